"""A workspace sized once for the longest batch serves the shorter ones: the
entry points take less than what the query names for a size (they then run
with the full lengths of runs and chunks), down to a need that grows with T.
Checked up to the first launch, which fails without a GPU: no GPU is needed,
and none may be there (the addresses are made up)."""

import ctypes

import pytest
import torch

from paper_2607_14530_amd import xhc as X

pytestmark = pytest.mark.skipif(torch.cuda.is_available(), reason="made-up addresses: runs where no launch can happen")

TS = (5, 64, 129, 300, 512, 600, 700, 777, 1000, 1024, 1025, 1500, 2000, 2048, 3000, 4000, 4096, 4097, 8192, 16384)
BWD = ("POST_BWD", "PRE_BWD", "FLASH_POST_BWD", "FLASH_PRE_BWD")
OPS = {"PRE": X.XHC_OP_PRE, "POST_BWD": X.XHC_OP_POST_BWD, "PRE_BWD": X.XHC_OP_PRE_BWD,
       "FLASH_PRE": X.XHC_OP_FLASH_PRE, "FLASH_POST": X.XHC_OP_FLASH_POST,
       "FLASH_POST_BWD": X.XHC_OP_FLASH_POST_BWD, "FLASH_PRE_BWD": X.XHC_OP_FLASH_PRE_BWD}


def dims(T, N, k, C, Kr, state="bf16", impl=X.XHC_IMPL_AUTO):
    return X.make_dims(T, N, k, k // 2, C, Kr=Kr, state=state, impl=impl)


def Q_of(d):
    return 4 if 5 * d.N <= 128 else 2


def need(d, op):
    return X.xhc_workspace_bytes(d, OPS[op], Q_of(d))


def status(d, op, nbytes):
    """What the entry point says to a workspace of nbytes, all other arguments being valid."""
    A = [(1 << 30) + (i << 20) for i in range(40)]   # distinct, aligned, never dereferenced
    D, Q, end = ctypes.byref(d), Q_of(d), (nbytes, None)
    L, conv = X.lib(), A[5] if d.Kr > 1 else None
    if op == "PRE":
        return L.xhc_pre(D, *A[:13], None, A[14], *end)
    if op == "POST_BWD":
        return L.xhc_post_bwd(D, *A[:4], conv, *A[5:14], A[15] if d.Kr > 1 else None, A[16], *end)
    if op == "PRE_BWD":
        return L.xhc_pre_bwd(D, *A[:27], *end)
    if op == "FLASH_PRE":
        return L.xhc_flash_pre(D, Q, *A[:16], *end)
    if op == "FLASH_POST":   # the last but one, whose successor has the residual mixing
        return L.xhc_flash_post(D, Q, Q - 1, A[0], A[1], None, A[2], A[3], A[4], None, *A[6:15], None, None, A[17], *end)
    if op == "FLASH_POST_BWD":   # the last sublayer
        return L.xhc_flash_post_bwd(D, Q, Q, *A[:4], conv, *A[5:18], None, A[19], A[20] if d.Kr > 1 else None,
                                    *A[21:30], *end)
    if op == "FLASH_PRE_BWD":
        return L.xhc_flash_pre_bwd(D, Q, *A[:21], *end)
    raise ValueError(op)


def accepted(d, op, nbytes):
    st = status(d, op, nbytes)
    assert st in (X.XHC_EHIP, X.XHC_EWORKSPACE), (op, X.STATUS_NAMES.get(st, st))
    return st == X.XHC_EHIP


@pytest.mark.parametrize("op", BWD)
@pytest.mark.parametrize("N,k,C,Kr,state", [(16, 4, 4096, 4, "bf16"), (16, 4, 1024, 4, "bf16"), (8, 4, 512, 4, "bf16"),
                                            (4, 4, 1536, 1, "bf16"), (32, 4, 2048, 4, "f32")])
def test_backward_workspace_of_a_longer_batch_serves_a_shorter_one(op, N, k, C, Kr, state):
    if op == "FLASH_PRE_BWD" and state == "f32":
        pytest.skip("the partials of the recomputed fp32 projection do not grow with T")
    at = {T: need(dims(T, N, k, C, Kr, state), op) for T in TS}
    for T in TS:
        assert accepted(dims(T, N, k, C, Kr, state), op, at[T]), (op, T)
        for longer in (L for L in TS if L > T):
            assert accepted(dims(T, N, k, C, Kr, state), op, at[longer]), (op, T, longer, at[T] / at[longer])
        assert not accepted(dims(T, N, k, C, Kr, state), op, 128), (op, T)


# the pre-projection of few tokens in short chunks, and of a dense sublayer in one pass: a batch one
# token tile longer names half the bytes
@pytest.mark.parametrize("op,T,longer,N,k,C,Kr", [("PRE", 512, 513, 32, 4, 1024, 4),
                                                  ("FLASH_PRE", 512, 513, 16, 4, 2048, 4),
                                                  ("FLASH_POST", 1024, 1025, 16, 4, 4096, 4)])
def test_forward_workspace_of_a_longer_batch_serves_a_shorter_one(op, T, longer, N, k, C, Kr):
    short, long = dims(T, N, k, C, Kr), dims(longer, N, k, C, Kr)
    assert need(long, op) < need(short, op), "not the case meant here"
    assert accepted(short, op, need(short, op))
    assert accepted(short, op, need(long, op)), need(short, op) / need(long, op)
    assert not accepted(short, op, 1024)


def test_single_pass_widths_take_the_multi_kernel_workspace():
    """AUTO at a width that impl = FUSED refuses: the multi-kernel path's bytes are enough."""
    for T, C in ((16, 2112), (2048, 2560), (16384, 2560)):
        multi = need(dims(T, 16, 4, C, 4, impl=X.XHC_IMPL_MULTI), "PRE")
        assert accepted(dims(T, 16, 4, C, 4), "PRE", multi), (T, C)


def test_dense_sublayer_takes_the_two_projection_workspace():
    """k = m = N: one pass for both mappings names more than two passes need."""
    T, C = 16384, 4096
    d = X.make_dims(T, 4, 4, 4, C, Kr=1)
    routed = need(X.make_dims(T, 4, 4, 2, C, Kr=1), "PRE")   # the same projections, one after the other
    assert need(d, "PRE") > routed
    assert accepted(d, "PRE", routed)
