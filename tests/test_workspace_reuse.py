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
OPS = {"POST_BWD": X.XHC_OP_POST_BWD, "PRE_BWD": X.XHC_OP_PRE_BWD,
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
    if op == "POST_BWD":
        return L.xhc_post_bwd(D, *A[:4], conv, *A[5:14], A[15] if d.Kr > 1 else None, A[16], *end)
    if op == "PRE_BWD":
        return L.xhc_pre_bwd(D, *A[:27], *end)
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


@pytest.mark.parametrize("op", OPS)
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
