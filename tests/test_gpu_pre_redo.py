"""The coefficient pass behind a single pass whose waits gave up: it forms the
whole sublayer's outputs again, against the oracle, with the records that the
multi-kernel path saves, and nothing behind the last token.  The count of
failed waits is set from here; no wait is made to fail."""

import ctypes

import pytest
import torch

from paper_2607_14530_amd import synth
from paper_2607_14530_amd import xhc as X
from tests.parity_util import check_sublayer

pytestmark = pytest.mark.gpu

NAME = "_ZN3xhc15launch_pre_coefEPKfllliiilS1_S1_S1_S1_fifPfS2_S2_S2_iiiP12ihipStream_tPKNS_7PreRedoE"
P, I64, I32, F32 = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int, ctypes.c_float
OUT = ("input", "idx", "p", "Hpre", "Hres", "Hpost")


class PreRedo(ctypes.Structure):
    _fields_ = ([("err", P), ("X", P), ("wfull", P), ("wact", P), ("act_grouped", I32)] +
                [(n, P) for n in ("colsum", "alpha_pre", "b_pre", "input", "idx", "p", "Hpre")] +
                [(n, I32) for n in ("C", "m", "softmax")])


def coef_pass(sub, state, part, count, out, saved):
    """The coefficient pass of `sub` into `out` and `saved`, on partials part [G, 34, T] of a single
    pass that counted `count` failed waits."""
    d = sub.d
    T, k, N, C, Kr = d.T, d.k, d.N, d.C, d.Kr
    f = getattr(X.lib(), NAME)
    f.restype = ctypes.c_int
    f.argtypes = [P, I64, I64, I64, I32, I32, I32, I64, P, P, P, P, F32, I32, F32, P, P, P, P, I32, I32, I32, P, P]
    err = torch.full((1,), count, dtype=torch.int32, device="cuda")
    full = N * C // 32 * 2 * 1024
    a = sub.alpha
    r = PreRedo(err.data_ptr(), state.data_ptr(), sub.packed_full.data_ptr(), sub.packed_act.data_ptr(),
                int(C % 128 == 0), sub.packed_full[full:].data_ptr(), a.data_ptr(), sub.b_pre.data_ptr(),
                *(out[n].data_ptr() for n in ("input", "idx", "p", "Hpre")), C, d.m, d.router)
    ns = saved.shape[1]
    st = f(part.data_ptr(), part.shape[0], k * Kr + k * k, T, k, Kr, 1, C, a[2:].data_ptr(), a[1:].data_ptr(),
           sub.b_post.data_ptr(), sub.b_res.data_ptr(), d.eps, d.sinkhorn_iters, d.clamp_delta,
           out["Hpost"].data_ptr(), out["Hres"].data_ptr(), None, saved.data_ptr(), ns, 2 * N, ns - 2,
           torch.cuda.current_stream().cuda_stream, ctypes.byref(r))
    assert st == 0
    torch.cuda.synchronize()


def _setup(T, C, Kr, m, router, pad):
    w = synth.Workload(T=T, N=16, k=4, m=m, C=C, Kr=Kr, router=router, alpha=(0.5, 1.0, 0.5), kappa=(4, 8, 12)[:Kr - 1] or (4, 8, 12),
                       name=f"redo-T{T}-C{C}-Kr{Kr}-{router}")
    print(f"[pre-redo] {w.name}", flush=True)
    inp = synth.sublayer_inputs(w, 53, device="cuda")
    sub = X.Sublayer(X.dims_for(w, impl=X.XHC_IMPL_MULTI), inp, "cuda")
    saved = torch.empty(T, X.xhc_saved_floats(sub.d), device="cuda")
    sub.pre(inp["X"], saved=saved)
    # outputs of another token count, with what must not be touched behind them
    out = {n: torch.full((T + pad, *getattr(sub, n).shape[1:]), 7, dtype=getattr(sub, n).dtype, device="cuda")
           for n in OUT}
    return w, inp, sub, saved, out, torch.full((T + pad, saved.shape[1]), 7.0, device="cuda")


@pytest.mark.parametrize("T,C,Kr,m,router", [(75, 160, 4, 2, "sigmoid"), (33, 4096, 1, 0, "sigmoid"),
                                             (40, 2112, 4, 2, "softmax"), (5, 32, 2, 4, "sigmoid")])
def test_outputs_formed_again(T, C, Kr, m, router):
    w, inp, sub, ref_saved, out, saved = _setup(T, C, Kr, m, router, pad=3)
    part = torch.full(((C + 127) // 128, 34, T), float("nan"), device="cuda")   # (not read)
    coef_pass(sub, inp["X"], part, 3, out, saved)
    for n, v in dict(out, saved=saved).items():
        assert bool((v[T:] == 7).all()), f"{n} written past the last token"
    for n in OUT:
        getattr(sub, n).copy_(out[n][:T])
    after = inp["X"].clone()
    sub.post(after, inp["F"])
    torch.cuda.synchronize()
    _, same = check_sublayer(sub, inp, w, inp["X"], after)
    n = saved.shape[1] - 1      # the last float is padding
    same = same.to("cuda")
    assert float((saved[:T][same, :n] - ref_saved[same, :n]).abs().max()) < 2e-4


def test_nothing_is_formed_again_without_a_failed_wait():
    w, inp, sub, _, out, saved = _setup(75, 160, 4, 2, "sigmoid", pad=0)
    part = torch.randn(2, 34, 75, device="cuda", generator=torch.Generator("cuda").manual_seed(3)).abs()
    coef_pass(sub, inp["X"], part, 0, out, saved)
    for n in ("input", "idx", "p", "Hpre"):
        assert bool((out[n] == 7).all()), n
    z = part.sum(0)
    want = z[:32].T * torch.rsqrt(z[33][:, None] / (4 * 160) + sub.d.eps)
    assert float((saved[:, 32:64] - want).abs().max()) < 1e-4
