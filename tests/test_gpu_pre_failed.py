"""The coefficient pass behind a single pass whose waits gave up: every float
output of the call becomes NaN, those that the single pass had written itself
among them, and the ones behind the last token stay as they are.  The count is
set from here; no wait is made to fail."""

import ctypes

import pytest
import torch

from paper_2607_14530_amd import xhc as X

pytestmark = pytest.mark.gpu

NAME = "_ZN3xhc15launch_pre_coefEPKfllliiilS1_S1_S1_S1_fifPfS2_S2_S2_iiiP12ihipStream_tPKNS_9PreFailedE"
P, I64, I32, F32 = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int, ctypes.c_float


class PreFailed(ctypes.Structure):
    _fields_ = [("err", P), ("input", P), ("p", P), ("Hpre", P), ("N", I32), ("C", I32)]


@pytest.mark.parametrize("count", [0, 3])
def test_float_outputs_after_a_failed_single_pass(count):
    T, k, Kr, N, C, G, pad = 75, 4, 4, 16, 160, 2, 5
    f = getattr(X.lib(), NAME)
    f.restype = ctypes.c_int
    f.argtypes = [P, I64, I64, I64, I32, I32, I32, I64, P, P, P, P, F32, I32, F32, P, P, P, P, I32, I32, I32, P, P]
    print(f"[pre-failed] T={T} C={C} count={count}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(3)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=gen)
    ns = 2 * N + k * Kr + k * k + 4
    part = rnd(G, 34, T).abs()
    alpha, b_post, b_res = torch.ones(3, device="cuda"), torch.zeros(k * Kr, device="cuda"), torch.zeros(k * k, device="cuda")
    out = {"input": rnd(T + pad, C).bfloat16(), "p": rnd(T + pad, k), "Hpre": rnd(T + pad, N),
           "Hpost": rnd(T + pad, k * Kr), "Hres": rnd(T + pad, k * k), "saved": rnd(T + pad, ns)}
    before = {n: v.clone() for n, v in out.items()}
    err = torch.full((1,), count, dtype=torch.int32, device="cuda")
    failed = PreFailed(err.data_ptr(), out["input"].data_ptr(), out["p"].data_ptr(), out["Hpre"].data_ptr(), N, C)
    st = f(part.data_ptr(), G, k * Kr + k * k, T, k, Kr, 1, C, alpha[2:].data_ptr(), alpha[1:].data_ptr(),
           b_post.data_ptr(), b_res.data_ptr(), 1e-5, 20, 1e-6, out["Hpost"].data_ptr(), out["Hres"].data_ptr(), None,
           out["saved"].data_ptr(), ns, 2 * N, ns - 2, torch.cuda.current_stream().cuda_stream, ctypes.byref(failed))
    assert st == 0
    torch.cuda.synchronize()
    for n, v in out.items():
        assert torch.equal(v[T:], before[n][T:]), f"{n} written past the last token"
        if count:
            assert bool(v[:T].isnan().all()), n
        else:
            assert not bool(v.isnan().any()), n
            if n in ("input", "p", "Hpre"):
                assert torch.equal(v, before[n]), n
