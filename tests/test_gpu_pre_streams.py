"""The single-pass pre on the streams a program has: the null and the
per-thread stream, torch's own, one under capture, and one with a CU mask,
which is launched cooperatively.  The results are those of the null stream."""

import ctypes

import pytest
import torch

from paper_2607_14530_amd import synth
from paper_2607_14530_amd import xhc as X

pytestmark = pytest.mark.gpu

NAMES = ("input", "idx", "p", "Hpre", "Hres", "Hpost")


def plain_workgroups(sub):
    """Workgroups the last pre() numbered as they started (the word 128 bytes into the workspace):
    0 for a cooperative launch and for the multi-kernel path, which clears it."""
    return int(sub.ws_pre[128:132].view(torch.int32).item())


def _setup(C, seed):
    w = synth.Workload(T=200, N=16, k=4, m=2, C=C, Kr=4, name=f"pre-streams-C{C}")
    print(f"[pre-streams] {w.name}", flush=True)
    inp = synth.sublayer_inputs(w, seed, device="cuda")
    sub = X.Sublayer(X.dims_for(w), inp, "cuda")
    sub.pre(inp["X"], stream=0)
    torch.cuda.synchronize()
    assert plain_workgroups(sub) > 0 and sub.pre_failures() == 0
    ref = {n: getattr(sub, n).clone() for n in NAMES}

    def check(plain):
        torch.cuda.synchronize()
        assert sub.pre_failures() == 0
        assert (plain_workgroups(sub) > 0) == plain
        for n in NAMES:
            assert torch.equal(getattr(sub, n), ref[n]), n
            getattr(sub, n).zero_()
        torch.cuda.synchronize()
    return inp, sub, check


def _hip():
    path = next(l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l)
    return ctypes.CDLL(path)


def test_streams_without_a_mask_are_launched_plainly():
    inp, sub, check = _setup(2112, 41)
    for stream in (0, 2, torch.cuda.Stream()):    # null, per-thread, torch's
        sub.pre(inp["X"], stream=stream)
        check(plain=True)


def test_under_capture():
    inp, sub, check = _setup(512, 43)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        sub.pre(inp["X"])
    for _ in range(3):
        g.replay()
        check(plain=True)


def test_a_masked_stream_is_launched_cooperatively():
    inp, sub, check = _setup(256, 45)
    hip, s = _hip(), ctypes.c_void_p()
    mask = (ctypes.c_uint32 * 8)(*([0xFFFFFFFF] * 4 + [0] * 4))    # 128 CUs; a team has 2 members here
    assert hip.hipExtStreamCreateWithCUMask(ctypes.byref(s), 8, mask) == 0
    try:
        sub.pre(inp["X"], stream=s.value)
        check(plain=False)
    finally:
        torch.cuda.synchronize()
        assert hip.hipStreamDestroy(s) == 0
