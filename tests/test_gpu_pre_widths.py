"""The single-pass pre over the widths AUTO takes it for: team sizes that do
not divide the 32 reducer jobs of a tile, short last slices (C no multiple of
128), empty ones (a team one larger than the width needs), both layouts of the
active weights; several tiles per team and a ragged last one.  Every output is
compared with the oracle, and the saved logits with the multi-kernel path."""

import pytest
import torch

from paper_2607_14530_amd import synth
from paper_2607_14530_amd import xhc as X
from tests.parity_util import check_sublayer
from tests.test_gpu_pre_streams import plain_workgroups

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,T,Kr", [(32, 75, 1), (96, 4100, 4), (160, 300, 1), (352, 1400, 4), (1184, 120, 1),
                                    (1408, 77, 4), (1760, 600, 4), (1888, 33, 1), (2112, 493, 4), (2336, 300, 1),
                                    (2560, 410, 4), (2816, 5, 4), (3072, 70, 1), (3712, 200, 1), (3936, 290, 4)])
def test_single_pass_widths(C, T, Kr):
    w = synth.Workload(T=T, N=16, k=4, m=2, C=C, Kr=Kr, name=f"width-C{C}-T{T}-Kr{Kr}")
    print(f"[width] {w.name}", flush=True)
    inp = synth.sublayer_inputs(w, 71, device="cuda")
    d = X.dims_for(w)
    sub = X.Sublayer(d, inp, "cuda")
    saved = torch.empty(T, X.xhc_saved_floats(d), device="cuda")
    before = inp["X"].clone()
    sub.pre(inp["X"], saved=saved)
    assert sub.pre_failures() == 0
    assert plain_workgroups(sub) > 0, "AUTO fell back to the multi-kernel path"
    assert torch.equal(inp["X"], before)
    sub.post(inp["X"], inp["F"])
    torch.cuda.synchronize()
    _, same = check_sublayer(sub, dict(inp, X=before), w, before, inp["X"])
    # the values kept for the backward: the multi-kernel path's, to the order of fp32 sums
    multi = X.Sublayer(X.dims_for(w, impl=X.XHC_IMPL_MULTI), inp, "cuda")
    ref = torch.empty_like(saved)
    multi.pre(before, saved=ref)
    torch.cuda.synchronize()
    assert plain_workgroups(multi) == 0
    same = same.to("cuda")
    n = saved.shape[1] - 1      # the last float is padding
    assert float((saved[same, :n] - ref[same, :n]).abs().max()) < 2e-4


@pytest.mark.parametrize("C", [4096, 2112])
def test_single_pass_on_several_streams(C):
    """Single-pass calls in flight on several streams at once (a plain launch each, whose
    last team may wait for CUs the others hold): the results of the calls one by one."""
    w = synth.Workload(T=600, N=16, k=4, m=2, C=C, Kr=4, name=f"streams-C{C}")
    inps = [synth.sublayer_inputs(w, 80 + i, device="cuda") for i in range(3)]
    subs = [X.Sublayer(X.dims_for(w), inp, "cuda") for inp in inps]
    names = ("input", "idx", "p", "Hpre", "Hres", "Hpost")
    refs = []
    for sub, inp in zip(subs, inps):
        sub.pre(inp["X"])
        torch.cuda.synchronize()
        refs.append({n: getattr(sub, n).clone() for n in names})
    streams = [torch.cuda.Stream() for _ in subs]
    for _ in range(6):
        for sub, inp, st in zip(subs, inps, streams):
            sub.pre(inp["X"], stream=st)
    torch.cuda.synchronize()
    for sub, ref in zip(subs, refs):
        assert sub.pre_failures() == 0 and plain_workgroups(sub) > 0
        for n in names:
            assert torch.equal(getattr(sub, n), ref[n]), n
