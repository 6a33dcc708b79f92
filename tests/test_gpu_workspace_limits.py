"""The entry points in the least workspace that they take, smaller than what
the query names: the full lengths of runs and chunks, at N = 8 the group's entry
reverse map by map, a dense sublayer's mappings from two projections, the
multi-kernel pre instead of the single pass.  The results are those of the
preferred forms to the order of the sums, and nothing is written past the end."""

import pytest
import torch

from paper_2607_14530_amd import synth
from paper_2607_14530_amd import xhc as X
from tests.parity_util import check_sublayer

pytestmark = pytest.mark.gpu

GUARD = 4096


class Least:
    """A workspace cut down to the least that `call` accepts, with guard bytes behind it."""

    def __init__(self, obj, attr, call):
        self.full = getattr(obj, attr).numel()
        lo, hi = 0, self.full          # refused, accepted
        while hi - lo > 1:
            n = (lo + hi) // 2
            setattr(obj, attr, torch.empty(n, dtype=torch.uint8, device="cuda"))
            try:
                call()
                hi = n
            except X.XhcError as e:
                assert e.status == X.XHC_EWORKSPACE, e
                lo = n
        self.n = hi
        buf = torch.full((hi + GUARD,), 0xA5, dtype=torch.uint8, device="cuda")
        self.end = buf[hi:]
        setattr(obj, attr, buf[:hi])

    def check(self):
        assert self.n < self.full, "nothing smaller is taken: not the case meant here"
        assert bool((self.end == 0xA5).all()), "written past the workspace"


def assert_same(got, ref, what, bf16=2.0 ** -9):
    """Per tensor, 2-norm of the difference over 2-norm: fp32 sums of at most 2^11 terms in another
    order (1e-5), bf16 results one rounding apart where such a sum lies at its edge."""
    for n, r in ref.items():
        for a, b in zip(got[n], r) if isinstance(r, list) else [(got[n], r)]:
            if b is not None:
                e = float((a.double() - b.double()).norm() / b.double().norm().clamp_min(1e-30))
                assert e < (bf16 if b.dtype == torch.bfloat16 else 1e-5), (what, n, e)


@pytest.mark.parametrize("T,N,C,Kr,state", [(777, 16, 4096, 4, "bf16"), (600, 4, 1536, 4, "bf16"),
                                            (300, 8, 1024, 4, "f32"), (100, 4, 256, 4, "bf16")])
def test_sublayer_backward(T, N, C, Kr, state):
    w = synth.Workload(T=T, S=T, N=N, k=4, m=2, C=C, Kr=Kr, state=state, name=f"wslim-T{T}-N{N}-C{C}-{state}")
    print(f"[ws] {w.name}", flush=True)
    inp = synth.sublayer_inputs(w, 31, device="cuda", grads=True)
    sub = X.TrainableSublayer(X.dims_for(w), inp, "cuda")
    after = inp["X"].clone()
    sub.forward(after, inp["F"])
    run = lambda: sub.backward(after.clone(), inp["G_X"], inp["G_in"], inp["F"])
    ref = run()
    least = [Least(sub, "ws_post_bwd", lambda: sub.backward_post(after.clone(), inp["G_X"], inp["F"]))]
    least.append(Least(sub, "ws_pre_bwd", run))
    got = run()
    torch.cuda.synchronize()
    for l in least:
        l.check()
    assert_same(got, ref, w.name)


@pytest.mark.parametrize("T,S,N,C,Q,recompute", [(300, 150, 8, 512, 4, False), (141, 47, 8, 256, 2, True),
                                                 (200, 200, 16, 512, 4, True), (600, 300, 4, 1536, 2, False)])
def test_group_backward(T, S, N, C, Q, recompute):
    w = synth.Workload(T=T, S=S, N=N, k=4, m=2, C=C, Kr=4, alpha=(0.5, 1.0, 0.5), name=f"wslim-flash-T{T}-N{N}-Q{Q}")
    print(f"[ws] {w.name}", flush=True)
    d = synth.flash_inputs(w, Q, 33, device="cuda", grads=True)
    grp = X.TrainableFlashGroup(X.dims_for(w), Q, d, "cuda")
    grp.forward(d["X"].clone(), d["F_list"])
    run = lambda: grp.backward(d["X"], d["G_X"], d["G_in_list"], d["F_list"], recompute=recompute)
    ref = run()
    least = [Least(grp, attr, run) for attr in ("ws_post_bwd", "ws_pre_bwd")]
    got = run()
    torch.cuda.synchronize()
    for l in least:
        l.check()
    # map by map the gradient rows are rounded to bf16 Q + 1 times (2^-9 of an element each)
    assert_same(got, ref, w.name, bf16=(Q + 1) ** 0.5 * 2.0 ** -9)


# short chunks of the projection; both mappings of a dense sublayer from one pass; the single pass
@pytest.mark.parametrize("T,N,k,m,C", [(512, 32, 4, 2, 1024), (1000, 4, 4, 4, 1024), (300, 16, 4, 2, 2112)])
def test_sublayer_forward(T, N, k, m, C):
    w = synth.Workload(T=T, S=T, N=N, k=k, m=m, C=C, Kr=4, name=f"wslim-pre-T{T}-N{N}-C{C}")
    print(f"[ws] {w.name}", flush=True)
    inp = synth.sublayer_inputs(w, 35, device="cuda")
    sub = X.Sublayer(X.dims_for(w), inp, "cuda")
    least = Least(sub, "ws_pre", lambda: sub.pre(inp["X"]))
    after = inp["X"].clone()
    sub.pre(after)
    sub.post(after, inp["F"])
    torch.cuda.synchronize()
    least.check()
    tok = torch.arange(0, T, max(1, T // 64), device="cuda")
    check_sublayer(sub, inp, w, inp["X"][tok], after[tok], tokens=tok)


@pytest.mark.parametrize("T,N,C,Q", [(512, 16, 2048, 4), (600, 8, 1024, 2)])
def test_group_forward(T, N, C, Q):
    w = synth.Workload(T=T, S=T, N=N, k=4, m=2, C=C, Kr=4, name=f"wslim-group-T{T}-N{N}-Q{Q}")
    print(f"[ws] {w.name}", flush=True)
    d = synth.flash_inputs(w, Q, 37, device="cuda")
    grp = X.FlashGroup(X.dims_for(w), Q, d, "cuda")
    names = ("idx", "p", "Hpre", "Hres", "base")
    out = lambda st: dict({n: getattr(grp, n).clone() for n in names}, X=st, inputs=[v.clone() for v in grp.inputs],
                          Hpost=[v.clone() for v in grp.Hpost])
    ref = out(grp.run(d["X"].clone(), d["F_list"]))
    least = [Least(grp, "ws_pre", lambda: grp.pre(d["X"]))]
    least.append(Least(grp, "ws_post", lambda: grp.run(d["X"].clone(), d["F_list"])))
    got = out(grp.run(d["X"].clone(), d["F_list"]))
    torch.cuda.synchronize()
    for l in least:
        l.check()
    assert torch.equal(got.pop("idx"), ref.pop("idx")), "routing differs (near-tie seed?)"
    assert_same(got, ref, w.name)
