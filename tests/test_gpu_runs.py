"""The run-based write-back and its reverse at every run length their launchers
choose (shorter runs where the full ones would leave the chip idle), against
the oracle's write-back differentiated in fp64: partial last runs, sequence
starts inside runs and at their edges."""

import pytest
import torch

from oracle import xhc_oracle as O
from paper_2607_14530_amd import synth
from paper_2607_14530_amd import xhc as X
from tests.parity_util import assert_bf16_close
from tests.test_gpu_bwd import assert_grad_close

pytestmark = pytest.mark.gpu
F64 = torch.float64

# (T, S, C): tokens per run of the conv reverse / the dot products / the forward
CASES = [(20, 4, 256),        # 16 / 4 / 4
         (1030, 515, 1024),   # 16 / 4 / 4, each sequence cut from its start
         (4100, 820, 1024),   # 32 / 8 / 8
         (2080, 2080, 4096)]  # 64 / 16 / 16


@pytest.mark.parametrize("T,S,C", CASES)
def test_run_lengths_match_oracle(T, S, C):
    w = synth.Workload(T=T, S=S, N=4, k=4, m=2, C=C, Kr=4, name=f"runs-T{T}-S{S}-C{C}")
    print(f"[runs] {w.name}", flush=True)
    inp = synth.sublayer_inputs(w, 61, device="cuda", grads=True)
    sub = X.TrainableSublayer(X.dims_for(w), inp, "cuda")
    state = inp["X"].clone()
    sub.forward(state, inp["F"])
    after = state.clone()
    g = sub.backward_post(state, inp["G_X"], inp["F"])
    torch.cuda.synchronize()
    assert torch.equal(state, inp["X"])
    c64 = lambda v: v.detach().to("cpu", F64)
    X0, Fd, cw = (c64(inp[n]).requires_grad_(True) for n in ("X", "F", "conv_w"))
    p, Hres, Hpost = (c64(v).requires_grad_(True) for v in (sub.p, sub.Hres, sub.Hpost))
    Xn = O.xhc_post(X0, Fd, cw, sub.idx.cpu().long(), p, Hres, Hpost, S=S, kappa=w.kappa)
    (Xn * c64(inp["G_X"])).sum().backward()
    assert_bf16_close(after, Xn, "X'")
    for got, ref, what in ((g["X"], X0, "dX"), (g["F"], Fd, "dF"), (g["dHres"], Hres, "dHres"),
                           (g["dHpost"], Hpost, "dHpost"), (g["dp"], p, "dp"), (g["conv_w"], cw, "dconv_w")):
        assert_grad_close(got, ref.grad, what)
