"""Sublayers whose streams are all active and fixed (k = m = N): both mappings
from one projection of the state, and where the layouts differ (C no multiple
of 128, fp32) from two, against the oracle, with the backward that reads the
saved logits."""

import pytest
import torch

from paper_2607_14530_amd import synth
from paper_2607_14530_amd import xhc as X
from tests.grad_util import assert_sublayer_state_grad
from tests.parity_util import check_sublayer
from tests.test_gpu_bwd import _oracle, _run, assert_grad_close

pytestmark = pytest.mark.gpu

CASES = [(37, 4, 256, 1, "bf16"), (300, 4, 1024, 4, "bf16"), (5, 2, 128, 2, "bf16"), (261, 4, 2112, 1, "bf16"),
         (70, 4, 256, 1, "f32")]


@pytest.mark.parametrize("T,N,C,Kr,state", CASES)
def test_dense_matches_oracle(T, N, C, Kr, state):
    w = synth.Workload(T=T, S=T, N=N, k=N, m=N, C=C, Kr=Kr, kappa=(4, 8, 12)[:Kr - 1] or (4, 8, 12), state=state,
                       name=f"dense-T{T}-N{N}-C{C}-Kr{Kr}-{state}")
    print(f"[dense] {w.name}", flush=True)
    inp = synth.sublayer_inputs(w, 29, device="cuda")
    sub = X.Sublayer(X.dims_for(w), inp, "cuda")
    after = inp["X"].clone()
    sub.pre(after)
    sub.post(after, inp["F"])
    torch.cuda.synchronize()
    check_sublayer(sub, inp, w, inp["X"], after)


def test_dense_backward_matches_oracle():
    w = synth.Workload(T=45, S=45, N=4, k=4, m=4, C=512, Kr=1, alpha=(0.5, 1.0, 0.5), name="dense-bwd")
    print(f"[dense] {w.name}", flush=True)
    inp, sub, state, g = _run(w, seed=14)
    ref = _oracle(w, inp)
    assert_sublayer_state_grad(g["X"], ref["X"], sub, inp["G_X"])
    for n in ("W_pre", "W_res", "W_post", "alpha", "b_pre", "b_res", "b_post"):
        assert_grad_close(g[n], ref[n], n)
