"""The mixing matrices with one element per lane, forward and reversed, against
the oracle: k at and below the padded sizes 2, 4 and 8, one iteration, and more
of them than the reverse keeps the normalisers of at a time."""

import pytest
import torch

from oracle import xhc_oracle as O
from paper_2607_14530_amd import synth
from paper_2607_14530_amd import xhc as X
from tests.grad_util import assert_sublayer_state_grad
from tests.parity_util import assert_coef_close
from tests.test_gpu_bwd import assert_grad_close

pytestmark = pytest.mark.gpu

# (k, m, Kr, N, iters): 40 normalisations (20 iterations) are one segment of the reverse
CASES = [(1, 1, 1, 4, 20), (2, 1, 4, 4, 20), (2, 2, 1, 8, 41), (3, 1, 2, 8, 20), (5, 2, 1, 16, 20), (5, 5, 1, 8, 21),
         (4, 2, 4, 16, 1), (4, 2, 4, 16, 2), (4, 2, 1, 8, 20), (4, 2, 4, 32, 33), (4, 4, 1, 4, 50)]


@pytest.mark.parametrize("k,m,Kr,N,iters", CASES)
def test_mixing_matches_oracle(k, m, Kr, N, iters):
    w = synth.Workload(T=37, S=37, N=N, k=k, m=m, C=256, Kr=Kr, kappa=(4, 8, 12)[:Kr - 1] or (4, 8, 12),
                       alpha=(0.5, 2.0, 0.5), name=f"mix-k{k}-m{m}-Kr{Kr}-N{N}-it{iters}")
    print(f"[mixing] {w.name}", flush=True)
    inp = synth.sublayer_inputs(w, 17, device="cuda", grads=True)
    sub = X.TrainableSublayer(X.dims_for(w, sinkhorn_iters=iters), inp, "cuda")
    state = inp["X"].clone()
    sub.forward(state, inp["F"])
    g = sub.backward(state, inp["G_X"], inp["G_in"], inp["F"])
    torch.cuda.synchronize()
    c = lambda v: v.cpu() if torch.is_tensor(v) else v
    ref = O.xhc_sublayer_grads(c(inp["X"]).double(), c(inp["F"]).double(), c(inp["conv_w"]), c(inp["W_r"]),
                               c(inp["W_pre"]), c(inp["W_res"]), c(inp["W_post"]), c(inp["alpha"]), c(inp["b_pre"]),
                               c(inp["b_res"]), c(inp["b_post"]), c(inp["G_X"]), c(inp["G_in"]), m=m, k=k, Kr=Kr,
                               S=w.S, kappa=w.kappa, sinkhorn_iters=iters)
    assert torch.equal(sub.idx.cpu().long(), ref["idx"]), "routing differs (near-tie seed?)"
    assert_coef_close(sub.Hres.cpu(), ref["Hres"], "Hres")
    assert_coef_close(sub.Hpost.cpu(), ref["Hpost"], "Hpost")
    assert_sublayer_state_grad(g["X"], ref["X"], sub, inp["G_X"])
    for n in ("W_r", "W_pre", "W_res", "W_post", "alpha", "b_pre", "b_res", "b_post"):
        assert_grad_close(g[n], ref[n], n)
