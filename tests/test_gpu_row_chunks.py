"""The row passes of the pre backward at the token chunks their launcher
chooses (64 tokens up, by the workgroups a chunk makes): several chunks with a
short last one, and one chunk shorter than a step, against the oracle."""

import pytest
import torch

from paper_2607_14530_amd import synth
from tests.grad_util import assert_sublayer_state_grad
from tests.test_gpu_bwd import _oracle, _run, assert_grad_close

pytestmark = pytest.mark.gpu

# (T, N, k, C, Kr): tokens per chunk of the full / the active rows
CASES = [(1101, 4, 2, 256, 1),    # 64 / 64
         (515, 16, 4, 1024, 4),   # 256 / 64
         (7, 8, 4, 512, 4)]       # one short chunk


@pytest.mark.parametrize("T,N,k,C,Kr", CASES)
def test_weight_gradients_over_chunks(T, N, k, C, Kr):
    w = synth.Workload(T=T, N=N, k=k, m=k // 2, C=C, Kr=Kr, name=f"chunks-T{T}-N{N}-C{C}")
    print(f"[chunks] {w.name}", flush=True)
    inp, sub, state, g = _run(w, seed=12)
    ref = _oracle(w, inp)
    assert torch.equal(sub.idx.cpu().long(), ref["idx"]), "routing differs (near-tie seed?)"
    assert_sublayer_state_grad(g["X"], ref["X"], sub, inp["G_X"])
    for n in ("W_r", "W_pre", "W_res", "W_post", "alpha", "b_pre", "b_res", "b_post"):
        assert_grad_close(g[n], ref[n], n)
