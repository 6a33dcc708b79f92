"""The projection's launch plans against the oracle: chunks of 2, 4 and 8 steps
(by the workgroups they make), and more tokens than a workgroup holds."""

import pytest
import torch

from paper_2607_14530_amd import synth
from paper_2607_14530_amd import xhc as X
from tests.parity_util import check_sublayer

pytestmark = pytest.mark.gpu

# (T, N, k, m, C): k-blocks per chunk of the full / the active rows
CASES = [(3, 8, 4, 2, 512),        # 8 / 8
         (19, 32, 4, 2, 1024),     # 8 / 8, 128 chunks
         (9, 32, 4, 2, 2560),      # 32 (80 chunks already) / 8
         (2500, 8, 4, 2, 1024),    # 16 / 8
         (261, 4, 2, 1, 2112)]     # 8 / per-wave chunks (2112 is no multiple of 128)


@pytest.mark.parametrize("T,N,k,m,C", CASES)
def test_pre_and_post_match_oracle(T, N, k, m, C):
    w = synth.Workload(T=T, S=T, N=N, k=k, m=m, C=C, Kr=1, name=f"plan-T{T}-N{N}-k{k}-C{C}")
    print(f"[plan] {w.name}", flush=True)
    inp = synth.sublayer_inputs(w, 23, device="cuda")
    sub = X.Sublayer(X.dims_for(w), inp, "cuda")
    state = inp["X"].clone()
    sub.pre(state)
    sub.post(state, inp["F"])
    torch.cuda.synchronize()
    tok = torch.arange(0, T, max(1, T // 64), device="cuda")
    check_sublayer(sub, inp, w, inp["X"][tok], state[tok], tokens=tok)
