"""The group entry reverse of all Q pre-maps in one pass at N = 8 (outputs that
fill neither 32 nor 64 columns), chunks and last steps that are not whole,
against the oracle."""

import pytest

from paper_2607_14530_amd import synth
from tests import test_gpu_flash_bwd as B

pytestmark = pytest.mark.gpu

CASES = [(37, 37, 256, 2), (70, 35, 256, 4), (141, 47, 512, 2)]


@pytest.mark.parametrize("T,S,C,Q", CASES)
def test_one_pass_entry_reverse(T, S, C, Q):
    w = synth.Workload(T=T, S=S, N=8, k=4, m=2, C=C, Kr=4, alpha=(0.5, 1.0, 0.5), name=f"fbwd-N8-T{T}-Q{Q}")
    print(f"[flash-bwd-n8] {w.name}", flush=True)
    B.test_flash_backward_matches_oracle(w, Q, 0.0)
