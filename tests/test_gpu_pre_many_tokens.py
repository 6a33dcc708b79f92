"""The single-pass pre of more tokens than 2^31 floats of saved records hold
(68 a token): about 60 GB, so only where the GPU has them to spare."""

import pytest
import torch

from paper_2607_14530_amd import synth
from paper_2607_14530_amd import xhc as X

pytestmark = pytest.mark.gpu


def test_saved_records_past_2_31_floats():
    if torch.cuda.mem_get_info()[0] < 80 << 30:
        pytest.skip("needs 80 GB of free GPU memory")
    block = 4096                                  # the same tokens over and over
    w = synth.Workload(T=block, N=16, k=4, m=2, C=32, Kr=4, name="pre-block")
    inp = synth.sublayer_inputs(w, 51, device="cuda")
    one = X.Sublayer(X.dims_for(w), inp, "cuda")
    ref = torch.empty(block, X.xhc_saved_floats(one.d), device="cuda")
    one.pre(inp["X"], saved=ref)
    ns = ref.shape[1]
    n = (1 << 31) // (ns * block) + 2
    print(f"[many-tokens] T={n * block} ({n * block * ns} floats of records)", flush=True)
    d = X.make_dims(n * block, 16, 4, 2, 32, Kr=4, S=block)
    many = X.Sublayer(d, inp, "cuda")
    saved = torch.zeros(n * block, ns, device="cuda")
    many.pre(inp["X"].repeat(n, 1, 1), saved=saved)
    torch.cuda.synchronize()
    assert many.pre_failures() == 0
    for b in (0, n // 2, n - 3, n - 2, n - 1):    # (the last float of a record is padding)
        at = slice(b * block, (b + 1) * block)
        assert torch.equal(saved[at, :ns - 1], ref[:, :ns - 1]), f"records of block {b} of {n}"
        for name in ("input", "idx", "Hpre", "Hres", "Hpost"):
            assert torch.equal(getattr(many, name)[at], getattr(one, name)), (name, b)
    del many, saved
    torch.cuda.empty_cache()
