"""The state gradient of one sublayer against the oracle's."""

import torch

from tests.test_gpu_flash_bwd import assert_state_grad_close


def assert_sublayer_state_grad(got, ref, sub, G_X, what="dX"):
    """dL/dX of a bf16 state is stored three times: what the write-back's
    reverse passes on (the mixing transpose of G_X on the active rows, G_X
    elsewhere), then with the full-row terms added, then with the active-row
    terms; an element is off by up to 2^-8 of what it holds each time, the whole by
    about sqrt(3) 2^-8 / sqrt(12) = 2e-3 in the 2-norm (twice that is allowed)."""
    t = torch.arange(G_X.shape[0], device=G_X.device)[:, None]
    first = G_X.double().clone()
    first[t, sub.idx.long()] = torch.matmul(sub.Hres.double().transpose(1, 2).contiguous(), first[t, sub.idx.long()])
    assert_state_grad_close(got, ref, 3, first, what)
    rel = (got.double().cpu() - ref.double().cpu()).norm() / ref.double().norm().cpu()
    assert float(rel) <= 4e-3, f"{what}: relative Frobenius error {float(rel):.2e}"
