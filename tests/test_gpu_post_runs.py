"""The run-based write-back at widths, sequence lengths and k that fill neither
a workgroup nor a group of tokens, over runs of one and of many sequences,
against the oracle's write-back, with the untouched rows unchanged; and the
per-token kernels where the fixed scratch holds only their partials."""

import pytest
import torch

from oracle import xhc_oracle as O
from paper_2607_14530_amd import synth
from paper_2607_14530_amd import xhc as X
from tests.parity_util import assert_bf16_close

pytestmark = pytest.mark.gpu
F64 = torch.float64

# (T, S, N, k, m, C, state): short last groups and runs, one-token
# sequences, widths with a partly and a wholly idle wave, one lane over
CASES = [(37, 37, 8, 4, 2, 96, "bf16"), (51, 17, 16, 4, 2, 2112, "bf16"), (66, 33, 4, 2, 1, 2560, "bf16"),
         (9, 1, 8, 4, 2, 1056, "bf16"), (130, 65, 16, 8, 2, 288, "bf16"), (70, 35, 16, 4, 2, 1056, "bf16"),
         (31, 31, 8, 4, 2, 544, "f32"), (22, 11, 8, 2, 1, 1024, "f32"), (1027, 1027, 8, 4, 2, 1024, "bf16")]
# many sequences to a run: starts on group edges, at every place inside a group, several in one
CASES += [(2056, 8, 4, 4, 2, 2048, "bf16"), (204, 12, 16, 8, 2, 1056, "bf16"), (2000, 100, 4, 4, 2, 2048, "bf16"),
          (2049, 3, 4, 4, 2, 2048, "bf16"), (2010, 5, 8, 8, 2, 2048, "bf16"), (1018, 2, 4, 2, 1, 2112, "bf16"),
          (1011, 1, 4, 4, 2, 2048, "f32"), (2002, 13, 8, 8, 2, 1024, "f32"), (2030, 7, 4, 2, 1, 1024, "f32")]
# one and two tokens a sequence, of so many that the per-token kernels take them, and one fewer
CASES += [(4096, 1, 4, 4, 2, 4096, "bf16"), (4096, 2, 2, 2, 1, 4096, "bf16"), (4095, 1, 2, 2, 1, 4096, "bf16")]


def _setup(T, S, N, k, m, C, state, seed=5):
    w = synth.Workload(T=T, S=S, N=N, k=k, m=m, C=C, Kr=4, state=state, name=f"post-T{T}-S{S}-k{k}-C{C}-{state}")
    print(f"[post-runs] {w.name}", flush=True)
    inp = synth.sublayer_inputs(w, seed, device="cuda")
    sub = X.Sublayer(X.dims_for(w), inp, "cuda")
    sub.pre(inp["X"])
    return w, inp, sub


def _check(w, inp, sub, after):
    ref = O.xhc_post(inp["X"].cpu().to(F64), inp["F"].cpu(), inp["conv_w"].cpu(), sub.idx.cpu().long(),
                     sub.p.cpu().to(F64), sub.Hres.cpu().to(F64), sub.Hpost.cpu().to(F64), S=w.S, kappa=w.kappa)
    assert_bf16_close(after, ref, "X'")
    act = torch.zeros(w.T, w.N, dtype=torch.bool)
    act[torch.arange(w.T)[:, None], sub.idx.cpu().long()] = True
    assert torch.equal(after.cpu()[~act], inp["X"].cpu()[~act]), "unwritten rows changed"


@pytest.mark.parametrize("T,S,N,k,m,C,state", CASES)
def test_post_matches_oracle(T, S, N, k, m, C, state):
    w, inp, sub = _setup(T, S, N, k, m, C, state)
    after = inp["X"].clone()
    sub.post(after, inp["F"])
    torch.cuda.synchronize()
    _check(w, inp, sub, after)


@pytest.mark.parametrize("T,S,N,C", [(1050, 5, 8, 1024), (1032, 12, 4, 2112)])
def test_group_write_backs_over_short_sequences(T, S, N, C):
    """The write-backs of a group's MLP-type sublayers, with the next input and with the mixing."""
    w = synth.Workload(T=T, S=S, N=N, k=4, m=2, C=C, Kr=4, name=f"group-T{T}-S{S}-C{C}")
    print(f"[post-runs] {w.name}", flush=True)
    d = synth.flash_inputs(w, 4, 19, device="cuda")
    grp = X.FlashGroup(X.dims_for(w), 4, d, "cuda")
    state = d["X"].clone()
    grp.pre(state)
    for q in range(1, 5):
        before, inp = state.clone(), [v.clone() for v in grp.inputs]
        grp.step(q, state, d["F_list"][q - 1])
        torch.cuda.synchronize()
        eye = torch.eye(4, dtype=F64).expand(T, 4, 4)
        ref = O.xhc_post(before.cpu().to(F64), d["F_list"][q - 1].cpu(),
                         d["conv_w_list"][q - 1].cpu() if q % 2 == 0 else None, grp.idx.cpu().long(),
                         grp.p.cpu().to(F64), grp.Hres.cpu().to(F64) if q == 4 else eye,
                         grp.Hpost[q - 1].cpu().to(F64), S=S, kappa=w.kappa)
        assert_bf16_close(state, ref, f"X after sublayer {q}")
        if q < 4:   # the next input: the base readout and the active rows as stored
            act = state[torch.arange(T, device="cuda")[:, None], grp.idx.long()].double()
            wts = grp.Hpre[q].gather(1, grp.idx.long()).double()
            want = grp.base[q - 1].double() + (wts[:, :, None] * act).sum(1)
            assert_bf16_close(grp.inputs[q], want, f"input {q + 1}")


def test_noalloc_past_the_run_kernels_partials():
    """18 MB of run partials against 16 MiB of scratch, where the per-token kernels' 10 MB fit:
    accepted as by size of the latter, and the same result as with a workspace."""
    import ctypes
    w, inp, sub = _setup(90000, 90000, 4, 2, 1, 2560, "bf16")
    a, b = inp["X"], inp["X"].clone()
    assert X.xhc_workspace_bytes(sub.d, X.XHC_OP_POST) > X.NOALLOC_SCRATCH_BYTES
    sub.post(a, inp["F"])
    st = X.lib().xhc_post_noalloc(ctypes.byref(sub.d), b.data_ptr(), inp["F"].data_ptr(), sub.conv_w.data_ptr(),
                                  sub.idx.data_ptr(), sub.p.data_ptr(), sub.Hres.data_ptr(), sub.Hpost.data_ptr(),
                                  None, torch.cuda.current_stream().cuda_stream)
    assert st == X.XHC_OK, X.STATUS_NAMES.get(st, st)
    torch.cuda.synchronize()
    tok = torch.arange(0, w.T, 997, device="cuda")
    assert_bf16_close(a[tok], b[tok].to("cpu", F64), "X' with a workspace / without")
