"""The bf16 intra-chunk stage at the sizes where its tiles end: chunks that stop at, before and after a 16-row block, both
head widths, the forward's and the backward's records, with and without the normalised read-out."""
import pytest
import torch

import kla_inputs
from oracle import token_oracle

pytestmark = pytest.mark.gpu
TOL = 2e-2          # the bf16 bar of the other parity tests


@pytest.fixture(scope="module")
def kla():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_08587_amd as m
    m.lib()
    return m


@pytest.mark.parametrize("T", [15, 16, 17, 31, 33, 48, 49, 64 + 47, 128])
@pytest.mark.parametrize("dk,nq", [(64, False), (128, False), (128, True)])
def test_block_edges(kla, T, dk, nq):
    d = kla_inputs.chunk_inputs(2, T, 3, dk, 64, seed=T + dk, h0_std=0.3, log_alpha_scale=0.1)
    x = [d[n].cuda() for n in ("q", "k", "v", "log_alpha", "eta")]
    f32 = [kla_inputs.to_numpy_f32(d[n]) for n in "qkv"] + [d["log_alpha"].numpy(), d["eta"].numpy()]
    o, hT = kla.kla_chunk_fwd(*x, d["eps"], h0=d["h0"].cuda(), normalize_q=nq, tune=kla.tune(unfused=True))
    ro, rh, _ = token_oracle.kla_recurrent(*f32, d["eps"], h0=d["h0"].numpy(), normalize_q=nq)
    assert token_oracle.rel_err(o.float().cpu().numpy(), ro) <= TOL and token_oracle.rel_err(hT.cpu().numpy(), rh) <= TOL
    d_o, d_hT = kla_inputs.grad_inputs(d, T)
    g = kla.kla_chunk_bwd(*x, d["eps"], d_o.cuda(), h0=d["h0"].cuda(), d_hT=d_hT.cuda(), normalize_q=nq)
    ref = token_oracle.kla_recurrent_bwd(*f32, d["eps"], kla_inputs.to_numpy_f32(d_o), h0=d["h0"].numpy(), d_hT=d_hT.numpy(),
                                         normalize_q=nq)
    errs = {n: token_oracle.rel_err(g[n].float().cpu().numpy(), ref[n]) for n in ref}
    assert max(errs.values()) <= TOL, errs
