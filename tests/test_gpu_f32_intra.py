"""The fp32 intra-chunk stage: the accuracy of beta, which the sums of the key norms decide, and the chunks where its tiles end,
both head widths, forward and backward."""
import numpy as np
import pytest
import torch

import kla_inputs
from oracle import token_oracle

pytestmark = pytest.mark.gpu
TOL = 1e-4          # the fp32 bar of the other parity tests


@pytest.fixture(scope="module")
def kla():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_08587_amd as m
    m.lib()
    return m


@pytest.mark.parametrize("dk", [64, 128])
def test_beta_accuracy(kla, dk):
    """T'[i][i] = beta_i exactly (the inverse has a unit diagonal).  Relative to its end a rounding moves a sum by 2^-24 / sqrt(12)
    to twice that, 0.43 * 2^-24 in the mean square.  In a tree the n nodes of a level add up to 1 / sqrt(n) of that, all levels
    to sqrt(2), the four squares of a leaf no more than another level, the sum with eps and the quotient (1 ulp at most) one
    and two: below sqrt(2 + 1 + 1 + 4) * 0.43 = 1.22 * 2^-24.  d_k roundings one after the other: 0.43 sqrt(d_k / 3) = 2.0
    and 2.8 * 2^-24 before the rest."""
    N, T, H = 4, 128, 3
    gen = torch.Generator().manual_seed(dk)
    k = torch.randn((N, T, H, dk), generator=gen)
    eta = torch.rand((N, T, H), generator=gen) + 0.01
    Tb, _, _ = kla.kla_debug_intra_chunk(k.cuda(), k.cuda(), torch.zeros((N, T, H), device="cuda"), eta.cuda(), 1e-6)
    got = torch.diagonal(Tb, dim1=2, dim2=3).cpu().double().reshape(N, T // 64, H, 64).permute(0, 1, 3, 2).reshape(N, T, H)
    ref = eta.double() / ((k.double() ** 2).sum(-1) + 1e-6)
    err = ((got - ref) / ref).abs().numpy()
    print("d_k=%d: beta off by %.2e at most, %.2e rms" % (dk, err.max(), np.sqrt((err ** 2).mean())), flush=True)
    assert np.sqrt((err ** 2).mean()) <= 1.22 * 2.0 ** -24


@pytest.mark.parametrize("T", [1, 15, 16, 17, 33, 48, 63, 64 + 47, 128])
@pytest.mark.parametrize("dk,nq", [(64, False), (128, False), (128, True)])
def test_block_edges(kla, T, dk, nq):
    d = kla_inputs.chunk_inputs(2, T, 3, dk, 64, dtype=torch.float32, seed=T + dk, h0_std=0.3, log_alpha_scale=0.1)
    x = [d[n].cuda() for n in ("q", "k", "v", "log_alpha", "eta")]
    f32 = [d[n].numpy() for n in ("q", "k", "v", "log_alpha", "eta")]
    o, hT = kla.kla_chunk_fwd(*x, d["eps"], h0=d["h0"].cuda(), normalize_q=nq)
    ro, rh, _ = token_oracle.kla_recurrent(*f32, d["eps"], h0=d["h0"].numpy(), normalize_q=nq)
    assert token_oracle.rel_err(o.cpu().numpy(), ro) <= TOL and token_oracle.rel_err(hT.cpu().numpy(), rh) <= TOL
    d_o, d_hT = kla_inputs.grad_inputs(d, T)
    g = kla.kla_chunk_bwd(*x, d["eps"], d_o.cuda(), h0=d["h0"].cuda(), d_hT=d_hT.cuda(), normalize_q=nq)
    ref = token_oracle.kla_recurrent_bwd(*f32, d["eps"], d_o.numpy(), h0=d["h0"].numpy(), d_hT=d_hT.numpy(), normalize_q=nq)
    errs = {n: token_oracle.rel_err(g[n].cpu().numpy(), ref[n]) for n in ref}
    assert max(errs.values()) <= TOL, errs
