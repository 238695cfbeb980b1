"""The fp32 forward with more column tiles than fit one round of two per workgroup (four waves per workgroup) and with fewer
(eight), over one to four chunks and ragged ends: both images of K and of the exchanged state are used and reused."""
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


@pytest.mark.parametrize("T", [1, 64, 65, 129, 250])
@pytest.mark.parametrize("N,H,dk,dv", [(3, 12, 128, 256), (3, 6, 128, 256), (2, 3, 128, 64), (2, 3, 64, 128)])
def test_forward(kla, T, N, H, dk, dv):
    d = kla_inputs.chunk_inputs(N, T, H, dk, dv, dtype=torch.float32, seed=T + H, h0_std=0.3, log_alpha_scale=0.1)
    o, hT = kla.kla_chunk_fwd(*(d[n].cuda() for n in ("q", "k", "v", "log_alpha", "eta")), d["eps"], h0=d["h0"].cuda(), normalize_q=T == 129)
    ro, rh, _ = token_oracle.kla_recurrent(*(d[n].numpy() for n in ("q", "k", "v", "log_alpha", "eta")), d["eps"], h0=d["h0"].numpy(),
                                           normalize_q=T == 129)
    assert token_oracle.rel_err(o.cpu().numpy(), ro) <= TOL and token_oracle.rel_err(hT.cpu().numpy(), rh) <= TOL
