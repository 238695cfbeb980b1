"""Segment-parallel forward with enough maps for the kernel of four compute waves (and with too few), both head widths, one to
fifteen steps of the composition, a long memory (so that the maps are not numerically zero) and a ragged last segment."""
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


@pytest.mark.parametrize("segs", [2, 3, 4, 5, 16])
@pytest.mark.parametrize("N,H,dk,dv,h0", [(4, 8, 128, 128, 0.3), (4, 8, 64, 64, None), (1, 3, 64, 256, 0.3), (2, 5, 128, 64, None)])
def test_segment_maps(kla, segs, N, H, dk, dv, h0):
    d = kla_inputs.chunk_inputs(N, 64 * 16 - 13, H, dk, dv, seed=segs + dv, h0_std=h0, log_alpha_scale=0.01)
    x = [d[n].cuda() for n in ("q", "k", "v", "log_alpha", "eta")]
    o, hT = kla.kla_chunk_fwd(*x, d["eps"], h0=None if h0 is None else d["h0"].cuda(), tune=kla.tune(segments=segs))
    ro, rh, _ = token_oracle.kla_recurrent(*(kla_inputs.to_numpy_f32(d[n]) for n in "qkv"), d["log_alpha"].numpy(), d["eta"].numpy(),
                                           d["eps"], h0=None if h0 is None else d["h0"].numpy())
    assert token_oracle.rel_err(o.float().cpu().numpy(), ro) <= TOL and token_oracle.rel_err(hT.cpu().numpy(), rh) <= TOL


def test_fixed_scratch_takes_what_it_took(kla):
    """8192 tokens of 8 heads, d_v = 256: with as many segments as pay the maps would not fit the fixed scratch, so both entry
    points run with fewer, and agree to the last bit."""
    d = kla_inputs.chunk_inputs(1, 8192, 8, 128, 256, seed=4, log_alpha_scale=0.1)
    x = [d[n].cuda() for n in ("q", "k", "v", "log_alpha", "eta")]
    o, hT = kla.kla_chunk_fwd(*x, d["eps"])
    o2, hT2 = torch.empty_like(o), torch.empty_like(hT)
    kla.kla_chunk_fwd_static(*x, d["eps"], o2, hT=hT2)
    assert torch.equal(o, o2) and torch.equal(hT, hT2)
