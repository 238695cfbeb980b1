"""The bf16 backward sweeps with four compute waves per workgroup (what batches of several rounds run): one to three chunks, last
chunks of 1, 63 and 64 rows, both head widths, one and several slices of d_v, packed sequences of no tokens."""
import numpy as np
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


@pytest.mark.parametrize("lens", [[64], [63], [65, 0, 127], [130, 129, 1, 200]])
@pytest.mark.parametrize("dk,dv,H", [(64, 64, 160), (128, 128, 72), (128, 256, 40)])
def test_four_waves(kla, lens, dk, dv, H):
    # every sequence nine times over: at least 320 pairs of column tiles
    lens = (lens * 9)[:9] if len(lens) > 1 else lens * 2
    H = H if len(lens) < 9 else H // 4
    cu = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32)
    chains = (len(lens) * H + 7) // 8 * 8
    assert chains * (dv // 32) > 256
    d = kla_inputs.chunk_inputs(1, int(cu[-1]), H, dk, dv, seed=dv + len(lens), h0_std=0.3, n_h0=len(lens), log_alpha_scale=0.1)
    x = [d[n].cuda() for n in ("q", "k", "v", "log_alpha", "eta")]
    gen = torch.Generator().manual_seed(7)
    d_o, d_hT = torch.randn(d["v"].shape, generator=gen).bfloat16(), torch.randn(d["h0"].shape, generator=gen)
    g = kla.kla_chunk_bwd(*x, d["eps"], d_o.cuda(), h0=d["h0"].cuda(), d_hT=d_hT.cuda(), cu_seqlens=cu.cuda(), cu_seqlens_host=cu)
    ref = token_oracle.kla_recurrent_bwd(*(kla_inputs.to_numpy_f32(d[n]) for n in "qkv"), d["log_alpha"].numpy(), d["eta"].numpy(), d["eps"],
                                         kla_inputs.to_numpy_f32(d_o), h0=d["h0"].numpy(), d_hT=d_hT.numpy(), cu_seqlens=cu.numpy())
    errs = {n: token_oracle.rel_err(g[n].float().cpu().numpy(), ref[n]) for n in ref}
    assert max(errs.values()) <= TOL, errs
