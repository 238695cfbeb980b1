"""The bf16 reverse sweep of few chains (a workgroup of four waves per 16 state columns, two rings, one visit of lead for the products that
do not depend on the state gradient): one to six chunks, last chunks of 1, 63 and 64 rows, packed sequences of no tokens, both head
widths, both sides of the line at 256 chains."""
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


@pytest.mark.parametrize("lens", [[64], [65], [127, 0, 1], [128, 192], [300, 63, 321]])
@pytest.mark.parametrize("dk,dv,H", [(64, 64, 2), (64, 256, 3), (128, 128, 2), (128, 64, 24)])
@pytest.mark.parametrize("normalize_q", [False, True])
def test_few_chains(kla, lens, dk, dv, H, normalize_q):
    if len(lens) < 3 and H == 24:
        H = 48          # 192 and 384 chains
    cu = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32)
    d = kla_inputs.chunk_inputs(1, int(cu[-1]), H, dk, dv, seed=dv + len(lens), h0_std=0.3, n_h0=len(lens), log_alpha_scale=0.1)
    x = [d[n].cuda() for n in ("q", "k", "v", "log_alpha", "eta")]
    gen = torch.Generator().manual_seed(11)
    d_o, d_hT = torch.randn(d["v"].shape, generator=gen).bfloat16(), torch.randn(d["h0"].shape, generator=gen)
    g = kla.kla_chunk_bwd(*x, d["eps"], d_o.cuda(), h0=d["h0"].cuda(), d_hT=d_hT.cuda(), cu_seqlens=cu.cuda(), cu_seqlens_host=cu,
                          normalize_q=normalize_q)
    ref = token_oracle.kla_recurrent_bwd(*(kla_inputs.to_numpy_f32(d[n]) for n in "qkv"), d["log_alpha"].numpy(), d["eta"].numpy(), d["eps"],
                                         kla_inputs.to_numpy_f32(d_o), h0=d["h0"].numpy(), d_hT=d_hT.numpy(), cu_seqlens=cu.numpy(),
                                         normalize_q=normalize_q)
    errs = {n: token_oracle.rel_err(g[n].float().cpu().numpy(), ref[n]) for n in ref}
    assert max(errs.values()) <= TOL, errs
