"""The fp32 chunk sweeps (four waves per column tile, one or two tiles per workgroup) at the sizes where their split can go
wrong: chunk counts 1 and 2, ragged last chunks of one row, one short of a tile, one into the next wave's rows; an empty
sequence in a packed batch; both tile counts, chosen by the rule and forced.  Bar: the fp32 bar of the other parity tests."""
import numpy as np
import pytest
import torch

import kla_inputs
from oracle import token_oracle

pytestmark = pytest.mark.gpu
TOL = 1e-4


@pytest.fixture(scope="module")
def kla():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_08587_amd as m
    m.lib()
    return m


def _c(t):
    return None if t is None else t.cuda()


def _case(T, dk, dv, packed, N=1, H=3):
    d = kla_inputs.chunk_inputs(1 if packed else N, T, H, dk, dv, dtype=torch.float32, seed=T + dk + dv, h0_std=0.5,
                                n_h0=4 if packed else None, log_alpha_scale=0.1)
    if packed:                                       # one token, nothing, the rest in two pieces
        d["cu_seqlens"] = torch.tensor([0, 1, 1, 1 + (T - 1) // 2, T], dtype=torch.int32)
    return d


def _np(d):
    return [d[n].numpy() for n in ("q", "k", "v", "log_alpha", "eta")]


@pytest.mark.parametrize("tiles", [0, 1, 2])
@pytest.mark.parametrize("T,dk,dv,packed", [(1, 64, 64, False), (63, 128, 64, False), (64, 64, 128, False), (65, 128, 128, False),
                                            (17, 128, 256, False), (113, 64, 256, False), (200, 128, 128, True), (150, 64, 64, True)])
def test_forward(kla, T, dk, dv, packed, tiles):
    d = _case(T, dk, dv, packed)
    cu = d["cu_seqlens"]
    o, hT = kla.kla_chunk_fwd(*(d[n].cuda() for n in ("q", "k", "v", "log_alpha", "eta")), d["eps"], h0=_c(d["h0"]), cu_seqlens=_c(cu),
                              tune=kla.tune(scan_waves=tiles))
    ro, rh, _ = token_oracle.kla_recurrent(*_np(d), d["eps"], h0=d["h0"].numpy(), cu_seqlens=None if cu is None else cu.numpy())
    assert token_oracle.rel_err(o.cpu().numpy(), ro) <= TOL and token_oracle.rel_err(hT.cpu().numpy(), rh) <= TOL


# 18 x 16 column tiles: two per workgroup by the rule; 3 x 4: one
@pytest.mark.parametrize("T,dk,dv,packed,N,H", [(1, 64, 64, False, 1, 3), (66, 128, 128, False, 1, 3), (129, 64, 256, False, 3, 6),
                                                (79, 128, 256, False, 3, 6), (140, 128, 64, True, 1, 3), (140, 64, 128, True, 1, 3)])
def test_backward(kla, T, dk, dv, packed, N, H):
    d = _case(T, dk, dv, packed, N, H)
    cu = d["cu_seqlens"]
    d_o, d_hT = kla_inputs.grad_inputs(d, 3)
    g = kla.kla_chunk_bwd(*(d[n].cuda() for n in ("q", "k", "v", "log_alpha", "eta")), d["eps"], d_o.cuda(), h0=_c(d["h0"]),
                          d_hT=d_hT.cuda(), cu_seqlens=_c(cu))
    ref = token_oracle.kla_recurrent_bwd(*_np(d), d["eps"], d_o.numpy(), h0=d["h0"].numpy(), d_hT=d_hT.numpy(),
                                         cu_seqlens=None if cu is None else cu.numpy())
    for n in ref:
        assert token_oracle.rel_err(g[n].cpu().numpy(), ref[n]) <= TOL, n


@pytest.mark.parametrize("T,dk,dv,N,H", [(65, 64, 64, 1, 3), (95, 128, 128, 1, 3), (70, 128, 256, 3, 6)])
def test_diagonal_gating(kla, T, dk, dv, N, H):
    d = _case(T, dk, dv, False, N, H)
    d["log_alpha"] = kla_inputs.diag_gates(d, 5, 0.1)
    o, hT = kla.kla_chunk_fwd_diag(*(d[n].cuda() for n in ("q", "k", "v", "log_alpha", "eta")), d["eps"], h0=_c(d["h0"]))
    ro, rh, _ = token_oracle.kla_recurrent_diag(*_np(d), d["eps"], h0=d["h0"].numpy())
    assert token_oracle.rel_err(o.cpu().numpy(), ro) <= TOL and token_oracle.rel_err(hT.cpu().numpy(), rh) <= TOL
