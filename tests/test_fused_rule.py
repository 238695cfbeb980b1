"""Which bf16 batches run the one-kernel forward (its workspace query reports 256 bytes), on both sides of the rule's lines.  The
two forms round different operands to 16 bits, so the line is part of a call's results: batches beside it give those of the
two-kernel form to the last bit, and the entry point with the fixed scratch gives what kla_chunk_fwd gives."""
import os

import numpy as np
import pytest
import torch

import kla_inputs
import paper_2605_08587_amd as kla

pytestmark = pytest.mark.skipif(not os.path.exists(kla.LIB_PATH), reason="libkla.so not built")


def _fused(N, T, H, dk, dv, lens=None, **t):
    cu = None if lens is None else torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32)
    return kla.kla_chunk_fwd_workspace_bytes(N, T if lens is None else sum(lens), H, dk, dv, torch.bfloat16, cu_seqlens=cu,
                                             tune=kla.tune(**t)) == 256


@pytest.mark.parametrize("N,T,H,dk,dv,fused", [
    (1, 1, 8, 128, 128, False), (1, 200, 8, 128, 128, False), (1, 200, 16, 128, 256, False), (5, 92, 8, 128, 128, False),
    (6, 92, 8, 128, 128, True), (41, 30, 1, 128, 128, True), (8, 4096, 8, 128, 128, True), (9, 4096, 8, 128, 128, True),
    (16, 4096, 8, 128, 128, True), (31, 500, 8, 128, 128, True), (32, 500, 8, 128, 128, False), (11, 92, 8, 64, 64, False),
    (12, 92, 8, 64, 64, True), (32, 1000, 8, 128, 64, True), (63, 100, 8, 64, 64, True), (64, 100, 8, 64, 64, False),
    (8, 4096, 8, 128, 256, False), (64, 4096, 16, 128, 256, False), (1, 65536, 8, 128, 128, False)])
def test_fixed_length(N, T, H, dk, dv, fused):
    assert _fused(N, T, H, dk, dv) == fused


@pytest.mark.parametrize("lens,H,dv,fused", [([20, 0, 120, 64], 8, 128, False), ([2000] * 4, 8, 128, False), ([900] * 16, 16, 256, False),
                                             ([1000, 1] * 3, 8, 128, True), ([70] * 64, 1, 128, True), ([70] * 65, 1, 128, True),
                                             ([70] * 64, 4, 128, False), ([70] * 65, 4, 64, True)])
def test_packed(lens, H, dv, fused):
    assert _fused(1, None, H, 128, dv, lens) == fused


def test_forced():
    for t, small, large in ((dict(fused=True), True, True), (dict(unfused=True), False, False), (dict(scan_waves=2), True, True),
                            (dict(scan_waves=1), False, False), (dict(scan_waves=4, fused=True), False, False)):
        assert _fused(1, 200, 8, 128, 128, **t) == small and _fused(32, 500, 8, 128, 128, **t) == large, t


def _correlated(N, T, H, dk, dv, n_seq=None):
    """Unit keys close to one another, slow decay: L is as large as it gets."""
    d = kla_inputs.chunk_inputs(N, T, H, dk, dv, seed=1, h0_std=0.1, n_h0=n_seq, log_alpha_scale=0.01)
    gen = torch.Generator().manual_seed(78)
    k = torch.randn((N, 1, H, dk), generator=gen) + 0.4 * torch.randn((N, T, H, dk), generator=gen)
    d["k"] = (k / k.norm(dim=-1, keepdim=True)).bfloat16()
    return d


@pytest.mark.gpu
@pytest.mark.parametrize("N,T,H,dk,dv,lens", [(1, 200, 8, 128, 128, None), (2, 250, 8, 64, 64, None), (1, 300, 4, 128, 256, None),
                                              (1, 450, 8, 128, 128, [100, 0, 300, 50])])
def test_small_batches_keep_the_fp32_inverse(N, T, H, dk, dv, lens):
    d = _correlated(N, T, H, dk, dv, lens and len(lens))
    x = [d[n].cuda() for n in ("q", "k", "v", "log_alpha", "eta")]
    packed = {}
    if lens:
        cu = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32)
        packed = dict(cu_seqlens=cu.cuda(), cu_seqlens_host=cu)
    for gdn in (False, True):
        o, hT = kla.kla_chunk_fwd(*x, d["eps"], h0=d["h0"].cuda(), gdn_beta=gdn, **packed)
        o2, hT2 = kla.kla_chunk_fwd(*x, d["eps"], h0=d["h0"].cuda(), gdn_beta=gdn, tune=kla.tune(unfused=True), **packed)
        assert torch.equal(o, o2) and torch.equal(hT, hT2)


@pytest.mark.gpu
@pytest.mark.parametrize("N,T", [(6, 200), (20, 1024), (31, 700)])
def test_fixed_scratch_agrees(N, T):
    """Also where the two-kernel form would not fit the fixed scratch (20 x 1024 tokens of 8 heads need 35 MB)."""
    d = _correlated(N, T, 8, 128, 128)
    x = [d[n].cuda() for n in ("q", "k", "v", "log_alpha", "eta")]
    o, hT = kla.kla_chunk_fwd(*x, d["eps"])
    o2, hT2 = torch.empty_like(o), torch.empty_like(hT)
    kla.kla_chunk_fwd_static(*x, d["eps"], o2, hT=hT2)
    assert torch.equal(o, o2) and torch.equal(hT, hT2)
