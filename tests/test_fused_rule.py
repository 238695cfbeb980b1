"""Which bf16 batches run the one-kernel forward (its workspace query reports 256 bytes), on both sides of the rule's lines."""
import os

import numpy as np
import pytest
import torch

import paper_2605_08587_amd as kla

pytestmark = pytest.mark.skipif(not os.path.exists(kla.LIB_PATH), reason="libkla.so not built")


def _fused(N, T, H, dk, dv, lens=None):
    cu = None if lens is None else torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32)
    return kla.kla_chunk_fwd_workspace_bytes(N, T if lens is None else sum(lens), H, dk, dv, torch.bfloat16, cu_seqlens=cu) == 256


@pytest.mark.parametrize("N,T,H,dk,dv,fused", [
    (1, 1, 8, 128, 128, True), (1, 256, 8, 128, 128, True), (1, 512, 8, 128, 128, False), (1, 200, 16, 128, 256, True),
    (1, 800, 16, 128, 256, False), (1, 200, 8, 64, 64, True), (1, 800, 8, 64, 64, False), (12, 92, 8, 128, 128, False),
    (4, 2000, 8, 128, 128, False), (8, 4096, 8, 128, 128, True), (9, 4096, 8, 128, 128, False), (8, 4096, 16, 128, 128, False),
    (32, 1000, 8, 128, 64, True), (16, 4096, 8, 64, 64, True), (64, 4096, 16, 128, 256, False), (1, 65536, 8, 128, 128, False)])
def test_fixed_length(N, T, H, dk, dv, fused):
    assert _fused(N, T, H, dk, dv) == fused


@pytest.mark.parametrize("lens,H,dv,fused", [([20, 0, 120, 64], 8, 128, True), ([100, 300, 150], 8, 128, True),
                                             ([2100, 100, 1000], 4, 128, False), ([900] * 16, 16, 256, False)])
def test_packed(lens, H, dv, fused):
    assert _fused(1, None, H, 128, dv, lens) == fused
