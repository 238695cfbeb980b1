"""The scan order of a packed batch and the room it takes: batches of more than 256 sequences have none."""
import os

import numpy as np
import pytest
import torch

import kla_inputs
import paper_2605_08587_amd as kla
from oracle import token_oracle

pytestmark = pytest.mark.skipif(not os.path.exists(kla.LIB_PATH), reason="libkla.so not built")


def test_many_sequences_fit_the_fixed_scratch():
    """Chunk offsets alone decide: seven million sequences, all but one empty, take 28 MB of the 32 MiB."""
    n = 7_000_000
    cu = np.full(n + 1, 64, np.int32)
    cu[0] = 0
    need = kla.lib().kla_chunk_fwd_workspace_bytes(1, 64, 1, 128, 256, 64, kla.KLA_BF16, cu.ctypes.data, n)
    assert 4 * (n + 1) <= need <= kla.KLA_STATIC_SCRATCH_BYTES


@pytest.mark.gpu
@pytest.mark.parametrize("n", [256, 257])
@pytest.mark.parametrize("dt,tol", [(torch.bfloat16, 2e-2), (torch.float32, 1e-4)])      # the bars of the other parity tests
def test_either_side(n, dt, tol):
    lens = [(37 * i) % 20 for i in range(n - 1)] + [150]
    cu = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32)
    T, H = int(cu[-1]), 1
    d = kla_inputs.chunk_inputs(1, T, H, 64, 256, dtype=dt, seed=n, h0_std=0.3, n_h0=n, log_alpha_scale=0.1)
    x = [d[m].cuda() for m in ("q", "k", "v", "log_alpha", "eta")]
    f32 = [kla_inputs.to_numpy_f32(d[m]) for m in "qkv"] + [d["log_alpha"].numpy(), d["eta"].numpy()]
    packed = dict(h0=d["h0"].cuda(), cu_seqlens=cu.cuda(), cu_seqlens_host=cu)
    ref = dict(h0=d["h0"].numpy(), cu_seqlens=cu.numpy())
    err = lambda a, b: token_oracle.rel_err(a.float().cpu().numpy(), b)
    ro, rh, _ = token_oracle.kla_recurrent(*f32, d["eps"], **ref)
    xd = x[:3] + [x[3][..., None].expand(1, T, H, 64).contiguous(), x[4]]                   # equal channels: the scalar gate
    for o, hT in (kla.kla_chunk_fwd(*x, d["eps"], **packed), kla.kla_chunk_fwd_diag(*xd, d["eps"], **packed)):
        assert err(o, ro) <= tol and err(hT, rh) <= tol
    o2, hT2 = torch.empty_like(x[2]), torch.empty_like(hT)
    kla.kla_chunk_fwd_static(*x, d["eps"], o2, hT=hT2, **packed)
    assert err(o2, ro) <= tol and err(hT2, rh) <= tol
    d_o = torch.randn(d["v"].shape, generator=torch.Generator().manual_seed(n)).to(dt)
    g = kla.kla_chunk_bwd(*x, d["eps"], d_o.cuda(), **packed)
    rg = token_oracle.kla_recurrent_bwd(*f32, d["eps"], kla_inputs.to_numpy_f32(d_o), **ref)
    errs = {m: err(g[m], rg[m]) for m in rg}
    assert max(errs.values()) <= tol, errs
