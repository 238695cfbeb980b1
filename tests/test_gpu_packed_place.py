"""Packed batches whose intra-chunk stage finds its chunks itself (up to 64 sequences) and those one above: empty sequences at
either end and in between, one token, whole chunks; forward in both element types, per-channel decay, backward."""
import numpy as np
import pytest
import torch

import kla_inputs
from oracle import token_oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def kla():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_08587_amd as m
    m.lib()
    return m


@pytest.mark.parametrize("lens", [[0, 70, 0, 1, 64, 129, 0], [128], [0, 0, 5], [0, 0], [(29 * i) % 70 for i in range(64)], [(29 * i) % 70 for i in range(65)]])
@pytest.mark.parametrize("dt,tol", [(torch.bfloat16, 2e-2), (torch.float32, 1e-4)])      # the bars of the other parity tests
def test_placement(kla, lens, dt, tol):
    cu = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32)
    T, H, n = int(cu[-1]), 2, len(lens)
    d = kla_inputs.chunk_inputs(1, T, H, 64, 128, dtype=dt, seed=n, h0_std=0.3, n_h0=n, log_alpha_scale=0.1)
    x = [d[m].cuda() for m in ("q", "k", "v", "log_alpha", "eta")]
    f32 = [kla_inputs.to_numpy_f32(d[m]) for m in "qkv"] + [d["log_alpha"].numpy(), d["eta"].numpy()]
    packed = dict(h0=d["h0"].cuda(), cu_seqlens=cu.cuda(), cu_seqlens_host=cu)
    ref = dict(h0=d["h0"].numpy(), cu_seqlens=cu.numpy())
    err = lambda a, b: token_oracle.rel_err(a.float().cpu().numpy(), b) if b.size else 0.0
    ro, rh, _ = token_oracle.kla_recurrent(*f32, d["eps"], **ref)
    o, hT = kla.kla_chunk_fwd(*x, d["eps"], tune=kla.tune(unfused=True), **packed)
    assert err(o, ro) <= tol and err(hT, rh) <= tol
    xd = x[:3] + [x[3][..., None].expand(1, T, H, 64).contiguous(), x[4]]                   # equal channels: the scalar gate
    o, hT = kla.kla_chunk_fwd_diag(*xd, d["eps"], **packed)
    assert err(o, ro) <= tol and err(hT, rh) <= tol
    if T < 100:
        return
    d_o = torch.randn(d["v"].shape, generator=torch.Generator().manual_seed(n)).to(dt)
    g = kla.kla_chunk_bwd(*x, d["eps"], d_o.cuda(), **packed)
    rg = token_oracle.kla_recurrent_bwd(*f32, d["eps"], kla_inputs.to_numpy_f32(d_o), **ref)
    errs = {m: err(g[m], rg[m]) for m in rg}
    assert max(errs.values()) <= tol, errs


@pytest.mark.parametrize("dt", [torch.bfloat16, torch.float32])
def test_no_tokens(kla, dt):
    """No token anywhere: h_T is h_0, whichever form runs."""
    h0 = torch.randn(2, 3, 128, 64, device="cuda")
    cu = torch.zeros(3, dtype=torch.int32)
    for shape, packed in (((2, 0, 3), {}), ((1, 0, 3), dict(cu_seqlens=cu.cuda(), cu_seqlens_host=cu))):
        e = lambda *s, t=dt: torch.empty(*shape, *s, dtype=t, device="cuda")
        for tune in (0, kla.tune(unfused=True), kla.tune(fused=True)):
            o, hT = kla.kla_chunk_fwd(e(128), e(128), e(64), e(t=torch.float32), e(t=torch.float32), 1e-6, h0=h0, tune=tune, **packed)
            assert o.numel() == 0 and torch.equal(hT, h0)
