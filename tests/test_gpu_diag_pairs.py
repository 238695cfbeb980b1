"""Per-channel decay: every entry of P = A o Q K^T of a chunk by itself.  Sequence j has a key at token j alone, so o_i = beta_j (sum_c
q_ic k_jc gamma_ic/gamma_jc) v_j for i >= j and 0 before: the pairs of each 8x8 block on the diagonal (running products), its
neighbours, the diagonal and the tiles below (products split at a reference row), at slow and at strong decay, each against the size
of its own terms."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt,tol", [(torch.float32, 1e-4), (torch.bfloat16, 6 * 2.0 ** -8)])   # bf16: both operands of a product, P, T', U and o are rounded
@pytest.mark.parametrize("dk", [64, 128])
@pytest.mark.parametrize("T", [64, 41])
@pytest.mark.parametrize("scale", [0.02, 3.0])
def test_every_pair(dt, tol, dk, T, scale):
    import paper_2605_08587_amd as kla
    gen = torch.Generator().manual_seed(T + dk)
    q = torch.randn((T, 2, dk), generator=gen).to(dt)
    kj = torch.randn((T, 2, dk), generator=gen).to(dt)
    vj = torch.randn((T, 2, 64), generator=gen).to(dt)
    la = -torch.nn.functional.softplus(torch.randn((T, 2, dk), generator=gen)) * scale
    eta = torch.sigmoid(torch.randn((T, 2), generator=gen))
    k, v = torch.zeros((T, T, 2, dk), dtype=dt), torch.zeros((T, T, 2, 64), dtype=dt)
    at = torch.arange(T)
    k[at, at], v[at, at] = kj, vj
    rep = lambda x: x[None].expand(T, *x.shape).contiguous().cuda()
    o, _ = kla.kla_chunk_fwd_diag(rep(q), k.cuda(), v.cuda(), rep(la), rep(eta), 1e-6)
    g = la.double().cumsum(0)
    low = (at[:, None] >= at[None, :])[:, :, None, None]                                # [i, j]
    ratio = torch.where(low, g[:, None] - g[None], torch.full((), -torch.inf, dtype=torch.float64)).exp()
    p = torch.einsum("ihc,jhc,ijhc->ijh", q.double(), kj.double(), ratio)
    beta = eta.double() / (kj.double().square().sum(-1) + 1e-6)
    ref = torch.einsum("ijh,jh,jhv->jihv", p, beta, vj.double())
    assert torch.equal(o.cpu().double()[~low[:, :, 0, 0].T], torch.zeros_like(ref)[~low[:, :, 0, 0].T])
    assert float((o.cpu().double() - ref).abs().max() / ref.abs().max()) <= (1e-4 if dt == torch.float32 else 2e-2)      # the bars of the other parity tests
    # The size of an entry's own terms; besides the element type's tolerance, the running log sums g_i and g_j are fp32 after at most 20
    # additions each (a segment of 16 rows, four offsets), every one rounded at the size of the sum; below 1e-35 factors underflow.
    size = torch.einsum("ihc,jhc,ijhc->ijh", q.double().abs(), kj.double().abs(), ratio)
    bound = size * (tol + 40 * 2.0 ** -24 * g.abs().amax(-1)[:, None])
    bound = torch.einsum("ijh,jh,jhv->jihv", bound, beta, vj.double().abs()) + 1e-35
    worst = (o.cpu().double() - ref).abs() / bound
    print("largest error %.3f of its bound" % float(worst.max()))
    assert float(worst.max()) <= 1.0
