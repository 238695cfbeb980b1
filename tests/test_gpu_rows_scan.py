"""The bf16 scan whose workgroups share sixteen columns among nine waves (batches of at most 256 chains of sixteen columns): the bits
of the scan with one wave per chain, at one to seven chunks (its ring holds five, its registers three), last chunks of 1, 63 and 64
rows, both head widths, packed batches with empty sequences, and what it leaves behind for the backward; against the oracle too."""
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


def _check(kla, d, cu, normalize_q, monkeypatch):
    x = [d[n].cuda() for n in ("q", "k", "v", "log_alpha", "eta")]
    h0 = d["h0"].cuda()
    packed = dict(cu_seqlens=None if cu is None else cu.cuda(), cu_seqlens_host=cu)

    def run(waves):
        monkeypatch.setattr(kla, "DEFAULT_TUNE", kla.tune(scan_waves=waves, unfused=True))
        y = [t.clone().requires_grad_(True) for t in x]
        o, hT = kla.kla_chunk(*y, d["eps"], h0=h0, normalize_q=normalize_q, **packed)
        w = torch.linspace(-1, 1, o.numel(), device="cuda").view(o.shape)
        plain = kla.kla_chunk_fwd(*x, d["eps"], h0=h0, normalize_q=normalize_q, **packed)
        return [*plain, o.detach(), hT.detach(), *torch.autograd.grad((o.float() * w).sum(), y)]
    got = run(0)
    for a, b in zip(got, run(1)):
        assert torch.equal(a, b)
    ro, rh, _ = token_oracle.kla_recurrent(*(kla_inputs.to_numpy_f32(d[n]) for n in "qkv"), d["log_alpha"].numpy(), d["eta"].numpy(), d["eps"],
                                           h0=d["h0"].numpy(), cu_seqlens=None if cu is None else cu.numpy(), normalize_q=normalize_q)
    assert token_oracle.rel_err(got[0].float().cpu().numpy(), ro) <= 2e-2 and token_oracle.rel_err(got[1].cpu().numpy(), rh) <= 2e-2


@pytest.mark.parametrize("T", [1, 64, 65, 191, 256, 320, 385, 448])
@pytest.mark.parametrize("dk,dv,H", [(64, 64, 3), (128, 128, 9), (64, 256, 1), (128, 256, 4)])
def test_fixed(kla, T, dk, dv, H, monkeypatch):
    _check(kla, kla_inputs.chunk_inputs(2, T, H, dk, dv, seed=T + dv, h0_std=0.3, log_alpha_scale=0.1), None, T == 191, monkeypatch)


@pytest.mark.parametrize("lens,H,dk,dv", [([70, 0, 200, 1, 64, 300], 2, 128, 128), ([0, 0, 5], 5, 64, 64), ([(37 * i) % 200 for i in range(64)], 1, 128, 64)])
def test_packed(kla, lens, H, dk, dv, monkeypatch):
    cu = torch.tensor([0] + [sum(lens[:i + 1]) for i in range(len(lens))], dtype=torch.int32)
    _check(kla, kla_inputs.chunk_inputs(1, int(cu[-1]), H, dk, dv, seed=len(lens), h0_std=0.3, n_h0=len(lens), log_alpha_scale=0.1), cu, False,
           monkeypatch)
