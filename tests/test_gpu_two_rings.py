"""Four compute waves at d_k = 128 read a chunk from two LDS rings of three and two stages; narrower workgroups have one ring. A
column's arithmetic is the same in both, so the results are the same bits for every number of chunks: in the forward scan, and in the
backward's reverse sweep, which has such rings of its own and visits the chunks from the last to the first."""
import pytest
import torch

import kla_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens", [[0, 1], [64, 63], [65, 128, 0], [129, 192, 193, 256], [257, 320, 449, 1]])
@pytest.mark.parametrize("dv", [64, 128, 256])
def test_same_bits_as_one_ring(lens, dv):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_08587_amd as kla
    cu = torch.tensor([0] + [sum(lens[:i + 1]) for i in range(len(lens))], dtype=torch.int32)
    d = kla_inputs.chunk_inputs(1, int(cu[-1]), 3, 128, dv, seed=dv + sum(lens), h0_std=0.3, n_h0=len(lens), log_alpha_scale=0.1)
    x = [d[n].cuda() for n in ("q", "k", "v", "log_alpha", "eta")]
    run = lambda w: kla.kla_chunk_fwd(*x, d["eps"], h0=d["h0"].cuda(), cu_seqlens=cu.cuda(), cu_seqlens_host=cu, tune=kla.tune(unfused=True, scan_waves=w))
    for a, b in zip(run(4), run(2)):
        assert torch.equal(a, b)


@pytest.mark.parametrize("lens,H,dv", [([T] * 9, 8, 128) for T in (320, 385, 449, 511, 576)] + [([511] * 5, 8, 256), ([576, 320, 385, 449, 511], 8, 256)])
def test_reverse_sweep(lens, H, dv):
    """Against the same sequences one by one, which run with one compute wave."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_08587_amd as kla
    # more than one round of workgroups of two waves, one of four
    assert len(lens) * H * (dv // 64) <= 256 < len(lens) * H * (dv // 32) and (H + 7) // 8 * 8 * (dv // 16) <= 256
    off = [sum(lens[:i]) for i in range(len(lens) + 1)]
    cu = torch.tensor(off, dtype=torch.int32)
    d = kla_inputs.chunk_inputs(1, off[-1], H, 128, dv, seed=dv + off[-1], h0_std=0.3, n_h0=len(lens), log_alpha_scale=0.1)
    x = [d[n].cuda() for n in ("q", "k", "v", "log_alpha", "eta")]
    gen = torch.Generator().manual_seed(off[-1])
    d_o, d_hT = (torch.randn(d[n].shape, generator=gen).to(d[n].dtype).cuda() for n in ("v", "h0"))
    h0 = d["h0"].cuda()
    if len(set(lens)) == 1:                              # fixed length: a batch
        split = lambda t: t.view(len(lens), lens[0], *t.shape[2:])
        got = kla.kla_chunk_bwd(*(split(t) for t in x), d["eps"], split(d_o), h0=h0, d_hT=d_hT)
        got = {n: t if n == "dh0" else t.reshape(1, off[-1], *t.shape[2:]) for n, t in got.items()}
    else:
        got = kla.kla_chunk_bwd(*x, d["eps"], d_o, h0=h0, d_hT=d_hT, cu_seqlens=cu.cuda(), cu_seqlens_host=cu)
    for i in range(len(lens)):
        a, b = off[i], off[i + 1]
        one = kla.kla_chunk_bwd(*(t[:, a:b].contiguous() for t in x), d["eps"], d_o[:, a:b].contiguous(), h0=h0[i:i + 1], d_hT=d_hT[i:i + 1])
        for n, t in one.items():
            assert torch.equal(t, got[n][i:i + 1] if n == "dh0" else got[n][:, a:b]), (i, n)
