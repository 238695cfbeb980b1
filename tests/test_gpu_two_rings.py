"""Four compute waves at d_k = 128 read a chunk from two LDS rings of three and two stages; the workgroups of two waves have one ring.
A column's arithmetic is the same in both, so the results are the same bits for every number of chunks."""
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
