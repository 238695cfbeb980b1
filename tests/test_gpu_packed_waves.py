"""Packed batches whose workgroups' width follows from their lengths (one, two, four or eight waves by the work of the busiest
CU; here 2, 2, 1, 4, 8 and 8): every column is a recurrence of its own, so any width gives the bits of one wave per workgroup."""
import pytest
import torch

import kla_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens,H,dv", [([130, 1, 64, 640, 65, 0, 400], 16, 128), ([650, 60, 600, 63, 580, 127, 64], 8, 256),
                                       ([640, 64, 60, 1, 64], 8, 128), ([575, 65, 449, 300, 1, 64, 130, 385, 0, 511], 8, 256),
                                       ([(29 * i) % 140 for i in range(64)], 4, 256), ([(29 * i) % 140 for i in range(65)], 4, 256)])
def test_any_width(lens, H, dv):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_08587_amd as kla
    cu = torch.tensor([0] + [sum(lens[:i + 1]) for i in range(len(lens))], dtype=torch.int32)
    d = kla_inputs.chunk_inputs(1, int(cu[-1]), H, 128, dv, seed=dv + len(lens), h0_std=0.3, n_h0=len(lens), log_alpha_scale=0.1)
    x = [d[n].cuda() for n in ("q", "k", "v", "log_alpha", "eta")]
    run = lambda **t: kla.kla_chunk_fwd(*x, d["eps"], h0=d["h0"].cuda(), cu_seqlens=cu.cuda(), cu_seqlens_host=cu, tune=kla.tune(unfused=True, **t))
    for a, b in zip(run(), run(scan_waves=1)):
        assert torch.equal(a, b)
