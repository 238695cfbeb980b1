"""The bf16 scan with eight compute waves per workgroup (what batches of d_v >= 128 run where they save rounds of workgroups)
and the scan order of packed batches (whose lengths give them two, eight, four and eight waves here), at the sizes where they
can go wrong: one to three chunks, last chunks of 1, 63 and 64 rows, both head widths, both slices of d_v = 256, empty
sequences, more sequences than the order is built for.  The two-kernel form is asked for: some of these batches run the
one-kernel form by themselves, which has neither."""
import numpy as np
import pytest
import torch

import kla_inputs
from oracle import token_oracle

pytestmark = pytest.mark.gpu
TOL = 2e-2          # the bf16 bar of the other parity tests


@pytest.fixture(scope="module")
def kla():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_08587_amd as m
    m.lib()
    return m


def _check(kla, d, cu=None, **opts):
    c = lambda t: None if t is None else t.cuda()
    o, hT = kla.kla_chunk_fwd(*(d[n].cuda() for n in ("q", "k", "v", "log_alpha", "eta")), d["eps"], h0=c(d["h0"]), cu_seqlens=c(cu),
                              tune=kla.tune(unfused=True), **opts)
    ro, rh, _ = token_oracle.kla_recurrent(*(kla_inputs.to_numpy_f32(d[n]) for n in "qkv"), d["log_alpha"].numpy(), d["eta"].numpy(),
                                           d["eps"], h0=None if d["h0"] is None else d["h0"].numpy(),
                                           cu_seqlens=None if cu is None else cu.numpy(), **opts)
    assert token_oracle.rel_err(o.float().cpu().numpy(), ro) <= TOL and token_oracle.rel_err(hT.cpu().numpy(), rh) <= TOL


@pytest.mark.parametrize("T", [1, 63, 64, 65, 130])
@pytest.mark.parametrize("dk,dv,H", [(64, 128, 17), (128, 128, 17), (128, 256, 9)])
def test_eight_waves(kla, T, dk, dv, H):
    _check(kla, kla_inputs.chunk_inputs(8, T, H, dk, dv, seed=T + dv, h0_std=0.3, log_alpha_scale=0.1), normalize_q=T == 65)


@pytest.mark.parametrize("lens,H,dv", [([70, 0, 200, 1, 64, 129, 0, 63, 300], 9, 256),
                                       ([70, 0, 200, 1, 64, 129, 0, 63, 300], 32, 256), ([(37 * i) % 75 for i in range(300)], 1, 64),
                                       ([(53 * i) % 131 for i in range(256)], 2, 128)])
def test_packed_order(kla, lens, H, dv):
    cu = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32)
    d = kla_inputs.chunk_inputs(1, int(cu[-1]), H, 128, dv, seed=len(lens), h0_std=0.3, n_h0=len(lens), log_alpha_scale=0.1)
    _check(kla, d, cu)
