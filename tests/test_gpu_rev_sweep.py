"""The bf16 reverse sweep of few chains (a workgroup of four waves per 16 state columns, two rings, one visit of lead for the products that
do not depend on the state gradient): one to six chunks, last chunks of 1, 63 and 64 rows, packed sequences of no tokens, both head
widths, both sides of the line at 256 chains.  And every width of the sweeps and of the per-channel scan gives the same bits: batches
against their sequences one by one, which are few chains."""
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


@pytest.mark.parametrize("lens", [[64], [65], [127, 0, 1], [128, 192], [300, 63, 321]])
@pytest.mark.parametrize("dk,dv,H", [(64, 64, 2), (64, 256, 3), (128, 128, 2), (128, 64, 24)])
@pytest.mark.parametrize("normalize_q", [False, True])
def test_few_chains(kla, lens, dk, dv, H, normalize_q):
    if len(lens) < 3 and H == 24:
        H = 48          # 192 and 384 chains
    cu = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32)
    d = kla_inputs.chunk_inputs(1, int(cu[-1]), H, dk, dv, seed=dv + len(lens), h0_std=0.3, n_h0=len(lens), log_alpha_scale=0.1)
    x = [d[n].cuda() for n in ("q", "k", "v", "log_alpha", "eta")]
    gen = torch.Generator().manual_seed(11)
    d_o, d_hT = torch.randn(d["v"].shape, generator=gen).bfloat16(), torch.randn(d["h0"].shape, generator=gen)
    g = kla.kla_chunk_bwd(*x, d["eps"], d_o.cuda(), h0=d["h0"].cuda(), d_hT=d_hT.cuda(), cu_seqlens=cu.cuda(), cu_seqlens_host=cu,
                          normalize_q=normalize_q)
    ref = token_oracle.kla_recurrent_bwd(*(kla_inputs.to_numpy_f32(d[n]) for n in "qkv"), d["log_alpha"].numpy(), d["eta"].numpy(), d["eps"],
                                         kla_inputs.to_numpy_f32(d_o), h0=d["h0"].numpy(), d_hT=d_hT.numpy(), cu_seqlens=cu.numpy(),
                                         normalize_q=normalize_q)
    errs = {n: token_oracle.rel_err(g[n].float().cpu().numpy(), ref[n]) for n in ref}
    assert max(errs.values()) <= TOL, errs


def _one_by_one(kla, run, lens, names, seqs, states):
    """run(inputs, states, packing) of the packed batch against that of each sequence, to the last bit."""
    cu = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32)
    got = run(seqs, states, dict(cu_seqlens=cu.cuda(), cu_seqlens_host=cu))
    for i in range(len(lens)):
        a, b = int(cu[i]), int(cu[i + 1])
        one = run([t[:, a:b].contiguous() for t in seqs], [t[i:i + 1] for t in states], {})
        for n, t, w in zip(names, one, got):
            assert torch.equal(t, w[i:i + 1] if n in ("dh0", "hT") else w[:, a:b]), (i, n)


def _backward(kla, lens, H, dk, dv):
    T, n = sum(lens), len(lens)
    d = kla_inputs.chunk_inputs(1, T, H, dk, dv, seed=dv + T, h0_std=0.3, n_h0=n, log_alpha_scale=0.1)
    gen = torch.Generator().manual_seed(T)
    d_o, d_hT = (torch.randn(d[m].shape, generator=gen).to(d[m].dtype).cuda() for m in ("v", "h0"))
    names = ["dq", "dk", "dv", "dlog_alpha", "deta", "dh0"]

    def run(x, st, packing):
        g = kla.kla_chunk_bwd(*x[:5], d["eps"], x[5], h0=st[0], d_hT=st[1], **packing)
        return [g[m] for m in names]
    _one_by_one(kla, run, lens, names, [d[m].cuda() for m in ("q", "k", "v", "log_alpha", "eta")] + [d_o], [d["h0"].cuda(), d_hT])


# more than 256 chains: two waves per workgroup (second rounds of one would be longer), four, one in two rounds (tests/test_sweep_widths.py)
MANY = [([65, 64, 63, 1, 128], 8, 128), ([200, 190, 180, 170, 129], 8, 128), ([385, 321, 320, 449, 448], 8, 128), ([257, 256, 255, 193, 192, 250], 16, 64),
        ([192, 129, 190, 65, 130, 191, 150, 180, 140], 8, 128),
        ([300, 64, 1, 130, 60], 8, 128), ([449, 100, 0, 64, 1, 127], 16, 64)]


@pytest.mark.parametrize("lens,H,dv", MANY)
@pytest.mark.parametrize("dk", [64, 128])
def test_same_bits_as_few_chains(kla, lens, H, dk, dv):
    _backward(kla, lens, H, dk, dv)


@pytest.mark.parametrize("lens,dk", [([2304, 2241, 2303, 2250, 2277, 2299], 128), ([3584, 3583, 3521, 3550, 3577, 3530], 64)])
def test_lines_asked_for_ahead(kla, lens, dk):
    """More than 144 MB of K, Q, M^T and P^T under two waves per workgroup: the only sweep that touches lines ahead of its copies."""
    assert 16 * sum((n + 63) // 64 for n in lens) * (2 * 64 * dk * 2 + 2 * 6144) > 144 << 20
    _backward(kla, lens, 16, dk, 64)


@pytest.mark.parametrize("lens,H,dv", MANY)
@pytest.mark.parametrize("dk", [64, 128])
def test_per_channel_scan(kla, lens, H, dk, dv):
    T, n = sum(lens), len(lens)
    d = kla_inputs.chunk_inputs(1, T, H, dk, dv, seed=dv + T, h0_std=0.3, n_h0=n, log_alpha_scale=0.1)
    la = -torch.nn.functional.softplus(torch.randn((1, T, H, dk), generator=torch.Generator().manual_seed(T))) * 0.1
    x = [d["q"], d["k"], d["v"], la, d["eta"]]
    run = lambda x, st, packing: kla.kla_chunk_fwd_diag(*x, d["eps"], h0=st[0], **packing)
    _one_by_one(kla, run, lens, ["o", "hT"], [t.cuda() for t in x], [d["h0"].cuda()])
