"""Infinities and NaN in the last row of a ragged fp32 chunk, whose rows beyond the end repeat it: they reach no output that the row
itself does not reach.  The products see 32 rows of the triangular operands at a time, so within the chunk that is the 32-row
block of the row and what follows; in V its own column, in Q its own row."""
import pytest
import torch

import kla_inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def kla():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_08587_amd as m
    m.lib()
    return m


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
@pytest.mark.parametrize("T", [1, 64 + 5, 64 + 32, 64 + 33, 64 + 50, 128])
@pytest.mark.parametrize("N,H,dv", [(2, 3, 64), (3, 12, 256)])     # eight and four waves per workgroup
def test_last_row(kla, N, H, dv, T, bad):
    d = kla_inputs.chunk_inputs(N, T, H, 64, dv, dtype=torch.float32, seed=T, h0_std=0.3, log_alpha_scale=0.1)
    x = {n: d[n].cuda() for n in ("q", "k", "v", "log_alpha", "eta")}
    run = lambda **o: kla.kla_chunk_fwd(*{**x, **o}.values(), d["eps"], h0=d["h0"].cuda())
    o, hT = run()
    assert o.isfinite().all() and hT.isfinite().all()
    n, h, c = N - 1, H - 1, 21
    v = x["v"].clone()
    v[n, T - 1, h, c] = bad
    ov, hv = run(v=v)
    reach = torch.zeros_like(o, dtype=torch.bool)
    reach[n, (T - 1) // 32 * 32:, h, c] = True
    state = torch.zeros_like(hT, dtype=torch.bool)
    state[n, h, :, c] = True
    assert torch.equal(ov[~reach], o[~reach]) and torch.equal(hv[~state], hT[~state])
    assert not ov[n, T - 1, h, c].isfinite() and not hv[state].isfinite().any()
    q = x["q"].clone()
    q[n, T - 1, h, c] = bad
    oq, hq = run(q=q)
    reach = torch.zeros_like(o, dtype=torch.bool)
    reach[n, T - 1, h] = True
    assert torch.equal(oq[~reach], o[~reach]) and torch.equal(hq, hT) and not oq[reach].isfinite().any()
