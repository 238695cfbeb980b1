"""The native half of the Python binding against the step-by-step half: the same results to the last bit for every form of a
call both take, the same exceptions for calls that are wrong, and subclasses, fakes and transforms left to the latter."""
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


class Nothing:
    """Takes no call."""
    def __getattr__(self, name):
        return lambda *a: None


def _both(kla, monkeypatch, f):
    fast = f()
    with monkeypatch.context() as m:
        m.setattr(kla, "_native", Nothing())
        slow = f()
    flat = lambda x: [x] if torch.is_tensor(x) else [] if x is None else [t for y in (x.values() if isinstance(x, dict) else x) for t in flat(y)]
    fast, slow = flat(fast), flat(slow)
    assert len(fast) == len(slow) > 0
    for a, b in zip(fast, slow):
        assert a.dtype == b.dtype and a.shape == b.shape and a.stride() == b.stride() and not a.requires_grad
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("diag", [False, True])
@pytest.mark.parametrize("nq,gdn,out", [(False, False, False), (True, True, True)])
def test_decode(kla, monkeypatch, dt, diag, nq, gdn, out):
    d = kla_inputs.decode_inputs(1, 3, 2, 64, 128, dtype=dt, seed=3)
    x = [d[n][0].contiguous().cuda() for n in ("q", "k", "v", "log_alpha", "eta")]
    if diag:
        x[3] = x[3][..., None].expand(3, 2, 64).contiguous()
    x[0] = torch.nn.Parameter(x[0])
    f = kla.kla_decode_step_diag if diag else kla.kla_decode_step

    def call():
        S = d["S"].cuda().clone()
        o = torch.empty(3, 2, 128, dtype=dt, device="cuda") if out else None
        r = f(*x, 1e-6, S, out=o, normalize_q=nq, gdn_beta=gdn)
        assert o is None or r is o
        return r, S
    _both(kla, monkeypatch, call)


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("form", ["plain", "options", "no_hT", "buffers", "packed", "packed_no_host"])
@pytest.mark.parametrize("diag", [False, True])
def test_chunk(kla, monkeypatch, dt, form, diag):
    packed = form.startswith("packed")
    d = kla_inputs.chunk_inputs(1 if packed else 2, 150, 2, 64, 128, dtype=dt, seed=5, h0_std=0.1, n_h0=3 if packed else 2)
    x = [d[n].cuda() for n in ("q", "k", "v", "log_alpha", "eta")]
    xd = list(x)
    if diag:
        xd[3] = x[3][..., None].expand(*x[0].shape).contiguous()
    kw = dict(h0=d["h0"].cuda())
    if packed:
        host = torch.tensor([0, 70, 71, 150], dtype=torch.int32)
        kw.update(cu_seqlens=host.cuda(), cu_seqlens_host=host.long() if form == "packed" and dt == torch.float32 else host)
        if form == "packed_no_host":
            del kw["cu_seqlens_host"]
    opts = dict(normalize_q=True, gdn_beta=True) if form == "options" else {}
    f = kla.kla_chunk_fwd_diag if diag else kla.kla_chunk_fwd

    def fwd():
        extra = dict(want_hT=False) if form == "no_hT" else {}
        if form == "buffers":
            extra = dict(out=torch.empty_like(x[2]), hT=torch.empty(2, 2, 64, 128, device="cuda"),
                         workspace=torch.empty(1 << 22, dtype=torch.uint8, device="cuda"))
        return f(*xd, 1e-6, **kw, **opts, **extra)
    _both(kla, monkeypatch, fwd)
    if not diag:
        d_o, d_hT = kla_inputs.grad_inputs(d, 5, d_hT=False)[0], torch.randn_like(d["h0"])
        _both(kla, monkeypatch, lambda: kla.kla_chunk_bwd(*x, 1e-6, d_o.cuda(), d_hT=None if form == "no_hT" else d_hT.cuda(),
                                                          want_dh0=form != "no_hT", **kw, **opts))


def test_refusals(kla, monkeypatch):
    d = kla_inputs.decode_inputs(1, 3, 2, 64, 128, seed=3)
    x = [d[n][0].contiguous().cuda() for n in ("q", "k", "v", "log_alpha", "eta")]
    S = d["S"].cuda()
    c = kla_inputs.chunk_inputs(2, 70, 2, 64, 64, seed=5)
    y = [c[n].cuda() for n in ("q", "k", "v", "log_alpha", "eta")]
    host = torch.tensor([0, 70], dtype=torch.int32)
    sub = lambda xs, i, t: [t if j == i else u for j, u in enumerate(xs)]
    odd = torch.empty(3 * 2 * 64 * 128 + 1, device="cuda")[1:].view(3, 2, 64, 128)          # not 16-byte aligned
    calls = [
        lambda: kla.kla_decode_step(*sub(x, 0, x[0].cpu()), 1e-6, S),
        lambda: kla.kla_decode_step(*sub(x, 1, x[1].float()), 1e-6, S),
        lambda: kla.kla_decode_step(*sub(x, 2, x[2][:2]), 1e-6, S),
        lambda: kla.kla_decode_step(*sub(x, 0, x[0].half()), 1e-6, S),
        lambda: kla.kla_decode_step(*sub(x, 4, x[4].t().contiguous().t()), 1e-6, S),
        lambda: kla.kla_decode_step(*x, 1e-6, odd),
        lambda: kla.kla_decode_step(*x, -1.0, S),
        lambda: kla.kla_decode_step(*x, "eps", S),
        lambda: kla.kla_decode_step(*x, 1e-6, None),
        lambda: kla.kla_decode_step(*x, 1e-6, S, tune=1 << 30),
        lambda: kla.kla_decode_step_diag(*x, 1e-6, S),
        lambda: kla.kla_chunk_fwd(*y, float("nan")),
        lambda: kla.kla_chunk_fwd(*y, 1e-6, chunk=32),
        lambda: kla.kla_chunk_fwd(*y, 1e-6, workspace=torch.empty(16, dtype=torch.uint8, device="cuda")),
        lambda: kla.kla_chunk_fwd(*y, 1e-6, cu_seqlens=host.cuda(), cu_seqlens_host=host),
        lambda: kla.kla_chunk_fwd(*y, 1e-6, cu_seqlens=host.cuda().float()),
        lambda: kla.kla_chunk_fwd(*y, 1e-6, h0=torch.zeros(2, 2, 64, 64, dtype=torch.bfloat16, device="cuda")),
        lambda: kla.kla_chunk_bwd(*y, 1e-6, None),
        lambda: kla.kla_chunk_bwd(*y, 1e-6, y[2].float()),
        lambda: torch.func.vmap(lambda q: kla.kla_decode_step(q, *x[1:], 1e-6, S))(x[0][None]),
    ]
    for i, f in enumerate(calls):
        with pytest.raises(Exception) as fast:
            f()
        with monkeypatch.context() as m:
            m.setattr(kla, "_native", Nothing())
            with pytest.raises(Exception) as slow:
                f()
        assert type(fast.value) is type(slow.value) and str(fast.value) == str(slow.value), i
        assert getattr(fast.value, "code", 0) == getattr(slow.value, "code", 0), i


def test_autograd_without_some_gradients(kla):
    """Only o, only h_T, or both used: as with the missing gradient passed as zeros."""
    c = kla_inputs.chunk_inputs(2, 70, 2, 64, 64, seed=5, h0_std=0.1)
    leaf = lambda n: c[n].cuda().requires_grad_(True)
    d_o, d_hT = (t.cuda() for t in kla_inputs.grad_inputs(c, 5))
    for use_o, use_h in ((True, True), (True, False), (False, True)):
        x = [leaf(n) for n in ("q", "k", "v", "log_alpha", "eta", "h0")]
        o, hT = kla.kla_chunk(*x[:5], 1e-6, h0=x[5])
        outs, gs = ([o] if use_o else []) + ([hT] if use_h else []), ([d_o] if use_o else []) + ([d_hT] if use_h else [])
        got = torch.autograd.grad(outs, x, gs)
        ref = kla.kla_chunk_bwd(*(t.detach() for t in x[:5]), 1e-6, d_o if use_o else torch.zeros_like(d_o), h0=x[5].detach(),
                                d_hT=d_hT if use_h else torch.zeros_like(d_hT))
        for a, b in zip(got, ref.values()):
            assert torch.equal(a, b)
