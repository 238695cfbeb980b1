"""kla_chunk as a C++ node of the autograd graph (the native half of the binding) against the Python function it stands for: which
inputs want a gradient, missing output gradients, gradients that are not contiguous, hooks on saved tensors, changed inputs,
a second backward, function transforms, forward mode, threads of the engine."""
import pytest
import torch
import torch.utils.checkpoint

import kla_inputs

pytestmark = pytest.mark.gpu
NAMES = ("q", "k", "v", "log_alpha", "eta", "h0")


@pytest.fixture(scope="module")
def kla():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_08587_amd as m
    m.lib()
    return m


def _leaves(seed=4, T=150, wrt=NAMES):
    d = kla_inputs.chunk_inputs(2, T, 3, 64, 128, seed=seed, h0_std=0.2)
    return [d[n].cuda().requires_grad_(n in wrt) for n in NAMES]


def _call(kla, x, **kw):
    return kla.kla_chunk(*x[:5], 1e-6, h0=x[5], **kw)


def _python(kla, f):
    with pytest.MonkeyPatch.context() as m:
        m.setattr(kla, "_native", kla._StepByStep)
        return f()


def _same(a, b):
    assert all((s is None and t is None) or torch.equal(s, t) for s, t in zip(a, b))


def test_native_node_runs(kla):
    assert "KlaChunk" in _call(kla, _leaves())[0].grad_fn.name()
    assert _call(kla, _leaves(wrt=()))[0].grad_fn is None


@pytest.mark.parametrize("wrt", [("q",), ("h0",), ("v", "eta"), NAMES[:5]])
@pytest.mark.parametrize("outs", [(0,), (1,), (0, 1)])
def test_some_gradients(kla, wrt, outs):
    def run():
        x = _leaves(wrt=wrt)
        o = _call(kla, x, normalize_q=True)
        loss = sum((o[i].float() * torch.linspace(-1, 1, o[i].numel(), device="cuda").view(o[i].shape)).sum() for i in outs)
        return torch.autograd.grad(loss, [t for t in x if t.requires_grad], allow_unused=True)
    _same(run(), _python(kla, run))


def test_without_h0_and_packed(kla):
    cu = torch.tensor([0, 100, 100, 150], dtype=torch.int32)

    def run(packed):
        x = [t.detach()[:1].requires_grad_(True) for t in _leaves()[:5]]
        o, hT = kla.kla_chunk(*x, 1e-6, **(dict(cu_seqlens=cu.cuda()) if packed else {}))
        return torch.autograd.grad([o.float().sum(), hT.sum()], x)
    for packed in (False, True):
        _same(run(packed), _python(kla, lambda: run(packed)))


def test_gradient_layouts_and_hooks(kla):
    def run(ctx=None):
        x = _leaves()
        with ctx or torch.enable_grad():
            o, hT = _call(kla, x)
        d = torch.randn(o.shape[::-1], generator=torch.Generator("cuda").manual_seed(1), device="cuda").bfloat16().permute(3, 2, 1, 0)
        return torch.autograd.grad([o, hT], x, [d, hT.detach().expand_as(hT)])
    ref = _python(kla, run)
    _same(run(), ref)
    _same(run(torch.autograd.graph.save_on_cpu()), ref)
    seen = []
    _same(run(torch.autograd.graph.saved_tensors_hooks(lambda t: seen.append(t.shape) or t.clone(), lambda t: t)), ref)
    assert len(seen) >= 7                                # the six inputs and what the forward leaves behind


def test_offsets_between_the_directions(kla):
    """A packed batch whose offsets change after its forward: the caller's host copy does not matter any more, the device's are
    refused (an inference tensor's, which count no changes, were copied); natively and step by step."""
    offs = torch.tensor([0, 100, 100, 150], dtype=torch.int32)

    def run(touch, host, inference=False):
        with torch.inference_mode(inference):
            cu = offs.cuda()
        mine = offs.clone() if host else None
        x = [t.detach()[:1].requires_grad_(True) for t in _leaves()[:5]]
        o, hT = kla.kla_chunk(*x, 1e-6, cu_seqlens=cu, cu_seqlens_host=mine)
        with torch.inference_mode(inference):
            touch(cu, mine)
        return torch.autograd.grad([o.float().sum(), hT.sum()], x)
    for call in (lambda f: f(), lambda f: _python(kla, f)):
        ref = call(lambda: run(lambda cu, mine: None, True))
        _same(ref, call(lambda: run(lambda cu, mine: mine.copy_(torch.tensor([0, 1, 2, 150])), True)))
        _same(ref, call(lambda: run(lambda cu, mine: cu.copy_(torch.tensor([0, 1, 2, 150])), False, True)))
        for host in (True, False):
            with pytest.raises(RuntimeError, match="modified by an inplace"):
                call(lambda: run(lambda cu, mine: cu.add_(0), host))


@pytest.mark.parametrize("swap", [lambda t: t.cpu(), lambda t: t.repeat_interleave(2)[::2], lambda t: t.view(torch.float32), lambda t: t[:-1]])
def test_hook_swaps_what_the_forward_left(kla, swap):
    """The bytes that the forward leaves behind go to the kernels as a pointer: others than it left are refused, natively and step by step."""
    def run():
        x = _leaves()
        with torch.autograd.graph.saved_tensors_hooks(lambda t: t, lambda t: swap(t) if t.dtype == torch.uint8 else t):
            o, _ = _call(kla, x)
        with pytest.raises((RuntimeError, ValueError, TypeError)):
            torch.autograd.grad(o.float().sum(), x)
    run()
    _python(kla, run)


def test_checkpointing(kla):
    x = _leaves()
    f = lambda *y: _call(kla, y)[0]
    ref = torch.autograd.grad(f(*x).float().sum(), x)
    _same(torch.autograd.grad(torch.utils.checkpoint.checkpoint(f, *x, use_reentrant=False).float().sum(), x), ref)


@pytest.mark.parametrize("N,T,H,dk,dv", [(8, 130, 8, 128, 128), (12, 65, 9, 64, 64), (30, 64, 8, 128, 128)])
def test_same_outputs_without_gradients(kla, N, T, H, dk, dv):
    """bf16 batches whose plain forward is one kernel: kla_chunk gives kla_chunk_fwd's bits whether a gradient is wanted or not, so that
    checkpointing whose first pass runs without gradients (re-entrant) differentiates the outputs it handed on."""
    d = kla_inputs.chunk_inputs(N, T, H, dk, dv, seed=T + dv, h0_std=0.1)
    x = [d[n].cuda().requires_grad_(True) for n in NAMES]
    plain = kla.kla_chunk_fwd(*(t.detach() for t in x[:5]), 1e-6, h0=x[5].detach())
    with torch.no_grad():
        _same(plain, _call(kla, x))
    got = _call(kla, x)
    _same(plain, got)
    w = torch.linspace(-1, 1, got[0].numel(), device="cuda").view(got[0].shape)
    ref = torch.autograd.grad((got[0].float() * w).sum() + got[1].sum(), x)
    again = torch.utils.checkpoint.checkpoint(lambda *y: _call(kla, y), *x, use_reentrant=True)
    _same(plain, again)
    # (the re-entrant form takes backward() only)
    ((again[0].float() * w).sum() + again[1].sum()).backward()
    _same(ref, [t.grad for t in x])


def test_refusals(kla):
    x = _leaves()
    o, _ = _call(kla, x)
    with torch.no_grad():
        x[1].add_(1.0)
    with pytest.raises(RuntimeError, match="modified by an inplace"):
        o.float().sum().backward()
    o, _ = _call(kla, _leaves())
    o.float().sum().backward()
    with pytest.raises(RuntimeError, match="second time"):
        o.float().sum().backward()
    y = [t.detach() for t in _leaves()]
    for f in (lambda: torch.func.grad(lambda q: kla.kla_chunk(q, *y[1:5], 1e-6, h0=y[5])[0].float().sum())(y[0]),
              lambda: torch.func.vmap(lambda q: kla.kla_chunk(q, *y[1:5], 1e-6, h0=y[5])[0])(y[0][None]),
              lambda: _call(kla, [y[0][:, :, :, :32]] + y[1:])):
        with pytest.raises(Exception) as fast:
            f()
        with pytest.raises(Exception) as slow:
            _python(kla, f)
        assert type(fast.value) is type(slow.value) and str(fast.value) == str(slow.value)
    with torch.autograd.forward_ad.dual_level():
        z = [torch.autograd.forward_ad.make_dual(y[0], torch.ones_like(y[0]))] + y[1:]
        with pytest.raises(RuntimeError):
            _call(kla, z)


def test_errors_of_the_backward(kla):
    """What the native node refuses in the backward raises what the Python function raises: type, code and text."""
    def unaligned():                                     # an output gradient that does not start at 16 bytes
        o, _ = _call(kla, _leaves())
        d = torch.zeros(o.numel() + 1, dtype=o.dtype, device="cuda")[1:].view(o.shape)
        torch.autograd.grad(o, o.grad_fn.next_functions[0][0].variable, d)

    def strided():                                       # a hook that hands back an input of other strides
        x = _leaves()
        with torch.autograd.graph.saved_tensors_hooks(lambda t: t, lambda t: t.transpose(0, 1) if t.dim() == 4 else t):
            o, _ = _call(kla, x)
        torch.autograd.grad(o.float().sum(), x[0])
    for f in (unaligned, strided):
        with pytest.raises(Exception) as fast:
            f()
        with pytest.raises(Exception) as slow:
            _python(kla, f)
        assert type(fast.value) is type(slow.value) and str(fast.value) == str(slow.value)
        assert getattr(fast.value, "code", None) == getattr(slow.value, "code", None)
    assert type(slow.value) is ValueError
    with pytest.raises(kla.KlaError) as e:
        unaligned()
    assert e.value.code == -4


def test_streams(kla):
    """Forward on a side stream: the backward runs there too, whatever stream is current when it is called."""
    x = _leaves()
    ref = torch.autograd.grad(_call(kla, x)[0].float().sum(), x)
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        y = _leaves()
        loss = _call(kla, y)[0].float().sum()
    torch.cuda.current_stream().wait_stream(s)
    got = torch.autograd.grad(loss, y)
    torch.cuda.synchronize()
    _same(got, ref)
