"""kla_chunk's forward leaves the per-chunk operands and states behind for its backward (kla_chunk_fwd_save, kla_chunk_bwd_saved):
the same bits as the two calls by hand, whose backward recomputes them, for the row-split bf16 scan, for its workgroups of 2, 4 and 8
waves and for each form of the fp32 one; last chunks of 1, 63 and 64 rows, packed batches with empty sequences, both options."""
import pytest
import torch

import kla_inputs

pytestmark = pytest.mark.gpu
B, F = torch.bfloat16, torch.float32


@pytest.fixture(scope="module")
def kla():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_08587_amd as m
    m.lib()
    return m


def _case(dt, N, T, H, dk, dv, lens, seed):
    cu = None
    if lens:
        cu = torch.tensor([0] + [sum(lens[:i + 1]) for i in range(len(lens))], dtype=torch.int32)
        N, T = 1, int(cu[-1])
    d = kla_inputs.chunk_inputs(N, T, H, dk, dv, dtype=dt, seed=seed, h0_std=0.3, n_h0=len(lens) if lens else None, log_alpha_scale=0.1)
    gen = torch.Generator().manual_seed(seed)
    d_o, d_hT = (torch.randn(d[n].shape, generator=gen).to(d[n].dtype).cuda() for n in ("v", "h0"))
    return [d[n].cuda() for n in ("q", "k", "v", "log_alpha", "eta", "h0")], d_o, d_hT, cu


@pytest.mark.parametrize("dt,N,T,H,dk,dv,lens,opts", [
    (B, 1, 1, 3, 128, 128, None, {}), (B, 2, 64, 2, 64, 64, None, {}), (B, 2, 200, 4, 128, 128, None, dict(normalize_q=True)),
    (B, 3, 70, 8, 128, 256, None, {}), (B, 6, 127, 8, 64, 256, None, dict(gdn_beta=True)), (B, 10, 65, 10, 128, 256, None, {}),
    (B, 0, 0, 5, 128, 128, [130, 0, 64, 1, 63], {}), (B, 0, 0, 9, 64, 256, [65] * 11, dict(normalize_q=True)),
    (B, 0, 0, 1, 64, 64, [3] * 70, {}),
    (F, 1, 1, 3, 128, 128, None, {}), (F, 2, 200, 4, 64, 64, None, dict(normalize_q=True)), (F, 5, 130, 8, 128, 128, None, {}),
    (F, 10, 65, 8, 64, 128, None, dict(gdn_beta=True)), (F, 0, 0, 3, 128, 128, [64, 0, 127, 2], {}),
])
def test_saved_equals_recomputed(kla, dt, N, T, H, dk, dv, lens, opts):
    x, d_o, d_hT, cu = _case(dt, N, T, H, dk, dv, lens, 11 + T)
    if opts.get("gdn_beta"):                         # the gated delta rule needs keys of length one
        x[1] = (x[1].float() / x[1].float().norm(dim=-1, keepdim=True)).to(dt)
    packed = dict(cu_seqlens=None if cu is None else cu.cuda(), cu_seqlens_host=cu)
    o, hT = kla.kla_chunk_fwd(*x[:5], 1e-6, h0=x[5], **packed, **opts)
    ref = kla.kla_chunk_bwd(*x[:5], 1e-6, d_o, h0=x[5], d_hT=d_hT, **packed, **opts)
    o_opts = (opts.get("normalize_q", False), opts.get("gdn_beta", False))
    assert kla._fwd_save(*x[:5], 1e-6, x[5], packed["cu_seqlens"], cu, *o_opts)[2] is not None
    for native in (True, False):                     # the native half of the binding and the calls step by step
        with pytest.MonkeyPatch.context() as m:
            if not native:
                m.setattr(kla, "_native", kla._StepByStep)
            y = [t.detach().requires_grad_(True) for t in x]
            o2, h2 = kla.kla_chunk(*y[:5], 1e-6, h0=y[5], **packed, **opts)
            assert torch.equal(o, o2) and torch.equal(hT, h2)
            for a, b in zip(torch.autograd.grad([o2, h2], y, [d_o, d_hT]), ref.values()):
                assert torch.equal(a, b)


@pytest.mark.parametrize("T,lens", [(1, None), (65, None), (300, None), (449, None), (0, [449, 320, 0, 449, 385, 449, 1, 400, 449])])
def test_four_waves(kla, T, lens):
    """d_k = 128, where four compute waves read from two LDS rings: these batches (512 workgroups of two waves, 256 of four) leave behind
    with four; the outputs, and the gradients from what was left, are those of one and two waves and of the two calls by hand."""
    x, d_o, d_hT, cu = _case(B, 8, T, 8, 128, 256, lens, 3 + T)
    packed = dict(cu_seqlens=None if cu is None else cu.cuda(), cu_seqlens_host=cu)

    def run(waves):
        with pytest.MonkeyPatch.context() as m:
            m.setattr(kla, "DEFAULT_TUNE", kla.tune(scan_waves=waves))
            y = [t.detach().requires_grad_(True) for t in x]
            assert kla._fwd_save(*x[:5], 1e-6, x[5], packed["cu_seqlens"], cu, False, False)[2] is not None
            out = kla.kla_chunk(*y[:5], 1e-6, h0=y[5], **packed)
            return [*(t.detach() for t in out), *torch.autograd.grad(out, y, [d_o, d_hT])]
    got = run(0)
    by_hand = [*kla.kla_chunk_fwd(*x[:5], 1e-6, h0=x[5], **packed), *kla.kla_chunk_bwd(*x[:5], 1e-6, d_o, h0=x[5], d_hT=d_hT, **packed).values()]
    for other in (by_hand, run(4), run(2), run(1)):
        assert all(torch.equal(a, b) for a, b in zip(got, other))


@pytest.mark.parametrize("N,T,H,dv", [(8, 70, 8, 128), (1, 4160, 2, 128), (2, 0, 2, 64)])
def test_nothing_saved(kla, N, T, H, dv):
    """One kernel, segments, no tokens: kla_chunk goes on as the two calls by hand do."""
    x, d_o, d_hT, _ = _case(B, N, T, H, 128, dv, None, 5)
    assert kla._fwd_save(*x[:5], 1e-6, x[5], None, None, False, False)[2] is None
    y = [t.detach().requires_grad_(True) for t in x]
    o, hT = kla.kla_chunk(*y[:5], 1e-6, h0=y[5])
    o2, h2 = kla.kla_chunk_fwd(*x[:5], 1e-6, h0=x[5])
    assert torch.equal(o, o2) and torch.equal(hT, h2)
    ref = kla.kla_chunk_bwd(*x[:5], 1e-6, d_o, h0=x[5], d_hT=d_hT)
    for a, b in zip(torch.autograd.grad([o, hT], y, [d_o, d_hT]), ref.values()):
        assert torch.equal(a, b)


def test_no_grad_saves_nothing(kla):
    x, _, _, _ = _case(B, 2, 200, 2, 128, 128, None, 3)
    y = [t.detach().requires_grad_(True) for t in x]
    torch.cuda.synchronize()
    with torch.no_grad():
        kla.kla_chunk(*y[:5], 1e-6, h0=y[5])
        before = torch.cuda.memory_allocated()
        keep = kla.kla_chunk(*y[:5], 1e-6, h0=y[5])
        assert torch.cuda.memory_allocated() - before < 2 * sum(t.numel() * t.element_size() for t in keep)
        assert not keep[0].requires_grad


@pytest.mark.parametrize("native", [True, False])
def test_save_switched_off(kla, native):
    """save=False: nothing but the outputs is held between the directions; same bits."""
    x, d_o, d_hT, _ = _case(B, 4, 1000, 16, 128, 256, None, 9)
    y = [t.detach().requires_grad_(True) for t in x]
    got, held = [], []
    with pytest.MonkeyPatch.context() as m:
        if not native:
            m.setattr(kla, "_native", kla._StepByStep)
        for save in (True, False):
            before = torch.cuda.memory_allocated()
            out = kla.kla_chunk(*y[:5], 1e-6, h0=y[5], save=save)
            held.append(torch.cuda.memory_allocated() - before - sum(t.nbytes for t in out))
            got.append([*out, *torch.autograd.grad(out, y, [d_o, d_hT])])
            del out
    assert all(torch.equal(a, b) for a, b in zip(*got))
    assert held[0] >= kla.lib().kla_chunk_saved_bytes(4, 1000, 16, 128, 256, 64, kla.KLA_BF16, None, 0, 0) and held[1] <= 1 << 20


@pytest.mark.parametrize("room", ["plain", "saved"])
@pytest.mark.parametrize("native", [True, False])
def test_no_memory_to_save(kla, native, room):
    """Memory for the plain forward but not for what it would leave behind, or for that and nothing else: the backward recomputes."""
    x, d_o, d_hT, _ = _case(B, 4, 1000, 16, 128, 256, None, 9)
    y = [t.detach().requires_grad_(True) for t in x]
    ref = torch.autograd.grad(kla.kla_chunk(*y[:5], 1e-6, h0=y[5]), y, [d_o, d_hT])
    sizes = (4, 1000, 16, 128, 256, 64, kla.KLA_BF16, None, 0)
    keep = kla.lib().kla_chunk_saved_bytes(*sizes, 0)
    plain = kla.lib().kla_chunk_fwd_workspace_bytes(*sizes) + x[2].nbytes + x[5].nbytes + (20 << 20)     # (20 MiB: the allocator's rounding)
    assert plain < 0.8 * keep
    total = torch.cuda.get_device_properties(0).total_memory
    kinds = []
    with pytest.MonkeyPatch.context() as m:
        if not native:
            m.setattr(kla, "_native", kla._StepByStep)
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        full = []                                        # what other tests hold may leave room in its segments: none of it counts
        try:
            torch.cuda.set_per_process_memory_fraction(torch.cuda.memory_reserved() / total)
            for mib in (1024, 256, 64, 16, 4, 1):
                try:
                    while True:
                        full.append(torch.empty(mib << 20, dtype=torch.uint8, device="cuda"))
                except torch.OutOfMemoryError:
                    pass
            limit = torch.cuda.memory_reserved() + int(0.8 * keep if room == "plain" else keep + (2 << 20))
            torch.cuda.set_per_process_memory_fraction(limit / total)
            with torch.autograd.graph.saved_tensors_hooks(lambda t: kinds.append(t.dtype) or t, lambda t: t):
                out = kla.kla_chunk(*y[:5], 1e-6, h0=y[5])
        finally:
            torch.cuda.set_per_process_memory_fraction(1.0)
        assert torch.uint8 not in kinds and len(kinds) >= 6
        for a, b in zip(torch.autograd.grad(out, y, [d_o, d_hT]), ref):
            assert torch.equal(a, b)
