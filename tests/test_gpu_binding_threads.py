"""The binding lets other Python threads run while it allocates and launches: two threads, each on a stream of its own, through
decode steps, forwards and training steps at once, every result equal to the one computed alone."""
import threading

import pytest
import torch

import kla_inputs

pytestmark = pytest.mark.gpu


def test_two_threads():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_08587_amd as kla
    assert kla._binding().__name__ == "kla_binding"
    host = torch.tensor([0, 70, 71, 150], dtype=torch.int32)

    def work(seed):
        d = kla_inputs.chunk_inputs(1, 150, 2, 64, 128, seed=seed, h0_std=0.1, n_h0=3)
        x = [d[n].cuda().requires_grad_(True) for n in ("q", "k", "v", "log_alpha", "eta", "h0")]
        e = kla_inputs.decode_inputs(1, 3, 2, 64, 128, seed=seed)
        y = [e[n][0].contiguous().cuda() for n in ("q", "k", "v", "log_alpha", "eta")]
        d_o, S0, cu = kla_inputs.grad_inputs(d, seed)[0].cuda(), e["S"].cuda(), host.cuda()

        def once():
            S = S0.clone()
            o = kla.kla_decode_step(*y, 1e-6, S)
            packed = dict(cu_seqlens=cu, cu_seqlens_host=host)
            f = kla.kla_chunk_fwd(*(t.detach() for t in x[:5]), 1e-6, **packed)
            t = kla.kla_chunk(*x[:5], 1e-6, h0=x[5], **packed)
            return (o, S, *f, *(u.detach() for u in t), *torch.autograd.grad(t[0], x, d_o))
        return once

    jobs = [work(1), work(2)]
    alone = [j() for j in jobs]
    torch.cuda.synchronize()
    wrong, done = [], []

    def loop(i):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            for it in range(50):
                got = jobs[i]()
                s.synchronize()
                if not all(torch.equal(a, b) for a, b in zip(got, alone[i])):
                    wrong.append((i, it))
        done.append(i)

    threads = [threading.Thread(target=loop, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert sorted(done) == [0, 1] and not wrong
