"""C ABI of the forward that leaves its intermediates and the backward that takes them: sizes and refusals, without a GPU."""
import ctypes
import timeit

import pytest

kla = pytest.importorskip("paper_2605_08587_amd")
E_NULL, E_SHAPE, E_DTYPE, E_ALIGN, E_WS = -1, -2, -3, -4, -5


@pytest.fixture(scope="module")
def lib():
    return kla.lib()


def test_sizes(lib):
    r256 = lambda x: (x + 255) // 256 * 256
    for dt, eb in ((kla.KLA_BF16, 2), (kla.KLA_F32, 4)):
        N, T, H, dk, dv = 3, 200, 2, 128, 256
        ch, rows = N * 4 * H, r256(N * T * H * dv * eb)
        a = (N, T, H, dk, dv, 64, dt, None, 0, 0)
        saved = r256(r256(ch * (3 * 384 * 8 * eb + 1280)) + 4) + r256(ch * dk * dv * eb) + (1 if eb == 2 else 2) * rows
        assert lib.kla_chunk_saved_bytes(*a) == saved
        # the two parts are the workspace of the backward that recomputes
        assert saved + lib.kla_chunk_bwd_saved_workspace_bytes(*a) == lib.kla_chunk_bwd_workspace_bytes(*a[:-1])
    for none in ((8, 4096, 8, 128, 128), (1, 8192, 2, 128, 128), (2, 0, 2, 64, 64), (1, 1 << 20, 8, 64, 64)):   # one kernel, segments, empty, too large
        assert lib.kla_chunk_saved_bytes(*none, 64, kla.KLA_BF16, None, 0, 0) == 0
        assert lib.kla_chunk_bwd_saved_workspace_bytes(*none, 64, kla.KLA_BF16, None, 0, 0) == 0
    for bits in (kla.tune(generic_bwd=True), kla.tune(generic_scan=True), kla.tune(generic_intra=True), kla.tune(fused=True)):
        assert lib.kla_chunk_saved_bytes(2, 200, 2, 64, 64, 64, kla.KLA_BF16, None, 0, bits) == 0


def test_refusals(lib):
    p = {n: ctypes.c_void_p(0x10000 * (i + 1)) for i, n in enumerate(("q", "k", "v", "la", "eta", "o", "dq", "dk", "dv", "dla", "deta", "do"))}
    sizes = [2, 200, 2, 64, 64, 64, kla.KLA_BF16]
    n_fwd = lib.kla_chunk_fwd_workspace_bytes(*sizes, None, 0)
    n_sv, n_bwd = lib.kla_chunk_saved_bytes(*sizes, None, 0, 0), lib.kla_chunk_bwd_saved_workspace_bytes(*sizes, None, 0, 0)

    def fwd(o=p["o"], sizes=sizes, ws=0x100000, nws=n_fwd, sv=0x200000, nsv=n_sv):
        return lib.kla_chunk_fwd_save(p["q"], p["k"], p["v"], p["la"], p["eta"], 1e-6, None, o, None, None, None, 0, *sizes, ws, nws, sv,
                                      nsv, None, 0)

    def bwd(do=p["do"], sizes=sizes, ws=0x100000, nws=n_bwd, sv=0x200000, nsv=n_sv):
        return lib.kla_chunk_bwd_saved(p["q"], p["k"], p["v"], p["la"], p["eta"], 1e-6, None, do, None, p["dq"], p["dk"], p["dv"], p["dla"],
                                       p["deta"], None, None, None, 0, *sizes, ws, nws, sv, nsv, None, 0)

    for f, n in ((fwd, n_fwd), (bwd, n_bwd)):
        assert f(None) == E_NULL
        assert f(sizes=[8, 4096, 8, 128, 128, 64, kla.KLA_BF16]) == E_SHAPE          # runs as one kernel: leaves nothing
        assert f(sizes=sizes[:-1] + [7]) == E_DTYPE
        assert f(ws=None) == E_WS and f(sv=None) == E_WS
        assert f(nws=n - 1) == E_WS and f(nsv=n_sv - 1) == E_WS
        assert f(ws=0x100010) == E_WS and f(sv=0x200010) == E_WS
    assert fwd(ctypes.c_void_p(0x10008)) == E_ALIGN and bwd(ctypes.c_void_p(0x10008)) == E_ALIGN
    assert lib.kla_chunk_saved_bytes(2, 200, 2, 96, 64, 64, kla.KLA_BF16, None, 0, 0) == 0


@pytest.mark.parametrize("entry", ["kla_chunk_fwd_workspace_bytes_opts", "kla_chunk_saved_bytes", "kla_chunk_bwd_workspace_bytes_opts"])
def test_sizes_of_a_packed_batch_are_cheap(lib, entry):
    """The sizes of a packed batch do not pay for the widths of its kernels' workgroups: 64 sequences hardly
    dearer than one (quickest of many calls; 2 to 5 times that if the schedule of the workgroups is played through)."""
    n = 64
    offs = [0]
    for i in range(n):
        offs.append(offs[-1] + 100 + 37 * i % 900)
    cu = (ctypes.c_int32 * (n + 1))(*offs)
    f = getattr(lib, entry)
    quickest = lambda n_seq, bits: min(timeit.repeat(lambda: f(1, offs[n_seq], 8, 128, 256, 64, kla.KLA_BF16, cu, n_seq, bits), number=50, repeat=200))
    assert quickest(n, 0) < 1.6 * quickest(1, 0)
