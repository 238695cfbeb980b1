"""Compute waves per workgroup of the bf16 sweeps by the lengths of the sequences (csrc/kla_widths.hpp, host code): up to 256 chains of
sixteen columns one; beyond, two, unless the batch is packed and so unequal that the workgroups of a second round fit behind the
longest sequence."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_08587_amd", "csrc")
WRAP = """#include "kla_widths.hpp"
extern "C" int sweep(int n, int NT, const int32_t* cu, int H, int dv) { return kla::sweep_waves({n, NT, cu}, H, dv, true); }
extern "C" int diag(int n, int NT, const int32_t* cu, int H, int dk, int dv) { return kla::diag_scan_waves({n, NT, cu}, H, dk, dv); }
"""


@pytest.fixture(scope="module")
def widths(tmp_path_factory):
    d = tmp_path_factory.mktemp("widths")
    (d / "w.cpp").write_text(WRAP)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I" + CSRC, str(d / "w.cpp"), "-o", str(d / "w.so")])
    lib = ctypes.CDLL(str(d / "w.so"))

    def of(lens, H, dk, dv):
        if isinstance(lens, tuple):                      # (N, T): equal lengths
            n, nt, cu = lens[0], (lens[1] + 63) // 64, None
        else:
            n, nt, cu = len(lens), 0, (ctypes.c_int32 * (len(lens) + 1))(*[sum(lens[:i]) for i in range(len(lens) + 1)])
        return lib.sweep(n, nt, cu, H, dv), lib.diag(n, nt, cu, H, dk, dv)
    return of


@pytest.mark.parametrize("lens,H,dk,dv,sweep,diag", [
    ([4000, 300, 300, 300, 200], 8, 128, 128, 1, 1), ([3000, 1500, 700, 400, 300], 8, 128, 128, 1, 1),
    ([2500, 1200, 1000, 800, 600], 8, 128, 128, 1, 1), ([4000, 300, 300, 300, 200], 8, 128, 256, 1, 1),
    ([8000] + [100] * 70, 8, 128, 128, 1, 1), ([3000, 1500, 700, 400, 300], 16, 64, 64, 1, 2),
    ([2000, 1800, 1700, 1600, 300], 8, 128, 128, 1, 2), ([3000, 100], 16, 128, 256, 1, 2), ([0, 2000, 0], 16, 128, 128, 1, 1),
    ([300, 64, 1, 130, 60], 8, 128, 128, 1, 1), ([449, 100, 0, 64, 1, 127], 16, 128, 64, 1, 1)])
def test_second_round_is_free(widths, lens, H, dk, dv, sweep, diag):
    assert widths(lens, H, dk, dv) == (sweep, diag)


@pytest.mark.parametrize("lens,H,dk,dv,sweep,diag", [
    ([2000] * 5, 8, 128, 128, 2, 2), ([2000, 1900, 1900, 1800, 300], 8, 128, 128, 2, 2), ([1500, 1400, 1300, 1200, 1100], 8, 128, 128, 2, 2), ([3000, 500], 16, 128, 256, 2, 2),
    ([130, 70, 60, 30, 20], 8, 128, 128, 2, 2), ([4000] + [200] * 40, 8, 128, 128, 2, 2), ([64] * 5, 8, 128, 128, 2, 2),
    ((4, 2000), 8, 128, 128, 1, 1), ((5, 2000), 8, 128, 128, 2, 2), ((5, 64), 8, 128, 128, 2, 2), ((8, 4096), 8, 128, 128, 2, 2),
    ((9, 2000), 8, 128, 128, 4, 2), ((1, 0), 64, 128, 128, 2, 2), ([65, 64, 63, 1, 128], 8, 128, 128, 2, 2),
    ([200, 190, 180, 170, 129], 8, 128, 128, 2, 2), ([192, 129, 190, 65, 130, 191, 150, 180, 140], 8, 64, 128, 4, 2),
    ([385, 321, 320, 449, 448], 8, 64, 128, 2, 2), ([257, 256, 255, 193, 192, 250], 16, 128, 64, 2, 2),
    ([2304, 2241, 2303, 2250, 2277, 2299], 16, 128, 64, 2, 2), ([3584, 3583, 3521, 3550, 3577, 3530], 16, 64, 64, 2, 2)])
def test_otherwise_by_the_number_of_chains(widths, lens, H, dk, dv, sweep, diag):
    assert widths(lens, H, dk, dv) == (sweep, diag)
