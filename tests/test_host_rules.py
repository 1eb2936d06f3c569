"""The host-side rules of the kernels' header, compiled for the CPU."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include "lbc_internal.h"
using namespace lbc;
extern "C" int order_pays_c(int sb, int K, long long np, long long N) { return order_pays(sb, K, np, N); }
extern "C" int rows_fit_c(int nx, int sb) { return rows_fit(nx, sb); }
extern "C" void image_bounds_c(double L, double* b) { image_bounds(L, b[0], b[1]); }
extern "C" void div_rem_c(const uint32_t* n, long long count, uint32_t d, uint32_t* q, uint32_t* r) {
  for (long long i = 0; i < count; ++i) q[i] = div_rem(n[i], d, div_magic((int)d), r[i]);
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.hip").write_text(SOURCE)
    lib = str(d / "rules.so")
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-host-only", "-O1", "-std=c++17",
                    "-fPIC", "-shared", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_1406_2211_amd", "csrc"), str(d / "rules.hip"), "-o", lib],
                   check=True)
    return C.CDLL(lib)


@pytest.mark.parametrize("K", [2, 3, 4])
def test_tile_order_is_not_taken_by_16_bit_boxes(rules, K):
    """Dense free particles are processed in tile order, except on 16-bit
    storage, whose populations a changed order of the sums moves by a quantum."""
    f = rules.order_pays_c
    f.argtypes = [C.c_int, C.c_int, C.c_longlong, C.c_longlong]
    for n, N in ((4096, 4096), (13694, 80 * 180 * 147), (1 << 20, 1 << 20)):
        assert not f(2, K, n, N)
    for sb in (4, 8):
        N = 4096 * K * K * 128 // sb  # one row of nodes per line
        assert f(sb, K, 4096, N) and not f(sb, K, 4095, N) and not f(sb, K, 4096, N + 128)


def test_rows_beyond_32_bit_offsets_take_the_linear_site_pass(rules):
    """The row-mapped pass holds x times the stored size in 32 bits; longer rows,
    which the grid check admits, go to the pass that has a 64-bit form."""
    for sb in (2, 4, 8):
        most = (2**32 - 1) // sb // 64 * 64  # the longest row whose offsets fit
        for nx in (64, 128, most, min(most + 64, 2**31 - 64)):
            assert bool(rules.rows_fit_c(nx, sb)) == (nx * sb < 2**32), (nx, sb)
        assert not rules.rows_fit_c(100, sb) and not rules.rows_fit_c(most - 1, sb)


def test_nearest_image_is_that_of_the_division(rules):
    """Two compares with the bounds give floor(d/L + 1/2) as the division rounds
    it, at every d within four units in the last place of half a box and over
    the whole range of |d| <= L."""
    f = rules.image_bounds_c
    f.argtypes = [C.c_double, C.c_void_p]
    lengths = list(range(1, 3000)) + [4095, 4097, 65535, 99991, 2**20 + 1, 2**24 - 1, 2**30 + 7, 2**31 - 1]
    for n in lengths:
        L, b = float(n), np.zeros(2)
        f(L, b.ctypes.data)
        d = [0.0, L, -L, np.nextafter(L, 0), np.nextafter(-L, 0)]
        for h in (0.5 * L, -0.5 * L):
            up = down = h
            d.append(h)
            for _ in range(4):
                up, down = np.nextafter(up, np.inf), np.nextafter(down, -np.inf)
                d += [up, down]
        d = np.concatenate([d, np.linspace(-L, L, 41)])
        image = np.where(d >= b[1], 1.0, np.where(d < b[0], -1.0, 0.0))
        assert (image == np.floor(d / L + 0.5)).all(), n


@pytest.mark.parametrize("d", [1, 2, 3, 5, 7, 45, 63, 64, 65, 117, 150, 255, 256, 257, 1000, 4095, 4097, 65535, 65536,
                               65537, 2**30, 2**31 - 1])
def test_quotient_of_the_linear_site_pass(rules, d):
    """div_rem with div_magic, as the kernels call them: the exact quotient and
    remainder of every 32-bit site index by a box side."""
    g = np.random.default_rng(d)
    k = g.integers(0, 2**32 // d, 50000, dtype=np.uint64) * np.uint64(d)  # multiples and their neighbours
    n = np.concatenate([g.integers(0, 2**32, 200000, dtype=np.uint64), np.arange(2000, dtype=np.uint64),
                        2**32 - 1 - np.arange(2000, dtype=np.uint64), k, k + np.uint64(1), k - np.uint64(1)])
    n = n[n < 2**32].astype(np.uint32)
    q, r = np.empty_like(n), np.empty_like(n)
    rules.div_rem_c(n.ctypes.data_as(C.c_void_p), C.c_longlong(n.size), C.c_uint32(d), q.ctypes.data_as(C.c_void_p),
                    r.ctypes.data_as(C.c_void_p))
    assert (q == n // np.uint32(d)).all() and (r == n % np.uint32(d)).all()
