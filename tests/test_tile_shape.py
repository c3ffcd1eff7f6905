"""Shapes of the row-flattened tiles, from the library's own functions
(csrc/tile_shape.hpp compiled for the host): the fixed LDS that the persistent
kernels reserve holds every grid's tile, a block has a thread for every chunk
that it loads, and the levels per tile fill the CUs in rounds."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r"""
#include "tile_shape.hpp"
extern "C" {
int max_chunks(int t) { return kl::rf_max_chunks(t); }
int rows(int j, int c, int t) { return kl::rf_rows(j, c, t); }
long lds(int c, int r) { return (long)kl::rf_lds_bytes(c, r); }
long lds_fixed(int t) { return (long)(t == 256 ? kl::RF_LDS_256 : kl::RF_LDS_512); }
int levels(int nby, int k, int t) { return kl::rf_levels(nby, k, t); }
int les_levels(int slab, int k) { return kl::les_rf_levels(slab, k); }
void les_shape(int kernel, int i, int j, int vx, long *o)
{
    const kl::LesRfShape s = kl::les_rf_shape(kernel, i, j, vx);
    o[0] = s.W; o[1] = s.R; o[2] = s.threads; o[3] = (long)s.lds;
}
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("tile_shape")
    (d / "t.cpp").write_text(SRC)
    so = d / "t.so"
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-Wall", "-Werror",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2303_12374_amd", "csrc"),
                    str(d / "t.cpp"), "-o", str(so)], check=True)
    lib = ctypes.CDLL(str(so))
    lib.lds.restype = lib.lds_fixed.restype = ctypes.c_long
    return lib


@pytest.mark.parametrize("threads", [256, 512])
def test_tiles_fit_the_block_and_the_reserved_lds(lib, threads):
    top = lib.max_chunks(threads)
    assert 2 * top <= threads  # a thread for every chunk of the two halo rows
    for cpr in range(1, top + 1):
        for j in (1, 2, 3, 4, 5, 7, 16, 63, 64, 255, 256, 257, 1000, 4096):
            R = lib.rows(j, cpr, threads)
            assert 1 <= R <= j and R * cpr <= threads
            assert -(-j // R) == -(-j // min(threads // cpr, j))  # equal heights, as few blocks
            assert lib.lds(cpr, R) <= lib.lds_fixed(threads) <= 160 * 1024


def cost(nby, ktot, kb):
    return -(-nby * -(-ktot // kb) // 256) * (kb + 5)


@pytest.mark.parametrize("nby", [1, 2, 3, 16, 25, 50, 64, 100, 107, 125, 128, 149, 185, 190, 200, 250, 256, 257, 300, 318,
                                 353, 400, 512, 513, 1000])
def test_levels_leave_no_round_nearly_empty(lib, nby):
    """Blocks of 512 threads run 256 at a time: no march of whole slabs that fills
    the chip needs a tenth less (levels and five more a tile, times rounds)."""
    for ktot in (1, 2, 7, 8, 9, 17, 32, 50, 64, 80, 100, 137, 151, 214, 264, 380, 512, 1000):
        kb = lib.levels(nby, ktot, 512)
        assert kb >= 2
        for n in range(1, min(16, ktot // 8) + 1):
            k = -(-ktot // n)
            if nby * -(-ktot // k) >= 240:
                assert cost(nby, ktot, kb) <= cost(nby, ktot, k) / 0.9 + 1e-9, (ktot, kb, k)
        # two blocks of 256 threads share a CU: about 512 tiles
        kb = lib.levels(nby, ktot, 256)
        assert kb == max(2, -(-ktot // max(1, 512 // nby)))


def test_thin_grids_of_the_papers_schemes_fill_the_cus(lib):
    for slab in (1, 2, 3):
        for ktot in (512, 1024, 2048, 4096):
            kb = lib.les_levels(slab, ktot)
            assert slab * -(-ktot // kb) >= 192, (slab, ktot, kb)
    for slab in range(4, 700, 37):  # whole range: a march of one to all levels
        for ktot in (1, 2, 3, 64, 151, 512):
            assert 1 <= lib.les_levels(slab, ktot) <= ktot


@pytest.mark.parametrize("kernel,vx", [(3, 4), (3, 2), (4, 4), (4, 2)])
def test_les_tiles_fit(lib, kernel, vx):
    o = (ctypes.c_long * 4)()
    for itot in list(range(8, 300)) + [512, 513, 1000, 1024, 4096, 4099]:
        for j in (1, 2, 5, 16, 180, 513):
            lib.les_shape(kernel, itot, j, vx, o)
            W, R, threads, lds = o
            assert 1 <= R <= j and R * W <= threads <= 512 and threads % 64 == 0 and lds <= 160 * 1024
