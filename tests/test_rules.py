"""The host's rules on sizes and tables (csrc/dyn_rules.h), compiled here for the CPU."""
import ctypes as C
import itertools
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = """
#include "dyn_rules.h"
extern "C" double even_scale(const double* rho, int n, int n_bucket) { return dyn_even_scale(rho, n, n_bucket); }
extern "C" int space_windows(long long cell_tiles, int tile, long long staged, int waves) { return dyn_space_windows(cell_tiles, tile, staged, waves); }
extern "C" int freq_axis_staged(long long axis_lds, long long lds, long long blocks, int n_cu) { return dyn_freq_axis_staged((size_t)axis_lds, (size_t)lds, blocks, n_cu); }
extern "C" void freq_shape(int n_window, int G, int n_tick, int n_f, long long axis_lds, int n_cu, long long* o) {
  const DynFreqShape f = dyn_freq_shape(n_window, G, n_tick, n_f, (size_t)axis_lds, n_cu);
  const long long v[] = {f.wins, f.run, f.n_run, f.chunk, f.tabled, f.staged, f.blocks, (long long)f.lds};
  for (int i = 0; i < 8; ++i) o[i] = v[i];
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "shim.cpp").write_text(SHIM)
    lib = str(d / "librules.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-ffp-contract=off", "-Wall", "-Werror", "-shared", "-fPIC", "-I" + os.path.join(ROOT, "paper_2408_00741_amd", "csrc"),
                    str(d / "shim.cpp"), "-o", lib], check=True)
    r = C.CDLL(lib)
    r.even_scale.restype = C.c_double
    return r


def _even_scale(rules, rho, n_bucket=None):
    rho = np.ascontiguousarray(rho, np.float64)
    if n_bucket is None:
        n_bucket = int(np.clip(np.ceil(3.0 * rho[-1] / np.diff(rho).min()), 16, 4096))
    return rules.even_scale(rho.ctypes.data_as(C.c_void_p), rho.size, n_bucket)


@pytest.mark.parametrize("n", [2, 3, 16, 33, 64, 900, 2000])
def test_even_load_points(rules, n):
    """Points that are even up to their roundings; a look-up starts at a point above the load only a rounding beside a point."""
    for rho in (np.linspace(0.0, 0.95, n), np.cumsum(np.r_[0.0, np.full(n - 1, 0.95 / (n - 1))]), 3.0e7 * np.arange(n)):
        s = _even_scale(rules, rho)
        assert s > 0.0
        load = np.random.default_rng(n).uniform(0.0, rho[-1], 100_000)
        first = np.minimum((load * s).astype(np.int64), n - 2)
        assert (rho[first] <= load).all()
        for side in (-np.inf, np.inf):               # a rounding beside every point: the start is the bracket or the one above
            x = np.clip(np.nextafter(rho, side), 0.0, rho[-1])
            true = np.clip(np.searchsorted(rho, x, side="right") - 1, 0, n - 2)
            first = np.minimum((x * s).astype(np.int64), n - 2)
            assert ((first == true) | (first == true + 1)).all()


@pytest.mark.parametrize("by", [0.3, 0.9, 1e-3, -1e-9])
def test_displaced_load_points(rules, by):
    """Points displaced within their buckets, for which most loads (or many) would start at a point above them, keep the other forms."""
    rho = np.linspace(0.0, 0.95, 33)
    one = rho.copy()
    one[7] += by * rho[1]
    rho[1:-1] += by * rho[1]
    assert _even_scale(rules, rho) == 0.0 and _even_scale(rules, one) == 0.0


@pytest.mark.parametrize("n,by", [(33, 0.95), (64, 0.9), (128, 0.8), (64, 5e-4), (900, 0.5), (2000, 0.999)])
def test_displaced_load_points_of_the_even_form(rules, n, by):
    """Points late by little, or by any part of a step where the bucket index would be large; a load starts at its bracket or the one above."""
    rho = np.linspace(0.0, 0.95, n)
    rho[1:-1] += by * rho[1]
    s = _even_scale(rules, rho)
    assert s > 0.0 and ((rho * s).astype(np.int64) == np.arange(n)).all()
    load = np.clip(np.r_[np.random.default_rng(n).uniform(0.0, rho[-1], 100_000), rho, np.nextafter(rho, -np.inf), np.nextafter(rho, np.inf)], 0.0, rho[-1])
    true = np.clip(np.searchsorted(rho, load, side="right") - 1, 0, n - 2)
    first = np.minimum((load * s).astype(np.int64), n - 2)
    assert ((first == true) | (first == true + 1)).all()
    rho[1] -= (by + 1e-9) * rho[1] / (1 + by)              # one point early
    assert _even_scale(rules, rho, 4096) == 0.0


@pytest.mark.parametrize("tiles,tile,staged,waves,want", [(1_600_000, 256, 1536, 32, 7), (1_600_000, 256, 1536, 24, 9), (830_000, 192, 2304, 24, 9), (1_250_000, 128, 1536, 22, 10),
                                                          (2_500_000, 64, 768, 20, 11), (1_250_000, 64, 768, 10, 22), (1_600_000, 256, 1536, 0, 32), (60_000, 256, 3600, 32, 8),
                                                          (250_000, 256, 1536, 32, 4), (8192, 64, 700, 32, 1), (20_000, 256, 2048, 32, 3)])
def test_windows_a_block(rules, tiles, tile, staged, waves, want):
    """Resident waves times windows stay at about 224 where the device is full, whatever the width of the tiles; few tiles keep 8192 blocks."""
    assert rules.space_windows(C.c_longlong(tiles), tile, C.c_longlong(staged), waves) == want


@pytest.mark.parametrize("axis,lds,blocks,staged", [(1512, 10_000, 10_000, 1), (40 * 1024, 56 * 1024, 10_000, 1), (46 * 1024, 54 * 1024, 512, 1), (46 * 1024, 54 * 1024, 513, 0),
                                                    (72 * 1024, 80 * 1024, 512, 1), (72 * 1024, 80 * 1024, 513, 0), (152 * 1024, 168 * 1024, 1, 0)])
def test_where_the_frequency_kernel_keeps_a_long_axis(rules, axis, lds, blocks, staged):
    assert rules.freq_axis_staged(C.c_longlong(axis), C.c_longlong(lds), C.c_longlong(blocks), 256) == staged


@pytest.mark.parametrize("G", [1, 4, 9, 25, 47, 48, 100, 257, 4096])
def test_cut_of_the_frequency_kernel(rules, G):
    """Every cell in one block, a thread for every cell, the LDS that a block is given room for, and no block of a few lanes where windows could fill it."""
    for n_window, n_tick, n_f, axis in itertools.product((1, 60, 511, 2016, 20160), (1, 5, 12, 64, 65, 1000), (1, 12, 128, 129), (1512, 60_000, 150_000)):
        o = (C.c_longlong * 8)()
        rules.freq_shape(n_window, G, n_tick, n_f, C.c_longlong(axis), 256, o)
        wins, run, n_run, chunk, tabled, staged, blocks, lds = o
        assert wins >= 1 and run >= 1 and chunk == min(n_tick, 64) and tabled == (n_f <= 128)
        assert run * n_run >= G > run * (n_run - 1) and (wins == 1 or n_run == 1)
        assert blocks == -(-n_window // wins) * n_run
        cells = wins * run
        assert cells <= 256
        need = cells * (chunk * 12 + (16 * n_f if tabled else 0) + 20)
        assert lds == need + (axis if staged else 0) <= 160 * 1024 and need <= 16 * 1024
        assert G - run * (n_run - 1) > run - n_run                   # runs alike: the last lacks less than one class a run
        if n_run == 1 and blocks >= 2 * 256:                        # more blocks than places: they are half full, or as full as LDS lets them
            assert 2 * cells * chunk > 256 or 2 * need > 16 * 1024 - need // cells * G
        if n_window * -(-G // (256 // chunk)) <= 2 * 256:            # few: every look-up of a block in one round
            assert run * chunk <= 256


def test_few_classes_share_a_block(rules):
    for n_window, G, n_tick, wins in ((20160, 1, 12, 21), (2016, 1, 12, 7), (2016, 1, 1, 7), (60, 1, 12, 1), (10000, 4, 5, 12), (1440, 9, 12, 2), (1440, 25, 12, 1)):
        o = (C.c_longlong * 8)()
        rules.freq_shape(n_window, G, n_tick, 12, C.c_longlong(1512), 256, o)
        assert o[0] == wins, (n_window, G, n_tick)
