"""Tiles of the moment step on lattices with solid cells (host code): every
row of every strip in exactly one tile, links only in tiles marked for them, and
no tile so tall that a few wavefronts march on alone: the tallest tile is at most
the rows that a SIMD marches on average, or queued ones' height."""
import ctypes
import os
import subprocess
import time

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2109_12565_amd", "csrc")
BELOW, ABOVE = 0b001100100, 0b110010000
SOURCE = r"""
#include "moment_tiles.hpp"
extern "C" int tiles(int lx, int ly, int strips, int strip, int rows, int fixed, long long slots,
                     long long simds, const uint16_t* link, int* out, int* nlinked) {
  const auto t = tlbk::moment_tiles({lx, ly, strips, strip, rows, fixed != 0, slots, simds, %d, %d},
                                    link, nlinked);
  for (size_t k = 0; k < t.size(); ++k) {
    const int v[4] = {t[k].strip, t[k].y0, t[k].y1, t[k].linked};
    for (int i = 0; i < 4; ++i) out[4 * k + i] = v[i];
  }
  return (int)t.size();
}
""" % (BELOW, ABOVE)
SIMDS = 1024


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("tiles")
    (d / "t.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O2", "-shared", "-fPIC", "-I", CSRC, str(d / "t.cpp"),
                    "-o", str(d / "t.so")], check=True)
    return ctypes.CDLL(str(d / "t.so"))


def links(solid):
    """Link masks as tlb_init forms them: bit 0 solid, bit i the source of direction i."""
    ly, lx = solid.shape
    wide = np.ones((ly + 2, lx), bool)
    wide[1:-1] = solid != 0
    m = (solid != 0).astype(np.uint16)
    cx, cy = (0, 1, 0, -1, 0, 1, -1, -1, 1), (0, 0, 1, 0, -1, 1, 1, -1, -1)
    for i in range(1, 9):
        m |= np.roll(wide, (cy[i], cx[i]), (0, 1))[1:-1].astype(np.uint16) << i
    return np.ascontiguousarray(m)


def tiles_of(lib, solid, slots=2 * SIMDS, fixed=0):
    ly, lx = solid.shape
    m = links(solid)
    strips = -(-lx // 58)
    strip = -(-lx // strips)
    rows = fixed or min(ly, -(-ly // max(1, slots // strips)))
    out = np.zeros((strips * ly, 4), np.int32)
    nl = ctypes.c_int()
    t0 = time.perf_counter()
    n = lib.tiles(lx, ly, strips, strip, rows, int(fixed > 0), ctypes.c_longlong(slots),
                  ctypes.c_longlong(SIMDS), ctypes.c_void_p(m.ctypes.data), ctypes.c_void_p(out.ctypes.data),
                  ctypes.byref(nl))
    dt = time.perf_counter() - t0
    t = out[:n]
    seen = np.zeros((strips, ly), int)
    flat = np.zeros(ly, np.uint16)
    flat[0] |= BELOW
    flat[-1] |= ABOVE
    for s, y0, y1, linked in t:
        assert y0 < y1
        seen[s, y0:y1] += 1
        if not linked:
            x0, x1 = s * strip, min((s + 1) * strip, lx)
            assert (m[y0:y1, x0:x1] == flat[y0:y1, None]).all()
    assert (seen == 1).all()
    assert (t[:nl.value, 3] == 1).all() and (t[nl.value:, 3] == 0).all()
    return t, rows, dt


def posts(lx, ly, upto, seed=5):
    rng = np.random.default_rng(seed)
    s = np.zeros((ly, lx), np.uint8)
    for y in range(4, min(ly - 12, upto), 32):
        for x in range(0, max(1, lx - 16), 32):
            dx, dy = rng.integers(0, 16, 2)
            s[y + dy % 12:y + dy % 12 + 8, x + dx:x + dx + 8] = 1
    return s


def discs(lx, ly):
    s = np.zeros((ly, lx), np.uint8)
    x, y = np.meshgrid(np.arange(lx), np.arange(ly))
    for k in range(12):
        s[(x - (k % 4 + .5) * lx / 4) ** 2 + (y - (k // 4 + .5) * ly / 3) ** 2 < (ly / 10) ** 2] = 1
    return s


def scattered(lx, ly):
    s = np.zeros((ly, lx), np.uint8)
    s[np.random.default_rng(1).random((ly, lx)) < 1 / 2000] = 1
    return s


def pillars(lx, ly):
    s = np.zeros((ly, lx), np.uint8)
    for x in range(0, lx - 8, 64):
        s[:ly // 3, x:x + 4] = 1
    return s


CASES = {
    "third": lambda: posts(2048, 1024, 341), "tenth": lambda: posts(4096, 2048, 204),
    "discs": lambda: discs(2048, 1024), "scattered": lambda: scattered(4096, 2048),
    "pillars": lambda: pillars(2048, 1024), "full": lambda: posts(1024, 512, 512),
    "all_solid": lambda: np.ones((40, 100), np.uint8), "small": lambda: posts(333, 129, 40),
    "one_column": lambda: (np.arange(90) % 17 == 3).astype(np.uint8)[:, None],
}


@pytest.mark.parametrize("slots", [SIMDS, 2 * SIMDS])
@pytest.mark.parametrize("name", sorted(CASES))
def test_tiles_cover_the_lattice_and_none_runs_on_alone(lib, name, slots):
    t, rows, _ = tiles_of(lib, CASES[name](), slots)
    height = t[:, 2] - t[:, 1]
    linked = t[:, 3] == 1
    share = (height.sum() + 3 * len(t)) * 2 / SIMDS    # a linked row costs up to two
    assert height[linked].max(initial=0) <= 8
    assert height[~linked].max(initial=0) <= max(rows, 24, share)


def test_bottom_posts_fit_in_one_wave(lib):
    """Posts along the bottom wall only: all tiles resident at once, a little
    taller than the flat lattice's chunks."""
    s = np.zeros((2048, 4096), np.uint8)
    for x in range(5, 4080, 40):
        s[:8, x:x + 8] = 1
    t, rows, _ = tiles_of(lib, s)
    assert rows == 74 and len(t) <= 2 * SIMDS
    assert (t[:, 2] - t[:, 1]).max() <= 80


@pytest.mark.parametrize("rows", [1, 7, 300])
def test_chosen_height_is_kept(lib, rows):
    t, _, _ = tiles_of(lib, posts(700, 600, 200), fixed=rows)
    plain = t[t[:, 3] == 0]
    assert (plain[:, 2] - plain[:, 1]).max() <= rows


def test_tall_lattice_is_cut_quickly(lib):
    """Five thousand short runs below a long one: one pass over the runs for each
    height tried, and few heights."""
    s = np.zeros((120000, 58), np.uint8)
    s[10:60000:12, 7] = 1
    t, _, dt = tiles_of(lib, s)
    assert (t[:, 2] - t[:, 1]).max() <= 64
    assert dt < 0.2
