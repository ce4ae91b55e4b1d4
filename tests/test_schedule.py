"""The rules that pick a clip's regression instance (esim_schedule.h, plain host
code): compiled here and called as they stand."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2303_02608_amd", "csrc")

SHIM = """
#include "esim_schedule.h"
extern "C" void route(int W, int H, int F, int r, int tr, double ridge, int cus, int* out) {
  const esim::ClipRoute c = esim::clip_route(W, H, F, r, tr, ridge, cus);
  out[0] = c.tile_lw, out[1] = c.tiles, out[2] = c.few, out[3] = c.kind;
}
extern "C" long long tiles(int W, int H, int lw) { return esim::tile_count(W, H, lw); }
extern "C" long long lds(int F, int r, int tr, int lw) {
  return static_cast<long long>(esim::tile_block_bytes(F, esim::tile_wave_units(F, r, tr, lw)));
}
extern "C" int member(int set, int tiles, int few, int kind) {
  esim::ClipRoute c{};
  c.tile_lw = 6, c.tiles = tiles != 0, c.few = few != 0, c.kind = kind;
  return esim::dense_member(set, c);
}
"""
LIMIT = 160 * 1024 - 64
CUS = 256


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("schedule")
    src, lib = d / "shim.cpp", d / "shim.so"
    src.write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, str(src), "-o",
                    str(lib)], check=True)
    so = ctypes.CDLL(str(lib))
    so.tiles.restype = so.lds.restype = ctypes.c_longlong

    class Rules:
        lds, tiles, member = so.lds, so.tiles, so.member

        @staticmethod
        def route(W, H, F, r, tr, ridge=1e-6):
            out = (ctypes.c_int * 4)()
            so.route(W, H, F, r, tr, ctypes.c_double(ridge), CUS, out)
            return dict(zip(("lw", "tiles", "few", "kind"), out))

    return Rules


def _fits(rules, F, r, tr, lw):
    return (1 << lw) + 2 * r <= 128 and rules.lds(F, r, tr, lw) <= LIMIT


@pytest.mark.parametrize("W,H,F,r,tr", [(752, 480, 7, 7, 2), (1000, 540, 7, 7, 2), (400, 300, 8, 5, 2),
                                        (752, 480, 8, 10, 1)])
def test_tiles_of_another_width(rules, W, H, F, r, tr):
    """Frames whose smallest cover does not fit LDS take the next one that does."""
    best = min((4, 5, 6), key=lambda lw: (rules.tiles(W, H, lw), -lw))
    assert not _fits(rules, F, r, tr, best)
    c = rules.route(W, H, F, r, tr)
    assert c["tiles"] and _fits(rules, F, r, tr, c["lw"])


def test_tiles_wherever_a_width_fits(rules):
    """Over sizes, features and windows: tiles exactly where a width fits, and of
    the widths that fit the one with the fewest tiles."""
    for W in (48, 64, 97, 320, 501, 752, 1280):
        for H in (40, 101, 720):
            for F in range(1, 13):
                for r in (1, 3, 5, 7, 8, 10, 16, 25, 33, 56, 57):
                    for tr in (0, 1, 2, 5):
                        c = rules.route(W, H, F, r, tr)
                        fit = [lw for lw in (4, 5, 6) if _fits(rules, F, r, tr, lw)]
                        assert c["tiles"] == bool(fit), (W, H, F, r, tr)
                        if fit:
                            assert c["lw"] in fit
                            assert rules.tiles(W, H, c["lw"]) == min(rules.tiles(W, H, lw) for lw in fit)


def test_dense_sets_cover_every_clip_once(rules):
    """The sets of each schedule (by hand 1 or 16 lanes, or automatic) hold every
    clip exactly once."""
    for tiles in (0, 1):
        for few in (0, 1):
            for kind in range(3):
                for sets in ((5, 6), (7, 8, 9), range(10, 15)):
                    assert sum(rules.member(s, tiles, few, kind) for s in sets) == 1
