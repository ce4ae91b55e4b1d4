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
                        best = min((rules.tiles(W, H, lw) for lw in fit), default=0)
                        # (at least three fifths of the tiles' pixels in the image)
                        assert c["tiles"] == (bool(fit) and 5 * W * H >= 3 * 64 * best), (W, H, F, r, tr)
                        if c["tiles"]:
                            assert c["lw"] in fit and rules.tiles(W, H, c["lw"]) == best


def test_dense_sets_cover_every_clip_once(rules):
    """The sets of each schedule (by hand 1 or 16 lanes, or automatic) hold every
    clip exactly once."""
    for tiles in (0, 1):
        for few in (0, 1):
            for kind in range(3):
                for sets in ((5, 6), (7, 8, 9), range(10, 15)):
                    assert sum(rules.member(s, tiles, few, kind) for s in sets) == 1


# Dense regressions on a device of 256 CUs, us: (W, H, F, r, tr), 16 lanes per item, tiles.
MEASURED = [
    ((96, 96, 3, 1, 0), 9, 8), ((128, 128, 7, 1, 0), 15, 11), ((96, 96, 7, 2, 1), 16, 22),
    ((192, 192, 7, 2, 1), 40, 26), ((96, 96, 1, 3, 0), 9, 10), ((192, 192, 3, 3, 0), 22, 15),
    ((256, 240, 7, 3, 0), 48, 22), ((128, 128, 7, 3, 1), 27, 37), ((224, 224, 7, 3, 1), 62, 37),
    ((96, 96, 10, 3, 0), 22, 29), ((192, 192, 10, 3, 0), 60, 30), ((240, 256, 10, 3, 2), 203, 91),
    ((128, 128, 7, 4, 1), 31, 54), ((224, 224, 7, 4, 1), 89, 54), ((128, 128, 3, 5, 1), 24, 41),
    ((240, 256, 3, 5, 1), 66, 41), ((160, 160, 7, 5, 0), 29, 38), ((240, 256, 7, 5, 2), 197, 116),
    ((96, 96, 10, 5, 1), 47, 110), ((224, 224, 10, 5, 1), 193, 115), ((160, 160, 7, 6, 1), 64, 99),
    ((256, 300, 7, 6, 0), 84, 80), ((96, 96, 7, 7, 1), 33, 125), ((192, 192, 7, 7, 1), 105, 136),
    ((256, 300, 7, 7, 1), 189, 237), ((128, 128, 10, 7, 1), 78, 193), ((224, 224, 8, 8, 1), 204, 199),
    ((160, 160, 10, 8, 0), 102, 109), ((240, 256, 10, 8, 0), 211, 113), ((192, 192, 12, 7, 1), 264, 452),
    ((240, 256, 12, 3, 0), 115, 49), ((128, 128, 12, 12, 0), 165, 399),
]


@pytest.mark.parametrize("shape,lanes16,tiles", MEASURED)
def test_small_frames_take_the_faster_instance(rules, shape, lanes16, tiles):
    """To within 40 % where the two are close: the rule knows the window's radius and
    the frame's size, not the rest."""
    W, H, F, r, tr = shape
    c = rules.route(W, H, F, r, tr)
    assert c["tiles"]
    assert (lanes16 if c["few"] else tiles) <= 1.4 * min(lanes16, tiles)


@pytest.mark.parametrize("W,H,tiles", [(4, 32768, 0), (8, 16384, 0), (16, 8192, 1), (20, 8192, 1), (33, 8192, 1),
                                       (64, 2048, 1)])
def test_narrow_images_read_from_memory(rules, W, H, tiles):
    assert rules.route(W, H, 7, 7, 1)["tiles"] == tiles
