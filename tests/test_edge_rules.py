"""CPU-only checks of the rules (plain C++ arithmetic) by which products on the ragged-shape kernel's tiles run as its kernels for few outputs and
for short rows."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_09825_amd", "csrc")
PRELUDE = """#include "edge_rules.h"
using namespace mxfp4;
// an output of t tiles of 32 x 32, or of 128 x 64, with rows of n bytes of codes
constexpr EdgeProduct few(int64_t t, int64_t n, bool e4m3 = false) { return {32 * t, 30, n, 60, e4m3, false, false}; }
constexpr bool on32(EdgeProduct p) { return small_tiles(p, nullptr) != 0; }
constexpr bool on32(EdgeProduct p, EdgeProduct q) { return small_tiles(p, &q) != 0; }
constexpr EdgeProduct shorts(int64_t t, int64_t n, int64_t pitch, bool fp32 = false, bool acc = false) { return {128 * t, 60, n, pitch, false, fp32, acc}; }
constexpr bool shrt(EdgeProduct p) { return runs_short(p, nullptr); }
constexpr bool shrt(EdgeProduct p, EdgeProduct q) { return runs_short(p, &q); }
static_assert(%s, "");
"""


def holds(condition):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    return subprocess.run([cxx, "-std=c++17", "-fsyntax-only", "-I", CSRC, "-x", "c++", "-"], input=PRELUDE % condition, text=True,
                          capture_output=True).returncode == 0


@pytest.mark.parametrize("condition", [
    # 32 x 32 tiles, whole stages: one up to 256 tiles, two up to 512
    "small_tiles(few(256, 128), nullptr) == 256 && !on32(few(257, 128)) && on32(few(512, 256)) && !on32(few(513, 256)) && !on32(few(513, 7168))",
    # a ragged last stage: MXFP4 from two stages on, from five beyond 256 tiles; MXFP8 from three, from eight
    "!on32(few(1, 16)) && !on32(few(256, 112)) && on32(few(1, 144)) && on32(few(256, 240))",
    "!on32(few(257, 496)) && on32(few(257, 528)) && on32(few(512, 624))",
    "!on32(few(1, 96, true)) && !on32(few(256, 224, true)) && on32(few(256, 288, true)) && on32(few(257, 256, true))",
    "!on32(few(257, 864, true)) && on32(few(257, 928, true)) && on32(few(512, 992, true))",
    # pairs: the tiles of both, and each of them long enough
    "on32(few(100, 128), few(156, 128)) && !on32(few(100, 128), few(157, 128)) && !on32(few(100, 128), few(1, 112)) && on32(few(256, 256), few(256, 528))",
    # short rows: up to two stages, rows of the output in no whole cache lines or more than 4096 tiles
    "shrt(shorts(600, 256, 120)) && !shrt(shorts(600, 272, 120)) && !shrt(shorts(4096, 256, 128)) && shrt(shorts(4097, 256, 128))",
    "shrt(shorts(600, 16, 120), shorts(1, 256, 120)) && !shrt(shorts(600, 16, 120), shorts(1, 256, 128)) && !shrt(shorts(600, 16, 120), shorts(1, 272, 120))",
    # ... of fp32 products alone not those with two stages and a last round that is nearly empty, nor few tiles that are added to
    "shrt(shorts(768, 256, 144, true)) && !shrt(shorts(769, 256, 144, true)) && !shrt(shorts(1024, 144, 144, true)) && shrt(shorts(1025, 256, 144, true))",
    "shrt(shorts(800, 128, 144, true)) && shrt(shorts(800, 256, 120, true)) && !shrt(shorts(800, 256, 120, true, true)) && shrt(shorts(800, 256, 144))",
    "!shrt(shorts(512, 128, 144, true, true)) && shrt(shorts(513, 128, 144, true, true)) && shrt(shorts(300, 128, 144, true))",
    "shrt(shorts(800, 256, 144), shorts(10, 256, 144, true, true))",
])
def test_rule(condition):
    assert holds(condition) and not holds("!(%s)" % condition)
