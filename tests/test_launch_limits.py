"""CPU-only checks of the host rules about launch grids (plain C++ constants): which tensors and calls share a launch."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_09825_amd", "csrc")


def holds(condition):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    src = '#include "launch_limits.h"\nusing namespace mxfp4;\nconstexpr int64_t ONE = 1;\nstatic_assert(%s, "");\n' % condition
    return subprocess.run([cxx, "-std=c++17", "-fsyntax-only", "-I", CSRC, "-x", "c++", "-"], input=src, text=True,
                          capture_output=True).returncode == 0


@pytest.mark.parametrize("condition", [
    # fewer than 2^32 threads along a dimension
    "grid_fits((ONE << 24) - 1, 256) && !grid_fits(ONE << 24, 256)",
    "grid_fits((ONE << 23) - 1, 512) && !grid_fits(ONE << 23, 512)",
    # workgroups of the quantisers: one block, a last workgroup of one block, one column more than a tile
    "rows_groups(1, 32) == 1 && rows_groups(257, 32) == 2 && rows_groups(8, 96) == 1",
    "cols_groups(32, 2) == 1 && cols_groups(256, 128) == 1 && cols_groups(288, 130) == 4",
    # dY and X of the weight gradient alone: together while one grid holds both
    "wgrad_operands_share_launch(32, 8, 8) && wgrad_operands_share_launch(16384, 4096, 4096)",
    "wgrad_operands_share_launch((ONE << 30) - 256, 8, 8) && !wgrad_operands_share_launch(ONE << 30, 8, 8)",
    "!wgrad_operands_share_launch(ONE << 31, 8, 8) && !wgrad_operands_share_launch(32, ONE << 40, 8)",
    # ... and while both are stored alike: one of them beyond the last-level cache
    "!wgrad_operands_share_launch(4096, 64, 32896) && wgrad_operands_share_launch(4096, 32776, 32896)",
    # waves of the column-wise workgroups (stochastic, rotated, regions, both axes, tiles, some beyond the last-level cache, all): stochastic four;
    # one axis eight from 512 tiles on; both axes eight from 1536 on, unless rotated; beyond the cache eight, rotated regions only if all are
    "cols_waves({true, false, false, true, 9999, true, true}) == 4 && cols_waves({false, true, true, true, 9999, true, true}) == 8",
    "cols_waves({false, true, false, false, 511, false, false}) == 4 && cols_waves({false, true, false, false, 512, false, false}) == 8",
    "cols_waves({false, false, true, false, 511, false, false}) == 4 && cols_waves({false, false, true, false, 512, false, false}) == 8",
    "cols_waves({false, false, false, true, 1535, false, false}) == 4 && cols_waves({false, false, false, true, 1536, false, false}) == 8",
    "cols_waves({false, false, true, true, 1535, false, false}) == 4 && cols_waves({false, false, true, true, 1536, false, false}) == 8",
    "cols_waves({false, true, false, true, 4096, false, false}) == 4 && cols_waves({false, true, true, true, 4096, false, false}) == 4",
    "cols_waves({false, true, false, true, 4096, true, false}) == 8 && cols_waves({false, true, true, true, 4096, true, false}) == 4",
    "cols_waves({false, false, true, true, 300, true, false}) == 8 && cols_waves({false, true, true, false, 4096, true, false}) == 4",
    # dY, W and X of a backward call (stochastic, rotated): together while W and X are fewer than 512 tiles, unless rounding is stochastic
    "cols_groups(18432, 896) + cols_groups(256, 896) == 511 && cols_groups(16128, 1024) + cols_groups(256, 1024) == 512",
    "backward_operands_share_launch(256, 18432, 896, false, false) && backward_operands_share_launch(256, 18432, 896, false, true)",
    "!backward_operands_share_launch(256, 16128, 1024, false, false) && !backward_operands_share_launch(256, 16128, 1024, false, true)",
    "backward_operands_share_launch(256, 16128, 1024, true, false) && backward_operands_share_launch(256, 16128, 1024, true, true)",
    # ... while dY is fewer than 1536 tiles, unless rotated
    "cols_groups(78592, 640) == 1535 && cols_groups(65536, 768) == 1536",
    "backward_operands_share_launch(78592, 640, 128, false, false) && !backward_operands_share_launch(65536, 768, 128, false, false)",
    "backward_operands_share_launch(65536, 768, 128, false, true) && backward_operands_share_launch(65536, 768, 128, true, false)",
    # ... and while each of the three is within the last-level cache
    "backward_operands_share_launch(16384, 8192, 8192, true, false)",
    "!backward_operands_share_launch(16384, 8224, 32, true, true) && !backward_operands_share_launch(32, 16384, 8224, true, true)",
    "!backward_operands_share_launch(16384, 32, 8224, true, true) && !backward_operands_share_launch(ONE << 31, 32, 32, true, true)",
    # a forward call in one launch (stochastic): 256 tiles of 32 x 32, rows of 16 blocks, or of 8
    "small_linear(1, 1, 32, false) && small_linear(512, 512, 512, false) && !small_linear(513, 512, 512, false) && !small_linear(512, 513, 32, true)",
    "small_linear(32, 32 * 256, 512, false) && !small_linear(32, 32 * 257, 64, false) && !small_linear(ONE << 40, ONE << 40, 32, false)",
    "!small_linear(1, 1, 544, false) && small_linear(1, 1, 256, true) && !small_linear(1, 1, 288, true)",
])
def test_rule(condition):
    assert holds(condition) and not holds("!(%s)" % condition)
