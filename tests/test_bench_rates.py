"""bench.py's count of the bytes one V-cycle moves, for the kernels as launched (CPU)."""
import os
import re

import bench

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2006_16764_amd", "csrc")


def test_two_dimensional_cycles_have_no_count():
    # iterates, residuals and directions stay in LDS and registers there: a byte
    # count of a launch per operation says nothing about them
    assert bench.vcycle_moved(2, 512, 8) is None
    assert bench.vcycle_moved(2, 75, 4) is None


def test_what_tiled_levels_save():
    # 8^3 elements: 9^3 nodes, tiled (small); no prolongation sweep over them
    assert bench.vcycle_moved(3, 8, 4) == bench.vcycle_bytes(3, 8, 4) - 4 * 4 * 9 ** 3
    # FP64: and no copy of the right-hand side on the finest level
    assert bench.vcycle_moved(3, 8, 8) == bench.vcycle_bytes(3, 8, 8) - (4 + 2) * 8 * 9 ** 3
    # 56, 28, 14, 7: the level of 29^3 nodes is neither small nor a tile wide
    assert (bench.vcycle_moved(3, 56, 4)
            == bench.vcycle_bytes(3, 56, 4) - 4 * 4 * (57 ** 3 + 15 ** 3))
    # 28, 14, 7: an untiled finest level keeps its prolongation sweep and its copy
    assert bench.vcycle_moved(3, 28, 8) == bench.vcycle_bytes(3, 28, 8) - 4 * 8 * 15 ** 3
    # one level: split, coarse solve, merge
    assert bench.vcycle_moved(3, 7, 8) == bench.vcycle_bytes(3, 7, 8)


def test_the_rule_is_that_of_the_kernels():
    with open(os.path.join(CSRC, "pf_gmg.hip")) as f:
        src = f.read()
    assert f"constexpr long long kTiledSmall = {bench.TILED_SMALL};" in src
    side = re.search(r"#define PF_SBX (\d+)\n.*?#define PF_SBY (\d+)\n", src, re.S)
    assert (int(side.group(1)), int(side.group(2))) == bench.TILED_SIDES
