"""CPU checks of bench.py's counts of the kernels as they run now, each against its
closed form, and of the name it gives the autotuner's choice."""
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402
from paper_1808_00128_amd import binding as B  # noqa: E402


def test_pair_chain_step_bytes():
    """Two steps of a window of four, by launch: cached words read once, written by
    every second launch; the rows of two proposals and of 4 and 2 pending steps; the
    constants."""
    chi, chains = 1000, 64
    window = [8 * chains + 8 * chains + 17 * (2 + 4) + 33, 8 * chains + 17 * (2 + 2) + 33]
    assert bench.pair_chain_step_bytes(chi, chains) == chi * sum(window) / 4


def test_amp_fp4_ops_per_pair():
    assert bench.amp_fp4_ops_per_pair(1) == 128  # 2 features: one step
    assert bench.amp_fp4_ops_per_pair(10) == 128  # 56
    assert bench.amp_fp4_ops_per_pair(11) == 256  # 67
    assert bench.amp_fp4_ops_per_pair(50) == 128 * 20
    assert bench.amp_fp4_ops_per_pair(60) == 128 * 29


def test_record_step_bytes():
    assert bench.record_step_bytes(50, 1 << 18) == 8192 * 23 * 1024
    assert bench.record_step_bytes(10, 33) == 2 * 4 * 1024  # a partial tile is read whole


def test_tuned_name():
    default = B.TUNE_SHAPES.index(0x104)
    ms = [1.0] * len(B.TUNE_SHAPES)
    assert bench.tuned_name(B, 0x108, ms) == bench.shape_name(0x108)
    ms[0] = 0.5
    assert bench.tuned_name(B, 0x104, ms) == "default (mixed by span)"
    ms[default] = 0.4
    assert bench.tuned_name(B, 0x104, ms).startswith("default, or")
