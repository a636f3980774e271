"""Launch sizes that follow from a call's sizes (csrc/launch_rules.hpp), compiled and asked on the
CPU."""
from __future__ import annotations

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
KIB = 1024
ROUND = 512  # workgroups of 1,024 threads that 256 compute units hold at once


@pytest.fixture(scope="module")
def scatter_grid(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("rules") / "dump")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-fsanitize=undefined",
                    "-fno-sanitize-recover=all", "-I", os.path.join(ROOT, "paper_2607_22648_amd", "csrc"),
                    os.path.join(ROOT, "tests", "c", "launch_rules_dump.cpp"), "-o", exe], check=True)

    def ask(entries, units, size, rnd=ROUND):
        p = subprocess.run([exe], input=f"{rnd} {entries} {units} {size}\n", capture_output=True, text=True,
                           check=True)
        return int(p.stdout)

    return ask


def test_scatter_grid_follows_bytes_not_units(scatter_grid):
    """A block of 1,280 KiB is worth forty pieces of 32 KiB whether its units hold 32 KiB or 256."""
    assert scatter_grid(24 * 224, 5, 1280 * KIB) == 16 * ROUND
    assert scatter_grid(24 * 224, 40, 1280 * KIB) == 16 * ROUND
    # units smaller than 32 KiB still count each
    assert scatter_grid(24 * 224, 64, 64 * 4 * KIB) == 16 * ROUND


def test_scatter_grid_of_small_blocks_and_layer_ranges(scatter_grid):
    """Four rounds at least: one layer (two slabs of 32 KiB, or one unit of 64 KiB), a small
    model's block of 128 KiB, a small call of large blocks."""
    assert scatter_grid(7168, 2, 64 * KIB) == 4 * ROUND
    assert scatter_grid(7168, 1, 64 * KIB) == 4 * ROUND
    assert scatter_grid(28928, 4, 128 * KIB) == 4 * ROUND
    assert scatter_grid(64, 64, 2048 * KIB) == 4 * ROUND
    assert scatter_grid(256, 64, 2048 * KIB) == 8 * ROUND


def test_scatter_grid_limits(scatter_grid):
    """Never more workgroups than units, nor than 16 rounds; no overflow at the largest sizes (the
    sanitizer ends the program at one)."""
    assert scatter_grid(3, 4, 128 * KIB) == 12
    assert scatter_grid(0, 4, 128 * KIB) == 0
    assert scatter_grid(1, 1, 32) == 1
    for units, size in ((1, 16), (1 << 21, 1 << 51), (64, 2 << 20)):
        assert scatter_grid(1 << 29, units, size) <= 16 * ROUND
