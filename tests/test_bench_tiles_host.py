"""Host checks of bench.py's accounting of time steps by tiles (no GPU), against counts
written out by hand from the tile kernel's reads and writes."""
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402

N = 33554432                    # graphene 4096 x 4096


def test_two_launches_with_a_table():
    info = {"format": 3, "ell_w": 4, "table_used": True, "table_diag": 2}
    # row number, one column word, one selector word, the diagonal's real part; launch 1: x read, out,
    # xout, yout written; launch 2: x, y, out, psi0 read, out written
    assert bench.tile_bytes_per_step(info, N, 1, "c128", 19, 10, True) == (N * (2 * (4 + 8 + 4 + 8) + 9 * 16), 2)


def test_one_launch_and_blocks_without_a_table():
    info = {"format": 1, "ell_w": 3, "table_used": False}
    assert bench.tile_bytes_per_step(info, 8192, 1, "c128", 19, 19, True) == (8192 * (16 + 3 * 8 + 3 * 16), 1)
    info["ell_w"] = 5           # two words
    assert bench.tile_bytes_per_step(info, 1000, 4, "c64", 19, 5, False) == (4000 * (4 * (28 + 5 * 8) + 21 * 8), 4)


def test_three_launches():
    info = {"format": 3, "ell_w": 8, "table_used": True, "table_diag": 0}
    assert bench.tile_bytes_per_step(info, 1000, 1, "c64", 19, 7, True) == (1000 * (3 * 28 + 15 * 8), 3)
