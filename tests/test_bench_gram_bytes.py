"""Bytes of the Gram blocks that bench.py counts for one object: half of each
block only where the half-block kernel takes the product."""
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402


@pytest.mark.parametrize("nz,nclass,groups,half", [(128, 5924, 6293, True), (64, 90, 100, True), (50, 90, 100, True),
                                                   (128, 900, 1000, False), (100, 5924, 6293, False), (160, 5924, 6293, False)])
def test_gram_read_info(nz, nclass, groups, half):
    row = -(-nz // 4) * 4
    info = {"nclass": nclass, "slab_bytes_A": nclass * 1000, "read_bytes_A": groups * 1000, "gram_bytes": nclass * nz * row * 4}
    got = bench.gram_read_info(info, nz)["gram_bytes"]
    # tile rows of 16: the columns from 32 * (i // 2) on
    want = sum(1 for i in range(nz) for j in range(row) if j >= 32 * (i // 32)) * nclass * 4
    assert got == (want if half else info["gram_bytes"])
