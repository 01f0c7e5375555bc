"""The index rules of the packed hash table and of the 3D row sweep, compiled
for the host: every key starts inside its table, spread over it; a table has
room for its item's pairs; no tile holds more voxels than its size class was
taken from; the 13 forward neighbours have 13 classes, whatever the sign."""
from __future__ import annotations

import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def rules():
    lib = os.path.join(ROOT, "tests", "libpacked_rules.so")
    hipcc = "/opt/rocm/bin/hipcc" if os.path.exists("/opt/rocm/bin/hipcc") else "hipcc"
    tmp = lib + ".tmp%d" % os.getpid()
    subprocess.check_call([hipcc, "--offload-arch=gfx950", "-O2", "-std=c++17", "-fPIC", "-shared",
                           "-I" + os.path.join(ROOT, "paper_2603_12016_amd", "csrc"), "-o", tmp,
                           os.path.join(ROOT, "tests", "packed_rules.hip")])
    os.replace(tmp, lib)
    L = ctypes.CDLL(lib)
    for f in (L.packed_histogram, L.packed_slot_count, L.packed_voxel_count, L.packed_item_bound):
        f.restype = ctypes.c_uint32
    return L


@pytest.mark.parametrize("slots", [12, 100, 384, 1288, 5128, 20488])
def test_first_slot_in_range_and_spread(rules, slots):
    n = 1 << 24
    hist = np.zeros(slots, np.uint32)
    top = rules.packed_histogram(n, slots, hist.ctypes.data_as(ctypes.c_void_p))
    assert top < slots and int(hist.sum()) == n
    assert hist.min() > 0 and hist.max() <= 2 * n / slots + 300


def test_room_for_an_item(rules):
    big = 0xFFFFFFFF
    for nb in list(range(1, 600)) + [1023, 2047, 4095, 4096, 16383]:
        s = rules.packed_slot_count(nb, ctypes.c_uint32(big))
        assert s % 4 == 0 and s >= nb + nb // 2 + 8 and s < 1 << 15
        assert rules.packed_slot_count(nb, s - 4) == s - 4
        # the table sized for nb voxels takes nb, and no item whose slots it cuts short
        most = rules.packed_voxel_count(s)
        assert most >= nb and rules.packed_slot_count(most, ctypes.c_uint32(big)) <= s


@pytest.mark.parametrize("n,rows,width,split", [(5000, 50, 130, 4096), (100, 10, 10, 4096), (9000, 3, 4000, 1024),
                                                (70000, 700, 200, 4096), (4097, 65, 64, 4096), (20000, 20000, 1, 512)])
def test_bound_covers_every_tile(rules, n, rows, width, split):
    bound = rules.packed_item_bound(n, rows, width, split)
    if n <= split:
        assert bound == n
        return
    tiles = -(-n // split)
    rb = min(tiles, rows)
    cb = max(1, min(-(-tiles // rb), width))
    assert bound == min(n, -(-rows // rb) * -(-width // cb))


def test_neighbour_classes(rules):
    seen = {}
    for z in (-1, 0, 1):
        for y in (-1, 0, 1):
            for x in (-1, 0, 1):
                if (z, y, x) != (0, 0, 0):
                    seen.setdefault(rules.packed_class3d(z, y, x), []).append((z, y, x))
    assert sorted(seen) == list(range(13))
    assert all(tuple(-v for v in a) == b for a, b in seen.values())
