"""CPU test of the small calls' closed-form split (paper_2607_12696_amd/csrc/split.hpp), compiled for the host:
the ranges cover every unit once and are equal to within a unit; an item's first and last workgroup are those
whose ranges hold its first and last unit; each workgroup's pieces of cut items go to different slots; items are
cut only where whole items would leave workgroups idle for longer than the stated bytes."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CUT_BYTES = 48 << 10


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("small_split") / "lib.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC",
                    "-I" + os.path.join(ROOT, "paper_2607_12696_amd", "csrc"),
                    os.path.join(ROOT, "tests", "small_split_shim.cpp"), "-o", out], check=True)
    return C.CDLL(out)


# (experts, items per expert, rounds, bytes per item): the three layers' gate/up items, one expert on many
# workgroups, fewer items than workgroups, one item.
CASES = [(4, 180, 3, 49 << 10), (15, 180, 3, 49 << 10), (32, 128, 7, 229376), (9, 128, 7, 229376), (11, 96, 4, 262144),
         (1, 96, 4, 262144), (1, 2, 8, 1 << 20), (1, 1, 1, 4096), (1, 1, 8, 4 << 20), (3, 7, 5, 300000)]


@pytest.mark.parametrize("experts,tiles,rounds,nbytes", CASES)
@pytest.mark.parametrize("G", [256, 304, 64, 7])
def test_small_split(lib, experts, tiles, rounds, nbytes, G):
    items = experts * tiles
    first, w0, w1 = np.zeros(G + 1, np.uint32), np.zeros(items, np.uint32), np.zeros(items, np.uint32)
    per = lib.small_split_table(items, rounds, nbytes, G, first.ctypes.data_as(C.c_void_p), w0.ctypes.data_as(C.c_void_p),
                                w1.ctypes.data_as(C.c_void_p))
    idle = -items % G
    assert per == (rounds if rounds > 1 and idle * nbytes > G * CUT_BYTES else 1)
    units = items * per
    size = np.diff(first.astype(np.int64))
    assert first[0] == 0 and first[G] == units and size.min() >= units // G and size.max() <= -(-units // G)
    owner = np.repeat(np.arange(G), size)  # brute force: the workgroup of each unit
    assert np.array_equal(w0, owner[::per]) and np.array_equal(w1, owner[per - 1::per])
    pieces = set()
    for i in np.nonzero(w0 != w1)[0]:
        for w in sorted(set(owner[i * per:(i + 1) * per])):
            key = (w, lib.small_piece_slot(int(first[w]), int(i * per)))
            assert key not in pieces
            pieces.add(key)
