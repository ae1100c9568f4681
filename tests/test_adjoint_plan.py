"""Which chunks make a brick of the adjoint: no brick may set the LDS of all."""
import ctypes

import numpy as np
import pytest

from tests.hostcode import compiled

SOURCE = r"""
#include "adjoint_plan.h"
#include <cstring>
extern "C" int most() { return sta::kBrickMost; }
// order: room for cap bricks; returns the number of bricks, -1: nothing halved
extern "C" int halve(int32_t* order, const int32_t* blocks, int n, int cap)
{
    std::vector<int32_t> o(order, order + n * sta::kBrickChunks), b(blocks, blocks + n);
    const bool halved = sta::halve_large_bricks(o, b);
    const int m = (int)o.size() / sta::kBrickChunks;
    if (m > cap)
        return -2;
    std::memcpy(order, o.data(), sizeof(int32_t) * o.size());
    return halved ? m : -1;
}
"""


def plan(lib, chunks, blocks_of):
    """Bricks of 8 of the chunks in turn, halved until none is too large."""
    n = (len(chunks) + 7) // 8
    order = np.full(8 * len(chunks), -1, np.int32)
    order[:len(chunks)] = chunks
    for _ in range(8):
        bricks = order[:8 * n].reshape(n, 8)
        blocks = np.array([blocks_of(b[b >= 0]) for b in bricks], np.int32)
        p = ctypes.POINTER(ctypes.c_int32)
        m = lib.halve(order.ctypes.data_as(p), blocks.ctypes.data_as(p), n, len(chunks))
        assert m != -2
        if m == -1:
            return [list(b[b >= 0]) for b in bricks], blocks
        n = m
    raise AssertionError("does not end")


@pytest.mark.parametrize("n", [1, 7, 8, 9, 64, 8195])
@pytest.mark.parametrize("kind", ["ordered", "scattered", "tail"])
def test_bricks_leave_room_for_others(tmp_path, n, kind):
    lib = compiled(tmp_path, SOURCE)
    most = lib.most()
    ordinary = set(range(n)) if kind == "ordered" else set() if kind == "scattered" else set(range(n - n // 50))
    # a chunk in no order holds 160 different blocks; of ordered ones a brick holds 400
    bricks, blocks = plan(lib, np.arange(n), lambda b: sum(50 if c in ordinary else 160 for c in b))
    assert [c for b in bricks for c in b] == list(range(n))  # every chunk once, in the order given
    if kind == "ordered":
        assert len(bricks) == (n + 7) // 8
    if kind == "tail":
        assert max(blocks) <= most  # a few in no order don't set the LDS of the others
    assert max(blocks) <= 640  # three workgroups on a compute unit whatever the mesh
