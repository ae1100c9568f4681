"""The rebuild's tiles of rows where a node is at their limits: 128 row blocks, 192 tets and 576
terms of a node fit in a tile, one more of any does not.  Values bitwise against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_11673_amd import workloads as W

pytestmark = pytest.mark.gpu


def apart(k):
    """k tets that share one vertex and nothing else: 3 k + 1 row blocks, k tets, 3 k terms."""
    g = np.random.default_rng(k)
    x = np.concatenate([[[0.5, 0.5, 0.5]], g.uniform(size=(3 * k, 3))])
    return x, np.concatenate([np.zeros((k, 1), int), 1 + np.arange(3 * k).reshape(k, 3)], 1)


def around(k):
    """k tets of one vertex over a ring of 16: 18 row blocks, k tets, 3 k terms."""
    a = 2 * np.pi * np.arange(16) / 16
    x = np.concatenate([[[0, 0, 0.7]], np.stack([np.cos(a), np.sin(a), 0 * a], -1), [[0.1, 0.0, -0.5]]])
    i = np.arange(k)
    return x, np.stack([0 * i, 1 + i % 16, 1 + (i + 1) % 16, 17 + 0 * i], -1)


@pytest.mark.parametrize("part", [lambda: apart(42), lambda: apart(43), lambda: apart(64), lambda: around(191),
                                  lambda: around(192), lambda: around(193), lambda: around(400)])
def test_a_node_at_the_limits_of_a_tile(part):
    """Beside an ordinary mesh, with some tets of the node off, in rebuilds and frames."""
    from paper_2605_11673_amd import stafem as Sm
    c = W.make_fracture(seed=1, n=3, counts=[3])
    x, tets = part()
    x, tets = np.concatenate([c.x, x + 3.0]), np.concatenate([c.tets, tets + c.n_nodes]).astype(np.int32)
    g = np.random.default_rng(len(tets))
    w = W.Workload("tile", x, tets, W.lognormal_E(len(tets), g), g.integers(0, 2, size=len(tets)).astype(np.uint8))
    pat = oracle.pattern(w.n_nodes, w.tets)
    asm = Sm.Assembler.from_workload(w)
    mask = w.mask0.copy()

    def check(what):
        got = asm.values().cpu().numpy()
        assert np.array_equal(got.view(np.uint64), oracle.rebuild_workload(w, mask, pat).view(np.uint64)), what

    check("build")
    for k in (1, 20, w.n_tets // 2):
        ids = g.permutation(w.n_tets)[:k].astype(np.int32)
        asm.apply_edits(*Sm.upload_frame(ids, 1 - mask[ids]))
        mask[ids] = 1 - mask[ids]
        check(f"{k} edits")
    asm.set_config(rebuild_nt=1)
    asm.full_rebuild()
    check("rebuild")
    assert asm.audit() == {"values_differing": 0, "tets_differing": 0} and asm.status_sync() == Sm.STA_OK
    asm.close()
