"""The adjoint's two kernels: bricks of tets that form their blocks in LDS (131,072 tets and
more) and tets that gather for themselves give the same bits, so that a mesh has one adjoint,
alone or in a batch."""
import numpy as np
import pytest
import torch

from paper_2605_11673_amd import workloads as W

pytestmark = pytest.mark.gpu


def S():
    from paper_2605_11673_amd import stafem
    return stafem


def bits(t):
    return t.cpu().numpy().reshape(-1).view(np.uint64)


def test_batch_of_many_tets_equals_each_mesh_alone():
    """170,256 tets together, so the batch takes bricks; 162 to 105,456 alone, which gather."""
    Sm = S()
    ws = W.make_batch(seed=7, count=4, frames=2, sizes=[22, 5, 26, 3])
    b = Sm.Batch.from_workloads(ws)
    off = b.offsets()
    assert off["tet"][-1] >= 131072 and max(w.n_tets for w in ws) < 131072
    g = torch.from_numpy(np.random.default_rng(12).standard_normal(b.nnz)).cuda()
    gl, gx = b.adjoint(g)
    for j, w in enumerate(ws):
        a = Sm.Assembler.from_workload(w)
        sl, sx = a.adjoint(g[off["nnz"][j]:off["nnz"][j + 1]].clone())
        assert np.array_equal(bits(gl[off["tet"][j]:off["tet"][j + 1]]), bits(sl)), j
        assert np.array_equal(bits(gx.reshape(-1, 3)[off["node"][j]:off["node"][j + 1]]), bits(sx)), j
        a.close()
    b.close()
