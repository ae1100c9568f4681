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


def check_against_oracle(w):
    import oracle
    from tests.bounds import adjoint_tolerances
    Sm = S()
    pat = oracle.pattern(w.n_nodes, w.tets)
    asm = Sm.Assembler.from_workload(w)
    g = np.random.default_rng(6).standard_normal(asm.nnz)
    gl, gx = (t.cpu().numpy() for t in asm.adjoint(torch.from_numpy(g).cuda()))
    ol, ox = oracle.adjoint(w.x, w.tets, w.E, w.nu, w.rho, w.dt, w.mask0, *pat, g)
    tl, tx = adjoint_tolerances(w, w.mask0, pat[0], pat[1], g)
    assert np.all(np.abs(gl - ol) <= tl) and np.all(np.abs(gx - ox) <= tx)
    assert np.all(gl[w.mask0 == 0] == 0.0)
    asm.close()


def reordered(w, perm, mask):
    return W.Workload("reordered", w.x, w.tets[perm], w.E[perm], mask, meta=w.meta)


def with_parts(w, parts):
    """The mesh and parts (x, tets) beside it."""
    x, tets = [w.x], [w.tets]
    for px, pt in parts:
        tets.append(pt + sum(len(v) for v in x))
        x.append(px)
    x, tets = np.concatenate(x), np.concatenate(tets).astype(np.int32)
    g = np.random.default_rng(len(tets))
    return W.Workload("parts", x, tets, W.lognormal_E(len(tets), g), g.integers(0, 2, size=len(tets)).astype(np.uint8),
                      meta=w.meta)


def apart(m):
    """m tets that share no vertex."""
    g = np.random.default_rng(m)
    corner = np.array([[0, 0, 0], [1, 0, 0], [0, 1, 0], [0, 0, 1.0]]) * 0.02
    x = g.uniform(size=(m, 1, 3)) + corner + g.uniform(-0.002, 0.002, size=(m, 4, 3))
    return x.reshape(-1, 3), np.arange(4 * m).reshape(m, 4)


def hub(k):
    """k tets around one vertex."""
    a = 2 * np.pi * np.arange(k) / k
    ring = np.stack([np.cos(a), np.sin(a), 0 * a], -1)
    x = np.concatenate([[[0, 0, 0.7]], ring, 0.5 * ring + [0, 0, 0.1]])
    i = np.arange(k)
    return x, np.stack([0 * i, 1 + i, 1 + (i + 1) % k, 1 + k + i], -1)


def full_bricks():
    """Ids in no order: 1,280 different blocks in 128 tets, 640 in the halves that bricks are."""
    w = W.make_fracture(0, 28, counts=[5])
    g = np.random.default_rng(1)
    return reordered(w, g.permutation(w.n_tets), np.ones(w.n_tets, np.uint8))


def some_full_bricks():
    """2,100 tets that share nothing, whose bricks are halved twice, and a hub over several bricks, beside a mesh in
    order; the last brick is short."""
    return with_parts(W.make_fracture(0, 28, counts=[5]), [apart(2100), hub(500)])


def few_active():
    """Of each brick 0 to 128 tets active, so on both sides of the count from which blocks are formed."""
    w = W.make_fracture(0, 28, counts=[5])
    g = np.random.default_rng(2)
    part = np.repeat(g.uniform(size=w.n_tets // 64 + 1), 64)[:w.n_tets]
    return reordered(w, np.arange(w.n_tets), (g.uniform(size=w.n_tets) < part).astype(np.uint8))


@pytest.mark.parametrize("mesh", [full_bricks, some_full_bricks, few_active])
def test_bricks(mesh):
    check_against_oracle(mesh())
