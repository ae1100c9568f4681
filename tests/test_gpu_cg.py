"""The linear solve where its kernels' shapes change: nodes with more neighbours than a
lane group holds at once, row counts around the workgroup's 16 nodes and one far below,
iteration limits around the host's chunks of launches, and converged solves.

Bound.  A solve that stops at relative (recurrence) residual rtol has a true residual of
at most rtol |b| plus the gap between the two, a rounding of a few u per iteration of
the recurrences r -= alpha q and x += alpha p, each bounded by u (|A| |x| + |b|) times a
small constant (8 is used, per iteration, with u = 2^-53)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_11673_amd import workloads as W
from tests.test_gpu_geometry import hub_mesh

pytestmark = pytest.mark.gpu
U = 2.0 ** -53


def S():
    from paper_2605_11673_amd import stafem
    return stafem


def single_tet():
    w = W.make_cube(0, n=1)
    return W.Workload("tet", w.x, w.tets[:1], w.E[:1], np.ones(1, np.uint8))


MESHES = {"tet": single_tet, "cube1": lambda: W.make_cube(0, n=1, frames=0), "cube2": lambda: W.make_cube(1, n=2, frames=2),
          "fracture7": lambda: W.make_fracture(seed=2, n=7, counts=[60, 90]),
          "refine3": lambda: W.make_refinement(seed=3, n=3, frames=2), "hub2": lambda: hub_mesh(2),
          "hub9": lambda: hub_mesh(9)}


def true_residual(pat, vals, x, b):
    rows = np.repeat(np.arange(len(pat[0]) - 1), np.diff(pat[0]))
    prod = vals.astype(np.longdouble) * x.astype(np.longdouble)[pat[1]]
    Ax, aAx = np.zeros(len(b), np.longdouble), np.zeros(len(b), np.longdouble)
    np.add.at(Ax, rows, prod)
    np.add.at(aAx, rows, np.abs(prod))
    return float(np.linalg.norm((b - Ax).astype(np.float64))), float(np.linalg.norm(aAx.astype(np.float64)))


@pytest.mark.parametrize("name", sorted(MESHES))
def test_solution_and_limits(name):
    Sm = S()
    w = MESHES[name]()
    pat = oracle.pattern(w.n_nodes, w.tets)
    asm = Sm.Assembler.from_workload(w)
    for ids, st in w.frames:
        asm.apply_edits(*Sm.upload_frame(ids, st))
    vals = asm.values()
    b = np.random.default_rng(4).standard_normal(asm.n_rows)
    bd = torch.from_numpy(b).cuda()
    v = vals.cpu().numpy()
    live = np.array([v[s:e][pat[1][s:e] == r].sum() != 0 if e > s else False
                     for r, (s, e) in enumerate(zip(pat[0][:-1], pat[0][1:]))])
    x, it, rr = asm.cg_solve(bd, rtol=1e-12)
    y, it2, rr2 = asm.cg_solve(bd, vals * 1.0, rtol=1e-12)  # given values: same bits
    assert it == it2 and rr == rr2 and torch.equal(x, y)
    xh = x.cpu().numpy()
    assert rr <= 1e-12 and np.all(xh[~live] == 0.0)
    bl = np.where(live, b, 0.0)
    res, size = true_residual(pat, v, xh, bl)
    nb = np.linalg.norm(bl)
    print(f"[cg] {name}: {asm.n_rows} rows, {it} iterations, true residual {res / nb:.2e}", flush=True)
    assert res <= 1e-12 * nb + 8 * U * max(it, 1) * (size + nb), (res / nb, it)
    for k in (0, 1, 15, 16, 17, 31, 48, 49):  # stops exactly at the limit, or where the free solve stopped
        xk, itk, rk = asm.cg_solve(bd, rtol=1e-12, max_iter=k)
        assert itk == min(k, it), (k, itk, it)
        assert itk < it or torch.equal(xk, x)
    assert asm.cg_solve(torch.zeros_like(bd))[1] == 0
    asm.close()


def bar(layers, stiff):
    """Stiff cells in a row, with their moduli far apart: 1,760 iterations at 70 layers and 1e9."""
    x1, t1 = W.grid_nodes(1), W.kuhn_tets(1)
    x = np.concatenate([x1[:4] + [i, 0, 0] if x1[3, 0] == 0 else x1[:4] + [0, 0, i] for i in range(layers + 1)])
    tets = np.concatenate([t1 + 4 * i for i in range(layers)]).astype(np.int32)
    E = stiff * 10.0 ** np.random.default_rng(layers).uniform(-2, 2, size=len(tets))
    return W.Workload("bar", x, tets, E, np.ones(len(tets), np.uint8))


def padded(nodes):
    """The largest fracture mesh of at most this many nodes, its nodes scattered among unused ones."""
    n = int(round(nodes ** (1 / 3) + 0.5))
    while (n + 1) ** 3 > nodes:
        n -= 1
    w = W.make_fracture(seed=8, n=n, counts=[1])
    g = np.random.default_rng(nodes)
    at = g.permutation(nodes)[:w.n_nodes]
    x = g.uniform(size=(nodes, 3))
    x[at] = w.x
    return W.Workload("padded", x, at[w.tets].astype(np.int32), w.E, w.mask0)


@pytest.mark.parametrize("nodes", [8, 32, 33, 256, 257, 288, 289, 343, 352, 353])
def test_small_systems(nodes):
    """Node counts where a small system's rounds, its blocks in LDS and the one launch itself
    begin and end, with unused nodes between the others."""
    Sm = S()
    w = padded(nodes)
    pat = oracle.pattern(w.n_nodes, w.tets)
    asm = Sm.Assembler.from_workload(w)
    vals = asm.values()
    v = vals.cpu().numpy()
    g = np.random.default_rng(3)
    live = np.diff(pat[0]) > 0
    b = g.standard_normal(asm.n_rows)
    x, it, rr = asm.cg_solve(torch.from_numpy(b).cuda(), rtol=1e-12)
    bl = np.where(live, b, 0.0)
    res, size = true_residual(pat, v, x.cpu().numpy(), bl)
    nb = np.linalg.norm(bl)
    assert rr <= 1e-12 and np.all(x.cpu().numpy()[~live] == 0.0)
    assert res <= 1e-12 * nb + 8 * U * it * (size + nb), (res / nb, it)
    for k in (0, 1, it - 1, it, it + 1):
        xk, itk, rk = asm.cg_solve(torch.from_numpy(b).cuda(), rtol=1e-12, max_iter=k)
        assert itk == min(k, it) and (itk < it or torch.equal(xk, x))
    asm.close()


def test_small_system_long_solve():
    """More iterations than one launch takes: the solve goes on where it stopped, and ends at the
    limit or at the tolerance as a shorter one does."""
    Sm = S()
    w = bar(70, 1e9)
    pat = oracle.pattern(w.n_nodes, w.tets)
    asm = Sm.Assembler.from_workload(w)
    vals = asm.values()
    b = np.random.default_rng(5).standard_normal(asm.n_rows)
    bl = np.where(np.diff(pat[0]) > 0, b, 0.0)
    nb = np.linalg.norm(bl)
    free = asm.cg_solve(torch.from_numpy(b).cuda(), rtol=1e-12)[1]
    assert free > 1100
    for k in (1023, 1024, 1025, 1100):
        x, it, rr = asm.cg_solve(torch.from_numpy(b).cuda(), rtol=1e-12, max_iter=k)
        res, size = true_residual(pat, vals.cpu().numpy(), x.cpu().numpy(), bl)
        assert it == k and abs(res - rr * nb) <= 8 * U * it * (size + nb), (k, it, res / nb, rr)
    asm.close()
