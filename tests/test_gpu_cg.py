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
