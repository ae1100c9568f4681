"""Meshes with vertices and edges of very many tets: the state is the oracle's, and a frame
does not take a time that grows with the square of what is around it."""
import time

import numpy as np
import pytest
import torch

from paper_2605_11673_amd import workloads as W

pytestmark = pytest.mark.gpu


def S():
    from paper_2605_11673_amd import stafem
    return stafem


def cone(n):
    """2 n^2 tets from the triangles of a square to one apex."""
    i, j = np.meshgrid(np.arange(n + 1), np.arange(n + 1), indexing="ij")
    x = np.concatenate([np.stack([0 * i, i / n, j / n], -1).reshape(-1, 3), [[1.0, 0.4, 0.6]]])
    ids = np.arange((n + 1) ** 2).reshape(n + 1, n + 1)
    tri = np.concatenate([np.stack([ids[:-1, :-1], ids[1:, :-1], ids[1:, 1:]], -1).reshape(-1, 3),
                          np.stack([ids[:-1, :-1], ids[:-1, 1:], ids[1:, 1:]], -1).reshape(-1, 3)])
    tets = np.concatenate([np.full((len(tri), 1), (n + 1) ** 2), tri], 1).astype(np.int32)
    return W.Workload("cone", x, tets, W.lognormal_E(len(tets), np.random.default_rng(n)),
                      np.ones(len(tets), np.uint8))


def seconds(f, reps=5):
    best = np.inf
    for _ in range(reps):
        torch.cuda.synchronize()
        t = time.perf_counter()
        f()
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t)
    return best


@pytest.mark.parametrize("n", [4, 7, 8, 50])
def test_proxy_frames_at_an_apex(n):
    """32 and 98 tets (one launch), 128 and 5,000 (two launches; in one, 7 and 13 ms a frame at 5,000)."""
    from oracle import proxy as P
    Sm = S()
    w = cone(n)
    pat = P.proxy_pattern(w.n_nodes, w.tets)
    px = Sm.Proxy.from_workload(w, W.PROXY_EPS)
    g = np.random.default_rng(n)
    mask = w.mask0.copy()
    for k in (1, 30, min(2304, w.n_tets)):
        ids = g.permutation(w.n_tets)[:k].astype(np.int32)
        frames = [Sm.upload_frame(ids, 1 - mask[ids]), Sm.upload_frame(ids, mask[ids])]
        px.apply_edits(*frames[0])
        mask[ids] = 1 - mask[ids]
        v, c, d = (t.cpu().numpy() for t in px.state())
        ov, oc, od = P.proxy_rebuild(w.n_nodes, w.tets, mask, W.PROXY_EPS, pat)
        assert np.array_equal(c, oc) and np.array_equal(d, od) and np.array_equal(v.view(np.uint64), ov.view(np.uint64))
        assert seconds(lambda: [px.apply_edits(*f) for f in (frames[1], frames[0])]) < 2e-3, k
    assert px.status_sync() == Sm.STA_OK
    px.close()


@pytest.mark.parametrize("n,m", [(40, 1000), (100, 400), (100, 2000), (350, 10000)])
def test_small_solves_with_many_neighbours(n, m):
    """Solved by one workgroup (the first two) and by launches: residuals within the bound of
    tests/test_gpu_cg.py."""
    import oracle
    from tests.test_gpu_cg import U, true_residual
    Sm = S()
    g = np.random.default_rng(n + m)
    tets = np.argsort(g.uniform(size=(m, n)), axis=1)[:, :4].astype(np.int32)
    w = W.Workload("dense", g.uniform(size=(n, 3)), tets, W.lognormal_E(m, g), np.ones(m, np.uint8))
    pat = oracle.pattern(w.n_nodes, w.tets)
    asm = Sm.Assembler.from_workload(w)
    live = np.diff(pat[0]) > 0
    b = np.where(live, g.standard_normal(asm.n_rows), 0.0)
    x, it, rr = asm.cg_solve(torch.from_numpy(b).cuda(), rtol=1e-12)
    res, size = true_residual(pat, asm.values().cpu().numpy(), x.cpu().numpy(), b)
    nb = np.linalg.norm(b)
    assert rr <= 1e-12 and res <= 1e-12 * nb + 8 * U * it * (size + nb), (res / nb, it)
    asm.close()


@pytest.mark.parametrize("n,one", [(22, True), (23, False), (50, False)])
def test_frames_at_an_apex(n, one):
    """968 tets of a vertex (one launch, which sums a block once for each edit), 1,058 and 5,000 (two,
    which sum it once; at 5,000 and 2,304 edits 257 us in one launch, 133 in two)."""
    import oracle
    Sm = S()
    w = cone(n)
    pat = oracle.pattern(w.n_nodes, w.tets)
    asm = Sm.Assembler.from_workload(w)
    asm.enable_kernel_timing(True)
    asm.kernel_times()
    g = np.random.default_rng(n)
    mask = w.mask0.copy()
    sizes = (1, 64, 65, min(2304, w.n_tets))
    for k in sizes:
        ids = g.permutation(w.n_tets)[:k].astype(np.int32)
        asm.apply_edits(*Sm.upload_frame(ids, 1 - mask[ids]))
        mask[ids] = 1 - mask[ids]
        got = asm.values().cpu().numpy()
        assert np.array_equal(got.view(np.uint64), oracle.rebuild_workload(w, mask, pat).view(np.uint64)), k
    times = asm.kernel_times()
    launches = tuple(times[k][0] if k in times else 0 for k in ("frame", "edits", "touched"))
    assert launches == ((4, 0, 0) if one else (0, 4, 4)), times
    asm.full_rebuild()
    assert np.array_equal(asm.values().cpu().numpy().view(np.uint64), got.view(np.uint64))
    assert asm.audit() == {"values_differing": 0, "tets_differing": 0} and asm.status_sync() == Sm.STA_OK
    asm.close()
