"""GPU connectivity (sta_components) against the oracle: per-tet component labels
(smallest vertex id of the component) bitwise, the component count, and the
paper's sampled breadth-first spot checks."""
import numpy as np
import pytest
import torch

from oracle import connectivity as C
from paper_2605_11673_amd import workloads as W

pytestmark = pytest.mark.gpu


def S():
    from paper_2605_11673_amd import stafem
    return stafem


def gpu_labels(asm):
    lab, k = asm.components()
    torch.cuda.synchronize()
    return lab.cpu().numpy().astype(np.int64), k


def check(asm, w, mask, what):
    lab, k = gpu_labels(asm)
    ref, rk = C.components(w.n_nodes, w.tets, mask)
    assert np.array_equal(lab, ref), f"{what}: {np.sum(lab != ref)} labels differ"
    assert k == rk, f"{what}: {k} vs {rk} components"
    return lab, k


def test_fracture_stream_every_frame():
    Sm = S()
    w = W.make_fracture(seed=4, n=12, counts=[100, 400, 900, 300, 60])
    frames = list(w.frames) + W.merge_stream(w.frames)
    asm = Sm.Assembler.from_workload(w)
    mask = w.mask0.copy()
    ks = [check(asm, w, mask, "initial")[1]]
    for t, (ids, st) in enumerate(frames):
        asm.apply_edits(*Sm.upload_frame(ids, st))
        mask[ids] = st
        ks.append(check(asm, w, mask, f"frame {t}")[1])
    assert ks[0] == 1 and max(ks) > 1 and ks[-1] == 1  # the cut separates pieces, reinsertion rejoins them
    asm.close()


@pytest.mark.parametrize("seed", range(6))
def test_random_small_meshes(seed):
    Sm = S()
    w = W.random_small_mesh(seed, max_tets=40)
    asm = Sm.Assembler.from_workload(w)
    check(asm, w, w.mask0, f"small{seed}")
    asm.close()


def test_full_size_with_bfs_spot_checks():
    """40^3 fracture stream: labels vs the oracle at frames 0, 12, 23 and at the end of the
    reinsertion; at the peak frame, breadth-first searches from 20 sampled active tets
    each reach exactly the tets that carry their GPU label; two calls agree."""
    Sm = S()
    w = W.make_fracture(seed=0)
    frames = list(w.frames) + W.merge_stream(w.frames)
    asm = Sm.Assembler.from_workload(w)
    mask = w.mask0.copy()
    for t, (ids, st) in enumerate(frames):
        asm.apply_edits(*Sm.upload_frame(ids, st))
        mask[ids] = st
        if t in (0, 12, 23, 47):
            lab, k = check(asm, w, mask, f"frame {t}")
            print(f"[connect] frame {t}: {k} components", flush=True)
        if t == 12:
            by = C.tets_by_node(w.n_nodes, w.tets, mask)
            g = np.random.default_rng(0)
            act = np.nonzero(mask)[0]
            for e in g.choice(act, size=20, replace=False):
                comp = C.bfs_component(w.n_nodes, w.tets, mask, int(e), by)
                assert comp == set(np.nonzero(lab == lab[e])[0].tolist())
            lab2, _ = gpu_labels(asm)
            assert np.array_equal(lab, lab2)
    asm.close()


def test_refinement_and_batch():
    """Refinement superset (hanging nodes join through shared corners) every 6th frame;
    a batch of disjoint meshes has at least one component per mesh."""
    Sm = S()
    r = W.make_refinement(seed=3, n=8, frames=12)
    asm = Sm.Assembler.from_workload(r)
    mask = r.mask0.copy()
    for t, (ids, st) in enumerate(r.frames):
        asm.apply_edits(*Sm.upload_frame(ids, st))
        mask[ids] = st
        if t % 6 == 5:
            check(asm, r, mask, f"refinement frame {t}")
    asm.close()
    ws = W.make_batch(seed=3, count=6, sizes=[2, 4, 3, 1, 5, 2])
    b = Sm.Batch.from_workloads(ws)
    lab, k = gpu_labels(b)
    assert k == 6
    off = b.offsets()
    for j in range(6):
        assert np.all(lab[off["tet"][j]:off["tet"][j + 1]] == off["node"][j])
    b.close()


# Face adjacency (sta_face_components): labels are the smallest tet id of the component.

def check_face(asm, w, mask, pairs, what):
    lab, k = gpu_face(asm)
    ref, rk = C.face_components(w.tets, mask, pairs)
    assert np.array_equal(lab, ref), f"{what}: {np.sum(lab != ref)} face labels differ"
    assert k == rk, f"{what}: {k} vs {rk} face components"
    return lab, k


def gpu_face(asm):
    lab, k = asm.components("face")
    torch.cuda.synchronize()
    return lab.cpu().numpy().astype(np.int64), k


def test_face_fracture_stream_every_frame():
    Sm = S()
    w = W.make_fracture(seed=4, n=12, counts=[100, 400, 900, 300, 60])
    frames = list(w.frames) + W.merge_stream(w.frames)
    pairs = C.face_pairs(w.tets)
    asm = Sm.Assembler.from_workload(w)
    mask = w.mask0.copy()
    ks = [check_face(asm, w, mask, pairs, "initial")[1]]
    for t, (ids, st) in enumerate(frames):
        asm.apply_edits(*Sm.upload_frame(ids, st))
        mask[ids] = st
        ks.append(check_face(asm, w, mask, pairs, f"frame {t}")[1])
        if t % 3 == 0:  # the vertex labels on the same context stay right in between
            check(asm, w, mask, f"vertex frame {t}")
    assert ks[0] == 1 and max(ks) > 1 and ks[-1] == 1
    asm.close()


@pytest.mark.parametrize("seed", range(6))
def test_face_random_small_meshes(seed):
    Sm = S()
    w = W.random_small_mesh(seed, max_tets=40)
    g = np.random.default_rng(seed)
    asm = Sm.Assembler.from_workload(w)
    pairs = C.face_pairs(w.tets)
    check_face(asm, w, w.mask0, pairs, f"small{seed}")
    every = np.arange(w.n_tets, dtype=np.int32)
    for r in range(3):
        mask = (g.uniform(size=w.n_tets) < 0.6).astype(np.uint8)
        asm.apply_edits(*Sm.upload_frame(every, mask))
        check_face(asm, w, mask, pairs, f"small{seed} mask {r}")
        check(asm, w, mask, f"small{seed} mask {r} (vertex)")
    asm.close()


def test_face_full_size_with_bfs_spot_checks():
    """40^3 fracture stream, face adjacency: labels vs the oracle at frames 0, 12, 23, 47;
    at the peak frame, breadth-first searches (neighbours by direct vertex-set comparison)
    from 20 sampled active tets reach exactly the tets with their GPU label."""
    Sm = S()
    w = W.make_fracture(seed=0)
    frames = list(w.frames) + W.merge_stream(w.frames)
    pairs = C.face_pairs(w.tets)
    asm = Sm.Assembler.from_workload(w)
    mask = w.mask0.copy()
    for t, (ids, st) in enumerate(frames):
        asm.apply_edits(*Sm.upload_frame(ids, st))
        mask[ids] = st
        if t in (0, 12, 23, 47):
            lab, k = check_face(asm, w, mask, pairs, f"frame {t}")
            print(f"[connect] face frame {t}: {k} components", flush=True)
        if t == 12:
            by = C.tets_by_node(w.n_nodes, w.tets, mask)
            g = np.random.default_rng(1)
            found = []  # components already searched: a sample inside one needs no new search
            for e in g.choice(np.nonzero(mask)[0], size=20, replace=False):
                comp = next((c for c in found if int(e) in c), None)
                if comp is None:
                    comp = C.bfs_face_component(w.tets, mask, int(e), by)
                    found.append(comp)
                assert comp == set(np.nonzero(lab == lab[e])[0].tolist())
    asm.close()


@pytest.mark.parametrize("seed", [1, 2])
def test_both_adjacencies_full_size_other_seeds(seed):
    """40^3 fracture+merge stream for two more seeds: face labels against the oracle at
    every frame, vertex labels every sixth frame, and the component counts' course."""
    Sm = S()
    w = W.make_fracture(seed=seed)
    frames = list(w.frames) + W.merge_stream(w.frames)
    pairs = C.face_pairs(w.tets)
    asm = Sm.Assembler.from_workload(w)
    mask = w.mask0.copy()
    ks = []
    for t, (ids, st) in enumerate(frames):
        asm.apply_edits(*Sm.upload_frame(ids, st))
        mask[ids] = st
        ks.append(check_face(asm, w, mask, pairs, f"seed {seed} frame {t}")[1])
        if t % 6 == 5:
            check(asm, w, mask, f"seed {seed} frame {t} (vertex)")
    print(f"[connect] seed {seed} face components along the stream: {ks}", flush=True)
    assert ks[-1] == 1 and np.all(mask == 1)
    asm.close()


def test_face_refinement_and_batch():
    """Refinement superset: hanging-node interfaces separate refined regions (many more
    face components than vertex components); a batch of disjoint cubes: one component per
    mesh, labelled by its first tet."""
    Sm = S()
    r = W.make_refinement(seed=3, n=8, frames=12)
    pairs = C.face_pairs(r.tets)
    asm = Sm.Assembler.from_workload(r)
    mask = r.mask0.copy()
    for t, (ids, st) in enumerate(r.frames):
        asm.apply_edits(*Sm.upload_frame(ids, st))
        mask[ids] = st
        if t % 6 == 5:
            _, kf = check_face(asm, r, mask, pairs, f"refinement frame {t}")
            _, kv = check(asm, r, mask, f"refinement frame {t}")
            assert kf >= kv
    asm.close()
    ws = W.make_batch(seed=3, count=6, sizes=[2, 4, 3, 1, 5, 2])
    b = Sm.Batch.from_workloads(ws)
    lab, k = gpu_face(b)
    assert k == 6
    off = b.offsets()
    for j in range(6):
        assert np.all(lab[off["tet"][j]:off["tet"][j + 1]] == off["tet"][j])
    b.close()


def test_all_inactive_and_all_active():
    """Every tet deleted in one frame: no components, every label -1; every tet back: one."""
    Sm = S()
    w = W.make_fracture(seed=6, n=10, counts=[10])
    pairs = C.face_pairs(w.tets)
    asm = Sm.Assembler.from_workload(w)
    every = np.arange(w.n_tets, dtype=np.int32)
    asm.apply_edits(*Sm.upload_frame(every, np.zeros(w.n_tets, np.uint8)))
    for adj in ("vertex", "face"):
        lab, k = asm.components(adj)
        assert k == 0 and bool((lab == -1).all())
    asm.apply_edits(*Sm.upload_frame(every, np.ones(w.n_tets, np.uint8)))
    check(asm, w, np.ones(w.n_tets, np.uint8), "all active (vertex)")
    lab, k = check_face(asm, w, np.ones(w.n_tets, np.uint8), pairs, "all active (face)")
    assert k == 1 and np.all(lab == 0)
    asm.close()


def apart(m):
    """m tets without a common vertex: every window of tets holds the most vertices it can."""
    g = np.random.default_rng(m)
    x = g.uniform(0.0, 1.0, size=(4 * m, 3))
    tets = g.permutation(4 * m).astype(np.int32).reshape(m, 4)
    return W.Workload("apart", x, tets, W.lognormal_E(m, g), np.ones(m, np.uint8))


def chain(m, seed):
    """m tets, each sharing a face with the next, ids scattered over the windows."""
    g = np.random.default_rng(seed)
    p = g.permutation(m)
    tets = (np.arange(m)[:, None] + np.arange(4)[None, :]).astype(np.int32)[p]
    return W.Workload("chain", g.uniform(0.0, 1.0, size=(m + 3, 3)), tets, W.lognormal_E(m, g), np.ones(m, np.uint8))


def shuffled(n):
    w = W.make_fracture(seed=5, n=n, counts=[50])
    g = np.random.default_rng(n)
    p, q = g.permutation(w.n_tets), g.permutation(w.n_nodes).astype(np.int32)
    x = np.empty_like(w.x)
    x[q] = w.x
    return W.Workload("shuffled", x, np.ascontiguousarray(q[w.tets[p]]), w.E[p], w.mask0[p])


@pytest.mark.parametrize("mesh", [lambda: apart(1), lambda: apart(1023), lambda: apart(1024), lambda: apart(1025),
                                  lambda: apart(2049), lambda: chain(1024, 1), lambda: chain(5000, 2),
                                  lambda: shuffled(9)])
def test_windows(mesh):
    """Windows of 1,024 tets, full and with a remainder, with no common vertex at all, one long
    chain, and scattered ids (nearly every tet the root of its window): both adjacencies, all
    active, then random masks of decreasing density and none."""
    Sm = S()
    w = mesh()
    pairs = C.face_pairs(w.tets)
    asm = Sm.Assembler.from_workload(w)
    g = np.random.default_rng(7)
    every = np.arange(w.n_tets, dtype=np.int32)
    for density in (1.0, 0.9, 0.5, 0.1, 0.0):
        mask = (g.uniform(size=w.n_tets) < density).astype(np.uint8)
        asm.apply_edits(*Sm.upload_frame(every, mask))
        check(asm, w, mask, f"{w.name} {w.n_tets} {density} (vertex)")
        check_face(asm, w, mask, pairs, f"{w.name} {w.n_tets} {density}")
    asm.close()
