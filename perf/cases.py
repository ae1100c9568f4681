"""What the performance of this package is measured on: the calls that a program makes
through the public entry points (stafem.Assembler, stafem.Batch, stafem.Proxy and the
autograd wrappers), from the 384-tet cube up to the 432,000-tet refinement superset.

Meshes, materials, edit streams and batches are the seeded ones of
paper_2605_11673_amd.workloads; sizes are the benchmark's and the tests' own, and odd ones
between them.  Everything is float64, the only type of the library.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2605_11673_amd import autograd, stafem
from paper_2605_11673_amd import workloads as W


def listed():
    return [
        # the smallest call there is: one frame that deletes up to 8 tets of the 384-tet
        # cube and one that reinserts them, each launched by the host as it comes
        {"name": "frames_cube4", "kind": "frames", "mesh": "cube", "n": 4, "frames": 1, "lo": 8, "hi": 8,
         "graph": False},
        # an ordinary interactive stream: fracture frames of a 118,098-tet cube and their
        # merge, launched by the host frame by frame
        {"name": "frames_fracture27", "kind": "frames", "mesh": "fracture", "n": 27, "frames": 12, "lo": 20,
         "hi": 700, "graph": False},
        # the preplanned stream of the benchmark: 24 fracture frames (50 to 2,000 tets each)
        # and 24 merge frames on 384,000 tets, captured once and replayed as one graph
        {"name": "stream_fracture40", "kind": "frames", "mesh": "fracture", "n": 40, "frames": 24, "lo": 50,
         "hi": 2000, "graph": True},
        # large frames: refinement and its undoing, 0.1 to 2 per cent of the parents per
        # frame (9 edits for each parent) on the 432,000-tet superset
        {"name": "frames_refine20", "kind": "frames", "mesh": "refinement", "n": 20, "frames": 8, "lo": 0,
         "hi": 0, "graph": False},
        # new positions and moduli, then the whole matrix anew, as each step of a fit or
        # of a design loop asks for it (half of the straddling tets are deleted)
        {"name": "rebuild_fracture40", "kind": "rebuild", "mesh": "fracture", "n": 40},
        # many uneven meshes as one context (1,000 to 120,000 tets each): all rebuilt
        {"name": "rebuild_batch16", "kind": "batch", "count": 16, "sizes": 0},
        # the linear solve of a frame on the large system, at the default tolerance
        {"name": "solve_fracture40", "kind": "solve", "mesh": "fracture", "n": 40},
        # the backward direction of the assembly alone, from given slot cotangents
        {"name": "adjoint_fracture40", "kind": "adjoint", "mesh": "fracture", "n": 40},
        # forward and backward through assembly and solve of an ordinary mesh: loss, gradients
        {"name": "gradient_fracture17", "kind": "gradient", "mesh": "fracture", "n": 17},
        # two implicit-Euler steps of a small mesh, an edit before each: launches count
        {"name": "euler_fracture11", "kind": "euler", "mesh": "fracture", "n": 11, "frames": 2, "lo": 60, "hi": 60},
        # which fragments there are, over shared vertices and over shared faces
        {"name": "fragments_fracture32", "kind": "fragments", "mesh": "fracture", "n": 32},
        # the graph-Laplacian proxy operator: a stream of frames, then one rebuild
        {"name": "proxy_fracture31", "kind": "proxy", "mesh": "fracture", "n": 31, "frames": 10, "lo": 30,
         "hi": 1000},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["frames", "frames", "frames", "rebuild", "batch", "solve", "adjoint", "gradient", "euler",
                       "fragments", "proxy"])
    if kind == "batch":
        return {"kind": kind, "count": rng.randint(3, 16), "sizes": rng.randint(1, 1 << 20)}
    mesh = rng.choice(["fracture", "fracture", "refinement"]) if kind in ("frames", "rebuild") else "fracture"
    c = {"kind": kind, "mesh": mesh, "n": _log_int(rng, 3, 20) if mesh == "refinement" else _log_int(rng, 4, 40)}
    if kind in ("gradient", "euler"):
        c["n"] = _log_int(rng, 4, 24)
    if kind in ("frames", "euler", "proxy"):
        # a stream deletes at most about half of what the mesh can fracture (a quarter of its tets)
        most = max(2, min(2000, 6 * c["n"] ** 3 // 8))
        c["frames"] = 2 if kind == "euler" else rng.randint(1, 8 if mesh == "refinement" else 20)
        c["hi"] = _log_int(rng, 2, max(2, most // max(1, c["frames"] // 2)))
        c["lo"] = max(1, _log_int(rng, 1, c["hi"]))
    if kind == "frames":
        c["graph"] = rng.random() < 0.5
    return c


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _counts(case):
    """Edits per frame: rising from lo to hi and falling again, geometrically."""
    k = case["frames"]
    if k == 24 and (case["lo"], case["hi"]) == (50, 2000):
        return W.fracture_counts(24)
    mid = (k - 1) / 2
    t = [1.0 - abs(i - mid) / mid if mid else 1.0 for i in range(k)]
    return [max(1, int(round(case["lo"] * (case["hi"] / case["lo"]) ** u))) for u in t]


def _workload(case, seed):
    if case["mesh"] == "cube":
        w = W.make_cube(seed, case["n"], case["frames"])
        ids = W.rng(seed, W.STREAM_EDITS, 1).permutation(w.n_tets)[: case["hi"]].astype(np.int32)
        w.frames = [(ids, np.zeros(len(ids), dtype=np.uint8))]
        return w
    if case["mesh"] == "refinement":
        w = W.make_refinement(seed, case["n"], case.get("frames", 4))
        w.frames = w.frames[: case.get("frames", 4)]  # the refining half; its undoing is made by _undo
        return w
    if "frames" in case:
        return W.make_fracture(seed, case["n"], counts=_counts(case))
    n = case["n"]  # one frame that deletes an eighth of the tets, along the fracture surfaces
    return W.make_fracture(seed, n, counts=[6 * n ** 3 // 8])


def _undo(frames):
    return [(ids, (1 - st).astype(np.uint8)) for ids, st in reversed(frames)]


class _View:
    """A zero-copy tensor over device memory that a context owns (its CSR values, its mask)."""

    def __init__(self, ptr, n, typestr):
        self.__cuda_array_interface__ = {"data": (ptr, False), "shape": (n,), "typestr": typestr, "version": 2}


def _view(owner, ptr, n, typestr):
    v = _View(ptr, n, typestr)
    v.owner = owner
    return torch.as_tensor(v, device="cuda")


def _values_view(asm):
    return _view(asm, asm.values_ptr(), asm.nnz, "<f8")


def _mask_view(asm):
    return _view(asm, asm.pattern_ptrs()[2], asm.n_tets, "|u1")


def _gpu(a, dtype=torch.float64):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda", dtype)


def _loads(w, seed, stream):
    """Gravity plus a random load, on every degree of freedom."""
    g = W.rng(seed, W.STREAM_LOADS, stream)
    f = g.standard_normal((w.n_nodes, 3)) * 1e-2
    f[:, 2] -= 9.81 * 1e-2
    return f


def _perturbed(w, seed):
    """New node positions and moduli of a design step."""
    g = W.rng(seed, W.STREAM_FD, 1)
    h = 1.0 / w.meta["n"] / (2 if w.name.startswith("refine") else 1)
    x = w.x + g.uniform(-0.02 * h, 0.02 * h, size=w.x.shape)
    return x, w.E * np.exp(0.1 * g.standard_normal(w.n_tets))


def _batch_cells(case):
    """Cells per side of every mesh of a batch (1e3 to 1.2e5 tets each, log-uniform)."""
    return W.batch_sizes(case["sizes"], case["count"])


def _batch(case, seed):
    cells = _batch_cells(case)
    return W.make_batch(seed, len(cells), frames=24, sizes=cells)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        ws = _batch(case, seed)
        b = stafem.Batch.from_workloads(ws)
        return {"kind": kind, "asm": b, "values": _values_view(b)}
    w = _workload(case, seed)
    s = {"kind": kind}
    if kind == "proxy":
        px = stafem.Proxy.from_workload(w, W.PROXY_EPS)
        s["asm"] = px
        s["frames"] = [stafem.upload_frame(*f) for f in _undo(w.frames) + w.frames]
        for f in s["frames"][len(w.frames):]:
            px.apply_edits(*f)
        s["values"] = _view(px, px.values_ptr(), px.nnz, "<f8")
        s["counts"] = _view(px, int(stafem.load().sta_proxy_counts_ptr(px._p)), px.n_edges, "<i4")
        return s
    asm = stafem.Assembler.from_workload(w)
    s["asm"] = asm
    done = [stafem.upload_frame(*f) for f in w.frames]
    for f in done:
        asm.apply_edits(*f)
    if kind in ("frames", "euler"):
        # a pass undoes the whole stream and runs it again, so that it ends as it began
        s["frames"] = [stafem.upload_frame(*f) for f in _undo(w.frames)] + done
        s["values"], s["mask"] = _values_view(asm), _mask_view(asm)
        if case.get("graph"):
            torch.cuda.synchronize()
            s["graph"] = torch.cuda.CUDAGraph()
            with torch.cuda.graph(s["graph"]):
                for f in s["frames"]:
                    asm.apply_edits(*f)
    if kind == "euler":
        g = W.rng(seed, W.STREAM_LOADS, 2)
        s["u0"] = _gpu(1e-3 * g.standard_normal(asm.n_rows))
        s["v0"] = _gpu(1e-1 * g.standard_normal(asm.n_rows))
        s["u"], s["v"] = torch.empty_like(s["u0"]), torch.empty_like(s["v0"])
        s["f"] = _gpu(_loads(w, seed, 1).reshape(-1))
    if kind in ("rebuild", "gradient"):
        x, E = _perturbed(w, seed)
        s["x"], s["E"], s["values"] = _gpu(x), _gpu(E), _values_view(asm)
    if kind == "solve":
        s["b"] = _gpu(_loads(w, seed, 1).reshape(-1))
    if kind == "adjoint":
        s["gA"] = _gpu(W.rng(seed, W.STREAM_LOADS, 3).standard_normal(asm.nnz))
    if kind == "gradient":
        s["logE"] = torch.log(s["E"]).requires_grad_(True)
        s["x"].requires_grad_(True)
        s["f"] = _gpu(_loads(w, seed, 1).reshape(-1))
        s["target"] = _gpu(W.rng(seed, W.STREAM_LOADS, 4).standard_normal(asm.n_rows))
    return s


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------

def run(s):
    kind, asm = s["kind"], s["asm"]
    if kind == "frames":
        if "graph" in s:
            s["graph"].replay()
        else:
            for ids, st in s["frames"]:
                asm.apply_edits(ids, st)
        return {"values": s["values"], "mask": s["mask"]}
    if kind == "batch":
        asm.full_rebuild()
        return {"values": s["values"]}
    if kind == "rebuild":
        asm.set_params(s["x"], s["E"])
        asm.full_rebuild()
        return {"values": s["values"]}
    if kind == "solve":
        x, _, _ = asm.cg_solve(s["b"])
        return {"x": x}
    if kind == "adjoint":
        g_logE, g_x = asm.adjoint(s["gA"])
        return {"g_logE": g_logE, "g_x": g_x}
    if kind == "gradient":
        s["logE"].grad = s["x"].grad = None
        values = autograd.assemble(s["logE"], s["x"], asm, s["E"])
        u = autograd.solve(values, s["f"], asm)
        loss = torch.dot(s["target"], u)
        loss.backward()
        return {"loss": loss.detach(), "u": u.detach(), "values": values.detach(), "g_logE": s["logE"].grad,
                "g_x": s["x"].grad}
    if kind == "euler":
        s["u"].copy_(s["u0"])
        s["v"].copy_(s["v0"])
        half = len(s["frames"]) // 2
        for part in (s["frames"][:half], s["frames"][half:]):
            for ids, st in part:
                asm.apply_edits(ids, st)
            asm.euler_step(s["u"], s["v"], s["f"])
        return {"u": s["u"], "v": s["v"], "values": s["values"]}
    if kind == "fragments":
        lv, kv = asm.components("vertex")
        lf, kf = asm.components("face")
        return {"vertex_labels": lv, "vertex_count": kv, "face_labels": lf, "face_count": kf}
    for ids, st in s["frames"]:  # proxy
        asm.apply_edits(ids, st)
    asm.full_rebuild()
    return {"values": s["values"], "counts": s["counts"]}


# ---------------------------------------------------------------------------
# Work
# ---------------------------------------------------------------------------

def _cube(n):
    """Nodes, node pairs that share a tet, and tets of the n^3-cell Kuhn cube."""
    return (n + 1) ** 3, 3 * n * (n + 1) ** 2 + 3 * n * n * (n + 1) + n ** 3, 6 * n ** 3


def _sizes(case):
    n = case["n"]
    if case["mesh"] != "refinement":
        return _cube(n)
    nodes, edges, tets = _cube(2 * n)
    return nodes, edges + _cube(n)[1], tets + _cube(n)[2]


# Element matrix of a tet: geometry about 120 operations, 78 distinct entries of about 6 each.
_TET_FLOPS = 600


def _rebuild_work(nodes, edges, tets):
    nnz = 9 * (nodes + 2 * edges)
    return {"bytes": 8 * nnz + 24 * nodes + 25 * tets, "flops": (_TET_FLOPS + 90) * tets}


def _frames_work(edits):
    """Per edit: its 5 bytes and its mask byte; about 44 distinct entries written (8 bytes
    each; the benchmark's fracture stream), and the 25 bytes of each of about 6 tets that
    share them with no other edit, with their entries summed again."""
    return {"bytes": edits * (6 + 44 * 8 + 6 * 25), "flops": edits * 6 * _TET_FLOPS}


def _edits(case):
    if case["mesh"] == "refinement":  # log-uniform 0.1 to 2 per cent of the parents, 9 edits each
        return 2 * case["frames"] * int(9 * 6 * case["n"] ** 3 * 0.0063)
    return 2 * sum(_counts(case)) if case["mesh"] != "cube" else 2 * case["hi"]


def _solve_work(nodes, edges, iterations):
    """A matrix (values and one column per block) and ten vectors per iteration."""
    blocks = nodes + 2 * edges
    return {"bytes": iterations * (76 * blocks + 240 * nodes), "flops": iterations * (18 * blocks + 36 * nodes)}


def _add(*ws):
    return {k: sum(w[k] for w in ws) for k in ("bytes", "flops")}


def work(case):
    kind = case["kind"]
    if kind == "batch":
        return _add(*(_rebuild_work(*_cube(n)) for n in _batch_cells(case)))
    nodes, edges, tets = _sizes(case)
    blocks = nodes + 2 * edges
    if kind == "frames":
        return _frames_work(_edits(case))
    if kind == "rebuild":
        return _rebuild_work(nodes, edges, tets)
    if kind == "solve":
        return _solve_work(nodes, edges, 200)
    if kind == "adjoint":
        return {"bytes": 72 * blocks + 33 * tets + 48 * nodes, "flops": 1100 * tets}
    if kind == "gradient":
        return _add(_rebuild_work(nodes, edges, tets), _solve_work(nodes, edges, 320),
                    {"bytes": 72 * blocks + 33 * tets + 48 * nodes, "flops": 1100 * tets + 18 * blocks})
    if kind == "euler":
        return _add(_frames_work(_edits(case)), _solve_work(nodes, edges, 200))
    if kind == "fragments":  # vertex ids, mask and labels twice, face pairs once
        return {"bytes": 16 * tets + 2 * 5 * tets + 8 * 2 * tets + 4 * nodes, "flops": 0}
    # proxy: per edit its six counts and entries and four diagonals; the rebuild reads every
    # edge's tets and writes every value
    return {"bytes": _edits(case) * (6 + 6 * 20 + 4 * 12) + 24 * tets + tets + 8 * blocks + 8 * edges, "flops": 0}


# ---------------------------------------------------------------------------
# The same in plain torch, in 64 bits
# ---------------------------------------------------------------------------

def _pairs(n_nodes, tets):
    """Block pattern: per tet the sorted-unique index of each of its 16 node pairs, the
    pairs' rows, and the first block of each row."""
    i = tets[:, :, None].expand(-1, 4, 4)
    j = tets[:, None, :].expand(-1, 4, 4)
    keys, inv = torch.unique((i * n_nodes + j).reshape(-1), return_inverse=True)
    rows = keys // n_nodes
    deg = torch.bincount(rows, minlength=n_nodes)
    first = torch.cumsum(deg, 0) - deg
    return inv.reshape(-1, 4, 4), rows, deg, first, keys % n_nodes


def _csr_positions(rows, deg, first):
    """CSR position of entry (p, q) of every block: rows 3i..3i+2 of node i share one column list."""
    b = torch.arange(len(rows), device=rows.device)
    start = 9 * first[rows]
    p = torch.arange(3, device=rows.device)[None, :, None]
    q = torch.arange(3, device=rows.device)[None, None, :]
    return start[:, None, None] + p * 3 * deg[rows][:, None, None] + 3 * (b - first[rows])[:, None, None] + q


def _elements(x, tets, E, w):
    """12 x 12 element matrices dt^2 K_e + M_e as (m, 4, 3, 4, 3), differentiable in x and E."""
    X = x[tets]
    D = X[:, 1:] - X[:, :1]
    c = torch.stack([torch.linalg.cross(D[:, 1], D[:, 2]), torch.linalg.cross(D[:, 2], D[:, 0]),
                     torch.linalg.cross(D[:, 0], D[:, 1])], 1)
    det = (D[:, 0] * c[:, 0]).sum(1)
    g = c / det[:, None, None]
    g = torch.cat([-g.sum(1, keepdim=True), g], 1)
    V = det.abs() / 6
    lam = E * w.nu / ((1 + w.nu) * (1 - 2 * w.nu)) * V * w.dt ** 2
    mu = E * 0.5 / (1 + w.nu) * V * w.dt ** 2
    outer = g[:, :, :, None, None] * g[:, None, None, :, :]              # g_a i  g_b j
    A = lam[:, None, None, None, None] * outer + mu[:, None, None, None, None] * outer.permute(0, 1, 4, 3, 2)
    eye = torch.eye(3, dtype=x.dtype, device=x.device)
    s = (g[:, :, None, :] * g[:, None, :, :]).sum(-1) * mu[:, None, None]
    s = s + torch.eye(4, dtype=x.dtype, device=x.device) * (w.rho * V / 4)[:, None, None]
    return A + s[:, :, None, :, None] * eye[None, None, :, None, :]


class _System:
    """A_t of one mesh at a mask, by scattered addition."""

    def __init__(self, w, x, E, mask):
        dev = "cuda" if torch.cuda.is_available() else "cpu"
        self.w, self.x, self.E = w, x.to(dev), E.to(dev)
        self.tets = torch.from_numpy(w.tets.astype(np.int64)).to(dev)
        self.on = torch.from_numpy(mask.astype(bool)).to(dev)
        self.inv, self.rows, self.deg, self.first, self.cols = _pairs(w.n_nodes, self.tets)
        self.pos = _csr_positions(self.rows, self.deg, self.first)

    def blocks(self):
        b = torch.zeros((len(self.rows), 3, 3), dtype=torch.float64, device=self.x.device)
        on = torch.nonzero(self.on).reshape(-1)
        for part in on.split(1 << 16):
            A = _elements(self.x, self.tets[part], self.E[part], self.w)
            b.index_add_(0, self.inv[part].reshape(-1), A.permute(0, 1, 3, 2, 4).reshape(-1, 3, 3))
        return b

    def values(self):
        out = torch.zeros(self.pos.numel(), dtype=torch.float64, device=self.x.device)
        out[self.pos.reshape(-1)] = self.blocks().reshape(-1)
        return out

    def multiply(self, b, u):
        y = torch.zeros((len(self.deg), 3), dtype=torch.float64, device=u.device)
        y.index_add_(0, self.rows, torch.bmm(b, u.reshape(-1, 3)[self.cols][:, :, None].contiguous())[:, :, 0])
        return y.reshape(-1)

    def solve(self, f, tol=1e-15, most=4000):
        """Conjugate gradients with the diagonal, restarted from the true residual."""
        b = self.blocks()
        d = torch.zeros((len(self.deg), 3), dtype=torch.float64, device=self.x.device)
        own = self.rows == self.cols
        d[self.rows[own]] = torch.diagonal(b[own], dim1=1, dim2=2)
        d = d.reshape(-1)
        live = d != 0
        m = torch.where(live, 1 / torch.where(live, d, torch.ones_like(d)), torch.zeros_like(d))
        f = torch.where(live, f.to(d.device), torch.zeros_like(d))
        u = torch.zeros_like(f)
        for _ in range(3):
            r = torch.where(live, f - self.multiply(b, u), torch.zeros_like(f))
            z = m * r
            p, rz = z.clone(), torch.dot(r, z)
            for k in range(most):
                if k % 16 == 0 and float(r.norm()) <= tol * float(f.norm()):
                    break
                q = torch.where(live, self.multiply(b, p), torch.zeros_like(p))
                a = rz / torch.dot(p, q)
                u, r = u + a * p, r - a * q
                z = m * r
                rz, old = torch.dot(r, z), rz
                p = z + (rz / old) * p
        return u

    def gradients(self, cotangents):
        """d/dlogE and d/dx of the sum over active tets of <cotangents(tets), element matrix>."""
        g_logE, g_x = torch.zeros_like(self.E), torch.zeros_like(self.x)
        for part in torch.nonzero(self.on).reshape(-1).split(1 << 16):
            x = self.x.detach().requires_grad_(True)
            logE = torch.zeros(len(part), dtype=torch.float64, device=x.device, requires_grad=True)
            A = _elements(x, self.tets[part], self.E[part] * torch.exp(logE), self.w)
            (A.permute(0, 1, 3, 2, 4) * cotangents(part)).sum().backward()
            g_logE[part] = logE.grad
            g_x += x.grad
        return g_logE, g_x


def _lumped(sys):
    X = sys.x[sys.tets]
    V = torch.linalg.det(X[:, 1:] - X[:, :1]).abs() / 6
    m = torch.zeros(len(sys.deg), dtype=torch.float64, device=sys.x.device)
    m.index_add_(0, sys.tets[sys.on].reshape(-1), (sys.w.rho * V[sys.on] / 4).repeat_interleave(4))
    return m.repeat_interleave(3)


def exact(case, seed):
    kind = case["kind"]
    if kind == "fragments":
        return None
    if kind == "batch":
        vs = [_System(w, torch.from_numpy(w.x), torch.from_numpy(w.E), w.mask0).values()
              for w in _batch(case, seed)]
        return {"values": torch.cat(vs)}
    w = _workload(case, seed)
    mask = w.mask_after(len(w.frames) - 1)
    x, E = torch.from_numpy(w.x), torch.from_numpy(w.E)
    if kind in ("rebuild", "gradient"):
        x, E = (torch.from_numpy(a) for a in _perturbed(w, seed))
    if kind == "proxy":
        return {"values": _proxy_values(w, mask), "counts": None}
    sys = _System(w, x, E, mask)
    if kind == "frames":
        return {"values": sys.values(), "mask": None}
    if kind == "rebuild":
        return {"values": sys.values()}
    f = torch.from_numpy(_loads(w, seed, 1).reshape(-1))
    if kind == "solve":
        return {"x": sys.solve(f)}
    if kind == "adjoint":
        gA = torch.from_numpy(W.rng(seed, W.STREAM_LOADS, 3).standard_normal(sys.pos.numel())).to(sys.x.device)
        g_logE, g_x = sys.gradients(lambda part: gA[sys.pos[sys.inv[part]]])
        return {"g_logE": g_logE, "g_x": g_x}
    if kind == "gradient":
        target = torch.from_numpy(W.rng(seed, W.STREAM_LOADS, 4).standard_normal(len(f))).to(sys.x.device)
        u, lam = sys.solve(f), sys.solve(target)
        ue, le = u.reshape(-1, 3)[sys.tets], lam.reshape(-1, 3)[sys.tets]
        # dL/dA = -lam u^T, per tet (a, b, p, q)
        g_logE, g_x = sys.gradients(lambda part: -le[part][:, :, None, :, None] * ue[part][:, None, :, None, :])
        return {"loss": torch.dot(target, u), "u": u, "values": sys.values(), "g_logE": g_logE, "g_x": g_x}
    # euler: a step on the undone mesh, then one on the edited mesh
    g = W.rng(seed, W.STREAM_LOADS, 2)
    u = torch.from_numpy(1e-3 * g.standard_normal(len(f))).to(sys.x.device)
    v = torch.from_numpy(1e-1 * g.standard_normal(len(f))).to(sys.x.device)
    f = f.to(u.device)
    for m in (w.mask0, mask):
        one = _System(w, x, E, m)
        u1 = one.solve(_lumped(one) * (u + w.dt * v) + w.dt ** 2 * f)
        u, v = u1, (u1 - u) / w.dt
    return {"u": u, "v": v, "values": sys.values()}


def _proxy_values(w, mask):
    tets = torch.from_numpy(w.tets.astype(np.int64))
    inv, rows, deg, first, cols = _pairs(w.n_nodes, tets)
    on = torch.zeros(len(rows), dtype=torch.float64)
    on[inv[torch.from_numpy(mask.astype(bool))].reshape(-1)] = 1.0
    own = rows == cols
    on[own] = 0.0
    degree = torch.zeros(w.n_nodes, dtype=torch.float64).index_add_(0, rows, on)
    return torch.where(own, degree[rows] + W.PROXY_EPS, torch.where(on > 0, -1.0, 0.0).to(torch.float64))
