"""Benchmark: exact streaming assembly vs GPU full rebuild on one MI355X.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--no-cpu-baseline] [--no-extras]

Headline workload: jittered Kuhn cube 40^3 x 6 (384,000 candidate tets,
68,921 nodes, 8,945,649 FP64 values), lognormal E, nu 0.3, rho 1000,
dt 1e-2.  One step = the 24-frame Voronoi fracture stream (50..2000
deletions per frame) followed by the 24 frames that reinsert the deleted
tets in reverse order (merge), so every step starts and ends at the
initial mask.  Edit lists are resident in HBM before timing.  The rebuild's
stores (and the mode of frames of more edits than one launch takes) are chosen
by the library's autotuner on the peak frame before timing.  The timed region
replays the whole step captured as one HIP graph.

Printed: one compact JSON line on stdout (the last line, a few KB): touched
slots/s over the timed steps, per-frame streaming and rebuild times (both
pipelined from HIP graphs and per-frame latency between events), their
ratios, the HBM roofline of the dominant streaming kernel from the
method's algorithmic bytes (the design's own byte count and the committed
counter traffic beside it), the oracle's CPU rebuild rate on a bounded
sample (one thread, and all host threads), parity (streaming bitwise equal
to the GPU rebuild at every frame, checked outside the timed region) and a
one-line summary per secondary workload.  Everything else (the per-frame
rows, the autotuner's report, every secondary section in full: refinement
superset, 64-mesh batch in both frame modes, +/- delta policy, proxy
operator, implicit Euler, connectivity, differentiation) goes to the file
named by --detail, with a one-line summary of each on stderr.
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "per-frame A_t update us + touched slots/s, streaming vs GPU rebuild; HBM GB/s"
HBM_PEAK_GBS = 8000.0
TRAFFIC_FILE = os.path.join(ROOT, "profiles", "traffic.json")


def log(*a):
    print(*a, file=sys.stderr, flush=True)


# ---------------------------------------------------------------------------
# Algorithmic bytes of the method (what any exact streaming update must move)
# ---------------------------------------------------------------------------

def alg_edits(st):
    """Edit phase: per edit 130 B (the edit, its mask byte read and written, the tet's
    10 block ids, the block-stamp read-modify-writes); per activation 780 B (vertex ids,
    coordinates and modulus, 624 B of contributions written)."""
    return 130 * st["edits"] + 780 * st["activated"]


def alg_touched(st):
    """Re-sum of the touched blocks: per incidence its tet id, mask byte and
    contribution (48 B diagonal, 72 B off-diagonal); 8 B per slot written (both
    triangles); 24 B of segment and row metadata per block."""
    return (53 * st["diag_incidences"] + 77 * st["off_incidences"] + 8 * st["touched_slots"]
            + 24 * (st["diag_blocks"] + st["off_blocks"]))


def alg_frame(st):
    return alg_edits(st) + alg_touched(st)


ALG_MODEL = {"edits": alg_edits, "touched": alg_touched, "frame": alg_frame}


# ---------------------------------------------------------------------------
# Design bytes (what these kernels move as designed, each byte once)
# ---------------------------------------------------------------------------

def bytes_sums(st):
    """Sums of the touched blocks: per incidence its 4-byte entry, mask byte and the parts
    of its tet's record (diagonal: one gradient and three scalars, 48 B; off-diagonal: two
    gradients and two scalars, 64 B); 9 values written per diagonal block (72 B), 18 per
    off-diagonal block (144 B)."""
    return (53 * st["diag_incidences"] + 69 * st["off_incidences"]
            + 72 * st["diag_blocks"] + 144 * st["off_blocks"])


def bytes_touched(st):
    """Two-launch frame, phase 2: per edit its 10 claim records (320 B), and the sums."""
    return 320 * st["edits"] + bytes_sums(st)


def bytes_edits(st):
    """Two-launch frame, phase 1: per edit id + state + tet stamp read/write + mask read +
    10 claim records written + undo byte (335 B); per changed tet its 10 block
    descriptors, 10 block stamp read/writes and mask write (401 B)."""
    return 335 * st["edits"] + 401 * st["changed"]


def bytes_frame(st):
    """One-launch frame: per edit id, state, mask byte read and written, undo byte and kept
    id (12 B); per changed tet its 10 block descriptors (320 B); the sums, each block once
    (edits that share a block read and write it again, from cache)."""
    return 12 * st["edits"] + 320 * st["changed"] + bytes_sums(st)


def bytes_delta(st):
    """+/- delta frame (k_delta_edits + k_delta_clear): per edit its id, state, tet stamp
    read/write and mask read, and its stamp cleared again (20 B); per changed tet its
    descriptors (320 B), vertex ids and geometry record (144 B), its mask write, and the
    144 CSR entries of its 10 blocks read and written by the atomic additions (2,769 B)."""
    return 20 * st["edits"] + 2769 * st["changed"]


def bytes_connectivity_pass(n_tets, n_nodes, n_pairs=0):
    """A lower bound for one connectivity rebuild: every tet's mask byte, vertex ids (16 B,
    vertex adjacency) and label (4 B), every node's parent (4 B), and for face adjacency
    every candidate pair (8 B) with its two mask bytes; one pass over the data."""
    if n_pairs:
        return 5 * n_tets + 10 * n_pairs
    return 21 * n_tets + 4 * n_nodes


def bytes_element(n_tets, n_nodes):
    """Rebuild geometry kernel: per tet its vertex ids, E and mask byte (25 B) and its
    128-byte record written; node coordinates once (24 B per node)."""
    return 153 * n_tets + 24 * n_nodes


def bytes_reduce(nd, no, n_tets):
    """Rebuild rows kernel: per tet its record and mask byte once, its 4 node incidences
    (4 B) and 12 row terms (2 B); per row block (diagonal once, off-diagonal twice) its
    8-byte plan entry and 9 values written."""
    return (129 + 16 + 24) * n_tets + 80 * (nd + 2 * no)


# ---------------------------------------------------------------------------

def pct(a, q):
    return float(np.percentile(np.asarray(a, dtype=np.float64), q))


LIB = os.path.join(ROOT, "paper_2605_11673_amd", "libstafem.so")


def source_sha():
    """Digest of the library's device code (its .hip_fatbin section): counter records taken
    with other kernels are not used.  The device code is rebuilt bit for bit from the same
    kernel sources, and host-only changes leave it alone."""
    import struct

    try:
        with open(LIB, "rb") as f:
            data = f.read()
    except OSError:
        return None
    shoff = struct.unpack_from("<Q", data, 0x28)[0]
    shentsize, shnum, shstrndx = struct.unpack_from("<HHH", data, 0x3A)
    secs = [struct.unpack_from("<IIQQQQ", data, shoff + i * shentsize) for i in range(shnum)]
    stroff = secs[shstrndx][4]
    for name, _typ, _flags, _addr, offset, size in secs:
        if data[stroff + name:data.index(b"\0", stroff + name)] == b".hip_fatbin":
            return hashlib.sha256(data[offset:offset + size]).hexdigest()[:16]
    return None


_TRAFFIC = None


def _traffic():
    global _TRAFFIC
    if _TRAFFIC is None:
        try:
            with open(TRAFFIC_FILE) as f:
                d = json.load(f)
        except (OSError, ValueError):
            d = {}
        sha = source_sha()
        _TRAFFIC = d if sha is not None and d.get("device_code_sha") == sha else {}
    return _TRAFFIC


def load_traffic(workload, kernels, per=None):
    """HBM bytes (FETCH_SIZE + WRITE_SIZE, scaled) from the committed rocprofv3 counter runs
    of `workload`: the kernels' summed bytes per unit, a unit being one dispatch of `per`
    (default: of the first kernel).  None if a kernel has no record or the library's device
    code changed since the counters were taken."""
    rec = _traffic().get("workloads", {}).get(workload, {}).get("kernels", {})
    if not all(k in rec for k in kernels) or (per is not None and per not in rec):
        return None
    units = rec[per or kernels[0]]["dispatches"]
    return round(sum(rec[k]["bytes"] for k in kernels) / max(units, 1), 1)


def load_frame_traffic(kernel):
    """Per-frame HBM bytes of the frame kernel (first pass over the headline step), or None."""
    return _traffic().get("frames", {}).get(kernel)


def kernel_instance(asm, kernel):
    """Template instantiation of `kernel` that the context launches: the key of its counter
    record (counters of another instantiation are not attached)."""
    if kernel == "k_rows":
        return f"k_rows<{'true' if asm.get_config()['rebuild_nt'] else 'false'}>"
    return kernel


ONE_LAUNCH_EDITS = 2304  # largest list that runs as one launch (include/stafem.h, sta_set_config)


def roofline(kernel, alg_bytes, seconds, launches, traffic=None, design_bytes=None):
    """alg_bytes: the method's algorithmic bytes over all launches; design_bytes (optional):
    the design's own byte count over the same launches, reported beside it; traffic: the
    counted HBM bytes per launch (load_traffic), or None."""
    achieved = alg_bytes / seconds / 1e9 if seconds > 0 else 0.0
    out = {"kernel": kernel, "bound": "hbm", "achieved": round(achieved, 2), "peak": HBM_PEAK_GBS,
           "unit": "GB/s", "frac": round(achieved / HBM_PEAK_GBS, 5),
           "traffic": traffic,
           "algorithmic_bytes_per_launch": round(alg_bytes / max(launches, 1), 1),
           "avg_launch_us": round(seconds / max(launches, 1) * 1e6, 3), "launches": launches}
    if design_bytes is not None:
        out["design_bytes_per_launch"] = round(design_bytes / max(launches, 1), 1)
    return out


def host_info():
    """The host the CPU baseline ran on: logical CPUs, those this process may use, the
    OpenMP thread setting and the CPU model as lscpu reports it."""
    import subprocess

    model = "unknown"
    try:
        out = subprocess.run(["lscpu"], capture_output=True, text=True, timeout=10).stdout
        for line in out.splitlines():
            if line.strip().startswith("Model name:"):
                model = line.split(":", 1)[1].strip()
                break
    except (OSError, subprocess.SubprocessError):
        pass
    if model == "unknown":
        try:
            for line in open("/proc/cpuinfo"):
                if line.startswith("model name"):
                    model = line.split(":", 1)[1].strip()
                    break
        except OSError:
            pass
    try:
        usable = len(os.sched_getaffinity(0))
    except AttributeError:
        usable = os.cpu_count()
    return {"nproc": os.cpu_count(), "usable_cpus": usable, "omp_num_threads": os.environ.get("OMP_NUM_THREADS"),
            "cpu_model": model}


# ---------------------------------------------------------------------------
# Measurement helpers
# ---------------------------------------------------------------------------

class Stream:
    """An assembler, its step (a list of device-resident frames) and per-frame stats."""

    def __init__(self, torch, asm, frames, n_tets, n_nodes, mask0, workload="fracture"):
        from paper_2605_11673_amd import stafem
        self.torch, self.asm = torch, asm
        self.workload = workload  # key of this workload's counter records
        self.frames_host = frames
        self.dframes = [stafem.upload_frame(ids, st) for ids, st in frames]
        self.n_tets, self.n_nodes, self.mask0 = n_tets, n_nodes, mask0
        self.stats = []
        torch.cuda.synchronize()

    def step(self):
        for di, ds in self.dframes:
            self.asm.apply_edits(di, ds)

    def tune(self, peak):
        di, ds = self.dframes[peak]
        rep = self.asm.autotune(di, ds, reps=7)
        cfg = self.asm.get_config()
        cfg["buckets"] = {k: self.asm.bucket_map(k) for k in ("rebuild", "stream")}
        return cfg, [r for r in rep.splitlines() if r.strip()]

    def stats_pass(self, check_parity):
        torch, asm = self.torch, self.asm
        stats, mismatches = [], 0
        ref = torch.empty(asm.nnz, dtype=torch.float64, device="cuda")
        for di, ds in self.dframes:
            asm.apply_edits(di, ds)
            stats.append(asm.last_frame_stats())
            if check_parity:
                got = asm.values()
                asm.full_rebuild()
                torch.cuda.synchronize()
                ref.copy_(asm.values())
                if not torch.equal(got.view(torch.int64), ref.view(torch.int64)):
                    mismatches += 1
        torch.cuda.synchronize()
        self.stats = stats
        return stats, mismatches

    def timed(self, steps, warmup, kernel_events=True):
        """Kernel durations (events), host-launched step time, graph-replayed step time."""
        torch, asm = self.torch, self.asm
        for _ in range(warmup):
            self.step()
        torch.cuda.synchronize()
        ktimes, eager_s = {}, 0.0
        if kernel_events:
            asm.enable_kernel_timing(True)
            asm.kernel_times()
            for _ in range(steps):
                self.step()
            ktimes = asm.kernel_times()
            asm.enable_kernel_timing(False)
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(steps):
                self.step()
            torch.cuda.synchronize()
            eager_s = (time.perf_counter() - t0) / steps
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            self.step()
        torch.cuda.synchronize()
        for _ in range(warmup):
            graph.replay()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(steps):
            graph.replay()
        torch.cuda.synchronize()
        step_s = (time.perf_counter() - t0) / steps
        del graph
        return ktimes, eager_s, step_s

    def stream_roofline(self, ktimes, steps):
        """Roofline of the dominant streaming kernel (largest summed duration): the method's
        algorithmic bytes over its launches, the design's bytes beside them."""
        design = {"touched": bytes_touched, "edits": bytes_edits, "frame": bytes_frame}
        kern = {k: {"launches": n, "avg_us": round(ms * 1e3 / max(n, 1), 3), "total_ms": round(ms, 3)}
                for k, (n, ms) in ktimes.items()}
        cands = [k for k in ("frame", "touched", "edits") if k in ktimes]
        dom = max(cands, key=lambda k: ktimes[k][1])
        # the frames that ran through the dominant kernel
        one = [st for st in self.stats if self.asm.get_config()["fused"] or st["edits"] <= ONE_LAUNCH_EDITS]
        mine = one if dom == "frame" else [st for st in self.stats if not any(st is o for o in one)]
        alg = steps * sum(ALG_MODEL[dom](st) for st in mine)
        des = steps * sum(design[dom](st) for st in mine)
        name = "k_once" if dom == "frame" and any(st["edits"] <= ONE_LAUNCH_EDITS for st in one) else "k_" + dom
        return kern, roofline(name, alg, ktimes[dom][1] * 1e-3, ktimes[dom][0],
                              traffic=load_traffic(self.workload, [kernel_instance(self.asm, name)]),
                              design_bytes=des)

    def rebuild_pipelined(self, reps=20):
        """Microseconds per full rebuild with `reps` rebuilds captured as one HIP graph and
        replayed (timed as the streaming step is), at the current mask."""
        torch, asm = self.torch, self.asm
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            for _ in range(reps):
                asm.full_rebuild()
        g.replay()
        torch.cuda.synchronize()
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        ev[0].record()
        for _ in range(5):
            g.replay()
        ev[1].record()
        ev[1].synchronize()
        del g
        return ev[0].elapsed_time(ev[1]) * 1e3 / (5 * reps)

    def rebuild_roofline(self, reps=5):
        """Rebuild kernels timed with events at every frame's mask (the step returns to the start)."""
        asm = self.asm
        asm.enable_kernel_timing(True)
        asm.kernel_times()
        for di, ds in self.dframes:
            asm.apply_edits(di, ds)
            for _ in range(reps):
                asm.full_rebuild()
        kt = asm.kernel_times()
        asm.enable_kernel_timing(False)
        nd, no = asm.n_diag_blocks, asm.n_off_blocks
        rb = bytes_reduce(nd, no, self.n_tets)
        eb = bytes_element(self.n_tets, self.n_nodes)
        n_e, ms_e = kt.get("element", (0, 0.0))
        n_r, ms_r = kt.get("reduce", (0, 0.0))
        # a large batch is rebuilt in mesh groups, a geometry and a row launch each (and, while
        # kernels are timed, one for large nodes, also with none): rates and counted bytes are
        # per rebuild, all groups together
        rebuilds = len(self.frames_host) * reps
        per_e, per_r = n_e / max(rebuilds, 1), n_r / max(rebuilds, 1)
        te = load_traffic(self.workload, ["k_geometry"])
        tr = load_traffic(self.workload, [kernel_instance(asm, "k_rows")])
        el = roofline("k_geometry", eb * rebuilds, ms_e * 1e-3, rebuilds,
                      traffic=None if te is None else round(te * per_e, 1))
        re = roofline("k_rows", rb * rebuilds, ms_r * 1e-3, rebuilds,
                      traffic=None if tr is None else round(tr * per_e, 1))
        el["launches_per_rebuild"], re["launches_per_rebuild"] = per_e, per_r
        return {"element": el, "reduce": re,
                "rebuild_us_mean": round((ms_e + ms_r) * 1e3 / max(rebuilds, 1), 3),
                "full_rebuild_alg_bytes": int(eb + rb)}

    def mask_before(self, k):
        m = self.mask0.copy()
        for ids, st in self.frames_host[:k]:
            m[ids] = st
        return m

    def per_frame(self, reps):
        """Per-frame latency: one sta_apply_edits between two HIP events on the launch
        stream, warm and after writing 1 GiB to evict the caches; the full rebuild at
        the same mask; medians."""
        torch, asm = self.torch, self.asm
        flush = torch.empty(1 << 30, dtype=torch.uint8, device="cuda")  # > 256 MB infinity cache
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]

        def timed(fn, cold):
            # queue the events and the launches behind GPU work (the cache flush, or
            # a spin that touches no memory), so that the interval is GPU time alone
            # and not the host's launch latency
            if cold:
                flush.fill_(1)
            else:
                torch.cuda._sleep(200000)
            ev[0].record()
            fn()
            ev[1].record()
            ev[1].synchronize()
            return ev[0].elapsed_time(ev[1]) * 1e3

        rows, t_stream, t_cold, t_reb, t_reb_cold = [], [], [], [], []
        ftr = load_frame_traffic("k_once") if self.workload == "fracture" else None
        for k, ((di, ds), st) in enumerate(zip(self.dframes, self.stats)):
            ids_h = self.frames_host[k][0]
            prev = torch.from_numpy(self.mask_before(k)[ids_h].copy()).cuda()  # undoes the frame
            warm, cold = [], []
            for r in range(reps):
                c = r % 2 == 1
                (cold if c else warm).append(timed(lambda: asm.apply_edits(di, ds), c))
                asm.apply_edits(di, prev)
            asm.apply_edits(di, ds)
            nreb = max(4, reps // 2)
            reb = [timed(asm.full_rebuild, False) for _ in range(nreb)]
            reb_cold = [timed(asm.full_rebuild, True) for _ in range(nreb // 2)]
            alg = alg_frame(st)
            rows.append({"frame": k, "edits": st["edits"], "touched_blocks": st["touched_blocks"],
                         "touched_slots": st["touched_slots"], "stream_us": round(float(np.median(warm)), 3),
                         "stream_cold_us": round(float(np.median(cold)), 3) if cold else None,
                         "rebuild_us": round(float(np.median(reb)), 3),
                         "rebuild_cold_us": round(float(np.median(reb_cold)), 3), "alg_bytes": alg,
                         "stream_gbs": round(alg / (np.median(warm) * 1e-6) / 1e9, 2)})
            if ftr and k < len(ftr):
                cb = ftr[k]["k_once"]
                rows[-1]["counter_bytes"] = cb
                rows[-1]["counter_gbs"] = round(cb / (np.median(warm) * 1e-6) / 1e9, 2)
                rows[-1]["counter_frac_of_peak"] = round(cb / (np.median(warm) * 1e-6) / 1e9 / HBM_PEAK_GBS, 5)
            t_stream.append(float(np.median(warm)))
            if cold:
                t_cold.append(float(np.median(cold)))
            t_reb.append(float(np.median(reb)))
            t_reb_cold.append(float(np.median(reb_cold)))
        del flush
        ratio = np.asarray(t_reb) / np.asarray(t_stream)
        peak = int(np.argmax([r["edits"] for r in rows]))

        def summ(a):
            return {"median": round(pct(a, 50), 3), "p10": round(pct(a, 10), 3), "p90": round(pct(a, 90), 3)}

        return {
            "stream_us_per_frame": {"mean": round(float(np.mean(t_stream)), 3), **summ(t_stream),
                                    "max": round(float(np.max(t_stream)), 3)},
            "stream_cold_us_per_frame": summ(t_cold) if t_cold else None,
            "rebuild_us": summ(t_reb),
            "rebuild_cold_us": summ(t_reb_cold),
            "stream_vs_rebuild": {"median_ratio": round(float(np.median(ratio)), 2),
                                  "min_ratio": round(float(np.min(ratio)), 2), "peak_frame": peak,
                                  "peak_frame_ratio": round(float(ratio[peak]), 2)},
            "frames": rows,
        }


def cpu_baseline(args, w, frames, stats):
    """The oracle (plain C, single thread) rebuilding A_t from the mask, on a sample of
    the step's frames, expressed in the same unit: touched slots delivered per second."""
    import oracle

    pat = oracle.pattern(w.n_nodes, w.tets)
    mask = w.mask0.copy()
    masks = []
    for ids, st in frames:
        mask[ids] = st
        masks.append(mask.copy())
    idx = np.linspace(0, len(frames) - 1, num=min(args.cpu_sample, len(frames))).round().astype(int)
    t_total, slots = 0.0, 0
    serial = {}
    for k in idx:
        t0 = time.perf_counter()
        serial[int(k)] = oracle.rebuild(w.x, w.tets, w.E, w.nu, w.rho, w.dt, masks[k], *pat)
        t_total += time.perf_counter() - t0
        slots += stats[k]["touched_slots"]
    # the same rebuilds row by row on every host thread, checked bitwise against the serial ones
    t_par, slots_par, threads, same = 0.0, 0, 0, True
    for k in idx:
        t0 = time.perf_counter()
        v, threads = oracle.rebuild_rows(w.x, w.tets, w.E, w.nu, w.rho, w.dt, masks[k], *pat)
        t_par += time.perf_counter() - t0
        slots_par += stats[k]["touched_slots"]
        same = same and bool(np.array_equal(v.view(np.uint64), serial[int(k)].view(np.uint64)))
    info = host_info()
    return {"value": slots / t_total, "unit": "touched slots/s", "cores": 1, "kind": "oracle",
            "sample": f"oracle full rebuild from the mask at {len(idx)} of the {len(frames)} frames of one step "
                      f"(frames {idx.tolist()}), single-threaded, {t_total:.1f} s",
            "rebuild_s_per_frame": round(t_total / len(idx), 4), **info,
            "multicore": {"value": slots_par / t_par, "unit": "touched slots/s", "cores": threads,
                          "rebuild_s_per_frame": round(t_par / len(idx), 4),
                          "bitwise_equal_to_serial": same,
                          "sample": "the same frames, row-parallel oracle rebuild on every host thread"}}


def secondary(torch, name, asm, frames, n_tets, n_nodes, mask0, peak, args, describe, fused_too=False,
              workload=None):
    """Tuned, parity-checked, graph-timed stream of another workload; with fused_too the
    same stream also in the one-launch frame mode (the tuned slot mapping, its own parity
    check and timing)."""
    log(f"[bench] {name}: {n_tets} tets, {len(frames)} frames")
    s = Stream(torch, asm, frames, n_tets, n_nodes, mask0, workload=workload)
    if args.config:  # forced (as for counter runs, where the tuner's repeated frames would skew averages)
        asm.set_config(*[int(v) for v in args.config.split(",")])
        cfg = {**asm.get_config(), "buckets": {k: asm.bucket_map(k) for k in ("rebuild", "stream")}}
    else:
        cfg, _ = s.tune(peak)
    stats, mism = s.stats_pass(check_parity=True)
    steps = max(3, args.steps // 4)
    kt, eager_s, step_s = s.timed(steps, 1)
    kern, roof = s.stream_roofline(kt, steps)
    reb = s.rebuild_roofline(reps=2)
    slots = int(sum(st["touched_slots"] for st in stats))
    frame_us = step_s * 1e6 / len(frames)
    out = {"workload": describe, "n_tets": n_tets, "nnz": asm.nnz, "frames_per_step": len(frames),
           "edits_per_step": int(sum(st["edits"] for st in stats)), "touched_slots_per_step": slots,
           "tuned_config": cfg, "value": slots / step_s, "unit": "touched slots/s",
           "ms_per_step": step_s * 1e3, "stream_pipelined_us_per_frame": round(frame_us, 3),
           "host_launched_ms_per_step": eager_s * 1e3, "rebuild_us_mean": reb["rebuild_us_mean"],
           "rebuild_vs_pipelined_frame": round(reb["rebuild_us_mean"] / frame_us, 2),
           "roofline": roof, "roofline_rebuild": {"element": reb["element"], "reduce": reb["reduce"]},
           "kernels": kern, "parity": {"frames_checked": len(frames), "mismatching_frames": mism}}
    log(f"[bench] {name}: {step_s * 1e3:.3f} ms/step, {frame_us:.2f} us/frame, "
        f"rebuild {reb['rebuild_us_mean']} us, parity mismatches {mism}")
    if fused_too:
        # the grid cap of the persistent launch: the fastest of a few, timed on the step
        best = None
        for cap in (32, 64, 128, 256):
            apply_config(asm, dict(cfg, fused=1, grid_cap=cap))
            _, _, t = s.timed(1, 1, kernel_events=False)
            if best is None or t < best[1]:
                best = (cap, t)
        fcfg = dict(cfg, fused=1, grid_cap=best[0])
        apply_config(asm, fcfg)
        _, fmism = s.stats_pass(check_parity=True)
        fkt, _, fstep_s = s.timed(steps, 1)
        fkern, froof = s.stream_roofline(fkt, steps)
        ffus = fstep_s * 1e6 / len(frames)
        out["one_launch"] = {"config": {k: v for k, v in fcfg.items() if k != "buckets"},
                             "stream_pipelined_us_per_frame": round(ffus, 3), "value": slots / fstep_s,
                             "rebuild_vs_pipelined_frame": round(reb["rebuild_us_mean"] / ffus, 2),
                             "roofline": froof, "kernels": fkern,
                             "parity": {"frames_checked": len(frames), "mismatching_frames": fmism}}
        assert asm.status_sync() == 0, "one-launch frame reported a device error"
        apply_config(asm, cfg)
        log(f"[bench] {name}, one launch per frame: {ffus:.2f} us/frame, parity mismatches {fmism}")
    return out


def proxy_rebuild_bytes(n_edges, n_incidences, n_nodes, nnz):
    """Algorithmic bytes of the proxy rebuild: per edge its segment bounds, incidence ids
    and mask bytes, count write, two positions and two value writes; per vertex its row
    bounds, diagonal position, the row's values, degree and diagonal writes."""
    return (n_edges * (8 + 4 + 8 + 16) + n_incidences * (4 + 1)
            + n_nodes * (8 + 4 + 4 + 8) + (nnz - n_nodes) * 8 + n_nodes * 8)


def proxy_section(torch, stafem, w, frames, args):
    """The graph-Laplacian proxy operator over the same mesh and stream: streaming state
    bitwise equal to the GPU rebuild at every frame, the whole stream graph-timed, the
    rebuild timed, and (unless disabled) the oracle's rebuild on the host."""
    from paper_2605_11673_amd.workloads import PROXY_EPS as eps

    px = stafem.Proxy.from_workload(w, eps)
    dfr = [stafem.upload_frame(ids, st) for ids, st in frames]
    # parity: streaming state vs a rebuild of a second context at every frame
    ref = stafem.Proxy.from_workload(w, eps)
    mism = 0
    trans = []
    for ids, st in dfr:
        px.apply_edits(ids, st)
        trans.append(px.last_frame_stats()["transitions"])
        a = px.state()
        ref.apply_edits(ids, st)
        ref.full_rebuild()
        b = ref.state()
        torch.cuda.synchronize()
        mism += int(not all(torch.equal(x.view(torch.uint8) if x.dtype == torch.float64 else x,
                                        y.view(torch.uint8) if y.dtype == torch.float64 else y)
                            for x, y in zip(a, b)))
    ref.close()
    # undo the stream so that each timed step starts from the initial state
    for ids, st in reversed(dfr):
        px.apply_edits(ids, (1 - st.to(torch.int32)).to(torch.uint8))
    inv = [(ids, (1 - st.to(torch.int32)).to(torch.uint8)) for ids, st in dfr]
    torch.cuda.synchronize()

    def step():
        for ids, st in dfr:
            px.apply_edits(ids, st)
        for ids, st in reversed(inv):
            px.apply_edits(ids, st)

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        step()
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    g.replay()
    torch.cuda.synchronize()
    ev[0].record()
    for _ in range(args.steps):
        g.replay()
    ev[1].record()
    torch.cuda.synchronize()
    step_s = ev[0].elapsed_time(ev[1]) * 1e-3 / args.steps
    frames_per_step = 2 * len(frames)
    reb = []
    for _ in range(max(5, args.reps)):
        torch.cuda._sleep(200000)
        ev[0].record()
        px.full_rebuild()
        ev[1].record()
        ev[1].synchronize()
        reb.append(ev[0].elapsed_time(ev[1]) * 1e3)
    assert px.status_sync() == stafem.STA_OK
    edits = int(sum(len(f[0]) for f in frames))
    reb_us = float(np.median(reb))
    alg = proxy_rebuild_bytes(px.n_edges, 6 * w.n_tets, w.n_nodes, px.nnz)
    out = {"workload": f"graph-Laplacian proxy L_t + eps I (eps {eps:g}) over the 40^3 fracture mesh: the 48-frame "
                       "fracture+reinsertion stream, then the same frames undone (96 frames per step)",
           "n_edges": px.n_edges, "nnz": px.nnz, "frames_per_step": frames_per_step,
           "edits_per_step": 2 * edits, "value": 2 * edits / step_s, "unit": "edits/s",
           "ms_per_step": step_s * 1e3, "stream_pipelined_us_per_frame": round(step_s * 1e6 / frames_per_step, 3),
           "transitions_per_stream": int(sum(trans)),
           "rebuild_us_median": round(reb_us, 3),
           "rebuild_roofline": {"bound": "hbm", "achieved": round(alg / (reb_us * 1e-6) / 1e9, 2), "peak": HBM_PEAK_GBS,
                                "unit": "GB/s", "frac": round(alg / (reb_us * 1e-6) / 1e9 / HBM_PEAK_GBS, 5),
                                "traffic": load_traffic("proxy", ["k_proxy_counts", "k_proxy_diagonal"]),
                                "algorithmic_bytes": alg},
           "rebuild_vs_pipelined_frame": round(reb_us / (step_s * 1e6 / frames_per_step), 2),
           "parity": {"frames_checked": len(frames), "mismatching_frames": mism,
                      "check": "streaming counts, degrees and values bitwise equal to a GPU rebuild at every frame"}}
    px.close()
    if not args.no_cpu_baseline:
        from oracle import proxy as oproxy

        pat = oproxy.proxy_pattern(w.n_nodes, w.tets)
        mask = w.mask0.copy()
        t_total, k = 0.0, 0
        for ids, st in frames[::8]:
            mask[ids] = st
            t0 = time.perf_counter()
            oproxy.proxy_rebuild(w.n_nodes, w.tets, mask, eps, pat)
            t_total += time.perf_counter() - t0
            k += 1
        out["cpu_baseline"] = {"value": round(t_total / k * 1e3, 3), "unit": "ms per rebuild", "cores": 1,
                               "kind": "oracle", "sample": f"proxy oracle rebuild (numpy) at {k} frames of the stream"}
    log(f"[bench] proxy: {step_s * 1e3:.3f} ms/step, {out['stream_pipelined_us_per_frame']} us/frame, "
        f"rebuild {reb_us:.1f} us, parity mismatches {mism}")
    return out


def graph_time(torch, fn, steps, warmup):
    """Seconds per call of fn() captured once as a HIP graph and replayed `steps` times."""
    for _ in range(warmup):
        fn()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        fn()
    g.replay()
    torch.cuda.synchronize()
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    ev[0].record()
    for _ in range(steps):
        g.replay()
    ev[1].record()
    torch.cuda.synchronize()
    return ev[0].elapsed_time(ev[1]) * 1e-3 / steps, g


def drift(torch, asm):
    """Largest difference between the maintained values and a rebuild of the same mask
    (the rebuild replaces the maintained values)."""
    got = asm.values()
    asm.full_rebuild()
    ref = asm.values()
    torch.cuda.synchronize()
    d = (got - ref).abs()
    nz = ref != 0
    rel = (d[nz] / ref[nz].abs()).max().item() if bool(nz.any()) else 0.0
    return {"max_abs": d.max().item(), "max_rel": rel, "entries_differing": int((d != 0).sum().item()),
            "entries": int(ref.numel())}


def apply_config(asm, cfg):
    """The tuned configuration of the headline context, bucket maps included."""
    asm.set_config(*[cfg[k] for k in ("fused", "rebuild_qd", "rebuild_qo", "stream_qd", "stream_qo", "grid_cap",
                                      "rebuild_nt")])
    for k, m in cfg.get("buckets", {}).items():
        asm.set_bucket_map(k, m["diag"], m["off"])


def delta_section(torch, stafem, w, frames, cfg, exact_step_s, args, stats=None, oracle_s_per_frame=None):
    """The paper's +/- delta policy (sta_apply_edits_delta) on the headline stream and on a
    repeated-locality stream (one slab deleted and reinserted frame after frame): time per
    frame against the exact policy, and the drift from the rebuild after many frames."""
    asm = stafem.Assembler.from_workload(w)
    apply_config(asm, cfg)
    dfr = [stafem.upload_frame(ids, st) for ids, st in frames]

    def delta_step():
        for ids, st in dfr:
            asm.apply_edits_delta(ids, st)

    step_s, _ = graph_time(torch, delta_step, args.steps, args.warmup)
    n_frames = len(frames) * (args.steps + args.warmup + 2)
    dr = drift(torch, asm)
    out = {"workload": "the headline fracture+reinsertion stream under the +/- delta policy",
           "delta_us_per_frame": round(step_s * 1e6 / len(frames), 3),
           "exact_us_per_frame": round(exact_step_s * 1e6 / len(frames), 3),
           "exact_over_delta": round(exact_step_s / step_s, 3),
           "drift_after_frames": n_frames, "drift": dr}
    if stats:
        # kernel events over one host-launched pass of the step (the same frames)
        asm.enable_kernel_timing(True)
        asm.kernel_times()
        delta_step()
        kt = asm.kernel_times()
        asm.enable_kernel_timing(False)
        n_d, ms_d = kt.get("delta", (0, 0.0))
        out["roofline"] = roofline("k_delta_edits+k_delta_clear", sum(bytes_delta(st) for st in stats),
                                   ms_d * 1e-3, n_d,
                                   traffic=load_traffic("delta", ["k_delta_edits", "k_delta_clear"]))
    if oracle_s_per_frame:
        out["cpu_baseline"] = {"value": round(oracle_s_per_frame * 1e6, 1), "unit": "us per frame", "cores": 1,
                               "kind": "oracle",
                               "sample": "the oracle's rebuild from the mask, against which the delta policy's "
                                         "drift is bounded (the headline CPU-baseline measurement)"}
    # repeated locality: the peak frame's tets (a slab near the impact point) deleted and
    # reinserted on alternate frames
    peak = int(np.argmax([len(f[0]) for f in frames[:24]]))
    slab = frames[peak][0]
    off = stafem.upload_frame(slab, np.zeros(len(slab), np.uint8))
    on = stafem.upload_frame(slab, np.ones(len(slab), np.uint8))
    cycle = [off, on] * 4

    def exact_loc():
        for ids, st in cycle:
            asm.apply_edits(ids, st)

    def delta_loc():
        for ids, st in cycle:
            asm.apply_edits_delta(ids, st)

    asm.full_rebuild()
    ex_s, _ = graph_time(torch, exact_loc, args.steps, args.warmup)
    de_s, g = graph_time(torch, delta_loc, args.steps, args.warmup)
    asm.full_rebuild()
    torch.cuda.synchronize()
    reps = 125  # 1000 frames
    for _ in range(reps):
        g.replay()
    out["locality"] = {"slab_tets": int(len(slab)), "frames_per_step": len(cycle),
                       "exact_us_per_frame": round(ex_s * 1e6 / len(cycle), 3),
                       "delta_us_per_frame": round(de_s * 1e6 / len(cycle), 3),
                       "exact_over_delta": round(ex_s / de_s, 3),
                       "drift_after_frames": reps * len(cycle), "drift": drift(torch, asm)}
    assert asm.status_sync() == stafem.STA_OK
    asm.close()
    if "roofline" in out:
        log(f"[bench] delta kernels: {out['roofline']['avg_launch_us']} us per frame, "
            f"{out['roofline']['frac'] * 100:.1f}% of HBM peak")
    log(f"[bench] delta: {out['delta_us_per_frame']} us/frame (exact {out['exact_us_per_frame']}), drift "
        f"{dr['max_abs']:.3e}; locality {out['locality']['delta_us_per_frame']} vs "
        f"{out['locality']['exact_us_per_frame']} us/frame, drift {out['locality']['drift']['max_abs']:.3e}")
    return out


def euler_section(torch, stafem, workloads, w, frames, cfg, args, rtol=1e-8):
    """Implicit-Euler loop of eq. (9) over the headline stream (one time step per frame,
    gravity plus a surface load, from rest): each policy's matrix update and the solve,
    timed per frame; the two policies' trajectories must agree bit for bit."""
    f = torch.from_numpy(workloads.loads_for(w, w.mask0).reshape(-1)).cuda()
    dfr = [stafem.upload_frame(ids, st) for ids, st in frames]
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(3)]
    res = {}
    traj = {}
    cg = {}
    for policy in ("stream", "rebuild"):
        asm = stafem.Assembler.from_workload(w)
        apply_config(asm, cfg)
        asm.kernel_times()
        u = torch.zeros(asm.n_rows, dtype=torch.float64, device="cuda")
        v = torch.zeros_like(u)
        upd, sol, its = [], [], []
        for ids, st in dfr:
            torch.cuda.synchronize()
            torch.cuda._sleep(200000)
            ev[0].record()
            asm.apply_edits(ids, st)
            if policy == "rebuild":
                asm.full_rebuild()
            ev[1].record()
            asm.enable_kernel_timing(True)  # the CG chunks, timed by events (both policies alike)
            it, _ = asm.euler_step(u, v, f, rtol=rtol)
            asm.enable_kernel_timing(False)
            ev[2].record()
            ev[2].synchronize()
            upd.append(ev[0].elapsed_time(ev[1]) * 1e3)
            sol.append(ev[1].elapsed_time(ev[2]) * 1e3)
            its.append(it)
        torch.cuda.synchronize()
        traj[policy] = (u.clone(), v.clone())
        kt = asm.kernel_times()
        cg[policy] = (kt.get("solve", (0, 0.0))[1], int(np.sum(its)), asm.n_rows, asm.nnz)
        assert asm.status_sync() == stafem.STA_OK
        asm.close()
        res[policy] = {"update_us_mean": round(float(np.mean(upd)), 3),
                       "solve_us_mean": round(float(np.mean(sol)), 3),
                       "frame_us_mean": round(float(np.mean(np.add(upd, sol))), 3),
                       "cg_iterations_mean": round(float(np.mean(its)), 2)}
    same = all(torch.equal(a.view(torch.int64), b.view(torch.int64)) for a, b in zip(traj["stream"], traj["rebuild"]))
    out = {"workload": "implicit Euler (M_t + h^2 K_t) u' = M_t (u + h v) + h^2 f, h = dt = 1e-2, one step per frame "
                       f"of the headline stream, Jacobi-PCG to relative residual {rtol:g}, gravity + surface load",
           "policies": res,
           "frame_speedup_stream_vs_rebuild": round(res["rebuild"]["frame_us_mean"] / res["stream"]["frame_us_mean"], 3),
           "update_speedup_stream_vs_rebuild": round(res["rebuild"]["update_us_mean"] / res["stream"]["update_us_mean"],
                                                     2),
           "trajectories_bitwise_equal": bool(same)}
    ms_cg, it_cg, n_rows, nnz = cg["stream"]
    out["roofline"] = roofline("cg_iteration", bytes_cg_iteration(n_rows, nnz) * it_cg, ms_cg * 1e-3, it_cg,
                               traffic=load_traffic("euler", ["k_cg_spmv", "k_cg_update"], per="k_cg_update"))
    if not args.no_cpu_baseline:
        # the oracle's step of eq. (9) at the frame-12 state: its matrix, lumped mass and PCG
        import oracle
        mask = w.mask0.copy()
        for ids, st in frames[:13]:
            mask[ids] = st
        pat = oracle.pattern(w.n_nodes, w.tets)
        fh = f.cpu().numpy()
        t0 = time.perf_counter()
        vals = oracle.rebuild(w.x, w.tets, w.E, w.nu, w.rho, w.dt, mask, *pat)
        m = oracle.lumped_mass(w.x, w.tets, w.rho, mask)
        _, _, it_o, _ = oracle.euler_step(*pat, vals, m, np.zeros_like(fh), np.zeros_like(fh), fh, w.dt, rtol=rtol)
        t_o = time.perf_counter() - t0
        out["cpu_baseline"] = {"value": round(t_o * 1e6, 1), "unit": "us per frame", "cores": 1, "kind": "oracle",
                               "sample": f"one step at the frame-12 state from rest (oracle matrix, lumped mass "
                                         f"and PCG, {it_o} iterations), single-threaded"}
    log(f"[bench] euler: CG {out['roofline']['avg_launch_us']} us per iteration "
        f"({out['roofline']['frac'] * 100:.1f}% of HBM peak)"
        + (f"; oracle step {out['cpu_baseline']['value'] * 1e-6:.2f} s" if "cpu_baseline" in out else ""))
    log(f"[bench] euler: stream frame {res['stream']['frame_us_mean']} us (update {res['stream']['update_us_mean']}), "
        f"rebuild frame {res['rebuild']['frame_us_mean']} us (update {res['rebuild']['update_us_mean']}), "
        f"CG {res['stream']['cg_iterations_mean']} it, same trajectory {same}")
    return out


def bytes_cg_iteration(n_rows, nnz):
    """One Jacobi-PCG iteration: the values once, one column index per 3x3 block, the row
    pointers, and 13 vector passes (product: z, previous p, new p, q, 1/diag; update: x read
    and written, new p, r read and written, q, 1/diag, z)."""
    return 8 * nnz + 4 * (nnz // 9) + 4 * (n_rows + 1) + 13 * 8 * n_rows


def bytes_adjoint(n_tets, n_active, n_nodes, n_blocks, nnz):
    """Adjoint kernels: per tet its mask, 10 positions, 10 block ids, vertex ids, E, the
    dL/dlogE and 4 vertex cotangent writes; the node coordinates; every block descriptor and
    slot cotangent once; then per node its descriptor and its diagonal segment of vertex
    cotangents (4 per tet), and dL/dx."""
    per_tet = 1 + 40 + 40 + 16 + 8 + 8 + 96
    return (n_tets * per_tet + 24 * n_nodes + 32 * n_blocks + 8 * nnz
            + 4 * n_tets * 24 + n_nodes * (4 + 32 + 24))


def gradient_section(torch, stafem, workloads, args, rtol=1e-10, reps=5):
    """The differentiation workload: the fracture state after frame 12, compliance
    L = f.u with A u = f.  Jacobi-PCG (time per iteration, bytes per iteration) and the
    adjoint kernels (dL/dlogE, dL/dx from the slot cotangents -u u^T), each against the
    HBM roofline; the GPU gradient against the oracle's complex-step adjoint for the same
    cotangents; the oracle's PCG and adjoint timed on the host."""
    w, mask, f, _, _ = workloads.make_gradient_case(args.seed)
    asm = stafem.Assembler(w.x, w.tets, w.E, w.nu, w.rho, w.dt, mask)
    fd = torch.from_numpy(f.reshape(-1)).cuda()
    u, it, rr = asm.cg_solve(fd, rtol=rtol)  # warm-up
    asm.enable_kernel_timing(True)
    asm.kernel_times()
    iters = 0
    for _ in range(reps):
        u, it, rr = asm.cg_solve(fd, rtol=rtol)
        iters += it
    ks = asm.kernel_times()
    gA = asm.slot_outer(u, u, -1.0)
    gl, gx = asm.adjoint(gA)  # warm-up
    asm.kernel_times()
    for _ in range(reps):
        gl, gx = asm.adjoint(gA)
    ka = asm.kernel_times()
    asm.enable_kernel_timing(False)
    torch.cuda.synchronize()
    n_solve, ms_solve = ks.get("solve", (0, 0.0))
    n_adj, ms_adj = ka.get("adjoint", (0, 0.0))
    it_us = ms_solve * 1e3 / max(iters, 1)
    cg_bytes = bytes_cg_iteration(asm.n_rows, asm.nnz)
    adj_bytes = bytes_adjoint(w.n_tets, int(mask.sum()), w.n_nodes, asm.n_diag_blocks + asm.n_off_blocks, asm.nnz)
    out = {"workload": "fracture 40^3 after frames 0..12, compliance f.u with A u = f (gravity + surface load)",
           "active_tets": int(mask.sum()),
           "cg": {"rtol": rtol, "iterations": it, "relres": rr, "us_per_iteration": round(it_us, 3),
                  "roofline": roofline("cg_iteration", cg_bytes * iters, ms_solve * 1e-3, iters,
                                       traffic=load_traffic("gradient", ["k_cg_spmv", "k_cg_update"],
                                                            per="k_cg_update"))},
           "adjoint": {"us": round(ms_adj * 1e3 / max(n_adj, 1), 3),
                       "roofline": roofline("k_adjoint_element+k_adjoint_nodes", adj_bytes * n_adj,
                                            ms_adj * 1e-3, n_adj,
                                            traffic=load_traffic("gradient", ["k_adjoint_element",
                                                                              "k_adjoint_nodes"]))}}
    if not args.no_cpu_baseline:
        # the CPU baseline leg: the oracle's complex-step adjoint on the same cotangents and
        # its PCG on the same system, timed on the host; the GPU gradient is compared with
        # the oracle's on the way
        import oracle

        uh = u.cpu().numpy()
        pat = oracle.pattern(w.n_nodes, w.tets)
        r = np.repeat(np.arange(asm.n_rows), np.diff(pat[0]))
        g_host = -(uh[r] * uh[pat[1]])
        t0 = time.perf_counter()
        ol, ox = oracle.adjoint(w.x, w.tets, w.E, w.nu, w.rho, w.dt, mask, pat[0], pat[1], g_host)
        t_adj = time.perf_counter() - t0
        gl_h, gx_h = gl.cpu().numpy(), gx.cpu().numpy()
        rel = lambda a, b: float(np.abs(a - b).max() / max(np.abs(b).max(), 1e-300))
        vals = asm.values().cpu().numpy()
        t0 = time.perf_counter()
        _, oit, _ = oracle.pcg(pat[0], pat[1], vals, f.reshape(-1), rtol=rtol)
        t_pcg = time.perf_counter() - t0
        out["cpu_baseline"] = {"adjoint_s": round(t_adj, 3), "pcg_s_per_iteration": round(t_pcg / max(oit, 1), 5),
                               "pcg_iterations": int(oit), "cores": 1, "kind": "oracle",
                               "sample": "one oracle adjoint (complex step, C) and one oracle PCG solve (C) on "
                                         "the same state, single-threaded",
                               "gpu_gradient_rel_err": {"dlogE": rel(gl_h, ol), "dx": rel(gx_h, ox)}}
    asm.close()
    log(f"[bench] gradient: CG {it} it, {it_us:.2f} us/it ({out['cg']['roofline']['frac'] * 100:.1f}% of HBM peak); "
        f"adjoint {out['adjoint']['us']} us ({out['adjoint']['roofline']['frac'] * 100:.1f}%)"
        + (f"; vs oracle {max(out['cpu_baseline']['gpu_gradient_rel_err'].values()):.2e}, oracle adjoint "
           f"{out['cpu_baseline']['adjoint_s']:.2f} s, PCG {out['cpu_baseline']['pcg_s_per_iteration'] * 1e3:.2f} ms/it"
           if "cpu_baseline" in out else ""))
    return out


def face_pair_count(tets):
    """Candidate tet pairs with a common face (for the face-adjacency byte count): every pair
    of tets on one sorted vertex triple."""
    tri = np.sort(tets.astype(np.int64), axis=1)
    faces = np.concatenate([tri[:, [1, 2, 3]], tri[:, [0, 2, 3]], tri[:, [0, 1, 3]], tri[:, [0, 1, 2]]])
    n = int(tri.max()) + 1
    key = (faces[:, 0] * n + faces[:, 1]) * n + faces[:, 2]
    _, counts = np.unique(key, return_counts=True)
    return int((counts * (counts - 1) // 2).sum())


# Connectivity is rebuilt from the mask periodically (paper Sec. 3.6), with no period given:
# here once per 4 frames, the frames per scenario of the paper's elasticity study (Sec. 5.2).
CONNECTIVITY_PERIOD = 4


def connectivity_section(torch, stafem, w, frames, args):
    """Connectivity rebuilt from the mask after every frame of the headline stream, for
    both adjacencies (union-find over the active tets' vertices; over the candidate face
    pairs): time per rebuild and the component count along the stream; each rebuild is
    repeated and must give identical labels."""
    asm = stafem.Assembler.from_workload(w)
    dfr = [stafem.upload_frame(ids, st) for ids, st in frames]
    lab = torch.empty(w.n_tets, dtype=torch.int32, device="cuda")
    import ctypes

    lib = stafem.load()
    fns = {"vertex": lib.sta_components, "face": lib.sta_face_components}
    if args.adjacency != "both":
        fns = {args.adjacency: fns[args.adjacency]}
    if "face" in fns:
        asm.components("face")  # the face pairs are found once per context, outside the timing
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    res = {a: {"times": [], "counts": [], "stable": True} for a in fns}
    for ids, st in dfr:
        asm.apply_edits(ids, st)
        for adj, fn in fns.items():
            torch.cuda.synchronize()
            torch.cuda._sleep(200000)
            ev[0].record()
            code = fn(asm.handle, ctypes.c_void_p(lab.data_ptr()), None,
                      ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
            ev[1].record()
            ev[1].synchronize()
            assert code == stafem.STA_OK
            r = res[adj]
            r["times"].append(ev[0].elapsed_time(ev[1]) * 1e3)
            again, k = asm.components(adj)
            r["stable"] = r["stable"] and bool(torch.equal(again, lab))
            r["counts"].append(k)
    n_pairs = face_pair_count(w.tets)
    asm.close()
    period = CONNECTIVITY_PERIOD
    out = {"workload": "components of the active tets rebuilt after every frame of the headline stream, "
                       "shared-vertex and shared-face adjacency; cost per frame when rebuilt every "
                       f"{period} frames", "period_frames": period}
    oracle_s = {}
    if not args.no_cpu_baseline:
        # the oracle's components at the peak frame's mask (library connected_components)
        from oracle import connectivity as C
        mask = w.mask0.copy()
        for ids, st in frames[:13]:
            mask[ids] = st
        t0 = time.perf_counter()
        C.components(w.n_nodes, w.tets, mask)
        oracle_s["vertex"] = time.perf_counter() - t0
        pairs = C.face_pairs(w.tets)
        t0 = time.perf_counter()
        C.face_components(w.tets, mask, pairs)
        oracle_s["face"] = time.perf_counter() - t0
    for adj, r in res.items():
        c = r["counts"]
        med = float(np.median(r["times"]))
        out[adj] = {"rebuild_us_median": round(med, 3),
                    "rebuild_us_max": round(float(np.max(r["times"])), 3),
                    "components_initial": c[0], "components_max": int(max(c)), "components_final": c[-1],
                    "repeat_labels_identical": r["stable"],
                    "us_per_frame_at_period": round(med / period, 3)}
        if adj == "vertex" or n_pairs:
            nb = bytes_connectivity_pass(w.n_tets, w.n_nodes, n_pairs if adj == "face" else 0)
            # the first kernel runs once per rebuild: the unit of the counted bytes
            ks = (["k_cc_init", "k_cc_windows", "k_cc_roots", "k_cc_label"] if adj == "vertex"
                  else ["k_ccf_windows", "k_ccf_cross", "k_cc_roots", "k_ccf_label"])
            out[adj]["roofline"] = roofline(f"connectivity ({adj}), one-pass lower bound", nb, med * 1e-6, 1,
                                            traffic=load_traffic(f"connectivity_{adj}", ks, per=ks[0]))
        if adj in oracle_s:
            out[adj]["cpu_baseline"] = {"value": round(oracle_s[adj] * 1e6, 1), "unit": "us per rebuild",
                                        "cores": 1, "kind": "oracle",
                                        "sample": "components at the frame-12 mask (library connected_components"
                                                  + (" over the candidate face pairs, pairs found beforehand)"
                                                     if adj == "face" else " over the vertex graph)")}
        log(f"[bench] connectivity ({adj}): {out[adj]['rebuild_us_median']} us per rebuild, components "
            f"{c[0]} -> {max(c)} -> {c[-1]}")
    return out


SECTIONS = ("delta", "proxy", "euler", "connectivity", "gradient", "refinement", "batch")


def compact_line(out, detail_path):
    """The default line: the headline numbers and a short summary of each section (the
    full report is in the detail file)."""
    pf = out.get("per_frame", {})
    line = {k: out[k] for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step",
                                "higher_is_better", "scaling", "vs_baseline", "dtype", "data")}
    line["config"] = {k: out["config"][k] for k in ("workload", "n_tets", "nnz", "frames_per_step",
                                                    "edits_per_step", "touched_slots_per_step", "seed")}
    line["config"]["frame_mode"] = f"one launch up to {ONE_LAUNCH_EDITS} edits, " + (
        "one with a grid barrier above" if out["tuned_config"]["fused"] else "two above")
    line["timing_mode"] = out["timing_mode"]
    if pf:
        line["per_frame_us"] = pf["us"]
        line["stream_vs_rebuild"] = pf["ratios"]
    line["roofline"] = out["roofline"]
    if "frame_roofline" in out:
        line["frame_roofline"] = out["frame_roofline"]
    if "roofline_rebuild" in out:
        rr = out["roofline_rebuild"]
        line["roofline_rebuild"] = {"element_frac": rr["element"]["frac"], "reduce_frac": rr["reduce"]["frac"],
                                    "whole_frac": rr["whole_frac"], "kernel_us": rr["rebuild_us_mean"]}
    if "hbm_measured" in out:
        line["hbm_measured_GBs"] = out["hbm_measured"]
    if "cpu_baseline" in out:
        cb = dict(out["cpu_baseline"])
        cb["sample"] = cb["sample"].split(" (frames")[0]
        cb["multicore"] = {k: v for k, v in cb["multicore"].items() if k != "sample"}
        line["cpu_baseline"] = cb
    line["parity"] = out["parity"]
    sec = {}
    for name in ("refinement", "batch"):
        if name in out:
            o = out[name]
            sec[name] = {"us_per_frame": o["stream_pipelined_us_per_frame"], "rebuild_us": o["rebuild_us_mean"],
                         "ratio": o["rebuild_vs_pipelined_frame"], "frac": o["roofline"]["frac"],
                         "mismatching_frames": o["parity"]["mismatching_frames"]}
            if "one_launch" in o:
                ol = o["one_launch"]
                sec[name]["one_launch_us_per_frame"] = ol["stream_pipelined_us_per_frame"]
                sec[name]["one_launch_mismatching_frames"] = ol["parity"]["mismatching_frames"]
    if "delta" in out:
        d = out["delta"]
        sec["delta"] = {"us_per_frame": d["delta_us_per_frame"], "exact_us_per_frame": d["exact_us_per_frame"],
                        "drift_max_abs": d["drift"]["max_abs"]}
    if "proxy" in out:
        p = out["proxy"]
        sec["proxy"] = {"us_per_frame": p["stream_pipelined_us_per_frame"], "rebuild_us": p["rebuild_us_median"],
                        "mismatching_frames": p["parity"]["mismatching_frames"]}
    if "euler" in out:
        e = out["euler"]
        sec["euler"] = {"frame_us_stream": e["policies"]["stream"]["frame_us_mean"],
                        "frame_us_rebuild": e["policies"]["rebuild"]["frame_us_mean"],
                        "cg_frac": e["roofline"]["frac"], "bitwise_same_trajectory": e["trajectories_bitwise_equal"]}
    if "gradient" in out:
        g = out["gradient"]
        sec["gradient"] = {"cg_us_per_iteration": g["cg"]["us_per_iteration"], "cg_frac": g["cg"]["roofline"]["frac"],
                           "adjoint_us": g["adjoint"]["us"], "adjoint_frac": g["adjoint"]["roofline"]["frac"]}
    if "connectivity" in out:
        c = out["connectivity"]
        sec["connectivity"] = {a: {"rebuild_us": c[a]["rebuild_us_median"],
                                   "us_per_frame_at_period": c[a]["us_per_frame_at_period"]}
                               for a in ("vertex", "face") if a in c}
        sec["connectivity"]["period_frames"] = c["period_frames"]
    if sec:
        line["sections"] = sec
    line["detail"] = detail_path
    text = json.dumps(line)
    if len(text) > 4000:  # keep the line short: the sections are in the detail file
        line.pop("sections", None)
        text = json.dumps(line)
    return text


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--reps", type=int, default=40,
                    help="repetitions per frame for the per-frame breakdown (half warm, half after a cache flush)")
    ap.add_argument("--seed", type=int, default=0)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-extras", action="store_true", help="skip the secondary workloads")
    ap.add_argument("--adjacency", default="both", choices=("both", "vertex", "face"),
                    help="connectivity section: which adjacencies to rebuild")
    ap.add_argument("--sections", default="all",
                    help="secondary sections to run: all, or a comma list of " + ",".join(SECTIONS)
                         + " (with --quick, only the named ones; default none)")
    ap.add_argument("--no-tune", action="store_true", help="keep the default configuration")
    ap.add_argument("--config", default=None,
                    help="force fused,rebuild_qd,rebuild_qo,stream_qd,stream_qo,grid_cap,rebuild_nt (skips tuning)")
    ap.add_argument("--cpu-sample", type=int, default=48, help="oracle rebuilds in the CPU baseline sample")
    ap.add_argument("--quick", action="store_true",
                    help="headline timed steps, 3 rebuilds and a 512 MiB reference copy only (for profiler runs)")
    ap.add_argument("--detail", default="bench_detail.json",
                    help="file for the full report (per-frame rows, autotuner report, every section)")
    args = ap.parse_args()

    world = int(os.environ.get("WORLD_SIZE", "1"))
    if args.gpus != 1 or world != 1:
        print(json.dumps({"error": "this implementation runs on one GPU only; sharding over several GPUs is "
                                   "described, not implemented", "n_gpus": args.gpus}))
        sys.exit(2)

    import torch
    from paper_2605_11673_amd import stafem, workloads

    torch.cuda.set_device(0)
    t0 = time.time()
    w = workloads.make_fracture(args.seed, n=40)
    frames = list(w.frames) + workloads.merge_stream(w.frames)
    asm = stafem.Assembler.from_workload(w)
    log(f"[bench] fracture 40^3: {w.n_tets} tets, nnz {asm.nnz}, {len(frames)} frames, setup {time.time() - t0:.1f}s")
    s = Stream(torch, asm, frames, w.n_tets, w.n_nodes, w.mask0)
    tune_report = None
    if args.config:
        asm.set_config(*[int(v) for v in args.config.split(",")])
        log(f"[bench] forced: {asm.get_config()}")
    elif not args.no_tune:
        cfg, tune_report = s.tune(12)
        log(f"[bench] tuned: {cfg}")
    stats, mismatches = s.stats_pass(check_parity=not args.quick)
    slots_per_step = int(sum(st["touched_slots"] for st in stats))
    edits_per_step = int(sum(st["edits"] for st in stats))
    ktimes, eager_s, step_s = s.timed(args.steps, args.warmup)
    value = slots_per_step / step_s
    log(f"[bench] graph {step_s * 1e3:.3f} ms/step ({value:.4g} slots/s), host-launched {eager_s * 1e3:.3f} ms/step")
    kern, roof = s.stream_roofline(ktimes, args.steps)
    frame_us = step_s * 1e6 / len(frames)
    alg_step = sum(alg_frame(st) for st in stats)

    out = {
        "metric": METRIC, "value": value, "unit": "touched slots/s", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": step_s * 1e3, "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "f64", "data": "synthetic",
        "config": {"workload": "fracture+merge stream, Kuhn cube 40^3x6 (384000 tets, 68921 nodes), "
                               "24 Voronoi fracture frames + 24 reinsertion frames, FP64",
                   "n_tets": w.n_tets, "n_nodes": w.n_nodes, "nnz": asm.nnz, "frames_per_step": len(frames),
                   "edits_per_step": edits_per_step, "touched_slots_per_step": slots_per_step, "seed": args.seed},
        "tuned_config": {**asm.get_config(),
                         "buckets": {k: asm.bucket_map(k) for k in ("rebuild", "stream")}},
        "timing_mode": "whole step captured as one HIP graph, replayed",
        "host_launched": {"ms_per_step": eager_s * 1e3, "value": slots_per_step / eager_s},
        "stream_pipelined_us_per_frame": round(frame_us, 3),
        "roofline": roof,
        # a frame's kernels as one unit: the method's bytes per frame over the pipelined frame time
        "frame_roofline": {"kernels": "every kernel of a frame (pipelined)", "bound": "hbm",
                           "achieved": round(alg_step / step_s / 1e9, 2), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                           "frac": round(alg_step / step_s / 1e9 / HBM_PEAK_GBS, 5),
                           "algorithmic_bytes_per_frame": round(alg_step / len(frames), 1)},
        "kernels": kern,
        "parity": {"frames_checked": 0 if args.quick else len(frames), "mismatching_frames": mismatches,
                   "check": "GPU streaming values bitwise equal to GPU full rebuild at every frame"},
    }
    if args.quick:
        for _ in range(3):
            asm.full_rebuild()
        # reference copy of known size (512 MiB read + 512 MiB written, larger than any other
        # copy the bench makes) for counter scaling
        src = torch.ones(1 << 26, dtype=torch.float64, device="cuda")
        dst = torch.empty_like(src)
        for _ in range(3):
            dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst
    if not args.quick:
        out["latency_floor"] = stafem.latency_probe()
        out["barrier_vs_boundary"] = stafem.barrier_probe()
        log(f"[bench] grid barrier vs kernel boundary (us per graph-replayed unit): {out['barrier_vs_boundary']}")
        out["hbm_measured"] = {k: round(x, 1) for k, x in stafem.bandwidth_probe().items()}
        rr = s.rebuild_roofline()
        rb = rr["element"]["algorithmic_bytes_per_launch"] + rr["reduce"]["algorithmic_bytes_per_launch"]
        rr["whole_frac"] = round(rb / (rr["rebuild_us_mean"] * 1e-6) / 1e9 / HBM_PEAK_GBS, 5)
        out["roofline_rebuild"] = rr
        reb_pipe = s.rebuild_pipelined()
        pfr = s.per_frame(args.reps)
        out["per_frame_detail"] = pfr
        out["per_frame"] = {
            "us": {"stream_pipelined": round(frame_us, 3), "rebuild_pipelined": round(reb_pipe, 3),
                   "stream_warm_median": pfr["stream_us_per_frame"]["median"],
                   "rebuild_warm_median": pfr["rebuild_us"]["median"],
                   "stream_cold_median": (pfr["stream_cold_us_per_frame"] or {}).get("median"),
                   "rebuild_cold_median": pfr["rebuild_cold_us"]["median"],
                   "stream_warm_max": pfr["stream_us_per_frame"]["max"]},
            "ratios": {"pipelined": round(reb_pipe / frame_us, 2),
                       "warm_median": pfr["stream_vs_rebuild"]["median_ratio"],
                       "cold_median": round(pfr["rebuild_cold_us"]["median"]
                                            / (pfr["stream_cold_us_per_frame"] or {"median": np.nan})["median"], 2),
                       "peak_frame_warm": pfr["stream_vs_rebuild"]["peak_frame_ratio"],
                       "target": 20.0}}
        out["autotune_report"] = tune_report
        log(f"[bench] per frame: stream {frame_us:.2f} us pipelined / {pfr['stream_us_per_frame']['median']} us "
            f"warm median; rebuild {reb_pipe:.1f} us pipelined / {pfr['rebuild_us']['median']} us warm median; "
            f"ratios {out['per_frame']['ratios']}")
    asm.close()
    if not args.quick and not args.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline(args, w, frames, stats)
        cb = out["cpu_baseline"]
        log(f"[bench] cpu baseline: {cb['rebuild_s_per_frame']} s per oracle rebuild (1 thread), "
            f"{cb['multicore']['rebuild_s_per_frame']} s on {cb['multicore']['cores']} threads "
            f"(bitwise equal: {cb['multicore']['bitwise_equal_to_serial']}); {cb['cpu_model']}, nproc {cb['nproc']}")
    if args.sections == "all":
        sections = [] if (args.quick or args.no_extras) else list(SECTIONS)
    else:
        sections = [x for x in args.sections.split(",") if x]
        bad = [x for x in sections if x not in SECTIONS]
        if bad:
            raise SystemExit(f"unknown sections {bad}; choose from {SECTIONS}")
        if args.no_extras:
            sections = []
    if "delta" in sections:
        out["delta"] = delta_section(torch, stafem, w, frames, out["tuned_config"], step_s, args, stats,
                                     out.get("cpu_baseline", {}).get("rebuild_s_per_frame"))
    if "proxy" in sections:
        out["proxy"] = proxy_section(torch, stafem, w, frames, args)
    if "euler" in sections:
        out["euler"] = euler_section(torch, stafem, workloads, w, frames, out["tuned_config"], args)
    if "connectivity" in sections:
        out["connectivity"] = connectivity_section(torch, stafem, w, frames, args)
    if "gradient" in sections:
        out["gradient"] = gradient_section(torch, stafem, workloads, args)
    if "refinement" in sections:
        r = workloads.make_refinement(args.seed)
        rf = r.frames[:24]
        rframes = rf + [(ids, (1 - st).astype(np.uint8)) for ids, st in reversed(rf)]
        peak = int(np.argmax([len(ids) for ids, _ in rf]))
        ra = stafem.Assembler.from_workload(r)
        out["refinement"] = secondary(torch, "refinement 20^3 x 8 children", ra, rframes, r.n_tets, r.n_nodes,
                                      r.mask0, peak, args,
                                      "red-refinement superset 432000 tets (48000 parents + 8 children each), "
                                      "24 refine frames (0.1-2% of parents swapped for children) then the same "
                                      "swaps undone in reverse (merge), FP64", workload="refinement")
        ra.close()
    if "batch" in sections:
        ws = workloads.make_batch(args.seed)
        b = stafem.Batch.from_workloads(ws)
        off = b.offsets()["tet"]
        bfr = []
        for t in range(24):
            bfr.append((np.concatenate([wj.frames[t][0].astype(np.int64) + off[j]
                                        for j, wj in enumerate(ws)]).astype(np.int32),
                        np.concatenate([wj.frames[t][1] for wj in ws]).astype(np.uint8)))
        bframes = bfr + [(ids, (1 - st).astype(np.uint8)) for ids, st in reversed(bfr)]
        mask0 = np.ones(b.n_tets, dtype=np.uint8)
        out["batch"] = secondary(torch, "batch of 64 meshes", b, bframes, b.n_tets, b.n_nodes, mask0, 12, args,
                                 f"64 jittered Kuhn cubes of 6n^3 tets (n log-uniform, {b.n_tets} tets in all), "
                                 "each with its own 24-frame fracture stream, then reinsertion; one context, "
                                 "one frame = all meshes' edits, FP64", fused_too=True, workload="batch")
        b.close()
    if args.detail:
        d = os.path.dirname(args.detail)
        if d:
            os.makedirs(d, exist_ok=True)
        with open(args.detail, "w") as f:
            json.dump(out, f, indent=1)
    print(compact_line(out, args.detail), flush=True)


if __name__ == "__main__":
    main()
