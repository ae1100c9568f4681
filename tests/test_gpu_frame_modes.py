"""Which launches frames take, as the kernel times and the trace tell it, and the frame with a grid
barrier where it is asked for: its errors undo what the first phase wrote."""
import ctypes
import json
import os

import numpy as np
import pytest
import torch

import oracle
from paper_2605_11673_amd import workloads as W

pytestmark = pytest.mark.gpu
POLLS = 1 << 25  # a limit that the caller sets asks for the barrier that it limits


def S():
    from paper_2605_11673_amd import stafem
    return stafem


def launches(asm):
    t = asm.kernel_times()
    return {k: t[k][0] for k in ("frame", "edits", "touched") if k in t}


def traced(w, path):
    os.environ["STA_TRACE"] = str(path)
    try:
        return S().Assembler.from_workload(w)
    finally:
        os.environ.pop("STA_TRACE")


def test_trace_names_the_launches(tmp_path):
    """2,304 and 2,305 edits, each with fused 0 and 1, a device count, and a limit of polls."""
    Sm = S()
    w = W.make_fracture(seed=6, n=10, counts=[50])
    asm = traced(w, tmp_path / "trace.jsonl")
    asm.enable_kernel_timing(True)
    want, ran = [], []
    n = torch.tensor([7], dtype=torch.int32, device="cuda")
    one, two, barrier = "one launch", "two launches", "one launch with a grid barrier"
    for fused, polls, k, mode in ((0, 0, 2304, one), (0, 0, 2305, two), (1, 0, 2304, one), (1, 0, 2305, barrier),
                                  (1, POLLS, 10, barrier), (0, POLLS, 10, one)):
        asm.set_config(fused=fused)
        asm.set_barrier_spin_limit(polls)
        frame = Sm.upload_frame(np.arange(k, dtype=np.int32), np.ones(k, np.uint8))
        asm.kernel_times()
        asm.apply_edits(*frame)
        asm.apply_edits_dev(*frame, n)
        ran.append(launches(asm))
        want += [mode, mode]
        assert ran[-1] == ({"edits": 2, "touched": 2} if mode == two else {"frame": 2}), (fused, polls, k)
    asm.apply_edits_delta(*frame)
    assert asm.status_sync() == Sm.STA_OK
    asm.close()
    lines = [json.loads(l) for l in (tmp_path / "trace.jsonl").read_text().splitlines()]
    assert [l["frame_mode"] for l in lines] == want + [two]


@pytest.mark.parametrize("k", [1, 40, 2304, 3000])
def test_barrier_frame_errors_roll_back(k):
    """A duplicate, a tet and a state out of range in a list of valid edits: nothing changes, and the next
    frame runs."""
    Sm = S()
    w = W.make_fracture(seed=k, n=9, counts=[10])
    pat = oracle.pattern(w.n_nodes, w.tets)
    asm = Sm.Assembler.from_workload(w)
    asm.set_config(fused=1)
    asm.set_barrier_spin_limit(POLLS)
    asm.enable_kernel_timing(True)
    asm.kernel_times()
    g = np.random.default_rng(k)
    ids = g.permutation(w.n_tets)[:k].astype(np.int32)
    zero = np.zeros(k + 1, np.uint8)
    before = asm.values()
    for bad, state, code in ((ids[0], 0, Sm.STA_EDUP), (w.n_tets, 0, Sm.STA_ERANGE), (-1, 0, Sm.STA_ERANGE),
                             (int(np.setdiff1d(np.arange(w.n_tets), ids)[0]), 2, Sm.STA_ERANGE)):
        st = zero.copy()
        st[-1] = state
        asm.apply_edits(*Sm.upload_frame(np.append(ids, bad).astype(np.int32), st))
        assert asm.status_sync() == code
        assert torch.equal(asm.values().view(torch.int64), before.view(torch.int64)), code
        assert asm.last_frame_stats()["rolled_back"] == 1
        assert asm.audit() == {"values_differing": 0, "tets_differing": 0}
    asm.apply_edits(*Sm.upload_frame(ids, zero[:k]))
    assert asm.status_sync() == Sm.STA_OK and launches(asm) == {"frame": 5}
    mask = w.mask0.copy()
    mask[ids] = 0
    got = asm.values().cpu().numpy()
    assert np.array_equal(got.view(np.uint64), oracle.rebuild_workload(w, mask, pat).view(np.uint64))
    asm.close()


@pytest.mark.parametrize("cached", [False, True])
def test_autotune_keeps_the_mode_that_it_cannot_tell(tmp_path, monkeypatch, cached):
    """A frame of one launch in either mode leaves fused and the grid cap as they are, with a tuning file
    that an earlier choice left or without."""
    Sm = S()
    w = W.make_fracture(seed=3, n=12, counts=[300, 50])
    asm = Sm.Assembler.from_workload(w)
    frame = Sm.upload_frame(*w.frames[0])
    path = tmp_path / "tune.txt"
    monkeypatch.setenv("STA_TUNE_CACHE", str(path))
    if cached:  # a file in which fused is 1 with the cap 256
        first = asm.autotune(*frame, reps=2)
        assert "chosen" in first
        key, values = path.read_text().splitlines()[0].split("|")
        v = values.split()
        v[0], v[5] = "1", "256"
        path.write_text(f"{key}| {' '.join(v)}\n")
    for fused, cap in ((0, 0), (1, 77)):
        asm.set_config(fused=fused, grid_cap=cap)
        rep = asm.autotune(*frame, reps=2)
        assert rep.startswith("cached") == (cached or (fused, cap) != (0, 0)), rep
        cfg = asm.get_config()
        assert (cfg["fused"], cfg["grid_cap"]) == (fused, cap), rep
    asm.close()


def test_autotune_tells_the_modes_of_a_long_list():
    """2,305 edits: two launches and the grid barrier under its caps are timed, each by itself."""
    Sm = S()
    w = W.make_fracture(seed=3, n=12, counts=[10])
    asm = Sm.Assembler.from_workload(w)
    rep = asm.autotune(*Sm.upload_frame(np.arange(2305, dtype=np.int32), np.zeros(2305, np.uint8)), reps=2)
    assert sum(l.startswith("frame ") for l in rep.splitlines()) == 4, rep
    asm.close()


def test_grouped_rebuild_launches_what_it_needs():
    """A batch rebuilt in groups and without large nodes: two launches a group, three while timed."""
    Sm = S()
    ws = W.make_batch(seed=0)
    b = Sm.Batch.from_workloads(ws)
    b.enable_kernel_timing(True)
    b.kernel_times()
    b.full_rebuild()
    times = b.kernel_times()
    b.enable_kernel_timing(False)
    groups = times["element"][0]
    assert groups > 1 and times["reduce"][0] == 2 * groups
    hip = ctypes.CDLL("libamdhip64.so.7")
    side = torch.cuda.Stream()
    handle, graph, nodes = ctypes.c_void_p(side.cuda_stream), ctypes.c_void_p(), ctypes.c_size_t()
    torch.cuda.synchronize()
    assert hip.hipStreamBeginCapture(handle, 2) == 0
    b.full_rebuild(stream=side)
    assert hip.hipStreamEndCapture(handle, ctypes.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(nodes)) == 0
    assert hip.hipGraphDestroy(graph) == 0
    assert nodes.value == 2 * groups, (nodes.value, groups)
    b.close()
