"""Statistics of frames are counted on the device with few atomics and few waits: the values after every
kind of frame, and what a call costs."""
import time

import numpy as np
import pytest
import torch

from paper_2605_11673_amd import workloads as W

pytestmark = pytest.mark.gpu


def S():
    from paper_2605_11673_amd import stafem
    return stafem


def seconds(f, reps=20):
    best = np.inf
    for _ in range(reps):
        t = time.perf_counter()
        f()
        best = min(best, time.perf_counter() - t)
    return best


def test_a_call_does_not_grow_with_the_frame():
    """59 us after 10 edits and 62 after 2,304; 580 with an atomic for each block."""
    Sm = S()
    w = W.make_fracture(seed=0, n=24, counts=[10])
    asm = Sm.Assembler.from_workload(w)
    times = []
    for k in (10, 2304):
        frame = Sm.upload_frame(np.arange(k, dtype=np.int32) * 7, np.zeros(k, np.uint8))
        asm.apply_edits(*frame)
        assert asm.last_frame_stats()["changed"] == k
        times.append(seconds(asm.last_frame_stats))
        asm.apply_edits(frame[0], 1 - frame[1])
    asm.close()
    assert times[1] < 3 * times[0], times


def test_proxy_statistics_of_alternating_frames():
    """Frames of one and of two launches in turn, refused ones among them, asked for twice each."""
    Sm = S()
    w = W.make_fracture(seed=1, n=10, counts=[10])
    px = Sm.Proxy.from_workload(w, W.PROXY_EPS)
    g = np.random.default_rng(3)
    mask = w.mask0.copy()
    _, counts, _ = px.state()
    for k in (5, 2400, 2304, 1, 3000, 64):
        ids = g.permutation(w.n_tets)[:k].astype(np.int32)
        st = 1 - mask[ids]
        px.apply_edits(*Sm.upload_frame(ids, st))
        mask[ids] = st
        before, (_, counts, _) = counts.clone(), px.state()
        flips = int(((before > 0) != (counts > 0)).sum())
        for _ in range(2):
            got = px.last_frame_stats()
            assert (got["edits"], got["changed"]) == (k, k)
            if k <= 2304:  # two launches count the changes on the way too
                assert got["transitions"] == flips
        twice = np.append(ids[:2], ids[0]).astype(np.int32)
        px.apply_edits(*Sm.upload_frame(twice, np.zeros(len(twice), np.uint8)))
        assert px.status_sync() == Sm.STA_EDUP
        assert px.last_frame_stats()["changed"] == 0
    px.close()
