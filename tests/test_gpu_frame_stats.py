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
