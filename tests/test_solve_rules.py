"""How a solve is launched: the iterations between two looks at its residual, and which
systems one workgroup solves."""
import ctypes
import math

import numpy as np
import pytest

import oracle
from paper_2605_11673_amd import workloads as W
from tests.hostcode import compiled

SOURCE = r"""
#include "solve_rules.h"
extern "C" int chunk(double rr, double bb, double tol2, int launched) { return sta::cg_chunk(rr, bb, tol2, launched); }
extern "C" int small_pays(long long nodes, const int32_t* rowptr) { return sta::cg_small_pays(nodes, rowptr); }
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    return compiled(tmp_path_factory.mktemp("rules"), SOURCE)


@pytest.fixture(scope="module")
def chunk(rules):
    rules.chunk.argtypes = [ctypes.c_double, ctypes.c_double, ctypes.c_double, ctypes.c_int]
    return rules.chunk


@pytest.mark.parametrize("ratio", [1.0, 1.5, 30.0, 1e8, math.inf, math.nan])
@pytest.mark.parametrize("tol", [1e-12, 0.0])
def test_no_rate_to_go_by(chunk, ratio, tol):
    """A residual at or above |b|, infinite or not a number: a look every 16 iterations."""
    for launched in (16, 48, 1000):
        assert chunk(ratio * 3.0, 3.0, tol * tol * 3.0, launched) == 16


def test_a_falling_residual(chunk):
    for launched in (16, 32, 100, 1000, 100000):
        most = min(2 * launched, 256)
        assert chunk(1e-3, 1.0, 0.0, launched) == most  # never to be reached
        assert chunk(1.0 - 1e-9, 1.0, 1e-24, launched) == most
        left = math.log(0.99) / (math.log(1e-23) / launched)  # all but there
        assert chunk(1e-23, 1.0, 0.99e-23, launched) == max(4, math.ceil(left))
        rate = math.log(1e-12) / launched
        assert chunk(1e-12, 1.0, math.exp(rate * (launched + 10.5)), launched) == 11


@pytest.mark.parametrize("rise", [0, 100, 1700])
def test_looks_of_a_solve(chunk, rise):
    """A residual above |b| for `rise` iterations, then falling: no more looks than one per 16, and no
    more than twice the iterations that have run, or 256, past the end."""
    fall = np.linspace(2.0, math.log(1e-24), 800)
    log_rr = np.concatenate([2.0 + np.sin(np.arange(rise)) ** 2, fall])
    launched, looks, n = 0, 0, 16
    while True:
        launched, looks = launched + n, looks + 1
        if launched >= len(log_rr):
            break
        n = chunk(math.exp(log_rr[launched]), 1.0, 1e-24, launched)
    assert looks <= math.ceil(len(log_rr) / 16) and launched - len(log_rr) <= 256


def small_pays(rules, degrees):
    """degrees: neighbours of each node, itself included."""
    rowptr = np.concatenate([[0], np.cumsum(np.repeat(3 * np.asarray(degrees), 3))]).astype(np.int32)
    return bool(rules.small_pays(ctypes.c_longlong(len(degrees)), rowptr.ctypes.data_as(ctypes.c_void_p)))


def test_one_workgroup_for_a_small_system(rules):
    for w in (W.make_cube(0, 4), W.make_fracture(0, 6, counts=[1]), W.make_refinement(0, 3, 1)):
        rowptr = oracle.pattern(w.n_nodes, w.tets)[0]
        assert rules.small_pays(ctypes.c_longlong(w.n_nodes), rowptr.ctypes.data_as(ctypes.c_void_p)), w.name
    assert small_pays(rules, [15] * 352) and not small_pays(rules, [15] * 353)
    assert small_pays(rules, [0] * 10) and small_pays(rules, [])
    assert small_pays(rules, [12] * 300 + [320])  # one vertex with many neighbours
    for n in (100, 200, 350):  # nearly all of them neighbours of each other
        assert not small_pays(rules, [min(n, 170)] * n), n
    assert small_pays(rules, [40] * 40)
