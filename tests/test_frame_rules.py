"""Which launches a frame takes: the rules, compiled on their own."""
import ctypes

import numpy as np
import pytest

from paper_2605_11673_amd import workloads as W
from tests.hostcode import compiled

SOURCE = r"""
#include "frame_rules.h"
using namespace sta;
extern "C" int route(long long edits, long long longest, int fused, int limited)
{
    return (int)frame_route(edits, longest, fused != 0, limited != 0);
}
extern "C" long long proxy_most() { return kProxyOnceRounds; }
extern "C" long long edge_rounds(long long t) { return proxy_edge_rounds(t); }
extern "C" long long vertex_rounds(long long t, long long c) { return proxy_vertex_rounds(t, c); }
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    lib = compiled(tmp_path_factory.mktemp("rules"), SOURCE)
    for f in ("proxy_most", "edge_rounds", "vertex_rounds"):
        getattr(lib, f).restype = ctypes.c_longlong
    return lib


def incidence(w):
    """Most tets of a vertex and of an edge, most columns of a row."""
    t = w.tets.astype(np.int64)
    e = np.sort(t[:, [[0, 1], [0, 2], [0, 3], [1, 2], [1, 3], [2, 3]]].reshape(-1, 2), 1)
    keys, of_edge = np.unique(e[:, 0] * w.n_nodes + e[:, 1], return_counts=True)
    columns = np.bincount(np.concatenate([keys // w.n_nodes, keys % w.n_nodes])) + 1
    return int(np.bincount(t.reshape(-1)).max()), int(of_edge.max()), int(columns.max())


def test_proxy_frames_of_one_launch(rules):
    """The workloads' meshes take one launch; a vertex or an edge of very many tets does not."""
    ll = ctypes.c_longlong
    for w in (W.make_fracture(0, 6, counts=[1]), W.make_refinement(0, 4, 1)):
        of_vertex, of_edge, columns = incidence(w)
        assert rules.vertex_rounds(ll(of_vertex), ll(columns)) <= rules.proxy_most()
        assert rules.edge_rounds(ll(of_edge)) <= rules.proxy_most()
    for tets, columns in ((200, 122), (5000, 2602), (160, 65), (1, 1025)):
        assert rules.vertex_rounds(ll(tets), ll(columns)) > rules.proxy_most(), tets
    assert rules.edge_rounds(ll(121)) > rules.proxy_most()


ONCE, TWO, BARRIER = 0, 1, 2


@pytest.mark.parametrize("edits,longest,fused,limited,want", [
    (0, 24, 0, 0, ONCE), (2304, 48, 0, 0, ONCE), (2305, 48, 0, 0, TWO), (2305, 48, 1, 0, BARRIER), (2304, 48, 1, 0, ONCE),
    (1, 1024, 0, 0, ONCE), (1, 1025, 0, 0, TWO), (2304, 5000, 0, 0, TWO), (10, 5000, 1, 0, BARRIER),
    (10, 24, 1, 1, BARRIER), (10, 24, 0, 1, ONCE), (5000, 24, 0, 1, TWO)])
def test_frame_route(rules, edits, longest, fused, limited, want):
    ll = ctypes.c_longlong
    assert rules.route(ll(edits), ll(longest), fused, limited) == want
