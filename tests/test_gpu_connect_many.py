"""Vertex connectivity of more windows of tets than the device has compute units."""
import numpy as np
import pytest

from oracle import connectivity as C
from paper_2605_11673_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shuffle", [False, True])
@pytest.mark.parametrize("windows", [256, 257])
@pytest.mark.parametrize("part", [0.35, 0.01])
def test_labels(windows, shuffle, part):
    """262,144 tets and one more; a hundredth of them active make some thousand pieces."""
    from paper_2605_11673_amd import stafem as Sm
    full = W.make_fracture(seed=2, n=36, counts=[10])
    g = np.random.default_rng(windows)
    m = 256 * 1024 + (windows - 256)
    pick = np.sort(g.permutation(full.n_tets)[:m]) if not shuffle else g.permutation(full.n_tets)[:m]
    mask = (g.uniform(size=m) < part).astype(np.uint8)
    w = W.Workload("many", full.x, full.tets[pick], full.E[pick], mask)
    asm = Sm.Assembler.from_workload(w)
    lab, k = asm.components()
    ref, rk = C.components(w.n_nodes, w.tets, mask)
    assert np.array_equal(lab.cpu().numpy(), ref) and k == rk
    asm.close()
