"""Row pointers of the assembled matrix, an exclusive scan of the rows' block
counts, for row counts around the scan's turns (4096 each) and the largest
that one workgroup scans (16384): against counts from the tetrahedra of a bar
far above the ground."""
import numpy as np
import pytest

from gpu_util import to_np
from test_gpu_wide_queries import _block

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [8, 4092, 4096, 4100, 8192, 16380, 16384, 16388])
def test_row_pointers(rows):
    from paper_2609_25653_amd import Sim
    sc = _block(rows // 4 - 1)
    assert len(sc["X"]) == rows
    sc["X"] = sc["X"] + [0.0, 0.0, 1.0]
    sim = Sim(sc)
    sim.begin_step(0)
    rp, col, _ = sim.hessian_bsr(sim.state()[0])
    i, j = (np.repeat(sc["tets"], 4, axis=1).ravel(), np.tile(sc["tets"], (1, 4)).ravel())
    edges = np.unique(i.astype(np.int64) * rows + j)
    want = np.concatenate([[0], np.cumsum(np.bincount(edges // rows, minlength=rows))])
    assert np.array_equal(to_np(rp), want) and len(col) == want[-1]
