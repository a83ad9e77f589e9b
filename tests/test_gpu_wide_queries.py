"""Broad-phase queries that meet most of a scene's tree (an edge or a vertex
of the ground's two large triangles, of a rigid box) leave the traversal and
scan the leaves 64 at a time (k_wide).  Pair sets and CCD bounds against the
oracle's, exactly, for primitive counts around the blocks' and the
workgroup's sizes, alone and batched (each scene's blocks start anew)."""
import numpy as np
import pytest

import ipcscenes as S
import oracle as O
from gpu_util import to_np

pytestmark = pytest.mark.gpu


def _block(n):
    """n x 1 x 1 cells of 1 cm, 0.6 mm above the ground's two triangles."""
    sc = S.block_drop(n_steps=1)
    g = np.stack(np.meshgrid(np.arange(n + 1), np.arange(2), np.arange(2), indexing="ij"), -1).reshape(-1, 3)
    rng = np.random.Generator(np.random.PCG64(n))
    X = 0.01 * g + [0.3 - 0.005 * n, 0.295, 6e-4] + rng.uniform(-1e-4, 1e-4, size=g.shape)
    T = S.hex_tets(n, 1, 1)
    e = X[T[:, 1:]] - X[T[:, :1]]
    neg = np.linalg.det(e) < 0
    T[neg, 1], T[neg, 2] = T[neg, 2].copy(), T[neg, 1].copy()
    nt = len(T)
    sc.update(X=X, V=np.zeros_like(X), tets=np.ascontiguousarray(T), tet_E=np.full(nt, 1e5), tet_nu=np.full(nt, 0.45),
              tet_rho=np.full(nt, 1000.0), vobj=np.zeros(len(X), np.int32))
    return sc


# 8 n + 4 + 2 triangles and 12 n + 6 + 5 edges: one block of leaves, around
# 128 edges (two blocks), past one round of the workgroup's blocks
@pytest.mark.parametrize("cells", [(1,), (6,), (10,), (11,), (60,), (1400,), (1, 11, 60, 2, 10)], ids=str)
def test_pairs_and_ccd_match_the_oracle(cells):
    from paper_2609_25653_amd import Sim
    scenes = [_block(n) for n in cells]
    sim = Sim(scenes)
    orc = [O.Oracle(sc) for sc in scenes]
    y = np.concatenate([o.state()[0] for o in orc])
    rng = np.random.default_rng(3)
    p = 3e-3 * rng.standard_normal(len(y))
    alpha = to_np(sim.ccd(y, p))
    for s, o in enumerate(orc):
        ys, ps = (a[sim.dof_offsets[s]:sim.dof_offsets[s + 1]] for a in (y, p))
        pt, ee = sim.pairs(y, scene=s)
        opt, oee = o.pairs(ys)
        assert len(opt) > 0 and np.array_equal(pt, opt) and np.array_equal(ee, oee), (cells, s)
        assert alpha[s] == o.ccd(ys, ps), (cells, s)
