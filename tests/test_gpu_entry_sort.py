"""The sort behind the assembly's run sums, over its three ways (one block up
to 1024 entries, one workgroup's passes up to 4096, a pass over several
workgroups beyond): copies of one scene in one context, whose contact pairs
give 4 entries each for the gradient and 16 for the matrix, against the scene
alone.  Only the places where a run's partial sums meet differ, runs of some
50 terms at most, so gradients and products agree within 1e-13 of their
largest entry."""
import numpy as np
import pytest

from gpu_util import to_np
from test_gpu_wide_queries import _block

pytestmark = pytest.mark.gpu
WAYS = (1024, 4096, 8192)   # the last entry of one block, of one workgroup, of two


def _eval(sim, y, d):
    import torch
    dev = lambda a: torch.as_tensor(a, dtype=torch.float64, device="cuda")
    e, g, hv = sim.energy_grad_hess(dev(y), dev(d))[:3]
    return to_np(e), to_np(g), to_np(hv)


@pytest.mark.parametrize("way", WAYS)
@pytest.mark.parametrize("per_pair", [4, 16])
@pytest.mark.parametrize("beyond", [False, True])
def test_copies_of_a_scene(way, per_pair, beyond):
    from paper_2609_25653_amd import Sim
    one = Sim(_block(2))
    y1, v1 = (to_np(a) for a in one.state())
    pt, ee = one.pairs(y1)
    pairs = len(pt) + len(ee)
    copies = way // (per_pair * pairs) + (1 if beyond else 0)   # the last count of this way, the first of the next
    assert copies >= 1 and (per_pair * pairs * copies > way) == beyond
    rng = np.random.default_rng(5)
    d1 = rng.standard_normal(len(y1))
    one.begin_step(0)
    e, g, hv = _eval(one, y1, d1)
    many = Sim([_block(2)] * copies)
    many.begin_step(0)
    es, gs, hvs = _eval(many, np.tile(y1, copies), np.tile(d1, copies))
    assert np.abs(g).max() > 0 and np.abs(hv).max() > 0
    assert np.abs(gs.reshape(copies, -1) - g).max() <= 1e-13 * np.abs(g).max()
    assert np.abs(hvs.reshape(copies, -1) - hv).max() <= 1e-13 * np.abs(hv).max()
