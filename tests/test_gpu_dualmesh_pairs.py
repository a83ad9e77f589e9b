"""The dual-mesh kernel that gives a thread two fine rows: shuffled meshes,
whose blocks fill up with distinct coarse vertices before they are full of
rows, frames split over workgroups (16, 17 and 50 of them, the last part
shorter), an odd number of rows, rows that do not pair, and positions that
are not finite, which must reach exactly the fine vertices whose row of W
names them.  Against W's own rows summed on the host: each coordinate within
1e-13 of the coordinates' magnitude, a few roundings of sums of at most 16
positive terms (needs a GPU)."""
import numpy as np
import pytest

import ipcscenes as S
from test_gpu_dualmesh import fan

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a ROCm GPU")]


def _shuffled(disk, layers, seed):
    rng = np.random.default_rng(seed)
    tri, frames = S.dualmesh_frames(n_frames=1, n_disk=disk, n_layers=layers)
    V = frames[0]
    perm = rng.permutation(len(V))                      # new number of each vertex
    W = np.empty_like(V)
    W[perm] = V
    return W, perm[np.asarray(tri)][rng.permutation(len(tri))]


def _host(dm, X):
    rp, col, val = dm.weights()
    return np.stack([np.add.reduceat(val[:, None] * x[col], rp[:-1], axis=0) for x in X])


def _mesh(name):
    if name == "shuffled":
        return _shuffled(20, 24, 3) + (2,)
    if name == "coarse rows only":
        return _shuffled(16, 20, 4) + (0,)
    if name == "unpaired":                              # rows of 16 next to rows of 4
        return fan(15, seed=2) + (1,)
    tri, frames = S.dualmesh_frames(n_frames=1, n_disk=6, n_layers=7)
    return frames[0], np.asarray(tri), 3


@pytest.mark.parametrize("name", ["shuffled", "coarse rows only", "unpaired", "cylinder"])
@pytest.mark.parametrize("frames", [1, 16, 17, 50])
def test_matches_the_rows_of_w(name, frames):
    from paper_2609_25653_amd.dualmesh import DualMesh
    V, F, levels = _mesh(name)
    rng = np.random.default_rng(frames)
    X = V[None] + 0.1 * rng.standard_normal((frames,) + V.shape)
    dm = DualMesh(F, len(V), levels)
    xc = torch.as_tensor(X, device="cuda")
    out = torch.full((frames, dm.n_fine, 3), float("nan"), dtype=torch.float64, device="cuda")
    dm.apply(xc, out)
    ref = _host(dm, X)
    assert np.abs(out.cpu().numpy() - ref).max() <= 1e-13 * np.abs(X).max()
    again = torch.full_like(out, float("nan"))
    dm.apply_noalloc(xc, again)
    torch.cuda.synchronize()
    assert torch.equal(out, again)


@pytest.mark.parametrize("value", [float("nan"), float("inf"), -float("inf")])
@pytest.mark.parametrize("name", ["shuffled", "cylinder"])
def test_positions_that_are_not_finite(name, value):
    from paper_2609_25653_amd.dualmesh import DualMesh
    V, F, levels = _mesh(name)
    X = np.repeat(V[None], 5, axis=0)
    X[1, 3, 0] = value
    X[4, len(V) - 1, 2] = value
    dm = DualMesh(F, len(V), levels)
    out = dm.apply(torch.as_tensor(X, device="cuda")).cpu().numpy()
    ref = _host(dm, X)
    fin = np.isfinite(ref)
    assert not fin[1].all() and not fin[4].all() and fin[0].all()
    assert np.array_equal(out[~fin], ref[~fin], equal_nan=True)
    assert np.abs(out[fin] - ref[fin]).max() <= 1e-13 * np.abs(V).max()
