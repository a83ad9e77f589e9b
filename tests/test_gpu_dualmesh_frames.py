"""Frames of the dual-mesh map taken one per workgroup (k_dm_frame: few blocks
or a single frame; whole blocks or halves) and several per workgroup
(k_dm_pairs): the same bits, for rows that pair and rows that do not, at the
counts where the launch changes, and positions that are not finite reach
exactly the fine vertices whose row of W names them in either kernel."""
import numpy as np
import pytest

from test_gpu_dualmesh import fan
from test_gpu_dualmesh_pairs import _host, _shuffled

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a ROCm GPU")]


def _torus(nu, nv):
    u, v = np.meshgrid(np.arange(nu), np.arange(nv), indexing="ij")
    a, b = 2 * np.pi * u / nu, 2 * np.pi * v / nv
    V = np.stack([(1 + 0.3 * np.cos(b)) * np.cos(a), (1 + 0.3 * np.cos(b)) * np.sin(a), 0.3 * np.sin(b)], -1).reshape(-1, 3)
    i = lambda x, y: (x % nu) * nv + y % nv
    F = np.stack([i(u, v), i(u + 1, v), i(u + 1, v + 1), i(u, v), i(u + 1, v + 1), i(u, v + 1)], -1).reshape(-1, 3)
    return V, F


def _mesh(name):
    if name == "unpaired":                 # rows of 16 next to rows of 4; a single block of under 128 groups
        return fan(15, seed=2) + (1,)
    if name == "one level":                # groups of at most 8 columns, one block of over 128 groups and a short one
        return _torus(13, 11) + (1,)
    if name == "many blocks":              # more than 64: 50 frames are several per workgroup
        return _shuffled(20, 24, 3) + (2,)
    return _torus(31, 20) + (3,)           # 78 blocks: one frame in whole blocks and in none halved


@pytest.mark.parametrize("name", ["unpaired", "one level", "many blocks", "three levels"])
def test_single_frames_and_runs_of_frames_agree(name):
    from paper_2609_25653_amd.dualmesh import DualMesh
    V, F, levels = _mesh(name)
    rng = np.random.default_rng(1)
    X = V[None] + 0.1 * rng.standard_normal((50,) + V.shape)
    X[7, 2, 1] = np.inf
    X[31, len(V) - 1, 0] = np.nan
    dm = DualMesh(F, len(V), levels)
    x = torch.as_tensor(X, device="cuda")
    all_at_once = dm.apply(x).cpu().numpy()
    with np.errstate(invalid="ignore"):
        ref = _host(dm, X)
    fin = np.isfinite(ref)
    assert not fin[7].all() and not fin[31].all() and fin[:7].all()
    assert np.array_equal(all_at_once[~fin], ref[~fin], equal_nan=True)
    assert np.abs(all_at_once[fin] - ref[fin]).max() <= 1e-13 * np.abs(X[np.isfinite(X)]).max()
    for frames in (1, 2, 3, 5, 20):
        for f in (0, 7, 30):
            part = x[f:f + frames].contiguous()
            assert np.array_equal(dm.apply(part).cpu().numpy(), all_at_once[f:f + len(part)], equal_nan=True), (frames, f)


def _large(name):
    V, F = _torus(328 if name == "rows staged" else 300, 200)
    if name == "rows staged":
        return V, F
    rng = np.random.default_rng(6)         # rows next to each other share no columns: blocks of more than 1024
    perm = rng.permutation(len(V))
    W = np.empty_like(V)
    W[perm] = V
    return W, perm[F][rng.permutation(len(F))]


@pytest.mark.parametrize("name", ["rows staged", "rows not staged"])
def test_the_forms_that_fit_the_fixed_array(name):
    """One level, 262400 and 240000 rows: W's pairs take more than the no-alloc
    path's 16 MiB, its own rows (at most 12 bytes per nonzero and 4 per row)
    less.  The same bits as through the library's own memory, for frames in
    one part and in several, also around positions that are not finite."""
    from paper_2609_25653_amd.dualmesh import DualMesh
    V, F = _large(name)
    dm = DualMesh(F, len(V), 1)
    assert 12 * dm.nnz + 4 * (dm.n_fine + 1) <= 16 << 20
    rng = np.random.default_rng(3)
    for frames in (1, 3, 40):
        X = V[None] + 0.1 * rng.standard_normal((frames,) + V.shape)
        X[0, 5, 1] = np.inf
        X[-1, len(V) - 2, 0] = np.nan
        xc = torch.as_tensor(X, device="cuda")
        a = dm.apply(xc)
        b = torch.full_like(a, 7.0)
        dm.apply_noalloc(xc, b)
        torch.cuda.synchronize()
        assert torch.equal(torch.isnan(a), torch.isnan(b))
        assert torch.equal(a.nan_to_num(nan=-9.0), b.nan_to_num(nan=-9.0)) and not torch.isfinite(a).all()


def test_few_frames_of_a_large_mesh_of_one_level():
    """Up to 4 frames go row by row from a copy of W's rows, more by pairs;
    the same bits, whichever call comes first on a handle."""
    from paper_2609_25653_amd.dualmesh import DualMesh
    V, F = _torus(300, 200)
    rng = np.random.default_rng(4)
    X = V[None] + 0.1 * rng.standard_normal((9,) + V.shape)
    X[2, 11, 2] = -np.inf
    x = torch.as_tensor(X, device="cuda")
    few, many = DualMesh(F, len(V), 1), DualMesh(F, len(V), 1)
    a = torch.cat([few.apply(x[f:f + 1].contiguous()) for f in range(5)] + [few.apply(x[5:9].contiguous())])
    b = many.apply(x)
    c = torch.cat([many.apply(x[:4].contiguous()), many.apply(x[4:].contiguous())])
    for q in (a, c):
        assert torch.equal(torch.isnan(q), torch.isnan(b)) and torch.equal(q.nan_to_num(nan=-9.0), b.nan_to_num(nan=-9.0))
    assert not torch.isfinite(b[2]).all() and torch.isfinite(b[3:]).all()
