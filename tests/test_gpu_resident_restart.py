"""When the PCG solve in one launch gives up (ipc_pcg_resident.hip): the solve
starts again in the launch-per-iteration form, with that form's bits, and the
context leaves the one-launch form alone for a while."""
import numpy as np
import pytest

import ipcscenes as S

pytestmark = pytest.mark.gpu


def _block(n, z=0.3):
    """n^3 cells of 1 cm, away from the ground."""
    sc = S.block_drop(n_steps=2)
    g = np.stack(np.meshgrid(*[np.arange(n + 1)] * 3, indexing="ij"), -1).reshape(-1, 3)
    X = 0.01 * g + [0.1, 0.1, z]
    T = S.hex_tets(n, n, n)
    e = X[T[:, 1:]] - X[T[:, :1]]
    neg = np.linalg.det(e) < 0
    T[neg, 1], T[neg, 2] = T[neg, 2].copy(), T[neg, 1].copy()
    nt = len(T)
    sc.update(X=X, V=np.zeros_like(X), tets=np.ascontiguousarray(T), tet_E=np.full(nt, 1e5), tet_nu=np.full(nt, 0.45),
              tet_rho=np.full(nt, 1000.0), vobj=np.zeros(len(X), np.int32))
    return sc


def _crossed(n=12, per=40, seed=0):
    """The block with weak springs from every vertex to 40 random ones: rows of
    at most 64 blocks, 64 of which read more vertices of other rows than a
    workgroup has places for (1024)."""
    sc = _block(n)
    rng = np.random.default_rng(seed)
    nv = len(sc["X"])
    a = np.tile(np.arange(nv), per // 2)
    b = np.concatenate([rng.permutation(nv) for _ in range(per // 2)])
    a, b = a[a != b], b[a != b]
    ns = len(a)
    sc.update(sp_ka=np.zeros(ns, np.int32), sp_ia=a.astype(np.int32), sp_xa=np.zeros((ns, 3)), sp_kb=np.zeros(ns, np.int32),
              sp_ib=b.astype(np.int32), sp_xb=np.zeros((ns, 3)), sp_k=np.full(ns, 1.0))
    return sc


def test_crossed_block_has_short_rows_that_do_not_fit():
    """(the input of the tests below, on the host: a tile's 64 rows are
    vertices near each other)"""
    sc = _crossed()
    X = sc["X"]
    adj = [set() for _ in range(len(X))]
    for t in sc["tets"]:
        for i in t:
            adj[i].update(int(j) for j in t)
    for i, j in zip(sc["sp_ia"], sc["sp_ib"]):
        adj[i].add(int(j))
        adj[j].add(int(i))
    assert max(len(a) for a in adj) <= 64 and len(X) <= 64 * 240
    for k in range(0, len(X), 200):
        own = set(np.argsort(np.abs(X - X[k]).max(1), kind="stable")[:64].tolist())
        assert len(set().union(*(adj[i] for i in own)) - own) > 1024


def _solve(sc, b_seed, eta=1e-8):
    import torch
    from paper_2609_25653_amd import Sim
    sim = Sim(sc)
    y, _ = sim.state()
    sim.begin_step(0)
    b = torch.randn(sim.ndof, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(b_seed))
    return sim, y, b


@pytest.mark.parametrize("with_others", [False, True])
def test_rows_that_do_not_fit(with_others, monkeypatch):
    """One workgroup's set-up refuses, the others wait for it and leave: the
    verdict stays "does not fit", whatever the order in which they leave."""
    import torch
    from paper_2609_25653_amd._lib import Q_PCG_RESIDENT, Q_PCG_SKIP
    monkeypatch.setenv("IPC_PCG_COARSE", "0")
    sc = _crossed()
    if with_others:   # scenes that fit, of which the first ends before the refusal is seen
        sc = [S.tiny_scene("tet", h=0.01, n_steps=2), sc, _block(6)]
    got = []
    for eager in ("1", "0"):
        monkeypatch.setenv("IPC_NO_GRAPH", eager)
        sim, y, b = _solve(sc, 3)
        x, it = sim.pcg(y, b, 1e-8)
        assert sim._query(Q_PCG_RESIDENT) == 0
        assert sim._query(Q_PCG_SKIP) == (0 if eager == "1" else 256)
        x2, it2 = sim.pcg(y, b, 1e-8)
        assert torch.equal(x, x2) and np.array_equal(it, it2)
        assert sim._query(Q_PCG_SKIP) == (0 if eager == "1" else 255)
        got.append((x.clone(), it.copy()))
    assert torch.equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1]) and got[0][1].max() > 10


@pytest.mark.parametrize("coarse", ["0", "1"])
@pytest.mark.parametrize("name", ["one_tile", "squeeze", "batch"])
def test_restart_after_giving_up(name, coarse, monkeypatch):
    """The abort word is up from the start: workgroups that need not wait
    (scenes of one tile) run to their end and write their solutions and
    counts, the others leave at the first wait; then the solve starts again.
    Steps and counts are those of the launch-per-iteration form."""
    import torch
    from paper_2609_25653_amd import Sim
    from paper_2609_25653_amd._lib import Q_PCG_RESIDENT, Q_PCG_SKIP
    if name == "one_tile":
        sc = S.tiny_scene("cube", h=0.01, n_steps=3)
    elif name == "squeeze":
        sc = S.gripper_squeeze(n_steps=3, pad_cells=(4, 2, 3))
    else:
        sc = [S.tiny_scene("cube", h=0.005, n_steps=3), S.gripper_squeeze(n_steps=3, pad_cells=(6, 3, 3)), S.block_drop(n_steps=3),
              S.tiny_scene("free_body", h=0.005, n_steps=3)]
    monkeypatch.setenv("IPC_PCG_COARSE", coarse)
    got = []
    for eager in ("1", "0"):
        monkeypatch.setenv("IPC_NO_GRAPH", eager)
        monkeypatch.setenv("IPC_PCG_GIVE_UP", "1")
        sim = Sim(sc)
        out = []
        for _ in range(3):
            _, st = sim.step(allow_status=(3,))
            out.append((sim.state(), [(q["newton_iters"], q["pcg_iters_total"], q["status"]) for q in st]))
        assert sim._query(Q_PCG_RESIDENT) == 0
        assert (sim._query(Q_PCG_SKIP) > 0) == (eager == "0")
        got.append(out)
    for ((ya, va), sa), ((yb, vb), sb) in zip(*got):
        assert sa == sb and torch.equal(ya, yb) and torch.equal(va, vb)


def test_two_contexts_on_two_streams(monkeypatch):
    """Two threads solve at the same time, each with its context on its own
    stream: one launch holds the device at a time, the other context takes
    the launch-per-iteration form meanwhile.  Solutions are those of a
    context alone, whichever form each solve took."""
    import threading

    import torch
    from paper_2609_25653_amd import Sim
    from paper_2609_25653_amd._lib import Q_PCG_RESIDENT
    scenes = [S.gripper_squeeze(n_steps=1, pad_cells=(12, 6, 6)), _block(9)]
    N = 40

    def solves(sc, n):
        with torch.cuda.stream(torch.cuda.Stream()):
            sim = Sim(sc)
            y, _ = sim.state()
            sim.begin_step(0)
            b = torch.randn(sim.ndof, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(7))
            torch.cuda.current_stream().synchronize()
            xs = [sim.pcg(y, b, 1e-8) for _ in range(n)]
            torch.cuda.current_stream().synchronize()
            return [(x.cpu(), int(it[0])) for x, it in xs], sim._query(Q_PCG_RESIDENT)

    alone = [solves(sc, 1) for sc in scenes]
    assert all(a[1] == 1 for a in alone)
    got = [None, None]

    def run(k):
        got[k] = solves(scenes[k], N)

    ts = [threading.Thread(target=run, args=(k,)) for k in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for k in range(2):
        out, taken = got[k]
        assert 0 <= taken <= N
        for x, it in out:
            assert it == alone[k][0][0][1] and torch.equal(x, alone[k][0][0][0])
    assert got[0][1] + got[1][1] > 0


def _with_bodies(cells, nb):
    """The block and nb free boxes above it, whose nodes follow each other."""
    from ipcscenes import scenes as M
    blk = _block(cells)
    b = M._Builder()
    b.add_fem(blk["X"], blk["tets"], 1e5, 0.45, 1000.0)
    for k in range(nb):
        b.add_body((0.1 * (k % 8), 0.1 * (k // 8), 0.9), (0.02, 0.03, 0.04), 0.05)
    return b.finish(M._params(h=0.01, n_steps=1), np.zeros((1, 0, 12)))


@pytest.mark.parametrize("cells,coarse,nb,taken", [
    (9, "0", 40, True),      # 64 nodes per workgroup: 16 bodies fill them
    (25, "0", 16, True),     # 128 per workgroup: as many bodies as it has places for
    (25, "0", 40, False),
    (9, "1", 13, True),      # 256 per workgroup, rows for 13 bodies' coarse groups
    (9, "1", 30, False),
])
def test_bodies_in_one_workgroup(cells, coarse, nb, taken, monkeypatch):
    """More bodies side by side than a workgroup has places for: the context
    keeps to the launch-per-iteration form from the start (nothing is thrown
    away: the skip count stays 0); up to there the forms agree bit for bit."""
    import torch
    from paper_2609_25653_amd._lib import Q_PCG_RESIDENT, Q_PCG_SKIP
    monkeypatch.setenv("IPC_PCG_COARSE", coarse)
    sc = _with_bodies(cells, nb)
    got = []
    for eager in ("1", "0"):
        monkeypatch.setenv("IPC_NO_GRAPH", eager)
        sim, y, b = _solve(sc, 4)
        x, it = sim.pcg(y, b, 1e-8)
        assert sim._query(Q_PCG_SKIP) == 0
        assert sim._query(Q_PCG_RESIDENT) == (1 if eager == "0" and taken else 0)
        got.append((x.clone(), int(it[0])))
    assert torch.equal(got[0][0], got[1][0]) and got[0][1] == got[1][1] > 5


def test_waits_that_run_out_again_lengthen_the_pause(monkeypatch):
    from paper_2609_25653_amd._lib import Q_PCG_RESIDENT, Q_PCG_SKIP
    monkeypatch.setenv("IPC_PCG_GIVE_UP", "1")
    sim, y, b = _solve(S.tiny_scene("tet", h=0.01, n_steps=1), 5)
    for pause in (64, 128, 256):
        sim.pcg(y, b, 1e-8)
        assert sim._query(Q_PCG_SKIP) == pause
        for _ in range(pause):
            sim.pcg(y, b, 1e-8)
        assert sim._query(Q_PCG_SKIP) == 0 and sim._query(Q_PCG_RESIDENT) == 0


@pytest.mark.parametrize("cells", [9, 25])
def test_stream_with_half_of_the_compute_units(cells, monkeypatch):
    """On a stream that may use half of the compute units the launch is cut
    for these: 17.6k nodes (25 cells), 138 workgroups of two tiles on the whole
    chip, take more tiles each.  No wait runs out, and the bits are the same."""
    import ctypes

    import torch
    from paper_2609_25653_amd._lib import Q_PCG_RESIDENT, Q_PCG_SKIP
    monkeypatch.setenv("IPC_PCG_COARSE", "0")
    sc = _block(cells)
    sim, y, b = _solve(sc, 6)
    want = sim.pcg(y, b, 1e-8)
    assert sim._query(Q_PCG_RESIDENT) == 1
    torch.cuda.synchronize()
    path = [ln.split()[-1] for ln in open("/proc/self/maps") if "libamdhip64" in ln][0]
    hip = ctypes.CDLL(path)
    p = ctypes.c_void_p()
    n = torch.cuda.get_device_properties(0).multi_processor_count // 32
    mask = (ctypes.c_uint32 * n)(*[0xFFFFFFFF if k < n // 2 else 0 for k in range(n)])
    assert hip.hipExtStreamCreateWithCUMask(ctypes.byref(p), n, mask) == 0
    try:
        with torch.cuda.stream(torch.cuda.ExternalStream(p.value)):
            sim, y, b = _solve(sc, 6)
            x, it = sim.pcg(y, b, 1e-8)
            assert sim._query(Q_PCG_SKIP) == 0 and sim._query(Q_PCG_RESIDENT) == 1
            torch.cuda.current_stream().synchronize()
        assert torch.equal(x, want[0]) and it[0] == want[1][0]
        del sim, y, b, x
        torch.cuda.synchronize()
    finally:
        hip.hipStreamDestroy(p)
