"""The PCG solve in one launch (ipc_pcg_resident.hip) against the solve of one
launch per iteration step: the same sums in the same order, so solutions and
iteration counts are compared bit for bit, at the sizes where its split
changes (1, 2 or 4 tiles of 64 rows per workgroup, with the coarse correction
or without) and with affine bodies (rows of their own, coarse groups that
stand for a body's node)."""
import numpy as np
import pytest

import ipcscenes as S

pytestmark = pytest.mark.gpu


def _squeeze(c):
    return S.gripper_squeeze(n_steps=1, pad_cells=c)


SCENES = {
    "one_tet": lambda: S.tiny_scene("tet"),                      # a single tile
    "block": lambda: S.block_drop(n_steps=1),                    # FEM only, a ragged last tile
    "free_body": lambda: S.tiny_scene("free_body"),              # bodies only
    "squeeze_small": lambda: _squeeze((4, 2, 3)),                # long rows, contact with a body
    "arm": lambda: S.arm_squeeze(n_steps=1),                     # 13 bodies, joint springs
    "rich_15k": lambda: S.contact_rich(n_steps=1, n_disk=16, n_layers=32),   # about 14.6k nodes
    "rich_27k": lambda: S.contact_rich(n_steps=1, n_disk=22, n_layers=40),   # about 26.8k nodes
    "rich_33k": lambda: S.contact_rich(n_steps=1, n_disk=26, n_layers=38),   # about 33.5k nodes
}


@pytest.mark.parametrize("coarse", ["0", "1"])
@pytest.mark.parametrize("name", list(SCENES))
def test_one_launch_solve_matches_iteration_launches(name, coarse, monkeypatch):
    import torch

    from paper_2609_25653_amd import Sim
    from paper_2609_25653_amd._lib import Q_PCG_RESIDENT
    sc = SCENES[name]()
    monkeypatch.setenv("IPC_PCG_COARSE", coarse)
    got = []
    for eager in ("1", "0"):
        monkeypatch.setenv("IPC_NO_GRAPH", eager)
        sim = Sim(sc)
        y, _ = sim.state()
        sim.begin_step(0)
        b = torch.randn(sim.ndof, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(5))
        out = []
        for cap, eta in ((1, 1e-10), (7, 1e-10), (None, 1e-6)):
            if cap is not None:
                s2 = dict(sc, max_pcg=np.asarray(float(cap)))
                one = Sim(s2)
                one.begin_step(0)
            else:
                one = sim
            x, it = one.pcg(y, b, eta)
            out.append((x.clone(), int(it[0])))
            # a right-hand side of zeros ends before the first update
            x0, it0 = one.pcg(y, torch.zeros_like(b), eta)
            assert it0[0] == 0 and not x0.any()
            solves = one._query(Q_PCG_RESIDENT)
            assert solves == (0 if eager == "1" else 2), (name, solves)
        got.append(out)
    for (xa, ia), (xb, ib) in zip(*got):
        assert ia == ib and torch.equal(xa, xb), (name, ia, ib)


@pytest.mark.parametrize("coarse", ["0", "1"])
def test_scenes_of_a_batch_match_iteration_launches(coarse, monkeypatch):
    """Uneven scenes, more than one launch holds with the coarse correction (4
    workgroups at least per scene), with and without bodies and contact: steps
    (each Newton iteration solves for the scenes still iterating) and counts."""
    import torch

    from paper_2609_25653_amd import Sim
    from paper_2609_25653_amd._lib import Q_PCG_RESIDENT
    cells = [(2, 2, 2), (6, 3, 3), (12, 6, 6), (3, 2, 2)]
    scenes = [S.gripper_squeeze(seed=i, n_steps=2, pad_cells=cells[i % 4]) for i in range(40)]
    scenes[3:3] = [S.block_drop(n_steps=2), S.tiny_scene("free_body", h=0.005, n_steps=2), S.tiny_scene("cube", h=0.005, n_steps=2)]
    monkeypatch.setenv("IPC_PCG_COARSE", coarse)
    got = []
    for eager in ("1", "0"):
        monkeypatch.setenv("IPC_NO_GRAPH", eager)
        sim = Sim(scenes)
        out = []
        for _ in range(2):
            _, st = sim.step(allow_status=(3,))
            out.append((sim.state(), [(q["newton_iters"], q["pcg_iters_total"], q["status"]) for q in st]))
        assert (sim._query(Q_PCG_RESIDENT) > 0) == (eager == "0")
        got.append(out)
    for ((ya, va), sa), ((yb, vb), sb) in zip(*got):
        assert sa == sb and torch.equal(ya, yb) and torch.equal(va, vb)


def test_rows_in_contact_past_a_chunk(monkeypatch):
    """The 200k-tet squeeze after 34 steps: one workgroup's rows have some 2200
    blocks past those in registers, three chunks of 1024; early on none has
    more than one."""
    import torch

    from paper_2609_25653_amd import Sim
    from paper_2609_25653_amd._lib import Q_PCG_RESIDENT
    sc = S.contact_rich(n_steps=100)
    got = []
    y = v = None
    for eager in ("0", "1"):
        monkeypatch.setenv("IPC_NO_GRAPH", eager)
        sim = Sim(sc)
        if y is None:
            for n in range(34):
                sim.step(n, allow_status=(3,))
            y, v = sim.state()
        else:
            sim.set_state(y, v)
        sim.begin_step(34)
        b = torch.randn(sim.ndof, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(6))
        before = sim._query(Q_PCG_RESIDENT)
        x, it = sim.pcg(y, b, 1e-6)
        assert sim._query(Q_PCG_RESIDENT) - before == (1 if eager == "0" else 0)
        got.append((x.clone(), int(it[0])))
    assert got[0][1] == got[1][1] > 10
    assert torch.equal(got[0][0], got[1][0])
