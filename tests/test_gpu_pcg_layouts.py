"""Which form of the PCG solve ran: the layouts by size, and each form's own test.

Every case asserts the layout it is meant for and that its solves ran in that
form, then compares bit for bit: the resident form with the launched one, the
launched form's thread per row with its two lanes per row (with and without a
resident form of the same scene, which add in different orders), and a list
whose workgroups share CUs with the scenes alone. A scene above every resident
layout (76,800 vertices FP64) follows the oracle's block-Jacobi PCG to 1e-9 of
the scene's size, as the smaller ones do in test_gpu_parity.
"""
import json

import numpy as np
import pytest

import oracle as O
from paper_2411_04776_amd import scenes as S
from test_gpu_fixed_partners import slab
from test_gpu_one_workgroup import crowd, patch
from test_gpu_parity import pressed
from test_gpu_pcg_forms import gel, hub, plate

pytestmark = pytest.mark.gpu

NARROW, WIDE, ONE_PAIR, ONE = 0, 1, 2, 3
# name: scene, mixed, Jacobi, resident layout, workgroups
CASES = {
    "one workgroup": (lambda: S.tiny_scene(), False, False, ONE_PAIR, 1),
    "one workgroup, a thread more a row": (lambda: patch(2e-3, 5e-5, (4, 4, 6), 1), False, False, ONE, 1),
    "one workgroup mixed": (lambda: S.tiny_scene(), True, False, ONE_PAIR, 1),
    "one workgroup mixed, a thread a row": (lambda: patch(2e-3, 5e-5, (9, 9, 4), 1), True, False, ONE, 1),
    "narrow": (lambda: gel((13, 11, 5)), False, False, NARROW, 7),
    "narrow mixed": (lambda: gel((19, 23, 5)), True, False, NARROW, 10),
    "narrow jacobi": (lambda: gel((11, 9, 4)), False, True, NARROW, 5),
    "narrow, long rows": (lambda: hub(3), True, False, NARROW, 3),
    "narrow, dense rows": (lambda: plate((28, 30, 3)), True, False, NARROW, 10),
    "narrow, rows without blocks": (lambda: slab((13, 13, 3)), False, False, NARROW, 5),
    "wide": (lambda: gel((64, 65, 9), steps=1), False, False, WIDE, 147),
    "wide mixed": (lambda: gel((57, 50, 12), steps=1), True, False, WIDE, 68),
}


@pytest.fixture(scope="module")
def ipc():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible MI355X"
    from paper_2411_04776_amd import ipc as I
    I.lib()
    return I


def scene(ipc, monkeypatch, tmp_path, sc, mixed, jacobi=False, pcg_tol=None, **tuning):
    f = tmp_path / "tuning.json"
    f.write_text(json.dumps({"classes": [dict(min_verts=0, **tuning)]}))
    monkeypatch.setenv("IPC_TUNING_FILE", str(f))
    return ipc.GelScene(sc, precision=ipc.IPC_MIXED if mixed else ipc.IPC_FP64,
                        pcg_tol=pcg_tol or (3e-5 if mixed else 1e-12),
                        precond=ipc.IPC_PRECOND_JACOBI if jacobi else ipc.IPC_PRECOND_MULTILEVEL)


def run(g):
    its = []
    for _ in range(g.scene.n_steps):
        rc, st = g.step()
        its.append((rc, st.newton_iters, st.pcg_iters))
    out = its, g.x.copy(), g.v.copy(), g.pcg_info()
    g.close()
    return out


def same(a, b):
    return a[0] == b[0] and np.array_equal(a[1], b[1]) and np.array_equal(a[2], b[2])


@pytest.mark.parametrize("name", list(CASES))
def test_resident_form_runs(ipc, monkeypatch, tmp_path, name):
    make, mixed, jacobi, layout, workgroups = CASES[name]
    sc = make()
    print("pcg layouts", name, len(sc.X) + len(sc.Y), "vertices", flush=True)
    got = run(scene(ipc, monkeypatch, tmp_path, sc, mixed, jacobi, team=1))
    info, newton = got[3], sum(i[1] for i in got[0])
    print("   ", info, newton, "newton iterations", flush=True)
    assert (info["layout"], info["workgroups"]) == (layout, workgroups)
    assert info["resident"] == newton > 0 and info["launched"] == info["given_up"] == info["compact"] == 0
    if layout in (ONE_PAIR, ONE):
        return  # has no launched form; pinned by test_gpu_one_workgroup
    launched = run(scene(ipc, monkeypatch, tmp_path, sc, mixed, jacobi, team=0))
    assert launched[3]["launched"] == newton and launched[3]["resident"] == launched[3]["given_up"] == 0
    assert same(got, launched)
    given_up = run(scene(ipc, monkeypatch, tmp_path, sc, mixed, jacobi, team=1, team_spin=0))
    print("    given up while forming:", given_up[3], flush=True)
    assert given_up[3]["given_up"] > 0 and given_up[3]["resident"] + given_up[3]["launched"] == newton
    assert same(got, given_up)


def test_given_up_teams_rest(ipc, monkeypatch, tmp_path):
    """Each given-up solve doubles the number of solves until the next try: tries 1, 3, 7, 15, ... (a team whose
    members all arrive at the same moment forms without waiting, and the count starts anew)."""
    sc = gel((13, 11, 5), steps=4)
    its, x, v, info = run(scene(ipc, monkeypatch, tmp_path, sc, False, team=1, team_spin=0))
    newton = sum(i[1] for i in its)
    print("given-up teams:", info, newton, "newton iterations", flush=True)
    assert newton >= 7 and info["launched"] + info["resident"] == newton
    tries = (newton + 1).bit_length() - 1
    assert info["given_up"] == tries if info["resident"] == 0 else info["given_up"] <= tries * (info["resident"] + 1)


# a scene with a resident form adds in its order, one without in a flat one
@pytest.mark.parametrize("grid,mixed,layout", [((24, 26, 5), False, NARROW), ((40, 41, 6), True, NARROW),
                                               ((88, 90, 9), False, -1)])
def test_launched_lanes_per_row(ipc, monkeypatch, tmp_path, grid, mixed, layout):
    sc = gel(grid, radius=3e-3, steps=1)
    p = []
    for rows in (0, 1 << 30):  # a thread per row in every list, in none
        g = scene(ipc, monkeypatch, tmp_path, sc, mixed, pcg_tol=1e-4, team=0, spmv_one_lane_rows=rows)
        g.begin_step(sc.poses[1])
        x = pressed(g.x, len(sc.X), sc.fixed, sc.dhat, 0.85, seed=4)
        p.append(g.pcg(x))
        info = g.pcg_info()
        print("lanes per row", grid, info, p[-1][1], "iterations", flush=True)
        assert info["layout"] == layout and info["launched"] == 1 and info["resident"] == 0
        g.close()
    assert p[0][1] == p[1][1] and abs(p[0][1]) > 10
    assert np.array_equal(p[0][0], p[1][0])


def test_large_list_launched_bitwise_equals_alone(ipc, monkeypatch, tmp_path):
    """Above 65,536 rows the launched form runs a thread per row, a scene alone two lanes per row."""
    scs = [S.uneven_scene(6000 + k, steps=2) for k in range(16)]
    assert sum(len(sc.X) + len(sc.Y) for sc in scs) >= 65536
    ref = []
    for sc in scs:
        g = scene(ipc, monkeypatch, tmp_path, sc, True, team=0)
        rc, st = g.step()
        ref.append((rc, st.newton_iters, st.pcg_iters, g.x))
        g.close()
    gs = [scene(ipc, monkeypatch, tmp_path, sc, True, team=0) for sc in scs]
    b = ipc.Batch()
    print("launched list of", len(gs), flush=True)
    for i, t in enumerate(b.submit(gs)):
        rc, st = b.wait(t)
        assert (rc, st.newton_iters, st.pcg_iters) == ref[i][:3]
        assert np.array_equal(gs[i].x, ref[i][3])
        info = gs[i].pcg_info()
        assert info["launched"] == st.newton_iters and info["resident"] == 0
    b.close()


def test_compact_list_bitwise_equals_alone(ipc, monkeypatch, tmp_path):
    """Narrow teams of more workgroups than CUs share them, two on each."""
    scs = [S.uneven_scene(6100 + k, steps=2) for k in range(24)]
    ref = []
    for sc in scs:
        g = scene(ipc, monkeypatch, tmp_path, sc, True)
        rc, st = g.step()
        ref.append((rc, st.newton_iters, st.pcg_iters, g.x))
        assert g.pcg_info()["compact"] == 0 and g.pcg_info()["resident"] == st.newton_iters
        g.close()
    gs = [scene(ipc, monkeypatch, tmp_path, sc, True) for sc in scs]
    narrow = sum(g.pcg_info()["workgroups"] for g in gs if g.pcg_info()["layout"] == NARROW)
    print("compact list of", len(gs), "scenes,", narrow, "narrow workgroups", flush=True)
    assert narrow > 256
    b = ipc.Batch()
    for i, t in enumerate(b.submit(gs)):
        rc, st = b.wait(t)
        assert (rc, st.newton_iters, st.pcg_iters) == ref[i][:3]
        assert np.array_equal(gs[i].x, ref[i][3])
    infos = [g.pcg_info() for g in gs]
    print("   ", sum(f["compact"] for f in infos), "compact of", sum(f["resident"] for f in infos), "resident", flush=True)
    assert sum(f["compact"] for f in infos) > 0 and sum(f["launched"] for f in infos) == 0
    b.close()


def test_flat_sums_follow_the_oracle(ipc, monkeypatch, tmp_path):
    sc = S.uneven_scene(7100, steps=2, grid=(80, 80, 12))
    g = scene(ipc, monkeypatch, tmp_path, sc, False, jacobi=True, pcg_tol=1e-6)
    assert g.pcg_info()["layout"] == -1
    o = O.OracleScene(sc, pcg_tol=1e-6)
    g.begin_step(sc.poses[1])
    o.begin_step(sc.poses[1])
    x = pressed(o.x, o.n_gel, sc.fixed, sc.dhat, 0.85, seed=4)
    pg, itg = g.pcg(x)
    po, ito = o.pcg(x)
    err = np.abs(pg - po).max() / sc.bbox_diag
    print("flat sums:", len(x), "vertices, iterations gpu/oracle", itg, ito, "max diff / L", err, flush=True)
    assert ito >= 10 and abs(itg - ito) <= 2
    assert g.pcg_info()["launched"] == 1
    assert err <= 1e-9
    g.close()
