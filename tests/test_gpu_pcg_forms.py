"""The PCG solve's forms and the contact rows that they share.

A scene's solve runs as one resident launch or iteration by iteration; both
form every sum in the same order, so the trajectories are compared bit for
bit, at the sizes where the resident form's layout changes: one workgroup and
several, a last workgroup with few rows, narrow and wide workgroups, rows of
more blocks than a thread's registers hold, no row and most rows in contact, no fixed rows, block-Jacobi
in place of the multilevel groups, and a resident launch that is given up
while it forms.

Contact rows are checked against the per-pair blocks of the same state, summed
on the host: tolerance 1e-11 of the largest entry of the row block (the order
of FP64 sums), with rows of more entries than are merged at a time.
"""
import json
import sys

import numpy as np
import pytest

from paper_2411_04776_amd import scenes as S
from parity_util import assert_rows_close

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def ipc():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible MI355X"
    from paper_2411_04776_amd import ipc as I
    I.lib()
    return I


def gel(grid, size=S.GEL_SIZE, radius=4e-3, subdiv=2, steps=2, gap=0.0):
    X, T, fixed = S.grid_gel(*grid, size=size)
    Y, F = S.icosphere(subdiv, radius)
    poses = S._descent_poses(np.eye(3), Y, size[2], (size[0] / 2, size[1] / 2), 0.1e-3, steps)
    poses[:, 2, 3] += gap
    return S.Scene("gel%dx%dx%d" % grid, X, T, fixed, Y, F, poses, dt=1e-2)


def hub(subdiv):
    """A ball of tets that share their centre: one row holds every column."""
    P, F = S.icosphere(subdiv, 3e-3)
    X = np.concatenate([P, np.zeros((1, 3))])
    T = np.concatenate([F, np.full((len(F), 1), len(P))], axis=1)
    D = X[T[:, 1:]] - X[T[:, :1]]
    T[np.linalg.det(D) < 0] = T[np.linalg.det(D) < 0][:, [1, 0, 2, 3]]
    fixed = (X[:, 2] < -1.5e-3).astype(np.uint8)
    Y, Fi = S.icosphere(1, 2e-3)
    poses = S._descent_poses(np.eye(3), Y, X[:, 2].max(), (0.0, 0.0), 0.1e-3, 2)
    return S.Scene(f"hub{subdiv}", X, T.astype(np.int32), fixed, Y, Fi, poses, dt=1e-2)


def plate(grid):
    """A coarse plate flat on a fine gel: each of its vertices meets every surface vertex of the gel."""
    X, T, fixed = S.grid_gel(*grid)
    Y, F = S.box(30e-3, target_edge=30e-3)
    poses = S._descent_poses(np.eye(3), Y, S.GEL_SIZE[2], (S.GEL_SIZE[0] / 2, S.GEL_SIZE[1] / 2), 0.05e-3, 2)
    return S.Scene("plate", X, T, fixed, Y, F, poses, dt=1e-2)


SCENES = {
    "one workgroup": (lambda: S.tiny_scene(), False),
    "one workgroup mixed": (lambda: S.tiny_scene(), True),
    "remainder": (lambda: gel((13, 11, 5)), False),
    "remainder mixed": (lambda: gel((19, 23, 5)), True),
    "apart": (lambda: gel((9, 8, 4), gap=1e-3), False),
    "hub": (lambda: hub(2), False),
    "hub mixed": (lambda: hub(3), True),
    "plate": (lambda: plate((12, 14, 4)), False),
    "plate mixed": (lambda: plate((28, 30, 3)), True),
    "jacobi": (lambda: gel((11, 9, 4)), False),
    "attached": (lambda: S.attached_scene(grid=(9, 11, 3), depth=2e-4, steps=2), False),
    "friction": (lambda: S.tiny_slide_scene(press_steps=1, slide_steps=1), False),
    "wide mixed": (lambda: gel((57, 50, 12), steps=1), True),
}


def run(ipc, monkeypatch, tmp_path, sc, mixed, team, spin, jacobi=False):
    f = tmp_path / f"t{team}{spin}.json"
    f.write_text(json.dumps({"classes": [{"min_verts": 0, "team": team, "team_spin": spin}]}))
    monkeypatch.setenv("IPC_TUNING_FILE", str(f))
    g = ipc.GelScene(sc, precision=ipc.IPC_MIXED if mixed else ipc.IPC_FP64, pcg_tol=3e-5 if mixed else 1e-12,
                     precond=ipc.IPC_PRECOND_JACOBI if jacobi else ipc.IPC_PRECOND_MULTILEVEL)
    its = []
    for _ in range(sc.n_steps):
        rc, st = g.step()
        its.append((rc, st.newton_iters, st.pcg_iters))
    out = its, g.x.copy(), g.v.copy()
    g.close()
    return out


@pytest.mark.parametrize("name", list(SCENES))
def test_forms_agree(ipc, monkeypatch, tmp_path, name):
    make, mixed = SCENES[name]
    sc = make()
    want = run(ipc, monkeypatch, tmp_path, sc, mixed, 0, 0, name == "jacobi")
    for team, spin in ((1, 1 << 14), (1, 0)):
        say("pcg forms", name, "resident" if spin else "given up while it forms")
        its, x, v = run(ipc, monkeypatch, tmp_path, sc, mixed, team, spin, name == "jacobi")
        assert its == want[0]
        assert np.array_equal(x, want[1]) and np.array_equal(v, want[2])
    assert sum(i[2] for i in want[0]) > 0


@pytest.mark.parametrize("grid,entries", [((6, 5, 3), 0), ((30, 32, 3), 680)])
def test_contact_rows(ipc, grid, entries):
    """Gradient and H v with the contact rows against the sums over the pairs."""
    sc = plate(grid)
    g = ipc.GelScene(sc)
    g.begin_step(sc.poses[1])
    x = g.x.copy()
    ng = len(sc.X)
    x[ng:, 2] -= 0.6 * sc.dhat
    rng = np.random.default_rng(8)
    x[:ng] += rng.normal(0, 0.02 * sc.dhat, (ng, 3)) * (1 - sc.fixed[:, None])
    kind, v4, g12, H = g.barrier_pairs(x)
    longest = np.bincount(v4.ravel(), minlength=len(x)).max()
    say("contact rows", grid, len(kind), "pairs, longest row", longest)
    assert longest > entries
    v = rng.normal(size=x.shape)
    gb, yb = g.assemble_elastic(x, v)
    np.add.at(gb, v4.ravel(), g12.reshape(-1, 3))
    np.add.at(yb, v4.ravel(), np.einsum("kij,kj->ki", H, v[v4].reshape(-1, 12)).reshape(-1, 3))
    assert_rows_close(g.gradient(x), gb, ng, 1e-11)
    assert_rows_close(g.hess_apply(x, v), yb, ng, 1e-11)
    g.close()
