"""Scenes that one workgroup holds: the outcome is pinned to the last bit.

A few dozen vertices make scenes whose outcome turns on rounding: an icosphere
whose lowest vertex comes down exactly over an edge of the gel's grid is a tie
of closest features, and one rounding in a Newton iterate grows to 1e-9 to
1e-4 of the positions. So the order in which such a scene's solve, its barrier
Hessians and its contact gradients are added is part of their result. The
golden positions are those of commit 2792d08, which ran every part of a PCG
iteration as a launch of its own and added contact pairs one by one. Equality
is the only tolerance: the same operations in the same order. What does not
turn on the last bit is pinned to the oracle: each Newton iterate from the
oracle's state, to 1e-9 of the scene's size.

The cases: ties of several radii (90 vertices) and larger patches, at both
layouts of each precision, with rows of more blocks than a thread holds (hub),
indenter rows of more entries than eight lanes or a wavefront take at once
(plate), more pairs than the workgroup's LDS keeps (crowd), no aggregates
(Jacobi) and friction.
"""
import os

import numpy as np
import pytest

import oracle as O
from paper_2411_04776_amd import scenes as S
from test_gpu_pcg_forms import gel, hub, plate

pytestmark = pytest.mark.gpu
GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "one_workgroup.npz")


@pytest.fixture(scope="module")
def ipc():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible MI355X"
    from paper_2411_04776_amd import ipc as I
    I.lib()
    return I


def patch(radius, depth, grid=(4, 4, 3), subdiv=1, steps=3):
    """A small patch of gel under the middle of which a sphere's lowest vertex comes down."""
    size = (4e-3, 4e-3, 2e-3)
    X, T, fixed = S.grid_gel(*grid, size=size)
    Y, F = S.icosphere(subdiv, radius)
    c = np.array([size[0] / 2, size[1] / 2, size[2] + S.DHAT - Y[:, 2].min()])
    down = np.array([0.0, 0.0, depth + S.DHAT / steps])
    poses = np.stack([S.pose_matrix(np.eye(3), c - k * down) for k in range(steps + 1)])
    return S.Scene("patch", X, T, fixed, Y, F, poses, dt=1e-2)


def crowd(grid):
    """A gel whose vertices stand closer than the barrier's range, in contact with itself all over."""
    size = tuple(0.6 * S.DHAT * (k - 1) for k in grid)
    X, T, fixed = S.grid_gel(*grid, size=size)
    Y, F = S.icosphere(1, 3 * S.DHAT)
    poses = S._descent_poses(np.eye(3), Y, size[2], (size[0] / 2, size[1] / 2), 0.02 * S.DHAT, 2)
    return S.Scene("crowd", X, T, fixed, Y, F, poses, dt=1e-2)


# name: scene, mixed, Jacobi
CASES = {f"tie {k}": (lambda k=k: patch(1.5e-3 + 0.83e-4 * k, 2.5e-5 + 0.9e-5 * (k % 7)), False, False) for k in range(12)}
CASES.update({
    "tie mixed": (lambda: patch(2e-3, 5e-5), True, False),
    "one thread more": (lambda: patch(2e-3, 5e-5, (4, 4, 6), 1), False, False),
    "larger": (lambda: patch(2e-3, 5e-5, (5, 6, 3), 2), False, False),
    "larger mixed": (lambda: patch(2e-3, 5e-5, (9, 9, 4), 1), True, False),
    "hub": (lambda: hub(2), False, False),
    "hub mixed": (lambda: hub(2), True, False),
    "plate": (lambda: plate((6, 5, 3)), False, False),
    "large plate": (lambda: plate((9, 8, 3)), False, False),
    "plate mixed": (lambda: plate((15, 16, 2)), True, False),
    "plate jacobi": (lambda: plate((9, 8, 3)), False, True),
    "crowd": (lambda: crowd((7, 7, 3)), False, False),
    "crowd mixed": (lambda: crowd((9, 9, 3)), True, False),
    "jacobi": (lambda: gel((4, 4, 3), size=(4e-3, 4e-3, 2e-3), radius=2e-3, subdiv=1), False, True),
    "friction": (lambda: S.tiny_slide_scene(press_steps=1, slide_steps=1), True, False),
})


def final_positions(ipc, name):
    make, mixed, jacobi = CASES[name]
    sc = make()
    g = ipc.GelScene(sc, precision=ipc.IPC_MIXED if mixed else ipc.IPC_FP64, pcg_tol=3e-5 if mixed else 1e-12,
                     precond=ipc.IPC_PRECOND_JACOBI if jacobi else ipc.IPC_PRECOND_MULTILEVEL)
    for _ in range(sc.n_steps):
        rc, st = g.step()
        print("one workgroup", name, len(sc.X) + len(sc.Y), "vertices: rc", rc, "newton", st.newton_iters, "pcg",
              st.pcg_iters, "pairs", st.n_active, flush=True)
    x = g.x.copy()
    g.close()
    return x


@pytest.mark.parametrize("name", list(CASES))
def test_outcome_to_the_last_bit(ipc, name):
    want = np.load(GOLDEN)[name]
    assert len(want) <= 512
    assert np.array_equal(final_positions(ipc, name), want)


@pytest.mark.parametrize("radius,depth", [(1.6e-3, 3e-5), (2e-3, 5e-5), (2.4e-3, 9e-5)])
def test_iterates_from_the_oracles_states(ipc, radius, depth):
    sc = patch(radius, depth)
    o, g = O.OracleScene(sc), ipc.GelScene(sc)
    worst, checked = 0.0, 0
    for step in range(1, sc.n_steps + 1):
        g.x, g.v = o.x, o.v
        o.begin_step(sc.poses[step])
        g.begin_step(sc.poses[step])
        x = o.x.copy()
        for _ in range(12):
            r, nxt, _ = o.newton_iterate(x)
            if r != 0:
                break
            rc, got, st = g.newton_iterate(x)
            assert rc == 0
            worst = max(worst, np.abs(got - nxt).max() / sc.bbox_diag)
            checked += 1
            x = nxt
        o.step()  # the whole step, from the state at its start
    print("iterates of", sc.name, radius, depth, ":", checked, "checked, worst err/L", worst, flush=True)
    assert checked >= 8
    assert worst <= 1e-9
    g.close()
