"""Contact rows without blocks: free vertices whose contact partners are all fixed.

Such a vertex has contact entries (its gradient and diagonal block count) but no
off-diagonal block, since fixed columns drop out. A fine free block stands just
above a coarse fixed slab of the same mesh: most of its lowest vertices touch
triangles of fixed vertices only. The resident solve's result is compared with
the launched form's bit for bit, and gradient and H v with the sums over the
pairs (1e-11 of the largest entry of the row block in FP64: the order of sums;
mixed: 2^-24 for each of the roundings to FP32 in an element, a pair and a
stored sum, some 40 of them in a row, of the row block's largest entry).
"""
import numpy as np
import pytest

from paper_2411_04776_amd import scenes as S
from parity_util import assert_rows_close
from test_gpu_pcg_forms import run

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ipc():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible MI355X"
    from paper_2411_04776_amd import ipc as I
    I.lib()
    return I


def slab(grid, gap=0.5):
    """A free block of gel `gap` barrier ranges above a fixed slab of 3 x 3 x 2 vertices."""
    size = (8e-3, 8e-3, 2e-3)
    X0, T0, _ = S.grid_gel(*grid, size=size)
    X1, T1, _ = S.grid_gel(3, 3, 2, size=(10e-3, 10e-3, 2e-3))
    X1 = X1 - np.array([1.1e-3, 0.9e-3, size[2] + gap * S.DHAT])
    X, T = np.concatenate([X0, X1]), np.concatenate([T0, T1 + len(X0)])
    fixed = np.concatenate([np.zeros(len(X0)), np.ones(len(X1))]).astype(np.uint8)
    Y, F = S.icosphere(1, 2e-3)
    poses = S._descent_poses(np.eye(3), Y, size[2], (4e-3, 4e-3), 0.05e-3, 2)
    return S.Scene("slab", X, T.astype(np.int32), fixed, Y, F, poses, dt=1e-2)


def rows_without_blocks(v4, fixed):
    """Free vertices with contact entries, and those of them whose partners are all fixed."""
    free = fixed[v4] == 0
    with_entries = np.unique(v4[free])
    partner = free & (free.sum(axis=1, keepdims=True) > 1)
    return with_entries, np.setdiff1d(with_entries, np.unique(v4[partner]))


# narrow layouts (several workgroups), the rows of a chunk more than its lanes hold at a time; one workgroup
@pytest.mark.parametrize("grid,mixed,held", [((13, 13, 3), False, 16), ((15, 15, 3), True, 32), ((9, 9, 2), False, 0)])
def test_partners_all_fixed(ipc, monkeypatch, tmp_path, grid, mixed, held):
    sc = slab(grid)
    n = len(sc.X) + len(sc.Y)
    g = ipc.GelScene(sc, precision=ipc.IPC_MIXED if mixed else ipc.IPC_FP64)
    g.begin_step(sc.poses[1])
    x = g.x.copy()
    rng = np.random.default_rng(2)
    x[:len(sc.X)] += rng.normal(0, 0.02 * sc.dhat, sc.X.shape) * (1 - sc.fixed[:, None])
    kind, v4, g12, H = g.barrier_pairs(x)
    fixed = np.concatenate([sc.fixed, np.zeros(len(sc.Y), dtype=np.uint8)])
    rows, bare = rows_without_blocks(v4, fixed)
    chunks = -(-n // (256 if mixed else 128))
    print("fixed partners", grid, n, "vertices", len(kind), "pairs", len(rows), "rows,", len(bare), "without a block",
          chunks, "chunks", flush=True)
    assert len(bare) > held * chunks
    v = rng.normal(size=x.shape)
    v[len(sc.X):] *= 1e-7
    gb, yb = g.assemble_elastic(x, v)
    np.add.at(gb, v4.ravel(), g12.reshape(-1, 3))
    yp = np.einsum("kij,kj->ki", H, v[v4].reshape(-1, 12)).reshape(-1, 3)
    np.add.at(yb, v4.ravel(), yp)
    tol = 40 * 2.0 ** -24 if mixed else 1e-11
    assert_rows_close(g.gradient(x), gb, len(sc.X), tol)
    assert_rows_close(g.hess_apply(x, v), yb, len(sc.X), tol)
    g.close()
    want = run(ipc, monkeypatch, tmp_path, sc, mixed, 0, 0)
    print("fixed partners, resident", grid, flush=True)
    its, xr, vr = run(ipc, monkeypatch, tmp_path, sc, mixed, 1, 1 << 14)
    assert its == want[0] and sum(i[2] for i in its) > 0
    assert np.array_equal(xr, want[1]) and np.array_equal(vr, want[2])
