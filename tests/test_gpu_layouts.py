"""Storage orders and work splits against the oracle, at the sizes where they change.

Tets: a regular grid, whose tets are stored by pattern, the same grid with its
tets shuffled, and a ball of tets around one vertex, which keeps its order.
Body gradient and H v to 1e-11 of the row block's largest entry (the order of
FP64 sums).

Height map: images whose triangles cover one pixel, part of a 16 x 4 tile and
many tiles; the same FP64 expressions, to 1e-15 m.
"""
import numpy as np
import pytest

import oracle as O
from oracle.height_map import height_map
from paper_2411_04776_amd import scenes as S
from parity_util import assert_rows_close
from test_gpu_pcg_forms import gel, hub

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ipc():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible MI355X"
    from paper_2411_04776_amd import ipc as I
    I.lib()
    return I


@pytest.mark.parametrize("name", ["grid", "shuffled", "hub"])
def test_tet_storage(ipc, name):
    print("tet storage", name, flush=True)
    sc = hub(2) if name == "hub" else gel((9, 7, 5))
    rng = np.random.default_rng(3)
    if name == "shuffled":
        sc.T = sc.T[rng.permutation(len(sc.T))]
    g, o = ipc.GelScene(sc), O.OracleScene(sc)
    g.begin_step(sc.poses[1])
    o.begin_step(sc.poses[1])
    x = o.x.copy()
    x[:o.n_gel] += rng.normal(0, 1e-5, (o.n_gel, 3)) * (1 - sc.fixed[:, None])
    t = o.gradient_terms(x)
    want = t["inertia"] + t["elastic"] + t["target"]
    want[:o.n_gel][sc.fixed.astype(bool)] = 0.0
    v = rng.normal(size=x.shape)
    gb, yb = g.assemble_elastic(x, v)
    assert_rows_close(gb, want, o.n_gel, 1e-11)
    assert_rows_close(yb, o.hess_apply_body(x, v), o.n_gel, 1e-11)
    g.close()


@pytest.mark.parametrize("nx,ny", [(3, 2), (17, 5), (130, 9), (7, 90), (301, 260)])
def test_height_map_tiles(ipc, nx, ny):
    print("height map", nx, ny, flush=True)
    sc = gel((5, 4, 3))
    g, o = ipc.GelScene(sc), O.OracleScene(sc)
    _, _, tris = o.surface()
    x = o.x.copy()
    x[:o.n_gel] += np.random.default_rng(5).normal(0, 1e-4, (o.n_gel, 3)) * (1 - sc.fixed[:, None])
    g.x = x
    ext = sc.X.max(0)
    spec = (-0.02 * ext[0], -0.03 * ext[1], 1.05 * ext[0] / nx, 1.04 * ext[1] / ny, nx, ny, ext[2])
    got = g.height_map(*spec)
    want = height_map(x, tris[:o.n_gel_tris], *spec)
    assert np.abs(got - want).max() <= 1e-15
    assert np.count_nonzero(want) > 0
    g.close()
