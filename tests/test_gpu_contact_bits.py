"""Contact products of the mixed form keep FP64 from the stored pair blocks on.

With the direction on the indenter's vertices alone, a gel row of H v is the
contact part alone: the sum over the row's pairs of their FP32 blocks times an
FP32 direction. Blocks of a column are merged and multiplied in FP64, so the
only rounding left is the result's to FP32: 2^-24 of its size, plus 1e-12 of the
terms' sizes for the FP64 sums. (Merged blocks rounded to FP32 and multiplied in
FP32 are off by several times that.) Rows with one pair and with hundreds.
"""
import numpy as np
import pytest

from test_gpu_pcg_forms import gel, plate

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ipc():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible MI355X"
    from paper_2411_04776_amd import ipc as I
    I.lib()
    return I


@pytest.mark.parametrize("name", ["gel", "plate"])
def test_one_rounding(ipc, name):
    sc = gel((33, 35, 3), radius=6e-3, subdiv=4) if name == "gel" else plate((20, 22, 3))
    ng = len(sc.X)
    g = ipc.GelScene(sc, precision=ipc.IPC_MIXED)
    g.begin_step(sc.poses[1])
    x = g.x.copy()
    x[ng:, 2] -= 0.7 * sc.dhat
    rng = np.random.default_rng(4)
    x[:ng] += rng.normal(0, 0.05 * sc.dhat, (ng, 3)) * (1 - sc.fixed[:, None])
    kind, v4, g12, H = g.barrier_pairs(x)
    v = np.zeros_like(x)
    v[ng:] = rng.normal(size=v[ng:].shape).astype(np.float32)
    want, size = np.zeros_like(x), np.zeros_like(x)
    d = v[v4].reshape(-1, 12)
    np.add.at(want, v4.ravel(), np.einsum("kij,kj->ki", H, d).reshape(-1, 3))
    np.add.at(size, v4.ravel(), np.einsum("kij,kj->ki", np.abs(H), np.abs(d)).reshape(-1, 3))
    err = np.abs(g.hess_apply(x, v) - want)[:ng]
    want, size = want[:ng], size[:ng]
    rows = size.max(axis=1) > 0
    entries = np.bincount(v4[v4 < ng].ravel(), minlength=ng)
    over = err[rows] / (2.0 ** -24 * np.abs(want[rows]) + 1e-12 * size[rows])
    print("contact bits", name, len(kind), "pairs,", rows.sum(), "gel rows of up to", entries.max(), "entries, largest error",
          over.max(), "of the bound", flush=True)
    assert rows.sum() >= 16 and entries.max() >= 3
    assert over.max() <= 1.0
    g.close()
