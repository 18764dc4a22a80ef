"""The grid of a run's sums follows the run's own weights in long rows.

Rows of up to 1152 FP64 markers may take one bound for all their runs where the
weights lie within a factor of four; longer ones take a shared bound only where it is
each run's own, whether the kernel stages them whole (up to 1536 markers) or not.  A
weight raised from below 2 to 3.9 in one column then leaves every cell out of its
reach as it was, bit for bit; a coarser shared bound would move the last bits of some.
(The first and last target rows are left out: the markers of half a cell beyond them
make short rows.)
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1804_03901_amd import avl, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ppc", [(64, 20), (64, 30), (128, 21), (256, 40)])
def test_long_rows_keep_each_runs_own_bound(nx, ppc):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    w = inputs.bump_on_tail(nx=nx, nv=24, ppc=ppc, seed=41)
    x, v, _ = inputs.markers(w)
    f = 1.0 + 0.99 * np.random.default_rng(5).random(x.size)
    raised = f.copy()
    col = 40
    pick = np.nonzero((x >= col * w.dx) & (x < (col + 1) * w.dx))[0]
    # one marker of that column in every velocity row
    row = np.floor((v.reshape(-1)[pick] - w.vmin[0]) / w.dv(0)).astype(int)
    raised[pick[np.unique(row, return_index=True)[1]]] = 3.9
    print(f"[case] {w.name} n={x.size} raised={int((raised != f).sum())}", flush=True)
    out = []
    for weights in (f, raised):
        sim = avl.Simulation(w, x, v.reshape(-1), weights, precision=avl.AVL_FP64)
        out.append(sim.reconstruct().cpu().numpy())
        sim.close()
    away = [c for c in range(nx) if not col - 2 <= c <= col + 2]
    assert np.array_equal(out[0][1:-1, away], out[1][1:-1, away])
    assert not np.array_equal(out[0], out[1])
