"""The reconstruction at the edges of its split over waves.

1D-3V: velocity rows cut into chunks of two rows (small grids, with a ragged
last chunk) and of 16 and more, grids of up to 64 columns as one ring of lanes
and wider ones in strips with a halo, rows that are staged and rows that are
not.  N = f D and D against the oracle's from the exported markers, rho against
the moments of the oracle's f; bounds as for a step elsewhere: 1e-12 normwise
in FP64, 1e-5 in the FP32 form.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from checks import nrel
from paper_1804_03901_amd import avl, inputs

pytestmark = pytest.mark.gpu


def _check(w, precision, steps=2):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    x, v, f = inputs.markers(w)
    print(f"[case] {w.name} nx={w.nx} nv={w.nv} n={x.size} prec={precision}", flush=True)
    sim = avl.Simulation(w, x, v.reshape(-1), f, precision=precision)
    sim.step(steps)
    fg, Dg = (t.double().cpu().numpy() for t in sim.reconstruct(want_D=True))
    rho = sim.moments().double().cpu().numpy()
    sim.check()
    xs, vs, fs = (t.double().cpu().numpy() for t in sim.markers())
    g = oracle.Grid.from_workload(w)
    No, Do, fo = oracle.reconstruct(g, xs, vs.reshape(w.vdim, -1), fs)
    rho_o, _, _ = oracle.moments(g, fo)
    tol = 1e-12 if precision == avl.AVL_FP64 else 1e-5
    assert nrel(Dg, Do) <= tol and nrel(fg * Dg, No) <= tol
    assert nrel(rho, rho_o) <= tol
    sim.close()


@pytest.mark.parametrize("precision", [avl.AVL_FP64, avl.AVL_FP32])
@pytest.mark.parametrize("nx,nv,ppc", [
    (8, (2, 2, 2), 3), (32, (5, 3, 2), 2), (64, (33, 4, 3), 1), (64, (7, 2, 2), 9),
    (128, (9, 3, 3), 2), (64, (70, 44, 40), 1), (128, (37, 24, 24), 1),
])
def test_3v_chunks_and_ring(nx, nv, ppc, precision):
    w = inputs.two_stream_3v(nx=nx, nv=8, ppc=ppc, seed=31).replace(name="ts3v_split", nv=nv)
    _check(w, precision)
