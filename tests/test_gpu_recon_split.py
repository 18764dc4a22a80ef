"""The reconstruction at the edges of its split over waves.

1D-1V: each capacity of the kernels (by markers a row and marker count), grids
of up to 64 columns as one ring of lanes, and rows beyond the capacity, staged
in pieces: by a concentrated placement, by many markers a cell, and by a wrapped
run longer than a wavefront; f spread over many exponents and over few.
Batches: chunks of rows longer than an instance's own.
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


def _check(w, precision, steps=2, markers=None, options=0):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    x, v, f = inputs.markers(w) if markers is None else markers
    print(f"[case] {w.name} nx={w.nx} nv={w.nv} n={x.size} prec={precision}", flush=True)
    sim = avl.Simulation(w, x, v.reshape(-1), f, precision=precision, options=options)
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


@pytest.mark.parametrize("form", ["fp64", "fp32", "kahan"])
@pytest.mark.parametrize("nx,nv,ppc,placement", [
    (8, 2, 1, "cells"), (16, 30, 3, "cells"), (32, 9, 90, "cells"), (64, 33, 4, "cells"), (64, 20, 30, "peak"),
    (128, 70, 4, "peak"), (128, 50, 7, "cells"), (256, 40, 11, "peak"), (64, 40, 16, "cells"), (128, 60, 17, "cells"),
    (256, 30, 20, "cells"), (128, 20, 27, "cells"), (128, 12, 70, "cells"), (1024, 520, 4, "cells"),
])
def test_1v_capacities_and_pieces(nx, nv, ppc, placement, form):
    w = inputs.bump_on_tail(nx=nx, nv=nv, ppc=ppc, seed=33).replace(L=0.25 * nx)
    x, v, f = inputs.markers(w)
    if placement == "peak":
        # a sixteenth of the velocity range holds most markers, f over 13 binades
        rng = np.random.default_rng(nx + ppc)
        v = 0.5 * (w.vmax[0] + w.vmin[0]) + (w.vmax[0] - w.vmin[0]) / 16 * rng.standard_normal(v.shape)
        f = np.exp(9.0 * rng.random(f.size) - 8.0)
    precision = avl.AVL_FP64 if form == "fp64" else avl.AVL_FP32
    _check(w, precision, markers=(x, v, f), options=avl.AVL_OPT_KAHAN32 if form == "kahan" else 0)


def test_1v_two_rows_in_flight():
    _check(inputs.bump_on_tail(nx=1024, nv=2050, ppc=4, seed=34), avl.AVL_FP64, steps=1)


@pytest.mark.parametrize("precision", [avl.AVL_FP64, avl.AVL_FP32])
def test_batch_chunks_longer_than_an_instances_own(precision):
    """Rows enough for a batch to walk them in longer chunks than each instance
    alone would: rho to the rounding of its chunk sums, f from the same markers."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ws = [inputs.bump_on_tail(nx=nx, nv=nv, ppc=2, seed=41 + i).replace(name=f"b{i}")
          for i, (nx, nv) in enumerate([(256, 2000), (256, 1801), (64, 900), (512, 1300), (256, 2400)])]
    mk = [inputs.markers(w) for w in ws]
    print(f"[case] batch of {len(ws)} prec={precision}", flush=True)
    b = avl.Batch(ws, [(x, v.reshape(-1), f) for x, v, f in mk], precision=precision)
    b.step(1)
    b.check()
    for i, w in enumerate(ws):
        sim = avl.Simulation(w, mk[i][0], mk[i][1].reshape(-1), mk[i][2], precision=precision)
        sim.step(1)
        rho_s, rho_b = (t.double().cpu().numpy() for t in (sim.field()[1], b.instance(i).field()[1]))
        assert nrel(rho_b, rho_s) <= 1e-12, w.name
        sim.close()
