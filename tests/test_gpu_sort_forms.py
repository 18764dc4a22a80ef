"""Which sort kernels a step takes: every choice against the oracle.

The sums N = f D and D of a state against the oracle's, from the exported markers,
hold only if each marker lies in the run of its cell; bounds as for a step
elsewhere, 1e-12 normwise in FP64 and 1e-5 in the FP32 form.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from checks import nrel
from paper_1804_03901_amd import avl, inputs

pytestmark = pytest.mark.gpu


def _sim(w, markers, precision, **kw):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    x, v, f = markers
    print(f"[case] {w.name} nx={w.nx} nv={w.nv} n={x.size} prec={precision}", flush=True)
    return avl.Simulation(w, x, v.reshape(-1), f, precision=precision, **kw)


def _check(sim, w, precision):
    sim.check()
    xs, vs, fs = (t.double().cpu().numpy() for t in sim.markers())
    fg, Dg = (t.double().cpu().numpy() for t in sim.reconstruct(want_D=True))
    No, Do, _ = oracle.reconstruct(oracle.Grid.from_workload(w), xs, vs.reshape(w.vdim, -1), fs)
    tol = 1e-12 if precision == avl.AVL_FP64 else 1e-5
    assert nrel(Dg, Do) <= tol and nrel(fg * Dg, No) <= tol


def _kick(sim, w):
    """Largest kick of the current field, in velocity cells."""
    return float(sim.field()[0].abs().max()) * abs(w.q / w.m) * w.dt / w.dv(0)


@pytest.mark.parametrize("nx,nv", [(8, 18300), (8, 18420), (8, 18500), (512, 17950)])
def test_drift_table_that_leaves_the_block_kernels_no_room(nx, nv):
    # FP32 drift and field tables of 146 to 148 KB: the wave kernels' maps still fit a
    # block's 160 KB, the block kernels' map fits the first case only
    w = inputs.paper_landau(ppc=1).replace(nx=nx, nv=(nv, 1, 1))
    sim = _sim(w, inputs.markers(w), avl.AVL_FP32)
    assert _kick(sim, w) > 1.0
    for graph in (False, True):
        sim.step(2, graph=graph)
        _check(sim, w, avl.AVL_FP32)
    sim.close()


@pytest.mark.parametrize("precision", [avl.AVL_FP64, avl.AVL_FP32])
@pytest.mark.parametrize("nx,nv,ppc", [(64, 700, 4), (512, 1500, 3), (16, 300, 7)])
def test_field_that_weakens_and_grows_after_loading(nx, nv, ppc, precision):
    # loaded with kicks of more than a velocity cell, then stepped by fields on
    # both sides of one cell, directly and by graph replay
    w = inputs.paper_landau(ppc=ppc).replace(nx=nx, nv=(nv, 1, 1), mode_amplitude=0.5)
    sim = _sim(w, inputs.markers(w), precision)
    loaded = _kick(sim, w)
    assert loaded > 1.0
    rho = sim.field()[1].clone()
    for kick, graph in ((0.05, False), (1.5, False), (0.99, True), (6.0, True), (0.3, True)):
        sim.poisson(rho * (kick / loaded))
        assert abs(_kick(sim, w) - kick) < 1e-9 * kick
        sim.step(1, graph=graph)
        _check(sim, w, precision)
    sim.close()


def _crowded(w, n, beyond, seed):
    """n markers: most in three cells, some anywhere, a share `beyond` off the velocity grid."""
    rng = np.random.default_rng(seed)
    x, v = rng.random(n) * w.L, w.vmin[0] + (w.vmax[0] - w.vmin[0]) * rng.random(n)
    crowd = rng.random(n) < 0.8
    cell = rng.integers(0, 3, n)
    x[crowd] = ((cell * (w.nx // 3) + rng.random(n)) * w.dx)[crowd]
    v[crowd] = (w.vmin[0] + (cell + 2 + rng.random(n)) * w.dv(0))[crowd]
    off = rng.random(n) < beyond
    v[off] = (w.vmax[0] + (1.0 + rng.random(n)) * (w.vmax[0] - w.vmin[0]))[off]
    return x, v, 0.1 + rng.random(n)


@pytest.mark.parametrize("nx,nv,n,beyond", [(32, 8, 40000, 0.0), (256, 64, 300001, 0.34), (64, 40, 70000, 0.97),
                                            (128, 30, 2047, 1.0)])
def test_runs_that_span_many_tiles(nx, nv, n, beyond):
    # the FP32 sort records where its tiles start in the runs of the order before:
    # runs of thousands of markers, and an overflow run of up to all of them
    w = inputs.bump_on_tail(nx=nx, nv=nv, ppc=1, seed=61).replace(dt=1e-3)
    sim = _sim(w, _crowded(w, n, beyond, n), avl.AVL_FP32)
    for graph in (False, True, False):
        sim.step(1, graph=graph)
        sim.sort()
        _check(sim, w, avl.AVL_FP32)
    sim.close()


@pytest.mark.parametrize("precision", [avl.AVL_FP64, avl.AVL_FP32])
@pytest.mark.parametrize("nx,nv", [(256, 382), (256, 383), (512, 8190), (512, 8191)])
def test_scan_changes_form(nx, nv, precision):
    # 24 and 25 scan tiles of 4096 buckets (the totals get a launch of their own),
    # 1024 and 1025 (and a scan of their own)
    tiles = (nx * (nv + 1) + 1 + 4095) // 4096
    assert tiles in (24, 25, 1024, 1025)
    w = inputs.bump_on_tail(nx=nx, nv=nv, ppc=1, seed=62)
    rng = np.random.default_rng(nv)
    n = 150001
    v = w.vmin[0] + (w.vmax[0] - w.vmin[0]) * rng.random(n)
    sim = _sim(w, (rng.random(n) * w.L, v, 0.1 + rng.random(n)), precision)
    for graph in (False, True):
        sim.step(2, graph=graph)
        _check(sim, w, precision)
    sim.close()


@pytest.mark.parametrize("precision,nx,nv,ppc", [
    (avl.AVL_FP32, 1024, 512, 10),      # 5 * 2^20 markers: eight a lane in the count
    (avl.AVL_FP32, 1024, 1024, 10),     # 10 * 2^20: and in the scatter
    (avl.AVL_FP64, 1024, 911, 9),       # 2^23 dense markers: the scatter by blocks
    (avl.AVL_FP64, 2048, 512, 9),       # wider grids stay with the waves
    (avl.AVL_FP64, 1024, 1024, 12),     # 12 * 2^20: eight a lane in the count
])
def test_large_sorts(precision, nx, nv, ppc):
    w = inputs.bump_on_tail(nx=nx, nv=nv, ppc=ppc, seed=63)
    sim = _sim(w, inputs.markers_threaded(w), precision)
    sim.step(1)
    sim.step(2, graph=True)
    _check(sim, w, precision)
    sim.close()


@pytest.mark.parametrize("precision,nv,ppc", [(avl.AVL_FP32, 1024, 10), (avl.AVL_FP64, 911, 9)])
def test_large_sorts_carry_identities(precision, nv, ppc):
    # the gradient is a function of the marker multiset: loaded in another order it
    # is the same bit for bit, marker by marker, only if each keeps its identity
    from paper_1804_03901_amd import adjoint
    w = inputs.bump_on_tail(nx=1024, nv=nv, ppc=ppc, seed=64)
    x, v, f = inputs.markers_threaded(w)
    v = v.reshape(-1)
    order = np.random.default_rng(1).permutation(x.size)
    sim = _sim(w, (x, v, f), precision)
    J, grad = adjoint.energy_and_gradient(sim, x, v, f, 2, 2)
    Jp, gradp = adjoint.energy_and_gradient(sim, x[order], v[order], f[order], 2, 2)
    sim.close()
    assert float(J) == float(Jp)
    assert torch.equal(grad[torch.as_tensor(order, device=grad.device)], gradp)
