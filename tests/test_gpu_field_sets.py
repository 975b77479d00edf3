"""The fused 2D field update between two field sets against the same steps with separate
in-place kernels (LPIC_FIELD_SEPARATE): boxes that no tile divides (1 + 64 k columns with Mur
ends among them), layers and antennas at odd places, odd and even numbers of fused updates in
a call, several calls in a row, a box without species, and a window that has moved.

The arithmetic per cell is the same in both paths: tolerances as in the tests of the fused
update on boxes that tiles divide (FP64 1e-12, FP32 1e-5)."""
import numpy as np
import pytest
import torch

from gpu_helpers import banner
from paper_2607_13507_amd import lpic as L
from paper_2607_13507_amd import workloads as W
from paper_2607_13507_amd.simulation import Simulation
from test_gpu_field_fused import FIELDS, LASER, PNAME, _rel

pytestmark = pytest.mark.gpu
PRECS = [L.F64_ABS, L.F32_CELLOFS]


def _wl(nx, ny, ends, seed=61):
    wl = W.thermal_2d(nx=nx, ny=ny, dx=0.1, ppc=2, T=0.2, order=2, seed=seed)
    wl.fields = W.random_fields(wl.ncell, seed + 1, 0.5)
    if ends != "periodic":
        wl.open_x = True
        wl.laser = dict(LASER, ia=10 if ends == "pml" else 3)
    if ends == "pml":
        wl.pml = dict(cells=7, order=3, a_order=1, kappa_max=2.0, a_max=0.3)
    for s in wl.species:
        s.w = s.w * (1.0 + 1e-3 * np.arange(s.n) / s.n)
    return wl


def _sim(wls, prec, flags, graph, diag=5):
    return Simulation(wls, prec=prec, tiling=(8, 8, 1), halo=4, chunk=128, sort_interval=4,
                      diag_interval=diag, use_graph=graph, flags=flags)


def _compare(fused, sep, prec, what):
    tol = 1e-12 if prec == L.F64_ABS else 1e-5
    fa, fb = fused.fields[0].numpy(), sep.fields[0].numpy()
    for k in FIELDS:
        err = _rel(fa[k], fb[k])
        assert err <= tol, f"{what} {k}: {err}"
    da, db = fused.diagnostics(0), sep.diagnostics(0)
    for k in ("field_energy", "kinetic_energy"):
        assert da[k] == pytest.approx(db[k], rel=tol, abs=1e-300), (what, k)
    for i in range(len(fused.species)):
        # particles matched by weight, and by position where FP32 weights coincide
        order = []
        for sim in (fused, sep):
            x, y = sim.positions(i)
            at = np.lexsort((y, x, sim.current(i).numpy("w")))
            order.append(at[x[at] >= 0.0])      # the live ones (dead slots keep no order)
        assert order[0].size == order[1].size, (what, i)
        for d in range(2):
            pa, pb = fused.positions(i)[d][order[0]], sep.positions(i)[d][order[1]]
            assert np.abs(pa - pb).max(initial=0) <= 10 * tol, (what, i, d)
        for k in ("ux", "uy", "uz"):
            ua, ub = (s.current(i).numpy(k)[o] for s, o in zip((fused, sep), order))
            assert _rel(ua, ub) <= 10 * tol, (what, i, k)


@pytest.mark.parametrize("prec", PRECS, ids=PNAME.get)
@pytest.mark.parametrize("nx,ny,ends", [(100, 37, "periodic"), (65, 18, "mur"), (129, 20, "mur"),
                                        (97, 33, "pml"), (21, 9, "periodic"), (30, 70, "mur"),
                                        (1000, 17, "pml")])
@pytest.mark.parametrize("calls", [(13,), (12, 1, 2, 7)], ids=["one", "several"])
def test_ragged_tiles_match_separate_kernels(prec, nx, ny, ends, calls):
    banner(f"field sets {nx}x{ny} {ends} prec={PNAME[prec]} calls={calls}")
    wl = _wl(nx, ny, ends)
    graph = len(calls) > 1
    fused, sep = _sim(wl, prec, 0, graph), _sim(wl, prec, L.FIELD_SEPARATE, graph)
    for n in calls:
        fused.step(n)
        sep.step(n)
    torch.cuda.synchronize()
    assert fused.stats()["field_tile"] != (0, 0)
    _compare(fused, sep, prec, ends)
    fused.close()
    sep.close()


@pytest.mark.parametrize("prec", PRECS, ids=PNAME.get)
def test_no_species(prec):
    banner(f"field sets without species prec={PNAME[prec]}")
    wl = _wl(70, 40, "mur")
    wl.species = []
    wl.fields["jx"] = np.linspace(-1.0, 1.0, wl.ncell)      # a current left in the caller's array
    fused, sep = _sim(wl, prec, 0, True, 6), _sim(wl, prec, L.FIELD_SEPARATE, True, 6)
    for n in (8, 3, 10):
        fused.step(n)
        sep.step(n)
    torch.cuda.synchronize()
    _compare(fused, sep, prec, "no species")
    fused.close()
    sep.close()


@pytest.mark.parametrize("nx", [96, 129])
def test_moved_window(nx):
    # FP64 only: the pulse has left the box by the end, and FP32 rounding of what passed
    # through is not small against what is left
    prec = L.F64_ABS
    banner(f"field sets under a moving window nx={nx}")
    wl = W.wakefield_2d(nx=nx, ny=24, ppc=4, moving=True, spare=4096, a0=1.0, T=1e-3,
                        pulse_cells=nx // 3)
    wl.species[0].w[:-4096] *= 1.0 + 1e-3 * np.arange(wl.species[0].n - 4096) / wl.species[0].n
    fused, sep = _sim(wl, prec, 0, True, 4), _sim(wl, prec, L.FIELD_SEPARATE, True, 4)
    for m in (5, 1, 40):
        for sim in (fused, sep):
            sim.step(7)
            sim.window_shift(0, m, dict(species=0, ppc_x=2, ppc_y=2, density=0.01))
            sim.step(6)
    torch.cuda.synchronize()
    tol = 1e-12
    fa, fb = fused.fields[0].numpy(), sep.fields[0].numpy()
    for k in ("ex", "ey", "ez", "bx", "by", "bz", "jx", "jy"):
        scale = max(np.abs(fb[k]).max(), 1e-3 * np.abs(fb["ey"]).max())
        assert np.abs(fa[k] - fb[k]).max() <= tol * scale, k
    fused.close()
    sep.close()
