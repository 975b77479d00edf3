"""Particles that have left their tile's staged region, in large numbers: the workgroups'
lists in LDS (and what overflows them), the escape kernel's short lists and its deposit boxes,
and the workgroups that push their own (2D boxes of up to 2^20 slots), against the split path
on a copy of the same slots (which uses neither tiles nor lists).

Tolerances: the arithmetic per particle is the same in both paths, so FP64 agrees to the order
of the sums (1e-11 of each component's largest value) and particles to 1e-12; FP32 sums are
rounded at different places (2e-5 of the largest value, particles 2e-6)."""
import numpy as np
import pytest
import torch

from gpu_helpers import banner
from paper_2607_13507_amd import lpic as L
from paper_2607_13507_amd import workloads as W
from paper_2607_13507_amd.simulation import DeviceFields, DeviceSpecies, Simulation, grid_struct

pytestmark = pytest.mark.gpu
CURRENT = ("jx", "jy", "jz")

CASES = [  # ndim, nx, ny, ppc, order, share of the particles moved away
    (2, 512, 256, 9, 2, 0.004), (2, 512, 256, 9, 2, 0.4), (2, 512, 256, 9, 1, 1.0),
    (2, 100, 60, 9, 2, 0.5), (3, 40, 0, 4, 2, 0.01), (3, 40, 0, 4, 1, 0.6),
]
# 3D rounds of a workgroup over long chunks, ragged at their end: few, some and all particles
# waiting for the escape list; compiled strides (halo 3 and, FP32, 4) and runtime strides
ROUNDS = [(3, 16, 0, 27, order, share, tile) for order, share, tile in [
    (2, 0.002, (8, 4, 4, 3)), (1, 0.2, (8, 4, 4, 3)), (2, 1.0, (8, 4, 4, 3)), (2, 0.1, (8, 4, 4, 4)),
    (2, 0.3, (4, 4, 4, 3)), (1, 0.03, (4, 8, 4, 3))]]
ROUNDS.append((3, 16, 0, 343, 2, 0.3, (8, 4, 4, 3)))   # more than 64 rounds of 512 in a chunk


@pytest.mark.parametrize("prec", [L.F64_ABS, L.F32_CELLOFS], ids=["f64", "f32"])
@pytest.mark.parametrize("ndim,nx,ny,ppc,order,share,tile", [c + (None,) for c in CASES] + ROUNDS)
def test_escaped_particles(prec, ndim, nx, ny, ppc, order, share, tile):
    if prec == L.F64_ABS and tile == (8, 4, 4, 4):
        pytest.skip("the region needs more LDS than a CU has")
    banner(f"escapes {ndim}D {nx}x{ny} ppc={ppc} order={order} share={share} prec={prec}")
    wl = (W.thermal_2d(nx=nx, ny=ny, dx=0.1, ppc=ppc, T=0.3, order=order, seed=31) if ndim == 2
          else W.thermal_3d(n=nx, dx=0.1, ppc=ppc, T=0.3, order=order, seed=32))
    wl.fields = W.random_fields(wl.ncell, 33, 0.5)
    grid = grid_struct(wl)
    F, G = DeviceFields(wl, prec), DeviceFields(wl, prec)
    a = DeviceSpecies.from_init(grid, wl.species[0], prec)
    n, st = a.n, a.struct()
    alt = a.like()
    t = L.Tiling(16, 16, 1, 5, 1024, 0) if ndim == 2 else L.Tiling(8, 4, 4, 3, 1024, 0)
    if tile:
        t = L.Tiling(*tile, 50000, 0)
    off = torch.empty(L.lpic_num_tiles(grid, t) + 2, dtype=torch.int32, device="cuda")
    size = L.lpic_sort_ws_bytes(grid, t, n)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    L.lpic_sort_tiles(grid, st, alt.struct(), t, off.data_ptr(), ws.data_ptr(), size, prec)
    torch.cuda.synchronize()
    a = alt                                    # the sorted arrays
    # a share of the slots, contiguous ranges among them, moves half a box away
    pos = a.positions(grid)
    rng = np.random.default_rng(3)
    move = rng.random(n) < share
    move[n // 3:n // 3 + int(0.2 * share * n)] = True
    for d in range(ndim):
        box = (grid.nx * grid.dx, grid.ny * grid.dy, grid.nz * grid.dz)[d]
        p = pos[d] + 0.5 * box * move
        pos[d] = np.where(p >= box, p - box, p)
    a.load_positions(grid, pos[0], pos[1], pos[2] if ndim == 3 else None)
    b = a.like()
    for k, v in a.a.items():
        b.a[k].copy_(v)
    size = L.lpic_fused_ws_bytes(grid, t, n)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    ke = torch.zeros(1, dtype=torch.float64, device="cuda")
    L.lpic_push_deposit_fused(grid, F.struct(), a.struct(), t, off.data_ptr(), ws.data_ptr(), size,
                              1, ke.data_ptr(), prec)
    size = L.lpic_old_state_bytes(ndim, n, prec)
    old = torch.empty(size, dtype=torch.uint8, device="cuda")
    L.lpic_gather_push(grid, G.struct(), b.struct(), old.data_ptr(), size, prec)
    L.lpic_deposit_esirkepov(grid, G.struct(), b.struct(), old.data_ptr(), size, 1, prec)
    torch.cuda.synchronize()
    tol, ptol = (1e-11, 1e-12) if prec == L.F64_ABS else (2e-5, 2e-6)
    f, g = F.numpy(), G.numpy()
    for k in CURRENT + ("rho0", "rho1"):
        scale = np.abs(g[k]).max()
        assert np.abs(f[k] - g[k]).max() <= tol * scale, k
    pa, pb = a.positions(grid), b.positions(grid)
    for d in range(ndim):
        box = (grid.nx * grid.dx, grid.ny * grid.dy, grid.nz * grid.dz)[d]
        e = pa[d] - pb[d]
        assert np.abs(e - box * np.round(e / box)).max() <= ptol * box, d
    u2 = 0.0
    for k in ("ux", "uy", "uz"):
        ua, ub = a.numpy(k).astype(np.float64), b.numpy(k).astype(np.float64)
        assert np.abs(ua - ub).max() <= ptol * max(1.0, np.abs(ub).max()), k
        u2 = u2 + ub * ub
    w = b.numpy("w").astype(np.float64)
    want = (w * u2 / (1.0 + np.sqrt(1.0 + u2))).sum()
    assert abs(ke.item() - want) <= (1e-11 if prec == L.F64_ABS else 1e-6) * want


@pytest.mark.parametrize("prec", [L.F64_ABS, L.F32_CELLOFS], ids=["f64", "f32"])
@pytest.mark.parametrize("nx,ny,ppc,order,chunk", [(48, 32, 8, 2, 1024), (40, 20, 3, 1, 100),
                                                   (16, 16, 40, 2, 257), (20, 12, 1, 2, 64)])
def test_stream_in_cell_order(prec, nx, ny, ppc, order, chunk):
    """The stateless fused call on tiles whose particles lie cell by cell (dealt to the waves in
    turn), in full and ragged batches, against the split path on the same slots."""
    banner(f"cell order {nx}x{ny} ppc={ppc} chunk={chunk} prec={prec}")
    wl = W.thermal_2d(nx=nx, ny=ny, dx=0.1, ppc=ppc, T=0.1, order=order, seed=41)
    wl.fields = W.random_fields(wl.ncell, 42, 0.5)
    s = wl.species[0]
    tile = (np.floor(s.y / 0.1).astype(int) // 16) * -(-nx // 16) + np.floor(s.x / 0.1).astype(int) // 16
    by = np.argsort(tile, kind="stable")
    for k in ("x", "y", "ux", "uy", "uz", "w"):
        setattr(s, k, np.ascontiguousarray(getattr(s, k)[by]))
    grid = grid_struct(wl)
    F, G = DeviceFields(wl, prec), DeviceFields(wl, prec)
    a, b = (DeviceSpecies.from_init(grid, s, prec) for _ in range(2))
    t = L.Tiling(16, 16, 1, 5, chunk, 0)
    nt = L.lpic_num_tiles(grid, t)
    off = np.concatenate([[0], np.cumsum(np.bincount(tile, minlength=nt)), [a.n]]).astype(np.int32)
    off = torch.from_numpy(off).cuda()
    size = L.lpic_fused_ws_bytes(grid, t, a.n)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    L.lpic_push_deposit_fused(grid, F.struct(), a.struct(), t, off.data_ptr(), ws.data_ptr(), size,
                              1, None, prec)
    size = L.lpic_old_state_bytes(2, a.n, prec)
    old = torch.empty(size, dtype=torch.uint8, device="cuda")
    L.lpic_gather_push(grid, G.struct(), b.struct(), old.data_ptr(), size, prec)
    L.lpic_deposit_esirkepov(grid, G.struct(), b.struct(), old.data_ptr(), size, 1, prec)
    torch.cuda.synchronize()
    tol, ptol = (1e-11, 1e-12) if prec == L.F64_ABS else (2e-5, 2e-6)
    f, g = F.numpy(), G.numpy()
    for k in CURRENT + ("rho0", "rho1"):
        assert np.abs(f[k] - g[k]).max() <= tol * np.abs(g[k]).max(), k
    for k in ("ux", "uy", "uz"):
        assert np.abs(a.numpy(k) - b.numpy(k)).max() <= ptol, k


def _two_species(nx, ny, ppc, orders, seed):
    wl = W.thermal_2d(nx=nx, ny=ny, dx=0.1, ppc=ppc, T=0.3, order=orders[0], seed=seed)
    ions = W.thermal_2d(nx=nx, ny=ny, dx=0.1, ppc=ppc, T=0.3, order=orders[1], seed=seed + 1)
    ions.species[0].q, ions.species[0].m = 1.0, 4.0
    wl.species.append(ions.species[0])
    wl.fields = W.random_fields(wl.ncell, seed + 2, 0.5)
    return wl


@pytest.mark.parametrize("prec", [L.F64_ABS, L.F32_CELLOFS], ids=["f64", "f32"])
@pytest.mark.parametrize("nx,ny", [(256, 192), (288, 256)], ids=["own", "list"])
def test_escapes_of_two_species(nx, ny, prec):
    """Two boxes of two species each (different orders), several chunks of a tile and a species
    per workgroup: a share of one species of a tile moved away, then of both, with diagnostics.
    `own`: 912,384 slots, pushed by the workgroup that meets them, which empties its list when
    the species changes inside a tile; `list`: 1,354,752 slots, the shared list."""
    banner(f"escapes of two species {nx}x{ny} prec={prec}")
    wls = [_two_species(nx, ny, 9, (2, 1), 51), _two_species(48, 32, 9, (1, 2), 54)]

    def sim():
        return Simulation(wls, prec=prec, tiling=(16, 16, 1), halo=5, chunk=256,
                          sort_interval=1000, diag_interval=1, use_graph=False)
    a, b = sim(), sim()
    b.register_hook("INTERPOLATOR", lambda *_: 0)      # the split path
    a.step(1)
    b.step(1)
    rng = np.random.default_rng(7)
    tol, ptol = (1e-11, 1e-12) if prec == L.F64_ABS else (2e-5, 2e-6)
    for moved in ((0, 3), (0, 1, 2, 3)):
        e0 = a.stats()["halo_escapes"]
        away = 0
        for i in moved:
            s, g = a.current(i), a.grids[a.species_run[i]]
            move = rng.random(s.n) < 0.3
            away += int(move.sum())
            pos = s.positions(g)
            for d, box in enumerate((g.nx * g.dx, g.ny * g.dy)):
                p = pos[d] + 0.5 * box * move
                pos[d] = np.where(p >= box, p - box, p)
            s.load_positions(g, pos[0], pos[1])
        for i in range(4):                             # the same slots in both
            for k, v in a.current(i).a.items():
                b.current(i).a[k].copy_(v)
        for r in range(2):
            for k, v in a.fields[r].t.items():
                b.fields[r].t[k].copy_(v)
        a.step(1)
        b.step(1)
        torch.cuda.synchronize()
        assert a.stats()["fused"] and not b.stats()["fused"]
        assert a.stats()["halo_escapes"] - e0 >= 0.5 * away, moved
        for r in range(2):
            f, g = a.fields[r].numpy(), b.fields[r].numpy()
            for k in g:
                assert np.abs(f[k] - g[k]).max() <= tol * np.abs(g[k]).max(), (moved, r, k)
            ka, kb = (x.diagnostics(r)["kinetic_energy"] for x in (a, b))
            assert abs(ka - kb) <= (1e-11 if prec == L.F64_ABS else 1e-6) * kb, (moved, r)
        for i in range(4):
            sa, sb, g = a.current(i), b.current(i), a.grids[a.species_run[i]]
            for d, box in enumerate((g.nx * g.dx, g.ny * g.dy)):
                e = sa.positions(g)[d] - sb.positions(g)[d]
                assert np.abs(e - box * np.round(e / box)).max() <= ptol * box, (moved, i, d)
            for k in ("ux", "uy", "uz"):
                ua, ub = sa.numpy(k).astype(np.float64), sb.numpy(k).astype(np.float64)
                assert np.abs(ua - ub).max() <= ptol * max(1.0, np.abs(ub).max()), (moved, i, k)
    a.close()
    b.close()
