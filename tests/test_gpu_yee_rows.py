"""Field half updates four cells of a row at a time, and one at a time, against the oracle:
rows of whole groups, one group wide, and not of whole groups; open (Mur) ends; arrays that
are not aligned to a group; J and charge cleared on the way.

Tolerances as for the other single kernels (FP64 1e-11, FP32 2e-5 of the largest value)."""
import numpy as np
import pytest
import torch

from gpu_helpers import TOL, banner
from oracle import OracleSim
from paper_2607_13507_amd import lpic as L
from paper_2607_13507_amd import workloads as W
from paper_2607_13507_amd.simulation import grid_struct, torch_dtype

pytestmark = pytest.mark.gpu
KEYS = ("ex", "ey", "ez", "bx", "by", "bz", "jx", "jy", "jz")

CASES = [  # ndim, nx, ny, nz, open_x, first element of every array
    (2, 44, 9, 1, 0, 0), (2, 41, 9, 1, 0, 0), (2, 44, 9, 1, 0, 1), (2, 8, 5, 1, 1, 0),
    (2, 260, 7, 1, 1, 0), (2, 261, 7, 1, 1, 0), (3, 4, 6, 5, 0, 0), (3, 24, 10, 9, 0, 0),
    (3, 24, 10, 9, 1, 0), (3, 25, 10, 9, 1, 0), (3, 24, 10, 9, 0, 3),
]


@pytest.mark.parametrize("prec", [L.F64_ABS, L.F32_CELLOFS], ids=["f64", "f32"])
@pytest.mark.parametrize("ndim,nx,ny,nz,open_x,shift", CASES)
def test_yee_rows(prec, ndim, nx, ny, nz, open_x, shift):
    banner(f"yee rows {nx}x{ny}x{nz} open={open_x} shift={shift} prec={prec}")
    wl = (W.thermal_2d(nx=nx, ny=ny, dx=0.1, ppc=1, seed=5) if ndim == 2
          else W.thermal_3d(n=4, dx=0.1, ppc=1, seed=5))
    wl.nx, wl.ny, wl.nz, wl.open_x, wl.species = nx, ny, nz, bool(open_x), []
    wl.fields = W.random_fields(wl.ncell, 7, names=KEYS)
    grid, dt = grid_struct(wl), torch_dtype(prec)
    arr = {}
    for k in KEYS + ("rho0", "rho1"):
        arr[k] = torch.empty(wl.ncell + 8, dtype=dt, device="cuda")[shift:shift + wl.ncell]
        arr[k].copy_(torch.from_numpy(wl.fields.get(k, np.ones(wl.ncell))).to(dt))
    F = L.Fields(*[arr[k].data_ptr() for k in KEYS + ("rho0", "rho1")])
    orc = OracleSim.from_workload(wl)
    for k in KEYS:
        orc.f[k][:] = arr[k].double().cpu().numpy()
    for flags in (0, L.YEE_ZERO_J):
        L.lpic_yee_update_EB(grid, F, 0, 0.5, flags, prec)
        orc.yee_e(0.5)
        L.lpic_yee_update_EB(grid, F, 1, 0.5, 0, prec)
        orc.yee_b(0.5)
    for k in KEYS[:6]:
        want = orc.f[k]
        err = np.abs(arr[k].double().cpu().numpy() - want).max() / np.abs(want).max()
        assert err <= TOL[prec], (k, err)
    for k in KEYS[6:] + ("rho0", "rho1"):
        assert torch.count_nonzero(arr[k]).item() == 0, k
