"""The split deposit's node boxes against the FP64 oracle: particles in cell order, shuffled
over the box (no pass fits its nodes), in two far clusters, a box smaller than a window's
reach, one particle, and enough passes that a workgroup keeps its box between them.

Tolerances as for the other kernels against the oracle (FP64 1e-11: only the order of the
sums differs; FP32 2e-5: the shapes and factors are single precision in both cases)."""
import numpy as np
import pytest
import torch

from gpu_helpers import banner, compare_fields, device_state
from paper_2607_13507_amd import lpic as L
from paper_2607_13507_amd import workloads as W

pytestmark = pytest.mark.gpu


def _arrange(s, how, rng):
    n = s.n
    if how == "shuffled":
        order = rng.permutation(n)
    elif how == "clusters":       # alternating halves of the list: two regions in every pass
        order = np.arange(n).reshape(2, -1).T.reshape(-1) if n % 2 == 0 else np.arange(n)
    else:
        order = np.arange(n)
    for k in ("x", "y", "z", "ux", "uy", "uz", "w"):
        v = getattr(s, k)
        if v is not None:
            setattr(s, k, np.ascontiguousarray(v[order]))


CASES = [  # ndim, order, nx, ny, ppc, arrangement
    (2, 2, 300, 70, 3, "cells"), (2, 1, 300, 70, 3, "shuffled"), (2, 2, 300, 70, 4, "clusters"),
    (2, 2, 6, 5, 9, "cells"), (2, 1, 257, 9, 1, "cells"), (2, 2, 1024, 520, 2, "cells"),
    (3, 2, 24, 0, 2, "cells"), (3, 1, 24, 0, 2, "shuffled"), (3, 2, 24, 0, 2, "clusters"),
    (3, 2, 5, 0, 3, "cells"),
]


@pytest.mark.parametrize("prec", [L.F64_ABS, L.F32_CELLOFS], ids=["f64", "f32"])
@pytest.mark.parametrize("ndim,order,nx,ny,ppc,how", CASES)
def test_deposit_boxes(prec, ndim, order, nx, ny, ppc, how):
    banner(f"deposit boxes {ndim}D order={order} {nx}x{ny} ppc={ppc} {how} prec={prec}")
    wl = (W.thermal_2d(nx=nx, ny=ny, dx=0.1, ppc=ppc, T=0.3, order=order, seed=21) if ndim == 2
          else W.thermal_3d(n=nx, dx=0.1, ppc=ppc, T=0.3, order=order, seed=22))
    _arrange(wl.species[0], how, np.random.default_rng(1))
    grid, F, S, orc = device_state(wl, prec, random_fields_seed=7, field_scale=0.5)
    d, o = S[0], orc.species[0]
    size = L.lpic_old_state_bytes(ndim, d.n, prec)
    old = torch.empty(size, dtype=torch.uint8, device="cuda")
    L.lpic_gather_push(grid, F.struct(), d.struct(), old.data_ptr(), size, prec)
    L.lpic_deposit_esirkepov(grid, F.struct(), d.struct(), old.data_ptr(), size, 1, prec)
    torch.cuda.synchronize()
    orc.zero_currents()
    orc.push_deposit(o)
    compare_fields(F, orc, prec, keys=("jx", "jy", "jz", "rho0", "rho1"), what=how)


@pytest.mark.parametrize("prec", [L.F64_ABS, L.F32_CELLOFS], ids=["f64", "f32"])
def test_deposit_of_one_and_of_dead(prec):
    banner(f"deposit of one particle among dead slots prec={prec}")
    wl = W.thermal_2d(nx=40, ny=36, dx=0.1, ppc=1, T=0.3, order=2, seed=23)
    s = wl.species[0]
    keep = 777
    s.x[np.arange(s.n) != keep] = -1.0      # a pass with one live lane, others with none
    grid, F, S, orc = device_state(wl, prec, random_fields_seed=8, field_scale=0.5)
    d, o = S[0], orc.species[0]
    size = L.lpic_old_state_bytes(2, d.n, prec)
    old = torch.empty(size, dtype=torch.uint8, device="cuda")
    L.lpic_gather_push(grid, F.struct(), d.struct(), old.data_ptr(), size, prec)
    L.lpic_deposit_esirkepov(grid, F.struct(), d.struct(), old.data_ptr(), size, 1, prec)
    torch.cuda.synchronize()
    orc.zero_currents()
    orc.push_deposit(o)
    compare_fields(F, orc, prec, keys=("jx", "jy", "jz", "rho0", "rho1"), what="one")
