"""fdetd_deposit_current over the forms a block of samples can take: long runs of one cell (summed with matrix
instructions, runs that are no multiple of four samples), many short runs (a lane per sample), a footprint
beyond the LDS tile and beyond the sort, fewer samples than a block, more modes than a pass, problems of
different grids in one plan, and 4-plane blocks with rho_xy.  Against the oracle; FP64 1e-12 and FP32C 1e-5
relative L2 per plane, as for the other deposition tests (the sums are FP64 in both, FP32C rounds each add)."""
import numpy as np
import pytest

import oracle
from helpers import dev, log, rel_l2

import paper_2605_12132_amd as F
import paper_2605_12132_amd.inputs as I

pytestmark = pytest.mark.gpu
DZ = I.LAMBDA0 / 20


def make(kind, n, nz, nr, rng):
    """Samples z, x, y, q w, v (3), unused: `cells` a few cells with many samples each (on and next to the axis,
    inside, beyond the last row), `bunch` z-ordered around the middle, `spread` unordered over the whole grid."""
    dr = 2 * DZ
    if kind == "cells":
        z = (20 + rng.integers(0, 3, n) + rng.uniform(0.3, 0.4, n)) * DZ
        r = rng.choice([0.0, 0.2, 1.7, 5.3, nr - 1.2, nr + 0.4], n) * dr * rng.uniform(0.99, 1.0, n)
    elif kind == "bunch":
        z = np.sort(0.5 * nz * DZ + 6 * DZ * rng.standard_normal(n))
        r = 3 * dr * np.abs(rng.standard_normal(n))
    else:
        z, r = rng.uniform(-2 * DZ, (nz + 2) * DZ, n), rng.uniform(0, 1.02 * nr * dr, n)
    th = rng.uniform(-np.pi, np.pi, n)
    v = rng.uniform(-0.8, 0.8, (n, 3))
    return np.column_stack([z, r * np.cos(th), r * np.sin(th), rng.uniform(-1, 1, n), v, np.zeros(n)])


@pytest.mark.parametrize("precision", [F.FP64, F.FP32C])
@pytest.mark.parametrize("kind,n,nz,nr,modes,rxy", [
    ("cells", 1, 60, 20, [0, 1], False),          # one sample
    ("cells", 127, 60, 20, [0, 1, 2], True),      # a run's remainder in every cell
    ("cells", 4099, 60, 20, [0, 1, 2, 3], False),  # several blocks, four modes: two passes
    ("bunch", 5000, 120, 24, [0, 1, 2], False),
    ("bunch", 5000, 120, 24, [2, 0], True),
    ("spread", 3000, 300, 90, [0, 1, 2], False),  # footprint beyond the tile and the sort
    ("spread", 3000, 40, 24, [1], True),
])
def test_deposit_current_runs(precision, kind, n, nz, nr, modes, rxy):
    import torch
    rng = np.random.default_rng(n + nz)
    s = make(kind, n, nz, nr, rng)
    cd = torch.complex128 if precision == F.FP64 else torch.complex64
    probs = [F.Problem(nz, nr, m, 8, 8, DZ, 2 * DZ, 0.5 * DZ) for m in modes]
    plan = F.Plan(probs, precision=precision, flags=F.PLAN_SKIP_STABILITY | (F.PLAN_CURRENT_CORRECTION if rxy else 0))
    J = [torch.zeros((4 if rxy else 3, nr, nz), dtype=cd, device="cuda") for _ in modes]
    plan.deposit_current(dev(s, torch.float64), J, eps=0.5)
    torch.cuda.synchronize()
    plan.close()
    tol = 1e-12 if precision == F.FP64 else 1e-5
    for p, m in enumerate(modes):
        g = oracle.Grid(nz=nz, nr=nr, m=m, fd_order=8, taylor_order=8, dz=DZ, dr=2 * DZ, dt=0.5 * DZ)
        wj, wr = oracle.deposit_current(g, s)
        got = J[p].cpu().numpy().astype(np.complex128)
        errs = [rel_l2(got[c], wj[c]) for c in range(3)] + ([rel_l2(got[3], wr)] if rxy else [])
        log(f"deposit runs {kind} n={n} m={m} precision={precision}: {[f'{e:.1e}' for e in errs]}")
        assert max(errs) < tol


@pytest.mark.parametrize("precision", [F.FP64, F.FP32C])
def test_deposit_current_grids_of_one_plan(precision):
    """Problems of two grids, modes of each interleaved: every problem gets its own deposit."""
    import torch
    s = make("bunch", 3000, 100, 20, np.random.default_rng(9))
    shapes = [(100, 20, 0), (140, 30, 1), (140, 30, 0), (100, 20, 2)]
    cd = torch.complex128 if precision == F.FP64 else torch.complex64
    plan = F.Plan([F.Problem(nz, nr, m, 8, 8, DZ, 2 * DZ, 0.5 * DZ) for nz, nr, m in shapes], precision=precision,
                  flags=F.PLAN_SKIP_STABILITY)
    J = [torch.zeros((3, nr, nz), dtype=cd, device="cuda") for nz, nr, _ in shapes]
    plan.deposit_current(dev(s, torch.float64), J, eps=0.25)
    torch.cuda.synchronize()
    plan.close()
    for (nz, nr, m), j in zip(shapes, J):
        g = oracle.Grid(nz=nz, nr=nr, m=m, fd_order=8, taylor_order=8, dz=DZ, dr=2 * DZ, dt=0.5 * DZ)
        want, _ = oracle.deposit_current(g, s, eps=0.25)
        got = j.cpu().numpy().astype(np.complex128)
        assert max(rel_l2(got[c], want[c]) for c in range(3)) < (1e-12 if precision == F.FP64 else 1e-5)
