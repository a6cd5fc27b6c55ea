"""fdetd_deposit_current against the oracle in FP64 blocks of every size: 256, 512 and 1024 samples (by the number of
samples), with runs of one cell that go on from one chunk of a wavefront to the next; and a sample whose half-step
positions lie more than 2^15 rows from it, which no run can hold.  1e-12 relative L2 per plane, as for the other FP64
depositions: the sums differ in their order only."""
import numpy as np
import pytest

import oracle
from helpers import dev, log, rel_l2

import paper_2605_12132_amd as F
import paper_2605_12132_amd.inputs as I

pytestmark = pytest.mark.gpu
DZ = I.LAMBDA0 / 20
DT = 0.5 * DZ


def check(s, nz, nr, modes, rxy, what):
    import torch
    print(what, flush=True)
    plan = F.Plan([F.Problem(nz, nr, m, 8, 8, DZ, 2 * DZ, DT) for m in modes], precision=F.FP64,
                  flags=F.PLAN_SKIP_STABILITY | F.PLAN_NO_AUTOTUNE | (F.PLAN_CURRENT_CORRECTION if rxy else 0))
    J = [torch.zeros((4 if rxy else 3, nr, nz), dtype=torch.complex128, device="cuda") for _ in modes]
    plan.deposit_current(dev(s, torch.float64), J, eps=0.5)
    torch.cuda.synchronize()
    plan.close()
    for j, m in zip(J, modes):
        wj, wr = oracle.deposit_current(oracle.Grid(nz=nz, nr=nr, m=m, fd_order=8, taylor_order=8, dz=DZ, dr=2 * DZ, dt=DT), s)
        got = j.cpu().numpy()
        errs = [rel_l2(got[c], wj[c]) for c in range(3)] + ([rel_l2(got[3], wr)] if rxy else [])
        log(f"  m={m}: {[f'{e:.1e}' for e in errs]}")
        assert max(errs) < 1e-12


@pytest.mark.parametrize("n,modes,rxy", [(131072 + 77, [0, 1], True), (262144 + 130, [1], False), (524288 + 1001, [1], False),
                                         (524288 + 5, [0], True)])
def test_fp64_blocks(n, modes, rxy):
    rng = np.random.default_rng(n)
    z = (20 + np.arange(n) * 20 // n + rng.uniform(0.2, 0.45, n)) * DZ  # 20 cells one after the other
    r, th = (rng.integers(0, 2, n) * 7 + rng.uniform(0.6, 0.95, n)) * 2 * DZ, rng.uniform(-np.pi, np.pi, n)
    s = np.column_stack([z, r * np.cos(th), r * np.sin(th), rng.uniform(-1, 1, n), rng.uniform(-0.3, 0.3, (n, 3)), np.zeros(n)])
    check(s, 60, 20, modes, rxy, f"blocks n={n} modes={modes}")


@pytest.mark.parametrize("rxy", [False, True])
def test_half_steps_beyond_16_bit_rows(rxy):
    rng = np.random.default_rng(1)
    n, nr = 200, 34000
    s = np.column_stack([rng.uniform(8, 30, n) * DZ, rng.uniform(1, 90, n) * 2 * DZ, rng.uniform(-9, 9, n) * DZ,
                         rng.uniform(0.5, 1, n), rng.uniform(-0.3, 0.3, (n, 3)), np.zeros(n)])
    s[::25, 4] = 33400 * 2 * DZ / (0.5 * DT)
    check(s, 40, nr, [0, 1], rxy, "half steps beyond 16-bit rows")
