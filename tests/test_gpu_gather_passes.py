"""fdetd_gather where the planes of a block of samples fit its LDS tile all at once, several at a time, one at a
time, or not at all: footprints from a few cells to the whole grid, one to four modes, against the oracle
(FP64 1e-12; FP32C 2e-6: destaggered planes rounded to float, relative 2^-24 each, over sums of weights 1)."""
import numpy as np
import pytest

import oracle
from helpers import dev, log, rel_l2

import paper_2605_12132_amd as F
import paper_2605_12132_amd.inputs as I

pytestmark = pytest.mark.gpu
DZ = I.LAMBDA0 / 20


@pytest.mark.parametrize("precision", [F.FP64, F.FP32C])
@pytest.mark.parametrize("n,width,rmax,modes", [
    (700, 3, 8, [0, 1]),           # every plane at once
    (513, 8, 60, [0, 1, 2]),       # a few planes per pass, a block of one sample
    (600, 25, 100, [0, 1, 2, 3]),  # one plane per pass
    (600, 290, 100, [1]),          # no tile
])
def test_gather_passes(precision, n, width, rmax, modes):
    import torch
    nz, nr = 300, 104
    rng = np.random.default_rng(n + width)
    z, r = (150 + width * rng.uniform(-0.5, 0.5, n)) * DZ, rmax * 2 * DZ * rng.uniform(0, 1, n)
    r[:: max(n // 2, 1)] = [0.0, 0.999 * rmax * 2 * DZ, 0.5][: len(r[:: max(n // 2, 1)])]
    th = rng.uniform(-np.pi, np.pi, n)
    # (+ 0.0: no negative zeros, with which the oracle's atan2 takes the angle of a sample on the axis as pi)
    s = np.column_stack([z, r * np.cos(th), r * np.sin(th), np.ones(n)]) + 0.0
    grids = [oracle.Grid(nz=nz, nr=nr, m=m, fd_order=8, taylor_order=8, dz=DZ, dr=2 * DZ, dt=0.5 * DZ) for m in modes]
    cd = torch.complex128 if precision == F.FP64 else torch.complex64
    states = [(rng.uniform(-1, 1, (6, nr, nz)) + 1j * rng.uniform(-1, 1, (6, nr, nz)) * (m != 0)) for m in modes]
    psi = [dev(x, cd) for x in states]
    states = [x.cpu().numpy().astype(np.complex128) for x in psi]
    plan = F.Plan([F.Problem(nz, nr, m, 8, 8, DZ, 2 * DZ, 0.5 * DZ) for m in modes], precision=precision,
                  flags=F.PLAN_SKIP_STABILITY)
    got = plan.gather(psi, dev(s, torch.float64)).cpu().numpy()
    plan.close()
    err = rel_l2(got, oracle.gather(grids, states, s))
    log(f"gather passes n={n} width={width} rmax={rmax} modes={modes} precision={precision}: rel L2 {err:.1e}")
    assert err < (1e-12 if precision == F.FP64 else 2e-6)
