"""The radial stencils of the current correction at the edges of their tiles (64 columns x 16 rows): columns and
rows one short of, at and one past a tile, grids as low as the stencil allows, the narrowest and widest stencil,
odd and even modes; the corrected step against the oracle's (FP64, 1e-12, as test_gpu_correction.py)."""
import numpy as np
import pytest

from helpers import gpu_maxwell, log, rel_l2
from test_gpu_correction import grid, inputs, workload

import oracle
import paper_2605_12132_amd as F

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order,nz,nr,m", [(2, 3, 2, 0), (2, 63, 15, 1), (8, 64, 16, 0), (8, 65, 17, 1), (16, 129, 33, 2),
                                           (32, 33, 17, 0), (32, 128, 48, 1)])
def test_correction_tile_edges(order, nz, nr, m):
    w = workload([m], [order], nz=nz, nr=nr, steps=1)
    psi0, J4 = inputs(w, 1, np.random.default_rng(nz + nr))
    print(f"correction tiles order {order} {nz} x {nr} m={m}", flush=True)
    got, _ = gpu_maxwell(w, psi0, J4, 1, precision=F.FP64, flags=1 | F.PLAN_CURRENT_CORRECTION)
    err = rel_l2(got[0], oracle.step_corrected(grid(w, 0), psi0[0], J4[0], 1))
    log(f"correction tiles order {order} {nz} x {nr} m={m}: rel L2 {err:.2e}")
    assert err < 1e-12
