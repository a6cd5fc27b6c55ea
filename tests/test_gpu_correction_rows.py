"""The radial stencils of the current correction in blocks of 4 rows (grids of less than 2^19 cells) and of 8: rows one
short of, at and one past a block, and each side of the line between the two; the corrected step against the oracle's
(FP64, 1e-12, as test_gpu_correction.py)."""
import numpy as np
import pytest

from helpers import gpu_maxwell, log, rel_l2
from test_gpu_correction import grid, inputs, workload

import oracle
import paper_2605_12132_amd as F

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order,nz,nr,m", [(8, 65, 11, 1), (8, 65, 12, 0), (8, 65, 13, 2), (2, 4096, 127, 1), (2, 4096, 128, 1), (4, 4100, 129, 0),
                                           (2, 4000, 135, 1), (6, 4000, 136, 2)])
def test_correction_rows_per_block(order, nz, nr, m):
    w = workload([m], [order], nz=nz, nr=nr, steps=1)
    psi0, J4 = inputs(w, 1, np.random.default_rng(nz + nr))
    print(f"correction rows order {order} {nz} x {nr} m={m}", flush=True)
    got, _ = gpu_maxwell(w, psi0, J4, 1, precision=F.FP64, flags=1 | F.PLAN_CURRENT_CORRECTION)
    err = rel_l2(got[0], oracle.step_corrected(grid(w, 0), psi0[0], J4[0], 1))
    log(f"correction rows order {order} {nz} x {nr} m={m}: rel L2 {err:.2e}")
    assert err < 1e-12
