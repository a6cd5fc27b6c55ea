"""fdetd_gather chooses per block between planes copied into LDS and direct reads, by the footprint, the samples of the
block and the number of blocks: whatever it takes, the fields are the same bits.  Footprints around the limits (6 values
of a plane per sample of a part block, 1400, 2048 and 4096 values, 256 blocks), the samples of one large call against
the same samples in calls of 1, 40, 300 and 512; a part of them against the oracle (1e-12)."""
import numpy as np
import pytest

import oracle
from helpers import dev, rel_l2

import paper_2605_12132_amd as F
import paper_2605_12132_amd.inputs as I

pytestmark = pytest.mark.gpu
DZ = I.LAMBDA0 / 20


@pytest.mark.parametrize("precision", [F.FP64, F.FP32C])
@pytest.mark.parametrize("width,height,modes", [(2, 2, [0, 1, 2]), (33, 32, [0]), (38, 36, [2, 0, 1]), (42, 40, [0, 1]), (60, 62, [1, 1, 3]),
                                                (80, 60, [0])])
def test_same_bits_in_any_call(precision, width, height, modes):
    import torch
    nz, nr, n = 100, 70, 256 * 512 + 77
    print(f"gather choice {width} x {height} modes {modes} precision {precision}", flush=True)
    rng = np.random.default_rng(width)
    z, r, th = (6 + width * rng.uniform(0, 1, n)) * DZ, height * 2 * DZ * rng.uniform(0, 1, n), rng.uniform(-np.pi, np.pi, n)
    s = np.column_stack([z, r * np.cos(th), r * np.sin(th), np.ones(n)])
    cd = torch.complex128 if precision == F.FP64 else torch.complex64
    psi = [dev(rng.uniform(-1, 1, (6, nr, nz)) + 1j * rng.uniform(-1, 1, (6, nr, nz)) * (m != 0), cd) for m in modes]
    plan = F.Plan([F.Problem(nz, nr, m, 8, 8, DZ, 2 * DZ, 0.5 * DZ) for m in modes], precision=precision,
                  flags=F.PLAN_SKIP_STABILITY | F.PLAN_NO_AUTOTUNE)
    get = lambda x: plan.gather(psi, dev(x, torch.float64)).cpu().numpy()  # noqa: E731
    whole = get(s)
    for start, size in ((0, 1), (100, 40), (1000, 300), (5000, 512), (7000, 512 + 40)):
        assert np.array_equal(get(s[start:start + size]), whole[start:start + size])
    plan.close()
    grids = [oracle.Grid(nz=nz, nr=nr, m=m, fd_order=8, taylor_order=8, dz=DZ, dr=2 * DZ, dt=0.5 * DZ) for m in modes]
    want = oracle.gather(grids, [x.cpu().numpy().astype(np.complex128) for x in psi], s[:400])
    assert rel_l2(whole[:400], want) < (1e-12 if precision == F.FP64 else 2e-6)
