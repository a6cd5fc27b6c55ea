"""FP32C plans of few cells share the rows of a near-axis segment out over several wavefronts: the results are the
bits of the unsplit segments (FDETD_SEG_AXIS = 16 takes them as they are), for bands of one short segment, of whole
segments and with a remainder, and on grids lower than the band."""
import numpy as np
import pytest

from helpers import gpu_envelope, gpu_maxwell

import paper_2605_12132_amd.inputs as I

pytestmark = pytest.mark.gpu


def noise(rng, *shape):
    return rng.uniform(-1, 1, shape) + 1j * rng.uniform(-1, 1, shape)


@pytest.mark.parametrize("nz,nr,order", [(67, 9, 2), (131, 23, 8), (203, 40, 12), (150, 17, 32), (97, 70, 20), (900, 180, 16)])
def test_split_segments_give_the_same_bits(monkeypatch, nz, nr, order):
    w = I.Workload("split", 0, [nz, nz], [nr, nr], [0, 1], [order, order], 4, 0.5, 0.7, 0.05, 2)
    we = I.Workload("split_env", 1, [nz, nz], [nr, nr], [0, 1], [order, order], 4, 0.5, 0.7, 0.05, 2)
    rng = np.random.default_rng(nz)
    psi = [noise(rng, 6, nr, nz) for _ in range(2)]
    J = [noise(rng, 2, 3, nr, nz) for _ in range(2)]
    a, at = ([noise(rng, nr, nz) for _ in range(2)] for _ in range(2))
    chi = [rng.uniform(0, 0.01, (nr, nz)) for _ in range(2)]
    print(f"near-axis split {nz} x {nr} order {order}", flush=True)
    out = []
    for forced in (None, "16"):
        if forced:
            monkeypatch.setenv("FDETD_SEG_AXIS", forced)
        m, info = gpu_maxwell(w, psi, J, 2, precision=1, flags=1)
        ga, gt, _ = gpu_envelope(we, a, at, chi, 2, precision=1, flags=1)
        assert info["seg_rows_axis"] == min(16, order, nr)
        out.append(list(m) + ga + gt)
    assert all(np.array_equal(x, y) for x, y in zip(*out))
