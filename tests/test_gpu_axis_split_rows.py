"""That the near-axis rows of small FP32C plans are shared out, and over how many wavefronts: the rows a wavefront
marches, as the plan reports them, by the cells of the plan; in the range of two wavefronts the results are the bits of
unshared segments (the range of four: test_gpu_axis_split.py)."""
import numpy as np
import pytest

from helpers import gpu_envelope, gpu_maxwell

import paper_2605_12132_amd as F
import paper_2605_12132_amd.inputs as I

pytestmark = pytest.mark.gpu


def rows(kind, nz, nr, order, n):
    w = I.Workload("rows", kind, [nz] * n, [nr] * n, [0] * n, [order] * n, 4, 0.5, 0.7, 0.05, 1)
    plan = F.Plan(w.problems(), precision=F.FP32C, flags=F.PLAN_SKIP_STABILITY | F.PLAN_NO_AUTOTUNE)
    info = plan.query()
    plan.close()
    assert info["seg_rows_axis"] == min(16, order, nr)
    return info["tile_rows_axis"]


@pytest.mark.parametrize("kind,nz,nr,n,part", [(0, 600, 150, 1, 4), (0, 1024, 256, 1, 2), (0, 1000, 262, 2, 2),
                                              (0, 1024, 256, 2, 1), (1, 1000, 150, 2, 4), (1, 2048, 512, 1, 2), (1, 1280, 1023, 1, 2), (1, 1280, 1024, 1, 2),
                                              (1, 2048, 512, 2, 1)])
def test_rows_of_a_wavefront(kind, nz, nr, n, part):
    for order in (2, 8, 16, 24, 32):
        # an envelope's segments of wide stencils are shared by two up to 5/4 of 2^20 cells only
        whole = kind == 1 and order > 24 and nz * nr * n >= 5 << 18
        assert rows(kind, nz, nr, order, n) == min(16 if whole else 16 // part, order)


def test_fp64_plans_have_no_near_axis_tiles():
    plan = F.Plan([F.Problem(64, 32, 0, 8, 4, 0.5, 0.7, 0.05)], precision=F.FP64, flags=F.PLAN_SKIP_STABILITY)
    assert plan.query()["tile_rows_axis"] == 0
    plan.close()


@pytest.mark.parametrize("kind,nz,nr,order", [(0, 1300, 180, 16), (0, 1300, 180, 12), (1, 2048, 300, 16)])
def test_two_wavefronts_give_the_same_bits(monkeypatch, kind, nz, nr, order):
    w = I.Workload("two", kind, [nz, nz], [nr, nr], [0, 1], [order, order], 4, 0.5, 0.7, 0.05, 1)
    rng = np.random.default_rng(nz + order)
    print(f"near-axis split by two {nz} x {nr} order {order}", flush=True)
    def noise(*shape):
        return rng.uniform(-1, 1, shape) + 1j * rng.uniform(-1, 1, shape)
    if kind == 0:
        psi, J = [noise(6, nr, nz) for _ in range(2)], [noise(1, 3, nr, nz) for _ in range(2)]
    else:
        a, at = ([noise(nr, nz) for _ in range(2)] for _ in range(2))
        chi = [rng.uniform(0, 0.01, (nr, nz)) for _ in range(2)]
    out, tiles = [], []
    for forced in (None, "16"):
        if forced:
            monkeypatch.setenv("FDETD_SEG_AXIS", forced)
        if kind == 0:
            m, info = gpu_maxwell(w, psi, J, 1, precision=1, flags=1)
            out.append(list(m))
        else:
            ga, gt, info = gpu_envelope(w, a, at, chi, 1, precision=1, flags=1)
            out.append(ga + gt)
        tiles.append(info["tile_rows_axis"])
    assert tiles == [8, min(16, order)]
    assert all(np.array_equal(x, y) for x, y in zip(*out))
