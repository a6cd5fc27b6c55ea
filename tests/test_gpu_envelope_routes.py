"""Which FP64 envelope steps run in fused groups: not on grids that leave most of a block's columns empty, and a call's
last step of one group not where the copies that end it cost more than the group saves (small grids in a batch).
Whatever the route, by rule (no autotuning), timed or forced, the bits are those of the single stages."""
import numpy as np
import pytest

from helpers import dev, gpu_envelope

import paper_2605_12132_amd as F
import paper_2605_12132_amd.inputs as I

pytestmark = pytest.mark.gpu
DZ = I.LAMBDA0 / 5


def launches(nz, nr, order, steps):
    """Stage launches of a call of `steps` steps of N = 4, without autotuning."""
    import torch
    w = I.Workload("routes", 1, nz, nr, [0] * len(nz), [order] * len(nz), 4, DZ, 0.2 * I.UM, 0.5 * DZ, steps)
    planes = [torch.zeros((y, x), dtype=torch.complex128, device="cuda") for x, y in zip(nz, nr)]
    chi = [torch.zeros((y, x), dtype=torch.float64, device="cuda") for x, y in zip(nz, nr)]
    plan = F.Plan(w.problems(), precision=F.FP64, flags=F.PLAN_SKIP_STABILITY | F.PLAN_NO_AUTOTUNE | F.PLAN_PROFILE)
    plan.envelope_step(planes, [p.clone() for p in planes], chi, n_steps=steps)
    torch.cuda.synchronize()
    n = plan.query()["profiled_launches"]
    plan.close()
    return n


@pytest.mark.parametrize("nz,nr,order,one,two", [
    ([122] * 40, [128] * 40, 2, 4, 2),    # one group per step; its copies are 80 launches
    ([2440], [860], 2, 1, 2),             # ... or two large ones
    ([2440], [300], 8, 3, 4),             # two groups per step, the last one of the call by stages
    ([20], [40000], 8, 4, 8),             # 17 % of a block's columns in the grid
    ([130], [6000], 6, 4, 8),             # 53 %
])
def test_routes_without_timing(nz, nr, order, one, two):
    print(f"routes {nz[0]} x {nr[0]} ({len(nz)}) order {order}", flush=True)
    assert (launches(nz, nr, order, 1), launches(nz, nr, order, 2)) == (one, two)


@pytest.mark.parametrize("nz,nr,order", [([122] * 5, [900] * 5, 2), ([300], [2400], 4), ([130], [6000], 8)])
@pytest.mark.parametrize("steps", [1, 2, 3])
def test_every_route_gives_the_same_bits(monkeypatch, nz, nr, order, steps):
    rng = np.random.default_rng(steps)
    w = I.Workload("routes", 1, nz, nr, [0] * len(nz), [order] * len(nz), 4, DZ, 0.2 * I.UM, 0.5 * DZ, steps)
    a, at = ([rng.uniform(-1, 1, (y, x)) + 1j * rng.uniform(-1, 1, (y, x)) for x, y in zip(nz, nr)] for _ in range(2))
    chi = [1e-3 * rng.uniform(0, 1, (y, x)) for x, y in zip(nz, nr)]
    print(f"bits {nz[0]} x {nr[0]} ({len(nz)}) order {order} steps {steps}", flush=True)
    monkeypatch.setenv("FDETD_ENV_FUSE", "0")
    sa, st, _ = gpu_envelope(w, a, at, chi, steps, flags=1)
    monkeypatch.delenv("FDETD_ENV_FUSE")
    for flags in (1, 3, 1 | F.PLAN_NO_AUTOTUNE):
        ga, gt, _ = gpu_envelope(w, a, at, chi, steps, flags=flags)
        assert all(np.array_equal(x, y) for x, y in zip(ga + gt, sa + st))


@pytest.mark.parametrize("order,N", [(2, 4), (2, 8), (8, 4), (6, 6)])
def test_query_counts_what_runs(monkeypatch, order, N):
    """bytes_per_step and launches_per_step of grouped steps: 4.5 complex values per cell for the first group and 6.5
    for each further one, as the profiled launches of a call of two steps are counted."""
    import torch
    monkeypatch.setenv("FDETD_ENV_FUSE", "1")
    nz, nr, groups = 250, 60, N // (4 if order == 2 else 2)
    plan = F.Plan([F.Problem(nz, nr, 0, order, N, DZ, 0.2 * I.UM, 0.5 * DZ, k0=1.0, kind=F.ENVELOPE)], precision=F.FP64,
                  flags=F.PLAN_SKIP_STABILITY | F.PLAN_PROFILE)
    planes = [torch.zeros((nr, nz), dtype=torch.complex128, device="cuda") for _ in range(2)]
    plan.envelope_step(planes[:1], planes[1:], [torch.zeros((nr, nz), dtype=torch.float64, device="cuda")], n_steps=2)
    torch.cuda.synchronize()
    info = plan.query()
    plan.close()
    assert info["launches_per_step"] == groups
    assert info["bytes_per_step"] == nz * nr * 16 * (6.5 * groups - 2)
    assert info["profiled_launches"] == 2 * groups and info["profiled_bytes"] == 2 * info["bytes_per_step"]
