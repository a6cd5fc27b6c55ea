"""Fused FP64 envelope stages at the edges of their tiles: grids of one column block, one cell more, of two blocks,
as narrow and as low as the stencil allows, taller than one segment; every stencil half width that takes the path,
one group of stages per step and several, odd and even step counts (the state ends in the caller's planes),
absorbing layers, batches of uneven grids and replayed graphs.  Against the CPU FP64 oracle to 1e-12 (as for the
stage-by-stage step), and bit for bit against the stage-by-stage step, whose operations they repeat in its order."""
import numpy as np
import pytest

from helpers import gpu_envelope, log, oracle_envelope, rel_l2

import paper_2605_12132_amd.inputs as I

pytestmark = pytest.mark.gpu

DZ = I.LAMBDA0 / 5


def depth(nd):
    return 4 if nd == 1 else 2


def columns(nd):
    """Output columns of a block: 4 wavefronts of 32 columns, less the halo of the later stages on both sides."""
    return 4 * 32 - 2 * (depth(nd) - 1) * nd


def check(monkeypatch, nz, nr, m, order, N, steps, flags=1, absorbers=()):
    rng = np.random.default_rng(nz[0] + 7 * nr[0] + order)
    w = I.Workload("env_fused", 1, nz, nr, m, [order] * len(nz), N, DZ, 0.2 * I.UM, 0.5 * DZ, steps)
    a, at, chi = [], [], []
    for x, y in zip(nz, nr):
        a.append(rng.uniform(-1, 1, (y, x)) + 1j * rng.uniform(-1, 1, (y, x)))
        at.append(rng.uniform(-1, 1, (y, x)) + 1j * rng.uniform(-1, 1, (y, x)))
        chi.append(1e-3 * (1 + 0.05 * rng.uniform(-1, 1, (y, x))))
    print(f"fused envelope {nz} x {nr} m={m} order {order} N {N} steps {steps}", flush=True)
    got = {}
    for fuse in ("1", "0"):
        monkeypatch.setenv("FDETD_ENV_FUSE", fuse)
        ga, gt, info = gpu_envelope(w, a, at, chi, steps, flags=flags, absorbers=absorbers)
        assert info["launches_per_step"] == (N // depth(order // 2) if fuse == "1" else N)
        got[fuse] = ga, gt
    oa, ot = oracle_envelope(w, a, at, chi, steps, absorbers=absorbers)
    for p in range(len(nz)):
        (fa, ft), (sa, st) = [(g[0][p], g[1][p]) for g in (got["1"], got["0"])]
        err = rel_l2(np.concatenate([fa.ravel(), ft.ravel()]), np.concatenate([oa[p].ravel(), ot[p].ravel()]))
        log(f"  problem {p}: rel L2 {err:.2e}")
        assert err < 1e-12
        assert np.array_equal(fa, sa) and np.array_equal(ft, st)
    return got["1"]


@pytest.mark.parametrize("order", [2, 4, 6, 8])
def test_tile_edges(monkeypatch, order):
    nd = order // 2
    oc = columns(nd)
    check(monkeypatch, [2 * nd + 1], [nd + 1], [1], order, 4, 1)          # smallest grid
    check(monkeypatch, [oc], [4 * nd + 3], [0], order, 4, 2)              # one block
    check(monkeypatch, [oc + 1], [70], [2], order, 4, 3)                  # one column more
    check(monkeypatch, [2 * oc - 1], [8 * nd + 1], [1], order, 8, 1)      # several groups per step
    check(monkeypatch, [97], [700], [0], order, 12, 2)                    # more rows than a block marches at most


@pytest.mark.parametrize("order", [2, 4, 8])
def test_many_steps_graph_and_layers(monkeypatch, order):
    """A captured call of several steps with absorbing layers equals the eager one bit for bit."""
    args = ([611], [149], [0], order, 4, 5)
    a = check(monkeypatch, *args, flags=1, absorbers=[(0, 16, 12, 0.2 / DZ, 2.0)])
    b = check(monkeypatch, *args, flags=3, absorbers=[(0, 16, 12, 0.2 / DZ, 2.0)])
    assert all(np.array_equal(x[0], y[0]) for x, y in zip(a, b))


def test_uneven_batch(monkeypatch):
    check(monkeypatch, [97, 611, 64], [23, 149, 300], [1, 0, 2], 8, 4, 4)
