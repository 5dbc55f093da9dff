"""Objectives with transcendental terms take the block of three wavefronts only
in large launches, the one of four in small ones: at the edges of the column
blocks, the same bits from both as the oracle.  (One unit makes 18 starts a
large launch.)  And without forcing anything a small launch takes as long as
with four wavefronts forced."""
import time

import numpy as np
import pytest

from paper_2603_28770_amd import workloads as W

pytestmark = pytest.mark.gpu

KEYS = ("f", "x", "iters", "status", "ls_trials", "skips", "resets")


@pytest.fixture(scope="module")
def Z():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_28770_amd import zeus
    return zeus


@pytest.fixture(scope="module")
def ctx(Z):
    c = Z.zeus_context_create(0)
    yield c
    Z.zeus_context_destroy(c)


@pytest.mark.parametrize("d", [65, 80, 81, 95, 96])
@pytest.mark.parametrize("objective", ["rastrigin", "ackley"])
def test_both_blocks(Z, ctx, oracle_mod, monkeypatch, objective, d):
    lo, hi = W.BOXES[objective]
    p = W.problem(objective=objective, dim=d, n=18, lower=lo, upper=hi, iter_pso=1, iter_bfgs=40, seed=d)
    print(f"\n[tile] {objective} d={d}", flush=True)
    four = Z.zeus_minimize(ctx, p)
    mixed_four = Z.zeus_minimize(ctx, dict(p, precision="mixed"))
    monkeypatch.setenv("ZEUS_BFGS_CUS", "1")
    three = Z.zeus_minimize(ctx, p)
    mixed_three = Z.zeus_minimize(ctx, dict(p, precision="mixed"))
    o = oracle_mod.bfgs(p, oracle_mod.pso(p)["x"])
    for k in KEYS:
        eq = o[k].dtype.kind == "f"
        assert np.array_equal(four[k], o[k], equal_nan=eq), k
        assert np.array_equal(three[k], o[k], equal_nan=eq), k
        assert np.array_equal(mixed_four[k], mixed_three[k], equal_nan=eq), k


def test_small_launch_time(Z, ctx, monkeypatch):
    # 1.18 with three wavefronts, 1.00 with four
    import torch
    p = W.problem(objective="ackley", dim=80, n=256, lower=-5.0, upper=5.0, iter_pso=1,
                  iter_bfgs=1000, seed=3, grad_tol=1e-13)
    run = Z.DeviceSolve(p)
    best = {0: float("inf"), 128: float("inf")}
    for rep in range(8):
        for lanes in best:
            if lanes:
                monkeypatch.setenv("ZEUS_TILE_LANES", str(lanes))
            else:
                monkeypatch.delenv("ZEUS_TILE_LANES", raising=False)
            torch.cuda.synchronize()
            t = time.perf_counter()
            run.enqueue(ctx)
            torch.cuda.synchronize()
            if rep:
                best[lanes] = min(best[lanes], time.perf_counter() - t)
    print(f"\n[tile] {1e3 * best[0]:.3f} ms, four wavefronts {1e3 * best[128]:.3f}", flush=True)
    assert best[0] < 1.09 * best[128]
