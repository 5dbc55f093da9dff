"""Gradient tolerances whose square underflows: a start whose gradient is exactly
zero has converged whatever the tolerance is (the norm test is decided as
sqrt(g'g) < Theta, not on the squares).  Sphere starts get there in one step.
Every kernel family, against the oracle, bit for bit."""
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


# (lanes forced or 0, dimension, L-BFGS pairs): lane groups, the cut tile, the
# blocks of three, four and eight wavefronts, and L-BFGS
CASES = [(0, 1, 0), (0, 7, 0), (0, 16, 0), (0, 30, 0), (52, 50, 0), (0, 64, 0), (96, 70, 0),
         (128, 100, 0), (208, 150, 0), (256, 230, 0), (0, 3, 5), (0, 8, 5), (0, 50, 5), (0, 200, 5)]


@pytest.mark.parametrize("lanes,d,m", CASES)
@pytest.mark.parametrize("tol", [1e-200, 5e-324])
def test_zero_gradient_converges(Z, ctx, oracle_mod, monkeypatch, lanes, d, m, tol):
    if lanes:
        monkeypatch.setenv("ZEUS_TILE_LANES", str(lanes))
    if lanes == 52:  # more starts than the whole tile would take on one unit
        monkeypatch.setenv("ZEUS_BFGS_CUS", "1")
    p = W.problem(objective="sphere", dim=d, n=14, lower=-2.0, upper=2.0, iter_pso=1, iter_bfgs=6,
                  grad_tol=tol, seed=d, lbfgs_m=m)
    print(f"\n[tiny] d={d} lanes={lanes} m={m} tol={tol}", flush=True)
    g = Z.zeus_minimize(ctx, p)
    o = oracle_mod.bfgs(p, oracle_mod.pso(p)["x"])
    assert (o["status"] == 1).any()  # some start gets to a gradient of zero
    for k in KEYS:
        assert np.array_equal(g[k], o[k], equal_nan=g[k].dtype.kind == "f"), k
