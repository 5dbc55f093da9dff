"""The two L-BFGS kernels that a launch can take, with a coordinate per lane and
with more, at the edges of the coordinate slots: the same bits as the oracle
from both (sums do not depend on which lane holds a coordinate).  One unit takes
the second kernel for as many starts as these, all of them the first."""
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


@pytest.mark.parametrize("d,m", [(5, 3), (8, 8), (9, 1), (16, 5), (17, 8), (32, 4), (33, 8), (64, 5),
                                 (65, 3), (128, 8)])
@pytest.mark.parametrize("objective", ["rosenbrock", "ackley", "styblinski_tang"])
def test_both_kernels(Z, ctx, oracle_mod, monkeypatch, objective, d, m):
    lo, hi = W.BOXES[objective]
    p = W.problem(objective=objective, dim=d, n=150, lower=lo, upper=hi, iter_pso=1, iter_bfgs=40,
                  seed=d, lbfgs_m=m)
    print(f"\n[lbfgs] {objective} d={d} m={m}", flush=True)
    spread = Z.zeus_minimize(ctx, p)
    mixed = Z.zeus_minimize(ctx, dict(p, precision="mixed"))
    monkeypatch.setenv("ZEUS_BFGS_CUS", "1")
    dense = Z.zeus_minimize(ctx, p)
    mixed_dense = Z.zeus_minimize(ctx, dict(p, precision="mixed"))
    o = oracle_mod.bfgs(p, oracle_mod.pso(p)["x"])
    for k in KEYS:
        eq = o[k].dtype.kind == "f"
        assert np.array_equal(spread[k], o[k], equal_nan=eq), k
        assert np.array_equal(dense[k], o[k], equal_nan=eq), k
        assert np.array_equal(mixed[k], mixed_dense[k], equal_nan=eq), k
