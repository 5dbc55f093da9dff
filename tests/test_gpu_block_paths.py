"""Starts that run off to infinity after updates, through every kernel whose H
has padding to restore, and the tilings of 52 and 96 lanes against the others."""
import numpy as np
import pytest

from paper_2603_28770_amd import workloads as W

pytestmark = pytest.mark.gpu

KEYS = ("f", "x", "iters", "status", "ls_trials", "skips", "resets")
NONFINITE = 3


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


@pytest.mark.parametrize("lanes,d", [(16, 13), (52, 50), (64, 60), (96, 70), (128, 100), (208, 150),
                                     (208, 200), (256, 230)])
@pytest.mark.parametrize("objective", ["rosenbrock", "styblinski_tang"])
def test_updates_before_infinity(Z, ctx, oracle_mod, monkeypatch, objective, lanes, d):
    # one trial per search: half the step is taken whatever it gives
    monkeypatch.setenv("ZEUS_TILE_LANES", str(lanes))
    if lanes == 52:
        monkeypatch.setenv("ZEUS_BFGS_CUS", "1")  # more starts than the whole tile takes on a unit
    p = W.problem(objective=objective, dim=d, n=14, lower=-5.0, upper=5.0, iter_pso=1, iter_bfgs=60,
                  iter_ls=1, seed=d)
    print(f"\n[paths] {objective} d={d} lanes={lanes}", flush=True)
    g = Z.zeus_minimize(ctx, p)
    o = oracle_mod.bfgs(p, oracle_mod.pso(p)["x"])
    assert (o["status"] == NONFINITE).all()
    assert (o["iters"] - o["skips"] >= 2).all()  # an update at least before the last step
    assert (o["resets"] > 0).any()               # from an H or a gradient that is no use any more
    for k in ("f", "x", "iters", "status", "ls_trials", "resets"):
        assert np.array_equal(g[k], o[k], equal_nan=o[k].dtype.kind == "f"), k
    # at the last point a whole pass of the oracle's gradient meets 0 * inf in the
    # terms that a kernel's lane does not evaluate, so only that y's may differ
    assert (np.abs(g["skips"] - o["skips"]) <= 1).all()


@pytest.mark.parametrize("objective", ["rosenbrock", "styblinski_tang", "ackley"])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("d,tilings", [(40, (64, 52, 96, 128)), (66, (96, 128, 208, 256)),
                                       (96, (96, 128, 208, 256))])
def test_tilings_of_52_and_96_agree(Z, ctx, monkeypatch, objective, precision, d, tilings):
    # (one unit: launches large enough for the cut tile and for three wavefronts
    # whatever the objective; no cut tile for Ackley, which then takes its own)
    monkeypatch.setenv("ZEUS_BFGS_CUS", "1")
    p = W.problem(objective=objective, dim=d, n=20, lower=-5.0, upper=5.0, iter_pso=2, iter_bfgs=80,
                  seed=d, precision=precision, grad_tol=1e-4)
    ref = None
    for lanes in tilings:
        print(f"\n[paths] {objective} {precision} d={d} lanes={lanes}", flush=True)
        monkeypatch.setenv("ZEUS_TILE_LANES", str(lanes))
        out = Z.zeus_minimize(ctx, p)
        ref = ref or out
        for k in KEYS:
            assert np.array_equal(out[k], ref[k], equal_nan=out[k].dtype.kind == "f"), (lanes, k)
