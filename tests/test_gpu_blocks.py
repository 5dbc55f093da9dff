"""The block kernels at the dimensions where the pieces of H change: the edges
of the column blocks, of the register tiles and of the parts in LDS and in the
device-memory slot, on each block that takes the dimension; and starts that run
off to infinity.  Against the oracle, bit for bit (the rounding order does not
depend on where H lives)."""
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


def _same(a, b):
    return np.array_equal(a, b, equal_nan=a.dtype.kind == "f")


# (lanes forced, dimensions): three and four wavefronts, eight with H on chip, eight
# with a slot
CASES = ([(96, d) for d in (33, 48, 49, 64, 65, 80, 81, 95, 96)]
         + [(128, d) for d in (65, 66, 80, 81, 97, 127, 128)]
         + [(208, d) for d in (100, 129, 144, 145, 160, 176, 177, 192, 193, 207, 208)]
         + [(256, d) for d in (65, 128, 129, 160, 192, 193, 209, 224, 225, 240, 241, 255, 256)])


@pytest.mark.parametrize("lanes,d", CASES)
@pytest.mark.parametrize("objective", ["rosenbrock", "ackley"])
def test_block_edges(Z, ctx, oracle_mod, monkeypatch, lanes, d, objective):
    monkeypatch.setenv("ZEUS_TILE_LANES", str(lanes))
    p = W.problem(objective=objective, dim=d, n=6, lower=-2.0, upper=2.0, iter_pso=1, iter_bfgs=40,
                  seed=d)
    print(f"\n[blocks] {objective} d={d} lanes={lanes}", flush=True)
    g = Z.zeus_minimize(ctx, p)
    o = oracle_mod.bfgs(p, oracle_mod.pso(p)["x"])
    for k in KEYS:
        assert _same(g[k], o[k]), k


@pytest.mark.parametrize("lanes,d", [(96, 90), (128, 100), (208, 150), (208, 200), (256, 230)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_blocks_share_a_launch(Z, ctx, monkeypatch, lanes, d, precision):
    # two dimensions and an early stop in one launch: a block goes from one
    # to the other with the vectors and pieces of the last start in its LDS
    monkeypatch.setenv("ZEUS_TILE_LANES", str(lanes))
    ps = [W.problem(objective="rosenbrock", dim=dd, n=n, lower=-2.0, upper=2.0, iter_pso=1,
                    iter_bfgs=30, seed=3, request_id=i, precision=precision, required_converged=c)
          for i, (dd, n, c) in enumerate(((d, 300, 0), (d - 37, 300, 0), (d, 290, 5)))]
    print(f"\n[blocks] batch d={d} lanes={lanes} {precision}", flush=True)
    for p, g in zip(ps, Z.zeus_minimize_batch(ctx, ps)):
        monkeypatch.setenv("ZEUS_BFGS_CUS", "3")
        alone = Z.zeus_minimize(ctx, p)
        monkeypatch.delenv("ZEUS_BFGS_CUS")
        for k in KEYS:
            assert _same(g[k], alone[k]), (p["dim"], k)


@pytest.mark.parametrize("lanes,d", [(96, 70), (128, 90), (208, 170), (208, 205), (256, 211)])
def test_blocks_diverging_starts(Z, ctx, oracle_mod, monkeypatch, lanes, d):
    # one trial per search: alpha = 1/2 is taken unverified and the starts run
    # off until a value is not finite, through updates whose coefficients are
    # not (the last, unusable y is not compared as a skip)
    monkeypatch.setenv("ZEUS_TILE_LANES", str(lanes))
    p = W.problem(objective="rosenbrock", dim=d, n=5, lower=-2.0, upper=2.0, iter_pso=1,
                  iter_bfgs=60, iter_ls=1, seed=d)
    print(f"\n[blocks] diverging d={d} lanes={lanes}", flush=True)
    g = Z.zeus_minimize(ctx, p)
    o = oracle_mod.bfgs(p, oracle_mod.pso(p)["x"])
    for k in ("f", "x", "iters", "status", "ls_trials", "resets"):
        assert _same(g[k], o[k]), k


@pytest.mark.parametrize("d", [1, 4, 16, 33, 47, 48, 49, 50, 51, 52])
@pytest.mark.parametrize("objective,iter_ls", [("rosenbrock", 20), ("rosenbrock", 1),
                                               ("styblinski_tang", 20), ("quartic", 3)])
def test_cut_tile(Z, ctx, oracle_mod, monkeypatch, d, objective, iter_ls):
    # more starts than two wavefronts on each SIMD of one unit: the kernel with
    # the cut tile.  One trial per search lets the starts run off (as above).
    monkeypatch.setenv("ZEUS_TILE_LANES", "52")
    monkeypatch.setenv("ZEUS_BFGS_CUS", "1")
    p = W.problem(objective=objective, dim=max(d, 2) if objective == "rosenbrock" else d, n=14,
                  lower=-2.0, upper=2.0, iter_pso=1, iter_bfgs=60, iter_ls=iter_ls, seed=d)
    print(f"\n[blocks] cut {objective} d={d} ls={iter_ls}", flush=True)
    g = Z.zeus_minimize(ctx, p)
    o = oracle_mod.bfgs(p, oracle_mod.pso(p)["x"])
    for k in ("f", "x", "iters", "status", "ls_trials", "resets"):
        assert _same(g[k], o[k]), k
    ended = o["status"] != 3  # not at a value that is not finite
    assert _same(g["skips"][ended], o["skips"][ended])


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_cut_tile_or_not(Z, ctx, monkeypatch, precision):
    # one request through the cut tile and through the whole one, and two
    # dimensions and an early stop in one launch
    ps = [W.problem(objective="rosenbrock", dim=d, n=n, lower=-2.0, upper=2.0, iter_pso=1,
                    iter_bfgs=30, seed=3, request_id=i, precision=precision, required_converged=c)
          for i, (d, n, c) in enumerate(((50, 1500, 0), (35, 900, 0), (48, 290, 5)))]
    print(f"\n[blocks] cut or not {precision}", flush=True)
    cut = Z.zeus_minimize_batch(ctx, ps)
    monkeypatch.setenv("ZEUS_TILE_LANES", "64")
    for p, g in zip(ps, cut):
        whole = Z.zeus_minimize(ctx, p)
        for k in KEYS:
            assert _same(g[k], whole[k]), (p["dim"], k)
