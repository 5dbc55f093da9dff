"""Results of a blocking call on their way through the context's pinned memory:
requests of up to 1 MB of results are staged there, up to 16 MB in one call, and
the others copied directly.  One call with requests on both sides of both
limits, with traces and the swarm's state, against the same solves into device
buffers, which stage nothing; and again, in the memory of the call before."""
import numpy as np
import pytest

from paper_2603_28770_amd import workloads as W

pytestmark = pytest.mark.gpu

TRACE = 6


@pytest.fixture(scope="module")
def Z():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_28770_amd import zeus
    return zeus


def test_both_limits_in_one_call(Z):
    import torch
    ctx = Z.zeus_context_create(0)
    # 17 requests just below 1 MB, of which the last do not fit 16 MB, one of
    # 2.5 MB between them, and small ones of other launch groups
    sizes = [(10, 1200)] * 9 + [(10, 3000), (70, 40)] + [(10, 1200)] * 8 + [(3, 64), (10, 1)]
    ps = [W.problem(objective=("rastrigin", "rosenbrock")[i % 2], dim=d, n=n, lower=-5.0, upper=5.0,
                    iter_pso=2, iter_bfgs=12, seed=9, request_id=i) for i, (d, n) in enumerate(sizes)]
    per_start = 8 * (4 * 10 + 2 + TRACE * 10) + 5 * 4
    assert 0.9 * 2**20 < 1200 * per_start < 2**20 < 3000 * per_start and 17 * 1200 * per_start > 2**24
    want = []
    for p in ps:
        s = Z.DeviceSolve(p, trace_len=TRACE, pso_state=True)
        s.enqueue(ctx)
        torch.cuda.synchronize()
        want.append(s.host())
    for rep, sub in enumerate((slice(None), slice(8, 12), slice(None))):
        print(f"\n[staging] call {rep}", flush=True)
        got = Z.zeus_minimize_batch(ctx, ps[sub], trace_len=TRACE, pso_state=True)
        for p, g, w in zip(ps[sub], got, want[sub]):
            for k, v in w.items():
                if k == "summary":
                    assert g[k]["best_f"] == v["best_f"] and g[k]["n_converged"] == v["n_converged"]
                else:
                    assert np.array_equal(g[k], v, equal_nan=v.dtype.kind == "f"), (p["request_id"], k)
    Z.zeus_context_destroy(ctx)
