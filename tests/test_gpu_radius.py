"""The time-step check where the sigma product is not finite: the bound says so, and a server refuses."""
import math

import numpy as np
import pytest
from conftest import say

from paper_2601_16949_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "mixed"])
@pytest.mark.parametrize("spoil", ["nan", "overflow"])
@pytest.mark.parametrize("o,v,nq", [(8, 33, 7), (20, 64, 40)])
def test_bound_of_an_operator_that_is_not_finite(gpu_lib, o, v, nq, spoil, prec):
    prob = I.make_problem(I.Shape(o, v, nq, 0.05, storage="f32" if prec == "fp32" else "bf16"), 5)
    ctx = gpu_lib.Context(gpu_lib.DeviceProblem(prob, prec), max_rhs=1)
    rho, bound = ctx.spectral_radius(20)
    assert math.isfinite(rho) and rho <= bound < 100.0
    dev = gpu_lib.DeviceProblem(prob, prec)
    if spoil == "nan":
        dev.b_vv[nq // 2, 3, 3] = float("nan")
    else:  # finite factors whose product overflows FP32
        dev.b_ov *= 1e30
    rho, bound = gpu_lib.Context(dev, max_rhs=1).spectral_radius(20)
    say(f"[radius] {prec} o={o} v={v} nq={nq} {spoil}: rho {rho!r} bound {bound!r}")
    assert not math.isfinite(bound)
    assert not bound * 1e-6 <= 2.5


def test_server_refuses_a_request_whose_bound_is_not_a_number(gpu_lib, monkeypatch):
    from paper_2601_16949_amd import serve

    reqs = I.serving_requests(2, rate=200.0, seed=11, o_min=4, o_max=12)
    for r in reqs:
        r.n_steps = 20
    real = gpu_lib.Context.spectral_radius
    bad = []

    def radius(ctx, n_iter=30):
        if not bad:  # the first request that is admitted
            bad.append(ctx)
            return 0.0, float("nan")
        return real(ctx, n_iter)

    monkeypatch.setattr(gpu_lib.Context, "spectral_radius", radius)
    say("[radius] server with a request whose bound is not a number")
    srv = serve.Server(budget_bytes=1 << 30, chunk_steps=32, precision="mixed")
    srv.run(reqs, realtime=False)
    refused = [r for r in srv.results.values() if r.refused]
    assert len(refused) == 1 and refused[0].trace is None
    assert all(np.isfinite(r.trace).all() for r in srv.results.values() if not r.refused)
