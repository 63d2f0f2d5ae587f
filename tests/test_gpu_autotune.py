"""The autotuner's sweep: each exchange tile is tried around its own split count, and the sweep leaves the
context as it was."""
import pytest
from conftest import say

from paper_2601_16949_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,o,v,nq,R", [("fp32", 40, 300, 200, 64), ("mixed", 40, 300, 200, 64), ("mixed", 72, 136, 60, 4)])
def test_each_tile_is_tried_around_its_own_split_count(gpu_lib, prec, o, v, nq, R):
    import torch

    from paper_2601_16949_amd import autotune

    dev = gpu_lib.DeviceProblem(I.make_problem(I.Shape(o, v, nq, 0.03, storage="f32" if prec == "fp32" else "bf16"), 3), prec)
    ctx = gpu_lib.Context(dev, max_rhs=R)
    base = ctx.get_tuning()
    c0, c = gpu_lib.to_planes(*I.random_state(o, v, R, seed=3))
    dirs, field = [(0.0, 0.0, 1.0)] * R, [0.0] * R
    _, before = ctx.sigma(field, dirs, c0, c)
    out = autotune.candidates(ctx)
    assert ctx.get_tuning() == base
    _, after = ctx.sigma(field, dirs, c0, c)
    torch.cuda.synchronize()
    assert torch.equal(before, after)
    staged = {}
    for k in {k for k, _, _ in out}:
        fresh = gpu_lib.Context(dev, max_rhs=R)
        fresh.set_tuning(exchange_variant=k)
        own = fresh.get_tuning()["exchange_splits"]
        assert own in {s for j, s, _ in out if j == k}, (fresh.variant_name(k), own)
        if "dl" in fresh.variant_name(k) or fresh.variant_name(k).startswith(("f32_", "bf16x2_")):
            staged[fresh.variant_name(k)] = own
    say(f"[autotune] {prec} o={o} v={v} nq={nq} {R} RHS: {ctx.variant_name(base['exchange_variant'])} "
        f"{base['exchange_splits']}, LDS-staged {staged}")
    # a count the caller has chosen stays with the context
    ctx.set_tuning(exchange_splits=base["exchange_splits"] + 1)
    ctx.set_tuning(exchange_variant=base["exchange_variant"])
    assert ctx.get_tuning()["exchange_splits"] == base["exchange_splits"] + 1
    # the LDS-staged tiles' workgroups take a part of the columns or rows each and want counts of their own
    assert any(s != base["exchange_splits"] for s in staged.values())
