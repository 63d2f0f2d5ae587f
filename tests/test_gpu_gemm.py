"""The GEMM exchange path at the edges of its tiles: slices' rows padded to multiples of 8 (any o from 65 on),
columns that end inside a tile and inside a K chunk, one and many row tiles, chunks of Q and Q splits of
uneven length, and workgroups that take more than one tile (with one, a few and many K chunks per tile).
Each against the FP64 oracle's sigma; a batch and one of its states alone give the same bits."""
import numpy as np
import pytest
from conftest import say

from oracle import rttda64 as O
from paper_2601_16949_amd import inputs as I

pytestmark = pytest.mark.gpu

# X and W carry 16 bits, so each product is off by at most 2^-16 of K = 1.5e-5 twice, and K is less than
# half of sigma here
TOL = 2e-5

SHAPES = [(65, 136, 5, 1), (66, 264, 3, 2), (72, 72, 7, 3), (77, 136, 4, 1), (96, 256, 9, 1), (96, 264, 4, 3),
          (104, 144, 3, 2), (121, 136, 3, 1), (127, 152, 3, 2), (129, 136, 4, 1), (250, 136, 2, 1), (256, 40, 3, 1),
          (128, 8, 5, 2), (65, 264, 300, 1), (130, 520, 130, 1), (128, 8, 600, 16), (72, 48, 1500, 6)]


@pytest.mark.parametrize("o,v,nq,nrhs", SHAPES)
def test_gemm_path_matches_oracle(gpu_lib, o, v, nq, nrhs):
    import torch

    prob = I.make_problem(I.Shape(o, v, nq, b_scale=0.05, cx=1.0, storage="bf16"), 41 + o)
    op = O.Operator.from_problem(prob)
    ctx = gpu_lib.Context(gpu_lib.DeviceProblem(prob, "mixed"), max_rhs=nrhs)
    tun = ctx.get_tuning()
    assert ctx.variant_name(tun["exchange_variant"]).startswith("bf16x2gemm")  # the default
    c0, c = I.random_state(o, v, nrhs, seed=o + v)
    dirs, field = np.tile([[1.0, 0.0, 0.0]], (nrhs, 1)), np.zeros(nrhs)
    checked = sorted({0, nrhs - 1})
    ref = {r: O.apply_H(op, O.dipole_blocks(op, dirs[r]), 0.0, c0[r], c[r])[1] for r in checked}
    c0d, cd = gpu_lib.to_planes(c0, c)
    n = ctx.lib.rttda_exchange_variants(ctx.desc.precision)
    kinds = [k for k in range(1, n + 1) if ctx.variant_name(k).startswith("bf16x2gemm")]
    tried = 0
    for k in kinds:
        for chunk, splits in ((-1, 0), (nq, 1), (max(1, nq // 3), min(nq, 4)), (1 if nq < 10 else nq, min(nq, 2))):
            try:
                ctx.set_tuning(exchange_variant=k, exchange_chunk=chunk,
                               exchange_splits=splits or tun["exchange_splits"])
            except gpu_lib.RttdaError:
                break  # (a tile of fewer than o rows)
            say(f"[gemm] {ctx.variant_name(k)} o={o} v={v} nq={nq} nrhs={nrhs} chunk {chunk} splits {splits}")
            _, sd = ctx.sigma(field, dirs, c0d, cd)
            torch.cuda.synchronize()
            s = gpu_lib.from_planes(torch.zeros_like(c0d), sd)[1]
            for r in checked:
                err = np.linalg.norm(s[r] - ref[r]) / np.linalg.norm(ref[r])
                assert err < TOL, (ctx.variant_name(k), chunk, splits, r, err)
            if nrhs > 1:
                _, s1 = ctx.sigma(field[-1:], dirs[-1:], c0d[-1:].contiguous(), cd[-1:].contiguous())
                torch.cuda.synchronize()
                assert torch.equal(s1[0], sd[-1]), (ctx.variant_name(k), chunk, splits)
            tried += 1
    assert tried >= 4
