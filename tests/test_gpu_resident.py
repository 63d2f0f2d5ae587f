"""The X-resident exchange tiles (X of a slice or two held in LDS, B_vv rows read straight into
registers) at the sizes where their layouts can go wrong: v around the 16-byte groups, the single and
double K steps, the 16-column blocks and the column remainders; o around the 16-row blocks and the
repeated last group of rows; odd slice counts, Q ranges shorter than the wave split, and the longest v
that fits.  Each against the FP64 oracle's sigma."""
import numpy as np
import pytest

from conftest import say
from oracle import rttda64 as O
from paper_2601_16949_amd import inputs as I

pytestmark = pytest.mark.gpu

# FP32: X and both products are rounded to 2^-24 relative with sums of at most ~1e3 terms in chains of
# a few hundred; 2e-6 is about 30 of those roundings in a row.  Split BF16: X and W carry 16 bits, so
# each product is off by at most 2^-16 of K = 1.5e-5 twice, and K is less than half of sigma here.
TOL = {"fp32": 2e-6, "mixed": 2e-5}

SHAPES = [(8, 8, 3, 1), (9, 9, 2, 2), (15, 15, 5, 1), (16, 16, 4, 3), (17, 17, 3, 2), (23, 31, 5, 1), (31, 32, 2, 3),
          (32, 33, 9, 1), (33, 47, 3, 2), (40, 63, 4, 1), (41, 64, 3, 3), (47, 65, 2, 1), (48, 96, 5, 2),
          (49, 127, 3, 1), (57, 129, 2, 2), (63, 255, 3, 1), (64, 257, 2, 1), (60, 400, 11, 2), (61, 431, 2, 1),
          (64, 512, 1, 1), (50, 639, 2, 1), (64, 640, 3, 1), (48, 832, 2, 1), (20, 1100, 2, 2)]


def _resident(name):
    return name.startswith("f32r_") or name.startswith("bf16x2r_")


@pytest.mark.parametrize("prec", ["fp32", "mixed"])
@pytest.mark.parametrize("o,v,nq,nrhs", SHAPES)
def test_resident_tiles_match_oracle(gpu_lib, o, v, nq, nrhs, prec):
    import torch
    from paper_2601_16949_amd import rttda

    shape = I.Shape(o, v, nq, b_scale=0.05, cx=1.0, storage="f32" if prec == "fp32" else "bf16")
    prob = I.make_problem(shape, 99 + o)
    op = O.Operator.from_problem(prob)
    ctx = rttda.Context(rttda.DeviceProblem(prob, prec), max_rhs=nrhs)
    c0, c = I.random_state(o, v, nrhs, seed=o + v)
    dirs, field = np.tile([[0.0, 0.0, 1.0]], (nrhs, 1)), np.zeros(nrhs)
    ref = [O.apply_H(op, O.dipole_blocks(op, dirs[r]), 0.0, c0[r], c[r])[1] for r in range(nrhs)]
    c0d, cd = gpu_lib.to_planes(c0, c)
    names = [ctx.variant_name(k) for k in range(1, ctx.lib.rttda_exchange_variants(ctx.desc.precision) + 1)]
    tried = 0
    for k, name in enumerate(names, 1):
        if not _resident(name):
            continue
        for splits in sorted({1, min(2, nq), nq}):
            try:
                ctx.set_tuning(exchange_variant=k, exchange_splits=splits)
            except gpu_lib.RttdaError:
                continue
            say(f"[resident] {name} o={o} v={v} nq={nq} nrhs={nrhs} splits {splits}")
            _, sd = ctx.sigma(field, dirs, c0d, cd)
            torch.cuda.synchronize()
            s = gpu_lib.from_planes(torch.zeros_like(c0d), sd)[1]
            for r in range(nrhs):
                err = np.linalg.norm(s[r] - ref[r]) / np.linalg.norm(ref[r])
                assert err < TOL[prec], (name, splits, r, err)
            # one state of the batch alone: the same bits
            if nrhs > 1:
                _, s1 = ctx.sigma(field[-1:], dirs[-1:], c0d[-1:].contiguous(), cd[-1:].contiguous())
                torch.cuda.synchronize()
                assert torch.equal(s1[0], sd[-1]), (name, splits)
            tried += 1
    assert tried > 0


@pytest.mark.parametrize("prec", ["fp32", "mixed"])
def test_resident_tile_is_the_default_for_every_alignment(gpu_lib, prec):
    """Contexts pick a resident tile wherever X fits the LDS, odd and even sizes alike; the split
    operator's launches (one plane per state) take their own split count."""
    import torch
    from paper_2601_16949_amd import rttda

    for o, v in ((20, 61), (33, 100), (60, 401)):
        prob = I.make_problem(I.Shape(o, v, 40, b_scale=0.05, storage="f32" if prec == "fp32" else "bf16"), 7)
        ctx = rttda.Context(rttda.DeviceProblem(prob, prec), max_rhs=2)
        assert _resident(ctx.variant_name(ctx.get_tuning()["exchange_variant"]))
        op = O.Operator.from_problem(prob)
        pulses = I.kick_pulses(axes=I.AXES[:2], kappa=1e-2)
        c0d, cd = gpu_lib.ground_state(2, o, v)
        tr = ctx.propagate(pulses, 0.05, 3, c0d, cd, integrator="sso").cpu().numpy()
        torch.cuda.synchronize()
        for r, p in enumerate(pulses):
            ref = O.propagate_sso(op, p, 0.05, 3)[0]
            assert np.max(np.abs(tr[:, r] - ref)) / np.max(np.abs(ref)) < TOL[prec]


@pytest.mark.parametrize("o,v,nq", [(17, 33, 5), (23, 40, 9), (24, 64, 6), (33, 47, 4), (39, 100, 7), (40, 96, 5)])
def test_packed_pairs_keep_their_slices_apart(gpu_lib, o, v, nq):
    """Two slices of different states share a packed tile in the split operator (one real plane per state):
    each state of an odd batch gives the bits that it gives alone, in either half of a tile and next to a
    state that is not finite, and follows the oracle."""
    import torch
    from paper_2601_16949_amd import rttda

    prob = I.make_problem(I.Shape(o, v, nq, b_scale=0.05, storage="f32"), 17 + o)
    op = O.Operator.from_problem(prob)
    pulses = I.kick_pulses()
    ctx = rttda.Context(rttda.DeviceProblem(prob, "fp32"), max_rhs=3)
    name = "f32r_p24" if o <= 24 else "f32r_p40"
    k = [k for k in range(1, ctx.lib.rttda_exchange_variants(ctx.desc.precision) + 1) if ctx.variant_name(k) == name]
    ctx.set_tuning(exchange_variant=k[0], exchange_splits=min(3, nq), small_path=2)
    say(f"[packed] {name} o={o} v={v} nq={nq}")

    def run(idx, spoil=None):
        c0, c = gpu_lib.ground_state(len(idx), o, v)
        if spoil is not None:
            c[spoil] = float("nan")
        tr = ctx.propagate([pulses[r] for r in idx], 0.05, 6, c0, c, integrator="sso")
        torch.cuda.synchronize()
        return tr.cpu().numpy(), c

    tr, c = run([0, 1, 2])
    for r in range(3):
        one, c1 = run([r])
        assert np.array_equal(one[:, 0], tr[:, r]) and torch.equal(c1[0], c[r]), r
        ref, _, _ = O.propagate_sso(op, pulses[r], 0.05, 6)
        assert np.max(np.abs(tr[:, r] - ref)) <= 1e-5 * np.max(np.abs(ref)), r
    for spoil in range(3):
        bad, cb = run([0, 1, 2], spoil)
        for r in range(3):
            if r != spoil:
                assert np.array_equal(bad[:, r], tr[:, r]) and torch.equal(cb[r], c[r]), (spoil, r)
