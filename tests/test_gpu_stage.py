"""The general path's Coulomb products and stage update where their layouts can go wrong: rows of ov values
that are and are not a multiple of the load widths (and shorter than one load), auxiliary counts around the
rows in flight and the wave split, one and many Q splits, and a few propagation steps with field and energy
output over few and many partial slabs.  Each against the FP64 oracle."""
import numpy as np
import pytest
from conftest import say

from oracle import rttda64 as O
from paper_2601_16949_amd import inputs as I

pytestmark = pytest.mark.gpu

# X is rounded to 2^-24 relative and both products are FP32 chains of at most a few hundred terms: 2e-6
# is about 30 such roundings in a row.
TOL_J = 2e-6

SHAPES = [(1, 1, 1, 1), (1, 3, 5, 2), (1, 7, 9, 1), (2, 4, 17, 1), (3, 4, 7, 3), (5, 8, 8, 1), (7, 9, 33, 2),
          (13, 5, 64, 1), (8, 32, 65, 4), (9, 57, 31, 1), (11, 36, 16, 2), (4, 514, 259, 1), (6, 350, 1100, 3),
          (15, 139, 257, 5), (24, 184, 63, 1)]


@pytest.mark.parametrize("prec", ["fp32", "mixed"])
@pytest.mark.parametrize("o,v,nq,nrhs", SHAPES)
def test_coulomb_rows_match_oracle(gpu_lib, o, v, nq, nrhs, prec):
    import torch

    # no exchange term: sigma is D X + J alone
    prob = I.make_problem(I.Shape(o, v, nq, 0.05, cx=0.0, storage="f32" if prec == "fp32" else "bf16"), 31 + o)
    op = O.Operator.from_problem(prob)
    ctx = gpu_lib.Context(gpu_lib.DeviceProblem(prob, prec), max_rhs=nrhs)
    ctx.set_tuning(small_path=2)
    c0, c = I.random_state(o, v, nrhs, seed=1000 * o + v)
    dirs, field = np.tile([[0.0, 1.0, 0.0]], (nrhs, 1)), np.zeros(nrhs)
    c0d, cd = gpu_lib.to_planes(c0, c)
    for splits in sorted({1, ctx.get_tuning()["coulomb_splits"]}):
        ctx.set_tuning(coulomb_splits=splits)
        say(f"[coulomb rows] {prec} o={o} v={v} nq={nq} nrhs={nrhs} splits {splits}")
        _, sd = ctx.sigma(field, dirs, c0d, cd)
        torch.cuda.synchronize()
        s = gpu_lib.from_planes(torch.zeros_like(c0d), sd)[1]
        for r in range(nrhs):
            ref = O.apply_H(op, O.dipole_blocks(op, dirs[r]), 0.0, c0[r], c[r])[1]
            assert np.linalg.norm(s[r] - ref) <= TOL_J * np.linalg.norm(ref), (splits, r)


# a relative 2^-24 (FP32) or 2^-16 (split BF16) per product, a few sums of each, over a handful of steps
TOL_STEP = {"fp32": 1e-5, "mixed": 1e-4}


@pytest.mark.parametrize("prec", ["fp32", "mixed"])
@pytest.mark.parametrize("o,v,nq", [(3, 5, 40), (7, 9, 33), (8, 8, 70), (13, 5, 64), (24, 40, 130)])
def test_stage_update_over_few_and_many_slabs(gpu_lib, o, v, nq, prec):
    import torch

    prob = I.make_problem(I.Shape(o, v, nq, 0.05, storage="f32" if prec == "fp32" else "bf16"), 7 + o)
    op = O.Operator.from_problem(prob)
    pulses = [I.Pulse(kind=I.PULSE_DELTA, e0=0.05, direction=(0.0, 0.0, 1.0)),
              I.Pulse(kind=I.PULSE_GAUSS, e0=0.05, omega=0.6, t0=0.2, fwhm=1.0, direction=(1.0, 0.0, 0.0))]
    dt, n = 0.05, 5
    refs = []
    for p in pulses:
        blocks = O.dipole_blocks(op, p.direction)
        s0, S = O.apply_kick(op, blocks, p, 1.0 + 0j, np.zeros((o, v), complex))
        en, mu = [O.energy(op, s0, S)], [O.dipole_expectation(blocks, s0, S)]
        for k in range(n):
            s0, S = O.rk4_step(op, blocks, p, dt, k, s0, S)
            en.append(O.energy(op, s0, S))
            mu.append(O.dipole_expectation(blocks, s0, S))
        refs.append((S, np.array(en), np.array(mu)))
    for splits in (1, nq):
        for graph in (1, 2):
            ctx = gpu_lib.Context(gpu_lib.DeviceProblem(prob, prec), max_rhs=2)
            ctx.set_tuning(small_path=2, exchange_splits=splits, use_graph=graph, steps_per_graph=2)
            say(f"[stage] {prec} o={o} v={v} nq={nq} exchange splits {splits} graph {graph}")
            c0, c = gpu_lib.ground_state(2, o, v)
            energy = torch.empty((n + 1, 2), dtype=torch.float64, device="cuda")
            tr = ctx.propagate(pulses, dt, n, c0, c, energy=energy).cpu().numpy()
            got = gpu_lib.from_planes(c0, c)[1]
            for r, (S, en, mu) in enumerate(refs):
                assert np.linalg.norm(got[r] - S) <= TOL_STEP[prec] * np.linalg.norm(S)
                assert np.max(np.abs(energy[:, r].cpu().numpy() - en)) <= TOL_STEP[prec] * np.max(np.abs(en))
                assert np.max(np.abs(tr[:, r] - mu)) <= TOL_STEP[prec] * np.max(np.abs(mu))


@pytest.mark.parametrize("o,v,nrhs", [(1, 1, 1), (2, 15, 2), (16, 16, 1), (17, 33, 2), (15, 64, 1), (9, 65, 3),
                                      (33, 129, 1), (64, 67, 2), (5, 257, 1)])
def test_field_product_tiles_alone_and_beside_other_launches(gpu_lib, o, v, nrhs):
    """The FP64 field product at the edges of its tiles and contraction quarters: the dipole expectation
    (its own launch), and steps under a field, where the small path's and the first Coulomb product's
    launches carry it, from graphs and directly."""
    import torch

    nq = 24
    prob = I.make_problem(I.Shape(o, v, nq, 0.05, storage="f32"), 3 * o + v)
    op = O.Operator.from_problem(prob)
    c0, c = I.random_state(o, v, nrhs, seed=o)
    dirs = np.random.default_rng(o + v).standard_normal((nrhs, 3))
    ctx = gpu_lib.Context(gpu_lib.DeviceProblem(prob, "fp32"), max_rhs=nrhs)
    c0d, cd = gpu_lib.to_planes(c0, c)
    mu = ctx.dipole_trace(dirs, c0d, cd).cpu().numpy()
    for r in range(nrhs):  # FP64 throughout
        ref = O.dipole_expectation(O.dipole_blocks(op, dirs[r] / np.linalg.norm(dirs[r])), c0[r], c[r])
        assert abs(mu[r] - ref) <= 1e-12 * max(1.0, abs(ref)), r
    pulses = [I.Pulse(kind=I.PULSE_CW, e0=0.05, omega=0.6, phase=0.4, direction=tuple(dirs[r] / np.linalg.norm(dirs[r])))
              for r in range(nrhs)]
    dt, n = 0.05, 4
    ref = [O.propagate(op, pulses[r], dt, n) for r in range(nrhs)]
    for path in (1, 2):
        for graph in (1, 2):
            ctx = gpu_lib.Context(gpu_lib.DeviceProblem(prob, "fp32"), max_rhs=nrhs)
            try:
                ctx.set_tuning(small_path=path, use_graph=graph, steps_per_graph=2)
            except gpu_lib.RttdaError:
                continue  # (too large for the small path)
            say(f"[field] o={o} v={v} nrhs={nrhs} path {path} graph {graph}")
            g0, g = gpu_lib.ground_state(nrhs, o, v)
            tr = ctx.propagate(pulses, dt, n, g0, g).cpu().numpy()
            got = gpu_lib.from_planes(g0, g)[1]
            for r, (t, c0f, cf) in enumerate(ref):
                assert np.max(np.abs(tr[:, r] - t)) <= TOL_STEP["fp32"] * np.max(np.abs(t))
                assert np.linalg.norm(got[r] - cf) <= TOL_STEP["fp32"] * np.linalg.norm(cf)


@pytest.mark.parametrize("o,v,nq,gaps", [(4, 5, 3, 1), (8, 33, 7, 2), (3, 4, 2, 3)])
def test_spectral_radius_where_the_start_spans_an_invariant_space(gpu_lib, o, v, nq, gaps):
    """A with `gaps` distinct eigenvalues (no two-electron part): Lanczos ends after that many steps, and the
    steps queued behind its end leave the answer alone."""
    prob = I.make_problem(I.Shape(o, v, nq, 0.05, storage="f32"), 5)
    prob.b_ov[:], prob.b_oo[:], prob.b_vv[:] = 0, 0, 0
    prob.e_occ[:] = -0.5
    prob.e_virt[:] = 0.25 + 0.5 * (np.arange(v) * gaps // v)
    ctx = gpu_lib.Context(gpu_lib.DeviceProblem(prob, "fp32"), max_rhs=1)
    rho, bound = ctx.spectral_radius(n_iter=20)
    top = prob.e_virt[-1] + 0.5
    say(f"[lanczos] {gaps} distinct gaps: rho {rho!r} bound {bound!r} exact {top!r}")
    assert abs(rho - top) <= 1e-12 * top and top * (1 - 1e-12) <= bound <= top * (1 + 1e-6)


@pytest.mark.parametrize("prec", ["fp32", "mixed"])
@pytest.mark.parametrize("o,v,nq,nrhs", [(5, 7, 3, 16), (9, 33, 70, 16), (8, 40, 64, 31), (7, 9, 65, 32), (6, 25, 33, 33),
                                         (11, 13, 129, 47), (8, 16, 31, 64), (5, 5, 40, 70)])
def test_coulomb_batches_match_oracle(gpu_lib, o, v, nq, nrhs, prec):
    """The matrix-core Coulomb pair over its widths (32, 64 and 128 slices and more than one such block) and
    rows that do and do not come in fours; under a field, which the first launch carries."""
    import torch

    prob = I.make_problem(I.Shape(o, v, nq, 0.05, cx=0.0, storage="f32" if prec == "fp32" else "bf16"), 77 + o)
    op = O.Operator.from_problem(prob)
    ctx = gpu_lib.Context(gpu_lib.DeviceProblem(prob, prec), max_rhs=nrhs)
    ctx.set_tuning(small_path=2)
    assert ctx.get_tuning()["coulomb_path"] == 2
    c0, c = I.random_state(o, v, nrhs, seed=o + v)
    dirs = [I.AXES[r % 3] for r in range(nrhs)]
    field = [0.01 * ((r % 5) - 2) for r in range(nrhs)]
    c0d, cd = gpu_lib.to_planes(c0, c)
    _, sd = ctx.sigma(field, dirs, c0d, cd)
    torch.cuda.synchronize()
    s = gpu_lib.from_planes(torch.zeros_like(c0d), sd)[1]
    for r in range(nrhs):
        ref = O.apply_H(op, O.dipole_blocks(op, dirs[r]), field[r], c0[r], c[r])[1]
        assert np.linalg.norm(s[r] - ref) <= TOL_J * np.linalg.norm(ref), r
    say(f"[coulomb batches] {prec} o={o} v={v} nq={nq} nrhs={nrhs}")
    pulses = [I.Pulse(kind=I.PULSE_CW, e0=0.05, omega=0.6, phase=0.1 * r, direction=dirs[r]) for r in range(nrhs)]
    g0, g = gpu_lib.ground_state(nrhs, o, v)
    tr = ctx.propagate(pulses, 0.05, 2, g0, g).cpu().numpy()
    for r in (0, nrhs - 1):
        t, _, _ = O.propagate(op, pulses[r], 0.05, 2)
        assert np.max(np.abs(tr[:, r] - t)) <= TOL_STEP[prec] * np.max(np.abs(t))
