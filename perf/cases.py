"""The work a user has this framework do, as cases that can be timed and compared.

Every case is one call (or, for the admission check and the spectra, the call that goes with a run)
through the public binding `paper_2601_16949_amd.rttda`, on seeded synthetic factors drawn on the
device by the recipe of `paper_2601_16949_amd/inputs.py` (orbital energies, N(0,1) factors capped so
that the Coulomb edge stays at 4.79 Ha, dipoles N(0, 0.5)).  A case is a dict of plain values:

  kind       "rk4" | "sso" (Context.propagate with that integrator), "radius"
             (Context.spectral_radius, the time-step check before a run), "spectrum"
  o, v, nq   occupied, virtual and auxiliary counts;  precision "fp32" | "mixed" (BF16 factors)
  nrhs       right-hand sides;  steps, dt: the propagation
  pulse      "kick" (delta kicks at step 0 along z, or x/y/z), "gauss" (Gaussian-envelope carriers,
             the call in the middle of the envelope, from excited states), "cw"
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2601_16949_amd import inputs as I
from paper_2601_16949_amd import rttda

DEV = "cuda:0"
KAPPA = 1e-4
CX = 0.2
# A fine step: RK4 keeps the norm to 1e-13 a step, so a run of many steps keeps it to 1e-10.  The work
# of a step does not depend on it; the amplitudes move by dt sigma, so the FP64 amplitudes that a call
# returns carry the FP32 sums behind sigma to about 1e-6 of a state's size.
DT = 0.002
T_MID = 400.0  # calls inside a pulse start at the envelope's centre (au)


def _case(name, kind, o, v, nq, precision, nrhs, pulse, steps, dt=DT):
    return {"name": name, "kind": kind, "o": o, "v": v, "nq": nq, "precision": precision, "nrhs": nrhs,
            "pulse": pulse, "steps": steps, "dt": dt}


def listed():
    return [
        # the smallest molecule (the smoke test's and workload 1's shape), a z kick: launch-bound, the
        # host path and the launches between a step's kernels count
        _case("small_kick_fp32", "rk4", 10, 40, 120, "fp32", 1, "kick", 16),
        # the serving stream's request sizes (v = 7.5 o, N_Q = 20 o, BF16 factors), served at padded
        # sizes in chunks of 8 steps: a small request with a pulse on, and a larger one after its kick
        _case("serve_pulse_mixed", "rk4", 24, 184, 480, "mixed", 1, "gauss", 8),
        _case("serve_kick_mixed", "rk4", 96, 720, 1920, "mixed", 1, "kick", 1),
        # sizes as a user's basis set gives them, on a context without the server's padding: odd
        # counts, a continuous wave or a pulse on, two and three states at once
        _case("odd_cw_fp32", "rk4", 27, 203, 541, "fp32", 3, "cw", 4),
        _case("odd_pulse_mixed", "rk4", 37, 277, 743, "mixed", 2, "gauss", 2),
        # an absorption spectrum's x/y/z kicks at the benchmark's shape: RK4 in both precisions and
        # the split operator
        _case("kick_xyz_fp32", "rk4", 60, 400, 1500, "fp32", 3, "kick", 2),
        _case("kick_xyz_mixed", "rk4", 60, 400, 1500, "mixed", 3, "kick", 2),
        _case("kick_xyz_sso_fp32", "sso", 60, 400, 1500, "fp32", 3, "kick", 4),
        # a 64-frequency strong-field scan, one step in the middle of the pulses
        _case("scan64_fp32", "rk4", 40, 300, 1000, "fp32", 64, "gauss", 1),
        # the largest molecule of the configurations, 37 GB of BF16 factors, one step
        _case("large_kick_mixed", "rk4", 240, 1800, 5000, "mixed", 3, "kick", 1),
        # the time-step check every served request and every benchmark run takes first (20 Lanczos
        # steps on the request's own operator)
        _case("admission_mixed", "radius", 48, 360, 960, "mixed", 1, "kick", 20),
        # the x/y/z spectrum of a whole 20000-step run, averaged
        _case("spectrum_20k", "spectrum", 60, 400, 1500, "fp32", 3, "kick", 20000, dt=0.05),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the same ranges; within each range sizes are spread over their logarithm."""
    k = rng.randrange(9)
    if k == 0:  # the smallest molecules
        o = rng.randint(6, 14)
        return _draw("rk4", o, rng.randint(3 * o, 5 * o), rng.randint(8 * o, 13 * o), rng.choice(["fp32", "mixed"]),
                     rng.randint(1, 2), rng.choice(["kick", "gauss"]), 16)
    if k in (1, 2):  # served requests, padded as the server pads them
        o = _log_int(rng, 12, 110)
        nq, v = 20 * o, (int(7.5 * o) + 7) // 8 * 8
        return _draw("rk4", (o + 1) // 2 * 2, v, nq, "mixed", 1, rng.choice(["kick", "gauss"]), 8 if o < 40 else 1)
    if k in (3, 4):  # unpadded sizes
        o = _log_int(rng, 15, 63)
        v = rng.randint(5 * o, 8 * o)
        return _draw("rk4", o, v, rng.randint(15 * o, 25 * o), rng.choice(["fp32", "mixed"]), rng.randint(1, 4),
                     rng.choice(["cw", "gauss", "kick"]), 2)
    if k in (5, 6):  # spectra of mid-sized molecules
        o = rng.randint(9, 16) * 4
        v = rng.randint(5 * o // 4, 8 * o // 4) * 4
        return _draw(rng.choice(["rk4", "sso"]), o, v, rng.randint(18 * o, 27 * o), rng.choice(["fp32", "mixed"]),
                     rng.choice([1, 3, 6]), "kick", 2)
    if k == 7:  # frequency scans
        o = rng.randint(5, 11) * 4
        return _draw("rk4", o, rng.randint(6 * o // 4, 8 * o // 4) * 4, 25 * o, rng.choice(["fp32", "mixed"]),
                     _log_int(rng, 8, 64), "gauss", 1)
    o = _log_int(rng, 128, 208) // 8 * 8  # large molecules
    return _draw("rk4", o, (int(7.5 * o) + 7) // 8 * 8, _log_int(rng, 500, 2500), "mixed", rng.choice([1, 3]), "kick", 1)


def _draw(*args):
    c = _case("", *args)
    del c["name"]
    return c


# ------------------------------------------------------------------------------------------------
# Inputs: made from the case and the seed alone, on the device.
# ------------------------------------------------------------------------------------------------
def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * int(seed) + 7919 * stream + 17)
    return g


def _sym(m):
    return torch.triu(m) + torch.triu(m, 1).transpose(-1, -2)


def _tensors(case, seed):
    o, v, nq = case["o"], case["v"], case["nq"]
    dt = torch.float32 if case["precision"] == "fp32" else torch.bfloat16
    s = min(0.02 if case["precision"] == "mixed" and o >= 128 else 0.05,
            1.547 / (math.sqrt(o * v) + math.sqrt(nq)))
    g = _gen(seed, 0)
    t = {"e_occ": torch.sort(torch.rand(o, generator=g, device=DEV, dtype=torch.float64) * 0.7 - 1.0)[0],
         "e_virt": torch.sort(torch.rand(v, generator=g, device=DEV, dtype=torch.float64) * 1.45 + 0.05)[0],
         "mu": (_sym(torch.randn((3, o + v, o + v), generator=g, device=DEV, dtype=torch.float64)) * 0.5).contiguous(),
         "b_ov": torch.empty((nq, o, v), dtype=dt, device=DEV), "b_oo": torch.empty((nq, o, o), dtype=dt, device=DEV),
         "b_vv": torch.empty((nq, v, v), dtype=dt, device=DEV)}
    for q in range(0, nq, 100):
        n = min(nq, q + 100) - q
        t["b_ov"][q:q + n] = torch.randn((n, o, v), generator=g, device=DEV).mul_(s).to(dt)
        t["b_oo"][q:q + n] = _sym(torch.randn((n, o, o), generator=g, device=DEV).mul_(s)).to(dt)
        t["b_vv"][q:q + n] = _sym(torch.randn((n, v, v), generator=g, device=DEV).mul_(s)).to(dt)
    return t


def _pulses(case):
    R = case["nrhs"]
    axes = [(0.0, 0.0, 1.0)] if R == 1 else [((1.0, 0.0, 0.0), (0.0, 1.0, 0.0), (0.0, 0.0, 1.0))[r % 3] for r in range(R)]
    if case["pulse"] == "kick":
        return [I.Pulse(kind=I.PULSE_DELTA, e0=KAPPA, direction=a) for a in axes]
    if case["pulse"] == "cw":
        return [I.Pulse(kind=I.PULSE_CW, e0=0.01, omega=0.3 + 0.05 * r, phase=0.3, direction=a)
                for r, a in enumerate(axes)]
    return I.gauss_cos_scan(0.39, 0.05, n=R)


def _states(case, seed):
    """The states a call starts from: the ground state before a kick; inside a pulse, ground states
    with a fifth of their weight in the singles."""
    R, o, v = case["nrhs"], case["o"], case["v"]
    c0 = torch.zeros((R, 2), dtype=torch.float64, device=DEV)
    c0[:, 0] = 1.0
    c = torch.zeros((R, 2, o, v), dtype=torch.float64, device=DEV)
    if case["pulse"] != "kick":
        c = torch.randn((R, 2, o, v), generator=_gen(seed, 1), device=DEV, dtype=torch.float64)
        c *= math.sqrt(0.2 / (2 * o * v))
        c0 *= math.sqrt(0.8)
    return c0, c


def _step0(case):
    return 0 if case["pulse"] == "kick" else round(T_MID / case["dt"])


def _signal(case, seed):
    """Dipole traces of a kicked run: a few hundred damped lines per signal, ~1e-4 in size."""
    n, R = case["steps"] + 1, case["nrhs"]
    g = _gen(seed, 2)
    t = torch.arange(n, device=DEV, dtype=torch.float64)[:, None] * case["dt"]
    out = torch.zeros((n, R), dtype=torch.float64, device=DEV)
    for r in range(R):
        w = torch.rand(200, generator=g, device=DEV, dtype=torch.float64) * 2.0 + 0.3
        a = torch.rand(200, generator=g, device=DEV, dtype=torch.float64) * 2e-4
        out[:, r] = (torch.sin(t * w) @ a)
    return out


def _omega(case):
    return np.linspace(0.2, 1.2, 2001)


class State:
    pass


def prepare(case, seed):
    st = State()
    st.case = case
    if case["kind"] == "spectrum":
        st.signal, st.omega = _signal(case, seed), _omega(case)
        return st
    shape = I.Shape(case["o"], case["v"], case["nq"], cx=CX, storage="f32" if case["precision"] == "fp32" else "bf16")
    st.dev = rttda.DeviceProblem.from_tensors(shape, _tensors(case, seed), case["precision"])
    st.ctx = rttda.Context(st.dev, max_rhs=case["nrhs"])
    if case["kind"] == "radius":
        return st
    st.ctx.use_tuned(case["nrhs"], case["kind"])
    st.pulses = _pulses(case)
    st.init = _states(case, seed)
    st.c0, st.c = torch.empty_like(st.init[0]), torch.empty_like(st.init[1])
    return st


def run(st):
    case = st.case
    if case["kind"] == "spectrum":
        return rttda.spectrum(st.signal, case["dt"], st.omega, kappa=KAPPA, average=True)
    if case["kind"] == "radius":
        return st.ctx.spectral_radius(case["steps"])
    st.c0.copy_(st.init[0])
    st.c.copy_(st.init[1])
    trace = st.ctx.propagate(st.pulses, case["dt"], case["steps"], st.c0, st.c, step0=_step0(case),
                             integrator=case["kind"])
    return {"trace": trace, "c0": st.c0, "c": st.c}


def _sigma_flops(case):
    """Two-electron flops of one complex sigma per state (Coulomb pair and exchange)."""
    o, v, nq = case["o"], case["v"], case["nq"]
    return 8.0 * nq * o * v + 4.0 * nq * o * v * (o + v)


def work(case):
    o, v, nq, R, n = case["o"], case["v"], case["nq"], case["nrhs"], case["steps"]
    if case["kind"] == "spectrum":
        m = len(_omega(case))
        return {"bytes": 8.0 * ((n + 1) * R + m), "flops": 2.0 * (n + 1) * R * m}
    b = 4 if case["precision"] == "fp32" else 2
    factors = float(nq) * (o * v + o * o + v * v) * b
    if case["kind"] == "radius":
        return {"bytes": factors + 8.0 * (o + v), "flops": n * 0.5 * _sigma_flops(case)}
    # states in and out, dipoles, energies, trace
    other = 8.0 * (2 * R * (2 * o * v + 2) + 3 * (o + v) ** 2 + o + v + (n + 1) * R)
    field = 4.0 * o * v * (o + v) * R  # one product with the dipole blocks, both planes
    per_step = 4 if case["kind"] == "rk4" else 1
    n_field = (4 if case["kind"] == "rk4" else 3) * n + 1 if case["pulse"] != "kick" else n + 2
    return {"bytes": factors + other, "flops": n * per_step * R * _sigma_flops(case) + n_field * field}


# ------------------------------------------------------------------------------------------------
# The same results in 64 bits, in plain torch.
# ------------------------------------------------------------------------------------------------
class _Exact:
    def __init__(self, case, seed):
        self.case, self.t = case, _tensors(case, seed)
        self.D = self.t["e_virt"][None, :] - self.t["e_occ"][:, None]
        self.axes = [torch.tensor(p.direction, dtype=torch.float64, device=DEV) for p in _pulses(case)]
        self.chunk = max(1, min(case["nq"], int(4e8 / (case["v"] * (case["v"] + 2 * case["nrhs"] * case["o"])))))

    def A(self, x):
        """A x for real slices x [n, o, v]."""
        n, o, v = x.shape
        out = self.D * x
        flat = x.reshape(n * o, v)
        for q in range(0, self.case["nq"], self.chunk):
            bov, boo, bvv = (self.t[k][q:q + self.chunk].double() for k in ("b_ov", "b_oo", "b_vv"))
            m = bov.shape[0]
            d = bov.reshape(m, o * v) @ x.reshape(n, o * v).t().contiguous()
            out += 2.0 * (d.t().contiguous() @ bov.reshape(m, o * v)).reshape(n, o, v)
            # W[s, i, (Q, b)] = sum_a x[s, i, a] B_vv[Q, a, b] (symmetric B_vv), then over (Q, j)
            w = (flat @ bvv.reshape(m * v, v).t().contiguous()).reshape(n, o, m, v)
            w = w.permute(0, 2, 1, 3).reshape(n, m * o, v).contiguous()
            boo = boo.permute(1, 0, 2).reshape(o, m * o).contiguous()
            for s in range(n):
                out[s] -= CX * (boo @ w[s])
        return out

    def M(self, r, c0, C):
        """The dipole operator along state r's axis on (c0, C), complex."""
        o = self.case["o"]
        mu = torch.tensordot(self.axes[r], self.t["mu"], 1)
        oo, ov, vv = mu[:o, :o].contiguous(), mu[:o, o:].contiguous(), mu[o:, o:].contiguous()
        f = torch.stack([P @ vv - oo @ P for P in (C.real.contiguous(), C.imag.contiguous())])
        return math.sqrt(2.0) * (ov * C).sum(), torch.complex(f[0], f[1]) + math.sqrt(2.0) * ov * c0


def _field(p, t):
    if p.kind == I.PULSE_CW:
        return p.e0 * math.sin(p.omega * t + p.phase)
    if p.kind == I.PULSE_GAUSS:
        s, tau = p.fwhm / 2.35482, t - p.t0
        return p.e0 * math.exp(-tau * tau / (2.0 * s * s)) * math.sin(p.omega * tau + p.phase)
    return 0.0


def _exact_propagate(case, seed):
    ex, pulses, R = _Exact(case, seed), _pulses(case), case["nrhs"]
    p0, pc = _states(case, seed)
    x0 = [torch.complex(p0[r, 0], p0[r, 1]) for r in range(R)]
    X = [torch.complex(pc[r, 0], pc[r, 1]) for r in range(R)]
    dt, step0 = case["dt"], _step0(case)
    if case["pulse"] == "kick":
        for r in range(R):
            m0, m = ex.M(r, x0[r], X[r])
            x0[r], X[r] = x0[r] + 1j * KAPPA * m0, X[r] + 1j * KAPPA * m
    trace = torch.empty((case["steps"] + 1, R), dtype=torch.float64, device=DEV)

    def sample(k):
        for r in range(R):
            m0, m = ex.M(r, x0[r], X[r])
            trace[k, r] = ((x0[r].conj() * m0).real + (X[r].conj() * m).real.sum())

    def H(y0, Y, t):
        planes = torch.stack([P for C in Y for P in (C.real, C.imag)])
        a = ex.A(planes)
        h0, h = [], []
        for r in range(R):
            E = _field(pulses[r], t)
            s0, s = torch.zeros_like(y0[r]), torch.complex(a[2 * r], a[2 * r + 1])
            if E != 0.0:
                m0, m = ex.M(r, y0[r], Y[r])
                s0, s = s0 - E * m0, s - E * m
            h0.append(s0)
            h.append(s)
        return h0, h

    def shifted(k, f):
        return [x0[r] + f * k[0][r] for r in range(R)], [X[r] + f * k[1][r] for r in range(R)]

    sample(0)
    for n in range(case["steps"]):
        t = (step0 + n) * dt
        if case["kind"] == "rk4":
            k1 = H(x0, X, t)
            k2 = H(*shifted(k1, -0.5j * dt), t + 0.5 * dt)
            k3 = H(*shifted(k2, -0.5j * dt), t + 0.5 * dt)
            k4 = H(*shifted(k3, -1j * dt), t + dt)
            x0 = [x0[r] - 1j * dt / 6 * (k1[0][r] + 2 * k2[0][r] + 2 * k3[0][r] + k4[0][r]) for r in range(R)]
            X = [X[r] - 1j * dt / 6 * (k1[1][r] + 2 * k2[1][r] + 2 * k3[1][r] + k4[1][r]) for r in range(R)]
        else:  # kick, drift, kick on X = q + ip; no field after a kick, so the ground row stays put
            q, p = torch.stack([C.real for C in X]), torch.stack([C.imag for C in X])
            p = p - 0.5 * dt * ex.A(q)
            q = q + dt * ex.A(p)
            p = p - 0.5 * dt * ex.A(q)
            X = [torch.complex(q[r], p[r]) for r in range(R)]
        sample(n + 1)
    return {"trace": trace, "c0": torch.stack([torch.view_as_real(z) for z in x0]),
            "c": torch.stack([torch.stack([C.real, C.imag]) for C in X])}


def _exact_spectrum(case, seed):
    y, w = _signal(case, seed), torch.from_numpy(_omega(case)).to(DEV)
    n = y.shape[0]
    t = torch.arange(n, device=DEV, dtype=torch.float64)
    h = 0.5 * (1.0 + torch.cos(math.pi * t / (n - 1)))
    g = h[:, None] * (y - y[:1])
    s = torch.stack([(torch.sin(wi * t * case["dt"]) @ g) * wi for wi in w]) * (case["dt"] / KAPPA)
    return s.mean(dim=1)


def exact(case, seed):
    if case["kind"] == "spectrum":
        return _exact_spectrum(case, seed)
    if case["kind"] == "radius":
        return None  # Ritz values of a short Lanczos run have no value of their own beyond their bound
    # a float64 product runs at a few tens of TFLOP/s: the frequency scan and the largest molecules
    # would take longer than the rest together
    if case["steps"] * case["nrhs"] * _sigma_flops(case) > 3e13:
        return None
    return _exact_propagate(case, seed)
