"""Device spectra (rttda_spectrum, eq. fourier_transform and eq. spectrum_average) of GPU dipole
traces and time correlations against the oracle's transforms of the same signals
(oracle.spectrum.dtft and oracle.spectrum.correlation_spectrum, FP64 on both sides).  (The signals themselves are checked against the oracle elsewhere: traces in the
parity tests, correlations in test_gpu_corr.)"""
import numpy as np
import pytest

from conftest import say
from oracle import spectrum as SP
from paper_2601_16949_amd import inputs as I

pytestmark = pytest.mark.gpu


def _run(gpu_lib, n):
    import torch
    from paper_2601_16949_amd import rttda

    o, v, nq = 10, 40, 120
    prob = I.make_problem(I.Shape(o, v, nq, b_scale=0.05, storage="f32"), 16949)
    ctx = rttda.Context(rttda.DeviceProblem(prob, "fp32"), max_rhs=3)
    pulses = I.kick_pulses(kappa=1e-3)
    c0d, cd = gpu_lib.ground_state(3, o, v)
    corr = torch.empty((n + 1, 3, 2), dtype=torch.float64, device="cuda")
    tr = ctx.propagate(pulses, 0.05, n, c0d, cd, corr=corr)
    torch.cuda.synchronize()
    return tr, corr


def test_spectra_match_the_transform_definition(gpu_lib):
    import torch

    n, kappa, dt = 1500, 1e-3, 0.05
    tr, corr = _run(gpu_lib, n)
    omega = np.linspace(0.2, 1.6, 701)
    S = gpu_lib.spectrum(tr, dt, omega, kappa=kappa).cpu().numpy()
    Sa = gpu_lib.spectrum(tr, dt, omega, kappa=kappa, average=True).cpu().numpy()
    C = gpu_lib.spectrum(corr, dt, omega).cpu().numpy()
    torch.cuda.synchronize()
    trh, ch = tr.cpu().numpy(), corr.cpu().numpy()
    worst = 0.0
    for s in range(3):
        for j in range(0, omega.size, 50):
            ref = SP.dtft(trh[:, s], dt, kappa, omega[j])
            worst = max(worst, abs(S[s, j] - ref) / np.max(np.abs(S[s])))
            refc = SP.correlation_spectrum(ch[:, s, 0] + 1j * ch[:, s, 1], dt, omega[j])[0]
            worst = max(worst, abs(C[s, j] - refc) / np.max(np.abs(C[s])))
    say(f"[spectrum] worst relative deviation from the transform definition {worst:.2e}")
    assert worst < 1e-10
    assert np.max(np.abs(Sa - S.mean(axis=0))) <= 1e-12 * np.max(np.abs(Sa))


def test_spectrum_argument_errors(gpu_lib):
    import torch

    sig = torch.zeros((10, 2), dtype=torch.float64, device="cuda")
    with pytest.raises(gpu_lib.RttdaError):
        gpu_lib.spectrum(sig, 0.05, np.linspace(0.1, 1.0, 5), kappa=0.0)
    with pytest.raises(gpu_lib.RttdaError):
        gpu_lib.spectrum(sig, -0.05, np.linspace(0.1, 1.0, 5), kappa=1.0)
    # the binding refuses what the library cannot check: a correlation without its (re, im)
    # pair and a frequency grid that is not uniform
    with pytest.raises(ValueError):
        gpu_lib.spectrum(torch.zeros((10, 2, 1), dtype=torch.float64, device="cuda"), 0.05, np.linspace(0.1, 1.0, 5))
    with pytest.raises(ValueError):
        gpu_lib.spectrum(sig, 0.05, np.array([0.1, 0.2, 0.4]), kappa=1.0)


@pytest.mark.parametrize("n_t,nsig,n_w", [(1, 1, 1), (2, 2, 3), (255, 3, 4), (257, 4, 5), (8193, 7, 9)])
def test_spectrum_edges(gpu_lib, n_t, nsig, n_w):
    """Sample counts around the block's 256 lanes and its 8192-sample phase refresh, signal counts
    around the groups of three and frequency counts around the groups of four, both kinds.  The
    phases reach w t = 655 rad, so each sine is good to about 655 x 1.1e-16 on either side: 1e-12 of
    the windowed sum of |y| leaves a factor of ten."""
    import torch

    rng = np.random.default_rng(5)
    dt, kappa = 0.05, 1e-3
    omega = 0.2 + 0.175 * np.arange(n_w)
    y = rng.standard_normal((n_t, nsig))
    z = rng.standard_normal((n_t, nsig, 2))
    S = gpu_lib.spectrum(torch.from_numpy(y).cuda(), dt, omega, kappa=kappa).cpu().numpy()
    Sa = gpu_lib.spectrum(torch.from_numpy(y).cuda(), dt, omega, kappa=kappa, average=True).cpu().numpy()
    C = gpu_lib.spectrum(torch.from_numpy(z).cuda(), dt, omega).cpu().numpy()
    n = np.arange(n_t)
    h = 0.5 * (1.0 + np.cos(np.pi * n / (n_t - 1))) if n_t > 1 else np.ones(1)
    for j, w in enumerate(omega):
        sn, cs = np.sin(w * (n * dt)), np.cos(w * (n * dt))
        ref = w * dt / kappa * ((h * sn) @ (y - y[0]))
        bar = 1e-12 * w * dt / kappa * (h @ np.abs(y - y[0]) + 1.0)
        assert np.all(np.abs(S[:, j] - ref) <= bar)
        assert abs(Sa[j] - ref.mean()) <= bar.max()
        refc = w * dt * ((h * cs) @ z[:, :, 0] - (h * sn) @ z[:, :, 1])
        assert np.all(np.abs(C[:, j] - refc) <= 1e-12 * w * dt * (h @ np.abs(z).sum(axis=2) + 1.0))
