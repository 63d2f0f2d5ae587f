"""Spectra of short records, which take blocks of one wave, or a thread per frequency where there are many: around the
wave's 64 samples, the length from which blocks of four are taken and the count from which threads are, and many
frequencies of a short record in a fraction of a long one's time."""
import ctypes

import numpy as np
import pytest
from conftest import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_t,nsig,n_w", [(1, 2, 5), (63, 4, 3), (64, 1, 4), (65, 3, 5), (129, 2, 1), (1023, 3, 6), (1024, 4, 4),
                                          (1025, 1, 7), (1, 4, 1024), (1, 1, 1300), (2, 5, 2047), (2, 5, 2048), (7, 2, 7169)])
def test_short_records_match_the_sums(gpu_lib, n_t, nsig, n_w):
    """The phases reach w t = 82 rad, so each sine is good to about 82 x 1.1e-16 on either side and 15 rotations
    add 15 roundings: 1e-13 of the windowed sum of |y| leaves a factor of ten."""
    import torch

    rng = np.random.default_rng(n_t)
    dt, kappa = 0.05, 1e-3
    omega = 0.2 + (0.175 if n_w < 20 else 1e-4) * np.arange(n_w)
    y = rng.standard_normal((n_t, nsig))
    z = rng.standard_normal((n_t, nsig, 2))
    S = gpu_lib.spectrum(torch.from_numpy(y).cuda(), dt, omega, kappa=kappa).cpu().numpy()
    Sa = gpu_lib.spectrum(torch.from_numpy(y).cuda(), dt, omega, kappa=kappa, average=True).cpu().numpy()
    C = gpu_lib.spectrum(torch.from_numpy(z).cuda(), dt, omega).cpu().numpy()
    n = np.arange(n_t)
    h = 0.5 * (1.0 + np.cos(np.pi * n / (n_t - 1))) if n_t > 1 else np.ones(1)
    for j in sorted({*range(min(n_w, 9)), n_w // 2, n_w - 2, n_w - 1} & set(range(n_w))):
        w = omega[j]
        sn, cs = np.sin(w * (n * dt)), np.cos(w * (n * dt))
        ref = w * dt / kappa * ((h * sn) @ (y - y[0]))
        bar = 1e-13 * w * dt / kappa * (h @ np.abs(y - y[0]) + 1.0)
        assert np.all(np.abs(S[:, j] - ref) <= bar)
        assert abs(Sa[j] - ref.mean()) <= bar.max()
        refc = w * dt * ((h * cs) @ z[:, :, 0] - (h * sn) @ z[:, :, 1])
        assert np.all(np.abs(C[:, j] - refc) <= 1e-13 * w * dt * (h @ np.abs(z).sum(axis=2) + 1.0))


def test_many_frequencies_of_a_short_record(gpu_lib):
    import torch

    n_w = 400000
    out = torch.empty((1, n_w), dtype=torch.float64, device="cuda")
    stream = torch.cuda.current_stream()
    t = {}
    for n_t in (10, 50, 4000):
        y = torch.randn((n_t, 1), dtype=torch.float64, device="cuda")
        ts = []
        for _ in range(6):
            ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            ev[0].record()
            gpu_lib._check(gpu_lib.load().rttda_spectrum(ctypes.c_void_p(stream.cuda_stream), 0, y.data_ptr(), n_t, 1, 0.05, 1e-4,
                                                         n_w, 0.1, 1e-5, 0, out.data_ptr()))
            ev[1].record()
            torch.cuda.synchronize()
            ts.append(ev[0].elapsed_time(ev[1]))
        t[n_t] = min(ts)
    say(f"[spectrum] {n_w} frequencies: 50 samples {t[50] * 1e3:.0f} us, 4000 samples {t[4000] * 1e3:.0f} us, "
        f"10 samples {t[10] * 1e3:.0f} us")
    assert t[50] < 0.4 * t[4000] and t[10] < 0.5 * t[50]
