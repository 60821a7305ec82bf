"""The tap that a window's end cuts, alone: free-field RIRs (one image) of many delay
fractions with windows just below an even number of samples, where the cut tap's polynomial
is worst, and just above a cap, where the moments take it.

With W/2 = h and j2 = floor(h) + 1, the samples k0 + j2 and k0 + 1 - j2 of an image at
k0 + f hold nothing but that tap (zero for half of the fractions). Errors are divided by the
image's amplitude. Tolerance: the fit (1.9e-9 under the cap of 64, 3.3e-8 above it), the
rounding of ten coefficients and as many steps of Horner's rule, 12 x 2^-24 of the tap's
largest value, and a delay fraction rounded to FP32, 2^-25 of its largest slope."""
import sys

import numpy as np
import pytest

from paper_1810_11359_amd import ism

pytestmark = pytest.mark.gpu

WINDOWS = [(4.1, 1.9e-9), (5.5, 1.9e-9), (5.925, 1.9e-9), (7.925, 1.9e-9), (9.8, 1.9e-9), (13.95, 1.9e-9),
           (31.9, 1.9e-9), (63.8, 1.9e-9), (64.9, 3.3e-8), (95.9, 3.3e-8)]


def cut_tap(u, W):
    """Eq. (6) at a distance u inside the window's end."""
    v = W / 2.0 - u
    return np.where(u > 0.0, np.sinc(v) * 0.5 * (1.0 + np.cos(2.0 * np.pi * v / W)), 0.0)


@pytest.mark.parametrize("W,fit", WINDOWS, ids=[f"W{w[0]:g}" for w in WINDOWS])
def test_cut_taps(W, fit):
    import torch

    fs, c, L = 16000.0, 343.0, [12.0, 9.0, 8.0]
    room = ism.Room(L, [0.5] * 6, (1, 1, 1), c, fs, 0.04, W / fs)
    src = np.array([[1.0, 4.0, 3.0]], dtype=np.float32)
    n = 1024
    rcv = np.tile(src, (n, 1))
    rcv[:, 0] += np.linspace(3.0, 9.0, n, dtype=np.float32)
    print(f"[case] cut taps W = {W:g}", flush=True)
    sys.stdout.flush()
    h = ism.simulate(room, src, rcv)[0]
    torch.cuda.synchronize()
    h = h.cpu().numpy().astype(np.float64)
    d = np.linalg.norm(rcv.astype(np.float64) - src.astype(np.float64), axis=1)
    x = d * fs / c
    k0 = np.floor(x).astype(int)
    f = x - k0
    amp = 1.0 / (4.0 * np.pi * d)
    j2 = int(np.floor(W / 2.0)) + 1
    grid = np.linspace(0.0, 1.0 - (j2 - W / 2.0), 4001)
    tap = cut_tap(grid, W)
    tol = fit + 12.0 * 2.0 ** -24 * np.max(np.abs(tap)) + 2.0 ** -25 * np.max(np.abs(np.gradient(tap, grid)))
    near = np.minimum(f, 1.0 - f) < 1e-5  # (either floor)
    i = np.arange(n)
    right = np.abs(h[i, k0 + j2] / amp - cut_tap(f - (j2 - W / 2.0), W))
    left = np.abs(h[i, k0 + 1 - j2] / amp - cut_tap(1.0 - (j2 - W / 2.0) - f, W))
    worst = max(np.max(right[~near]), np.max(left[~near]))
    print(f"W = {W:g}: cut taps off by {worst:.2e} of the amplitude, bound {tol:.2e}", flush=True)
    assert worst <= tol
