"""Samples and taps that are not finite in automatic filter calls that take segment blocks in
place of the direct sum: only the outputs that use such a value are infinite or NaN, as in
the sum, and the others are the oracle's with those values set to zero (they do not use
them), within the 1e-6 of the norm that segment blocks keep."""
import sys
import zlib

import numpy as np
import pytest

from paper_1810_11359_amd import ism

pytestmark = pytest.mark.gpu

TOL = 1e-6

CASES = [
    # name, n_x, n_pos, n_mic, n_rir: segments, several groups of partitions, ragged ends
    ("segments_of_1", 700, 700, 1, 2048),
    ("segments_of_29", 2000, 70, 3, 2050),
    ("segments_of_201", 20001, 100, 2, 2148),
]

INF, NAN = float("inf"), float("nan")
# (sample positions, taps), as fractions of their ranges: values
BAD = {
    "sample_nan": ([(0.4, NAN)], []),
    "sample_inf_first_and_last": ([(0.0, INF), (1.0, -INF)], []),
    "tap_nan": ([], [(0.5, 0.3, NAN)]),
    "tap_inf_first_and_last": ([], [(0.0, 0.0, INF), (1.0, 1.0, -INF)]),
    "whole_rir_nan": ([], [(0.7, None, NAN)]),
}


@pytest.mark.parametrize("bad", list(BAD))
@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_only_outputs_that_use_it(oracle_mod, case, bad):
    import torch

    name, n_x, n_pos, n_mic, n_rir = case
    seg = -(-n_x // n_pos)
    n_seg = -(-n_x // seg)
    rng = np.random.default_rng(zlib.crc32((name + bad).encode()))
    x = rng.standard_normal(n_x).astype(np.float32)
    rirs = (rng.standard_normal((n_pos, n_mic, n_rir)) * np.exp(-3.0 * np.arange(n_rir) / n_rir)).astype(np.float32)
    x0, r0 = x.copy(), rirs.copy()
    used = np.zeros((n_mic, n_x + n_rir - 1), dtype=bool)
    samples, taps = BAD[bad]
    for where, value in samples:
        i = round(where * (n_x - 1))
        x[i], x0[i] = value, 0.0
        used[:, i:i + n_rir] = True
    for point, where, value in taps:
        p, m = round(point * (n_seg - 1)), n_mic - 1
        first, last = p * seg, min(p * seg + seg, n_x)
        for k in ([round(where * (n_rir - 1))] if where is not None else range(n_rir)):
            rirs[p, m, k], r0[p, m, k] = value, 0.0
            used[m, first + k:last + k] = True
    print(f"[case] {name} {bad}", flush=True)
    sys.stdout.flush()
    xd, rd = torch.from_numpy(x).cuda(), torch.from_numpy(rirs).cuda()
    y = ism.filter_trajectory(xd, rd)
    again = ism.filter_trajectory(xd, rd)
    torch.cuda.synchronize()
    got = y.cpu().numpy().astype(np.float64)
    assert np.array_equal(got, again.cpu().numpy(), equal_nan=True)
    assert np.array_equal(~np.isfinite(got), used)
    ref = oracle_mod.filter_trajectory(x0, r0)
    err = np.linalg.norm(np.where(used, 0.0, got - ref), axis=1) / np.linalg.norm(ref, axis=1)
    print(name, bad, "rel err", err.max())
    assert err.max() <= TOL
