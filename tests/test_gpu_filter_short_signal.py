"""Segment blocks of signals with fewer segments than an RIR's partitions span, where an
output block meets only some of the partitions: against the FP64 oracle, several transforms
per workgroup and one, one and several partitions per block, in one group and in several.

Tolerance, of the norm of y per microphone: as for the other segment blocks, 1e-6."""
import sys
import zlib

import numpy as np
import pytest

from paper_1810_11359_amd import ism

pytestmark = pytest.mark.gpu

CASES = [
    # n_x, n_pos, n_mic, n_rir, method: transform size, segments per partition, partitions (met per block)
    (303, 3, 8, 20879, "fft"),      # 512, 4, 52 (1)
    (345, 5, 8, 16669, "fft"),      # 512, 6, 41 (1)
    (1001, 10, 2, 9000, "auto"),    # 512, 4, 23 (3), ragged last segment
    (500, 50, 1, 5000, "auto"),     # 512, 50, 10 (1): as many segments as one partition spans
    (6000, 6, 1, 30000, "auto"),    # 4096, 3, 10 (2): two groups
    (9000, 3, 2, 60000, "auto"),    # 8192, 1, 20 (3): a transform per workgroup
    (7000, 2, 1, 40001, "auto"),    # 8192, 1, 12 (2)
    (4000, 1, 3, 9001, "fft"),      # 8192, 1, 3 (1): a single segment
]


@pytest.mark.parametrize("case", CASES, ids=["_".join(map(str, c)) for c in CASES])
def test_short_signal(oracle_mod, case):
    import torch

    n_x, n_pos, n_mic, n_rir, method = case
    rng = np.random.default_rng(zlib.crc32(repr(case).encode()))
    x = rng.standard_normal(n_x).astype(np.float32)
    rirs = (rng.standard_normal((n_pos, n_mic, n_rir)) * np.exp(-3.0 * np.arange(n_rir) / n_rir)).astype(np.float32)
    xd, rd = torch.from_numpy(x).cuda(), torch.from_numpy(rirs).cuda()
    need = ism.filter_workspace_size(n_x, n_pos, n_mic, n_rir, method)
    assert need > 0
    print(f"[case] short signal {case}", flush=True)
    sys.stdout.flush()
    ws = torch.full((need + 4096,), 255, dtype=torch.uint8, device="cuda")  # NaN
    y = ism.filter_trajectory(xd, rd, method=method, ws=ws)
    torch.cuda.synchronize()
    assert bool((ws[need:] == 255).all())
    assert torch.equal(y, ism.filter_trajectory(xd, rd, method=method, ws=ws))
    got, ref = y.cpu().numpy().astype(np.float64), oracle_mod.filter_trajectory(x, rirs)
    err = np.linalg.norm(got - ref, axis=1) / np.linalg.norm(ref, axis=1)
    print(case, "rel err", err.max())
    assert err.max() <= 1e-6
