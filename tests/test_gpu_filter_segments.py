"""The moving-source filter on segment blocks (one input block per segment) against the
FP64 oracle, at each transform size and at the edges of its grid: single-sample segments,
several transforms and several partition groups per workgroup, ragged ends.

Tolerance, of the norm of y per microphone: an output passes three transforms (segment,
RIR, inverse) of at most 14 radix-2 levels and three steps of sums of at most 512 terms.
Each level and step rounds with an rms of at most 0.6 * 2^-24 of the norm, products
(twiddles, spectra) as much again: sqrt(2 * 3 * 17) * 0.6 * 2^-24 = 3.6e-7. Twice that and
rounding of the inputs to the transforms' constants: 1e-6."""
import ctypes
import sys
import zlib

import numpy as np
import pytest

from paper_1810_11359_amd import ism

pytestmark = pytest.mark.gpu

TOL = 1e-6

CASES = [
    # name, n_x, n_pos, n_mic, n_rir (transform size, segments per partition, partitions)
    ("one_sample", 700, 700, 1, 2048),          # 512, 512, 4 in 2 groups of 2
    ("two_samples", 600, 300, 1, 2048),         # 512, 255, 5 in 5 groups
    ("three_samples_ragged", 3001, 1500, 1, 2100),  # 512, 170, 5: unused trailing points
    ("short_many_mics", 2000, 70, 40, 2050),    # 512, 16, 5 in one group
    ("points_1024", 20000, 40, 2, 2200),        # 1024, 1, 5
    ("points_1024_four", 20001, 100, 1, 2048),  # 1024, 4, 3: last segment shorter
    ("points_2048", 30000, 64, 32, 6001),       # 2048, 3, 5 in one group
    ("points_4096", 30000, 20, 3, 4100),        # 4096, 1, 3
    ("one_partition", 20000, 13, 2, 1100),      # 4096, 1, 1: RIR shorter than a segment
    ("points_8192", 40000, 10, 64, 2500),       # 8192, 1, 1
    ("points_16384", 64000, 8, 9, 9001),        # 16384, 1, 2
]


def signals(name, n_x, n_pos, n_mic, n_rir):
    rng = np.random.default_rng(zlib.crc32(name.encode()))
    x = rng.standard_normal(n_x).astype(np.float32)
    rirs = (rng.standard_normal((n_pos, n_mic, n_rir)) * np.exp(-3.0 * np.arange(n_rir) / n_rir)).astype(np.float32)
    return x, rirs


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_segment_blocks(oracle_mod, case):
    import torch

    name, n_x, n_pos, n_mic, n_rir = case
    assert ism.filter_workspace_size(n_x, n_pos, n_mic, n_rir, "auto") > 0  # a transform plan
    x, rirs = signals(*case)
    print(f"[case] {name}", flush=True)
    sys.stdout.flush()
    xd, rd = torch.from_numpy(x).cuda(), torch.from_numpy(rirs).cuda()
    y = ism.filter_trajectory(xd, rd)
    y2 = ism.filter_trajectory(xd, rd)
    torch.cuda.synchronize()
    assert torch.equal(y, y2)  # fixed summation order
    got, ref = y.cpu().numpy().astype(np.float64), oracle_mod.filter_trajectory(x, rirs)
    err = np.linalg.norm(got - ref, axis=1) / np.linalg.norm(ref, axis=1)
    print(name, "rel err", err.max())
    assert err.max() <= TOL


def test_auto_without_workspace_is_the_direct_sum():
    """Segments too short for fixed blocks: auto takes the direct sum where the caller
    brings no workspace or too small a one, as a call that needs none may."""
    import torch

    case = ("no_workspace", 3000, 60, 2, 2100)
    x, rirs = signals(*case)
    xd, rd = torch.from_numpy(x).cuda(), torch.from_numpy(rirs).cuda()
    _, n_x, n_pos, n_mic, n_rir = case
    need = ism.filter_workspace_size(n_x, n_pos, n_mic, n_rir, "auto")
    assert need > 0
    direct = ism.filter_trajectory(xd, rd, method="direct")
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    for p, n in ((None, 0), (ws.data_ptr(), need - 1)):
        y = torch.full_like(direct, 7.0)
        rc = ism.lib().ism_filter_trajectory_ex(xd.data_ptr(), n_x, rd.data_ptr(), n_pos, n_mic, n_rir,
                                                ism.FILTER_METHODS["auto"], y.data_ptr(), p, n, st)
        torch.cuda.synchronize()
        assert rc == ism.ISM_OK
        assert torch.equal(y, direct)


def test_fft_without_workspace_is_refused():
    import torch

    x, rirs = signals("refused", 20000, 13, 2, 1100)
    xd, rd = torch.from_numpy(x).cuda(), torch.from_numpy(rirs).cuda()
    y = torch.empty((2, 20000 + 1100 - 1), device="cuda")
    for method in ("auto", "fft"):
        rc = ism.lib().ism_filter_trajectory_ex(xd.data_ptr(), 20000, rd.data_ptr(), 13, 2, 1100,
                                                ism.FILTER_METHODS[method], y.data_ptr(), None, 0, None)
        assert rc == ism.ISM_E_WORKSPACE
