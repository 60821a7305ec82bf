"""The moving-source filter on fixed blocks against the FP64 oracle. Automatic and FFT calls
prefer segment blocks, so these calls are such that only fixed blocks are left: segments
longer than half the longest transform, or a workspace of exactly the fixed blocks' size
where segment blocks ask for more (up to 16 segments per block). Every block size, ragged
last segments, partial last partitions, blocks across segment boundaries, several
transforms per workgroup with a partial last one.

The workspace is NaN before the call and its surroundings are checked after it. Tolerance,
of the norm of y per microphone: as on segment blocks (three transforms of at most 14
levels and sums of at most 512 terms, twice 3.6e-7 and the inputs' rounding), 1e-6."""
import ctypes
import sys
import zlib

import numpy as np
import pytest

from paper_1810_11359_amd import ism

pytestmark = pytest.mark.gpu

TOL = 1e-6

# n_x, n_pos, n_mic, n_rir, method: block size, pieces per block, segment
LONG = [
    (27001, 3, 2, 300, "fft"),     # 256, 2, 9001: partial second partition
    (27001, 3, 2, 255, "fft"),     # 256, 2: one partition, shorter than a block
    (8300, 1, 3, 1, "fft"),        # 256, 1: a single tap, a single segment
    (27001, 3, 5, 1500, "auto"),   # 512, 2, 9001
    (40000, 4, 2, 3001, "auto"),   # 1024, 2, 10000
    (18001, 2, 3, 6000, "auto"),   # 2048, 2, 9001
    (27003, 3, 1, 16500, "auto"),  # 4096, 2, 9001: 5 partitions, the last of 116 taps
    (60000, 13, 1, 4000, "auto"),  # 1024, 2, 4616: too few partitions for the longest transform
]
SHORT = [
    (709, 4, 1, 915, "fft"),       # 256, 3
    (526, 9, 2, 434, "fft"),       # 256, 6
    (733, 24, 1, 491, "fft"),      # 256, 10
    (549, 31, 2, 496, "fft"),      # 256, 16
    (1560, 4, 2, 2024, "auto"),    # 512, 3
    (161, 8, 1, 2041, "fft"),      # 512, 8
    (1785, 51, 8, 1448, "fft"),    # 512, 16
    (3113, 7, 2, 2965, "auto"),    # 1024, 4
    (3588, 24, 8, 2438, "fft"),    # 1024, 8
    (3140, 46, 8, 3032, "fft"),    # 1024, 16
    (8896, 20, 1, 8069, "fft"),    # 2048, 6
    (7788, 53, 1, 7637, "fft"),    # 2048, 15
    (116, 4, 1, 24832, "auto"),    # 4096, 4: 7 partitions
    (104, 7, 1, 32771, "fft"),     # 4096, 7: the last partition of 3 taps
    (114, 16, 1, 15548, "fft"),    # 4096, 16
]


def fixed_plan(n_x, n_pos, n_mic, n_rir):
    """Workspace bytes and pieces per block of fixed blocks, from their description in ism.h."""
    n2 = 1
    while n2 < n_rir:
        n2 *= 2
    B = 4096 if n2 >= 16384 else max(256, n2 // 4)
    P, seg = -(-n_rir // B), -(-n_x // n_pos)
    R = min(-(-B // seg) + 1, n_pos)
    n_in, n_out = -(-n_x // B), -(-(n_x + n_rir - 1) // B)
    size = 0
    for part in (8 * n_pos * n_mic * P * B, 8 * n_in * R * B, 8 * n_mic * n_out * B, 8 * n_mic * n_out * B):
        size = (size + part + 255) // 256 * 256
    return size, R


@pytest.mark.parametrize("case", LONG + SHORT, ids=["_".join(map(str, c)) for c in LONG + SHORT])
def test_fixed_blocks(oracle_mod, case):
    import torch

    n_x, n_pos, n_mic, n_rir, method = case
    size, R = fixed_plan(*case[:4])
    need = ism.filter_workspace_size(*case)
    if case in LONG:
        assert need == size
    else:
        assert need > size and R > 2  # segment blocks do not fit: fixed blocks are taken
    rng = np.random.default_rng(zlib.crc32(repr(case).encode()))
    x = rng.standard_normal(n_x).astype(np.float32)
    rirs = (rng.standard_normal((n_pos, n_mic, n_rir)) * np.exp(-3.0 * np.arange(n_rir) / n_rir)).astype(np.float32)
    xd, rd = torch.from_numpy(x).cuda(), torch.from_numpy(rirs).cuda()
    print(f"[case] fixed {case}", flush=True)
    sys.stdout.flush()
    guard, nan = 4096, float("nan")
    buf = torch.full((size // 4 + 2 * guard,), nan, device="cuda")
    st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)

    def run():
        buf.fill_(nan)
        buf[:guard] = 7.0
        buf[-guard:] = 7.0
        y = torch.full((n_mic, n_x + n_rir - 1), nan, device="cuda")
        rc = ism.lib().ism_filter_trajectory_ex(xd.data_ptr(), n_x, rd.data_ptr(), n_pos, n_mic, n_rir,
                                                ism.FILTER_METHODS[method], y.data_ptr(), buf[guard:].data_ptr(),
                                                size, st)
        torch.cuda.synchronize()
        assert rc == ism.ISM_OK
        assert bool((buf[:guard] == 7.0).all()) and bool((buf[-guard:] == 7.0).all())
        return y

    y = run()
    assert torch.equal(y, run())  # fixed summation order
    got, ref = y.cpu().numpy().astype(np.float64), oracle_mod.filter_trajectory(x, rirs)
    err = np.linalg.norm(got - ref, axis=1) / np.linalg.norm(ref, axis=1)
    print(case, "rel err", err.max())
    assert err.max() <= TOL
