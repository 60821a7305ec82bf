"""The diffuse tail at the edges of its launch: rows that start off the 16-byte grid, an
ISM part that ends inside a thread's four samples, several segments per block with a
partial last block. The tail is formed again in FP64 from the call's own ISM part.

Tolerance, of the tail's envelope: the two FP32 logarithms of up to 32 differ by at most
an ulp each (2 * 1.9e-6, times the scale of 0.38), the envelope, the level (a sum of FP32
squares) and their products by 16 roundings (1e-6) of a variate of at most 12.4: 1.4e-5
together, 2e-5."""
import sys

import numpy as np
import pytest

from paper_1810_11359_amd import ism

pytestmark = pytest.mark.gpu

TOL = 2e-5

CASES = [
    # name, n_rcv, t_diff, t_max (at 16 kHz): ISM samples, samples
    ("aligned", 3, 0.06, 0.128),          # 960, 2048: whole segments
    ("ragged_rows", 5, 0.0600625, 0.1500625),  # 961, 2401: rows at every alignment
    ("all_but_two", 2, 0.0999375, 0.1000625),  # 1599, 1601
    ("segments", 330, 0.0300625, 0.8),    # 481, 12800: 13 segments of 1024, two per block
    ("segments_ragged", 700, 0.03025, 0.8003125),  # 484, 12805: four per block
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_tail(oracle_mod, case):
    import torch

    name, n_rcv, t_diff, t_max = case
    L, t60, fs, seed = [3.0, 4.0, 2.5], 0.7, 16000.0, 77
    room = ism.Room(L, list(ism.beta_from_t60(L, t60)), ism.n_img_for_time(L, 343.0, t_diff), 343.0, fs, t_max, 0.004)
    rng = np.random.default_rng(n_rcv)
    src = [[1.0, 1.5, 1.2]]
    rcv = rng.uniform(0.4, 0.6, (n_rcv, 3)) * L + [0.3, 0.3, 0.1]
    print(f"[case] {name} nS={room.n_samples}", flush=True)
    sys.stdout.flush()
    got = ism.simulate_diffuse(room, src, rcv, t_diff, t60, seed)[0].cpu().numpy().astype(np.float64)
    torch.cuda.synchronize()
    part = ism.simulate(ism.Room(L, room.beta, room.n_img, 343.0, fs, t_diff, 0.004), src, rcv)[0].cpu().numpy()
    k_diff = oracle_mod.n_samples(t_diff, fs)
    assert np.array_equal(got[:, :k_diff], part.astype(np.float64))
    k = np.arange(k_diff, got.shape[1])
    scale = np.sqrt(oracle_mod.envelope_level(got[:, :k_diff], fs, t_diff, t60)[:, None] *
                    oracle_mod.envelope(k, fs, t_diff, t60))
    worst = 0.0
    for i in range(0, n_rcv, max(1, n_rcv // 40)):
        noise = oracle_mod.logistic_from_bits(oracle_mod.noise_bits(seed, i, k))
        worst = max(worst, np.max(np.abs(got[i, k_diff:] - noise * scale[i]) / scale[i]))
    print(name, "tail err / envelope", worst)
    assert worst <= TOL
