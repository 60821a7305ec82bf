"""FP32 taps by moments and table taps by pulses (ism_simulate) where their paths
meet, against the FP64 oracle: windows around the limits of the directly summed and the edge taps, a
room whose images coincide in delay (long lists), items smaller and larger than
the image pool, and RIR lengths around the tile."""
import sys

import numpy as np
import pytest

from paper_1810_11359_amd import ism

pytestmark = pytest.mark.gpu

# An image's taps are within 1e-7 of its amplitude of Eq. (6) (polynomial fit and
# rounded coefficients), its amplitude within 3e-7; sums of FP32 values add a
# few ulp (6e-8) of the largest partial sum, which the peak bounds in these short
# RIRs: 2e-6 of the peak leaves a factor of four.
TOL = 2e-6

# name, fs, W, T_max [s], room, centred, item_taps
CASES = [
    ("w_3.2_direct", 16000.0, 3.2, 0.05, [3.0, 4.0, 2.5], False, 0.0),
    ("w_3.99_direct", 16000.0, 3.99, 0.05, [3.0, 4.0, 2.5], False, 0.0),
    ("w_4_moments", 16000.0, 4.0, 0.05, [3.0, 4.0, 2.5], False, 0.0),
    ("w_5_edge", 16000.0, 5.0, 0.05, [3.0, 4.0, 2.5], False, 0.0),
    ("w_31.9_edge", 16000.0, 31.9, 0.05, [3.0, 4.0, 2.5], False, 0.0),
    ("w_33_edge", 16000.0, 33.0, 0.05, [3.0, 4.0, 2.5], False, 0.0),
    ("w_63.9_edge", 16000.0, 63.9, 0.05, [3.0, 4.0, 2.5], False, 0.0),
    ("w_64.1", 16000.0, 64.1, 0.05, [3.0, 4.0, 2.5], False, 0.0),
    ("w_255.5", 16000.0, 255.5, 0.05, [3.0, 4.0, 2.5], False, 0.0),
    ("cube_coincident", 16000.0, 64.0, 0.12, [2.0, 2.0, 2.0], True, 0.0),
    ("pool_refilled", 16000.0, 64.0, 0.2, [2.1, 2.3, 1.9], False, 1e9),
    ("small_items", 16000.0, 64.0, 0.2, [2.1, 2.3, 1.9], False, 1e4),
    ("one_sample", 16000.0, 64.0, 1.0 / 16000.0, [3.0, 4.0, 2.5], False, 0.0),
    ("tile_less_one", 16000.0, 64.0, 255.0 / 16000.0, [3.0, 4.0, 2.5], False, 0.0),
    ("tile_plus_one", 16000.0, 64.0, 257.0 / 16000.0, [3.0, 4.0, 2.5], False, 0.0),
    # few images per tile: tiles of 512 samples (a given item size takes them on small calls too)
    ("long_w_32", 16000.0, 32.0, 0.06, [9.0, 8.0, 7.0], False, 1e9),
    ("long_w_64_split", 16000.0, 64.0, 0.12, [9.0, 8.0, 7.0], False, 1e3),
    ("long_w_128", 16000.0, 128.0, 513.0 / 16000.0, [9.0, 8.0, 7.0], False, 1e9),
    ("long_w_33_edge", 16000.0, 33.0, 511.0 / 16000.0, [9.0, 8.0, 7.0], False, 1e9),
    ("long_w_3.2_direct", 16000.0, 3.2, 0.06, [9.0, 8.0, 7.0], False, 1e9),
    ("long_w_176.4_two_passes", 44100.0, 176.4, 0.03, [9.0, 8.0, 7.0], False, 1e9),
]


# Table taps: entries and weights are rounded to FP32 (an entry moves by 6e-8, the
# weight of a slope of at most 0.1 per entry by 16 x 6e-8): the same bound.
LUT_CASES = [(f"lut_{c[0]}",) + c[1:] for c in CASES if c[2] == 64.0] + [
    ("lut_w_32", 8000.0, 32.0, 0.1, [3.0, 4.0, 2.5], False, 0.0),
    ("lut_w_96", 48000.0, 96.0, 0.02, [3.0, 4.0, 2.5], False, 0.0),
    ("lut_w_128", 32000.0, 128.0, 0.04, [3.0, 4.0, 2.5], False, 1e9),
]


@pytest.mark.parametrize("case", CASES + LUT_CASES, ids=[c[0] for c in CASES + LUT_CASES])
def test_moments_match_oracle(oracle_mod, case):
    import torch

    name, fs, W, t_max, L, centred, item_taps = case
    prec, lut_q = ("lut", 16) if name.startswith("lut") else ("fp32", 0)
    n = ism.n_img_for_time(L, 343.0, t_max + W / fs)
    room = ism.Room(L, [0.9, 0.85, 0.8, 0.9, 0.7, 0.95], n, 343.0, fs, t_max, W / fs)
    if centred:
        src = np.array([[1.0, 1.0, 1.0]], dtype=np.float32)
        rcv = np.array([[1.0, 1.0, 0.5], [0.5, 1.0, 1.0]], dtype=np.float32)
    else:
        rng = np.random.default_rng(len(name))
        src = rng.uniform(0.3, np.array(L) - 0.3, (1, 3)).astype(np.float32)
        rcv = rng.uniform(0.3, np.array(L) - 0.3, (2, 3)).astype(np.float32)
    print(f"[case] moments {name}: n_img {n}", flush=True)
    sys.stdout.flush()
    sched = ism.Schedule(item_taps=item_taps) if item_taps else None
    h = ism.simulate(room, src, rcv, prec, schedule=sched)
    torch.cuda.synchronize()
    got = h.cpu().numpy().astype(np.float64)
    # lists are joined in a fixed order: the same bits again
    assert torch.equal(h.cpu(), ism.simulate(room, src, rcv, prec, schedule=sched).cpu())
    ref = oracle_mod.rir(room.room, room.beta, room.n_img, room.c, room.fs, room.t_max, room.t_w, src, rcv,
                         lut_q=lut_q)
    peak = np.max(np.abs(oracle_mod.rir(room.room, room.beta, room.n_img, room.c, room.fs, max(t_max, 0.02),
                                        room.t_w, src, rcv)), axis=-1)
    err = float(np.max(np.max(np.abs(got - ref), axis=-1) / peak))
    print(f"moments {name}: max err / peak {err:.2e}", flush=True)
    assert err <= TOL
