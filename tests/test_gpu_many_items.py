"""Calls of more work items than one launch holds: 2048 sources to 2048 receivers (the most
pairs of a call) with RIRs of five output tiles, 21 million items of 256 threads, where a
launch takes 16.7 million. The items are dispatched last tile first, so the first tile,
which holds the direct sound, falls to the second launch.

Every output has to be written (the buffer is filled with NaN first); sampled pairs are
compared with the oracle within 1e-5 of their peak (FP32 taps) or with its table taps."""
import sys

import numpy as np
import pytest

from paper_1810_11359_amd import ism

pytestmark = pytest.mark.gpu

CASES = [
    # precision, samples per RIR: five tiles of 512 samples (few images) or of 256 (table taps)
    ("fp32", 2040),
    ("lut", 1016),
]


@pytest.mark.parametrize("precision,n_samples", CASES, ids=[c[0] for c in CASES])
def test_more_items_than_a_launch(oracle_mod, precision, n_samples):
    import torch

    fs, t_w, L, n = 8000.0, 0.004, [6.0, 7.0, 3.0], 2048
    room = ism.Room(L, [0.9] * 6, (1, 1, 1), 343.0, fs, n_samples / fs, t_w)
    assert room.n_samples == n_samples
    rng = np.random.default_rng(21)
    src = rng.uniform(0.3, np.array(L) - 0.3, (n, 3)).astype(np.float32)
    rcv = rng.uniform(0.3, np.array(L) - 0.3, (n, 3)).astype(np.float32)
    tile = 512 if precision == "fp32" else 256
    items = n * n * -(-(n_samples + 16 - 1) // tile)
    assert n * n == ism.ISM_MAX_PAIRS and items * 256 >= 1 << 32
    print(f"[case] {precision}: {items} items", flush=True)
    sys.stdout.flush()
    sim = ism.Simulator(room, src, rcv, precision)
    sim.out.fill_(float("nan"))
    h = sim.run()
    torch.cuda.synchronize()
    for i in range(0, n, 64):
        assert bool(torch.isfinite(h[i:i + 64]).all()), f"sources {i} ..: samples that were not written"
    picks = [0, 1, 1023, 1024, 2046, 2047]
    got = h[picks][:, picks].cpu().numpy().astype(np.float64)
    del h, sim
    torch.cuda.empty_cache()
    ref = oracle_mod.rir(room.room, room.beta, room.n_img, room.c, room.fs, room.t_max, room.t_w, src[picks],
                         rcv[picks], lut_q=16 if precision == "lut" else 0)
    err = np.max(np.abs(got - ref), axis=-1) / np.max(np.abs(ref), axis=-1)
    print(f"{precision}: max err / peak {err.max():.2e}", flush=True)
    assert err.max() <= 1e-5
