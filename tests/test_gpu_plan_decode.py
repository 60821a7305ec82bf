"""Work items and reduce launches of single calls against the FP64 oracle at the edges of
the plan's tables: one block of 16 dispatch positions, one more, more blocks than lanes;
tiles in one item (plain reduce), in up to eight and more (gather), in 64 and more (sliced).

Tolerance, of the RIR's peak: as for the FP32 taps elsewhere, 2e-6 (amplitudes and moments
of FP32 accuracy, 1.2e-7 each, added over at most 16 images of like size per sample)."""
import sys

import numpy as np
import pytest

from paper_1810_11359_amd import ism

pytestmark = pytest.mark.gpu

TOL = 2e-6

CASES = [
    # name, samples, fs, n_img, item_taps
    ("one_tile", 200, 16000.0, (6, 6, 6), 0.0),
    ("block_of_positions", 4000, 16000.0, (12, 2, 2), 0.0),
    ("one_position_more", 4200, 16000.0, (34, 4, 4), 0.0),
    ("65_blocks", 262144, 96000.0, (602, 2, 2), 0.0),
    ("up_to_8_items", 4000, 16000.0, (60, 46, 70), 2.0e5),
    ("more_than_8_items", 4000, 16000.0, (60, 46, 70), 5.0e4),
    ("more_than_64_items", 4000, 16000.0, (60, 46, 70), 1.0e4),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_plan_edges(oracle_mod, case):
    import torch

    name, n, fs, n_img, item_taps = case
    room = ism.Room([3.0, 4.0, 2.5], [0.97, 0.98, 0.9, 0.92, 0.85, 0.95], n_img, 343.0, fs, n / fs, 64 / fs)
    src = np.array([[1.1, 1.3, 0.9]], dtype=np.float32)
    rcv = np.array([[2.0, 2.9, 1.6], [0.6, 3.1, 1.2], [2.4, 0.7, 1.9]], dtype=np.float32)
    print(f"[case] plan {name}", flush=True)
    sys.stdout.flush()
    h = ism.simulate(room, src, rcv, schedule=ism.Schedule(item_taps=item_taps) if item_taps else None)
    torch.cuda.synchronize()
    got = h.cpu().numpy().astype(np.float64)
    ref = oracle_mod.rir(room.room, room.beta, room.n_img, room.c, room.fs, room.t_max, room.t_w, src, rcv)
    err = float(np.max(np.max(np.abs(got - ref), axis=-1) / np.max(np.abs(ref), axis=-1)))
    print(f"plan {name}: max err / peak {err:.2e}", flush=True)
    assert err <= TOL
