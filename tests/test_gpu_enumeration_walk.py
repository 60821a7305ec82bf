"""The enumeration check at the seams of the walk that four waves share: lattices whose
columns (x and y indices together) number just around multiples of a wave's 64 lanes, of the
four waves and of their 256 lanes, and around a block of 64 x indices, in tiles that reach
every column. A column that two waves take, or none, shows as an image owned twice or
missing. The one-wave walk of the FP16 items, and the items of table taps, run the same
lattices; small fixed items cut the x range between workgroups as well."""
import functools
import sys

import numpy as np
import pytest

from paper_1810_11359_amd import ism

from .test_gpu_enumeration import check_enumeration

pytestmark = pytest.mark.gpu

# images per axis, x and y: columns
COLUMNS = [(1, 1), (3, 1), (2, 2), (5, 1), (9, 7), (8, 8), (13, 5), (17, 15), (16, 16), (37, 7), (63, 4), (64, 4),
           (65, 4), (1, 257), (31, 33), (32, 32), (41, 25), (129, 3)]
LONGEST = 2.4  # metres: the z axis, the shortest, is the innermost of the walk


def _room(nx, ny, nz):
    L = [LONGEST, 2.3, 2.0]
    far = np.sqrt(sum(((n / 2 + 1) * a) ** 2 for n, a in zip((nx, ny, nz), L)))
    t_max = np.ceil(far / 343.0 * 16000.0 + 40) / 16000.0  # every image inside
    return ism.Room(L, [0.99, 0.98, 0.97, 0.99, 0.98, 0.97], (nx, ny, nz), 343.0, 16000.0, t_max, 0.004)


@pytest.mark.parametrize("precision", ["fp32", "lut", "fp16"])
@pytest.mark.parametrize("nx,ny", COLUMNS, ids=[f"{a}x{b}" for a, b in COLUMNS])
def test_column_counts(oracle_mod, monkeypatch, nx, ny, precision):
    monkeypatch.setattr(ism, "debug_enumerate", functools.partial(ism.debug_enumerate, precision=precision))
    src = np.array([[1.1, 0.9, 0.7]], dtype=np.float32)
    rcv = np.array([[0.4, 1.7, 1.3], [2.1, 0.3, 0.9]], dtype=np.float32)
    for nz in (1, 6):
        room = _room(nx, ny, nz)
        args = (np.array(room.room), np.array(room.beta), room.n_img, room.c, room.fs, room.t_max, room.t_w)
        for sched in (None, ism.Schedule(item_taps=1e9), ism.Schedule(item_taps=1e3)):
            print(f"[case] walk {nx}x{ny}x{nz} {precision} {sched}", flush=True)
            sys.stdout.flush()
            n, _ = check_enumeration(oracle_mod, room, args, src, rcv, sched)
            assert n == 2 * nx * ny * nz


@pytest.mark.parametrize("precision", ["fp16", "lut"])
def test_other_precisions_on_a_room(oracle_mod, monkeypatch, precision):
    """The signed-beta room of the FP32 check."""
    monkeypatch.setattr(ism, "debug_enumerate", functools.partial(ism.debug_enumerate, precision=precision))
    L, beta, n_img = [3.3, 2.7, 2.9], [0.9, -0.7, 0.8, 0.6, -0.95, 0.5], (21, 19, 23)
    room = ism.Room(L, beta, n_img, 343.0, 16000.0, 0.12, 0.004)
    args = (np.array(L), np.array(beta), n_img, 343.0, 16000.0, 0.12, 0.004)
    src = np.array([[1.0, 1.1, 1.2]], dtype=np.float32)
    rcv = np.array([[2.6, 0.5, 2.1], [0.4, 2.2, 0.3]], dtype=np.float32)
    check_enumeration(oracle_mod, room, args, src, rcv, ism.Schedule(item_taps=5000.0))
