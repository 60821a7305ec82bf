"""Calls of few images per tile, whose FP32 and table taps run on one-wave items, image by
image: every window cap (exact, cut taps, windows shorter than four samples), directional
receivers, tiles of no, one and some hundred images, against the FP64 oracle, against the
same pairs in a launch small enough for moments, and in batches.

Tolerance: as for moments (taps within 1e-7 of an image's amplitude, the amplitude within
3e-7, sums of FP32 values in short RIRs): 2e-6 of the peak."""
import sys

import numpy as np
import pytest

from paper_1810_11359_amd import ism

pytestmark = pytest.mark.gpu

TOL = 2e-6

WINDOWS = [32.0, 64.0, 96.0, 128.0, 3.2, 3.99, 4.0, 5.925, 13.95, 31.9, 33.0, 40.0, 63.9, 64.9, 88.2, 100.0, 150.0,
           176.4, 201.0, 244.5, 255.5]
EXACT = (32.0, 64.0, 96.0, 128.0)


def _say(msg):
    print(f"[case] {msg}", flush=True)
    sys.stdout.flush()


def _err(oracle_mod, room, src, rcv, got, lut_q=0):
    ref = oracle_mod.rir(room.room, room.beta, room.n_img, room.c, room.fs, room.t_max, room.t_w, src, rcv,
                         lut_q=lut_q)
    return float(np.max(np.max(np.abs(got - ref), axis=-1) / np.max(np.abs(ref), axis=-1)))


@pytest.mark.parametrize("n", [1, 3])
@pytest.mark.parametrize("W", WINDOWS)
def test_small_lattices(oracle_mod, W, n):
    """The direct path alone and with first reflections, tiles beyond the last image."""
    import torch

    L, fs = [5.0, 4.0, 3.0], 16000.0
    room = ism.Room(L, [0.9, -0.85, 0.8, 0.9, 0.7, 0.95], (n, n, n), 343.0, fs, 900.0 / fs, W / fs)
    rng = np.random.default_rng(int(10 * W))
    src = rng.uniform(0.3, np.array(L) - 0.3, (2, 3)).astype(np.float32)
    rcv = rng.uniform(0.3, np.array(L) - 0.3, (40, 3)).astype(np.float32)
    for prec, lut_q in (("fp32", 0), ("lut", 16)) if W in EXACT else (("fp32", 0),):
        _say(f"few W={W:g} n={n} {prec}")
        h = ism.simulate(room, src, rcv, prec)
        fine = ism.simulate(room, src, rcv, prec, schedule=ism.Schedule(item_taps=1e3))
        torch.cuda.synchronize()
        assert torch.equal(h, ism.simulate(room, src, rcv, prec))
        for x in (h, fine):
            e = _err(oracle_mod, room, src, rcv, x.cpu().numpy().astype(np.float64), lut_q)
            print(f"W={W:g} n={n} {prec}: {e:.2e}", flush=True)
            assert e <= TOL


@pytest.mark.parametrize("W", [32.0, 64.0, 96.0, 128.0, 33.0, 176.4])
def test_some_hundred_images_per_tile(oracle_mod, W):
    """512 RIRs of 2000 samples, about 150 images per tile: one-wave items (several chunks of
    candidates and a carried rest per item); four of the pairs alone take moments."""
    import torch

    L, fs = [4.6, 3.9, 3.3], 16000.0
    k = 2000.0
    room = ism.Room(L, [0.9, 0.85, 0.8, 0.9, 0.7, 0.95], ism.n_img_for_time(L, 343.0, (k + W) / fs), 343.0, fs, k / fs,
                    W / fs)
    rng = np.random.default_rng(int(W))
    src = rng.uniform(0.3, np.array(L) - 0.3, (1, 3)).astype(np.float32)
    rcv = rng.uniform(0.3, np.array(L) - 0.3, (2048, 3)).astype(np.float32)
    # (thinned to the rule's range by the room's size)
    room.room[0] *= 4.0
    room.n_img = tuple(ism.n_img_for_time(room.room, 343.0, (k + W) / fs))
    for prec, lut_q in (("fp32", 0), ("lut", 16)) if W in EXACT else (("fp32", 0),):
        _say(f"hundreds W={W:g} {prec}")
        h = ism.simulate(room, src, rcv, prec)[0]
        few = [0, 1, 1000, 2047]
        alone = ism.simulate(room, src, rcv[few], prec)[0]
        torch.cuda.synchronize()
        got = h[few].cpu().numpy().astype(np.float64)
        peak = np.max(np.abs(got), axis=-1, keepdims=True)
        assert np.max(np.abs(got - alone.cpu().numpy()) / peak) <= TOL
        e = _err(oracle_mod, room, src, rcv[few], got[None], lut_q)
        print(f"W={W:g} {prec}: {e:.2e}", flush=True)
        assert e <= TOL


@pytest.mark.parametrize("W", [64.0, 5.925, 176.4])
def test_directional(oracle_mod, W):
    import torch

    L, fs = [5.0, 4.0, 3.0], 16000.0
    room = ism.Room(L, [0.9, 0.85, 0.8, 0.9, 0.7, 0.95], (3, 3, 3), 343.0, fs, 600.0 / fs, W / fs)
    rng = np.random.default_rng(3)
    src = rng.uniform(0.3, np.array(L) - 0.3, (1, 3)).astype(np.float32)
    rcv = rng.uniform(0.3, np.array(L) - 0.3, (9, 3)).astype(np.float32)
    o = rng.standard_normal(rcv.shape).astype(np.float32)
    _say(f"few directional W={W:g}")
    got = ism.simulate_polar(room, src, rcv, o, "cardioid")
    omni = ism.simulate_polar(room, src, rcv, o, "omni")
    plain = ism.simulate(room, src, rcv)
    torch.cuda.synchronize()
    assert torch.equal(omni, plain)
    ref = oracle_mod.rir_polar(room.room, room.beta, room.n_img, room.c, room.fs, room.t_max, room.t_w, src, rcv, o,
                               0.5)
    omni_peak = np.max(np.abs(plain.cpu().numpy()), axis=-1)
    assert np.all(np.max(np.abs(got.cpu().numpy() - ref), axis=-1) <= TOL * omni_peak)


@pytest.mark.parametrize("precision", ["fp32", "lut"])
def test_batches_of_both_kinds(precision):
    """Jobs of few and of many images in one batch (and 60 small jobs that only together fill
    the chip): each job is its single call with a shared item size, bit for bit, and the
    default plan's within rounding."""
    import torch

    rng = np.random.default_rng(8)
    jobs = []
    for i in range(64):
        L = [4.0 + 0.05 * i, 5.0, 3.0]
        many = i >= 60
        t = 0.12 if many else 0.05
        n = ism.n_img_for_time(L, 343.0, t) if many else (5, 5, 5)
        fs, t_w = (8000.0, 0.004) if i % 3 == 0 else (16000.0, 0.004)
        room = ism.Room(L, [0.9, 0.85, 0.8, 0.9, 0.7, 0.95], n, 343.0, fs, t, t_w)
        jobs.append((room, rng.uniform(0.3, np.array(L) - 0.3, (1, 3)).astype(np.float32),
                     rng.uniform(0.3, np.array(L) - 0.3, (12, 3)).astype(np.float32)))
    _say(f"batch of both kinds {precision}")
    sched = ism.Schedule(item_taps=40000.0)
    outs = [o.clone() for o in ism.BatchSimulator(jobs, precision=precision).run()]
    shared = [o.clone() for o in ism.BatchSimulator(jobs, precision=precision, schedule=sched).run()]
    torch.cuda.synchronize()
    for i, ((room, src, rcv), o, sh) in enumerate(zip(jobs, outs, shared)):
        assert torch.equal(sh, ism.simulate(room, src, rcv, precision, schedule=sched)), i
        single = ism.simulate(room, src, rcv, precision)
        peak = torch.amax(torch.abs(single), dim=-1, keepdim=True)
        assert float((torch.abs(o - single) / peak).max()) <= 1e-6, i
        if i % 9 == 0:
            alone = ism.BatchSimulator([(room, src, rcv)], precision=precision).run()[0]
            untapered = ism.simulate(room, src, rcv, precision, schedule=ism.Schedule(tail_rounds=0.0))
            assert torch.equal(alone, untapered), i


@pytest.mark.parametrize("per_tile", [10, 60, 200])
@pytest.mark.parametrize("n_jobs,n_rcv", [(2, 1), (20, 16), (70, 16)])
@pytest.mark.parametrize("precision", ["fp32", "lut"])
def test_batch_on_either_side_of_its_limits(oracle_mod, precision, n_jobs, n_rcv, per_tile):
    """Batches of 8, 1280 and 4480 tiles of few and of some more images: within rounding of
    the single calls (1e-6 of the peak), one pair of each fourth job against the oracle."""
    import torch

    rng = np.random.default_rng(n_jobs + per_tile)
    jobs = []
    for i in range(n_jobs):
        k, fs = 900.0, 16000.0
        side = (4 / 3 * np.pi * (k + 32) ** 3 / (4 * per_tile)) ** (1 / 3) * 343.0 / fs
        L = [side * 1.1, side, side / 1.1]
        room = ism.Room(L, [0.9, 0.85, 0.8, 0.9, 0.7, 0.95], ism.n_img_for_time(L, 343.0, (k + 32) / fs), 343.0, fs,
                        k / fs, 0.004)
        src = rng.uniform(0.4 * side, 0.6 * side, (1, 3)).astype(np.float32)
        jobs.append((room, src, (src + rng.uniform(-0.2, 0.2, (n_rcv, 3)) * side).astype(np.float32)))
    _say(f"batch limits {precision} {n_jobs} x {n_rcv}, {per_tile}")
    outs = [o.clone() for o in ism.BatchSimulator(jobs, precision=precision).run()]
    torch.cuda.synchronize()
    for i, ((room, src, rcv), o) in enumerate(zip(jobs, outs)):
        single = ism.simulate(room, src, rcv, precision)
        peak = torch.amax(torch.abs(single), dim=-1, keepdim=True)
        assert float((torch.abs(o - single) / peak).max()) <= 1e-6, i
        if i % 4 == 0:
            e = _err(oracle_mod, room, src, rcv[:1], o[:, :1].cpu().numpy().astype(np.float64),
                     16 if precision == "lut" else 0)
            assert e <= TOL, i
