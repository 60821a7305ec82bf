"""Timed cases of the Image Source Method library, one pass each through its Python entry points.

The listed cases are the work that a program has the library do: the smallest
call (one RIR of a small room), a microphone set in one room, a long 48 kHz
room, the prepared batch of many rooms, serving batches planned on each call,
directional receivers with a general window, the diffuse model, the table and
FP16 taps, and the moving-source filter with short and long RIRs. ``draw``
gives further cases of the same kinds and ranges.

A case's rooms and reverberation times follow from the case alone, positions,
wall jitter, orientations and signals from the seed.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1810_11359_amd import ism

C_SOUND = 343.0
LUT_Q = 16  # table points per sample of the "lut" taps


# ---------------------------------------------------------------------------
# Cases
# ---------------------------------------------------------------------------
def _single(name, call, lx, ly, lz, t60, n_src, n_rcv, fs=16000.0, t_w=0.004, precision="fp32", **more):
    c = dict(name=name, kind="room", call=call, lx=lx, ly=ly, lz=lz, t60=t60, n_src=n_src, n_rcv=n_rcv, fs=fs,
             t_w=t_w, precision=precision)
    c.update(more)
    return c


def listed():
    return [
        # the smallest call: one source, one microphone, a short RIR (latency and launches)
        _single("single_rir", "simulator", 3.0, 4.0, 2.5, 0.3, 1, 1),
        # one call of the problem statement with positions from host memory, checked and copied on each call
        _single("host_call_4rcv", "host", 3.0, 4.0, 2.5, 0.7, 1, 4),
        # an ordinary call: one room, 32 microphones, 16 kHz
        _single("room_32rcv", "simulator", 4.0, 5.0, 3.0, 0.7, 1, 32),
        # the same room with table taps
        _single("room_32rcv_lut", "simulator", 4.0, 5.0, 3.0, 0.7, 1, 32, precision="lut"),
        # the longest RIRs: a large reverberant room at 48 kHz, a 64-microphone circular array
        _single("uca64_48k", "simulator", 6.0, 9.0, 3.5, 2.0, 1, 64, fs=48000.0, t_w=0.002, uca=True),
        # directional microphones at 44.1 kHz: a window that is no even number of samples (176.4)
        _single("cardioid_44k1", "polar", 5.0, 6.3, 2.9, 0.45, 1, 6, fs=44100.0, pattern=0.5),
        # the diffuse model: early ISM part, noise tail, many receivers
        _single("diffuse_1024rcv", "diffuse", 3.0, 4.0, 2.5, 0.7, 1, 1024, att_db=13.0),
        # data generation: 1024 independent rooms in one prepared batch, FP32 and (a quarter of them) FP16 taps
        dict(name="batch_1024_rooms", kind="batch", call="prepared", n_rooms=1024, t60_lo=0.2, t60_hi=1.0,
             max_rcv=8, mixed=False, precision="fp32"),
        dict(name="batch_256_rooms_fp16", kind="batch", call="prepared", n_rooms=256, t60_lo=0.2, t60_hi=1.0,
             max_rcv=8, mixed=False, precision="fp16"),
        # serving: a batch of waiting jobs at 16 and 48 kHz with host positions, planned on each call
        dict(name="serving_12_jobs", kind="batch", call="host", n_rooms=12, t60_lo=0.1, t60_hi=1.5, max_rcv=64,
             mixed=True, precision="fp32"),
        # a 10 s signal at 16 kHz along 100 points to 8 microphones, 0.5 s RIRs
        dict(name="moving_16k", kind="filter", n_x=160000, n_pos=100, n_mic=8, n_rir=8000, fs=16000.0),
        # the same at 48 kHz with 2 s RIRs: the largest filter
        dict(name="moving_48k", kind="filter", n_x=480000, n_pos=100, n_mic=8, n_rir=96000, fs=48000.0),
    ]


def _log(rng, lo, hi):
    return lo * (hi / lo) ** rng.random()


def draw(rng):
    what = rng.choice(["room", "room", "room", "batch", "filter"])
    if what == "batch":
        if rng.random() < 0.5:
            return dict(kind="batch", call="prepared", n_rooms=int(_log(rng, 4, 1000)), t60_lo=0.2, t60_hi=1.0,
                        max_rcv=8, mixed=False, precision=rng.choice(["fp32", "fp32", "fp16"]))
        return dict(kind="batch", call="host", n_rooms=int(_log(rng, 1, 16)), t60_lo=0.1, t60_hi=1.5, max_rcv=64,
                    mixed=True, precision="fp32")
    if what == "filter":
        fs, n_mic = rng.choice([16000.0, 48000.0]), rng.randint(1, 8)
        return dict(kind="filter", n_x=int(_log(rng, 5000, 10 * fs)), n_pos=rng.randint(1, 100), n_mic=n_mic,
                    n_rir=int(_log(rng, 200, 2 * fs)), fs=fs)
    fs, t_w = rng.choice([(16000.0, 0.004), (16000.0, 0.004), (48000.0, 0.002), (44100.0, 0.004), (32000.0, 0.004),
                          (8000.0, 0.004)])
    call = rng.choice(["simulator", "simulator", "host", "polar", "diffuse"])
    even = fs != 44100.0
    c = dict(kind="room", call=call, lx=round(rng.uniform(3.0, 10.0), 2), ly=round(rng.uniform(3.0, 10.0), 2),
             lz=round(rng.uniform(2.3, 4.0), 2), t60=round(_log(rng, 0.12, 1.1), 3), n_src=rng.choice([1, 1, 1, 2, 3]),
             n_rcv=int(_log(rng, 1, 40)), fs=fs, t_w=t_w,
             precision=rng.choice(["fp32", "fp32", "fp32", "fp16", "lut"] if even else ["fp32"]))
    if call == "polar":
        c["pattern"] = rng.choice([0.0, 0.25, 0.5, 0.75])
    if call == "diffuse":
        c["att_db"] = 13.0
    lo = 0.161 * _volume_over_surface([c["lx"], c["ly"], c["lz"]])
    c["t60"] = max(c["t60"], round(1.3 * lo, 3))  # Sabine's formula needs an absorption of at most 1
    return c


# ---------------------------------------------------------------------------
# Rooms
# ---------------------------------------------------------------------------
def _volume_over_surface(L):
    return L[0] * L[1] * L[2] / (2.0 * (L[0] * L[1] + L[0] * L[2] + L[1] * L[2]))


def _beta(L, t60):
    return math.sqrt(1.0 - 0.161 * _volume_over_surface(L) / t60)


def _n_img(L, t):
    return [4 * math.ceil(C_SOUND * t / (2.0 * a)) + 2 for a in L]


def _n_samples(t, fs):
    v = t * fs
    r = round(v)
    return int(r) if abs(v - r) <= 1e-9 * v else math.ceil(v)


def _positions(rng, L, n, margin=0.5):
    return rng.uniform([margin] * 3, [a - margin for a in L], size=(n, 3)).astype(np.float32)


def _geometry(case):
    """The rooms of a case: [(L, t60, n_src, n_rcv, fs, t_w, t_ism)], from the case alone."""
    if case["kind"] == "room":
        L = [case["lx"], case["ly"], case["lz"]]
        t_ism = case["t60"] * case["att_db"] / 60.0 if case["call"] == "diffuse" else case["t60"]
        return [(L, case["t60"], case["n_src"], case["n_rcv"], case["fs"], case["t_w"], t_ism)]
    g = np.random.default_rng(1000 + case["n_rooms"])
    rooms = []
    for _ in range(case["n_rooms"]):
        L = [float(v) for v in g.uniform(3.0, 10.0, 3)]
        t60 = float(g.uniform(case["t60_lo"], case["t60_hi"]))
        while 0.161 * _volume_over_surface(L) / t60 > 1.0:
            t60 = float(g.uniform(case["t60_lo"], case["t60_hi"]))
        fs, t_w = (48000.0, 0.002) if case["mixed"] and g.random() < 0.5 else (16000.0, 0.004)
        rooms.append((L, t60, 1, int(g.integers(1, case["max_rcv"] + 1)), fs, t_w, t60))
    return rooms


def _inputs(case, seed):
    """Rooms with walls, positions and orientations: [(Room fields, src, rcv, orient)]."""
    rng = np.random.default_rng(seed)
    out = []
    for L, t60, n_src, n_rcv, fs, t_w, t_ism in _geometry(case):
        b = _beta(L, t60)
        beta = [b] * 6 if case["kind"] == "room" else \
            [float(v) for v in np.minimum(b * (1.0 + rng.uniform(-0.1, 0.1, 6)), 0.999)]
        src = _positions(rng, L, n_src)
        if case.get("uca"):
            a = 2.0 * np.pi * np.arange(n_rcv) / n_rcv
            rcv = np.stack([L[0] / 2 + 0.1 * np.cos(a), L[1] / 2 + 0.1 * np.sin(a), np.full(n_rcv, 1.5)],
                           axis=1).astype(np.float32)
        else:
            rcv = _positions(rng, L, n_rcv)
        orient = rng.standard_normal((n_rcv, 3)).astype(np.float32)
        out.append((dict(room=L, beta=beta, n_img=_n_img(L, t_ism), c=C_SOUND, fs=fs, t_max=t60, t_w=t_w), src, rcv,
                    orient))
    return out


# ---------------------------------------------------------------------------
# Passes
# ---------------------------------------------------------------------------
def prepare(case, seed):
    if case["kind"] == "filter":
        g = torch.Generator(device="cuda").manual_seed(seed)
        n_rir = case["n_rir"]
        x = torch.randn(case["n_x"], generator=g, device="cuda")
        env = torch.exp(-torch.arange(n_rir, device="cuda") * (6.9 / n_rir))  # 60 dB over the RIR
        rirs = torch.randn(case["n_pos"], case["n_mic"], n_rir, generator=g, device="cuda").mul_(env)
        ws = torch.empty(max(ism.filter_workspace_size(case["n_x"], case["n_pos"], case["n_mic"], n_rir), 1),
                         dtype=torch.uint8, device="cuda")
        return dict(kind="filter", x=x, rirs=rirs, ws=ws)
    inputs = [(ism.Room(**r), src, rcv, orient) for r, src, rcv, orient in _inputs(case, seed)]
    call, prec = case["call"], case["precision"]
    if case["kind"] == "room":
        room, src, rcv, orient = inputs[0]
        if call == "simulator":
            return dict(kind="sim", sim=ism.Simulator(room, src, rcv, prec))
        if call == "diffuse":
            t_diff = case["t60"] * case["att_db"] / 60.0
            return dict(kind="sim", sim=ism.DiffuseSimulator(room, src, rcv, t_diff, case["t60"], seed % 1000003,
                                                             prec))
        out = torch.empty((len(src), len(rcv), room.n_samples), dtype=torch.float32, device="cuda")
        return dict(kind=call, room=room, src=src, rcv=rcv, orient=orient, prec=prec, out=out,
                    pattern=case.get("pattern"))
    # batches: the RIRs of all rooms in one device buffer, one view per room
    n = [len(src) * len(rcv) * room.n_samples for room, src, rcv, _ in inputs]
    flat = torch.empty(sum(n), dtype=torch.float32, device="cuda")
    outs = [flat[e - k:e].view(len(src), len(rcv), -1)
            for k, e, (_, src, rcv, _) in zip(n, np.cumsum(n).tolist(), inputs)]
    jobs = [(room, src, rcv) for room, src, rcv, _ in inputs]
    if call == "host":
        return dict(kind="batch_host", jobs=jobs, outs=outs, flat=flat, prec=prec)
    return dict(kind="batch", batch=_Batch(jobs, outs, prec), flat=flat)


class _Batch:
    """A prepared batch (ism_batch_prepare) whose RIRs go to the caller's own buffer."""

    def __init__(self, jobs, outs, precision):
        import ctypes

        self.keep, arr = [outs], (ism._Job * len(jobs))()
        pos = torch.from_numpy(np.concatenate([p for j in jobs for p in j[1:3]])).to("cuda")
        at = pos.data_ptr()
        for a, (room, src, rcv), out in zip(arr, jobs, outs):
            a.room, a.n_src, a.n_rcv, a.out = room._c(), len(src), len(rcv), out.data_ptr()
            a.src, a.rcv = at, at + 12 * len(src)
            at += 12 * (len(src) + len(rcv))
        size, prec, lib = ctypes.c_size_t(), ism.PRECISIONS[precision], ism.lib()
        ism._check(lib.ism_batch_workspace_size(arr, len(jobs), prec, ctypes.byref(size)), "ism_batch_workspace_size")
        ws = torch.empty(size.value, dtype=torch.uint8, device="cuda")
        self.keep += [pos, ws]
        self.batch = ism._Batch()
        self.ref = ctypes.byref(self.batch)
        st = torch.cuda.current_stream().cuda_stream
        ism._check(lib.ism_batch_prepare(arr, len(jobs), prec, ws.data_ptr(), size.value, st, self.ref),
                   "ism_batch_prepare")

    def run(self):
        ism._check(ism.lib().ism_batch_run(self.ref, torch.cuda.current_stream().cuda_stream), "ism_batch_run")


def run(state):
    kind = state["kind"]
    if kind == "sim":
        return state["sim"].run()
    if kind == "host":
        return ism.simulate_host(state["room"], state["src"], state["rcv"], state["prec"], out=state["out"])
    if kind == "polar":
        return ism.simulate_polar(state["room"], state["src"], state["rcv"], state["orient"], state["pattern"],
                                  state["prec"])
    if kind == "batch_host":
        ism.simulate_batch(state["jobs"], state["prec"], outs=state["outs"])
        return state["flat"]
    if kind == "batch":
        state["batch"].run()
        return state["flat"]
    return ism.filter_trajectory(state["x"], state["rirs"], ws=state["ws"])


def work(case):
    """Bytes: positions or signals and RIRs in, results out. FLOP: 24 per image for its
    distance, delay and amplitude and 20 for its share of the band-limited RIR (ten
    numbers describe an image's windowed sinc within its sample to FP32 accuracy),
    and 20 per sample and window tap to turn these into the RIR; filters by FFT."""
    if case["kind"] == "filter":
        n_y = case["n_x"] + case["n_rir"] - 1
        n = 4.0 * (case["n_x"] + case["n_pos"] * case["n_mic"] * case["n_rir"] + case["n_mic"] * n_y)
        points = case["n_pos"] * case["n_mic"] * case["n_rir"] + case["n_mic"] * n_y
        return {"bytes": n, "flops": 2.5 * 2.0 * points * math.log2(2.0 * min(case["n_rir"], 4096))}
    bytes_, flops = 0.0, 0.0
    for L, t60, n_src, n_rcv, fs, t_w, t_ism in _geometry(case):
        q, w = fs / C_SOUND, t_w * fs
        n, n_full = _n_samples(t_ism, fs), _n_samples(t60, fs)
        images = min(4.0 / 3.0 * math.pi * (n + w / 2) ** 3 / (L[0] * L[1] * L[2] * q ** 3),
                     float(np.prod([float(v) for v in _n_img(L, t_ism)])))
        bytes_ += 12.0 * (n_src + n_rcv) + 4.0 * n_src * n_rcv * n_full
        flops += n_src * n_rcv * (44.0 * images + 20.0 * n * w)
    return {"bytes": bytes_, "flops": flops}


# ---------------------------------------------------------------------------
# The same results in 64 bits
# ---------------------------------------------------------------------------
def _axis(L, b0, b1, n_img, s, r, q):
    """Image displacements [samples] and gains along one axis."""
    n = torch.arange(-(n_img // 2), (n_img + 1) // 2, device="cuda", dtype=torch.float64)
    odd = torch.remainder(n, 2.0) == 1.0
    coord = torch.where(odd, (n + 1) * L - s, n * L + s)
    gain = torch.pow(torch.tensor(b0, dtype=torch.float64, device="cuda"), torch.abs(torch.floor(n / 2))) * \
        torch.pow(torch.tensor(b1, dtype=torch.float64, device="cuda"), torch.abs(torch.floor((n + 1) / 2)))
    return (coord - r) * q, gain


def _windowed_sinc(v, w):
    return torch.where(v.abs() < w / 2, torch.sinc(v) * (0.5 + 0.5 * torch.cos(2.0 * math.pi / w * v)), 0.0)


def _taps(v, w, precision):
    if precision != "lut":
        return _windowed_sinc(v, w)
    lo = torch.floor(v * LUT_Q)
    a, b = _windowed_sinc(lo / LUT_Q, w), _windowed_sinc((lo + 1) / LUT_Q, w)
    return a + (v * LUT_Q - lo) * (b - a)


def _rir(r, n, s, m, precision, orient=None, pattern=1.0):
    """RIR of n samples of one source and receiver: every image's taps, added up image by image."""
    q, w = r["fs"] / r["c"], r["t_w"] * r["fs"]
    ax = [_axis(r["room"][a], r["beta"][2 * a], r["beta"][2 * a + 1], r["n_img"][a], float(s[a]), float(m[a]), q)
          for a in range(3)]
    d2 = (ax[0][0] ** 2)[:, None, None] + (ax[1][0] ** 2)[None, :, None] + (ax[2][0] ** 2)[None, None, :]
    at = torch.nonzero(d2.view(-1) < (n + w / 2 + 1) ** 2).view(-1)
    x = torch.sqrt(d2.view(-1)[at])
    n1, n2 = len(ax[1][0]), len(ax[2][0])
    i0, i1, i2 = at // (n1 * n2), (at // n2) % n1, at % n2
    amp = ax[0][1][i0] * ax[1][1][i1] * ax[2][1][i2] * (q / (4.0 * math.pi)) / x
    if orient is not None:
        o = [float(v) for v in orient]
        norm = math.sqrt(sum(v * v for v in o))
        cos = (ax[0][0][i0] * o[0] + ax[1][0][i1] * o[1] + ax[2][0][i2] * o[2]) / (norm * x)
        amp = amp * (pattern + (1.0 - pattern) * cos)
    k0 = torch.floor(x)
    order = torch.argsort(k0)
    k0, frac, amp = k0[order].long(), (x - k0)[order], amp[order]
    half = math.ceil(w / 2)
    j = torch.arange(1 - half, half + 1, device="cuda", dtype=torch.float64)[:, None]
    # per integer delay and tap: the sum over the images of that delay, from running sums
    n_bins = n + half
    sums = torch.zeros((len(j), n_bins + 1), dtype=torch.float64, device="cuda")
    step = max(1, 60_000_000 // len(j))
    for a in range(0, len(k0), step):
        k = k0[a:a + step]
        val = _taps(j - frac[a:a + step], w, precision) * amp[a:a + step]
        run_ = torch.nn.functional.pad(torch.cumsum(val, dim=1), (1, 0))
        ends = torch.searchsorted(k, torch.arange(n_bins + 1, device="cuda"))
        sums[:, :n_bins] += run_[:, ends[1:]] - run_[:, ends[:-1]]
    h = torch.zeros(n, dtype=torch.float64, device="cuda")
    for t in range(len(j)):
        off = t + 1 - half
        a, b = max(0, off), min(n, n_bins + off)
        h[a:b] += sums[t, a - off:b - off]
    return h


def _words(seed, rir, k):
    """Philox4x32-10 words of samples k (counter (k / 4, rir, 0, 0), word k % 4)."""
    m32 = 0xFFFFFFFF
    blk = torch.unique(k // 4)
    c = [blk.clone(), torch.full_like(blk, rir), torch.zeros_like(blk), torch.zeros_like(blk)]
    k0, k1 = seed & m32, (seed >> 32) & m32

    def mul(a, b):  # 32 x 32 -> (high, low) words
        lo = a * (b & 0xFFFF)
        hi = a * (b >> 16) + (lo >> 16)
        return hi >> 16, ((hi & 0xFFFF) << 16) | (lo & 0xFFFF)

    for i in range(10):
        if i:
            k0, k1 = (k0 + 0x9E3779B9) & m32, (k1 + 0xBB67AE85) & m32
        h0, l0 = mul(c[0], 0xD2511F53)
        h1, l1 = mul(c[2], 0xCD9E8D57)
        c = [h1 ^ c[1] ^ k0, l1, h0 ^ c[3] ^ k1, l0]
    return torch.stack(c, dim=1).view(-1)[k - 4 * (k[0] // 4)]


def _with_tail(early, rir, n, fs, t_diff, t60, seed):
    kd = len(early)
    k = torch.arange(kd - max(1, kd // 5), n, device="cuda")
    env = torch.pow(10.0, -6.0 * (k.double() / fs - t_diff) / t60)
    nw = max(1, kd // 5)
    level = torch.mean(early[kd - nw:] ** 2 / env[:nw])
    u = (_words(seed, rir, k[nw:]).double() + 0.5) / 2.0 ** 32
    z = torch.log(u / (1.0 - u)) * (math.sqrt(3.0) / math.pi)
    return torch.cat([early, z * torch.sqrt(level * env[nw:])])


def exact(case, seed):
    if case["kind"] == "filter":
        s = prepare(case, seed)
        x, rirs = s["x"].double(), s["rirs"]
        n_x, n_pos, n_rir = len(x), rirs.shape[0], rirs.shape[2]
        seg = -(-n_x // n_pos)
        y = torch.zeros((rirs.shape[1], n_x + n_rir - 1), dtype=torch.float64, device="cuda")
        size = 1 << (seg + n_rir - 1).bit_length()
        for p in range(n_pos):
            part = x[p * seg:min((p + 1) * seg, n_x)]
            if len(part) == 0:
                break
            z = torch.fft.irfft(torch.fft.rfft(part, size) * torch.fft.rfft(rirs[p].double(), size), size)
            e = len(part) + n_rir - 1
            y[:, p * seg:p * seg + e] += z[:, :e]
        return y
    t_diff = case["t60"] * case["att_db"] / 60.0 if case.get("call") == "diffuse" else None
    outs = []
    for r, src, rcv, orient in _inputs(case, seed):
        n_full = _n_samples(r["t_max"], r["fs"])
        n = n_full if t_diff is None else _n_samples(t_diff, r["fs"])
        h = []
        for i in range(len(src)):
            for m in range(len(rcv)):
                o = (orient[m], case["pattern"]) if case.get("call") == "polar" else (None, 1.0)
                v = _rir(r, n, src[i], rcv[m], case["precision"], *o)
                if t_diff is not None:
                    v = _with_tail(v, len(h), n_full, r["fs"], t_diff, case["t60"], seed % 1000003)
                h.append(v)
        outs.append(torch.stack(h).view(len(src), len(rcv), n_full))
    return outs[0] if case["kind"] == "room" else torch.cat([v.view(-1) for v in outs])
