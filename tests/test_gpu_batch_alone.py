"""A batch of one job is bitwise the untapered single call (tail_rounds = 0), also where the
item size that the images ask for would take more workspace than the call reserves: few
images, tiles of 512 samples, a short window."""
import numpy as np
import pytest

from paper_1810_11359_amd import ism

pytestmark = pytest.mark.gpu

CASES = [
    # room, fs, t_w, t_max, sources, receivers
    ([9.138, 5.564, 8.079], 16000.0, 0.002, 0.1661902, 3, 7),
    ([7.633, 3.183, 2.198], 8000.0, 0.004, 0.0787676, 1, 7),
    ([7.633, 3.183, 2.198], 8000.0, 0.004, 0.08, 1, 8),
    ([4.0, 5.0, 3.0], 16000.0, 0.004, 0.3, 1, 8),
    ([9.0, 8.0, 7.0], 48000.0, 0.002, 0.1, 1, 30),
]


@pytest.mark.parametrize("precision", ["fp32", "lut", "fp16"])
@pytest.mark.parametrize("case", CASES, ids=[f"{c[1] / 1000:g}k_{c[3]:g}s_{c[4]}x{c[5]}" for c in CASES])
def test_one_job_is_the_untapered_call(case, precision):
    import torch

    L, fs, t_w, t_max, n_src, n_rcv = case
    room = ism.Room(L, [0.9] * 6, ism.n_img_for_time(L, 343.0, t_max), 343.0, fs, t_max, t_w)
    rng = np.random.default_rng(n_rcv)
    src = rng.uniform(0.3, np.array(L) - 0.3, (n_src, 3)).astype(np.float32)
    rcv = rng.uniform(0.3, np.array(L) - 0.3, (n_rcv, 3)).astype(np.float32)
    print(f"[case] one job {case} {precision}", flush=True)
    alone = ism.BatchSimulator([(room, src, rcv)], precision=precision).run()[0]
    untapered = ism.simulate(room, src, rcv, precision, schedule=ism.Schedule(tail_rounds=0.0))
    torch.cuda.synchronize()
    assert torch.equal(alone, untapered)
