"""ism.filter_trajectory on another stream than the current one: its workspace, its copies
of strided inputs and its output stay the call's until that stream is done with them.

The stream is held up by a copy of a large buffer many times over while the current stream
allocates and overwrites memory of every size that the call may have dropped; the result is
that of the same call on the current stream, bit for bit."""
import pytest

from paper_1810_11359_amd import ism

pytestmark = pytest.mark.gpu

CASES = [
    # name, n_x, n_pos, n_mic, n_rir, strided inputs
    ("segments_of_160", 16000, 100, 2, 4000, False),   # segment blocks
    ("segments_of_9000", 27000, 3, 2, 5000, False),    # fixed blocks
    ("strided_inputs", 16000, 100, 2, 4000, True),     # copies made by the call
]


class _Handle:
    """A stream of another library: only its handle."""

    def __init__(self, stream):
        self.cuda_stream = stream.cuda_stream


@pytest.mark.parametrize("handle", [False, True], ids=["torch_stream", "foreign_handle"])
@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_call_on_another_stream(case, handle):
    import torch

    name, n_x, n_pos, n_mic, n_rir, strided = case
    print(f"[case] {name}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(5)
    step = 2 if strided else 1
    x = torch.randn(n_x * step, generator=g, device="cuda")[::step]
    rirs = torch.randn(n_pos, n_mic, n_rir * step, generator=g, device="cuda")[:, :, ::step]
    expected = ism.filter_trajectory(x, rirs)
    need = ism.filter_workspace_size(n_x, n_pos, n_mic, n_rir)
    assert need > 0
    busy = torch.empty(1 << 28, device="cuda"), torch.empty(1 << 28, device="cuda")
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        for _ in range(60):  # 2 GiB a copy: some 30 ms in all
            busy[0].copy_(busy[1])
    y = ism.filter_trajectory(x, rirs, stream=_Handle(side) if handle else side)
    # what the call allocated and dropped would be given out again here
    junk = [torch.full((n // 4,), float("nan"), device="cuda") for n in (need, 4 * n_x, rirs.numel() * 4) * 2]
    torch.cuda.current_stream().wait_stream(side)
    got = y.clone()
    torch.cuda.synchronize()
    assert torch.equal(got, expected)
    assert all(bool(torch.isnan(j).all()) for j in junk)  # and the call did not write there


def test_inputs_dropped_after_the_call():
    """Temporaries passed as inputs may go as soon as the call returns."""
    import torch

    n_x, n_pos, n_mic, n_rir = 16000, 100, 2, 4000
    g = torch.Generator(device="cuda").manual_seed(6)
    x = torch.randn(n_x, generator=g, device="cuda")
    rirs = torch.randn(n_pos, n_mic, n_rir, generator=g, device="cuda")
    expected = ism.filter_trajectory(x * 2.0, rirs * 0.5)
    busy = torch.empty(1 << 28, device="cuda"), torch.empty(1 << 28, device="cuda")
    side = torch.cuda.Stream()
    x2, r2 = x * 2.0, rirs * 0.5
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        for _ in range(60):
            busy[0].copy_(busy[1])
    y = ism.filter_trajectory(x2, r2, stream=side)
    del x2, r2
    junk = [torch.full((n,), float("nan"), device="cuda") for n in (n_x, n_pos * n_mic * n_rir) * 2]
    torch.cuda.current_stream().wait_stream(side)
    got = y.clone()
    torch.cuda.synchronize()
    assert torch.equal(got, expected)
    assert all(bool(torch.isnan(j).all()) for j in junk)
