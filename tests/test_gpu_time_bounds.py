"""Orders of time that hold by what each form moves through memory (GPU).

Each test times two ways to the same result in turn, on the same buffers, and
takes the best of several repeats of each, so that neither the machine's
speed nor a passing disturbance decides; the bounds lie well between what the
bytes give and the time of the mistake each one guards against."""

import pytest

from paper_2106_10207_amd import harness as H
from paper_2106_10207_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda"


def _best_us(forms, repeats=9, calls=10):
    """Best time of one call of each form, the forms timed in turn."""
    best = [float("inf")] * len(forms)
    for _ in range(repeats):
        for i, f in enumerate(forms):
            f()
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(calls):
                f()
            b.record()
            b.synchronize()
            best[i] = min(best[i], a.elapsed_time(b) * 1e3 / calls)
    return best


def test_local_gradient_in_the_round_beats_its_own_encode():
    """Two passes (161 tensors): the round that encodes the local peer's
    gradient reads 4 and writes 2 bytes an element where an encode of its own
    before the round reads 4, writes 2 and has them read again, one launch
    more.  Measured 438 against 448 us; with plain loads of the gradient the
    round took 456 to 460."""
    print("\n[time] local gradient", flush=True)
    dr = H.DeviceRound(W.WORKLOADS["resnet50"], DEV, fused_local=True)

    def separate():
        dr.encode_local()
        dr.call_round_only()

    fused, apart = _best_us([dr.call, separate])
    print(f"in the round {fused:.1f} us, encoded before it {apart:.1f} us", flush=True)
    assert fused <= apart
