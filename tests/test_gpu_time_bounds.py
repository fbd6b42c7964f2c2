"""Orders of time that hold by what each form moves through memory (GPU).

Each test times two ways to the same result in turn, on the same buffers, and
takes the best of several repeats of each, so that neither the machine's
speed nor a passing disturbance decides; the bounds lie well between what the
bytes give and the time of the mistake each one guards against."""

import numpy as np
import pytest

from paper_2106_10207_amd import dedloc as D
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


def _step(sizes):
    """A call of the LAMB step on an fp32 gradient, tensors of these sizes."""
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.uint64)
    P = int(off[-1])
    x = torch.randn(P, device=DEV).mul_(0.02)
    m, v, g = torch.zeros(P, device=DEV), torch.full((P,), 1e-6, device=DEV), torch.randn(P, device=DEV).mul_(1e-3)
    flags, cfg, ws = np.full(len(sizes), 3, np.uint8), D.lamb_cfg(step=10), D.make_workspace(P, off)
    return lambda stream=None: D.dedloc_lamb_step(x, m, v, g, off, flags, cfg, ws=ws, stream=stream)


@pytest.mark.parametrize("polls", [4096, 0])
def test_one_large_tensor_takes_no_longer_than_its_bytes(polls):
    """2^28 elements in one tensor: nearly all of its rows are updated by the
    second pass, 40 bytes an element against 28 for the same elements in 64
    tensors (measured 1.92 against 1.38 ms; given up by every workgroup that
    waits, 1.96 to 2.05).  With a partial sum per 4096 elements and the ratio
    formed again by every workgroup of the second pass it took 34 ms."""
    print(f"\n[time] one large tensor, polls {polls}", flush=True)
    one, split = _step([1 << 28]), _step([1 << 22] * 64)
    (apart,) = _best_us([split], 3, 3)
    old = D.dedloc_test_trust_polls(polls)
    try:
        (whole,) = _best_us([one], 3, 3)
    finally:
        D.dedloc_test_trust_polls(old)
    print(f"one tensor {whole:.0f} us, 64 tensors {apart:.0f} us", flush=True)
    assert whole <= 2.5 * apart


def test_two_streams_take_little_longer_than_one():
    """Two one-pass steps, each in the other's way on a stream of its own: a
    workgroup whose tensor waits for workgroups that cannot start gives up
    soon, and the second pass does what is left.  Measured for the pair, two
    streams against one: 463 / 439 us; with waits of 512 polls and a ratio
    formed by every workgroup of the second pass 1255 / 447."""
    print("\n[time] two streams", flush=True)
    steps = [_step([1 << 25]) for _ in range(2)]
    streams = [torch.cuda.Stream() for _ in range(2)]

    def apart():
        for f, s in zip(steps, streams):
            s.wait_stream(torch.cuda.current_stream())
            for _ in range(4):
                f(s)
        for s in streams:
            torch.cuda.current_stream().wait_stream(s)

    def together():
        for _ in range(4):
            for f in steps:
                f()

    two, one = _best_us([apart, together], 5, 3)
    print(f"two streams {two:.0f} us, one {one:.0f} us", flush=True)
    assert two <= 1.7 * one
