"""The elementwise kernels' rows of 2048 elements (GPU): lengths at the edges
of a row and of a wave's 512, against the oracle, bit for bit, with the bytes
past the end untouched."""

import numpy as np
import pytest

import oracle
from paper_2106_10207_amd import dedloc as D

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LENGTHS = [1, 3, 511, 513, 2047, 2048, 2049, 4096, 3 * 2048 + 257]


@pytest.mark.parametrize("n", LENGTHS)
def test_rows(n):
    print(f"\n[rows] {n}", flush=True)
    rng = np.random.default_rng(n)
    g = (rng.standard_normal(n) * 1e-2).astype(np.float32)
    acc = rng.standard_normal(n).astype(np.float32)
    want = oracle.encode_fp16(g)
    pad = 16  # room past the end
    up = lambda a: torch.from_numpy(a).cuda()
    codes = torch.full((n + pad,), 0x1234, dtype=torch.int16, device="cuda")
    D.dedloc_encode(up(g), D.DEDLOC_CODEC_FP16, codes=codes)
    back = torch.full((n + pad,), 7.0, device="cuda")
    D.dedloc_decode(codes, None, n, D.DEDLOC_CODEC_FP16, out=back)
    back8 = torch.full((n + pad,), 7.0, device="cuda")
    c8, s8 = oracle.encode_i8(g, 1024)
    D.dedloc_decode(up(c8), up(s8), n, D.DEDLOC_CODEC_I8, out=back8)
    torch.cuda.synchronize()
    got = codes.cpu().numpy()
    assert np.array_equal(got[:n].view(np.uint16), want) and np.all(got[n:] == 0x1234)
    got = back.cpu().numpy()
    assert np.array_equal(got[:n], want.view(np.float16).astype(np.float32)) and np.all(got[n:] == 7.0)
    got = back8.cpu().numpy()
    assert np.array_equal(got[:n], c8.astype(np.float32) * np.repeat(s8, 1024)[:n]) and np.all(got[n:] == 7.0)
    # fma(b, g, acc) and acc / count: products and sums of these are exact in float64
    for grad, h in ((up(g), g), (up(want.view(np.int16)), want.view(np.float16).astype(np.float32))):
        a = up(acc.copy())
        D.dedloc_accumulate(a, grad, 3.0)
        expect = (np.float64(3.0) * h + acc).astype(np.float32)
        assert np.array_equal(a.cpu().numpy(), expect)
        out = torch.full((n + pad,), 0x1234, dtype=torch.int16, device="cuda")
        D.dedloc_finalize(a, 8, D.DEDLOC_CODEC_FP16, codes=out, reset=True)
        o = out.cpu().numpy()
        assert np.array_equal(o[:n].view(np.uint16), oracle.encode_fp16(expect / np.float32(8.0)))
        assert np.all(o[n:] == 0x1234) and not np.any(a.cpu().numpy())


@pytest.mark.parametrize("n", [(1 << 20) - 1, 1 << 20, (1 << 21) - 1, 1 << 21, (1 << 21) + 2049])
def test_decode_on_both_sides_of_its_store_rule(n):
    """The decoders take other stores from 2^20 (fp16) and 2^21
    (int8) elements on: whole rows and
    blocks and the partial last ones, bit for bit, nothing past the end."""
    print(f"\n[decode] {n}", flush=True)
    rng = np.random.default_rng(n)
    c16 = rng.integers(0, 0x7C00, n, np.uint16)  # finite, non-negative
    c8 = rng.integers(-127, 128, n, np.int8)
    s8 = rng.random((n + 1023) // 1024, np.float32)
    up = lambda a: torch.from_numpy(a).cuda()
    for codes, scales, codec, want in (
            (c16.view(np.int16), None, D.DEDLOC_CODEC_FP16, c16.view(np.float16).astype(np.float32)),
            (c8, s8, D.DEDLOC_CODEC_I8, c8.astype(np.float32) * np.repeat(s8, 1024)[:n])):
        back = torch.full((n + 16,), 7.0, device="cuda")
        D.dedloc_decode(up(codes), None if scales is None else up(scales), n, codec, out=back)
        got = back.cpu().numpy()
        assert np.array_equal(got[:n].view(np.uint32), want.view(np.uint32)) and np.all(got[n:] == 7.0)
