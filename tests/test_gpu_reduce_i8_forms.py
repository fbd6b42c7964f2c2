"""The int8 reduce's two forms (GPU): 12 and 13 peers (the rule on the group's
size), and lengths just below and above where the form changes (1024, 2048 and
3072 workgroups of four 1024-element blocks), with whole and partial last
blocks: the first, last and some middle blocks bit for bit with the oracle."""

import numpy as np
import pytest

import oracle
from paper_2106_10207_amd import dedloc as D

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

WG = 4096  # elements per workgroup


@pytest.mark.parametrize("n_peers", [12, 13])
@pytest.mark.parametrize("n", [700, 1023 * WG, 1024 * WG, 2048 * WG + 1, 3072 * WG + 5])
def test_reduce_i8_forms(n_peers, n):
    print(f"\n[reduce i8 forms] {n_peers} peers, n={n}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n % 1000 + n_peers)
    nb = (n + 1023) // 1024
    codes = [torch.randint(-127, 128, (n,), generator=gen, device="cuda", dtype=torch.int8) for _ in range(n_peers)]
    scales = [torch.rand(nb, generator=gen, device="cuda").mul_(1e-5) for _ in range(n_peers)]
    counts = np.arange(1, n_peers + 1, dtype=np.uint32)
    mean = torch.empty(n, device="cuda")
    oc, osc = D.dedloc_reduce_shard(codes, counts, n, D.DEDLOC_CODEC_I8, scales, out_mean=mean)
    torch.cuda.synchronize()
    for b in sorted({0, nb - 1, max(0, nb - 2), nb // 2, nb // 3}):
        sl = slice(b * 1024, min(n, b * 1024 + 1024))
        rc, rs, rm = oracle.reduce([c[sl].cpu().numpy() for c in codes], counts, oracle.CODEC_I8,
                                   [s[b:b + 1].cpu().numpy() for s in scales], 1024)
        assert np.array_equal(mean[sl].cpu().numpy().view(np.uint32), rm.view(np.uint32)), b
        assert np.array_equal(oc[sl].cpu().numpy().view(np.int8), rc), b
        assert np.array_equal(osc[b:b + 1].cpu().numpy().view(np.uint32), rs.view(np.uint32)), b
