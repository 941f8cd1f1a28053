"""Second moments of 256-channel tiles split over several workgroups, against
fp64 sums: tiles of 1 to 16 pieces, whole tiles, ragged edges and last slabs,
diagonal tiles of which only the upper half is kept, packed groups of small
blocks, onto a non-zero symmetric start."""
import numpy as np
import pytest

import paper_2603_04359_amd as cat
from paper_2603_04359_amd import binding as B

from gpu_common import host, say, torch_mod

pytestmark = pytest.mark.gpu

# (d, k or 0 for the whole matrix, n); a slab is 32 tokens, a launch 256 slabs
CASES = [(256, 0, 1), (256, 0, 200), (288, 0, 700), (1024, 0, 4099), (544, 0, 8192 + 33),
         (256, 256, 8192), (2560, 256, 130), (14336, 256, 321), (65536, 256, 64), (65792, 256, 40),
         (1536, 512, 515), (2048, 512, 96), (1024, 128, 777), (512, 64, 4000), (768, 32, 95)]


@pytest.mark.parametrize("d,k,n", CASES)
def test_cov_split_tiles(d, k, n):
    torch = torch_mod()
    say(f"cov split d={d} k={k} n={n}")
    g = torch.Generator(device="cuda").manual_seed(d + k + n)
    X = (torch.randn(n, d, generator=g, device="cuda") * torch.exp(torch.randn(d, generator=g, device="cuda")))
    X = X.bfloat16()
    kk = k or d
    xb = X.double().view(n, d // kk, kk).transpose(0, 1).contiguous()
    S = torch.randn(d // kk, kk, kk, generator=g, device="cuda")
    S = (S + S.transpose(1, 2)).contiguous()
    want = S.double() + torch.matmul(xb.transpose(1, 2).contiguous(), xb)
    acc = S.clone() if k else S[0].clone()
    cat.cat_cov_accumulate(X, acc, B.CAT_COV_BLOCK_DIAG if k else B.CAT_COV_FULL, k or 1)
    got = acc.view_as(want)
    # an entry is an fp32 sum of n exact products in a fixed order, cut into a
    # few partial sums: with each addition off by at most an ulp, (n + 20) 2^-23
    # of the sum of their sizes
    size = S.double().abs() + torch.matmul(xb.abs().transpose(1, 2).contiguous(), xb.abs())
    bound = (n + 20) * 2.0 ** -23 * size
    assert bool(((got.double() - want).abs() <= bound).all())
    rel = float((got.double() - want).norm() / want.norm())
    say(f"  rel fro {rel:.2e}")
    assert rel <= 1.2e-6         # what 32-bit sums of up to 8192 terms show, times four
    assert bool(((got - got.transpose(1, 2)).abs() <= 2 * bound).all())


def test_cov_split_deterministic_and_mirrored():
    """The pieces of a tile are added in one fixed order: two calls agree bit
    for bit, and a diagonal tile's two triangles are mirror images."""
    torch = torch_mod()
    say("cov split determinism")
    g = torch.Generator(device="cuda").manual_seed(4)
    X = torch.randn(5003, 2560, generator=g, device="cuda").bfloat16()
    res = []
    for _ in range(2):
        acc = torch.zeros(10, 256, 256, device="cuda")
        cat.cat_cov_accumulate(X, acc, B.CAT_COV_BLOCK_DIAG, 256)
        res.append(host(acc))
    assert np.array_equal(res[0], res[1])
    off = res[0][:, :64, 64:]
    assert np.array_equal(off, res[0][:, 64:, :64].transpose(0, 2, 1))
