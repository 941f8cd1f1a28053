"""Calls of more workgroups than one launch can have (fewer than 2^32 threads),
and rows wider than 32-bit byte offsets."""
import numpy as np
import pytest

import paper_2603_04359_amd as cat
from paper_2603_04359_amd import binding as B

from gpu_common import dev, host, say, torch_mod
from test_gpu_parity import _rand_T

pytestmark = pytest.mark.gpu


def test_second_moments_of_more_blocks_than_a_launch():
    torch = torch_mod()
    d, k = (1 << 27) + 4096, 16
    say(f"cov 1 x {d}, k={k}")
    x = torch.randn(1, d, dtype=torch.float32, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    acc = torch.zeros((d // k, k, k), dtype=torch.float32, device="cuda")
    cat.cat_cov_accumulate(x, acc, B.CAT_COV_BLOCK_DIAG, k)
    xb = x.view(-1, k)
    for i in range(0, d // k, 1 << 20):
        v = xb[i:i + (1 << 20)]
        assert torch.equal(acc[i:i + (1 << 20)], v[:, :, None] * v[:, None, :]), f"block {i} on"


def test_second_moments_of_rows_beyond_32_bit_offsets():
    torch = torch_mod()
    n, d = 5, (1 << 28) + 24
    say(f"cov {n} x {d}, k=1")
    x = torch.randn(n, d, dtype=torch.float32, device="cuda", generator=torch.Generator("cuda").manual_seed(2))
    acc = torch.zeros((d, 1, 1), dtype=torch.float32, device="cuda")
    cat.cat_cov_accumulate(x, acc, B.CAT_COV_BLOCK_DIAG, 1)
    for i in range(0, d, 1 << 26):
        ref = x[:, i:i + (1 << 26)].double().square_().sum(0)
        # the fp64 sum rounded once
        err = (acc[i:i + (1 << 26), 0, 0].double() - ref).abs_() / ref
        assert err.max().item() <= 2.0 ** -24 * 1.001


# whole rows, and channel pairs on the vector ALU
@pytest.mark.parametrize("n,d,k,x_dtype,border", [((1 << 26) + 33, 16, 16, "float32", 1 << 25),
                                                  (2_089_100, 4112, 16, "bfloat16", 1_044_506)])
@pytest.mark.parametrize("asym", [False, True])
def test_transform_quant_of_more_threads_than_a_launch(n, d, k, x_dtype, border, asym):
    torch = torch_mod()
    say(f"tq {n} x {d}, k={k} asym={asym}")
    X = torch.randn(n, d, dtype=getattr(torch, x_dtype), device="cuda",
                    generator=torch.Generator("cuda").manual_seed(3))
    T = dev(_rand_T(d, k, seed=4), "f32")

    def call(x):
        m = x.shape[0]
        codes = torch.full((m, d // 2), 77, dtype=torch.uint8, device="cuda")
        s_x, zmin = (torch.full((m,), 5.0, dtype=torch.float32, device="cuda") for _ in range(2))
        if asym:
            ws = torch.empty(cat.cat_transform_quant_asym_workspace_bytes(m, d, k), dtype=torch.uint8, device="cuda")
            cat.cat_transform_quant_asym(x, T, k, codes, s_x, zmin, ws)
        else:
            ws = torch.empty(cat.cat_transform_quant_workspace_bytes(m, d, k), dtype=torch.uint8, device="cuda")
            cat.cat_transform_quant(x, T, k, codes, s_x, ws)
        return codes, s_x, zmin

    whole = call(X)
    # around the launches' borders and at both ends, against calls of their own
    for lo in (0, border - 16, n - 50):
        part = call(X[lo:lo + 50].clone())
        for a, b in zip(part, whole):
            assert torch.equal(a, b[lo:lo + 50]), f"tokens {lo} on"
    assert not np.isnan(host(whole[1]).min())
