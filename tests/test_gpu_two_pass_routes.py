"""bf16 two-pass transform+quant on both sides of the rules that pick its kernel
by the number of tokens: the same tokens alone and at the front of a larger
call, which takes another kernel, give the same bits; a few rows also against
the CPU oracle."""
import functools

import numpy as np
import pytest

import paper_2603_04359_amd as cat
from oracle import cat_oracle as o

from gpu_common import dev, host, say, torch_mod
from test_gpu_asym import _check_asym
from test_gpu_wide_two_pass import _check_codes, _inputs

pytestmark = pytest.mark.gpu


@functools.lru_cache(maxsize=1)
def _case(d, k, n):
    X, T = _inputs(d, k, n)
    return X, T, dev(X, "bf16"), dev(T, "bf16")


# kernels on a 256-CU device, for m tokens and for n
@pytest.mark.parametrize("d,k,m,n", [
    (14336, 128, 300, 2341),       # wide; group (n d just above 2^25)
    (65536, 128, 64, 129),         # wide with slots, a span per CU; group
    (66048, 128, 3, 65),           # group, more spans than CUs
    (65536, 256, 64, 65),          # wide with slots; group
    (66048, 256, 130, 257),        # group; wide
    (2048, 256, 64 * 32 * 2, 64 * 32 * 2 + 1),      # wide with slots, two tiles; cleared words
    (2304, 256, 64 * 28, 64 * 28 * 2),              # wide with slots, one tile; two, cleared words
    (49152, 512, 96, 97),          # ring; wide
    (66048, 512, 65, 161),         # ring; wide
])
@pytest.mark.parametrize("mode", [4, 8, "asym"])
def test_routes_agree(d, k, m, n, mode):
    torch = torch_mod()
    say(f"tq routes d={d} k={k} m={m} n={n} {mode}")
    asym, bits = mode == "asym", 4 if mode == "asym" else mode
    X, T, Xd, Td = _case(d, k, n)
    size = cat.cat_transform_quant_asym_workspace_bytes if asym else cat.cat_transform_quant_workspace_bytes
    res = []
    for c in (m, n):
        codes = torch.full((c, d // 2 if bits == 4 else d), 77, device="cuda",
                           dtype=torch.uint8 if bits == 4 else torch.int8)
        s_x, zmin = (torch.full((c,), 5.0, dtype=torch.float32, device="cuda") for _ in range(2))
        ws = torch.full((size(c, d, k),), 0xFF, dtype=torch.uint8, device="cuda")
        if asym:
            cat.cat_transform_quant_asym(Xd[:c], Td, k, codes, s_x, zmin, ws)
        else:
            cat.cat_transform_quant(Xd[:c], Td, k, codes, s_x, ws, bits=bits)
        res.append([host(v) for v in (codes, s_x, zmin)])
    for a, b in zip(*res):
        assert np.array_equal(a, b[:m])
    rows = np.unique([0, m - 1, n // 2, n - 1])
    codes, s_x, zmin = (v[rows] for v in res[1])
    label = f"d={d} k={k} n={n} {mode}"
    if asym:
        _check_asym(o.unpack_int4(codes).astype(np.int16) + 8, s_x, zmin, X[rows], T, label)
    else:
        s_or = _check_codes(codes, X[rows], T, bits, label)
        assert np.all(np.abs(s_x.astype(np.float64) - s_or) <= 1e-6 * s_or)
