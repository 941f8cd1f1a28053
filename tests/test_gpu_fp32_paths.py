"""The fp64-summed kernels of fp32 operands (and of bf16 blocks the bf16
kernels do not take) at the edges of their tiles: second moments against
fp64 sums, whole-row transform+quant against the CPU oracle."""
import numpy as np
import pytest

import paper_2603_04359_amd as cat
from oracle import cat_oracle as o
from paper_2603_04359_amd import binding as B

from gpu_common import check_codes, dev, host, say, torch_mod

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode,d,k,n,dtype", [
    ("full", 5, 1, 3, "f32"),            # one 16 x 16 tile, mostly outside the matrix
    ("full", 100, 1, 4097, "f32"),       # 16 x 16 tiles, a second flush of one token
    ("full", 1040, 1, 37, "f32"),        # 32 x 32 tiles, ragged last one
    ("full", 1604, 1, 50, "f32"),        # the same, ragged by a part of a fragment
    ("block", 40, 8, 130, "f32"),        # blocks smaller than a tile
    ("block", 256, 32, 512, "f32"),      # three 16 x 16 tiles per block
    ("block", 16384, 64, 9, "f32"),      # three 32 x 32 tiles per block
    ("block", 8192, 32, 70, "f32"),      # one 32 x 32 tile per block
    ("block", 96, 16, 200, "bf16"),
    ("block", 17, 1, 5, "f32"),          # several blocks to a tile, a ragged last one
    ("block", 18, 2, 300, "f32"),
    ("block", 148, 4, 33, "bf16"),
    ("block", 24, 8, 4100, "f32"),       # and a second flush
    ("block", 4096, 1, 70, "bf16"),
    ("block", 8224, 32, 70, "bf16"),     # 32 x 32 tiles, two channels at once
    ("block", 8224, 32, 300, "bf16"),
])
def test_second_moment_fp64_path(mode, d, k, n, dtype):
    torch = torch_mod()
    say(f"cov {mode} d={d} k={k} n={n} {dtype}")
    rng = np.random.default_rng(d + n)
    X = o.round_storage(rng.standard_normal((n, d)) * np.exp(rng.standard_normal(d)), dtype)
    acc = torch.zeros((d, d) if mode == "full" else (d // k, k, k), dtype=torch.float32, device="cuda")
    cat.cat_cov_accumulate(dev(X, dtype), acc, B.CAT_COV_FULL if mode == "full" else B.CAT_COV_BLOCK_DIAG, k)
    got = host(acc).astype(np.float64)
    X = X.astype(np.float64)
    if mode == "full":
        ref, mag = X.T @ X, np.abs(X).T @ np.abs(X)
    else:
        xb = X.reshape(n, d // k, k).transpose(1, 0, 2)
        ref = xb.transpose(0, 2, 1) @ xb
        mag = np.abs(xb).transpose(0, 2, 1) @ np.abs(xb)
    # fp64 sums, rounded to fp32 once per 4096 tokens
    flushes = -(-n // 4096)
    assert np.all(np.abs(got - ref) <= flushes * 2.0 ** -24 * mag * 1.001)


# On a 256-CU device full matrices of 481 channels and more run 32 x 32 tiles, up
# to 128 tokens with four groups of 4 in flight per wave and beyond with eight;
# an odd width reads channels one by one.  The accumulator starts with values.
@pytest.mark.parametrize("dtype,d", [("f32", 480), ("f32", 512), ("f32", 560), ("f32", 561), ("f32", 1041),
                                     ("bf16", 561), ("bf16", 1041)])
@pytest.mark.parametrize("n", [1, 15, 17, 127, 129, 259])
def test_second_moment_fp64_path_accumulates(dtype, d, n):
    torch = torch_mod()
    say(f"cov full d={d} n={n} {dtype}, non-zero start")
    rng = np.random.default_rng(d + n)
    X = o.round_storage(rng.standard_normal((n, d)) * np.exp(rng.standard_normal(d)), dtype)
    start = rng.standard_normal((d, d)).astype(np.float32)
    start = start + start.T
    acc = dev(start, "f32")
    cat.cat_cov_accumulate(dev(X, dtype), acc, B.CAT_COV_FULL, 1)
    got = host(acc).astype(np.float64)
    X = X.astype(np.float64)
    ref = start.astype(np.float64) + X.T @ X
    # one rounding of the fp64 sum to fp32
    assert np.all(np.abs(got - ref) <= 2.0 ** -24 * 1.001 * np.abs(ref) + 2.0 ** -45 * (np.abs(X).T @ np.abs(X)))
    assert np.array_equal(got, got.T)


@pytest.mark.parametrize("x_dtype,t_dtype,d,k,n,bits", [
    ("f32", "f32", 16, 16, 1, 4),            # one tile, fifteen waves without work
    ("f32", "f32", 256, 32, 512, 8),         # the tiny layer
    ("f32", "bf16", 1024, 64, 33, 6),        # four tiles per wave, one token in the last workgroup
    ("bf16", "f32", 1040, 16, 17, 4),        # more than four, ragged over the waves
    ("f32", "f32", 4096, 512, 18, 4),        # the widest row and block
    ("bf16", "f32", 4096, 512, 2, 4),        # one zero token and another: the two-pass kernels
    ("f32", "bf16", 4096, 512, 3, 8),
    ("f32", "f32", 4112, 16, 5, 4),          # wider: the two-pass kernels
    ("bf16", "bf16", 4096, 16, 40, 8),
])
def test_transform_quant_whole_rows(x_dtype, t_dtype, d, k, n, bits):
    torch = torch_mod()
    say(f"tq rows {x_dtype}/{t_dtype} d={d} k={k} n={n} bits={bits}")
    rng = np.random.default_rng(d + k + n)
    X = o.round_storage(rng.standard_normal((n, d)) * np.exp(rng.standard_normal(d)), x_dtype).astype(np.float64)
    X[0] = 0.0
    T = o.round_storage(rng.standard_normal((d // k, k, k)) / np.sqrt(k), t_dtype).astype(np.float64)
    codes = torch.empty((n, d // 2) if bits == 4 else (n, d), device="cuda",
                        dtype=torch.uint8 if bits == 4 else torch.int8)
    s_x = torch.empty(n, dtype=torch.float32, device="cuda")
    ws = torch.empty(cat.cat_transform_quant_workspace_bytes(n, d, k), dtype=torch.uint8, device="cuda")
    cat.cat_transform_quant(dev(X, x_dtype), dev(T, t_dtype), k, codes, s_x, ws, bits=bits)
    got = host(codes)
    _, _, s_or = check_codes(got, X, T, bits=bits, label=f"d={d} k={k}")
    s = host(s_x).astype(np.float64)
    # z is the fp32 rounding of an fp64 sum, the scale one more rounding
    assert np.all(np.abs(s - s_or) <= 2.0 ** -22 * s_or)
    assert s[0] == 0 and not got[0].any()


def test_transform_quant_whole_rows_asymmetric_infinite_and_nan_rows():
    # a row with an infinity or a NaN stays its own affair: other rows are
    # untouched, and its scale is not finite
    torch = torch_mod()
    say("tq rows inf/nan")
    n, d, k = 20, 128, 32
    rng = np.random.default_rng(4)
    X = rng.standard_normal((n, d)).astype(np.float32)
    T = rng.standard_normal((d // k, k, k)).astype(np.float32)
    bad = X.copy()
    bad[3, 5], bad[17, 99] = np.inf, np.nan
    out = []
    for x in (X, bad):
        codes = torch.empty((n, d // 2), dtype=torch.uint8, device="cuda")
        s_x, zmin = (torch.empty(n, dtype=torch.float32, device="cuda") for _ in range(2))
        ws = torch.empty(cat.cat_transform_quant_asym_workspace_bytes(n, d, k), dtype=torch.uint8, device="cuda")
        cat.cat_transform_quant_asym(torch.from_numpy(x).cuda(), dev(T, "f32"), k, codes, s_x, zmin, ws)
        sym = torch.empty(n, dtype=torch.float32, device="cuda")
        c2 = torch.empty_like(codes)
        cat.cat_transform_quant(torch.from_numpy(x).cuda(), dev(T, "f32"), k, c2, sym, ws)
        out.append([host(a) for a in (codes, s_x, zmin, c2, sym)])
    ok = np.setdiff1d(np.arange(n), [3, 17])
    for a, b in zip(*out):
        assert np.array_equal(a[ok], b[ok])
    assert not np.isfinite(out[1][4][[3, 17]]).any()
