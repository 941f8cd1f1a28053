"""Small-tile integer GEMM (few output tiles, the reduction split over a
workgroup's waves) against the CPU oracle: every tile shape, at ragged rows,
outputs and row lengths.  The sums are exact integers and the epilogue has
one fp32 order, so sums and outputs must equal the oracle's bit for bit."""
import numpy as np
import pytest

import paper_2603_04359_amd as cat
from oracle import cat_oracle as o

from gpu_common import dev, host, say, torch_mod

pytestmark = pytest.mark.gpu

# (n, d_in, d_out); the tile shape a 256-CU device launches with is beside it
CASES = [
    (1, 32, 1),            # 16 x 16: one unit of a row, seven waves without work
    (1, 4096, 4096),       # 16 x 16: the decode shape, every CU one tile
    (16, 96, 4097),        # 16 x 32: a row of one ragged chunk, one output in the last tile
    (17, 4128, 4100),      # 32 x 32: one row in the last tile, ragged last chunk
    (33, 2080, 4000),      # 32 x 32
    (31, 4096, 8200),      # 32 x 64
    (47, 4128, 16001),     # 48 x 64, one output in the last tile
    (63, 4096, 4100),      # 64 x 32
    (250, 4096, 4096),     # 64 x 64
    (257, 4128, 4000),     # 80 x 64
    (190, 4096, 8000),     # 96 x 64
    (128, 2080, 14300),    # 128 x 64
    (1000, 4128, 500),     # 64 x 32: many rows, few outputs
]


@pytest.mark.parametrize("n,d_in,d_out", CASES)
@pytest.mark.parametrize("kind", ["int4", "int8", "asym"])
def test_small_tile_gemm_matches_oracle(kind, n, d_in, d_out):
    torch = torch_mod()
    say(f"{kind} n={n} d_in={d_in} d_out={d_out}")
    rng = np.random.default_rng(n + d_in + d_out)
    lim = 127 if kind == "int8" else 7
    qw = rng.integers(-lim, lim + 1, size=(d_out, d_in)).astype(np.int8)
    sx = rng.uniform(0.01, 1.0, n).astype(np.float32)
    sw = rng.uniform(0.01, 1.0, d_out).astype(np.float32)
    y = torch.full((n, d_out), float("nan"), dtype=torch.float32, device="cuda")
    acc = torch.full((n, d_out), -1, dtype=torch.int32, device="cuda")
    if kind == "asym":
        qx = rng.integers(0, 16, size=(n, d_in)).astype(np.int8)
        zmin = -rng.uniform(0.1, 2.0, n).astype(np.float32)
        rsum = qw.sum(1, dtype=np.int64).astype(np.int32)
        acc_or = qx.astype(np.float64) @ qw.astype(np.float64).T      # exact: below 2^53
        acc_or = acc_or.astype(np.int32)
        t1 = acc_or.astype(np.float32) * sx[:, None]
        t2 = zmin[:, None] * rsum.astype(np.float32)[None, :]
        y_or = (t1 + t2) * sw[None, :]
        args = (dev(o.pack_int4((qx - 8).astype(np.int8)), "u8"), dev(sx, "f32"), dev(zmin, "f32"),
                dev(o.pack_int4(qw), "u8"), dev(sw, "f32"), dev(rsum, "i32"))
        call = cat.cat_w4a4_linear_asym
    else:
        qx = rng.integers(-lim, lim + 1, size=(n, d_in)).astype(np.int8)
        acc_or = (qx.astype(np.float64) @ qw.astype(np.float64).T).astype(np.int32)
        y_or = acc_or.astype(np.float32) * sx[:, None] * sw[None, :]
        if kind == "int8":
            args = (dev(qx, "i8"), dev(sx, "f32"), dev(qw, "i8"), dev(sw, "f32"))
            call = cat.cat_int8_linear
        else:
            args = (dev(o.pack_int4(qx), "u8"), dev(sx, "f32"), dev(o.pack_int4(qw), "u8"),
                    dev(sw, "f32"))
            call = cat.cat_w4a4_linear
    call(*args, y, acc)
    assert np.array_equal(host(acc), acc_or)
    assert np.array_equal(host(y), y_or)
    y2 = torch.full((n, d_out), float("nan"), dtype=torch.float32, device="cuda")
    call(*args, y2)                                   # without the int32 sums
    assert np.array_equal(host(y2), y_or)
