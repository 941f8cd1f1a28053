"""Integer GEMMs at sizes that a 256-CU device runs on the 128- and 256-token
tiles (smaller ones take the small tiles): epilogues with scales across the
fp32 range, the longest rows with the largest sums, a last 128-token panel of
one row, and calls with and without the int32 sums."""
import numpy as np
import pytest

import paper_2603_04359_amd as cat
import workloads as wl
from oracle import cat_oracle as o
from paper_2603_04359_amd import binding as B

from gpu_common import check_tile_rows, dev, host, say, torch_mod

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("int8", [False, True])
@pytest.mark.parametrize("n,d_in,d_out,with_acc,rows", [
    (1921, 4160, 3000, True, 128),     # ragged outputs and K, one row in the last panel
    (1921, 4128, 4001, False, 128),    # one output in the last tile
    (2048, 1024, 4096, False, 128),    # full tiles: the store path without the sums
    (4097, 160, 4100, True, 256),
    (4352, 96, 4096, False, 256),      # full 256-token tiles without the sums
])
def test_large_tiles_scales_across_the_fp32_range(n, d_in, d_out, with_acc, rows, int8):
    # y~ = fl(fl(acc) s_x) s_w runs into subnormal and infinite values, which
    # the epilogue rounds as IEEE fp32 does, bit for bit
    say(f"large tiles n={n} d_in={d_in} d_out={d_out} acc={with_acc} int8={int8}")
    check_tile_rows(n, d_out, rows)
    torch = torch_mod()
    rng = np.random.default_rng(n + d_out + int8)
    sx = np.exp(rng.uniform(np.log(1e-30), np.log(1e30), n)).astype(np.float32)
    sw = np.exp(rng.uniform(np.log(1e-30), np.log(1e30), d_out)).astype(np.float32)
    sx[rng.random(n) < 0.05] = 0.0
    qmax = 127 if int8 else 7
    qx, qw = wl.random_codes(n, d_in, n + 1, qmax=qmax), wl.random_codes(d_out, d_in, n + 2, qmax=qmax)
    acc_or = (qx.astype(np.float32) @ qw.astype(np.float32).T if d_in * qmax * qmax < 1 << 24
              else qx.astype(np.float64) @ qw.astype(np.float64).T).astype(np.int32)      # exact either way
    with np.errstate(over="ignore"):
        y_or = (acc_or.astype(np.float32) * sx[:, None]) * sw[None, :]
    assert np.isinf(y_or).any() and ((y_or != 0) & (np.abs(y_or) < np.finfo(np.float32).tiny)).any()
    y = torch.full((n, d_out), 5.0, dtype=torch.float32, device="cuda")
    acc = torch.full((n, d_out), -1, dtype=torch.int32, device="cuda") if with_acc else None
    if int8:
        cat.cat_int8_linear(dev(qx, "i8"), dev(sx, "f32"), dev(qw, "i8"), dev(sw, "f32"), y, acc)
    else:
        cat.cat_w4a4_linear(dev(o.pack_int4(qx), "u8"), dev(sx, "f32"), dev(o.pack_int4(qw), "u8"),
                            dev(sw, "f32"), y, acc)
    assert np.array_equal(host(y), y_or)
    if with_acc:
        assert np.array_equal(host(acc), acc_or)


@pytest.mark.parametrize("kind", ["int4", "int8", "asym"])
def test_large_tiles_extreme_codes_at_max_d_in(kind):
    # rows of all +-qmax over the longest reduction: sums of +-qmax^2 d_in
    torch = torch_mod()
    n, d_in, d_out = 2048, B.CAT_MAX_D_IN, 4096
    say(f"large tiles {kind} extreme codes d_in={d_in}")
    check_tile_rows(n, d_out, 128)
    q = 127 if kind == "int8" else 7
    byte = lambda v: v if kind == "int8" else (v & 0xF) | (v & 0xF) << 4
    sign_x = torch.where(torch.arange(n, device="cuda") % 3 == 1, -1, 1)
    sign_w = torch.where(torch.arange(d_out, device="cuda") % 5 == 2, -1, 1)

    def rows(sign, lo, hi):
        t = torch.where(sign[:, None] > 0, byte(hi), byte(lo)).to(torch.int8 if kind == "int8" else torch.uint8)
        return t.expand(-1, d_in if kind == "int8" else d_in // 2).contiguous()

    cw = rows(sign_w, -q, q)
    sx, sw = torch.ones(n, device="cuda"), torch.ones(d_out, device="cuda")
    y = torch.empty((n, d_out), dtype=torch.float32, device="cuda")
    acc = torch.empty((n, d_out), dtype=torch.int32, device="cuda")
    ref = sign_x[:, None] * sign_w[None, :] * (q * q * d_in)
    if kind == "asym":
        # codes 0 and 15, stored less 8; sums of 0 or +-15 * 7 d_in
        cx = rows(sign_x, -8, 7)
        ref = (sign_x[:, None] > 0) * sign_w[None, :] * (15 * q * d_in)
        cat.cat_w4a4_linear_asym(cx, sx, torch.zeros(n, device="cuda"), cw, sw,
                                 (sign_w * (q * d_in)).to(torch.int32), y, acc)
    else:
        (cat.cat_int8_linear if kind == "int8" else cat.cat_w4a4_linear)(rows(sign_x, -q, q), sx, cw, sw, y, acc)
    assert torch.equal(acc.long(), ref)
    assert torch.equal(y, ref.float())
