"""bf16 two-pass transform+quant of blocks of 128, 256 and 512 (256 output rows
per workgroup) against the CPU oracle: one tile and several per workgroup (odd
and even counts), ragged last tiles, every code width, and the few-token calls
at k = 512 that stay on the ring kernel."""
import numpy as np
import pytest

import paper_2603_04359_amd as cat
from oracle import cat_oracle as o

from gpu_common import dev, host, say, torch_mod
from test_gpu_asym import _check_asym, _tq_asym

pytestmark = pytest.mark.gpu

# tiles are 64 tokens; on a 256-CU device d = 14336 gives 4 tile rows (k <= 256)
# or 4 (k = 512), d = 7680 8, d = 256 one per CU
CASES = [
    (256, 128, 1), (768, 128, 64), (14336, 128, 65), (14336, 128, 64 * 9 + 1),     # 2 and 3 tiles
    (256, 256, 63), (14336, 256, 64 * 4), (14336, 256, 64 * 8 + 3), (14336, 256, 64 * 13),
    (7680, 512, 140), (14336, 512, 64 * 9 + 2), (14336, 512, 64 * 16), (14336, 512, 200),
    (1024, 512, 1024), (1024, 512, 1025),       # the last few-token size and the first beyond
]


def _inputs(d, k, n):
    rng = np.random.default_rng(d + k + n)
    X = o.round_storage(rng.standard_normal((n, d)) * np.exp(rng.standard_normal(d)), "bf16")
    X[n // 2] = 0.0
    return X, o.round_storage(rng.standard_normal((d // k, k, k)) / np.sqrt(k), "bf16")


def _check_codes(codes, X, T, bits, label):
    """A code may differ from the oracle's by one where its multiplier u = z
    qmax / amax is nearer to a half-integer than fp32 resolves: z is an fp32
    sum of k exact products, so off by at most k 2^-24 sum |T_ji x_i|, and
    amax, its inverse and the product round once more each (with amax itself
    off by its own sum's error).  Such ties are rare and independent: with a
    share of 1e-6 qmax / 7 expected at most, their count stays within mu + 4
    sqrt(mu) + 3 of that Poisson mean mu (a miss below 1e-4 a case)."""
    q_or, s_or = o.transform_quant(X, T, bits)
    q = o.unpack_int4(codes) if bits == 4 else np.asarray(codes).view(np.int8)
    bad = np.argwhere(q != q_or)
    nb, k, _ = T.shape
    qmax = o.qmax_of(bits)
    Z = o.transform_rows(X, T)
    for t, c in bad:
        b, j = divmod(c, k)
        amax = np.abs(Z[t]).max()
        jm = int(np.abs(Z[t]).argmax())
        terms = lambda ch: np.abs(T[ch // k, ch % k] * X[t, ch // k * k:ch // k * k + k]).sum()
        u = abs(Z[t, c] * qmax / amax)
        err = 2.0 ** -24 * (k * terms(c) * qmax / amax + u * (k * terms(jm) / amax + 4))
        assert abs(int(q[t, c]) - int(q_or[t, c])) == 1 and abs(u - np.floor(u) - 0.5) <= err, (
            f"{label}: code at token {t}, channel {c}: {q[t, c]} against {q_or[t, c]}, u = {u}")
    mu = 1e-6 * qmax / 7.0 * q.size
    assert len(bad) <= mu + 4 * np.sqrt(mu) + 3, f"{label}: {len(bad)} differ"
    say(f"  {label}: codes {q.size}, tie mismatches {len(bad)}")
    return s_or


@pytest.mark.parametrize("d,k,n", CASES)
def test_wide_two_pass_symmetric(d, k, n):
    torch = torch_mod()
    bits = (4, 8, 6)[(n + d // 256) % 3]
    say(f"tq wide d={d} k={k} n={n} bits={bits}")
    X, T = _inputs(d, k, n)
    codes = torch.full((n, d // 2 if bits == 4 else d), 77, device="cuda",
                       dtype=torch.uint8 if bits == 4 else torch.int8)
    s_x = torch.full((n,), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(cat.cat_transform_quant_workspace_bytes(n, d, k), dtype=torch.uint8, device="cuda")
    cat.cat_transform_quant(dev(X, "bf16"), dev(T, "bf16"), k, codes, s_x, ws, bits=bits)
    got = host(codes)
    s_or = _check_codes(got, X, T, bits, f"d={d} k={k} n={n}")
    s = host(s_x).astype(np.float64)
    assert np.all(np.abs(s - s_or) <= 1e-6 * s_or)       # as the other bf16 kernels
    assert s[n // 2] == 0 and not got[n // 2].any()


@pytest.mark.parametrize("d,k,n", CASES[1:-2:2])
def test_wide_two_pass_asymmetric(d, k, n):
    say(f"tq wide asym d={d} k={k} n={n}")
    X, T = _inputs(d, k, n)
    q, s, m = _tq_asym(X, T, k, "bf16", "bf16")
    _check_asym(q, s, m, X, T, f"asym d={d} k={k} n={n}")
    assert s[n // 2] == 0 and m[n // 2] == 0 and not q[n // 2].any()


# n tokens in one tile per workgroup (two up to d = 2048; row words in slots)
# or in two or three (row words cleared and folded) against the same tokens at
# the front of a call with more;
# on a 256-CU device R = 64 tile rows at d = 1024, 4 at 14336, 8 at 7680 (k = 512)
@pytest.mark.parametrize("asym", [False, True])
@pytest.mark.parametrize("d,k,n,more", [(14336, 256, 64 * 8, 600), (14336, 128, 449, 600), (14336, 256, 1, 600),
                                        (1024, 256, 64 * 128, 64 * 128 + 1), (7680, 512, 64 * 16 - 5, 1100),
                                        (768, 128, 3, 64 * 200), (14336, 512, 260, 530)])
def test_wide_two_pass_slots_equal_folded_words(d, k, n, more, asym):
    torch = torch_mod()
    say(f"tq wide slots d={d} k={k} n={n} asym={asym}")
    X, T = _inputs(d, k, more)
    X[0, :5] = np.inf, -np.inf, 1.0, -1.0, 2.0 ** 127
    Xd, Td = dev(X, "bf16"), dev(T, "bf16")
    res = []
    for m in (n, more):
        codes = torch.full((m, d // 2), 77, device="cuda", dtype=torch.uint8)
        s_x, zmin = (torch.full((m,), 5.0, dtype=torch.float32, device="cuda") for _ in range(2))
        size = cat.cat_transform_quant_asym_workspace_bytes if asym else cat.cat_transform_quant_workspace_bytes
        ws = torch.full((size(m, d, k),), 0xFF, dtype=torch.uint8, device="cuda")     # no clean workspace needed
        for _ in range(2):
            if asym:
                cat.cat_transform_quant_asym(Xd[:m], Td, k, codes, s_x, zmin, ws)
            else:
                cat.cat_transform_quant(Xd[:m], Td, k, codes, s_x, ws)
        res.append([host(t[:n]).view(np.uint8) for t in (codes, s_x, zmin)])
    for a, b in zip(*res):
        assert np.array_equal(a, b)
