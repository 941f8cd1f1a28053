"""Fused full-dimension Hadamard transform+quant (z of whole rows held in
registers) against the CPU oracle, over its block counts, block sizes and
token groups, with ragged last workgroups."""
import numpy as np
import pytest

from oracle import cat_oracle as o

from gpu_common import say
from test_gpu_full_hadamard import _check_full, _tq_full

pytestmark = pytest.mark.gpu


# the token counts are ones the launcher takes the fused kernel for on a
# 256-CU device: 16 tokens per workgroup, or 32 from 8192 tokens on
@pytest.mark.parametrize("d,k,n", [
    (256, 128, 1), (512, 128, 50), (1024, 128, 33), (2048, 128, 1000), (3584, 128, 700), (4096, 128, 1001),
    (512, 256, 17), (1024, 256, 33), (2048, 256, 1500), (4096, 256, 4001),
    (1024, 128, 8193), (2048, 128, 8200), (2048, 256, 8193),
])
def test_fused_full_hadamard_matches_oracle(d, k, n):
    say(f"tq full fused d={d} k={k} (m={d // k}) n={n}")
    rng = np.random.default_rng(d + k + n)
    X = o.round_storage((rng.standard_normal((n, d)) * np.exp(rng.standard_normal(d))).astype(np.float32), "bf16")
    X[n // 2] = 0.0
    T = o.round_storage(rng.standard_normal((d // k, k, k)) / np.sqrt(k), "bf16")
    q, s = _tq_full(X, T, k)
    _check_full(q, s, X, T, k, f"d={d} k={k}")
    assert s[n // 2] == 0 and not q[n // 2].any()
