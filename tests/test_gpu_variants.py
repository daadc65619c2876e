"""Kernel variants that the dispatch picks by size or geometry, at the sizes where each can go
wrong (tile edges, remainders, the smallest call), against the fp64 oracle."""

import pytest

from test_gpu_prefill import _prefill_case

pytestmark = pytest.mark.gpu


# 8 query heads per KV head on MFMA: a q-tile is 32 rows at head_dim 64 / 128 and two sets of 4
# heads by 32 rows at 256.
GROUP8_CASES = [
    # dtype, D, Hq, Hkv, ctx_lens, chunk, q sigma_log2, needle divisor, windows
    ("bf16", 64, 8, 1, [0, 63], 33, -1, 0, (0, 0)),
    ("bf16", 128, 16, 2, [64, 5], 1, -1, 0, (0, 40)),
    ("bf16", 128, 8, 1, [130], 97, 2, 2, (0,)),            # harsh needles
    ("bf16", 256, 16, 2, [0, 500], 65, -1, 0, (0, 100)),
    ("bf16", 256, 8, 1, [77], 31, 2, 2, (0,)),
    ("fp8", 256, 8, 1, [64], 32, -1, 0, (0,)),
    ("fp8", 128, 16, 2, [0, 31], 64, -1, 0, (0, 33)),
    ("fp8", 64, 8, 1, [200], 5, -1, 0, (0,)),
    # several 512-key segments: boundaries inside the chunk, windows starting inside a segment
    ("bf16", 128, 8, 1, [1023, 511], 2, -1, 0, (0, 600)),
    ("bf16", 256, 8, 1, [1100], 40, -1, 0, (0, 513)),
]


@pytest.mark.parametrize("dtype,D,Hq,Hkv,ctxs,chunk,qsig,div,windows", GROUP8_CASES)
def test_group8_prefill(dtype, D, Hq, Hkv, ctxs, chunk, qsig, div, windows):
    _prefill_case(dtype, D, Hq, Hkv, ctxs, chunk, qsig, windows, div)
