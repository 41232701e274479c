"""The shard counts that the library chooses for a decode (pd_decode_splits, on the CPU) and that its workspace
sizes follow them."""

import pytest

from paper_2606_10537_amd import _lib
from paper_2606_10537_amd._lib import PD_BF16, Dims

# B, Hq, Hkv, Ld, d, K, Bt -> shards
CASES = [
    ((1, 32, 32, 256, 128, 2, 512), 4),      # 64 tiles of 128 rows: one workgroup a CU
    ((1, 28, 4, 256, 128, 4, 256), 4),
    ((1, 32, 8, 32, 128, 4, 1024), 17),      # 2 sqrt(tiles)
    ((8, 32, 32, 512, 128, 4, 256), 1),
    ((4, 32, 32, 512, 128, 4, 256), 1),
    ((2, 32, 32, 256, 128, 4, 1000), 4),     # eight waves: 64 tiles of 256 rows, 66 tiles of keys
    ((1, 64, 64, 256, 128, 4, 1000), 4),
    ((2, 32, 32, 256, 64, 4, 1000), 3),      # four waves only at d = 64; 3 shards fit the row table
    ((2, 32, 32, 128, 128, 4, 1000), 4),     # 64 tiles of 128 rows
    ((1, 32, 32, 256, 128, 4, 1000), 4),     # 8 shards of eight waves would be too short
    ((1, 4, 4, 40, 128, 2, 100), 1),         # under 8 tiles of keys
]


@pytest.mark.parametrize("case,want", CASES, ids=[str(c[0]) for c in CASES])
def test_chosen_shards(case, want):
    B, Hq, Hkv, Ld, D, K, Bt = case
    d = Dims(B, 32, 1024, 64, 64, Ld, Hq, Hkv, D, PD_BF16)
    assert _lib.pd_decode_splits(d, K, Bt, 64) == want
    rows = want * B * Hq * Ld
    up = lambda x: (x + 255) // 256 * 256
    assert _lib.pd_workspace_bytes(d, K, Bt, 0, 2) == (up(rows * D * 4) + up(rows * 4) if want > 1 else 0)
