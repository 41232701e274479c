"""fp32 attention at the edges of its tiles: 16- and 32-row query tiles, 32-key blocks dealt to the waves,
the 512-row address table, shards without a key for some waves.  Tolerance: the fp32 rule of the parity
tests (1e-5 absolute on outputs of N(0, 1/64) inputs)."""

import pytest
import torch

from gpu_path import random_decode_inputs, random_indices, random_prefill_inputs, run_decode, run_prefill
from paper_2606_10537_amd._lib import PD_FP32, Dims
from test_gpu_parity import decode_check, prefill_units_check

pytestmark = pytest.mark.gpu

# B, N, C, Lq, Lm, Hq, Hkv, D; S_c = 1 + C + Lq + Lm.  Heads * chunks * ceil(S_c / 32) >= 512 takes 32-row tiles.
PREFILL = [
    (1, 1, 13, 1, 0, 2, 1, 64),          # S_c = 15
    (1, 1, 14, 1, 1, 2, 1, 128),         # 17 rows, 17 content columns + query
    (1, 1, 494, 15, 2, 1, 1, 64),        # 512: the table exactly
    (1, 1, 494, 15, 3, 1, 1, 128),       # 513: one key in the second table
    (1, 1, 250, 5, 1, 2, 2, 64),         # 257 = 8 waves * 32 + 1
    (1, 8, 240, 10, 6, 8, 2, 64),        # 32-row tiles, 257 rows
    (2, 8, 112, 8, 7, 8, 4, 128),        # 32-row tiles, 128 rows: every wave one block
]


@pytest.mark.parametrize("case", PREFILL, ids=[str(c) for c in PREFILL])
def test_prefill_tiles(case):
    B, N, C, Lq, Lm, Hq, Hkv, D = case
    d = Dims(B, N, C, Lq, Lm, 4, Hq, Hkv, D, PD_FP32)
    x = random_prefill_inputs(d, seed=C + D, scale=0.125)
    out = run_prefill(d, x)
    torch.cuda.synchronize()
    prefill_units_check(d, x, out, [(0, 0), (B - 1, N - 1)])


# B, Ld, Hq, Hkv, D, K, Bt, n_static, splits; 512 or more (sequence, KV head, shard, 32-row tile) take 32-row tiles.
DECODE = [
    (1, 1, 1, 1, 64, 1, 1, 0, 1),        # 3 keys
    (1, 16, 2, 1, 128, 1, 12, 3, 1),     # 32 keys, 32 rows in two tiles
    (1, 17, 1, 1, 128, 2, 100, 0, 5),    # 219 keys in 5 shards
    (2, 33, 4, 2, 64, 3, 120, 16, 1),    # 412 keys, tiles crossing a head
    (1, 40, 2, 2, 128, 4, 128, 0, 2),    # 556 keys: shards of 288 and 268
    (16, 64, 16, 8, 64, 2, 60, 7, 1),    # 32-row tiles
    (16, 50, 16, 8, 128, 4, 128, 16, 1), # 32-row tiles, 582 keys: two tables
]


@pytest.mark.parametrize("case", DECODE, ids=[str(c) for c in DECODE])
def test_decode_tiles(case):
    B, Ld, Hq, Hkv, D, K, Bt, ns, S = case
    d = Dims(B, 4, 128, 12, 4, Ld, Hq, Hkv, D, PD_FP32)
    x = random_prefill_inputs(d, seed=Ld + D, scale=0.125)
    cache = run_prefill(d, x)
    dec = random_decode_inputs(d, seed=Ld, scale=0.125)
    ci, ts = random_indices(d, K, Bt, seed=5)
    o, lse = run_decode(d, K, Bt, dec, cache, ci, ts, x["k_qm"], x["v_qm"], ns, num_splits=S)
    torch.cuda.synchronize()
    decode_check(d, K, Bt, dec, cache, ci, ts, x["k_qm"], x["v_qm"], ns, o, lse, batches=[0, B - 1])


@pytest.mark.parametrize("C", [1, 63, 1024, 1025, 2049, 4096])
def test_rank_sort_sizes(C):
    """Token ranks where the sort's threads hold one, two and four keys."""
    d = Dims(1, 2, C, 3, 2, 4, 2, 1, 64, PD_FP32)
    out = run_prefill(d, random_prefill_inputs(d, seed=C, scale=0.125), chunk_score=True)
    torch.cuda.synchronize()
    e, rank = out["tok_score"].cpu(), out["tok_rank"].cpu().long()
    order = torch.sort(e, dim=2, descending=True, stable=True)[1]
    want = torch.empty_like(order).scatter_(2, order, torch.arange(C).expand(1, 2, C).contiguous())
    assert torch.equal(rank, want)
