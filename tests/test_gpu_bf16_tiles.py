"""bf16 decode at the edges of its tiles and of the rule that chooses its sweep: tiles that mix gathered,
static and own rows, one to three tiles, 32-row waves and 128-row workgroups without rows, and, with at least
16 tiles on workgroups that fill the CUs, the eight-wave sweep.  Checked against the fp64 oracle with the
parity tests' bounds."""

import pytest
import torch

from gpu_path import random_decode_inputs, random_indices, random_prefill_inputs, run_decode, run_prefill
from paper_2606_10537_amd._lib import PD_BF16, Dims
from test_gpu_parity import decode_check, prefill_units_check

pytestmark = pytest.mark.gpu

# B, N, C, Ld, Hq, Hkv, D, K, Bt, n_static, splits; L_kv = K (1 + Bt) + n_static + Ld
DECODE = [
    (1, 2, 64, 1, 1, 1, 128, 1, 1, 0, 1),          # 3 keys, one row
    (1, 2, 64, 31, 2, 1, 128, 1, 32, 0, 1),        # 64 keys, the tile mixes gathered and own rows
    (1, 2, 64, 33, 2, 1, 128, 1, 20, 11, 1),       # 65 keys: one in the second tile; three kinds in the first
    (1, 2, 64, 32, 4, 1, 64, 1, 63, 32, 1),        # regions cut exactly at the tile
    (1, 3, 128, 129, 2, 2, 128, 2, 100, 13, 1),    # 129 rows: a second workgroup with one row
    (1, 3, 128, 65, 4, 2, 64, 3, 128, 40, 3),      # shards that start inside the gathered rows
    (8, 2, 512, 17, 32, 32, 128, 2, 500, 5, 1),    # 256 workgroups, 1024 keys: eight waves, whole tiles
    (8, 2, 512, 18, 32, 32, 128, 2, 500, 5, 1),    # 1025 keys: one in the last tile
    (8, 2, 512, 50, 30, 30, 128, 2, 511, 9, 1),    # 240 workgroups, 17 tiles, 1 of 8 waves with 18 rows
    (8, 2, 512, 33, 32, 32, 128, 2, 500, 5, 1),    # 16 keys in the last tile of eight waves
    (8, 2, 512, 34, 32, 32, 128, 2, 500, 5, 1),    # 17
    (1, 2, 64, 40, 2, 1, 128, 1, 30, 9, 1),        # 80 keys: 16 in the last tile
    (1, 2, 64, 41, 2, 1, 64, 1, 30, 9, 1),         # 81
    (4, 2, 512, 260, 32, 32, 128, 2, 480, 0, 1),   # 256 rows and 4 more: two workgroups a head
]


@pytest.mark.parametrize("case", DECODE, ids=[str(c) for c in DECODE])
def test_decode_tiles(case):
    B, N, C, Ld, Hq, Hkv, D, K, Bt, ns, S = case
    d = Dims(B, N, C, 24, 16, Ld, Hq, Hkv, D, PD_BF16)
    x = random_prefill_inputs(d, seed=Ld + D)
    cache = {"k_cache": x["k_pre"].transpose(2, 3).contiguous(), "v_cache": x["v_pre"].transpose(2, 3).contiguous()}
    dec = random_decode_inputs(d, seed=Ld)
    ci, ts = random_indices(d, K, Bt, seed=5)
    o, lse = run_decode(d, K, Bt, dec, cache, ci, ts, x["k_qm"], x["v_qm"], ns, num_splits=S)
    torch.cuda.synchronize()
    decode_check(d, K, Bt, dec, cache, ci, ts, x["k_qm"], x["v_qm"], ns, o, lse, heads=sorted({0, Hq - 1}),
                 batches=sorted({0, B - 1}))


# C, Lq, Lm, D: chunk sequences of 1 + C + Lq + Lm rows
PREFILL = [(63, 1, 0, 128), (62, 1, 0, 64), (64, 63, 0, 128), (63, 64, 1, 64), (63, 16, 0, 128), (63, 10, 6, 64),
           (63, 17, 0, 128), (126, 1, 0, 128), (127, 1, 0, 128),
           (70, 190, 3, 64),
           # token scores with the keys of a head split: 4 blocks of 32 a workgroup, 1 in the last; two passes
           (513, 5, 0, 128), (300, 190, 3, 64)]


@pytest.mark.parametrize("case", PREFILL, ids=[str(c) for c in PREFILL])
def test_prefill_tiles(case):
    C, Lq, Lm, D = case
    d = Dims(1, 2, C, Lq, Lm, 4, 6, 2, D, PD_BF16)
    x = random_prefill_inputs(d, seed=C + D)
    out = run_prefill(d, x, chunk_score=True)
    torch.cuda.synchronize()
    prefill_units_check(d, x, out, [(0, 0), (0, 1)])
