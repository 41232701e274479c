"""The eight-wave sweep of the bf16 decode (d = 128, at least 16 tiles a shard, workgroups that fill the CUs) with
shards, grouped heads and a compact prefix, and calls just beside its rule, against the fp64 oracle with the
parity tests' bounds."""

import pytest
import torch

from gpu_path import random_decode_inputs, random_indices, random_prefill_inputs, run_decode
from paper_2606_10537_amd._lib import PD_BF16, Dims
from test_gpu_parity import decode_check
from test_gpu_static import run_compact, run_gather

pytestmark = pytest.mark.gpu

# B, N, C, Lq, Ld, Hq, Hkv, K, Bt, n_static, shards asked for; L_kv = K (1 + Bt) + n_static + Ld
CASES = [
    (4, 2, 1024, 60, 130, 32, 32, 2, 1000, 45, 2),   # 34 and a half tiles, 256 workgroups
    (4, 2, 1024, 60, 130, 32, 32, 2, 1000, 50, 2),   # 6 keys in the last tile of the last shard
    (4, 2, 1024, 60, 130, 32, 32, 2, 1000, 46, 2),   # 2
    (4, 3, 1024, 60, 200, 32, 32, 3, 700, 9, 0),     # more kept rows than one shard's table: shards chosen
    (1, 2, 128, 900, 1000, 32, 32, 2, 100, 900, 2),  # the second shard starts in the static rows
    (1, 2, 128, 300, 1100, 32, 32, 2, 40, 300, 2),   # and in the own rows
    (4, 2, 1024, 60, 64, 128, 32, 2, 1000, 45, 2),   # four heads of 64 rows
    (4, 2, 1024, 60, 128, 32, 32, 2, 1000, 45, 2),   # 128 rows: a half of the waves without rows
    (4, 2, 1024, 60, 128, 32, 32, 2, 1000, 45, 3),   # the same on more four-wave workgroups than CUs
    (4, 2, 1024, 60, 260, 32, 32, 2, 1000, 45, 2),   # 4 rows in the second tile of rows
    (4, 2, 1024, 60, 385, 32, 32, 2, 1000, 45, 2),   # 129
]


@pytest.mark.parametrize("case", CASES, ids=[str(c) for c in CASES])
def test_sharded_decode(case):
    B, N, C, Lq, Ld, Hq, Hkv, K, Bt, ns, S = case
    d = Dims(B, N, C, Lq, 0, Ld, Hq, Hkv, 128, PD_BF16)
    x = random_prefill_inputs(Dims(B, N, C, Lq, 0, Ld, 1, Hkv, 128, PD_BF16), seed=Ld + ns)
    cache = {"k_cache": x["k_pre"].transpose(2, 3).contiguous(), "v_cache": x["v_pre"].transpose(2, 3).contiguous()}
    dec = random_decode_inputs(d, seed=Ld)
    ci, ts = random_indices(d, K, Bt, seed=5)
    o, lse = run_decode(d, K, Bt, dec, cache, ci, ts, x["k_qm"], x["v_qm"], ns, num_splits=S)
    torch.cuda.synchronize()
    print(f"[sharded {case}] gathered decode done", flush=True)
    decode_check(d, K, Bt, dec, cache, ci, ts, x["k_qm"], x["v_qm"], ns, o, lse, heads=sorted({0, Hq - 1}),
                 batches=sorted({0, B - 1}))
    ks, vs = run_gather(d, K, Bt, cache, ci, ts)
    o2, lse2 = run_compact(d, K * (1 + Bt), dec, ks, vs, x["k_qm"], x["v_qm"], ns, S)
    torch.cuda.synchronize()
    assert torch.equal(o.cpu(), o2.cpu()) and torch.equal(lse.cpu(), lse2.cpu())
