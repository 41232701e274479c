"""A query row with a NaN, an infinite or an overflowing score leaves every other row of a bf16 call as it is,
bit for bit: decode (four and eight waves, d = 64 and 128, one head per KV head and several) and prefill."""

import pytest
import torch

from gpu_path import random_decode_inputs, random_indices, random_prefill_inputs, run_decode, run_prefill
from paper_2606_10537_amd._lib import PD_BF16, Dims

pytestmark = pytest.mark.gpu

POISON = {"nan": float("nan"), "inf": float("inf"), "overflow": 3e38}


def same_but(a, b, rows):
    """a and b (leading axes indexed by `rows`) hold the same bits everywhere else."""
    a, b = a.clone(), b.clone()
    for r in rows:
        a[r] = 0
        b[r] = 0
    assert torch.equal(a.cpu(), b.cpu())


# B, Ld, Hq, Hkv, D, C, Bt, n_static; two chunks kept
DECODE = [
    (1, 40, 2, 2, 128, 64, 40, 9),       # 32-row wave and one of 8 rows
    (2, 24, 8, 2, 64, 200, 150, 16),     # four heads share a wave's rows
    (2, 24, 8, 2, 128, 200, 150, 16),
    (8, 130, 32, 32, 128, 512, 500, 5),  # eight waves
]


@pytest.mark.parametrize("kind", POISON)
@pytest.mark.parametrize("case", DECODE, ids=[str(c) for c in DECODE])
def test_decode_row_stays_alone(case, kind):
    B, Ld, Hq, Hkv, D, C, Bt, ns = case
    d = Dims(B, 2, C, 12, 4, Ld, Hq, Hkv, D, PD_BF16)
    x = random_prefill_inputs(d, seed=3)
    cache = {"k_cache": x["k_pre"].transpose(2, 3).contiguous(), "v_cache": x["v_pre"].transpose(2, 3).contiguous()}
    dec = random_decode_inputs(d, seed=4)
    ci, ts = random_indices(d, 2, Bt, seed=5)
    run = lambda: run_decode(d, 2, Bt, dec, cache, ci, ts, x["k_qm"], x["v_qm"], ns, num_splits=1)
    o, lse = run()
    rows = [(0, 0, 0), (B - 1, 17, Hq - 1), (0, Ld - 1, Hq // 2)]
    for b, r, h in rows:
        dec["q_dec"][b, r, h, 3] = POISON[kind]
    o2, lse2 = run()
    torch.cuda.synchronize()
    assert torch.isfinite(o.float()).all()
    same_but(o, o2, rows)
    same_but(lse, lse2, [(b, h, r) for b, r, h in rows])
    if kind == "nan":
        for r in rows:
            assert torch.isnan(o2[r].float()).all()


@pytest.mark.parametrize("kind", POISON)
@pytest.mark.parametrize("D", [64, 128])
def test_prefill_row_stays_alone(D, kind):
    d = Dims(1, 2, 200, 12, 9, 4, 4, 2, D, PD_BF16)
    x = random_prefill_inputs(d, seed=D)
    out = run_prefill(d, x)
    x["q_pre"][0, 1, 60, 2, 3] = POISON[kind]   # content row 60 of chunk 1
    x["q_qm"][0, 20, 1, 3] = POISON[kind]       # the last pseudo-label row, in both chunks
    out2 = run_prefill(d, x)
    torch.cuda.synchronize()
    assert torch.isfinite(out["o"].float()).all()
    same_but(out["o"], out2["o"], [(0, 1, 60, 2), (0, 0, d.seq_len - 1, 1), (0, 1, d.seq_len - 1, 1)])
    same_but(out["tok_score"], out2["tok_score"], [(0, 1, 59)])
    for t in ("k_cache", "v_cache", "key_mean"):
        assert torch.equal(out[t], out2[t])
