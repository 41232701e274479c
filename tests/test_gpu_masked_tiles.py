"""Keys whose scores are -inf have weight zero, also where a whole tile, all keys of a wave or a whole shard have
none other.  The masked keys hold -inf in channel 0, where every query holds a positive value.  Reference:
float64 on the CPU; bounds of the parity tests."""

import pytest
import torch

from gpu_path import random_decode_inputs, random_prefill_inputs, run_prefill
from paper_2606_10537_amd._lib import PD_BF16, PD_FP32, Dims
from test_gpu_parity import assert_lse_close, assert_out_close
from test_gpu_static import run_compact

pytestmark = pytest.mark.gpu


def attend(q, k, v):
    """softmax(q k^T / sqrt(d)) v and its log-sum-exp in float64, [rows][H][d] operands, H_kv = H."""
    q, k, v = (x.double().cpu().transpose(0, 1) for x in (q, k, v))
    s = q @ k.transpose(1, 2) / q.shape[-1] ** 0.5
    return (torch.softmax(s, dim=-1) @ v).transpose(0, 1).numpy(), torch.logsumexp(s, dim=-1).numpy()


# dtype, d, masked keys of 656, shards asked for (0: chosen)
DECODE = [
    (PD_BF16, 128, [(64, 128)], 0), (PD_BF16, 64, [(64, 128)], 0),
    (PD_BF16, 128, [(0, 64), (576, 640)], 1), (PD_BF16, 64, [(0, 128)], 1),
    (PD_BF16, 128, [(0, 192)], 4),           # the first shard has no weight
    (PD_FP32, 128, [(32, 64)], 1), (PD_FP32, 64, [(96, 160), (512, 544)], 1),
    (PD_FP32, 64, [(0, 160)], 4), (PD_FP32, 128, [(64, 128)], 0),
]


@pytest.mark.parametrize("case", DECODE, ids=[str(c) for c in DECODE])
def test_decode_masked_keys(case):
    dtype, D, masked, S = case
    n_sel, Ld = 624, 32
    d = Dims(1, 1, 1, 4, 0, Ld, 2, 2, D, dtype, 0.0, 0, 1)
    scale = 0.125 if dtype == PD_FP32 else 1.0
    dec = random_decode_inputs(d, seed=D, scale=scale)
    pre = random_decode_inputs(Dims(1, 1, 1, 4, 0, n_sel, 2, 2, D, dtype), seed=7, scale=scale)
    dec["q_dec"][..., 0] = 0.5
    k = torch.cat([pre["k_dec"][0], dec["k_dec"][0]])
    for lo, hi in masked:
        k[lo:hi, :, 0] = float("-inf")
    ks = k[:n_sel].transpose(0, 1).contiguous()[None]
    vs = pre["v_dec"][0].transpose(0, 1).contiguous()[None]
    dec["k_dec"] = k[n_sel:].contiguous()[None]
    o, lse = run_compact(d, n_sel, dec, ks, vs, None, None, 0, S)
    torch.cuda.synchronize()
    ref, lref = attend(dec["q_dec"][0], k, torch.cat([pre["v_dec"][0], dec["v_dec"][0]]))
    assert_out_close(d, o[0].double().cpu().numpy(), ref, "o")
    kept = ~torch.isinf(k[:, 0, 0]).cpu()
    for h in range(2):
        assert_lse_close(d, lse[0, h].double().cpu().numpy(), lref[h], dec["q_dec"][0, :, h].double().cpu().numpy(),
                         k[:, h].double().cpu().numpy()[kept.numpy()], f"lse of head {h}")


@pytest.mark.parametrize("dtype,D", [(PD_BF16, 128), (PD_BF16, 64), (PD_FP32, 128), (PD_FP32, 64)])
def test_prefill_masked_keys(dtype, D):
    d = Dims(1, 1, 300, 19, 0, 4, 2, 2, D, dtype, 0.0, 0, 1)
    x = random_prefill_inputs(d, seed=D, scale=0.125 if dtype == PD_FP32 else 1.0)
    x["q_pre"][..., 0] = x["q_qm"][..., 0] = 0.5
    x["k_pre"][0, 0, :64, :, 0] = float("-inf")
    x["k_pre"][0, 0, 96:128, :, 0] = float("-inf")
    out = run_prefill(d, x)
    torch.cuda.synchronize()
    q, k, v = (torch.cat([x[t + "_pre"][0, 0], x[t + "_qm"][0]]) for t in "qkv")
    assert_out_close(d, out["o"][0, 0].double().cpu().numpy(), attend(q, k, v)[0], "o")
