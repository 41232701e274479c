"""Attention whose logits spread over more than +-100: tiles, the waves of an fp32 workgroup, its two address tables
and the shards hold very different maxima, so that rescaling and merging decide the result, and exp2 of a plain
logit overflows.  One key can be planted 60 above the others in the first, a middle or the last block of 32 keys, or
beyond the 512 keys of the first table.  Reference: float64 on the CPU.

Bounds: a logit is a sum of d products of magnitude sum |q k| / sqrt(d), 220 here, rounded to 24 bits each,
which adds up like sqrt(d) 2^-24 220 = 1.5e-4 at most; a weight has that relative error, and the weights that multiply V
in bf16 another 2^-8.  V has standard deviation 1/64 in fp32 and 1/4 in bf16, so the 1e-5 and 1e-2 of the parity
tests hold for the outputs, 2e-4 (bf16: + ln(1 + 2^-8)) for the LSE and 2e-4, relative, for the token scores."""

import pytest
import torch

from gpu_path import random_decode_inputs, random_prefill_inputs, run_prefill
from paper_2606_10537_amd._lib import PD_BF16, PD_FP32, Dims
from test_gpu_static import run_compact

pytestmark = pytest.mark.gpu

SIGMA = 5.5     # of Q and K elements: logits of standard deviation 30
V_SIGMA = {PD_FP32: 1 / 64, PD_BF16: 1 / 4}
O_TOL = {PD_FP32: 1e-5, PD_BF16: 1e-2}
LSE_TOL = {PD_FP32: 2e-4, PD_BF16: 2e-4 + 2.0 ** -8}


def plant(q, k, key):
    """Adds 60 to the logits of one key row of every head: channel 0 is 1 in Q, 0 in the other keys."""
    q[..., 0] = 1.0
    k[..., 0] = 0.0
    k[key, :, 0] = 60.0 * q.shape[-1] ** 0.5


def attend(q, k, v):
    """[rows][H][d] queries, [keys][H][d] keys: outputs [rows][H][d], LSE [H][rows], weights [H][rows][keys]."""
    q, k, v = (x.double().cpu().transpose(0, 1) for x in (q, k, v))
    s = q @ k.transpose(1, 2) / q.shape[-1] ** 0.5
    assert s.max() > 100 and s.min() < -100
    p = torch.softmax(s, dim=-1)
    return (p @ v).transpose(0, 1), torch.logsumexp(s, dim=-1), p


# dtype, B, H, Ld, d, shards; in fp32 16 * 16 heads of 64 rows take 32-row tiles
@pytest.mark.parametrize("key", [None, 3, 333, 600, 715])
@pytest.mark.parametrize("case", [
    (PD_FP32, 1, 2, 17, 64, 1), (PD_FP32, 1, 2, 17, 128, 1), (PD_FP32, 1, 2, 17, 128, 5), (PD_FP32, 16, 16, 64, 64, 1),
    (PD_FP32, 16, 16, 64, 128, 1), (PD_BF16, 1, 2, 40, 64, 1), (PD_BF16, 1, 2, 40, 128, 1), (PD_BF16, 1, 2, 40, 128, 5),
    (PD_BF16, 8, 32, 130, 128, 1),   # eight waves: 1024 keys and more
], ids=str)
def test_decode_large_logits(case, key):
    dtype, B, H, Ld, D, S = case
    n_sel = (1100 if Ld == 130 else 720) - Ld
    d = Dims(B, 1, 1, 4, 0, Ld, H, H, D, dtype, 0.0, 0, 1)
    dec = random_decode_inputs(d, seed=Ld + D, scale=SIGMA)
    pre = random_decode_inputs(Dims(B, 1, 1, 4, 0, n_sel, H, H, D, dtype), seed=7, scale=SIGMA)
    dec["v_dec"] *= V_SIGMA[dtype] / SIGMA
    pre["v_dec"] *= V_SIGMA[dtype] / SIGMA
    k = torch.cat([pre["k_dec"], dec["k_dec"]], dim=1)
    if key is not None:
        for b in range(B):
            plant(dec["q_dec"][b], k[b], key)
    dec["k_dec"] = k[:, n_sel:].contiguous()
    ks, vs = k[:, :n_sel].transpose(1, 2).contiguous(), pre["v_dec"].transpose(1, 2).contiguous()
    o, lse = run_compact(d, n_sel, dec, ks, vs, None, None, 0, S)
    torch.cuda.synchronize()
    for b in sorted({0, B - 1}):
        ref, lref, _ = attend(dec["q_dec"][b], k[b], torch.cat([pre["v_dec"][b], dec["v_dec"][b]]))
        assert (o[b].double().cpu() - ref).abs().max() <= O_TOL[dtype]
        assert (lse[b].double().cpu() - lref).abs().max() <= LSE_TOL[dtype]


# dtype, B, N, H, d; in fp32 2 * 4 * 4 heads of 731 rows take 32-row tiles
@pytest.mark.parametrize("key", [None, 3, 333, 600, 715])
@pytest.mark.parametrize("case", [(PD_FP32, 1, 1, 2, 64), (PD_FP32, 1, 1, 2, 128), (PD_FP32, 2, 4, 4, 64),
                                  (PD_FP32, 2, 4, 4, 128), (PD_BF16, 1, 1, 2, 64), (PD_BF16, 1, 1, 2, 128)], ids=str)
def test_prefill_large_logits(case, key):
    dtype, B, N, H, D = case
    C, Lq = 710, 20
    d = Dims(B, N, C, Lq, 0, 4, H, H, D, dtype, 0.0, 0, 1)
    x = random_prefill_inputs(d, seed=D, scale=SIGMA)
    for t in ("v_pre", "v_qm"):
        x[t] *= V_SIGMA[dtype] / SIGMA
    if key is not None:
        x["q_pre"][..., 0] = x["q_qm"][..., 0] = 1.0
        x["k_pre"][..., 0] = x["k_qm"][..., 0] = 0.0
        at = x["k_pre"][:, :, key] if key <= C else x["k_qm"][:, key - 1 - C]
        at[..., 0] = 60.0 * D ** 0.5
    out = run_prefill(d, x)
    torch.cuda.synchronize()
    for b, n in sorted({(0, 0), (B - 1, N - 1)}):
        q, k, v = (torch.cat([x[t + "_pre"][b, n], x[t + "_qm"][b]]) for t in "qkv")
        ref, _, p = attend(q, k, v)
        assert (out["o"][b, n].double().cpu() - ref).abs().max() <= O_TOL[dtype]
        e = p[:, 1 + C:, 1:1 + C].sum(dim=(0, 1)) + p[:, 1:1 + C, 1 + C:].sum(dim=(0, 2))
        assert ((out["tok_score"][b, n].double().cpu() - e).abs() <= 2e-4 * e + 1e-7).all()
