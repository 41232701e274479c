"""Ranks, selection and merge where their kernels change over: 64 and 65 chunks, one token and 4096 (one and 16
a thread), all and one kept, equal scores, few and many chunks, numbers of terms and shards around the batches.
Whole numbers are compared exactly."""

import numpy as np
import pytest
import torch

import oracle
from gpu_path import random_decode_inputs, random_indices, random_prefill_inputs, run_decode, run_prefill, run_select
from paper_2606_10537_amd import _lib
from paper_2606_10537_amd._lib import PD_BF16, PD_FP32, Dims
from test_gpu_parity import decode_check, prefill_units_check

pytestmark = pytest.mark.gpu

# B, N, C, K, Bt
CASES = [(1, 1, 1, 1, 1), (2, 63, 17, 63, 5), (3, 64, 256, 1, 256), (2, 64, 257, 64, 1), (2, 65, 257, 65, 100),
         (1, 65, 40, 2, 40), (1, 4, 4096, 3, 4095), (2, 3, 1025, 2, 511)]


@pytest.mark.parametrize("lowest", [0, 1])
@pytest.mark.parametrize("case", CASES, ids=[str(c) for c in CASES])
def test_select_ranked_edges(case, lowest):
    B, N, C, K, Bt = case
    d = Dims(B, N, C, 4, 0, 8, 2, 1, 64, PD_FP32)
    g = torch.Generator().manual_seed(N * C)
    # Scores in steps of 1/4: many equal ones, the lower index first.
    s = torch.randint(-6, 7, (B, N), generator=g).float() / 4
    rank = torch.argsort(torch.rand((B, N, C), generator=g), dim=2).to(torch.int32)
    ci = torch.full((B, K), -1, dtype=torch.int32, device="cuda")
    ts = torch.full((B, K, Bt), -1, dtype=torch.int32, device="cuda")
    _lib.pd_select_ranked(d, K, Bt, s.cuda(), lowest, rank.cuda(), ci, ts)
    torch.cuda.synchronize()
    order = np.argsort(s.numpy() if lowest else -s.numpy(), axis=1, kind="stable")
    want = np.sort(order[:, :K], axis=1)
    assert np.array_equal(ci.cpu().numpy(), want)
    assert np.array_equal(ts.cpu().numpy(), oracle.tokens_by_rank_ref(rank.numpy(), want, Bt))


@pytest.mark.parametrize("N", [64, 65])
def test_score_select_both_kernels(N):
    """The same sequence's chunks with and without one more: the scores and the kept sets agree."""
    d = Dims(2, N, 33, 4, 0, 40, 4, 2, 64, PD_FP32)
    g = torch.Generator().manual_seed(9)
    q = torch.randn((2, 40, 4, 64), generator=g).cuda()
    km = torch.randn((2, 65, 2, 64), generator=g)
    km[:, 64] = -km[:, :64].mean(dim=1)
    rank = torch.argsort(torch.rand((2, 65, 33), generator=g), dim=2).to(torch.int32)
    ci, ts, cs = run_select(d, 5, 9, q, km[:, :N].contiguous().cuda(), rank[:, :N].contiguous().cuda())
    torch.cuda.synchronize()
    ref = oracle.chunk_scores_ref(q.cpu().double().numpy(), km[:, :N].double().numpy())
    np.testing.assert_allclose(cs.cpu().double().numpy(), ref, rtol=1e-5, atol=1e-5)
    want = np.sort(np.argsort(-ref, axis=1, kind="stable")[:, :5], axis=1)
    assert np.array_equal(ci.cpu().numpy(), want)
    assert np.array_equal(ts.cpu().numpy(), oracle.tokens_by_rank_ref(rank[:, :N].numpy(), want, 9))


# C, N: at most 512 workgroups of 64 tokens count the ranks, more chunks sort them
@pytest.mark.parametrize("C,N", [(1, 2), (64, 2), (65, 2), (1000, 2), (1025, 2), (4096, 2), (1, 513), (64, 513), (65, 257),
                                 (1000, 33), (1025, 31), (4096, 9)])
def test_rank_both_kernels(C, N):
    """Ranks are those of a stable descending sort of the scores written beside them, with equal scores
    (every second token repeats the one before it)."""
    d = Dims(1, N, C, 3, 2, 4, 2, 1, 64, PD_FP32)
    x = random_prefill_inputs(d, seed=C, scale=0.125)
    for k in ("q_pre", "k_pre"):
        x[k][:, :, 2::2] = x[k][:, :, 1:C:2]
    out = run_prefill(d, x, chunk_score=True)
    torch.cuda.synchronize()
    e, rank = out["tok_score"].cpu(), out["tok_rank"].cpu().long()
    order = torch.sort(e, dim=2, descending=True, stable=True)[1]
    want = torch.empty_like(order).scatter_(2, order, torch.arange(C).expand(1, N, C).contiguous())
    assert torch.equal(rank, want)
    prefill_units_check(d, x, out, [(0, N - 1)])


@pytest.mark.parametrize("Hq,Ld", [(1, 1), (7, 1), (8, 5), (9, 40), (16, 1024), (43, 300)])
def test_score_terms(Hq, Ld):
    """Score terms per chunk (heads x 128-row splits): 1 to 129, eight threads a chunk, 16 terms a batch."""
    d = Dims(2, 5, 33, 4, 0, Ld, Hq, 1, 64, PD_FP32)
    g = torch.Generator().manual_seed(Hq + Ld)
    q = torch.randn((2, Ld, Hq, 64), generator=g).cuda()
    km = torch.randn((2, 5, 1, 64), generator=g)
    rank = torch.argsort(torch.rand((2, 5, 33), generator=g), dim=2).to(torch.int32)
    ci, ts, cs = run_select(d, 2, 9, q, km.cuda(), rank.cuda())
    torch.cuda.synchronize()
    ref = oracle.chunk_scores_ref(q.cpu().double().numpy(), km.double().numpy())
    # fp32 sums of Hq * Ld * 64 products of N(0, 1) values over Ld rows
    np.testing.assert_allclose(cs.cpu().double().numpy(), ref, rtol=1e-5, atol=1e-5 * Hq ** 0.5)
    want = np.sort(np.argsort(-cs.cpu().numpy(), axis=1, kind="stable")[:, :2], axis=1)
    assert np.array_equal(ci.cpu().numpy(), want)
    assert np.array_equal(ts.cpu().numpy(), oracle.tokens_by_rank_ref(rank.numpy(), want, 9))


@pytest.mark.parametrize("dtype", [PD_BF16, PD_FP32])
@pytest.mark.parametrize("S", [2, 4, 5, 8, 9, 16, 17, 24, 25, 33])
def test_merge_shards(S, dtype):
    """Shard counts around the merge's variants of 4, 8, 16 and 24, and beyond."""
    d = Dims(1, 4, 600, 8, 4, 9, 2, 1, 64, dtype)
    scale = 0.125 if dtype == PD_FP32 else 1.0
    x = random_prefill_inputs(d, seed=S, scale=scale)
    cache = {"k_cache": x["k_pre"].transpose(2, 3).contiguous(), "v_cache": x["v_pre"].transpose(2, 3).contiguous()}
    dec = random_decode_inputs(d, seed=S, scale=scale)
    ci, ts = random_indices(d, 4, 560, seed=5)
    o, lse = run_decode(d, 4, 560, dec, cache, ci, ts, x["k_qm"], x["v_qm"], 7, num_splits=S)
    torch.cuda.synchronize()
    decode_check(d, 4, 560, dec, cache, ci, ts, x["k_qm"], x["v_qm"], 7, o, lse, batches=[0])
