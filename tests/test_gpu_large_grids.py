"""Calls of very many small problems, whose launches hold more threads than one grid dimension takes."""

import pytest
import torch

from gpu_path import workspace
from paper_2606_10537_amd import _lib
from paper_2606_10537_amd._lib import PD_FP32, Dims

pytestmark = pytest.mark.gpu


def rnd(*s):
    return torch.empty(s, device="cuda").normal_(generator=torch.Generator(device="cuda").manual_seed(sum(s))).mul_(0.125)


def test_select_many_sequences():
    """2^18 sequences of 64 chunks."""
    B, N = 1 << 18, 64
    s = rnd(B, N)
    ci = torch.full((B, 1), -1, dtype=torch.int32, device="cuda")
    ts = torch.full((B, 1, 1), -1, dtype=torch.int32, device="cuda")
    rank = torch.zeros((B, N, 1), dtype=torch.int32, device="cuda")
    _lib.pd_select_ranked(Dims(B, N, 1, 1, 0, 1, 1, 1, 64, PD_FP32), 1, 1, s, 0, rank, ci, ts)
    torch.cuda.synchronize()
    assert torch.equal(torch.gather(s, 1, ci.long())[:, 0], s.max(dim=1)[0])
    assert (ts == 1).all()


def test_fp32_prefill_many_chunks():
    """2^21 chunks of one token and 8 heads: 2^24 row tiles."""
    B, N, H, D = 2048, 1024, 8, 64
    d = Dims(B, N, 1, 1, 0, 1, H, 1, D, PD_FP32)
    q, k, v = rnd(B, N, 2, H, D), rnd(B, N, 2, 1, D), rnd(B, N, 2, 1, D)
    qq, kq, vq = rnd(B, 1, H, D), rnd(B, 1, 1, D), rnd(B, 1, 1, D)
    o = torch.full((B, N, 3, H, D), float("nan"), device="cuda")
    kc, vc = torch.empty((B, N, 1, 2, D), device="cuda"), torch.empty((B, N, 1, 2, D), device="cuda")
    e, km = torch.full((B, N, 1), float("nan"), device="cuda"), torch.empty((B, N, 1, D), device="cuda")
    rank = torch.full((B, N, 1), -1, dtype=torch.int32, device="cuda")
    _lib.pd_prefill_chunks(d, q, k, v, qq, kq, vq, o, kc, vc, e, rank, km,
                           workspace(_lib.pd_workspace_bytes(d, which=0)))
    torch.cuda.synchronize()
    assert torch.equal(kc[:, :, 0], k[:, :, :, 0]) and torch.equal(vc[:, :, 0], v[:, :, :, 0])
    assert torch.equal(km[:, :, 0], k[:, :, 1, 0]) and (rank == 0).all()
    assert torch.isfinite(o.sum(dim=(2, 3, 4))).all()
    for b in (0, 1, 1023, 2047):   # every chunk of these sequences in float64
        qs = torch.cat([q[b], qq[b].expand(N, 1, H, D)], dim=1).double()
        ks, vs = (torch.cat([x[b], y[b].expand(N, 1, 1, D)], dim=1).double()[:, :, 0] for x, y in ((k, kq), (v, vq)))
        p = torch.softmax(torch.einsum("nrhd,ncd->nrhc", qs, ks) / D ** 0.5, dim=-1)
        assert (o[b].double() - torch.einsum("nrhc,ncd->nrhd", p, vs)).abs().max() <= 1e-5
        ref = p[:, 2, :, 1].sum(dim=1) + p[:, 1, :, 2].sum(dim=1)
        assert (e[b, :, 0].double() - ref).abs().max() <= 1e-4


def test_fp32_decode_many_rows():
    """2^24 KV heads of one row over one key: the output is the value row."""
    B, H, D = 1 << 20, 16, 64
    d = Dims(B, 1, 1, 1, 0, 1, H, H, D, PD_FP32)
    q, v = rnd(B, 1, H, D), rnd(B, 1, H, D)
    o = torch.full((B, 1, H, D), float("nan"), device="cuda")
    _lib.pd_sparse_decode_attn_compact(d, 0, q, q, v, None, None, None, None, 0, o, None, 1, None)
    torch.cuda.synchronize()
    assert (o - v).abs().max() <= 1e-6
