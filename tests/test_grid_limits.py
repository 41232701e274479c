"""Host limits of the fp32 launches, whose workgroups are smaller than 64 rows: grids of 2^31 workgroups and more are
refused before anything is launched.  The pointers are fake: only the host reads them."""

import ctypes

from paper_2606_10537_amd import _lib
from paper_2606_10537_amd._lib import PD_FP32, Dims
from test_abi import A, prefill

BAD_DIMS = 2


def dims(**kw):
    base = dict(batch=1, n_chunks=1, chunk_len=1, q_len=1, m_len=0, dec_len=1, n_heads_q=1, n_heads_kv=1, head_dim=64,
                dtype=PD_FP32)
    return Dims(**dict(base, **kw))


def test_prefill_row_tiles():
    """2^30 (sequence, chunk, head) of 40 rows: one tile of 64 rows each, two of 32."""
    d = dims(batch=1 << 20, n_chunks=1024, chunk_len=30, q_len=9)
    assert _lib.pd_workspace_bytes(d, which=0) == 0
    assert prefill(d, ws=None, wsn=0) == BAD_DIMS
    d.n_chunks = 256
    assert _lib.pd_workspace_bytes(d, which=0) > 0


def test_prefill_copies():
    """A tile each and as many copying workgroups: 2^31."""
    d = dims(batch=1 << 20, n_chunks=1024)
    assert _lib.pd_workspace_bytes(d, which=0) == 0
    assert prefill(d, ws=None, wsn=0) == BAD_DIMS


def test_token_score_blocks():
    """2^23 heads of 4096 keys: 65 tiles of 64 rows each, 256 blocks of 16 keys."""
    d = dims(batch=1 << 20, n_chunks=8, chunk_len=4096)
    assert _lib.pd_workspace_bytes(d, which=0) == 0
    assert prefill(d, ws=None, wsn=0) == BAD_DIMS


def test_decode_row_tiles():
    """2^29 KV heads of 33 rows in 2 shards: one tile of 64 rows each, two of 32."""
    d = dims(batch=1 << 24, n_heads_q=32, n_heads_kv=32, dec_len=33)
    lib = _lib.load()
    assert _lib.pd_workspace_bytes(d, 1, 1, 2, 2) == 0
    dd = d.c()
    rc = lib.pd_sparse_decode_attn(ctypes.byref(dd), 1, 1, A, A, A, A, A, A, A, None, None, 0, A, None, 2, None, 0, None)
    assert rc == BAD_DIMS
    assert b"too large" in lib.pd_last_error_message()
