"""The calls that the block-sparse attention path is timed on.

Five kinds of pass, each through the binding's entry points (one layer, as a model's layer calls them):

* ``prefill``  -- pd_prefill_chunks: chunk attention, KV cache, token scores and ranks, key means and,
  where asked, the prefill-time chunk score;
* ``step``     -- one denoising step: pd_score_select, then pd_sparse_decode_attn over what it kept;
* ``static``   -- the select-once schedule: pd_score_select_static, pd_gather_selected, then ``steps``
  calls of pd_sparse_decode_attn_compact with new decode rows;
* ``joint``    -- the full-mask cache: pd_select_ranked, pd_gather_joint and the dense joint pass;
* ``layer``    -- a whole layer of a short job: prefill with chunk score, selection, one decode.

Sizes are those of the synthetic workloads (8K to 32K contexts, chunks of 1024), of the block decode
with 32 rows, and odd ones.  ``draw`` covers the same ranges.
"""

import math

import torch

from paper_2606_10537_amd import _lib
from paper_2606_10537_amd._lib import PD_BF16, PD_FP32, Dims

_BASE = {"kind": "prefill", "dtype": "bf16", "batch": 1, "n_chunks": 8, "chunk_len": 1024, "q_len": 64,
         "m_len": 256, "dec_len": 256, "n_heads_q": 32, "n_heads_kv": 32, "head_dim": 128, "top_k": 2,
         "tok_budget": 512, "n_static": 64, "plant": 0, "lognormal": 0.0, "steps": 1, "qm_per_chunk": 0,
         "out_fp32": 0, "tok_score_dir": 0, "chunk_score": False, "lse": False}


def _case(name=None, **kw):
    c = dict(_BASE, **kw)
    if name is not None:
        c["name"] = name
    return c


_32K = dict(batch=8, n_chunks=32, q_len=128, m_len=512, dec_len=512, top_k=4, tok_budget=256, n_static=128,
            lognormal=0.3)
_16K = dict(n_chunks=16, n_heads_q=28, n_heads_kv=4, top_k=4, tok_budget=256, plant=4)


def listed():
    return [
        # The smallest job: four chunks of 128 tokens in fp32, every stage once.  Launches count.
        _case("layer_tiny_fp32", kind="layer", dtype="fp32", n_chunks=4, chunk_len=128, q_len=16, m_len=32,
              dec_len=32, n_heads_q=4, n_heads_kv=4, head_dim=64, top_k=2, tok_budget=128, n_static=16, plant=1),
        # Prefill of one 8K prompt, as many KV heads as query heads.
        _case("prefill_8k", plant=2),
        # Prefill of one 16K prompt, 7 query heads per KV head; the chunks are scored on the way.
        _case("prefill_16k_gqa", chunk_score=True, **_16K),
        # The largest call: one layer's prefill of eight 32K prompts.
        _case("prefill_32k_b8", **_32K),
        # A short-chunk prefill with odd sizes, d = 64, q/m rows per chunk and fp32 results.
        _case("prefill_ragged_d64", batch=2, n_chunks=5, chunk_len=777, q_len=45, m_len=83, n_heads_q=12,
              n_heads_kv=4, head_dim=64, qm_per_chunk=1, out_fp32=1),
        # A denoising step of a single 8K prompt: the latency of selection and decode.
        _case("step_8k", kind="step", plant=2, lse=True),
        # The same at 16K with grouped heads.
        _case("step_16k_gqa", kind="step", **_16K),
        # The step that a 32K batch job spends most of its time in.
        _case("step_32k_b8", kind="step", **_32K),
        # Block decode: 32 rows of one prompt over 4 x 1024 kept tokens, 4 query heads per KV head.
        _case("step_block32_gqa", kind="step", n_chunks=32, dec_len=32, n_heads_kv=8, top_k=4, tok_budget=1024),
        # The select-once schedule of a batch of four 32K prompts: selection, compaction, four steps.
        _case("static_32k_b4", kind="static", **dict(_32K, batch=4, steps=4)),
        # Full-mask cache of two 32K prompts: joint rows at continuous positions, dense joint pass.
        _case("joint_32k_b2", kind="joint", **dict(_32K, batch=2)),
        # A step in fp32 with odd sizes, as a check of a model in full precision runs it.
        _case("step_ragged_fp32", kind="step", dtype="fp32", n_chunks=6, chunk_len=300, q_len=33, m_len=40,
              dec_len=72, n_heads_q=16, n_heads_kv=4, top_k=3, tok_budget=117, n_static=73, lse=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    largest = max(work(c)["flops"] for c in listed())
    while True:
        kind = rng.choice(["prefill", "prefill", "step", "step", "step", "static", "joint", "layer"])
        fp32 = rng.random() < 0.2
        hkv = rng.choice([1, 2, 4, 8, 32] if not fp32 else [1, 2, 4])
        hq = hkv * (rng.choice([1, 2, 4, 7]) if hkv < 32 else 1)
        n = _log(rng, 1, 32)
        c = _log(rng, 64, 1024) if not fp32 else _log(rng, 32, 512)
        k = rng.randint(1, min(n, 4))
        lq, lm = _log(rng, 16, 128), _log(rng, 16, 512)
        case = _case(kind=kind, dtype="fp32" if fp32 else "bf16", batch=rng.choice([1, 1, 2, 3, 4, 8]), n_chunks=n,
                     chunk_len=c, q_len=lq, m_len=lm, dec_len=_log(rng, 16, 512), n_heads_q=hq, n_heads_kv=hkv,
                     head_dim=rng.choice([64, 128, 128]), top_k=k,
                     # a layer's own ranks feed its selection: all tokens kept, so that a tie cannot change the set
                     tok_budget=c if kind == "layer" else rng.randint(max(1, c // 8), c),
                     n_static=rng.choice([0, lq, lq + lm]), plant=rng.choice([0, 1]), lognormal=rng.choice([0.0, 0.3]),
                     steps=rng.randint(1, 4) if kind == "static" else 1, qm_per_chunk=rng.choice([0, 0, 1]),
                     out_fp32=rng.choice([0, 0, 1]), tok_score_dir=rng.choice([0, 0, 1]),
                     chunk_score=rng.random() < 0.5, lse=rng.random() < 0.5)
        if kind in ("prefill", "layer") and case["batch"] * n * c < 1024:
            continue   # too few ranks for a share of them to say anything
        w = work(case)
        # fp32 runs on the vector units: a fp32 case counts for 30 times its operations.
        if w["flops"] * (30 if fp32 else 1) <= largest / 2:
            return case


# ------------------------------------------------------------------------------------------- sizes

def _dims(c, dec_len=None):
    return Dims(c["batch"], c["n_chunks"], c["chunk_len"], c["q_len"], c["m_len"], dec_len or c["dec_len"],
                c["n_heads_q"], c["n_heads_kv"], c["head_dim"], PD_BF16 if c["dtype"] == "bf16" else PD_FP32, 0.0,
                c["qm_per_chunk"], c["out_fp32"], c["tok_score_dir"])


def _n_sel(c):
    return c["top_k"] * (1 + c["tok_budget"])


def work(case):
    """Operations and bytes that one pass cannot do without: every input row read once, every output
    written once, the two products of each attention."""
    c = case
    eb, d, B, N, C = (2 if c["dtype"] == "bf16" else 4), c["head_dim"], c["batch"], c["n_chunks"], c["chunk_len"]
    ob = 4 if c["out_fp32"] else eb
    Hq, Hkv, Lqm, Ld, K, Bt = c["n_heads_q"], c["n_heads_kv"], c["q_len"] + c["m_len"], c["dec_len"], c["top_k"], c["tok_budget"]
    Sc = 1 + C + Lqm
    by = fl = 0
    if c["kind"] in ("prefill", "layer"):
        rows = B * N * (1 + C)
        qm = B * (N if c["qm_per_chunk"] else 1) * Lqm
        by += (rows + qm) * (Hq + 2 * Hkv) * d * eb + rows * 2 * Hkv * d * eb + B * N * Sc * Hq * d * ob
        by += B * N * C * 8 + B * N * Hkv * d * 4
        fl += 4 * B * N * Hq * Sc * Sc * d
    L_kv = _n_sel(c) + c["n_static"] + Ld
    dec_rows = B * Ld * (Hq * d * (eb + ob) + 2 * Hkv * d * eb)
    sel = B * (N * Hkv * d * 4 + K * C * 4 + K * Bt * 4)
    if c["kind"] in ("step", "layer"):
        by += sel + dec_rows + B * (_n_sel(c) + c["n_static"]) * 2 * Hkv * d * eb
        fl += 4 * B * Hq * Ld * L_kv * d + (2 * B * N * Hq * d if c["kind"] == "step" else 0)
    if c["kind"] == "static":
        by += sel + B * c["m_len"] * Hq * d * eb + B * _n_sel(c) * 4 * Hkv * d * eb
        by += c["steps"] * (dec_rows + B * (_n_sel(c) + c["n_static"]) * 2 * Hkv * d * eb)
        fl += c["steps"] * 4 * B * Hq * Ld * L_kv * d + 2 * B * N * Hq * d
    if c["kind"] == "joint":
        Lj = _n_sel(c) + c["q_len"]
        by += B * (K * C * 4 + K * Bt * 4) + B * Lj * d * (eb * (2 * Hq + 6 * Hkv) + Hq * (eb + ob) + 2 * Hkv * eb)
        fl += 4 * B * Hq * Lj * Lj * d
    return {"bytes": by, "flops": fl}


def tolerance(case):
    """About four times what the passes of these ranges measured against ``exact``: fp32 results 9e-7 (32-bit
    sums, the hardware's exp2), bf16 calls 2.3e-3 (the weights that multiply V and the results are rounded to
    8 significant bits).  Two tokens whose fp32 scores differ by their last bits may swap ranks: up to 0.4 %
    of the ranks of a small call."""
    if case["dtype"] == "fp32":
        return {"rel": 4e-6, "max": 1e-4, "differ": 0.01}
    return {"rel": 1e-2, "max": 0.4, "differ": 0.01}


# ------------------------------------------------------------------------------------------ inputs

def _inputs(case, seed):
    """The pass's inputs: N(0, 1) rows (an eighth of that in fp32, d = 64), one BOS row per head shared by
    all chunks, heavy-tailed key norms and a planted direction in some chunks where the case has them."""
    c = case
    g = torch.Generator(device="cuda")
    g.manual_seed(1_000_003 * (int(seed) % 2_000_000_011) + 7)
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    B, N, C, d = c["batch"], c["n_chunks"], c["chunk_len"], c["head_dim"]
    Hq, Hkv, Lqm, K = c["n_heads_q"], c["n_heads_kv"], c["q_len"] + c["m_len"], c["top_k"]
    sigma = 0.125 if c["dtype"] == "fp32" and d == 64 else 1.0

    def rnd(*s, dtype=dt):
        x = torch.empty(s, dtype=dtype, device="cuda").normal_(generator=g)
        return x.mul_(sigma) if sigma != 1.0 else x

    def norms(x):
        if c["lognormal"]:
            z = torch.empty(x.shape[:-2], device="cuda").normal_(generator=g)
            x.mul_(torch.exp(c["lognormal"] * z)[..., None, None].to(dt))
        return x

    u = torch.nn.functional.normalize(torch.empty((Hkv, d), device="cuda").normal_(generator=g), dim=1)
    amp = 0.5 * math.sqrt(d) * sigma
    plant = torch.stack([torch.randperm(N, generator=g, device="cuda")[:min(c["plant"], N)] for _ in range(B)])
    uq = (amp * u.repeat_interleave(Hq // Hkv, dim=0)).to(dt)
    x = {}
    qm = (B, N, Lqm) if c["qm_per_chunk"] else (B, Lqm)
    x["q_qm"], x["k_qm"], x["v_qm"] = rnd(*qm, Hq, d), norms(rnd(*qm, Hkv, d)), rnd(*qm, Hkv, d)
    if c["plant"]:
        x["q_qm"][..., :c["q_len"], :, :] += uq
    if c["kind"] in ("prefill", "layer", "joint"):
        x["q_pre"] = rnd(B, N, 1 + C, Hq, d)
        x["q_pre"][:, :, 0] = rnd(Hq, d)
    if c["kind"] in ("prefill", "layer"):
        x["k_pre"], x["v_pre"] = norms(rnd(B, N, 1 + C, Hkv, d)), rnd(B, N, 1 + C, Hkv, d)
        x["k_pre"][:, :, 0], x["v_pre"][:, :, 0] = rnd(Hkv, d), rnd(Hkv, d)
        for b in range(B):
            for n in plant[b].tolist():
                x["k_pre"][b, n, 1:] += (amp * u).to(dt)
    else:   # what an earlier prefill left in the cache
        x["k_cache"], x["v_cache"] = rnd(B, N, Hkv, 1 + C, d), rnd(B, N, Hkv, 1 + C, d)
        if c["lognormal"]:
            z = torch.empty((B, N, 1, 1 + C, 1), device="cuda").normal_(generator=g)
            x["k_cache"].mul_(torch.exp(c["lognormal"] * z).to(dt))
        for b in range(B):
            for n in plant[b].tolist():
                x["k_cache"][b, n, :, 1:] += (amp * u).to(dt)[:, None]
        x["key_mean"] = x["k_cache"][:, :, :, 1:].mean(dim=3, dtype=torch.float32).contiguous()
        x["tok_rank"] = torch.rand((B, N, C), generator=g, device="cuda").argsort(dim=-1).to(torch.int32)
    if c["kind"] == "joint":
        x["scores"] = torch.empty((B, N), device="cuda").normal_(generator=g)
    if c["kind"] in ("step", "static", "layer"):
        x["dec"] = []
        for _ in range(c["steps"]):
            q = rnd(B, c["dec_len"], Hq, d)
            if c["plant"]:
                q += uq
            x["dec"].append((q, norms(rnd(B, c["dec_len"], Hkv, d)), rnd(B, c["dec_len"], Hkv, d)))
    return x


def prepare(case, seed):
    """Inputs, and the output buffers and workspaces that the caller of this library owns and keeps."""
    c = case
    x = _inputs(c, seed)
    d = _dims(c)
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    odt = torch.float32 if c["out_fp32"] else dt
    B, N, C, D, Hq, Hkv = c["batch"], c["n_chunks"], c["chunk_len"], c["head_dim"], c["n_heads_q"], c["n_heads_kv"]
    K, Bt, Ld = c["top_k"], c["tok_budget"], c["dec_len"]

    def new(*s, dtype=torch.float32):
        return torch.empty(s, dtype=dtype, device="cuda")

    def ws(nbytes):
        return torch.empty(max(16, nbytes), dtype=torch.uint8, device="cuda")

    st = {"case": c, "dims": d, "x": x}
    if c["kind"] in ("prefill", "layer"):
        st["pre"] = {"o": new(B, N, d.seq_len, Hq, D, dtype=odt), "k_cache": new(B, N, Hkv, 1 + C, D, dtype=dt),
                     "v_cache": new(B, N, Hkv, 1 + C, D, dtype=dt), "tok_score": new(B, N, C),
                     "tok_rank": new(B, N, C, dtype=torch.int32), "key_mean": new(B, N, Hkv, D)}
        if c["chunk_score"] or c["kind"] == "layer":
            st["pre"]["chunk_score"] = new(B, N)
        st["ws_pre"] = ws(_lib.pd_workspace_bytes(d, which=0))
    if c["kind"] != "prefill":
        st["chunk_idx"], st["tok_slot"] = new(B, K, dtype=torch.int32), new(B, K, Bt, dtype=torch.int32)
        st["ws_sel"] = ws(_lib.pd_workspace_bytes(d, K, Bt, 0, 1))
    if c["kind"] in ("step", "static", "layer"):
        st["o"] = [new(B, Ld, Hq, D, dtype=odt) for _ in range(c["steps"])]
        st["lse"] = [new(B, Hq, Ld) if c["lse"] else None for _ in range(c["steps"])]
        if c["kind"] != "layer":
            st["score"] = new(B, N)
        # The static rows are the prompt's q/m rows, in one copy per sequence.
        st["k_st"], st["v_st"] = ((x["k_qm"][:, 0].contiguous(), x["v_qm"][:, 0].contiguous())
                                  if c["qm_per_chunk"] else (x["k_qm"], x["v_qm"]))
    if c["kind"] in ("step", "layer"):
        st["ws_dec"] = ws(_lib.pd_workspace_bytes(d, K, Bt, 0, 2))
    if c["kind"] == "static":
        st["k_sel"], st["v_sel"] = new(B, Hkv, _n_sel(c), D, dtype=dt), new(B, Hkv, _n_sel(c), D, dtype=dt)
        st["ws_dec"] = ws(_lib.pd_compact_workspace_bytes(d, _n_sel(c), 0))
    if c["kind"] == "joint":
        Lj = _n_sel(c) + c["q_len"]
        st["dims_joint"] = _dims(c, Lj)
        st["joint"] = {"q": new(B, Lj, Hq, D, dtype=dt), "k": new(B, Lj, Hkv, D, dtype=dt),
                       "v": new(B, Lj, Hkv, D, dtype=dt), "k_pref": new(B, Hkv, Lj, D, dtype=dt),
                       "v_pref": new(B, Hkv, Lj, D, dtype=dt), "o": new(B, Lj, Hq, D, dtype=odt)}
        st["lse"] = new(B, Hq, Lj) if c["lse"] else None
        st["ws_dec"] = ws(_lib.pd_compact_workspace_bytes(st["dims_joint"], 0, 0))
    return st


_ROPE_BASE = 500000.0


def run(state):
    st, c, d, x = state, state["case"], state["dims"], state["x"]
    K, Bt, ns = c["top_k"], c["tok_budget"], c["n_static"]
    out = {}
    if c["kind"] in ("prefill", "layer"):
        p = st["pre"]
        _lib.pd_prefill_chunks(d, x["q_pre"], x["k_pre"], x["v_pre"], x["q_qm"], x["k_qm"], x["v_qm"], p["o"],
                               p["k_cache"], p["v_cache"], p["tok_score"], p["tok_rank"], p["key_mean"],
                               st["ws_pre"], chunk_score=p.get("chunk_score"))
        out.update(p)
        if c["kind"] == "prefill":
            return out
    ci, ts = st["chunk_idx"], st["tok_slot"]
    if c["kind"] == "layer":
        _lib.pd_select_ranked(d, K, Bt, p["chunk_score"], 1, p["tok_rank"], ci, ts)
        x = dict(x, k_cache=p["k_cache"], v_cache=p["v_cache"])
    elif c["kind"] == "step":
        _lib.pd_score_select(d, K, Bt, x["dec"][0][0], x["key_mean"], x["tok_rank"], ci, ts, st["score"],
                             st["ws_sel"])
        out["score"] = st["score"]
    elif c["kind"] == "static":
        _lib.pd_score_select_static(d, K, Bt, x["q_qm"], x["key_mean"], x["tok_rank"], ci, ts, st["score"],
                                    st["ws_sel"])
        _lib.pd_gather_selected(d, K, Bt, x["k_cache"], x["v_cache"], ci, ts, st["k_sel"], st["v_sel"])
        out.update(score=st["score"], k_sel=st["k_sel"], v_sel=st["v_sel"])
    elif c["kind"] == "joint":
        j = st["joint"]
        _lib.pd_select_ranked(d, K, Bt, x["scores"], 1, x["tok_rank"], ci, ts)
        _lib.pd_gather_joint(d, K, Bt, ci, ts, x["q_pre"], x["k_cache"], x["v_cache"], x["q_qm"], x["k_qm"],
                             x["v_qm"], _ROPE_BASE, j["q"], j["k"], j["v"], j["k_pref"], j["v_pref"])
        _lib.pd_sparse_decode_attn_compact(st["dims_joint"], 0, j["q"], j["k"], j["v"], None, None, None, None, 0,
                                           j["o"], st["lse"], 0, st["ws_dec"])
        out.update(j)
        if st["lse"] is not None:
            out["lse"] = st["lse"]
    out.update(chunk_idx=ci, tok_slot=ts)
    if c["kind"] == "joint":
        return out
    for i, (q, k, v) in enumerate(x["dec"]):
        kst, vst = st["k_st"], st["v_st"]
        if c["kind"] == "static":
            _lib.pd_sparse_decode_attn_compact(d, _n_sel(c), q, k, v, st["k_sel"], st["v_sel"], kst, vst, ns,
                                               st["o"][i], st["lse"][i], 0, st["ws_dec"])
        else:
            _lib.pd_sparse_decode_attn(d, K, Bt, q, k, v, x["k_cache"], x["v_cache"], ci, ts, kst, vst, ns,
                                       st["o"][i], st["lse"][i], 0, st["ws_dec"])
    out["o_dec"] = list(st["o"])
    if c["lse"]:
        out["lse"] = list(st["lse"])
    return out


# ------------------------------------------------------------------------------- the same in 64 bits

def _attend(q, k, v, scale):
    """softmax(scale q k^T) v and the logits' LSE for [H][rows][d] operands in float64."""
    s = torch.matmul(q, k.transpose(1, 2).contiguous()).mul_(scale)
    lse = torch.logsumexp(s, dim=-1)
    p = s.sub_(lse[..., None]).exp_()
    return torch.matmul(p, v), lse, p


def _exact_prefill(c, x, with_score):
    B, N, C, Lq, Lm = c["batch"], c["n_chunks"], c["chunk_len"], c["q_len"], c["m_len"]
    Hq, Hkv, d = c["n_heads_q"], c["n_heads_kv"], c["head_dim"]
    G, Sc = Hq // Hkv, 1 + C + Lq + Lm
    o = torch.empty((B, N, Sc, Hq, d), dtype=torch.float64, device="cuda")
    e = torch.empty((B, N, C), dtype=torch.float64, device="cuda")
    cs = torch.empty((B, N), dtype=torch.float64, device="cuda")
    for b in range(B):
        for n in range(N):
            q, k, v = (torch.cat([x[t + "_pre"][b, n], x[t + "_qm"][(b, n) if c["qm_per_chunk"] else b]]).double()
                       .transpose(0, 1).contiguous() for t in "qkv")
            rows, _, p = _attend(q, k.repeat_interleave(G, dim=0), v.repeat_interleave(G, dim=0), d ** -0.5)
            o[b, n] = rows.transpose(0, 1)
            qc = slice(1 + C, 1 + C + Lq)
            e[b, n] = p[:, qc, 1:1 + C].sum(dim=(0, 1))
            if not c["tok_score_dir"]:
                e[b, n] += p[:, 1:1 + C, qc].sum(dim=(0, 2))
            a = -torch.log(p[:, 1 + C:, 1:1 + C].sum(dim=2).mean(dim=0))
            cs[b, n] = a[:Lq].mean() + (a[Lq:].mean() if Lm else 0.0)
    rank = torch.empty((B, N, C), dtype=torch.int32, device="cuda")
    order = torch.sort(e, dim=-1, descending=True, stable=True)[1]
    rank.scatter_(2, order, torch.arange(C, dtype=torch.int32, device="cuda").expand(B, N, C).contiguous())
    out = {"o": o, "k_cache": x["k_pre"].transpose(2, 3).contiguous(), "v_cache": x["v_pre"].transpose(2, 3).contiguous(),
           "tok_score": e, "tok_rank": rank, "key_mean": x["k_pre"][:, :, 1:].double().mean(dim=2)}
    if with_score:
        out["chunk_score"] = cs
    return out


def _exact_scores(c, q_rows, key_mean):
    """s[b][n] = sum over heads of scale <mean row, key mean>."""
    G = c["n_heads_q"] // c["n_heads_kv"]
    q = q_rows.double().mean(dim=1).reshape(c["batch"], 1, c["n_heads_kv"], G, c["head_dim"]).sum(dim=3)
    return c["head_dim"] ** -0.5 * (q * key_mean.double()).sum(dim=(2, 3))


def _exact_select(c, score, lowest, tok_rank):
    order = torch.sort(score, dim=-1, descending=not lowest, stable=True)[1]
    ci = torch.sort(order[:, :c["top_k"]], dim=-1)[0]
    kept = torch.gather(tok_rank.long(), 1, ci[..., None].expand(-1, -1, c["chunk_len"])) < c["tok_budget"]
    ts = kept.nonzero()[:, 2].reshape(c["batch"], c["top_k"], c["tok_budget"]) + 1
    return ci.to(torch.int32), ts.to(torch.int32)


def _kept_rows(c, cache, ci, ts):
    """[B][Hkv][K*(1+Bt)][d]: BOS and kept slots of every kept chunk."""
    slots = torch.cat([torch.zeros_like(ts[..., :1]), ts], dim=-1).long()
    rows = [torch.cat([cache[b, int(ci[b, k])][:, slots[b, k]] for k in range(c["top_k"])], dim=1)
            for b in range(c["batch"])]
    return torch.stack(rows)


def _exact_decode(c, q, k, v, k_sel, v_sel, k_st, v_st, ns):
    G = c["n_heads_q"] // c["n_heads_kv"]
    os, lses = [], []
    for b in range(c["batch"]):
        kk, vv = (torch.cat([s[b].double(), st[b, :ns].double().transpose(0, 1), own[b].double().transpose(0, 1)], dim=1)
                  .repeat_interleave(G, dim=0) for s, st, own in ((k_sel, k_st, k), (v_sel, v_st, v)))
        o, lse, _ = _attend(q[b].double().transpose(0, 1).contiguous(), kk, vv, c["head_dim"] ** -0.5)
        os.append(o.transpose(0, 1))
        lses.append(lse)
    return torch.stack(os), torch.stack(lses)


def _rotate(x, shift):
    """Rotate-half rotary of x [rows][H][d] by shift[row] positions, in float64."""
    d = x.shape[-1]
    f = _ROPE_BASE ** (-2.0 * torch.arange(d // 2, dtype=torch.float64, device="cuda") / d)
    a = shift.double()[:, None, None] * f
    lo, hi = x[..., :d // 2].double(), x[..., d // 2:].double()
    return torch.cat([lo * a.cos() - hi * a.sin(), hi * a.cos() + lo * a.sin()], dim=-1)


def exact(case, seed):
    c, x = case, _inputs(case, seed)
    ns, B = c["n_static"], c["batch"]
    out = {}
    if c["kind"] in ("prefill", "layer"):
        out = _exact_prefill(c, x, c["chunk_score"] or c["kind"] == "layer")
        if c["kind"] == "prefill":
            return out
        x.update(k_cache=out["k_cache"], v_cache=out["v_cache"])
        ci, ts = _exact_select(c, out["chunk_score"], True, out["tok_rank"])
    elif c["kind"] == "joint":
        ci, ts = _exact_select(c, x["scores"], True, x["tok_rank"])
    else:
        qm = x["q_qm"][:, 0] if c["qm_per_chunk"] else x["q_qm"]
        out["score"] = _exact_scores(c, x["dec"][0][0] if c["kind"] == "step" else qm[:, c["q_len"]:], x["key_mean"])
        ci, ts = _exact_select(c, out["score"], False, x["tok_rank"])
    out.update(chunk_idx=ci, tok_slot=ts)
    k_sel, v_sel = _kept_rows(c, x["k_cache"], ci, ts), _kept_rows(c, x["v_cache"], ci, ts)
    dt = x["k_qm"].dtype
    if c["kind"] == "joint":
        K, Bt, Lq, C1 = c["top_k"], c["tok_budget"], c["q_len"], 1 + c["chunk_len"]
        shift = torch.cat([torch.arange(K, device="cuda").repeat_interleave(1 + Bt) * C1,
                           torch.full((Lq,), (K - 1) * C1, device="cuda")])
        rows = {}
        for t, sel in (("k", k_sel), ("v", v_sel)):
            qm = x[t + "_qm"][:, 0] if c["qm_per_chunk"] else x[t + "_qm"]
            rows[t] = torch.cat([sel.transpose(1, 2), qm[:, :Lq]], dim=1)
        q_sel = _kept_rows(c, x["q_pre"].transpose(2, 3), ci, ts)
        rows["q"] = torch.cat([q_sel.transpose(1, 2), (x["q_qm"][:, 0] if c["qm_per_chunk"] else x["q_qm"])[:, :Lq]], dim=1)
        for t in "qk":   # rounded once to the element type, which the joint pass then reads
            rows[t] = torch.stack([_rotate(rows[t][b], shift) for b in range(B)]).to(dt)
        out.update(rows, k_pref=rows["k"].transpose(1, 2).contiguous(), v_pref=rows["v"].transpose(1, 2).contiguous())
        none = torch.empty((B, c["n_heads_kv"], 0, c["head_dim"]), dtype=dt, device="cuda")
        out["o"], lse = _exact_decode(c, rows["q"], rows["k"], rows["v"], none, none, rows["k"], rows["v"], 0)
        if c["lse"]:
            out["lse"] = lse
        return out
    if c["kind"] == "static":
        out.update(k_sel=k_sel, v_sel=v_sel)
    k_st, v_st = (x["k_qm"][:, 0], x["v_qm"][:, 0]) if c["qm_per_chunk"] else (x["k_qm"], x["v_qm"])
    got = [_exact_decode(c, q, k, v, k_sel, v_sel, k_st, v_st, ns) for q, k, v in x["dec"]]
    out["o_dec"] = [o for o, _ in got]
    if c["lse"]:
        out["lse"] = [lse for _, lse in got]
    return out
