"""Workloads of the selective-prefill library for timing and for comparing builds.

Every case is one pass of a user's program through the public binding (`paper_2601_12904_amd.binding`, `.stack`), on
device tensors that the program already holds:

  layer    one layer's online step for one request: stitch the cached keys, score and select, attention of the
           recomputed rows, write-back (`fused` = the write-back inside the attention call)
  shared   several requests over one chunk store that is never written: selection per request, then one batched attention
  offline  preprocessing of one chunk for the store: its rows attend to the retrieved chunks and causally to themselves
  decode   one decoding step of a batch over the chunk store and the requests' own pages
  stack    decoder layers (projections, norms, feed-forward and the layer step above) over the recomputed rows
  stitch   every layer's cached keys moved to their prompt positions, then the KV-deviation selector on one layer

Inputs are random with planted structure: `k` context tokens per request stand out to the question (or deviate between
the two K tensors), so the set that a selection has to return is known and does not hang on the last bits of a score.
"""
import math

import numpy as np
import torch

from paper_2601_12904_amd import binding as B
from paper_2601_12904_amd import stack as S

NORMS = {"chunk": B.FR_NORM_PER_CHUNK, "global": B.FR_NORM_GLOBAL, "raw": B.FR_NORM_RAW}
TORCH = {"bf16": torch.bfloat16, "f32": torch.float32}

GQA4 = dict(q_heads=32, kv_heads=8, head_dim=128, dtype="bf16", rope_base=500000.0)    # the 8B-class layer
GQA7 = dict(q_heads=28, kv_heads=4, head_dim=128, dtype="bf16", rope_base=1000000.0)   # the 7B-class layer with 4 KV heads
GQA8 = dict(q_heads=64, kv_heads=8, head_dim=128, dtype="bf16", rope_base=500000.0)
MHA64 = dict(q_heads=16, kv_heads=8, head_dim=64, dtype="bf16", rope_base=500000.0)    # small models, head_dim 64
TINY32 = dict(q_heads=4, kv_heads=4, head_dim=64, dtype="f32", rope_base=10000.0)      # fp32: verification runs

PROMPT = dict(norm="chunk", half_layout=False, fused=False, ragged=False)


def listed():
    return [
        # The smallest request in fp32, 4 x 128 + 32 tokens: a verification run, all launches and latency.
        dict(PROMPT, name="layer_tiny_f32", kind="layer", **TINY32, chunks=4, ctx=512, question=32, ratio=0.15),
        # A short prompt of odd chunks (880 + 40 tokens): interactive use, where launches count.
        dict(PROMPT, name="layer_short_ragged", kind="layer", **GQA4, chunks=4, ctx=880, question=40, ratio=0.15) | dict(ragged=True),
        # The ordinary request: 16 x 1024 + 512 tokens, 15 % recomputed.
        dict(PROMPT, name="layer_17k", kind="layer", **GQA4, chunks=16, ctx=16384, question=512, ratio=0.15),
        # A long request: 64 ragged chunks, 33.8k tokens, write-back fused into the attention call.
        dict(PROMPT, name="layer_33k_ragged", kind="layer", **GQA4, chunks=64, ctx=32768, question=1024, ratio=0.15) | dict(ragged=True, fused=True),
        # The ordinary request on a layer with 28 query and 4 KV heads, in the half-split rotary layout such models use.
        dict(PROMPT, name="layer_17k_group7", kind="layer", **GQA7, chunks=16, ctx=16384, question=512, ratio=0.15) | dict(half_layout=True),
        # Every row recomputed: the dense end of the ratio sweep, equal to a full causal prefill.
        dict(PROMPT, name="layer_17k_full", kind="layer", **GQA4, chunks=16, ctx=16384, question=512, ratio=1.0),
        # Eight requests served together, each drawing 16 of 32 cached chunks.
        dict(name="shared_8_requests", kind="shared", **GQA4, half_layout=False, requests=8, store_chunks=32, chunks=16, chunk=1024, question=512, ratio=0.15),
        # A 1024-token chunk preprocessed behind a 64-token system prompt and its 10 nearest chunks.
        dict(name="offline_chunk", kind="offline", **GQA4, half_layout=False, top=10, chunk=1024, system=64),
        # A decoding step of a full batch, every request with 16 chunks of its own: streaming.
        dict(name="decode_32", kind="decode", **GQA4, half_layout=False, requests=32, chunks=16, chunk=1024, store_chunks=512, page=2978, ratio=0.15),
        # A decoding step of two requests: too few of them to fill the chip by number.
        dict(name="decode_2", kind="decode", **GQA4, half_layout=False, requests=2, chunks=16, chunk=1024, store_chunks=32, page=2978, ratio=0.15),
        # Two of the decoder layers of the ordinary request: the projections of 2970 rows around the layer step.
        dict(name="stack_17k", kind="stack", **GQA4, half_layout=False, layers=2, hidden=4096, ffn=14336, chunks=16, ctx=16384, question=512, ratio=0.15, select=True),
        # All 32 layers' cached keys stitched for a request, then the KV-deviation selector on the second layer.
        dict(name="stitch_32_layers", kind="stitch", **GQA4, half_layout=False, layers=32, chunks=16, ctx=16384, question=512, ratio=0.15),
    ]


def _spread(rng, lo, hi):
    """A whole number of [lo, hi], uniform in its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["layer"] * 6 + ["shared", "offline", "decode", "decode", "stack", "stitch"])
    ratio = rng.choice([0.0] + [round(math.exp(rng.uniform(math.log(0.02), math.log(0.5))), 3)] * 7)
    half = rng.random() < 0.5
    if kind == "layer":
        layer = rng.choice([GQA4] * 4 + [GQA7, GQA8, MHA64, TINY32])
        ctx = _spread(rng, 256, 32768 if layer in (GQA4, GQA8) else 16384 if layer is GQA7 else 8192 if layer is MHA64 else 1024)
        question = _spread(rng, 16, 1024 if ctx >= 4096 else 256)
        if ctx <= 16384 and layer in (GQA4, GQA8) and rng.random() < 0.08:
            ratio = 1.0
        case = dict(kind=kind, **layer, norm=rng.choice(["chunk"] * 5 + ["global", "raw"]), half_layout=half, fused=rng.random() < 0.5,
                    ragged=rng.random() < 0.7, chunks=_spread(rng, 1, max(1, min(64, ctx // 128))), ctx=ctx, question=question, ratio=ratio)
        while work(case)["flops"] > (4.7e11 if layer is GQA7 else 2.4e12):     # no more than the listed requests of the layer
            case["ratio"] = round(0.8 * case["ratio"], 3)
        return case
    if kind == "shared":
        chunks = rng.randint(2, 16)
        return dict(kind=kind, **rng.choice([GQA4, GQA4, GQA8]), half_layout=half, requests=rng.randint(1, 8), store_chunks=rng.randint(chunks, 32),
                    chunks=chunks, chunk=_spread(rng, 100, 1024), question=_spread(rng, 16, 512), ratio=min(ratio, 0.25))
    if kind == "offline":
        return dict(kind=kind, **rng.choice([GQA4, GQA4, GQA8]), half_layout=half, top=rng.randint(1, 10), chunk=_spread(rng, 128, 1536), system=rng.randint(1, 200))
    if kind == "decode":
        requests, chunks, chunk = _spread(rng, 1, 32), rng.randint(2, 16), _spread(rng, 100, 1024)
        own = rng.random() < 0.5
        ratio = max(ratio, 0.02)
        page = int(ratio * chunks * chunk) + rng.randint(20, 520)
        return dict(kind=kind, **rng.choice([GQA4, GQA4, GQA8]), half_layout=half, requests=requests, chunks=chunks, chunk=chunk,
                    store_chunks=requests * chunks if own else max(chunks, 48), page=page, ratio=ratio)
    if kind == "stack":
        ctx = _spread(rng, 512, 16384)
        return dict(kind=kind, **GQA4, half_layout=False, layers=rng.randint(1, 2), hidden=4096, ffn=14336, chunks=max(1, ctx // 1000), ctx=ctx,
                    question=_spread(rng, 16, 512), ratio=min(ratio, 0.15), select=rng.random() < 0.5)
    ctx = _spread(rng, 1024, 16384)
    return dict(kind=kind, **rng.choice([GQA4, GQA7]), half_layout=half, layers=rng.randint(2, 32), chunks=max(1, ctx // 1000), ctx=ctx,
                question=_spread(rng, 16, 512), ratio=ratio)


# ---- sizes that follow from a case ----------------------------------------------------------------------------------

def _offsets(case):
    """Chunk boundaries of a prompt: equal parts, or ragged ones between a half and one and a half of the mean."""
    n, total = case["chunks"], case["ctx"]
    if case.get("ragged"):
        w = 0.5 + np.random.default_rng([n, total]).random(n)
        cut = np.floor(np.cumsum(w) / w.sum() * total).astype(np.int32)
    else:
        cut = (np.arange(1, n + 1, dtype=np.int64) * total // n).astype(np.int32)
    cut[-1] = total
    return np.concatenate([np.zeros(1, np.int32), cut])


def _count(tokens, ratio):
    return min(tokens, int(math.floor(ratio * tokens + 0.5)))


def _pairs(ctx, k, question):
    """(row, key) pairs of the causal attention of k context rows, spread over the context, and the question's rows."""
    return k * (ctx + 1) / 2 + question * ctx + question * (question + 1) / 2


def _shared_count(case):
    """Chosen context tokens of a request over the store: the same number from each of its chunks."""
    return case["chunks"] * -(-_count(case["chunks"] * case["chunk"], case["ratio"]) // case["chunks"])


# ---- inputs ---------------------------------------------------------------------------------------------------------

class _Draws:
    """Random device tensors of one layer shape from one seed.  Unit-scale logits: q ~ N(0, d), k, v ~ N(0, 1/d)."""

    def __init__(self, case, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(1000003 * seed + 17)
        self.rng = np.random.default_rng(seed)
        self.d, self.hq, self.hkv = case["head_dim"], case["q_heads"], case["kv_heads"]
        self.t = TORCH[case["dtype"]]
        # One direction per KV head, inside the lowest-frequency rotary pairs, which a prompt's length hardly turns: what
        # the question asks for.
        d, p = self.d, max(1, self.d // 16)
        dims = list(range(d // 2 - p, d // 2)) + list(range(d - p, d)) if case.get("half_layout") else list(range(d - 2 * p, d))
        u = torch.zeros((self.hkv, d), device="cuda")
        u[:, dims] = torch.randn((self.hkv, 2 * p), generator=self.g, device="cuda")
        self.u = u / u.norm(dim=1, keepdim=True)

    def kv(self, *shape):
        return (torch.randn((*shape, self.hkv, self.d), generator=self.g, device="cuda") / math.sqrt(self.d)).to(self.t)

    def keys(self, rows, focus):
        """Keys [rows, Hkv, d] of which those of `focus` lie along the direction the question asks for."""
        k = torch.randn((rows, self.hkv, self.d), generator=self.g, device="cuda") / math.sqrt(self.d)
        k -= (k * self.u).sum(-1, keepdim=True) * self.u
        if len(focus):
            k[torch.from_numpy(focus).cuda()] += 3.0 / math.sqrt(self.d) * self.u
        return k.to(self.t)

    def queries(self, rows, question=0):
        """Queries [rows, Hq, d], the last `question` of them the question's."""
        q = torch.randn((rows, self.hq, self.d), generator=self.g, device="cuda") * math.sqrt(self.d)
        if question:
            q[rows - question:] += self.d * self.u.repeat_interleave(self.hq // self.hkv, dim=0)
        return q.to(self.t)

    def choose(self, n, k):
        return np.sort(self.rng.choice(n, size=k, replace=False)).astype(np.int64)


def _context(case, tokens, chunks, question):
    return B.Context(case["q_heads"], case["kv_heads"], case["head_dim"], B.FR_F32 if case["dtype"] == "f32" else B.FR_BF16, case["rope_base"],
                     max_tokens=tokens, max_chunks=chunks, max_question_tokens=question,
                     rope_layout=B.FR_ROPE_HALF if case["half_layout"] else B.FR_ROPE_INTERLEAVED)


def _prompt(case, seed, s):
    """What a request brings: its row set (context tokens the question asks for, then the question) and its chunks."""
    r = _Draws(case, seed)
    ctx, nq = case["ctx"], case["question"]
    k = _count(ctx, case["ratio"])
    focus = r.choose(ctx, k)
    s.update(ctx_tokens=ctx, nq=nq, k=k, R=k + nq, L=ctx + nq, offs=_offsets(case), focus=focus, draws=r)
    s["src"] = r.rng.integers(0, min(4096, ctx), size=case["chunks"]).astype(np.int32)
    s["q_index"] = torch.empty(k + nq, dtype=torch.int32, device="cuda")
    return r


def _prepare_layer(case, seed, s):
    r = _prompt(case, seed, s)
    s["c"] = _context(case, s["L"], case["chunks"], s["nq"])
    s["k_cached"] = r.keys(s["ctx_tokens"], s["focus"])
    s["k_cache"] = torch.zeros((s["L"], r.hkv, r.d), dtype=r.t, device="cuda")
    s["v_cache"] = r.kv(s["L"])
    s["q_rows"] = r.queries(s["R"], s["nq"])
    s["q_question"] = s["q_rows"][s["k"]:].contiguous()
    s["k_new"], s["v_new"] = r.kv(s["R"]), r.kv(s["R"])
    s["scores"] = torch.empty(s["ctx_tokens"], dtype=torch.float32, device="cuda")
    s["out"] = torch.empty_like(s["q_rows"])


def _run_layer(s):
    c, case = s["c"], s["case"]
    c.fr_rope_shift(s["k_cached"], s["k_cache"], s["offs"], s["src"])
    c.fr_score_select(s["q_question"], s["nq"], s["k_cache"], s["offs"], s["k"], NORMS[case["norm"]], s["scores"], s["q_index"])
    args = (s["q_rows"], s["q_index"], s["R"], s["k_cache"], s["v_cache"], s["L"], s["k_new"], s["v_new"], s["out"])
    if case["fused"]:
        c.fr_sparse_prefill_attn_writeback(*args)
    else:
        c.fr_sparse_prefill_attn(*args)
        c.fr_kv_scatter(s["k_new"], s["v_new"], s["q_index"], s["R"], s["k_cache"], s["v_cache"], s["L"])
    return {"scores": s["scores"], "q_index": s["q_index"], "out": s["out"], "k_cache": s["k_cache"], "v_cache": s["v_cache"]}


def _prepare_shared(case, seed, s):
    r = _Draws(case, seed)
    n, clen, nq = case["store_chunks"] * case["chunk"], case["chunk"], case["question"]
    ctx, k = case["chunks"] * clen, _shared_count(case)
    R = k + nq
    s.update(n=n, k=k, nq=nq, L=ctx + nq, R=R, offs=np.arange(0, ctx + 1, clen, dtype=np.int32))
    s["c"] = _context(case, s["L"], case["chunks"], nq)
    # the same tokens of a chunk stand out in every request that uses it
    marks = [r.rng.choice(clen, size=k // case["chunks"], replace=False) + c * clen for c in range(case["store_chunks"])]
    s["k_store"], s["v_store"] = r.keys(n, np.concatenate(marks).astype(np.int64)), r.kv(n)
    s["requests"] = []
    for _ in range(case["requests"]):
        ids = r.rng.choice(case["store_chunks"], size=case["chunks"], replace=False)
        q = r.queries(R, nq)
        s["requests"].append(dict(
            q_rows=q, q_question=q[k:].contiguous(), q_index=torch.empty(R, dtype=torch.int32, device="cuda"), R=R, chunk_offsets=s["offs"],
            chunk_store_row0=(ids * clen).astype(np.int32), chunk_src_pos0=r.rng.integers(0, 4096, size=case["chunks"]).astype(np.int32), L=s["L"],
            k_new=r.kv(R), v_new=r.kv(R), out=torch.empty_like(q)))
    s["work"] = torch.empty(s["c"].fr_shared_batch_workspace_bytes(case["requests"], s["L"]), dtype=torch.uint8, device="cuda")


def _run_shared(s):
    c = s["c"]
    for q in s["requests"]:
        c.fr_score_select_shared(q["q_question"], s["nq"], s["k_store"], s["n"], s["offs"], q["chunk_store_row0"], q["chunk_src_pos0"], s["k"],
                                 B.FR_NORM_PER_CHUNK, None, q["q_index"])
    c.fr_sparse_prefill_attn_shared_batch(s["requests"], s["k_store"], s["v_store"], s["n"], s["work"])
    return {"q_index": [q["q_index"] for q in s["requests"]], "out": [q["out"] for q in s["requests"]]}


def _prepare_offline(case, seed, s):
    r = _Draws(case, seed)
    lens = [case["system"]] + [case["chunk"]] * case["top"]
    offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    p, n = int(offs[-1]), case["chunk"]
    s.update(offs=offs, L=p + n, R=n, src=r.rng.integers(0, 4096, size=len(lens)).astype(np.int32))
    s["c"] = _context(case, p + n, len(lens), 16)
    s["k_cached"] = r.kv(p)
    s["k_cache"] = torch.zeros((p + n, r.hkv, r.d), dtype=r.t, device="cuda")
    s["v_cache"] = r.kv(p + n)
    s["q_rows"], s["k_new"], s["v_new"] = r.queries(n), r.kv(n), r.kv(n)
    s["q_index"] = torch.arange(p, p + n, dtype=torch.int32, device="cuda")
    s["out"] = torch.empty_like(s["q_rows"])


def _run_offline(s):
    c = s["c"]
    c.fr_rope_shift(s["k_cached"], s["k_cache"], s["offs"], s["src"])
    c.fr_sparse_prefill_attn(s["q_rows"], s["q_index"], s["R"], s["k_cache"], s["v_cache"], s["L"], s["k_new"], s["v_new"], s["out"])
    return {"out": s["out"]}


def _prepare_decode(case, seed, s):
    r = _Draws(case, seed)
    nb, per, clen, page = case["requests"], case["chunks"], case["chunk"], case["page"]
    n = case["store_chunks"] * clen
    words = (n + 31) // 32
    own = case["store_chunks"] == nb * per
    s.update(nb=nb, n=n, words=words, page=page, n_seg=nb * per)
    s["c"] = _context(case, 1024, 4, 8)
    s["k_store"], s["v_store"] = r.kv(n), r.kv(n)
    s["bits"] = torch.zeros((nb, words), dtype=torch.int32, device="cuda")
    row0, delta = [], []
    for b in range(nb):
        ids = np.arange(b * per, (b + 1) * per) if own else r.rng.choice(case["store_chunks"], size=per, replace=False)
        row0 += [int(i) * clen for i in ids]
        delta += [j * clen - int(r.rng.integers(0, 4096)) for j in range(per)]
        stale = r.choose(per * clen, _count(per * clen, case["ratio"]))
        rows = torch.from_numpy((ids[stale // clen] * clen + stale % clen).astype(np.int32)).cuda()
        s["c"].fr_mark_stale_rows(s["bits"][b], words, rows, len(stale), clear=True)
    i32 = lambda v: torch.tensor(v, dtype=torch.int32, device="cuda")  # noqa: E731
    s["seg_offsets"], s["row0"], s["len"], s["delta"] = i32(list(range(0, nb * per + 1, per))), i32(row0), i32([clen] * (nb * per)), i32(delta)
    s["q"], s["k_pages"], s["v_pages"] = r.queries(nb), r.kv(nb, page), r.kv(nb, page)
    s["page_len"] = i32([page - int(v) for v in r.rng.integers(0, 12, size=nb)])   # the requests are at different tokens
    s["out"] = torch.empty_like(s["q"])


def _run_decode(s):
    s["c"].fr_decode_attn(s["q"], s["nb"], s["k_store"], s["v_store"], s["n"], s["seg_offsets"], s["row0"], s["len"], s["delta"], s["n_seg"],
                          s["bits"], s["words"], s["k_pages"], s["v_pages"], s["page"], s["page_len"], s["out"])
    return {"out": s["out"]}


def _prepare_stack(case, seed, s):
    r = _prompt(case, seed, s)
    n, hidden = case["layers"], case["hidden"]
    s["c"] = _context(case, s["L"], case["chunks"], s["nq"])
    s["rows"] = torch.from_numpy(np.concatenate([s["focus"], s["ctx_tokens"] + np.arange(s["nq"])]).astype(np.int32)).cuda()
    layers = [S.random_layer(hidden, case["ffn"], r.hq, r.hkv, r.d, r.g) for _ in range(n)]
    s["stack"] = S.SelectivePrefillStack(s["c"], layers, hidden, case["ffn"])
    s["k_cached"] = [r.kv(s["ctx_tokens"]) for _ in range(n)]
    s["k_cache"] = [torch.zeros((s["L"], r.hkv, r.d), dtype=r.t, device="cuda") for _ in range(n)]
    s["v_cache"] = [r.kv(s["L"]) for _ in range(n)]
    s["h"] = torch.randn((s["R"], hidden), generator=r.g, device="cuda").to(torch.bfloat16)


def _run_stack(s):
    h = s["h"].clone()      # forward() works in place
    s["stack"].forward(h, s["rows"], s["k_cached"], s["k_cache"], s["v_cache"], s["offs"], s["src"], s["nq"], s["L"],
                       select_every_layer=s["case"]["select"], k_select=s["k"], q_index_scratch=s["q_index"])
    return {"h": h, "k_cache": s["k_cache"], "v_cache": s["v_cache"]}


def _prepare_stitch(case, seed, s):
    r = _prompt(case, seed, s)
    n, ctx = case["layers"], case["ctx"]
    s["c"] = _context(case, s["L"], case["chunks"], s["nq"])
    s["k_cached"] = torch.stack([r.kv(ctx) for _ in range(n)])
    s["k_cache"] = torch.zeros((n, s["L"], r.hkv, r.d), dtype=r.t, device="cuda")
    # the second layer's keys of full attention: near the stitched ones but for the tokens that deviate
    s["c"].fr_rope_shift(s["k_cached"][1], s["k_cache"][1], s["offs"], s["src"])
    full = s["k_cache"][1, :ctx].float() + 0.02 * r.kv(ctx).float()
    if s["k"]:
        full[torch.from_numpy(s["focus"]).cuda()] += 0.3 * r.kv(s["k"]).float()
    s["k_full"] = full.to(r.t)
    s["k_cache"].zero_()
    s["deviation"] = torch.empty(ctx, dtype=torch.float32, device="cuda")


def _run_stitch(s):
    c, (n, L, hkv, d) = s["c"], s["k_cache"].shape
    c.fr_rope_shift(s["k_cached"], s["k_cache"], s["offs"], s["src"], n_batch=n, src_batch_stride=s["ctx_tokens"] * hkv * d, dst_batch_stride=L * hkv * d)
    c.fr_kv_deviation(s["k_full"], s["k_cache"][1], s["ctx_tokens"], s["deviation"])
    c.fr_select_topk(s["deviation"], s["ctx_tokens"], s["k"], s["nq"], s["q_index"])
    return {"k_cache": s["k_cache"], "deviation": s["deviation"], "q_index": s["q_index"]}


PREPARE = {"layer": _prepare_layer, "shared": _prepare_shared, "offline": _prepare_offline, "decode": _prepare_decode, "stack": _prepare_stack,
           "stitch": _prepare_stitch}
RUN = {"layer": _run_layer, "shared": _run_shared, "offline": _run_offline, "decode": _run_decode, "stack": _run_stack, "stitch": _run_stitch}


def prepare(case, seed):
    s = {"case": case}
    PREPARE[case["kind"]](case, seed, s)
    s.pop("draws", None)
    return s


def run(state):
    return RUN[state["case"]["kind"]](state)


def work(case):
    d, hq, hkv = case["head_dim"], case["q_heads"], case["kv_heads"]
    e = 4 if case["dtype"] == "f32" else 2
    row, kind = hkv * d * e, case["kind"]          # bytes of one token's keys or values
    qrow = hq * d * e
    if kind == "decode":
        nb, per = case["requests"], case["chunks"] * case["chunk"]
        stale = _count(per, case["ratio"])
        used = nb * (per - stale + case["page"])
        shared = case["store_chunks"] != nb * case["chunks"]
        once = (min(case["store_chunks"] * case["chunk"], nb * (per - stale)) if shared else nb * (per - stale)) + nb * case["page"]
        return {"bytes": 2 * once * row + 2 * nb * qrow, "flops": 4 * used * hq * d}
    if kind == "offline":
        p, n = case["system"] + case["top"] * case["chunk"], case["chunk"]
        return {"bytes": (2 * p + p + 2 * n) * row + 2 * n * qrow, "flops": 4 * d * hq * (n * p + n * (n + 1) / 2)}
    if kind == "shared":
        nb, ctx, nq = case["requests"], case["chunks"] * case["chunk"], case["question"]
        k = _shared_count(case)
        store = min(case["store_chunks"], nb * case["chunks"]) * case["chunk"]
        return {"bytes": 2 * store * row + nb * ((k + nq) * (2 * row + 2 * qrow) + 4 * (k + nq)),
                "flops": nb * (2 * nq * hq * ctx * d + 4 * d * hq * _pairs(ctx, k, nq))}
    ctx, nq = case["ctx"], case["question"]
    k = _count(ctx, case["ratio"])
    R = k + nq
    if kind == "stitch":
        return {"bytes": 2 * case["layers"] * ctx * row + ctx * row + 4 * ctx + 4 * R, "flops": 6 * case["layers"] * ctx * hkv * d / 2}
    # stitched keys in and out, values in, the recomputed rows' K/V in and into the cache, queries in, output out
    data = (3 * ctx + 4 * R) * row + 2 * R * qrow + 4 * ctx + 4 * R
    score = 2 * nq * hq * ctx * d if case.get("norm") != "raw" else 2 * ctx * hkv * d
    attn = 4 * d * hq * _pairs(ctx, k, nq)
    if kind == "layer":
        return {"bytes": data, "flops": score + attn}
    hidden, ffn = case["hidden"], case["ffn"]
    weights = (hq + 2 * hkv) * d * hidden + hq * d * hidden + 3 * hidden * ffn
    data = (3 * ctx + 2 * R) * row                 # queries, fresh K/V and attention output stay inside a layer
    return {"bytes": case["layers"] * (data + 2 * weights) + 2 * R * hidden * 2,
            "flops": case["layers"] * (2 * R * weights + attn + (score if case["select"] else 0))}


def tolerance(case):
    # bf16: results and the weights of the value sums are rounded to 8 bits.  Against float64 an attention output is 2.1e-3
    # off (2-norm) and 0.027 at most; two layers of the stack with their products in another order 5.0e-3 and 0.045.  fp32:
    # 2e-7 and 3e-6 for an attention output, whose exponentials and sums may go in any order.
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-4, "differ": 0.0}
    if case["kind"] == "stack":
        return {"rel": 2e-2, "max": 0.2, "differ": 0.0}
    return {"rel": 1e-2, "max": 0.1, "differ": 0.0}
