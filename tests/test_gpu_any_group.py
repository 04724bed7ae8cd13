"""The matrix-core kernels at group sizes and head dimensions that have no instance of their own (any number of query
heads per KV head up to 64, head_dim 64), against the oracle: `pytest -m gpu`."""
import numpy as np
import pytest
import torch

from oracle import fusionrag_oracle as orc
from paper_2601_12904_amd import binding as B
from paper_2601_12904_amd import synth
from tests import harness as H
from tests.test_gpu_parity import assembled_cache, one_launch, run_attention, run_attention_over_store, staged

pytestmark = pytest.mark.gpu

# Outputs are rounded to bf16 once: 8 significant bits (one of them implicit), so half a unit is up to 2^-8 of the element
# and of the tensor's largest value at most.  The weights and the sums are fp32, so nothing else shows at this scale.
OUT_TOL = 2.0 ** -8 + 2.0 ** -14


def workload(Hq, Hkv, d, lens, nq, ratio=0.2):
    shape = synth.LayerShape(n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, dtype="bf16", rope_base=500000.0)
    return synth.config_small_bf16(seed=Hq + d, ratio=ratio, chunk_lens=lens, nq=nq, shape=shape)


# (query heads, KV heads, head_dim): rows per wave floor(64 / G) from 64 down to 1; columns left idle: none, 1 (G = 7), 4 (5), 21 (43)
SHAPES = [(7, 1, 128), (28, 4, 128), (6, 2, 128), (5, 1, 128), (16, 1, 128), (43, 1, 128), (64, 1, 128), (2, 2, 64), (8, 4, 64), (14, 2, 64), (64, 2, 64)]


@pytest.mark.parametrize("split", [B.FR_ATTN_SPLIT_OFF, B.FR_ATTN_SPLIT_ON])
@pytest.mark.parametrize("Hq,Hkv,d", SHAPES)
def test_attention(Hq, Hkv, d, split):
    w = workload(Hq, Hkv, d, (130, 0, 333, 61), 37)
    k_ctx, _, k, qi = staged(w)
    k_cache, v_cache = assembled_cache(w, k_ctx)
    ctx = H.make_ctx(w.shape, w.L, w.n_chunks, w.nq)
    ctx.fr_set_option(B.FR_OPT_ATTN_SPLIT, split)
    got, lse = run_attention(ctx, w, qi, k_cache, v_cache)
    want, want_lse = orc.sparse_prefill_attn(w.q_full[qi], qi, k_cache, v_cache, w.k_full[qi], w.v_full[qi])
    assert H.max_rel_err(got, want) <= OUT_TOL
    assert np.max(np.abs(lse - want_lse)) <= 1e-4
    kc, vc = H.dev(k_cache, "bf16"), H.dev(v_cache, "bf16")
    out = torch.zeros((len(qi), Hq, d), dtype=torch.bfloat16, device="cuda")
    ctx.fr_sparse_prefill_attn_writeback(H.dev(w.q_full[qi], "bf16"), torch.from_numpy(qi.astype(np.int32)).cuda(), len(qi), kc, vc,
                                         w.L, H.dev(w.k_full[qi], "bf16"), H.dev(w.v_full[qi], "bf16"), out)
    torch.cuda.synchronize()
    assert H.max_rel_err(H.host(out), want) <= OUT_TOL
    k_eff, v_eff = orc.kv_scatter(qi, w.k_full[qi], w.v_full[qi], k_cache, v_cache)
    assert np.array_equal(H.host(kc), k_eff) and np.array_equal(H.host(vc), v_eff)
    ctx.close()


@pytest.mark.parametrize("split", [B.FR_ATTN_SPLIT_AUTO, B.FR_ATTN_SPLIT_OFF, B.FR_ATTN_SPLIT_ON])
@pytest.mark.parametrize("Hq,Hkv,d", [(7, 1, 128), (2, 1, 64)])
def test_weights_keep_32_bits(Hq, Hkv, d, split):
    """Values whose weighted sum nearly cancels for the last row and head 0 (signs against the running sum, the rest into one
    key): what is left, about 1e-6, is rounded to bf16 at 1e-9 and shows the weights' own errors.  A weight in fp32 is off
    by some 2^-22 (a logit's sum, its scale and the exponential, 2^-24 each of a few units), one of 16 bits by up to 2^-17;
    independent errors of unit values add up to that times the root of the weights' squares.  2^-20 lies between.  In one launch (AUTO) and
    tiled, whole and in parts."""
    w = workload(Hq, Hkv, d, (200, 120), 20)
    L, rng = w.L, np.random.default_rng(d)
    logits = (w.k_full[:, 0].astype(np.float64) @ w.q_full[L - 1, 0].astype(np.float64)) / np.sqrt(d)
    weight = np.exp(logits - logits.max())
    weight /= weight.sum()
    v = np.zeros((L, Hkv, d), dtype=np.float32)
    for e in range(d):
        order, total = rng.permutation(L), 0.0
        for j in order[:-3]:
            v[j, 0, e] = -1.0 if total > 0 else 1.0
            total += weight[j] * v[j, 0, e]
        for j in order[-3:]:
            v[j, 0, e] = synth.round_to_storage(np.float32([-total / weight[j]]), "bf16")[0]
            total += weight[j] * v[j, 0, e]
    want = weight @ v[:, 0].astype(np.float64)
    assert one_launch(w, np.arange(L))      # (AUTO)
    ctx = H.make_ctx(w.shape, L, w.n_chunks, w.nq)
    ctx.fr_set_option(B.FR_OPT_ATTN_SPLIT, split)
    got, _ = run_attention(ctx, w, np.arange(L), w.k_full, v, with_new=False)
    ctx.close()
    assert np.max(np.abs(want)) < 1e-4
    assert np.sqrt(np.mean((got[L - 1, 0] - want) ** 2)) <= 2.0 ** -20 * np.sqrt(np.sum((weight[:, None] * v[:, 0]) ** 2) / d)


@pytest.mark.parametrize("split", [B.FR_ATTN_SPLIT_OFF, B.FR_ATTN_SPLIT_ON])
@pytest.mark.parametrize("Hq,Hkv,d", [(7, 1, 128), (4, 2, 64)])
def test_attention_logits_beyond_the_fixed_reference(Hq, Hkv, d, split):
    """A few keys whose logits lie far above those of the first 32 keys: the sums overflow and the rows are recomputed."""
    w = workload(Hq, Hkv, d, (200, 120), 20, ratio=0.1)
    k_ctx, _, k, qi = staged(w)
    k_cache, v_cache = assembled_cache(w, k_ctx)
    q = w.q_full.copy()
    hot = [150, 210]
    for j in hot:
        k_cache[j] = 0.0
        k_cache[j, :, 0] = 40.0
    q[:, :, 0] = 60.0
    q, k_cache = synth.round_to_storage(q, "bf16"), synth.round_to_storage(k_cache, "bf16")
    qi = np.array([i for i in qi if i not in hot])
    w.q_full = q
    ctx = H.make_ctx(w.shape, w.L, w.n_chunks, w.nq)
    ctx.fr_set_option(B.FR_OPT_ATTN_SPLIT, split)
    got, _ = run_attention(ctx, w, qi, k_cache, v_cache)
    want, _ = orc.sparse_prefill_attn(q[qi], qi, k_cache, v_cache, w.k_full[qi], w.v_full[qi])
    assert H.max_rel_err(got, want) <= OUT_TOL
    ctx.close()


# Parts of an item in 32 bits (short prompts; more than four; split weights, in up to eight parts beyond the positions of the one-launch kernel) and in half
# precision (two, four parts of 33 key tiles), parts without a key among them, whole items, and the one-launch kernel
STORE = "over a store"      # (the tiled kernels, AUTO)


@pytest.mark.parametrize("Hq,Hkv,d,total,split", [(8, 2, 128, 1300, B.FR_ATTN_SPLIT_AUTO), (2, 2, 128, 700, B.FR_ATTN_SPLIT_ON), (7, 1, 128, 1300, B.FR_ATTN_SPLIT_AUTO),
                                                  (4, 2, 64, 1300, B.FR_ATTN_SPLIT_AUTO), (8, 2, 128, 2100, B.FR_ATTN_SPLIT_ON), (80, 10, 128, 2100, B.FR_ATTN_SPLIT_AUTO),
                                                  (8, 2, 128, 2100, B.FR_ATTN_SPLIT_AUTO), (8, 2, 128, 700, B.FR_ATTN_SPLIT_OFF), (7, 1, 128, 2100, B.FR_ATTN_SPLIT_ON),
                                                  (8, 2, 128, 1300, STORE), (8, 2, 128, 2100, STORE), (7, 1, 128, 6300, B.FR_ATTN_SPLIT_AUTO), (4, 2, 64, 6300, B.FR_ATTN_SPLIT_AUTO)])
@pytest.mark.parametrize("size", [16.25, 40.0])
def test_two_parts_beyond_the_reference(Hq, Hkv, d, total, split, size):
    """Two keys far apart whose logits, for one head of each group, lie 2^124 or 2^300 above the first ones (half of the latter at
    head_dim 64 and more): what overflows is done again with a reference of its own, the rest is not, and both come together.  Weights and
    sums stay as precise as without."""
    w = workload(Hq, Hkv, d, (total - 20,), 20, ratio=0.05)
    w.q_full[:, ::Hq // Hkv, 0] = 60.0
    w.k_full[:, :, 0] *= 0.01
    for j, x in ((total // 4, size), (3 * total // 4, size + 0.125)):
        w.k_full[j] *= 0.01
        w.k_full[j, :, 0] = x
    w.k_full = synth.round_to_storage(w.k_full, "bf16")
    qi = np.concatenate([np.sort(np.random.default_rng(total).choice(total - 20, size=150, replace=False)), np.arange(total - 20, total)])
    assert one_launch(w, qi) == (total <= 2100 and Hkv < 10)      # (AUTO)
    ctx = H.make_ctx(w.shape, total, w.n_chunks, w.nq)
    ctx.fr_set_option(B.FR_OPT_ATTN_SPLIT, B.FR_ATTN_SPLIT_AUTO if split == STORE else split)
    got, lse = (run_attention_over_store if split == STORE else run_attention)(ctx, w, qi, w.k_full, w.v_full)
    want, want_lse = orc.sparse_prefill_attn(w.q_full[qi], qi, w.k_full, w.v_full, w.k_full[qi], w.v_full[qi])
    ctx.close()
    if Hq // Hkv == 7 or d == 64:
        assert H.max_rel_err(got, want) <= OUT_TOL
    else:
        H.assert_close(got, want, "bf16", "attention")
    assert np.max(np.abs(lse - want_lse) / np.maximum(1.0, np.abs(want_lse))) <= 1e-4


# Row tiles hold 4 floor(64 / G) rows.  Short prompts are cut up to 128 items (row tiles x KV heads; half of 256 compute units),
# prompts of 33 key tiles up to 64 log2(33 / 4) + 32 = 226: one case on either side of both lines, and two of few columns, which run in one launch.
@pytest.mark.parametrize("Hq,Hkv,d,lens", [(7, 1, 128, (500, 413)), (4, 2, 64, (500, 413)),                      # one launch
                                           (28, 4, 128, (500, 413)), (56, 8, 128, (500, 413)),                  # 112 in two parts, 224 whole
                                           (32, 16, 64, (500, 413)), (34, 17, 64, (500, 413)),                  # 128 in two parts, 136 whole
                                           (21, 3, 128, (1000, 990)), (42, 6, 128, (1000, 990)), (56, 8, 128, (1000, 990))])   # 174 in two parts, 348 and 464 whole
def test_items_on_both_sides_of_the_split_rules(Hq, Hkv, d, lens):
    """Every row of a prompt of several key tiles (100 % recompute equals dense causal attention)."""
    w = workload(Hq, Hkv, d, lens, 65, ratio=1.0)
    qi = np.arange(w.L)
    assert one_launch(w, qi) == (Hq <= 7)
    k_cache, v_cache = assembled_cache(w, w.k_cached)
    ctx = H.make_ctx(w.shape, w.L, w.n_chunks, w.nq)
    got, _ = run_attention(ctx, w, qi, k_cache, v_cache)
    rows = qi if Hq <= 7 else np.unique(np.concatenate([np.arange(0, w.L, 29), [w.L - 1]]))
    want, _ = orc.sparse_prefill_attn(w.q_full[qi], qi, k_cache, v_cache, w.k_full[qi], w.v_full[qi], rows=rows)
    assert H.max_rel_err(got[rows], want) <= OUT_TOL
    ctx.close()


# Items of split weights in more than two parts: few rows of a prompt beyond the positions of the one-launch kernel.  Items (row tiles x KV heads) of 256 compute
# units: 5 and 4 in eight parts, 32 in eight, 48 in five, 68 in three, 112 in two (two and more by counts), 16 of head_dim 64 in eight.
@pytest.mark.parametrize("Hq,Hkv,d,rows,parts", [(7, 1, 128, 150, 8), (16, 1, 128, 90, 8), (28, 4, 128, 280, 8), (28, 4, 128, 400, 5), (28, 4, 128, 600, 3), (28, 4, 128, 1000, 2),
                                                 (4, 2, 64, 1000, 8), (3, 1, 128, 84, 8)])
def test_items_of_split_weights_in_several_parts(Hq, Hkv, d, rows, parts):
    """Against the oracle, and against whole items: the parts keep 32 bits.  fp32 sums of n = 6200 weights differ by some 2^-24 sqrt(n) = 4.7e-6 of an
    element, which moves 2^-8 relative (one bf16 unit) in a share of 4.7e-6 / 2^-8 = 1.2e-3 of the elements: sqrt(1.2e-3) 2^-8 = 1.4e-4 of the norm."""
    w = workload(Hq, Hkv, d, (3000, 3140), 60)
    qi = np.concatenate([np.sort(np.random.default_rng(rows).choice(w.L_ctx, size=rows - w.nq, replace=False)), np.arange(w.L_ctx, w.L)])
    items = -(-rows // (4 * (64 // (Hq // Hkv)))) * Hkv
    assert not one_launch(w, qi) and min(8, torch.cuda.get_device_properties(0).multi_processor_count // items) == parts
    k_cache, v_cache = assembled_cache(w, w.k_cached)
    outs = []
    for split in (B.FR_ATTN_SPLIT_OFF, B.FR_ATTN_SPLIT_AUTO):
        ctx = H.make_ctx(w.shape, w.L, w.n_chunks, w.nq)
        ctx.fr_set_option(B.FR_OPT_ATTN_SPLIT, split)
        outs.append(run_attention(ctx, w, qi, k_cache, v_cache))
        ctx.close()
    some = np.unique(np.concatenate([np.arange(0, rows, 5), [rows - 1]]))
    want, want_lse = orc.sparse_prefill_attn(w.q_full[qi], qi, k_cache, v_cache, w.k_full[qi], w.v_full[qi], rows=some)
    for got, lse in outs:
        assert H.max_rel_err(got[some], want) <= OUT_TOL
        assert np.max(np.abs(lse[some] - want_lse)) <= 1e-4
    off = np.linalg.norm(outs[1][0] - outs[0][0]) / np.linalg.norm(outs[0][0])
    assert 0.0 < off <= 2e-4 or np.any(outs[1][1] != outs[0][1])      # (the order of the sums shows that there are parts)
    assert off <= 2e-4


@pytest.mark.parametrize("Hq,Hkv,d,total,parts", [(64, 1, 128, 448, 1), (64, 1, 128, 449, 2), (60, 20, 64, 448, 1), (60, 20, 64, 460, 2)])
def test_where_items_of_split_weights_stay_whole(Hq, Hkv, d, total, parts):
    """More columns than one launch takes, up to 128 items (row tiles of 4 and of 84 rows x KV heads): seven key tiles stay whole, bit for bit the result with the cutting off, eight are
    cut in two."""
    w = workload(Hq, Hkv, d, (total - 10,), 10)
    qi = np.arange(total) if Hkv == 1 else np.sort(np.random.default_rng(total).choice(total, 400, replace=False))
    items = -(-len(qi) // (4 * (64 // (Hq // Hkv)))) * Hkv
    assert not one_launch(w, qi) and 64 < items <= 128 and -(-total // 64) == 6 + parts
    outs = []
    for split in (B.FR_ATTN_SPLIT_OFF, B.FR_ATTN_SPLIT_AUTO):
        ctx = H.make_ctx(w.shape, w.L, w.n_chunks, w.nq)
        ctx.fr_set_option(B.FR_OPT_ATTN_SPLIT, split)
        outs.append(run_attention(ctx, w, qi, w.k_full, w.v_full))
        ctx.close()
    assert np.any(outs[1][1] != outs[0][1]) == (parts == 2)
    assert np.linalg.norm(outs[1][0] - outs[0][0]) <= (0.0 if parts == 1 else 1.2e-4) * np.linalg.norm(outs[0][0])
    some = np.arange(0, len(qi), 7)
    want, _ = orc.sparse_prefill_attn(w.q_full[qi], qi, w.k_full, w.v_full, w.k_full[qi], w.v_full[qi], rows=some)
    assert H.max_rel_err(outs[1][0][some], want) <= OUT_TOL


# Key tiles are 64 keys in two halves, one per wave of a row group, and the tile loop runs three tiles ahead: prompts of one half tile to
# five tiles, whole and in parts of one tile and of none (by the rule: over a store), and the one-launch kernel (AUTO).  (bf16 weights: the tolerance of the other
# tests of those shapes.)
@pytest.mark.parametrize("Hq,Hkv,d,split", [(*shape, split) for shape in ((4, 4, 128), (8, 2, 128), (7, 1, 128), (4, 2, 64))
                                            for split in (B.FR_ATTN_SPLIT_OFF, B.FR_ATTN_SPLIT_ON, B.FR_ATTN_SPLIT_AUTO)] + [(4, 4, 128, STORE), (8, 2, 128, STORE)])
@pytest.mark.parametrize("total", [2, 31, 32, 33, 63, 64, 65, 128, 129, 191, 256, 319, 320])
def test_few_key_tiles(Hq, Hkv, d, total, split):
    w = workload(Hq, Hkv, d, (total - 1,), 1, ratio=1.0)
    qi = np.arange(w.L)
    assert one_launch(w, qi)      # (AUTO)
    k_cache, v_cache = assembled_cache(w, w.k_cached)
    ctx = H.make_ctx(w.shape, w.L, w.n_chunks, w.nq)
    ctx.fr_set_option(B.FR_OPT_ATTN_SPLIT, B.FR_ATTN_SPLIT_AUTO if split == STORE else split)
    got, lse = (run_attention_over_store if split == STORE else run_attention)(ctx, w, qi, k_cache, v_cache)
    want, want_lse = orc.sparse_prefill_attn(w.q_full[qi], qi, k_cache, v_cache, w.k_full[qi], w.v_full[qi])
    if (Hq, d) == (7, 128) or d == 64:
        assert H.max_rel_err(got, want) <= OUT_TOL
    else:
        H.assert_close(got, want, "bf16", "few key tiles")
    assert np.max(np.abs(lse - want_lse)) <= 1e-4
    ctx.close()


# Scores: products of bf16 are exact in fp32; the sums, the exponentials and the normalisers are fp32 (2^-24 relative each,
# arguments of the exponentials up to about 30 in base 2, i.e. 2^-19 of a weight): 1e-5 of the largest score covers both
# storage types.
SCORE_TOL = 1e-5

# (query heads, KV heads, head_dim, dtype, question tokens, chunk lengths): key blocks of a wave from 1 to 8 (16, 128, 129, 1024 keys) and
# the last block partial; chunks of more than one workgroup's keys (1025; 513 for fp32 at head_dim 128); one column, a
# whole and a partial step and tile of columns, more than one range of columns (2048)
SCORES = [(7, 1, 128, "bf16", 1, (16, 1, 0, 128)), (7, 1, 128, "bf16", 37, (129, 640, 513)), (28, 4, 128, "bf16", 16, (1024, 900)),
          (7, 1, 128, "bf16", 300, (70, 50)), (3, 1, 128, "bf16", 21, (1025, 300, 2100)), (4, 2, 64, "bf16", 33, (1024, 255, 17)),
          (4, 1, 64, "bf16", 16, (1500, 40)), (4, 4, 64, "f32", 32, (128, 127, 1024)), (5, 1, 64, "f32", 7, (1030, 3)),
          (8, 2, 128, "f32", 9, (512, 100)), (8, 2, 128, "f32", 5, (513, 64)), (8, 2, 128, "bf16", 65, (768, 1024, 33))]


@pytest.mark.parametrize("norm", [B.FR_NORM_PER_CHUNK, B.FR_NORM_GLOBAL])
@pytest.mark.parametrize("Hq,Hkv,d,dt,nq,lens", SCORES)
def test_scores(Hq, Hkv, d, dt, nq, lens, norm):
    shape = synth.LayerShape(n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, dtype=dt, rope_base=500000.0)
    w = synth.config_small_bf16(seed=Hq + nq, chunk_lens=lens, nq=nq, shape=shape)
    k_ctx = synth.round_to_storage(orc.rope_shift(w.k_cached, w.chunk_offsets, w.src_pos0, None, shape.rope_base), dt)
    want = orc.critical_scores(w.q_question, k_ctx, w.chunk_offsets, "global" if norm == B.FR_NORM_GLOBAL else "per_chunk")
    ctx = H.make_ctx(shape, w.L, w.n_chunks, w.nq)
    scores = torch.full((w.L_ctx,), -7.0, dtype=torch.float32, device="cuda")
    qi = torch.zeros(w.nq, dtype=torch.int32, device="cuda")
    ctx.fr_score_select(H.dev(w.q_question, dt), w.nq, H.dev(k_ctx, dt), w.chunk_offsets, 0, norm, scores, qi)
    torch.cuda.synchronize()
    assert H.max_rel_err(scores.cpu().numpy().astype(np.float64), want) <= SCORE_TOL
    # from a chunk store, the keys moved on the way.  The fp32 rotation may differ from the position shift's in its last bit,
    # and an element that lies between two bf16 numbers may then round the other way: 2^-8 of one element, which is
    # |q_e k_e| 2^-8 / sqrt(d) on a unit-scale logit, at most 5e-3 for elements of four standard deviations each.
    store = torch.cat([torch.zeros_like(H.dev(w.k_cached, dt))[:5], H.dev(w.k_cached, dt)])
    shifted = torch.zeros_like(H.dev(w.k_cached, dt))
    scores2, scores3 = torch.zeros_like(scores), torch.zeros_like(scores)
    ctx.fr_rope_shift(H.dev(w.k_cached, dt), shifted, w.chunk_offsets, w.src_pos0)
    ctx.fr_score_select(H.dev(w.q_question, dt), w.nq, shifted, w.chunk_offsets, 0, norm, scores2, qi)
    ctx.fr_score_select_shared(H.dev(w.q_question, dt), w.nq, store, len(store), w.chunk_offsets, w.chunk_offsets[:-1] + 5, w.src_pos0,
                               0, norm, scores3, qi)
    torch.cuda.synchronize()
    assert H.max_rel_err(scores3.cpu().numpy(), scores2.cpu().numpy()) <= 5e-3
    ctx.close()


# One to eight key blocks per wave (128 keys each; of which at 512 bytes a row one to four), the last one whole, of one key and with a rest; steps of 16 and
# 32 columns with and without a rest; columns of one token and of several in a copy.
@pytest.mark.parametrize("Hq,Hkv,d,dt,nq", [(8, 2, 128, "bf16", 25), (7, 1, 128, "bf16", 33), (1, 1, 128, "bf16", 70), (6, 2, 64, "bf16", 11), (4, 4, 64, "f32", 31), (6, 2, 128, "f32", 17)])
def test_scores_at_every_number_of_key_blocks(Hq, Hkv, d, dt, nq):
    test_scores(Hq, Hkv, d, dt, nq, (128, 129, 255, 257, 400, 512) + ((513, 640, 750, 769, 1000, 1024) if (d, dt) != (128, "f32") else ()), B.FR_NORM_PER_CHUNK)


def enough_for_four_waves(Hq, Hkv, nq, lens):
    """(chunk, KV head, 32 columns) in all: four per compute unit."""
    return len(lens) * Hkv * -(-nq * Hq // Hkv // 32) >= 4 * torch.cuda.get_device_properties(0).multi_processor_count


# Workgroups of four waves: chunks of one to eight blocks of 64 keys, from 1024 (chunk, KV head, 32 columns) on; one chunk of 513 keys: eight waves for all.
@pytest.mark.parametrize("longest", [512, 513])
@pytest.mark.parametrize("Hq,Hkv,d,dt,nq", [(32, 8, 128, "bf16", 121), (28, 4, 128, "bf16", 170), (16, 8, 64, "bf16", 241), (8, 8, 64, "f32", 500)])
def test_scores_of_chunks_for_four_waves(Hq, Hkv, d, dt, nq, longest):
    lens = (1, 64, 65, 130, 255, 300, 449, longest)
    assert enough_for_four_waves(Hq, Hkv, nq, lens)
    test_scores(Hq, Hkv, d, dt, nq, lens, B.FR_NORM_PER_CHUNK)


# The keys of a store are rotated to their prompt positions on the way into the registers, as the position shift does but for which product of a pair is rounded: 2^-24 of a
# rotated element.  In fp32 the scores are those of the shifted prompt within twice the tolerance of one side.  In bf16 an element in 2^15 or so is rounded to the other
# side, one of some 250 keys of 128 elements has one, which moves that key's own scores by what test_scores derives and all others by a fp32 sum's error.  Both layouts, workgroups of eight and of four waves, one to eight key blocks per wave, rows of the store in any order, distances of both signs.
@pytest.mark.parametrize("layout", [B.FR_ROPE_HALF, B.FR_ROPE_INTERLEAVED])
@pytest.mark.parametrize("Hq,Hkv,d,dt,nq", [(7, 1, 128, "bf16", 33), (6, 2, 64, "bf16", 11), (4, 4, 64, "f32", 31), (6, 2, 128, "f32", 17), (28, 4, 128, "bf16", 170),
                                            (16, 8, 64, "bf16", 300), (8, 8, 64, "f32", 600)])
def test_scores_of_a_store_are_those_of_the_shifted_prompt(Hq, Hkv, d, dt, nq, layout):
    lens = (1, 64, 130, 255, 300, 449, 512) if nq >= 170 else (128, 129, 400, 512) + ((640, 769, 1024) if (d, dt) != (128, "f32") else ())
    assert enough_for_four_waves(Hq, Hkv, nq, lens) == (nq >= 170)
    shape = synth.LayerShape(n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, dtype=dt, rope_base=10000.0)
    w = synth.config_small_bf16(seed=4, chunk_lens=lens, nq=nq, shape=shape)
    ctx = H.make_ctx(shape, w.L, w.n_chunks, w.nq, rope_layout=layout)
    offs = np.asarray(w.chunk_offsets)
    src_pos = np.asarray([(0, 3, 5000, 70000)[c % 4] for c in range(len(lens))], np.int32)
    row0, at = np.zeros(len(lens), np.int32), 5
    for c in reversed(range(len(lens))):   # the store holds them last chunk first, with gaps of 5 rows
        row0[c], at = at, at + lens[c] + 5
    store = np.zeros((at, Hkv, d), np.float32)
    for c in range(len(lens)):
        store[row0[c]:row0[c] + lens[c]] = w.k_cached[offs[c]:offs[c + 1]]
    q, prompt = H.dev(w.q_question, dt), H.dev(w.k_cached, dt)
    ctx.fr_rope_shift(prompt, prompt, w.chunk_offsets, src_pos)
    got = [torch.full((w.L_ctx,), -7.0, dtype=torch.float32, device="cuda") for _ in range(2)]
    qi = torch.zeros(w.nq, dtype=torch.int32, device="cuda")
    ctx.fr_score_select(q, w.nq, prompt, w.chunk_offsets, 0, B.FR_NORM_PER_CHUNK, got[0], qi)
    ctx.fr_score_select_shared(q, w.nq, H.dev(store, dt), at, w.chunk_offsets, row0, src_pos, 0, B.FR_NORM_PER_CHUNK, got[1], qi)
    torch.cuda.synchronize()
    off = torch.abs(got[1] - got[0]) / torch.max(torch.abs(got[0]))
    assert torch.max(off) <= (5e-3 if dt == "bf16" else 2 * SCORE_TOL)
    assert torch.sum(off > 2 * SCORE_TOL) <= Hkv * w.L_ctx / 250 + 3
    ctx.close()


@pytest.mark.parametrize("norm", [B.FR_NORM_PER_CHUNK, B.FR_NORM_GLOBAL])
def test_scores_of_more_columns_than_the_workspace_holds(norm):
    """A context of two million tokens holds the partial sums of 4096 query columns and the normalisers of 2048 at a time: 4400
    columns take two and three turns."""
    shape = synth.LayerShape(n_q_heads=16, n_kv_heads=4, head_dim=64, dtype="f32", rope_base=10000.0)
    w = synth.config_small_bf16(seed=2, chunk_lens=(500, 1030, 40), nq=1100, shape=shape)
    want = orc.critical_scores(w.q_question, w.k_cached, w.chunk_offsets, "global" if norm == B.FR_NORM_GLOBAL else "per_chunk")
    ctx = H.make_ctx(shape, 2 << 20, w.n_chunks, w.nq)
    scores = torch.full((w.L_ctx,), -7.0, dtype=torch.float32, device="cuda")
    qi = torch.zeros(w.nq, dtype=torch.int32, device="cuda")
    ctx.fr_score_select(H.dev(w.q_question, "f32"), w.nq, H.dev(w.k_cached, "f32"), w.chunk_offsets, 0, norm, scores, qi)
    torch.cuda.synchronize()
    assert H.max_rel_err(scores.cpu().numpy().astype(np.float64), want) <= SCORE_TOL
    ctx.close()


@pytest.mark.parametrize("shape", [synth.LLAMA3_8B_BF16, synth.TINY_F32, synth.LayerShape(28, 4, 128, "bf16", 1e6)])
def test_workspace_of_many_question_tokens(shape):
    """What the question tokens add to a context of 131072 tokens: one normaliser per (KV head, chunk or whole prompt, column),
    and the columns' partial sums and segments' normalisers of one turn, 64 MB each."""
    tokens, chunks, size = 131072, 16, []
    for max_q in (512, tokens):
        ctx = H.make_ctx(shape, tokens, chunks, max_q)
        size.append(ctx.workspace_bytes())
        ctx.close()
    assert size[1] - size[0] <= 4 * shape.n_kv_heads * (chunks + 1) * shape.group * (tokens - 512) + 2 * (64 << 20)


@pytest.mark.parametrize("norm", [B.FR_NORM_PER_CHUNK, B.FR_NORM_GLOBAL])
def test_scores_beyond_the_first_reference(norm):
    """Logits far above those of a chunk's first 16 keys: the column ranges that overflow are repeated with exact maxima."""
    shape = synth.LLAMA3_8B_BF16
    w = synth.config_small_bf16(seed=3, chunk_lens=(300, 150), nq=20, shape=shape)
    q, k = w.q_question.copy(), w.k_cached.copy()
    q[:, :, 0] = 60.0
    k[:, :, 0] = 0.0
    k[[100, 101, 170, 350], :, 0] = 45.0
    q, k = synth.round_to_storage(q, "bf16"), synth.round_to_storage(k, "bf16")
    want = orc.critical_scores(q, k, w.chunk_offsets, "global" if norm == B.FR_NORM_GLOBAL else "per_chunk")
    ctx = H.make_ctx(shape, w.L, w.n_chunks, w.nq)
    scores = torch.zeros(w.L_ctx, dtype=torch.float32, device="cuda")
    qi = torch.zeros(w.nq, dtype=torch.int32, device="cuda")
    ctx.fr_score_select(H.dev(q, "bf16"), w.nq, H.dev(k, "bf16"), w.chunk_offsets, 0, norm, scores, qi)
    torch.cuda.synchronize()
    # exponents of several hundred: 2^-24 of them is 2^-14 of a weight
    assert H.max_rel_err(scores.cpu().numpy().astype(np.float64), want) <= 2e-4
    ctx.close()


# fp32 products (fp32 storage; bf16 with more than 64 heads per KV head): sums of a few hundred fp32 terms, 1e-5 of the
# largest output as everywhere for fp32; prompts below and above the size whose position map fits LDS (8192), column tiles
# with rows of several and of less than one tile, fewer key blocks than waves, one block a wave, one wave with two, all with two, one with three.
@pytest.mark.parametrize("Hq,Hkv,d,dt,lens,nq,ratio", [(4, 4, 64, "f32", (5,), 3, 0.5), (4, 4, 64, "f32", (128, 77), 32, 0.15),
                                                       (6, 2, 64, "f32", (300, 0, 129), 17, 1.0), (5, 1, 128, "f32", (260, 40), 9, 0.2),
                                                       (2, 1, 64, "f32", (8100, 200), 21, 0.01), (80, 1, 64, "bf16", (90, 60), 5, 0.2),
                                                       (4, 4, 64, "f32", (120,), 8, 0.1), (4, 4, 64, "f32", (121,), 8, 0.1), (8, 2, 128, "f32", (121,), 8, 0.1),
                                                       (8, 2, 128, "f32", (248,), 8, 0.1), (8, 2, 128, "f32", (249,), 8, 0.1)])
def test_attention_with_fp32_products(Hq, Hkv, d, dt, lens, nq, ratio):
    shape = synth.LayerShape(n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, dtype=dt, rope_base=500000.0)
    w = synth.config_small_bf16(seed=Hq + nq, ratio=ratio, chunk_lens=lens, nq=nq, shape=shape)
    k_ctx, _, k, qi = staged(w)
    k_cache, v_cache = assembled_cache(w, k_ctx)
    ctx = H.make_ctx(w.shape, w.L, w.n_chunks, w.nq)
    tol = 1e-5 if dt == "f32" else OUT_TOL
    for with_new in (True, False):
        kc, vc = (k_cache, v_cache) if with_new else orc.kv_scatter(qi, w.k_full[qi], w.v_full[qi], k_cache, v_cache)
        got, lse = run_attention(ctx, w, qi, kc, vc, with_new=with_new)
        want, want_lse = orc.sparse_prefill_attn(w.q_full[qi], qi, k_cache, v_cache, w.k_full[qi], w.v_full[qi])
        assert H.max_rel_err(got, want) <= tol
        assert np.max(np.abs(lse - want_lse)) <= 1e-5
    ctx.close()


@pytest.mark.parametrize("Hq,Hkv,d", [(8, 2, 128), (4, 4, 128), (14, 2, 128), (4, 2, 64)])
def test_parts_of_short_prompts_keep_32_bits(Hq, Hkv, d):
    """A short prompt in one launch gives what whole tiled items give, and so do items cut into parts, over a store (several by the rule) and in two: their
    sums stay fp32.  fp32 sums of about 700 weights differ by 1e-6 of an element at most, which moves 2^-8 relative (one bf16 unit) in a share
    of about 1e-6 / 2^-8 < 1e-3 of the elements: sqrt(1e-3) 2^-8 = 1.2e-4 of the norm.  (Half-precision partial sums: 9e-4.)"""
    w = workload(Hq, Hkv, d, (130, 0, 333, 161), 77)
    k_ctx, _, k, qi = staged(w)
    k_cache, v_cache = assembled_cache(w, k_ctx)
    assert one_launch(w, qi)      # (AUTO)
    own = d == 128 and Hq // Hkv in (1, 4)
    outs = []
    for split in [B.FR_ATTN_SPLIT_OFF, B.FR_ATTN_SPLIT_AUTO, B.FR_ATTN_SPLIT_ON] + [STORE] * own:
        ctx = H.make_ctx(w.shape, w.L, w.n_chunks, w.nq)
        ctx.fr_set_option(B.FR_OPT_ATTN_SPLIT, B.FR_ATTN_SPLIT_AUTO if split == STORE else split)
        outs.append((run_attention_over_store if split == STORE else run_attention)(ctx, w, qi, k_cache, v_cache))
        ctx.close()
    for out, lse in outs[1:]:
        assert np.linalg.norm(out - outs[0][0]) <= 1.2e-4 * np.linalg.norm(outs[0][0])
        assert np.any(lse != outs[0][1])      # (sums in another order: not the whole items once more)


@pytest.mark.parametrize("d", [64, 128])
def test_fp32_sums_round_once_per_key_block(d):
    """Keys of zeros: every weight is 1 and the sums of the values, from [1, 2), show nothing but their own rounding.  The oracle's
    counterpart adds 16 keys at a time with one rounding, in eight chains (the waves; blocks dealt in turn), and the chains one after
    the other.  A matrix product onto the running sum rounds that several times a block: 2.4 times the error measured; with two
    roundings a block it would be the root of 2 in the chains, 1.25 in all, so 1.2."""
    L, R, rng = 8000, 16, np.random.default_rng(d)
    shape = synth.LayerShape(n_q_heads=4, n_kv_heads=4, head_dim=d, dtype="f32", rope_base=10000.0)
    v = (1.0 + rng.random((L, 4, d))).astype(np.float32)
    ctx = H.make_ctx(shape, L, 1, R)
    out = torch.zeros((R, 4, d), dtype=torch.float32, device="cuda")
    ctx.fr_sparse_prefill_attn(H.dev(rng.standard_normal((R, 4, d)).astype(np.float32), "f32"), torch.arange(L - R, L, dtype=torch.int32, device="cuda"), R,
                               torch.zeros((L, 4, d), device="cuda"), H.dev(v, "f32"), L, None, None, out)
    torch.cuda.synchronize()
    ctx.close()
    got = out.cpu().numpy().astype(np.float64)[-1]
    want = v.astype(np.float64).mean(axis=0)
    blocks = v.astype(np.float64).reshape(L // 16, 16, 4, d).sum(axis=1)
    total = np.zeros((4, d), dtype=np.float32)
    for wave in range(8):
        chain = np.zeros((4, d), dtype=np.float32)
        for b in blocks[wave::8]:
            chain = (chain + b).astype(np.float32)
        total = total + chain
    once = (total / np.float32(L)).astype(np.float64)
    assert np.linalg.norm(got - want) <= 1.2 * np.linalg.norm(once - want)


# (query heads, recomputed context rows, split): two parts are asked for; eight parts of the few items of a small call (over a store; over a cache of its own such
# a call runs in one launch); four parts (64 items of 32 rows)
@pytest.mark.parametrize("Hq,Hkv,rows,split,parts", [(Hq, 2, 30, B.FR_ATTN_SPLIT_ON, 2) for Hq in (2, 4, 8, 16)] +
                         [(8, 2, 30, B.FR_ATTN_SPLIT_AUTO, 8), (8, 2, 30, STORE, 8), (64, 8, 190, B.FR_ATTN_SPLIT_AUTO, 4), (64, 8, 190, STORE, 4)])
@pytest.mark.parametrize("key_tiles", [31, 32, 33])
@pytest.mark.parametrize("runaway", [False, True])
def test_parts_in_half_precision_and_in_32_bits(Hq, Hkv, rows, split, parts, key_tiles, runaway):
    """Up to four parts of a prompt of 32 key tiles and more hold their sums in half precision, all others in 32 bits.  Against
    whole items: sums of 2000 fp32 terms differ by 2^-24 sqrt(2000) = 2.7e-6 of an element, which turns the bf16 rounding of
    2.7e-6 / 2^-8 of them: 1e-4 of the norm.  Half precision: 2^-12 of a column's largest partial sum, about 3.5 times its
    norm's share, uniform, for two parts and more: 7e-4 to 1e-3, and the rounding of a fifth of the elements turned: 1.5e-3."""
    shape = synth.LayerShape(n_q_heads=Hq, n_kv_heads=Hkv, head_dim=128, dtype="bf16", rope_base=500000.0)
    L, nq = 64 * key_tiles - 5, 40
    w = synth.config_small_bf16(seed=Hq, chunk_lens=(L - nq,), nq=nq, shape=shape)
    qi = np.concatenate([np.sort(np.random.default_rng(1).choice(L - nq, size=rows, replace=False)), np.arange(L - nq, L)])
    k_cache, v_cache = assembled_cache(w, w.k_cached)
    if runaway:      # one key far above the first ones: the sums of the rows behind it overflow, and their items are done again
        w.q_full[:, :, 0] = 60.0
        k_cache[1200] = w.k_full[1200] = 0.0
        k_cache[1200, :, 0] = w.k_full[1200, :, 0] = 40.0
    assert one_launch(w, qi) == (Hkv == 2)      # (AUTO)
    outs = []
    for mode in (B.FR_ATTN_SPLIT_OFF, split):
        ctx = H.make_ctx(shape, L, 1, nq)
        ctx.fr_set_option(B.FR_OPT_ATTN_SPLIT, B.FR_ATTN_SPLIT_AUTO if mode == STORE else mode)
        outs.append((run_attention_over_store if mode == STORE else run_attention)(ctx, w, qi, k_cache, v_cache)[0])
        ctx.close()
    some = np.unique(np.concatenate([np.arange(0, len(qi), 7), [len(qi) - 1]]))
    want, _ = orc.sparse_prefill_attn(w.q_full[qi], qi, k_cache, v_cache, w.k_full[qi], w.v_full[qi], rows=some)
    H.assert_close(outs[1][some], want, "bf16", "attention")
    before = slice(0, np.searchsorted(qi, 1200) // (4 * 64 // shape.group) * (4 * 64 // shape.group)) if runaway else slice(None)
    off = np.linalg.norm((outs[1] - outs[0])[before]) / max(np.linalg.norm(outs[0][before]), 1e-30)
    if key_tiles < 32 or parts > 4:
        assert off <= 2e-4
    else:
        assert off <= 2.5e-3 and (runaway or off > 2e-4)


@pytest.mark.parametrize("rows,key_tiles,parts", [(768, 33, 2), (769, 33, 1), (1024, 64, 2), (1025, 64, 1), (1408, 257, 2), (1409, 257, 1)])
def test_where_items_stay_whole(rows, key_tiles, parts):
    """Row tiles of 32 rows and 8 KV heads.  64 log2(33 / 4) = 194.7: of 33 key tiles, 192 items are the last to be cut in two by
    themselves (half-precision sums: the bound above); one row more and every item is whole, bit for bit the result with the cutting off.
    64 key tiles: 256 items; 182 and more: 352, 11 / 8 of 256 compute units."""
    shape = synth.LayerShape(n_q_heads=64, n_kv_heads=8, head_dim=128, dtype="bf16", rope_base=500000.0)
    L, nq = 64 * key_tiles - 5, 40
    w = synth.config_small_bf16(seed=3, chunk_lens=(L - nq,), nq=nq, shape=shape)
    qi = np.concatenate([np.sort(np.random.default_rng(1).choice(L - nq, size=rows - nq, replace=False)), np.arange(L - nq, L)])
    k_cache, v_cache = assembled_cache(w, w.k_cached)
    assert not one_launch(w, qi)
    outs = []
    for mode in (B.FR_ATTN_SPLIT_OFF, B.FR_ATTN_SPLIT_AUTO):
        ctx = H.make_ctx(shape, L, 1, nq)
        ctx.fr_set_option(B.FR_OPT_ATTN_SPLIT, mode)
        outs.append(run_attention(ctx, w, qi, k_cache, v_cache)[0])
        ctx.close()
    off = np.linalg.norm(outs[1] - outs[0]) / np.linalg.norm(outs[0])
    assert off == 0.0 if parts == 1 else 2e-4 < off <= 2.5e-3


@pytest.mark.parametrize("in_bin", [1, 2, 255, 256, 257, 300])
@pytest.mark.parametrize("n", [900, 8193, 32768])
def test_select_rank_inside_a_histogram_bin(n, in_bin):
    """The k-th largest score lies in a bin of `in_bin` keys, around the number that is ranked directly: every rank in it,
    with distinct keys and with ties."""
    ctx = H.make_ctx(synth.TINY_F32, 70000, 4, 16)
    rng = np.random.default_rng(n + in_bin)
    top = n // 10
    for ties in (1, 3):
        s = np.empty(n, dtype=np.float32)
        s[:top] = 64.0 + rng.random(top)                                       # larger than all of the bin
        s[top:top + in_bin] = 8.0 + (np.arange(in_bin) // ties) * 2.0 ** -20    # one unit in the last place apart: one bin
        s[top + in_bin:] = 1.0 + rng.random(n - top - in_bin)
        s = s[rng.permutation(n)]
        dev = torch.from_numpy(s).cuda()
        for k in sorted({top, top + 1, top + 2, top + in_bin // 2 + 1, top + in_bin, min(n - 1, top + in_bin + 1)}):
            out = torch.full((k + 1,), -7, dtype=torch.int32, device="cuda")
            ctx.fr_select_topk(dev, n, k, 1, out)
            torch.cuda.synchronize()
            assert np.array_equal(out.cpu().numpy(), orc.select_q_index(s, k, 1)), (ties, k)
    ctx.close()


def ranked(s, k, nq):
    """The selection's own order, NaN included: scores by their bits, larger first, then lower index (orc.select_q_index where all are numbers and zeros have one sign)."""
    u = s.view(np.uint32)
    key = np.where(u >> 31, ~u, u | np.uint32(1 << 31)).astype(np.int64)
    return np.concatenate([np.sort(np.lexsort((np.arange(len(s)), -key))[:k]), len(s) + np.arange(nq)])


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 63, 64, 65, 80, 127, 128, 129, 191, 192, 193, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025, 2047, 2048, 2049])
def test_select_in_one_wave(n):
    """Small numbers of scores: up to 128 counted, a wave for each 64, from there on by the workgroup's histogram (one wave selects behind sums of up to 512 scores only:
    test_selection_beside_the_sums).  Distinct scores, ties, one value, extremes of every bit, infinities, NaN of both signs; no score at all where none is taken; fewer and
    more question tokens than the scores' waves hold."""
    ctx = H.make_ctx(synth.TINY_F32, 4096, 4, 600)
    rng = np.random.default_rng(n)
    inputs = {"distinct": rng.permutation(n).astype(np.float32) - n / 3, "ties": rng.integers(0, 5, size=n).astype(np.float32),
              "constant": np.full(n, -2.5, dtype=np.float32), "extremes": rng.standard_normal(n).astype(np.float32)}
    inputs["extremes"][rng.integers(0, n, size=4)] = [3.0e38, -3.0e38, np.inf, -np.inf]
    inputs["runs"] = np.repeat(rng.permutation(n // 30 + 1), 30)[:n].astype(np.float32)      # ties in a wave and across two
    inputs["not numbers"] = inputs["extremes"].copy()
    inputs["not numbers"].view(np.uint32)[rng.integers(0, n, size=n // 8 + 2)] = rng.choice(np.array([0x7FC00000, 0xFFC00000, 0xFFFFFFFF, 0x7F800001], dtype=np.uint32), size=n // 8 + 2)
    for name, s in inputs.items():
        dev = torch.from_numpy(s).cuda()
        for k in sorted({0, 1, n // 7, n // 3, n // 2, n - 1, n}):
            for nq in (3, 600) if k == n // 3 else (3,):
                out = torch.full((k + nq + 1,), -7, dtype=torch.int32, device="cuda")
                ctx.fr_select_topk(dev if k else None, n, k, nq, out)
                torch.cuda.synchronize()
                got = out.cpu().numpy()
                assert got[-1] == -7 and np.array_equal(got[:-1], ranked(s, k, nq)), (name, k, nq)
                assert name == "not numbers" or np.array_equal(got[:-1], orc.select_q_index(s, k, nq)), (name, k, nq)
    ctx.close()
