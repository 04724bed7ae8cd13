"""Attention of short bf16 prompts in one launch, at the edges of its key blocks, column tiles and dispatch rule, against the
oracle and against the tiled kernels (FR_ATTN_SPLIT_OFF asks for those): `pytest -m gpu`."""
import numpy as np
import pytest
import torch

from oracle import fusionrag_oracle as orc
from paper_2601_12904_amd import binding as B
from paper_2601_12904_amd import synth
from tests import harness as H
from tests import test_gpu_unfilled_rows as unfilled

pytestmark = pytest.mark.gpu

# Output elements are rounded to bf16 once (half a unit: 2^-8 of the tensor's largest value at most).  Weights of shapes with an instance
# of their own are rounded to bf16 too: 2^-9 of each weight, as often up as down, at most 2^-8 of the largest value with signs against us.
TOL = {True: 2.0 ** -8 + 2.0 ** -14, False: 2.0 ** -7 + 2.0 ** -14}


def inputs(Hq, Hkv, d, L, R, seed, at_end=False):
    rng = np.random.default_rng(seed)
    qi = np.arange(L - R, L) if at_end else np.sort(np.concatenate([rng.choice(L - 1, R - 1, replace=False), [L - 1]]))
    bf = lambda *s, scale=1.0: synth.round_to_storage((rng.standard_normal(s) * scale).astype(np.float32), "bf16")  # noqa: E731
    return (qi, bf(R, Hq, d, scale=d ** 0.5), *(bf(L, Hkv, d, scale=d ** -0.5) for _ in range(2)), *(bf(R, Hkv, d, scale=d ** -0.5) for _ in range(2)))


def attend(Hq, Hkv, d, qi, q, kc, vc, kn, vn, split, writeback=False):
    L, R = len(kc), len(qi)
    c = B.Context(Hq, Hkv, d, B.FR_BF16, 500000.0, max_tokens=L, max_chunks=1, max_question_tokens=1)
    c.fr_set_option(B.FR_OPT_ATTN_SPLIT, split)
    out = torch.zeros((R, Hq, d), dtype=torch.bfloat16, device="cuda")
    lse = torch.zeros((R, Hq), dtype=torch.float32, device="cuda")
    k, v = H.dev(kc, "bf16"), H.dev(vc, "bf16")
    call = c.fr_sparse_prefill_attn_writeback if writeback else c.fr_sparse_prefill_attn
    call(H.dev(q, "bf16"), torch.from_numpy(qi.astype(np.int32)).cuda(), R, k, v, L, *(None if x is None else H.dev(x, "bf16") for x in (kn, vn)), out, lse)
    torch.cuda.synchronize()
    c.close()
    return H.host(out), lse.cpu().numpy(), H.host(k), H.host(v)


# (query heads, KV heads, head_dim): 32-column tiles of 32, 8, 4, 4 4/7 and half a row; head_dim 64; one KV head and a number that is no power of two
SHAPES = [(1, 1, 128), (12, 3, 128), (16, 2, 128), (7, 1, 128), (64, 1, 128), (3, 3, 64), (14, 2, 64)]
# positions: one, the last of a key block, one behind, one behind a round of eight blocks; rows: one, tiles with and without a rest
SIZES = [(1, 1), (31, 5), (32, 32), (33, 8), (64, 9), (257, 40), (530, 100)]


@pytest.mark.parametrize("L,R", SIZES)
@pytest.mark.parametrize("Hq,Hkv,d", SHAPES)
def test_against_the_oracle(Hq, Hkv, d, L, R):
    assert H.in_one_launch(Hq, Hkv, d, R, L)
    qi, q, kc, vc, kn, vn = inputs(Hq, Hkv, d, L, R, seed=L + Hq)
    want, want_lse = orc.sparse_prefill_attn(q, qi, kc, vc, kn, vn)
    k_eff, v_eff = orc.kv_scatter(qi, kn, vn, kc, vc)
    tol = TOL[d == 64 or Hq // Hkv not in (1, 2, 4, 8)]
    for new, kv, writeback in (((kn, vn), (kc, vc), False), ((kn, vn), (kc, vc), True), ((None, None), (k_eff, v_eff), False)):
        got, lse, k, v = attend(Hq, Hkv, d, qi, q, *kv, *new, B.FR_ATTN_SPLIT_AUTO, writeback)
        assert H.max_rel_err(got, want) <= tol
        assert np.max(np.abs(lse - want_lse)) <= 1e-4
        assert np.array_equal(k, k_eff if writeback else kv[0]) and np.array_equal(v, v_eff if writeback else kv[1])


# Either side of the rule's lines for 256 compute units: 32-column tiles (R x 32 heads / 32, R x 16 heads / 32 at head_dim 64, R x 7 / 32 for each of 4 KV heads) and
# positions; and of the line between 16 and 32 columns per workgroup.
@pytest.mark.parametrize("at_end", [False, True])
@pytest.mark.parametrize("Hq,Hkv,d,L,R,one", [(32, 8, 128, 700, 128, True), (32, 8, 128, 700, 129, True), (32, 8, 128, 1024, 512, True), (32, 8, 128, 1024, 513, False),
                                              (32, 8, 128, 1025, 384, True), (32, 8, 128, 1025, 385, False), (32, 8, 128, 1792, 384, True), (32, 8, 128, 1792, 385, False),
                                              (32, 8, 128, 1793, 256, True), (32, 8, 128, 1793, 257, False), (28, 4, 128, 6144, 288, True), (28, 4, 128, 6144, 293, False),
                                              (32, 8, 128, 6144, 20, True), (32, 8, 128, 6145, 20, False), (16, 8, 64, 4096, 768, True), (16, 8, 64, 4096, 769, False),
                                              (16, 8, 64, 4097, 512, True), (16, 8, 64, 4097, 513, False)])
def test_both_sides_of_the_rule(Hq, Hkv, d, L, R, one, at_end):
    assert H.in_one_launch(Hq, Hkv, d, R, L) == one
    args = inputs(Hq, Hkv, d, L, R, seed=L + R, at_end=at_end)
    got, lse, _, _ = attend(Hq, Hkv, d, *args, B.FR_ATTN_SPLIT_AUTO)
    tiled, tiled_lse, _, _ = attend(Hq, Hkv, d, *args, B.FR_ATTN_SPLIT_OFF)
    assert H.max_rel_err(got, tiled) <= 2 * TOL[d == 64 or Hq // Hkv == 7]      # both are off float64
    assert np.max(np.abs(lse - tiled_lse)) <= 2e-4


AUTO = (B.FR_OPT_ATTN_SPLIT, B.FR_ATTN_SPLIT_AUTO)


@pytest.mark.parametrize("with_new", [True, False])
@pytest.mark.parametrize("case_args", unfilled.TILED)
def test_rows_that_hold_nothing(case_args, with_new):
    unfilled.test_rows_that_hold_nothing(case_args, AUTO, with_new)


@pytest.mark.parametrize("case_args", unfilled.TILED + unfilled.SPARSE)
def test_values_that_are_not_finite_reach_later_rows_only(case_args):
    unfilled.test_values_that_are_not_finite_reach_later_rows_only(case_args, AUTO)


@pytest.mark.parametrize("rise", [16.0, 320.0])
@pytest.mark.parametrize("Hq,Hkv,d", [(8, 2, 128), (7, 1, 128), (4, 2, 64)])
def test_rising_references(Hq, Hkv, d, rise):
    """Logits that rise along the prompt.  A reference goes up where a lane's eight weights of a block, against the columns' maximum over keys 0..31 or what they have been
    raised to, sum to more than 2^10: with a rise of 320 every block of every wave does that for all of its columns (its largest logit is more than 2^11 above that
    of any block in front), with 16, 2^20 to 2^28 over the prompt, only some of the later ones do."""
    L = 600
    qi, q, kc, vc, kn, vn = inputs(Hq, Hkv, d, L, 90, seed=5)
    assert H.in_one_launch(Hq, Hkv, d, len(qi), L)
    ramp = np.linspace(0.0, rise, L, dtype=np.float32)
    q[:, :, 0], kc[:, :, 0], kn[:, :, 0] = 10.0, ramp[:, None], ramp[qi][:, None]
    q, kc, kn = (synth.round_to_storage(x, "bf16") for x in (q, kc, kn))
    if rise == 320.0:
        k_eff, _ = orc.kv_scatter(qi, kn, vn, kc, vc)
        s = np.einsum("rgqd,jgd->rgqj", q.reshape(len(qi), Hkv, Hq // Hkv, d), k_eff) / np.sqrt(d) * np.log2(np.e)
        blocks = s[..., :L // 32 * 32].reshape(*s.shape[:3], -1, 32).max(axis=-1)
        assert np.min(np.diff(blocks)) > 11
    got, lse, _, _ = attend(Hq, Hkv, d, qi, q, kc, vc, kn, vn, B.FR_ATTN_SPLIT_AUTO)
    want, want_lse = orc.sparse_prefill_attn(q, qi, kc, vc, kn, vn)
    # a logit of up to 577 in base 2 is rounded to 2^-24 of that, 3.4e-5, and its weight is off by as much; the sum's logarithm by three of them
    assert H.max_rel_err(got, want) <= TOL[d == 64 or Hq // Hkv == 7] + 2.0 ** -14
    assert np.max(np.abs(lse - want_lse)) <= (1e-4 if rise == 16.0 else 2e-4)


# Sums and selection in one launch: up to 1024 tokens and 64 partial sums (KV heads x column ranges); quads of tokens with a rest, fewer than four tokens
@pytest.mark.parametrize("Hq,Hkv,d,dt,nq", [(4, 4, 64, "f32", 9), (32, 8, 128, "bf16", 40), (64, 32, 128, "bf16", 70)])
@pytest.mark.parametrize("L", [1, 2, 3, 4, 5, 63, 511, 512, 513, 1021, 1024, 1025])
def test_selection_beside_the_sums(Hq, Hkv, d, dt, nq, L):
    shape = synth.LayerShape(n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, dtype=dt, rope_base=10000.0)
    w = synth.config_small_bf16(seed=L, chunk_lens=tuple(len(x) for x in np.array_split(np.arange(L), min(4, L))), nq=nq, shape=shape)
    k = synth.round_to_storage(w.k_cached, dt)
    if L % 2 == 0:
        k[L // 2:] = k[:L // 2]     # equal scores in pairs of chunks
    want = orc.critical_scores(w.q_question, k, w.chunk_offsets)
    ctx = H.make_ctx(shape, w.L, w.n_chunks, nq)
    q, kd = H.dev(w.q_question, dt), H.dev(k, dt)
    for take in {0, 1, (L + 6) // 7, L - 1, L}:
        scores = torch.full((L,), -7.0, dtype=torch.float32, device="cuda")
        qi, again = (torch.full((take + nq,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
        ctx.fr_score_select(q, nq, kd, w.chunk_offsets, take, B.FR_NORM_PER_CHUNK, scores, qi)
        ctx.fr_select_topk(scores, L, take, nq, again)
        torch.cuda.synchronize()
        assert H.max_rel_err(scores.cpu().numpy().astype(np.float64), want) <= 1e-4
        assert np.array_equal(qi.cpu().numpy(), again.cpu().numpy())
        ctx.fr_score_select(q, nq, kd, w.chunk_offsets, take, B.FR_NORM_PER_CHUNK, None, again)
        assert np.array_equal(qi.cpu().numpy(), again.cpu().numpy())
    ctx.close()


# Scores of few values: keys of zeros (every score of chunks of equal length the same, the selection's first bit is none) and two or seven different keys in turn; chunks
# of garbage (NaN: all scores of the chunk).  Up to 512 tokens one wave selects by ballots, up to 1024 the workgroup by a histogram; fr_select_topk the workgroup.
@pytest.mark.parametrize("kind", ["one", "two", "seven", "garbage"])
@pytest.mark.parametrize("L", [64, 65, 300, 511, 512, 513, 700, 1021, 1024])
def test_tied_scores_beside_the_sums(L, kind):
    Hq, Hkv, d, nq, chunks = 8, 2, 128, 9, 4
    shape = synth.LayerShape(n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, dtype="bf16", rope_base=10000.0)
    rng = np.random.default_rng(L)
    bf = lambda *s: synth.round_to_storage(rng.standard_normal(s).astype(np.float32), "bf16")  # noqa: E731
    some = bf({"one": 1, "two": 2, "seven": 7, "garbage": 7}[kind], Hkv, d) * (0.0 if kind == "one" else 1.0)
    k = some[rng.integers(0, len(some), size=L)]
    cut = np.array([len(x) for x in np.array_split(np.arange(L), chunks)])
    offs = np.concatenate([[0], np.cumsum(cut)]).astype(np.int32)
    if kind == "garbage":
        k[int(offs[1]) + 3, 1, 5], k[int(offs[3]) + 1, 0, 0] = np.nan, np.inf
    ctx = H.make_ctx(shape, L + nq, chunks, nq)
    q, kd = H.dev(bf(nq, Hq, d), "bf16"), H.dev(k, "bf16")
    scores = torch.full((L,), -7.0, dtype=torch.float32, device="cuda")
    for take in sorted({1, 2, L // 7, L // 2, L - 1, L}):
        got, again = (torch.full((take + nq,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
        ctx.fr_score_select(q, nq, kd, offs, take, B.FR_NORM_PER_CHUNK, scores, got)
        ctx.fr_select_topk(scores, L, take, nq, again)
        torch.cuda.synchronize()
        s = scores.cpu().numpy()
        if kind == "garbage":
            assert np.isnan(s).sum() == cut[1] + cut[3]
            assert torch.equal(got, again)
        else:
            assert len(np.unique(s)) <= chunks * len(some)            # (every chunk has a normaliser of its own)
            assert np.array_equal(got.cpu().numpy(), orc.select_q_index(s, take, nq))
    ctx.close()
