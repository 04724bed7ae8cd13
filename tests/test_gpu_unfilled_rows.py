"""Attention must not depend on values that no row sees: stale cache rows of listed positions, rows behind the last listed
one (a cache with room to spare, rows that the write-back has not reached yet), and for a row whatever lies behind its own
position.  All of them hold NaN or infinity here, which a weight of zero does not take away: `pytest -m gpu`."""
import numpy as np
import pytest
import torch

from oracle import fusionrag_oracle as orc
from paper_2601_12904_amd import binding as B
from paper_2601_12904_amd import synth
from tests import harness as H
from tests.test_gpu_parity import assembled_cache, staged

pytestmark = pytest.mark.gpu

SPARE = 75   # cache rows behind the prompt: more than a 64-key tile


def case(Hq, Hkv, d, dt, lens, nq, ratio):
    shape = synth.LayerShape(n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, dtype=dt, rope_base=500000.0)
    w = synth.config_small_bf16(seed=Hq + nq, ratio=ratio, chunk_lens=lens, nq=nq, shape=shape)
    k_ctx, _, _, qi = staged(w)
    k_cache, v_cache = assembled_cache(w, k_ctx)
    ctx = H.make_ctx(shape, w.L + SPARE, w.n_chunks, w.nq)
    return w, qi, k_cache, v_cache, ctx


def with_spare_rows(x, listed=()):
    """The cache with SPARE rows more; those and the `listed` ones hold NaN."""
    x = np.concatenate([x, np.full((SPARE,) + x.shape[1:], np.nan)]).astype(np.float32)
    x[np.asarray(listed, dtype=np.int64)] = np.nan
    return x


def attend(ctx, w, qi, q, k_cache, v_cache, k_new=None, v_new=None, writeback=False):
    dt = w.shape.dtype
    out = torch.zeros((len(qi), w.shape.n_q_heads, w.shape.head_dim), dtype=H.TORCH_DTYPE[dt], device="cuda")
    lse = torch.zeros((len(qi), w.shape.n_q_heads), dtype=torch.float32, device="cuda")
    kc, vc = H.dev(k_cache, dt), H.dev(v_cache, dt)
    new = (None, None) if k_new is None else (H.dev(k_new, dt), H.dev(v_new, dt))
    call = ctx.fr_sparse_prefill_attn_writeback if writeback else ctx.fr_sparse_prefill_attn
    call(H.dev(q, dt), torch.from_numpy(qi.astype(np.int32)).cuda(), len(qi), kc, vc, len(k_cache), *new, out, lse)
    torch.cuda.synchronize()
    return H.host(out), lse.cpu().numpy(), H.host(kc), H.host(vc)


# fp32 products: prompts below and above the size whose position map fits LDS, column tiles of 16 and of 4 rows and less,
# head_dim 64 and 128, bf16 with more than 64 heads per KV head
FP32_PRODUCTS = [(4, 4, 64, "f32", (128, 77), 32, 0.15), (4, 1, 64, "f32", (130, 60), 9, 0.15), (5, 1, 128, "f32", (260, 40), 9, 0.2),
                 (2, 2, 64, "f32", (8100, 200), 21, 0.01), (80, 1, 64, "bf16", (90, 60), 5, 0.2)]
# the tiled kernels: group sizes with and without an instance of their own, head_dim 64; items whole, in parts, and against the
# largest logit throughout
TILED = [(Hq, Hkv, d, "bf16", (130, 0, 333, 61), 37, 0.2) for Hq, Hkv, d in ((4, 4, 128), (4, 2, 128), (8, 2, 128), (16, 2, 128), (7, 1, 128), (14, 2, 64))]
WHOLE, PARTS, RUNNING = (B.FR_OPT_ATTN_SPLIT, B.FR_ATTN_SPLIT_OFF), (B.FR_OPT_ATTN_SPLIT, B.FR_ATTN_SPLIT_ON), (B.FR_OPT_ATTN_SOFTMAX, B.FR_ATTN_SOFTMAX_RUNNING_MAX)
CASES = [(c, WHOLE) for c in FP32_PRODUCTS] + [(c, option) for c in TILED for option in (WHOLE, PARTS, RUNNING)]


@pytest.mark.parametrize("with_new", [True, False])
@pytest.mark.parametrize("case_args,option", CASES)
def test_rows_that_hold_nothing(case_args, option, with_new):
    """Also with the question rows left out of the index: its last row then ends in the middle of a key block."""
    w, qi_all, k_cache, v_cache, ctx = case(*case_args)
    ctx.fr_set_option(*option)
    dt = w.shape.dtype
    for qi in (qi_all, qi_all[:-w.nq]):
        k_new, v_new = w.k_full[qi], w.v_full[qi]
        want, want_lse = orc.sparse_prefill_attn(w.q_full[qi], qi, k_cache, v_cache, k_new, v_new)
        k_eff, v_eff = orc.kv_scatter(qi, k_new, v_new, k_cache, v_cache)
        behind = np.arange(qi[-1] + 1, w.L)      # nothing is known about them
        if with_new:
            kc, vc = (with_spare_rows(x, np.concatenate([qi, behind])) for x in (k_cache, v_cache))
            got, lse, _, _ = attend(ctx, w, qi, w.q_full[qi], kc, vc, k_new, v_new)
        else:
            kc, vc = (with_spare_rows(x, behind) for x in (k_eff, v_eff))
            got, lse, _, _ = attend(ctx, w, qi, w.q_full[qi], kc, vc)
        H.assert_close(got, want, dt, "attention")
        assert np.max(np.abs(lse - want_lse)) <= (1e-5 if dt == "f32" else 1e-4)
        if with_new:
            got, _, kw, vw = attend(ctx, w, qi, w.q_full[qi], kc, vc, k_new, v_new, writeback=True)
            H.assert_close(got, want, dt, "attention with write-back")
            kc[qi], vc[qi] = k_new, v_new
            assert np.array_equal(kw, kc, equal_nan=True) and np.array_equal(vw, vc, equal_nan=True)
    ctx.close()


# few rows of a long prompt: the 64 / G rows of a wave lie a dozen key tiles apart, as do the value and the rows in front of it
SPARSE = [(Hq, Hkv, 128, "bf16", (700, 611, 800), 20, 0.03) for Hq, Hkv in ((2, 2), (4, 2), (8, 2), (16, 2), (7, 1))]


@pytest.mark.parametrize("case_args,option", CASES + [(c, option) for c in SPARSE for option in (WHOLE, PARTS, RUNNING)])
def test_values_that_are_not_finite_reach_later_rows_only(case_args, option):
    """A fresh value row with a NaN and an infinity, and a cached one that no listed row has replaced: rows in front of them
    are as without them, rows behind them have the NaN and the infinity in those elements and are otherwise as without them."""
    w, qi, k_cache, v_cache, ctx = case(*case_args)
    ctx.fr_set_option(*option)
    dt = w.shape.dtype
    k_new, v_new = w.k_full[qi], w.v_full[qi].copy()
    at = len(qi) // 2                                               # a row in the middle of the index
    cached = [j for j in range(int(qi[at]) + 1, int(qi[-1])) if j not in set(qi.tolist())][:1]   # and a stale position behind it
    elements = [(0, 3, np.nan), (0, 5, np.inf), (w.shape.n_kv_heads - 1, w.shape.head_dim - 1, -np.inf)]
    vc, vn = v_cache.copy(), v_new.copy()
    for g, e, bad in elements:
        v_new[:, g, e] = v_cache[:, g, e] = 0.25                    # (elements of their own: any finite values)
        vn[:, g, e] = vc[:, g, e] = 0.25
        vn[at, g, e] = bad
        vc[cached, g, (e + 8) % w.shape.head_dim] = bad
        v_cache[cached, g, (e + 8) % w.shape.head_dim] = 0.25
    want, _ = orc.sparse_prefill_attn(w.q_full[qi], qi, k_cache, v_cache, k_new, v_new)
    got, _, _, _ = attend(ctx, w, qi, w.q_full[qi], k_cache, vc, k_new, vn)
    G = w.shape.group
    for g, e, bad in elements:
        heads = slice(g * G, (g + 1) * G)
        for first, el in ((at, e), *((int(np.searchsorted(qi, j)), (e + 8) % w.shape.head_dim) for j in cached)):
            assert np.all(np.isfinite(got[:first, heads, el])) and not np.any(np.isfinite(got[first:, heads, el]))
            got[first:, heads, el] = want[first:, heads, el]
    H.assert_close(got, want, dt, "attention")
    ctx.close()
