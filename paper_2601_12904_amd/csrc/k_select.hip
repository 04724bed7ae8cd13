// Selection half of Query-Guided Selection: argTopk of the critical scores (Table 1, Sec. 3.2)
// and the Q index of Sec. 4.3 (ascending critical tokens, then the question tokens).
//
// Integer work only.  Scores are mapped to order-preserving 32-bit keys; a most-significant-digit
// radix select (digits of 12 bits, LDS histogram) finds the key of the k-th largest score: passes go on until the bin that
// holds it has at most CANDIDATES keys (after the first one as a rule), whose ranks are then counted directly; an
// ordered compaction then emits, in index order, every token above that key plus the first
// (lowest-index) tokens equal to it that are still needed.  The result is unique, so it does not
// depend on scheduling.  One workgroup: the 64 KB of scores of a 17k-token prompt fit its registers, and the
// whole selection is latency- rather than bandwidth-sized (longer score vectors: k_select_large.hip).  Scores of one prompt are clustered (their sign and
// most exponent bits agree), which would pile a plain histogram onto one or two bins; the digits are therefore
// taken from key - min(key), starting at the highest bit in which the largest and the smallest key differ.  Even so most scores lie near the smallest
// one: with 256 bins the adds of a wave queued up behind one LDS word, and every pass costs its barriers and scans (four
// passes of 8 bits 9.6 / 19.5 / 33.0 us at 880 / 16384 / 32768 scores of a prompt, one of 12 bits 8.1 / 14.7 / 25.2, and with what stands at select_in_workgroup 4.7 / 9.7 / 18.0).
#include "fr_internal.hpp"

#include <algorithm>

namespace fr {

__device__ __forceinline__ uint32_t score_key(float f) {
    const uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);  // larger score <=> larger key
}

constexpr int SEL_THREADS = 1024;

constexpr int BINS = 4 * SEL_THREADS;   // one 16-byte vector of bins per thread
constexpr int DIGIT = 12;
constexpr uint32_t CANDIDATES = 256;
static_assert(BINS == 1 << DIGIT, "digit");

template <int CTRL>
__device__ __forceinline__ uint32_t moved(uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true); }

// Over four (quad) and sixteen (row) neighbouring lanes, in every one of them.
template <typename F>
__device__ __forceinline__ uint32_t over_quad(uint32_t v, F f) {
    v = f(v, moved<0xB1>(v));        // quad_perm [1,0,3,2]
    return f(v, moved<0x4E>(v));     // quad_perm [2,3,0,1]
}
template <typename F>
__device__ __forceinline__ uint32_t over_row(uint32_t v, F f) {
    v = over_quad(v, f);
    v = f(v, moved<0x141>(v));       // row_half_mirror: the other quad of eight
    return f(v, moved<0x140>(v));    // row_mirror: the other eight
}
__device__ __forceinline__ uint32_t add(uint32_t a, uint32_t b) { return a + b; }
__device__ __forceinline__ uint32_t lower(uint32_t a, uint32_t b) { return min(a, b); }
__device__ __forceinline__ uint32_t higher(uint32_t a, uint32_t b) { return max(a, b); }

// Among the candidates of this pass (keys that share the digits fixed so far), the digit of the k-th largest
// key is the largest d whose suffix count S[d] = sum_{b >= d} hist[b] still reaches `remaining`.  Four bins
// per thread: suffix sums by lane moves, then the single thread that holds the matching bin publishes it.
// `remaining` is read before the first barrier: between the two barriers the matching thread overwrites it, and the
// waves do not run in lockstep, so a read behind the first barrier could see the reduced value and let a
// second bin match.  (The caller's barrier after the histogram orders this read behind the previous pass's write.)
__device__ __forceinline__ void pick_digit(const uint32_t* hist, uint32_t* wave_tot, uint32_t* s_prefix,
                                           uint32_t* s_remaining, uint32_t* s_count, int shift) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t remaining = *s_remaining;
    const uint4 own = reinterpret_cast<const uint4*>(hist)[tid];
    uint32_t suf = own.x + own.y + own.z + own.w;
    const uint32_t mine = suf;
    suf += moved<0x101>(suf);   // row_shl: the lanes above in the row, zero behind its end
    suf += moved<0x102>(suf);
    suf += moved<0x104>(suf);
    suf += moved<0x108>(suf);
    const uint32_t row1 = __builtin_amdgcn_readlane(suf, 16), row2 = __builtin_amdgcn_readlane(suf, 32), row3 = __builtin_amdgcn_readlane(suf, 48);
    suf += (lane < 16 ? row1 : 0u) + (lane < 32 ? row2 : 0u) + (lane < 48 ? row3 : 0u);
    if (lane == 0) wave_tot[wave] = suf;   // total of the wave's 256 bins
    __syncthreads();
    const int w2 = lane & (SEL_THREADS / 64 - 1);
    suf += over_row(w2 > wave ? wave_tot[w2] : 0u, add);
    uint32_t above = suf - mine;           // candidates with a larger digit than any of this thread's
    if (suf >= remaining && above < remaining) {
        const uint32_t bins[4] = {own.x, own.y, own.z, own.w};
        int d = 3;
        while (d > 0 && above + bins[d] < remaining) above += bins[d--];
        *s_remaining = remaining - above;  // still to take among keys with this digit
        *s_count = bins[d];
        *s_prefix |= (uint32_t)(4 * tid + d) << shift;
    }
    __syncthreads();
}

__device__ __forceinline__ uint32_t lanes_below(uint64_t ballot) {   // set bits of lanes lower than this one
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(ballot >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)ballot, 0u));
}

// Wave w owns the contiguous index range [w * 64 * PER, (w + 1) * 64 * PER); its i-th load covers the 256
// consecutive tokens base + 256 i + 4 lane .. + 3, so (i, lane, e) order is index order (one CU's loads of 4 bytes a lane come at a quarter of the rate).  A
// lane whose four tokens pass the end loads the last four, of which those before its own are another lane's.
// Every thread keeps its PER keys in registers (1 <= n <= SEL_THREADS * PER, k >= 1; all threads of the workgroup).
// Against loads of one score, reductions and scans by LDS permutes and the waves' totals read one after the other: 16384 scores 13.0 -> 9.7 us, 32768 23.5 -> 18.0, 4000 8.7 -> 5.0.
// (A launch of one wave, as select_in_wave below, 4.6 to 10 us at 128 to 1024 scores, 15 with ties; this one 4.5.)
template <int PER>
__device__ __forceinline__ void select_in_workgroup(const float* scores, int n, int64_t k, int32_t* __restrict__ out) {
    constexpr int WAVES = SEL_THREADS / 64;
    __shared__ __attribute__((aligned(16))) uint32_t hist[BINS];
    __shared__ uint32_t wave_a[WAVES], wave_b[WAVES];
    __shared__ uint32_t wave_tot[WAVES];
    __shared__ __attribute__((aligned(16))) uint32_t candidates[CANDIDATES];
    __shared__ uint32_t s_prefix, s_remaining, s_count, s_listed;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

    constexpr int QUADS = PER / 4;
    const int last = n - 4;
    auto quad = [&](int i) { return wave * 64 * PER + 256 * i + 4 * lane; };
    auto own = [&](int i) { return (i & 3) >= quad(i >> 2) - last; };   // key i: token min(quad(i / 4), last) + i % 4
    uint32_t keys[PER];
    {
        // branch-free: every load is issued before the first one is waited for
        typedef __attribute__((ext_vector_type(4), aligned(4))) float f32x4_any;
        f32x4_any raw[QUADS];
        if (n >= 4) {
#pragma unroll
            for (int i = 0; i < QUADS; ++i) raw[i] = *reinterpret_cast<const f32x4_any*>(scores + min(quad(i), last));
        } else {
#pragma unroll
            for (int i = 0; i < QUADS; ++i) raw[i] = f32x4_any{0.f, scores[max(n - 3, 0)], scores[max(n - 2, 0)], scores[n - 1]};   // tokens n - 4 .. n - 1
        }
#pragma unroll
        for (int i = 0; i < PER; ++i) keys[i] = own(i) ? score_key(raw[i >> 2][i & 3]) : 0u;
    }

    uint32_t thr_key = 0u;     // key of the k-th largest score
    uint32_t need_eq = 0u;     // how many tokens equal to it are taken
    const bool take_all = (k >= n);
    if (!take_all) {
        // range of the keys: block-wide minimum and maximum
        uint32_t kmin = 0xFFFFFFFFu, kmax = 0u;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            kmin = min(kmin, own(i) ? keys[i] : 0xFFFFFFFFu);
            kmax = max(kmax, keys[i]);   // (another lane's: 0)
        }
        kmin = over_row(kmin, lower);
        kmax = over_row(kmax, higher);
        for (int o = 32; o >= 16; o >>= 1) {
            kmin = min(kmin, (uint32_t)__shfl_xor((int)kmin, o));
            kmax = max(kmax, (uint32_t)__shfl_xor((int)kmax, o));
        }
        if (lane == 0) { wave_a[wave] = kmin; wave_b[wave] = kmax; }
        if (tid == 0) { s_prefix = 0u; s_remaining = (uint32_t)k; s_listed = 0u; }
        reinterpret_cast<uint4*>(hist)[tid] = make_uint4(0u, 0u, 0u, 0u);
        __syncthreads();
        kmin = __builtin_amdgcn_readfirstlane(over_row(wave_a[lane & (WAVES - 1)], lower));
        kmax = __builtin_amdgcn_readfirstlane(over_row(wave_b[lane & (WAVES - 1)], higher));
        // relative keys rk = key - kmin lie in [0, kmax - kmin]; digits of 12 bits (the last one narrower) are taken
        // from the highest bit in which the two extremes differ downwards
        const uint32_t span = kmax - kmin;
        int shift = (span == 0u) ? 1 : 32 - __clz((int)span);   // number of significant bits of the relative keys
        uint32_t mask = 0u;
        for (;;) {
            const int width = min(DIGIT, shift);
            shift -= width;
            const uint32_t digit_mask = (1u << width) - 1u;
            const uint32_t prefix = s_prefix;
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const uint32_t rk = keys[i] - kmin;
                if (own(i) && (rk & mask) == prefix) atomicAdd(&hist[(rk >> shift) & digit_mask], 1u);
            }
            __syncthreads();
            pick_digit(hist, wave_tot, &s_prefix, &s_remaining, &s_count, shift);
            mask |= digit_mask << shift;
            if (shift == 0 || s_count <= CANDIDATES) break;
            reinterpret_cast<uint4*>(hist)[tid] = make_uint4(0u, 0u, 0u, 0u);   // (read before pick_digit's barriers)
            __syncthreads();
        }
        if (shift > 0) {   // the remaining digits of at most CANDIDATES keys: count how many are larger than, and equal to, each
            const uint32_t prefix = s_prefix, count = s_count, remaining = s_remaining;
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const uint32_t rk = keys[i] - kmin;
                if (own(i) && (rk & mask) == prefix) candidates[atomicAdd(&s_listed, 1u)] = rk;
            }
            __syncthreads();
            // four threads per candidate, each counts in every fourth vector of the list (one thread each: 16 us instead of 12 for
            // 6196 scores of 50 different values, whose bins hold over a hundred)
            static_assert(4 * CANDIDATES <= SEL_THREADS, "candidates per pass");
            const uint32_t mine = candidates[min(tid >> 2, (int)count - 1)];
            uint32_t larger = 0u, equal = 0u;
            for (uint32_t j = 4 * (tid & 3); j < count; j += 16) {
                const uint4 c = *reinterpret_cast<const uint4*>(&candidates[j]);   // entries past `count` do not count
                const uint32_t v[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    larger += (j + e < count && v[e] > mine) ? 1u : 0u;
                    equal += (j + e < count && v[e] == mine) ? 1u : 0u;
                }
            }
            larger = over_quad(larger, add);
            equal = over_quad(equal, add);
            if (larger < remaining && larger + equal >= remaining) {   // (every copy of the k-th largest key writes the same)
                s_prefix = mine;
                s_remaining = remaining - larger;
            }
            __syncthreads();
        }
        thr_key = s_prefix + kmin;
        need_eq = s_remaining;
    }

    // ordered compaction: per-wave counts by ballots, one exchange of the 16 wave totals, then every wave
    // writes its tokens in (i, lane, e) order
    auto is_gt = [&](int i) { return own(i) && (take_all || keys[i] > thr_key); };
    auto is_eq = [&](int i) { return own(i) && !take_all && keys[i] == thr_key; };
    uint32_t w_gt = 0u, w_eq = 0u;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        w_gt += (uint32_t)__popcll(__ballot(is_gt(i)));
        w_eq += (uint32_t)__popcll(__ballot(is_eq(i)));
    }
    __syncthreads();   // wave_a / wave_b are free again
    if (lane == 0) { wave_a[wave] = w_gt; wave_b[wave] = w_eq; }
    __syncthreads();
    // equal keys and outputs of the waves before this one (of equal keys the first need_eq are taken)
    const int w2 = lane & (WAVES - 1);
    uint32_t eq_seen = __builtin_amdgcn_readfirstlane(over_row(w2 < wave ? wave_b[w2] : 0u, add));
    uint32_t pos = __builtin_amdgcn_readfirstlane(over_row(w2 < wave ? wave_a[w2] : 0u, add)) + min(eq_seen, need_eq);
#pragma unroll
    for (int i = 0; i < QUADS; ++i) {
        bool sel[4];
        uint32_t eq_at = eq_seen, at = pos;    // equal keys, outputs before this lane's four
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint64_t beq = __ballot(is_eq(4 * i + e));
            eq_at += lanes_below(beq);
            eq_seen += (uint32_t)__popcll(beq);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const bool eq = is_eq(4 * i + e);
            sel[e] = is_gt(4 * i + e) || (eq && eq_at < need_eq);
            eq_at += eq ? 1u : 0u;
            const uint64_t bsel = __ballot(sel[e]);
            at += lanes_below(bsel);
            pos += (uint32_t)__popcll(bsel);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (sel[e]) out[at] = min(quad(i), last) + e;
            at += sel[e] ? 1u : 0u;
        }
    }
}

template <int PER>
__global__ __launch_bounds__(SEL_THREADS) void select_topk_kernel(const float* __restrict__ scores, int64_t n,
                                                                  int64_t k, int nq, int32_t* __restrict__ out) {
    // question tokens: positions n .. n + nq - 1
    for (int i = threadIdx.x; i < nq; i += SEL_THREADS) out[k + i] = (int32_t)(n + i);
    if (k <= 0 || n <= 0) return;   // (there need be no scores then)
    select_in_workgroup<PER>(scores, (int)n, k, out);
}

// At most 128 scores: a lane has a token and counts the keys above its own, one broadcast after the other; a wave for each 64 tokens, each of which holds all keys.  Fewer than k
// of them: chosen, or tied at the k-th largest key, of whose tokens the first are taken.  No histogram, a barrier at most, nearly the same time whatever the scores are; what bounds
// it are the launch and three instructions a key.  Other waves are there for the question tokens only.
constexpr int FEW_WAVES = 2;
__global__ __launch_bounds__(SEL_THREADS) void select_few_kernel(const float* __restrict__ scores, int n, int k, int nq, int32_t* __restrict__ out) {
    __shared__ int s_chosen[FEW_WAVES], s_most[FEW_WAVES], s_tied[FEW_WAVES];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), token = threadIdx.x;
    for (int i = threadIdx.x; i < nq; i += blockDim.x) out[k + i] = n + i;   // question tokens: positions n .. n + nq - 1
    if (k <= 0) return;                                                      // (there need be no scores then)
    uint32_t keys[FEW_WAVES], key = 0u;   // (0, past the end: above no key)
#pragma unroll
    for (int i = 0; i < FEW_WAVES; ++i) keys[i] = 64 * i + lane < n ? score_key(scores[min(64 * i + lane, n - 1)]) : 0u;
#pragma unroll
    for (int i = 0; i < FEW_WAVES; ++i) key = wave == i ? keys[i] : key;
    int above = token < n ? 0 : k;
    if (64 * wave < n) {
#pragma unroll
        for (int i = 0; i < FEW_WAVES; ++i)
            for (int j = 0; j < min(64, n - 64 * i); j += 16)
#pragma unroll
                for (int u = 0; u < 16; ++u) above += __builtin_amdgcn_readlane(keys[i], j + u) > key ? 1 : 0;
    }
    // the tied key, if it has more tokens than are taken, is the chosen one with the most keys above it
    auto largest = [&] {
        const uint32_t v = over_row(above < k ? (uint32_t)above : 0u, higher);
        return (int)max(max(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)), max(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
    };
    uint64_t chosen = __ballot(above < k);
    int total = __popcll(chosen), at = 0, most = 0, tied_before = 0;
    if (n > 64) {
        const int own = largest();
        if (wave < FEW_WAVES && lane == 0) { s_chosen[wave] = total; s_most[wave] = own; }
        const int own_tied = __popcll(__ballot(above < k && above == own));
        if (wave < FEW_WAVES && lane == 0) s_tied[wave] = own_tied;
        __syncthreads();
        if (64 * wave >= n) return;
        const int waves = (n + 63) / 64;
        total = 0;
        for (int w = 0; w < waves; ++w) { total += s_chosen[w]; most = max(most, s_most[w]); }
        int above_before = 0;
        for (int w = 0; w < wave; ++w) {
            const int tied = s_most[w] == most ? s_tied[w] : 0;
            tied_before += tied;
            above_before += s_chosen[w] - tied;
        }
        at = above_before + min(tied_before, k - most);
    } else {
        if (wave > 0) return;
        if (total > k) most = largest();
    }
    if (total > k) {
        const uint64_t tied = __ballot(above == most);
        chosen = __ballot(above < most || (above == most && tied_before + (int)lanes_below(tied) < k - most));
    }
    if (chosen >> lane & 1) out[at + lanes_below(chosen)] = token;
}

// The same for n <= 64 PER scores in one wave: no histogram, no barrier, no LDS.  Token 64 i + lane is key i of the lane, so
// (i, lane) order is index order.  The threshold key is found bit by bit from the highest one in which the keys differ: a bit
// stays set if at least k keys reach it, counted by ballots (PER compares and scalar adds); as soon as exactly k keys reach the threshold, the set
// is known (with n distinct scores after about log2(n) + 4 bits; ties go on to the last bit and take the lowest indices).  What bounds it is the one wave's
// issue, 12 PER cycles a bit.
template <int PER>
__device__ __forceinline__ void select_in_wave(const float (&raw)[PER], int n, int k, int32_t* __restrict__ out) {
    const int lane = threadIdx.x & 63;
    uint32_t keys[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) keys[i] = score_key(raw[i]);
    // keys past the end are copies of the last token's: `valid` leaves them out of every count
    auto valid = [&](int i) { return 64 * i + lane < n; };
    uint32_t thr = 0u, need_eq = 0u;      // taken: keys above thr, and the first need_eq that equal it
    if (k < n) {
        const uint32_t key0 = __builtin_amdgcn_readfirstlane(keys[0]);
        uint32_t diff = 0u;
#pragma unroll
        for (int i = 0; i < PER; ++i) diff |= keys[i] ^ key0;
        for (int o = 32; o > 0; o >>= 1) diff |= (uint32_t)__shfl_xor((int)diff, o);
        diff = __builtin_amdgcn_readfirstlane(diff);
        int bit = diff ? 31 - __clz((int)diff) : -1;                       // highest bit in which two keys differ
        thr = bit >= 31 ? 0u : bit < 0 ? key0 : key0 >> (bit + 1) << (bit + 1);   // (at least k keys reach it)
        bool exact = false;
        for (; bit >= 0 && !exact; --bit) {
            const uint32_t cand = thr | 1u << bit;
            int count = 0;
#pragma unroll
            for (int i = 0; i < PER; ++i) count += __popcll(__ballot(valid(i) && keys[i] >= cand));
            if (count >= k) thr = cand;
            exact = count == k;
        }
        int above = 0;
#pragma unroll
        for (int i = 0; i < PER; ++i) above += __popcll(__ballot(valid(i) && keys[i] > thr));
        need_eq = (uint32_t)(k - above);      // (exact: as many as there are)
    }
    const bool take_all = k >= n;
    // ordered compaction
    int pos = 0;
    uint32_t eq_seen = 0u;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const bool gt = valid(i) && (take_all || keys[i] > thr), eq = valid(i) && !take_all && keys[i] == thr;
        const uint64_t beq = __ballot(eq);
        const bool sel = gt || (eq && eq_seen + lanes_below(beq) < need_eq);
        const uint64_t bsel = __ballot(sel);
        if (sel) out[pos + lanes_below(bsel)] = 64 * i + lane;
        pos += __popcll(bsel);
        eq_seen += (uint32_t)__popcll(beq);
    }
}

// The scores' partial sums added up and selected from in one launch (score_reduce_kernel's sums in its order): a launch less for short prompts, whose calls are bound
// by them on the device and on the host (4 x 128 tokens, 4 partial sums: the host's part of a selection call 13.0 -> 8.3 us).  Thread (quad of tokens, a): group w = a, a + 4, ..
// of eight partial sums, 16 bytes a load (one token a thread is a quarter of a compute unit's load rate: 880 tokens, 40 partial sums 2 us more); then a token a thread; then
// the selection, behind the sums by wave 0 alone up to 512 tokens (4 x 128 tokens 3.8 us, 5.2 by the workgroup), else by the workgroup (880 tokens 6.4 us, 8.4 by a wave).
constexpr int SUM_GROUPS = 8;   // of eight partial sums at most
template <bool ONE_WAVE>
__global__ __launch_bounds__(SEL_THREADS) void sum_and_select_kernel(const float* __restrict__ partial, int n_parts, int n, float* __restrict__ scores, int k,
                                                              int nq, int32_t* __restrict__ out) {
    typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    __shared__ __attribute__((aligned(16))) float sums[SUM_GROUPS][1024];
    const int tid = threadIdx.x, groups = (n_parts + 7) / 8;
    const int j = min(4 * (tid & 255), max(n - 4, 0));   // (the last quad of a number that is none of fours overlaps the one in front: the same sums twice)
    for (int w = tid >> 8; w < groups; w += 4) {         // group w: parts w, w + groups, ...
        f32x4u v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const float* p = partial + (size_t)min(w + u * groups, n_parts - 1) * n + j;
            if (n >= 4) v[u] = *reinterpret_cast<const f32x4u*>(p);
            else v[u] = f32x4u{p[0], p[min(1, n - 1)], p[min(2, n - 1)], 0.f};
        }
        f32x4 g = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (w + u * groups < n_parts) g += f32x4(v[u]);
#pragma unroll
        for (int e = 0; e < 4; ++e) sums[w][j + e] = g[e];
    }
    for (int i = tid; i < nq; i += 1024) out[k + i] = n + i;   // question tokens: positions n .. n + nq - 1
    __syncthreads();
    if (tid < n) {
        float t = 0.f;
        for (int w = 0; w < groups; ++w) t += sums[w][tid];
        scores[tid] = t;
        sums[0][tid] = t;   // (this token's words are this thread's)
    }
    __syncthreads();
    if (k <= 0) return;
    if constexpr (ONE_WAVE) {
        if (tid >= 64) return;
        float raw[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) raw[i] = sums[0][min(64 * i + tid, n - 1)];
        select_in_wave<8>(raw, n, k, out);
    } else {
        select_in_workgroup<4>(sums[0], n, k, out);
    }
}

bool sum_and_select_pays(int64_t n, int n_parts) { return n > 0 && n <= 1024 && n_parts <= 8 * SUM_GROUPS; }

hipError_t launch_sum_and_select(const float* partial, int n_parts, int n, float* scores, int k, int nq, int32_t* q_index, hipStream_t st) {
    if (n <= 512)
        sum_and_select_kernel<true><<<dim3(1), dim3(SEL_THREADS), 0, st>>>(partial, n_parts, n, scores, k, nq, q_index);
    else
        sum_and_select_kernel<false><<<dim3(1), dim3(SEL_THREADS), 0, st>>>(partial, n_parts, n, scores, k, nq, q_index);
    return hipGetLastError();
}

static_assert(SELECT_ONE_WORKGROUP_MAX == (int64_t)SEL_THREADS * 32, "largest score vector of the one-workgroup kernel");

hipError_t launch_select(const float* scores, int64_t n, int64_t k, int nq, int32_t* q_index, uint32_t* tmp,
                         size_t tmp_bytes, hipStream_t st) {
    if (k + nq == 0) return hipSuccess;
    // Up to 128 scores by counting, a wave for each 64 of them and of the question tokens (us, counted : workgroup, 3, 64, 100, 128 scores 2.2, 2.7, 3.9, 4.1 : 4.6, 160 and 256
    // 4.8 and 6.4 : 4.6; a bit-by-bit search in one wave took 3.1 to 5.3, 8.6 with ties).
    if (n <= 64 * FEW_WAVES)
        select_few_kernel<<<dim3(1), dim3(64 * std::max((int)(n + 63) / 64, std::min(SEL_THREADS / 64, std::max(1, (nq + 63) / 64)))), 0, st>>>(scores, (int)n, (int)k, nq, q_index);
    else if (n <= (int64_t)SEL_THREADS * 4)
        select_topk_kernel<4><<<dim3(1), dim3(SEL_THREADS), 0, st>>>(scores, n, k, nq, q_index);
    else if (n <= (int64_t)SEL_THREADS * 8)
        select_topk_kernel<8><<<dim3(1), dim3(SEL_THREADS), 0, st>>>(scores, n, k, nq, q_index);
    else if (n <= (int64_t)SEL_THREADS * 16)
        select_topk_kernel<16><<<dim3(1), dim3(SEL_THREADS), 0, st>>>(scores, n, k, nq, q_index);
    else if (n <= (int64_t)SEL_THREADS * 32)
        select_topk_kernel<32><<<dim3(1), dim3(SEL_THREADS), 0, st>>>(scores, n, k, nq, q_index);
    else
        return launch_select_large(scores, n, k, nq, q_index, tmp, tmp_bytes, st);
    return hipGetLastError();
}

}  // namespace fr
