// Query-Guided Selection, critical scores (Sec. 3.2) on the gfx950 matrix cores: bf16 and fp32, head_dim 64 and 128, any
// group size.
//
// The score of context token j is the column sum, over all question rows and query heads, of the softmax-normalised
// attention weights.  A weight needs its row's normaliser, i.e. the logits of every key in the softmax's scope, before it
// can be added up.  Where the scope is a chunk of at most SEG keys (the usual case: chunks of 1024 tokens, softmax per
// chunk) one workgroup holds the whole chunk: its keys sit in the registers of its eight (four) waves and the query columns
// stream past them, so every logit and every exponential is formed once.  Otherwise the chunk (or, for one softmax over
// the whole context, the prompt) is cut into segments of at most SEG keys and walked twice.
//
//   MODE_FUSED   logits -> weights exp2(s - ref) -> sum l per query column (exchanged between the waves through LDS) ->
//                score[key] += weight / l
//   MODE_LSE     the same up to l; leaves ref + log2 l per (segment, column)
//   MODE_GIVEN   score[key] += exp2(s - lse) with the normalisers that score_lse_combine_kernel made of those
//   reduce       scores[j] = sum over column ranges and KV heads of the partial sums, in a fixed order
//
// A "query column" n of KV head g is the pair (question token n / G, query head g G + n % G).
//
// Layout.  S^T = K Q^T with 16 x 16 tiles: keys on the accumulator's register dimension, query columns on lanes.  A wave
// owns key blocks w, w + 8, w + 16, ... (16 keys each; the chunk's last, possibly partial block is then the last of its
// wave, the only one that needs a mask).  Per 16 columns a wave has 4 NB logits per lane; its accumulators of
// the score (4 NB per lane, one per key and column mod 16) are added up across the 16 lanes once at the end.
// 128 keys x 256 bytes per wave are 128 registers; with 32 x 32 tiles the weights and the accumulators would be 64
// registers each and would not fit beside them, with 16 x 16 tiles they are 32.  What bounds the kernel is the vector
// ALU: fma + exp2 + add + fma per logit, 20 issue cycles of a wave for 64 logits against 16 of the matrix pipe (head_dim
// 128, bf16).  The weights of a step are kept until the next one: its barrier is also the one that makes the other waves'
// sums visible, so a step has a single barrier.
//
// Exponent reference.  exp2(s - ref) / sum exp2(s - ref) does not depend on ref.  The reference of a column is the maximum
// over the segment's first 16 keys, whose logits wave 0 has a step ahead; l >= 1 then, and fp32 has 2^127 of headroom.  If a later logit
// exceeds the reference by more than about 2^100 the sum shows it, and the workgroup repeats its range with the exact
// maxima.
//
// Measured (16 x 1024 keys, 512 question tokens, 32/8 heads, bf16, back to back, with the reduction): 83 us, of which 5 load the keys and a step of 16 columns
// takes 0.99; with keys loaded straight into fragment registers (12 us: see there), the order of a step's instructions left to the compiler (1.19 us a step) and a
// spilled index that was waited for in the loop together with the copies 96; the two passes of k_score_mfma.hip 66 + 62 + 5 us.  3 x 900 keys, 100 question tokens 20.3 -> 15.7.  28/4
// heads 90 -> 79; fp32, 4 x 128 keys, 32 question tokens: 7 us.  Vector instructions are issued in 70 % of the kernel's cycles (the matrix pipes work in 37 %): four per logit are the sums' own, one more
// per logit is the references, the sums' exchange and the fragments' addresses.
// All sums run in a fixed order: the scores are reproducible bit for bit.
#include "fr_internal.hpp"
#include "k_rotate.hpp"

#include <algorithm>
#include <type_traits>
#include <utility>

namespace fr {

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

enum { MODE_FUSED = 0, MODE_LSE = 1, MODE_GIVEN = 2 };
enum { SRC_PROMPT = 0, SRC_STORE_INTERLEAVED = 1, SRC_STORE_HALF = 2 };

constexpr int MOST_WAVES = 8;     // of a workgroup; chunks of up to half as many keys have four
constexpr int TILE = 64;          // query columns per LDS tile
constexpr int RANGE_UNIT = 32;    // column ranges are multiples of the longest step
constexpr int MAX_COLS = 2048;    // query columns per workgroup (their references sit in LDS)
constexpr int CG2_MAX_KEYS = 20;  // most 4-register key vectors per lane with two column groups per step in MODE_FUSED

template <typename T, int D, int WAVES = MOST_WAVES>
struct Op {
    static constexpr int ROWB = D * (int)sizeof(T);            // bytes of a head row: 128, 256 or 512
    static constexpr int NV = ROWB / 16;                       // its 16-byte vectors
    static constexpr int NJ = NV / 4;                          // vectors per lane: lane (row x, quarter kg) holds vectors 4 j + kg
    static constexpr int NB_MAX = ROWB == 512 ? 4 : 8;         // key blocks per wave: NB x NJ x 4 registers
    static constexpr int SEG = 16 * WAVES * NB_MAX;            // most keys of a workgroup
    static constexpr int STAGED = ROWB == 512 ? 1 : 512 / ROWB;   // key blocks of a wave in LDS at a time (two workgroups of four waves share the LDS)
    // 16-byte vector c of row r sits in slot c ^ swz(r) of the row: any 16 rows' vectors c then start in 16 different
    // 16-byte bank groups (two 128-byte rows share one stretch of banks)
    static __device__ __forceinline__ int swz(int r) { return ROWB == 128 ? (r >> 1) & 7 : r & 15; }
    static __device__ __forceinline__ void multiply(const u32x4& a, const u32x4& b, f32x4& acc) {
        if constexpr (sizeof(T) == 2) {
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[e]), __uint_as_float(b[e]), acc, 0, 0, 0);
        }
    }
};

struct ScoreArgs {
    const void* q;
    const void* k;
    const double* theta;      // [D / 2] rotary frequencies, stores only
    float* lse2;              // [Hkv][lse_rows][col_end - col0] base-2 normalisers of the two-pass modes
    float* partial;           // [n_split][Hkv][L_ctx]
    int col0, col_end;        // the launch's query columns
    int nq, Hq, Hkv, G, lse_rows, n_split, split_cols, max_parts, src, global_scope;
    uint32_t magic;           // ceil(2^32 / G): n / G = mulhi(n, magic) for G > 1
    float scale_log2e;
    ChunkTable ct;
    ChunkRows rows;
    ChunkDeltas deltas;       // stores only
    uint8_t order[FR_MAX_CHUNKS];   // chunks, longest first
};

// A chunk of `len` keys as segments of equal length (the last one may be shorter): keys per segment, and their number.
template <int SEG>
__host__ __device__ __forceinline__ int segment_keys(int len) {
    const int parts = (len + SEG - 1) / SEG;
    return (len + parts - 1) / parts;
}
template <int SEG>
__host__ __device__ __forceinline__ int segments(int len) {
    return len <= SEG ? (len > 0 ? 1 : 0) : (len + segment_keys<SEG>(len) - 1) / segment_keys<SEG>(len);
}
// Row of lse2 that holds segment 0 of chunk c: chunks before it have at most c + off[c] / SEG segments together.
template <int SEG>
__host__ __device__ __forceinline__ int lse_row(int c, int off) { return c + off / SEG; }

__device__ __forceinline__ uint32_t lds_address(const void* p) {
    return __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) const unsigned char*)p);
}
__device__ __forceinline__ void plain_barrier() {   // without the fences of __syncthreads(): the waits are explicit
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}
// f(0), f(1), ... f(N - 1), each with its own constant (`#pragma unroll` gives up on long bodies, and arrays indexed by them go to memory).
template <typename F, int... I>
__device__ __forceinline__ void static_for(F&& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
// Until all but the wave's last n copies have landed; n is a constant once loops are unrolled.
__device__ __forceinline__ void wait_copies_but(int n) {
    switch (n) {
#define FR_WAIT(N) case N: __builtin_amdgcn_s_waitcnt(0x0f70 | N); break;
        FR_WAIT(2) FR_WAIT(4) FR_WAIT(6) FR_WAIT(8) FR_WAIT(10)
#undef FR_WAIT
        default: __builtin_amdgcn_s_waitcnt(0x0f70);
    }
}
// Sum and maximum over the four lanes that hold the same column (lanes x, x + 16, x + 32, x + 48).
__device__ __forceinline__ float column_sum(float v) {
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float column_max(float v) {
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
template <int CTRL>
__device__ __forceinline__ float add_rotated(float v) {
    return v + __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float row_sum(float v) {   // over the 16 lanes of a row: rotations by 8, 4, 2, 1
    v = add_rotated<0x128>(v);
    v = add_rotated<0x124>(v);
    v = add_rotated<0x122>(v);
    return add_rotated<0x121>(v);
}

template <typename T, int D, int WAVES>
struct Smem {
    alignas(1024) unsigned char q[2][TILE * Op<T, D>::ROWB];
    float ref[MAX_COLS + 32];      // exponent references, or the given normalisers (and room for those of a step too many)
    alignas(16) float l[2][32][WAVES];
    float2 rotation[D / 2];        // of the chunk's keys, stores only
    alignas(1024) unsigned char stage[WAVES][Op<T, D>::STAGED * 16 * Op<T, D>::ROWB];   // key blocks on their way into registers
};

// Work of one workgroup: keys [s0, s0 + len) of chunk c, query columns [n0, n1).  NB = key blocks per wave.
template <typename T, int D, int WAVES, int MODE, int NB>
__device__ __forceinline__ void walk_columns(const ScoreArgs& a, Smem<T, D, WAVES>& sm, int g, int c, int s0, int len, int row,
                                             int n0, int n1, int split) {
    using O = Op<T, D, WAVES>;
    // Column groups of 16 per step.  A step costs about 0.2 us besides its logits (barrier, exchange of the sums, LDS
    // latency), so it takes two groups wherever the registers hold them: the weights are the only ones that double.
    constexpr int CG = (MODE == MODE_FUSED && NB * Op<T, D>::NJ > CG2_MAX_KEYS) ? 1 : 2;
    constexpr int STEP = 16 * CG, SPT = TILE / STEP;                 // columns per step, steps per tile
    // The logits of a step come as NB x CG units of 16 keys x 16 columns, in pairs (two independent chains of matrix
    // instructions): unit k is block k / CG, group k % CG.
    constexpr int NU = NB * CG, NP = (NU + 1) / 2;
    constexpr int NJ = O::NJ;                                        // vectors per lane
    const int tid = threadIdx.x, lane = tid & 63, x = lane & 15, kg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int NQG = a.nq * a.G;
    const T* __restrict__ q = static_cast<const T*>(a.q);
    const T* __restrict__ k = static_cast<const T*>(a.k);
    // row of the queries that holds column n (past the end: a copy of the last one): (n / G) Hq + g G + n % G
    const uint32_t per_column = a.G > 1 ? 1u : (uint32_t)a.Hq, per_token = a.G > 1 ? (uint32_t)(a.Hq - a.G) : 0u;
    auto column_row = [&](int n) -> uint32_t {
        n = min(n, NQG - 1);
        return (uint32_t)n * per_column + __umulhi((uint32_t)n, a.magic) * per_token + (uint32_t)(g * a.G);
    };
    // copies of one tile of query columns, global -> LDS directly: 1 KB per wave instruction, lane = (row, slot)
    auto copy_tile = [&](int t, int buf) {
        constexpr int COPIES = TILE * O::ROWB / 1024 / WAVES;
        int ln = lane;   // (opaque: the addresses are formed anew for every tile, no register holds parts of them meanwhile)
        asm volatile("" : "+v"(ln));
#pragma unroll
        for (int i = 0; i < COPIES; ++i) {
            const int r = (1024 / O::ROWB) * (COPIES * wave + i) + ln / O::NV;
            const unsigned char* src = reinterpret_cast<const unsigned char*>(q) + ((uint64_t)column_row(n0 + TILE * t + r) * (uint32_t)O::ROWB + 16 * ((ln % O::NV) ^ O::swz(r)));
            const uint32_t dst = lds_address(sm.q[buf]) + (uint32_t)(COPIES * wave + i) * 1024u;
            asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(src), "s"(dst) : "memory");
        }
    };
    const int n_steps = (n1 - n0 + STEP - 1) / STEP, n_tiles = (n_steps + SPT - 1) / SPT;
    copy_tile(0, 0);
    if (n_tiles > 1) copy_tile(1, 1);

    // This lane's vectors 4 j + kg of keys 16 (wave + 8 b) + x; keys past the end: a copy of the last one.  Through LDS, STAGED blocks of a wave at a
    // time: a fragment's 16 rows x 64 bytes per instruction, neighbouring lanes in different rows, take the vector cache 64 accesses per KB, rows side by
    // side 16.
    u32x4 kf[NB][NJ];
    {
        constexpr int BLOCK = 16 * O::ROWB, COPIES = BLOCK / 1024, RC = 1024 / O::ROWB;
        auto copy_block = [&](int b) {
#pragma unroll
            for (int i = 0; i < COPIES; ++i) {
                const int r = RC * i + lane / O::NV;
                const int j = min(16 * (wave + WAVES * b) + r, len - 1) + s0;
                const int64_t at = a.src == SRC_PROMPT ? (int64_t)j : (int64_t)a.rows.row0[c] + (j - a.ct.off[c]);
                const unsigned char* src = reinterpret_cast<const unsigned char*>(k + (at * a.Hkv + g) * D) + 16 * ((lane % O::NV) ^ O::swz(r));
                const uint32_t dst = lds_address(sm.stage[wave]) + (uint32_t)(b % O::STAGED) * BLOCK + (uint32_t)i * 1024u;
                asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(src), "s"(dst) : "memory");
            }
        };
        static_assert(COPIES * (O::STAGED - 1) <= 10 && COPIES % 2 == 0, "wait_copies_but");
#pragma unroll
        for (int b = 0; b < O::STAGED && b < NB; ++b) copy_block(b);
        auto load_blocks = [&](auto rotate) __attribute__((always_inline)) {
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                asm volatile("" ::: "memory");
                wait_copies_but(COPIES * min(NB - 1 - b, O::STAGED - 1));   // the later blocks'
                asm volatile("" ::: "memory");
                const unsigned char* row = sm.stage[wave] + (b % O::STAGED) * BLOCK;
#pragma unroll
                for (int j = 0; j < NJ; ++j) kf[b][j] = *reinterpret_cast<const u32x4*>(row + ((x * O::ROWB + 16 * (kg ^ O::swz(x))) ^ (64 * j)));
                if (b + O::STAGED < NB) {
                    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0): the slot has been read
                    copy_block(b + O::STAGED);
                }
                rotate(b);
#pragma unroll
                for (int j = 0; j < NJ; ++j) asm volatile("" : "+v"(kf[b][j]));   // rounded here: the compiler moves what the layouts' paths end
                __builtin_amdgcn_sched_barrier(0);                                // with behind them, with twice the registers
            }
        };
        // From a store: moved to their prompt positions on the way.  A lane meets the same NJ vectors of every key row, so their rotations, which the
        // workgroup forms itself, stay in its registers meanwhile.  Selection call, 28 query heads on 4 KV heads of 128 in bf16: 16 chunks of 1024 keys and
        // 512 question tokens 95.1 -> 80.4 us (from a prompt 80.3), 3 of 900 and 100 28.7 -> 19.3 (14.9), against a table in memory, which took a launch of
        // its own, and the rotations loaded from it block by block after all keys.
        if (a.src == SRC_PROMPT) {
            load_blocks([](int) __attribute__((always_inline)) {});
        } else {
            constexpr int N = 16 / (int)sizeof(T);
            if (tid < D / 2) sm.rotation[tid] = chunk_rotation(a.deltas.delta[c], a.theta[tid]);
            __syncthreads();
            if (a.src == SRC_STORE_INTERLEAVED) {
                float2 t[NJ][N / 2];
#pragma unroll
                for (int j = 0; j < NJ; ++j)
#pragma unroll
                    for (int e = 0; e < N / 2; ++e) t[j][e] = sm.rotation[N / 2 * (4 * j + kg) + e];
                load_blocks([&](int b) __attribute__((always_inline)) {
#pragma unroll
                    for (int j = 0; j < NJ; ++j) kf[b][j] = rotate_vector<T, FR_ROPE_INTERLEAVED>(kf[b][j], kf[b][j], t[j], false);
                });
            } else {   // (p, p + D/2): the partner of vector 4 j + kg is vector 4 (j + NJ / 2) + kg of the same lane
                static_assert(NJ % 2 == 0, "pairs inside a lane");
                float2 t[NJ / 2][N];
#pragma unroll
                for (int j = 0; j < NJ / 2; ++j)
#pragma unroll
                    for (int e = 0; e < N; ++e) t[j][e] = sm.rotation[N * (4 * j + kg) + e];
                load_blocks([&](int b) __attribute__((always_inline)) {
#pragma unroll
                    for (int j = 0; j < NJ / 2; ++j) {
                        const u32x4 lo = kf[b][j], hi = kf[b][j + NJ / 2];
                        kf[b][j] = rotate_vector<T, FR_ROPE_HALF>(lo, hi, t[j], true);
                        kf[b][j + NJ / 2] = rotate_vector<T, FR_ROPE_HALF>(hi, lo, t[j], false);
                    }
                });
            }
        }
    }
    const int last_key = 16 * (wave + WAVES * (NB - 1)) + 4 * kg;   // of the wave's last block: the lane's four keys
    f32x4 last_block;   // its products start from here: keys past the end come to weight 0
#pragma unroll
    for (int i = 0; i < 4; ++i) last_block[i] = last_key + i < len ? 0.f : -INFINITY;
    if constexpr (MODE == MODE_GIVEN) {
        const float* src = a.lse2 + ((size_t)g * a.lse_rows + row) * (a.col_end - a.col0) + (n0 - a.col0);
        for (int i = tid; i < n_steps * STEP; i += 64 * WAVES) sm.ref[i] = n0 + i < n1 ? src[i] : INFINITY;
    }

    float sc[NB][4], p[CG][NB][4];
    // fragments of step st's columns (vector 4 j + kg of row 16 cg + x), and the products of a pair of units
    u32x4 qv[CG][NJ];
    const int q_lane = x * O::ROWB + 16 * (kg ^ O::swz(x));   // (swz(16 i + x) = swz(x))
    auto q_at = [&](int st) {
        return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)sm.q +
               ((st / SPT) & 1) * (uint32_t)sizeof(sm.q[0]) + (st % SPT) * (STEP * O::ROWB) + (uint32_t)q_lane;
    };
    auto load_vector = [&](uint32_t at, int cg, int j) {   // 16 ((4 j + kg) ^ swz) = 64 j ^ 16 (kg ^ swz): one register for all vectors
        qv[cg][j] = *(__attribute__((address_space(3))) const u32x4*)(uintptr_t)((at ^ (64u * j)) + cg * (16 * O::ROWB));
    };
    auto load_q = [&](int st) {
        const uint32_t at = q_at(st);
#pragma unroll
        for (int cg = 0; cg < CG; ++cg)
#pragma unroll
            for (int j = 0; j < NJ; ++j) load_vector(at, cg, j);
    };
    f32x4 s[2][2];
    // Multiplication m of a pair's 2 NJ: vector m / 2 of unit m % 2.
    auto product = [&](int pr, int m) {
        const int unit = 2 * pr + m % 2;
        if (unit >= NU) return;
        f32x4& acc = s[pr & 1][m % 2];
        if (m < 2) acc = unit / CG == NB - 1 ? last_block : f32x4{0.f, 0.f, 0.f, 0.f};
        O::multiply(kf[unit / CG][m / 2], qv[unit % CG][m / 2], acc);
    };
    auto products = [&](int pr) {
#pragma unroll
        for (int m = 0; m < 2 * NJ; ++m) product(pr, m);
    };
    auto wait_copies = [&] { __builtin_amdgcn_s_waitcnt(0x0f70); };   // vmcnt(0)
    auto wait_lds = [&] { __builtin_amdgcn_s_waitcnt(0xc07f); };      // lgkmcnt(0)
    bool bad = false;
    int column = x;   // (its own register: one that came back from scratch memory at the loop's entry would be waited for in every step, with the copies)
    // 1 / l of this lane's column of group cg of step st (0 past the last column); MODE_LSE: the normaliser goes out
    auto finish_column = [&](int st, int cg, const f32x4 (&sums)[WAVES / 4]) -> float {
        const int i = STEP * st + 16 * cg + column;
        float l = (sums[0][0] + sums[0][1]) + (sums[0][2] + sums[0][3]);
        if constexpr (WAVES == 8) l += (sums[1][0] + sums[1][1]) + (sums[1][2] + sums[1][3]);
        bad = bad || !(l < 0x1p100f);
        if constexpr (MODE == MODE_LSE) {
            if (wave == 0 && kg == 0 && i < n1 - n0)
                a.lse2[((size_t)g * a.lse_rows + row) * (a.col_end - a.col0) + (n0 - a.col0) + i] = sm.ref[i] + __builtin_amdgcn_logf(l);
            return 0.f;
        } else {
            return i < n1 - n0 ? __builtin_amdgcn_rcpf(l) : 0.f;
        }
    };
    // the references of step st's columns: keys 0 .. 15 are block 0 of wave 0, whose logits are units 0 and (CG = 2) 1
    auto set_references = [&](int st) {
#pragma unroll
        for (int cg = 0; cg < CG; ++cg) {
            const f32x4& t = s[0][cg];
            sm.ref[STEP * st + 16 * cg + x] = column_max(fmaxf(fmaxf(t[0], t[1]), fmaxf(t[2], t[3]))) * a.scale_log2e;
        }
    };
    for (int attempt = 0;; ++attempt) {
        const bool fixed = MODE != MODE_GIVEN && attempt == 0 && wave == 0;   // this wave sets the references as it goes
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                sc[b][i] = 0.f;
#pragma unroll
                for (int cg = 0; cg < CG; ++cg) p[cg][b][i] = 0.f;
            }
        bad = false;
        wait_copies();
        wait_lds();
        plain_barrier();
        load_q(0);
        products(0);
        if (fixed) set_references(0);
        // Step st: its first pair's products were issued in the step before.  The barrier makes the other waves' sums and the
        // references visible; in a tile's last step also the next tile, which the fragments of the next step come from, and
        // it frees this tile's slot (the fragments of the tile's last step were read before the barrier).
        asm volatile("" : "+v"(column));
        for (int st = 0; st < n_steps; ++st) {
            const bool last_of_tile = st % SPT == SPT - 1;
            if (last_of_tile) wait_copies();
            wait_lds();
            plain_barrier();
            if (last_of_tile && st / SPT + 2 < n_tiles) copy_tile(st / SPT + 2, (st / SPT) & 1);
            float f[CG], ref[CG], lsum[CG][2], w[4];
            f32x4 l[CG][WAVES / 4];   // the waves' sums
            const uint32_t next_q = q_at(st + 1);
#pragma unroll
            for (int cg = 0; cg < CG; ++cg) {   // all of the step's first reads at once
                ref[cg] = sm.ref[STEP * st + 16 * cg + x];
                if constexpr (MODE != MODE_GIVEN) {
#pragma unroll
                    for (int h = 0; h < WAVES / 4; ++h) l[cg][h] = *reinterpret_cast<const f32x4*>(&sm.l[(st + 1) & 1][16 * cg + x][4 * h]);
                }
                lsum[cg][1] = f[cg] = 0.f;   // (of one block: nothing else comes to it)
            }
            // The step's logits one after the other, each with its share of the next pair's products (the last pair's: of the next step's first one): multiply,
            // add and exponentiate stand one logit apart, so that no instruction waits for the one in front of it, and a matrix instruction runs
            // beside the vector instructions of its own wave.  (The order is pinned: left to the compiler, also with scheduling groups, the matrix instructions
            // gather in dependent chains, and both waves of a SIMD, which leave the barrier together, first wait for the one pipe and then for the other.)
            // A weight takes the register of the step before, whose weight joins the score in front of it; those of the first LATE logits wait in registers of
            // their own (1 / l has come through LDS and a sum by then).
            constexpr int LOGITS = 4 * NU;
            constexpr int LATE = MODE == MODE_FUSED && LOGITS >= 8 ? 4 : 0;
            auto finish = [&] {
#pragma unroll
                for (int cg = 0; cg < CG; ++cg) f[cg] = (MODE != MODE_GIVEN && st > 0) ? finish_column(st - 1, cg, l[cg]) : 0.f;
            };
            if (LATE == 0) finish();
            float t[2], e[2];
            auto unit_of = [](int n) { return n / 4; };
            auto settle = [&](int n) {
                const int b = unit_of(n) / CG, cg = unit_of(n) % CG;
                sc[b][n % 4] = __builtin_fmaf(p[cg][b][n % 4], f[cg], sc[b][n % 4]);
                asm volatile("" : "+v"(sc[b][n % 4]));   // (here, not behind the branch below)
            };
            static_for([&](auto index) __attribute__((always_inline)) {
                constexpr int n = decltype(index)::value, pr = n / 8, in_pair = pr == NP - 1 ? LOGITS - 8 * pr : 8;   // logits of this pair
                constexpr int next = n >= LOGITS ? -1 : pr + 1 < NP ? pr + 1 : NP % 2 == 0 ? 0 : -1;
                if constexpr (next >= 0) {
#pragma unroll
                    for (int m = (n % 8) * 2 * NJ / in_pair; m < (n % 8 + 1) * 2 * NJ / in_pair; ++m) {
                        product(next, m);
                        if (pr == NP - 2 && m % 2 == 1) {   // the last products with these columns: the next step's follow
#pragma unroll
                            for (int cg = 0; cg < CG; ++cg) load_vector(next_q, cg, m / 2);   // (past the last step: read, never used)
                        }
                    }
                }
                if constexpr (n < LOGITS) {
                    t[n & 1] = __builtin_fmaf(s[pr & 1][unit_of(n) & 1][n % 4], a.scale_log2e, -ref[unit_of(n) % CG]);
                    if (MODE == MODE_FUSED && n >= LATE) settle(n);
                    if constexpr (n >= LATE && n < 2 * LATE) {
                        settle(n - LATE);
                        p[unit_of(n - LATE) % CG][unit_of(n - LATE) / CG][n % 4] = w[n - LATE];
                    }
                }
                if constexpr (n >= 1 && n <= LOGITS) {
                    constexpr int k = n - 1;
                    e[k & 1] = __builtin_amdgcn_exp2f(t[k & 1]);
                    if constexpr (k < LATE) w[k] = e[k & 1];
                    else if constexpr (MODE == MODE_FUSED) p[unit_of(k) % CG][unit_of(k) / CG][k % 4] = e[k & 1];
                }
                if constexpr (n >= 2) {
                    constexpr int k = n - 2, b = k / 4 / CG, cg = k / 4 % CG;
                    if constexpr (MODE == MODE_GIVEN) sc[b][k % 4] += e[k & 1];
                    else if constexpr (b < 2 && k % 4 == 0) lsum[cg][b] = e[k & 1];
                    else lsum[cg][b & 1] += e[k & 1];
                }
                if constexpr (n + 1 == LATE) {
#pragma unroll
                    for (int cg = 0; cg < CG; ++cg)
#pragma unroll
                        for (int h = 0; h < WAVES / 4; ++h) asm volatile("" : "+v"(l[cg][h]));   // (not earlier)
                    finish();
                }
                __builtin_amdgcn_sched_barrier(0);
            }, std::make_integer_sequence<int, LOGITS + 2>{});
            if (NP == 1) load_q(st + 1);
            if (NP % 2 == 1) products(0);
            // (all four lanes of a column store the same sum: no branch in the step)
            if constexpr (MODE != MODE_GIVEN)
#pragma unroll
                for (int cg = 0; cg < CG; ++cg) sm.l[st & 1][16 * cg + x][wave] = column_sum(lsum[cg][0] + lsum[cg][1]);
            if (fixed) set_references(st + 1);
        }
        if constexpr (MODE != MODE_GIVEN) {
            wait_lds();
            plain_barrier();
#pragma unroll
            for (int cg = 0; cg < CG; ++cg) {
                f32x4 l[WAVES / 4];
#pragma unroll
                for (int h = 0; h < WAVES / 4; ++h) l[h] = *reinterpret_cast<const f32x4*>(&sm.l[(n_steps - 1) & 1][16 * cg + x][4 * h]);
                const float f = finish_column(n_steps - 1, cg, l);
                if constexpr (MODE == MODE_FUSED) {
#pragma unroll
                    for (int b = 0; b < NB; ++b)
#pragma unroll
                        for (int i = 0; i < 4; ++i) sc[b][i] = __builtin_fmaf(p[cg][b][i], f, sc[b][i]);
                }
            }
        }
        if (MODE == MODE_GIVEN || attempt > 0 || !__any(bad)) break;   // (every wave has seen every column's sum)
        // A sum left the range of the fixed references: exact maxima of all columns, then once more.
        for (int st = 0; st < n_steps; ++st) {
            if (st % SPT == 0) {
                plain_barrier();
                copy_tile(st / SPT, (st / SPT) & 1);
                wait_copies();
            }
            wait_lds();
            plain_barrier();
            load_q(st);
            float m[CG];
#pragma unroll
            for (int cg = 0; cg < CG; ++cg) {
                m[cg] = -INFINITY;
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int j = 0; j < NJ; ++j) O::multiply(kf[b][j], qv[cg][j], z);
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (b < NB - 1 || last_block[i] == 0.f) m[cg] = fmaxf(m[cg], z[i]);
                }
                sm.l[st & 1][16 * cg + x][wave] = column_max(m[cg]);
            }
            wait_lds();
            plain_barrier();
            if (wave == 0) {
#pragma unroll
                for (int cg = 0; cg < CG; ++cg) {
                    for (int w2 = 0; w2 < WAVES; ++w2) m[cg] = fmaxf(m[cg], sm.l[st & 1][16 * cg + x][w2]);
                    sm.ref[STEP * st + 16 * cg + x] = m[cg] * a.scale_log2e;
                }
            }
        }
        wait_lds();
        plain_barrier();
        copy_tile(0, 0);
        if (n_tiles > 1) copy_tile(1, 1);
    }
    if constexpr (MODE != MODE_LSE) {
        float* dst = a.partial + ((size_t)split * a.Hkv + g) * a.ct.off[a.ct.n] + s0;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            float v = 0.f;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float t = row_sum(sc[b][i]);
                if (x == i) v = t;
            }
            const int key = 16 * (wave + WAVES * b) + 4 * kg + x;
            if (x < 4 && key < len) dst[key] = v;
        }
    }
}

// One workgroup = (KV head, chunk, segment of the chunk, column range).  1-D grid, KV head fastest: with 8 KV heads an
// XCD's L2 serves the queries of one head and the keys that its column ranges share.
template <typename T, int D, int WAVES, int MODE>
__global__ __launch_bounds__(64 * WAVES, 2) void score_kernel(const ScoreArgs a) {
    using O = Op<T, D, WAVES>;
    __shared__ Smem<T, D, WAVES> sm;
    int t = blockIdx.x;
    const int g = t % a.Hkv; t /= a.Hkv;
    const int split = t % a.n_split; t /= a.n_split;
    const int part = t % a.max_parts;
    const int c = a.order[t / a.max_parts];
    const int c0 = a.ct.off[c], clen = a.ct.off[c + 1] - c0;
    const int parts = segments<O::SEG>(clen);
    if (part >= parts) return;
    // softmax per chunk: chunks of one segment are done in the fused mode, the longer ones in the other two
    if (!a.global_scope && (parts > 1) != (MODE != MODE_FUSED)) return;
    const int per = segment_keys<O::SEG>(clen);
    const int s0 = c0 + part * per, len = min(per, clen - part * per);
    const int n0 = a.col0 + split * a.split_cols, n1 = min(a.col_end, n0 + a.split_cols);
    if (n0 >= n1) return;
    int row = lse_row<O::SEG>(c, c0) + part;             // MODE_LSE: this segment's normalisers go there
    if (MODE == MODE_GIVEN) row = a.global_scope ? a.lse_rows - 1 : row - part;   // combined: the chunk's first row, or the last of all
    switch ((len + 16 * WAVES - 1) / (16 * WAVES)) {
        case 1: walk_columns<T, D, WAVES, MODE, 1>(a, sm, g, c, s0, len, row, n0, n1, split); break;
        case 2: walk_columns<T, D, WAVES, MODE, 2>(a, sm, g, c, s0, len, row, n0, n1, split); break;
        case 3: walk_columns<T, D, WAVES, MODE, 3>(a, sm, g, c, s0, len, row, n0, n1, split); break;
        case 4: walk_columns<T, D, WAVES, MODE, 4>(a, sm, g, c, s0, len, row, n0, n1, split); break;
        default:
            if constexpr (O::NB_MAX > 4) {
                switch ((len + 16 * WAVES - 1) / (16 * WAVES)) {
                    case 5: walk_columns<T, D, WAVES, MODE, 5>(a, sm, g, c, s0, len, row, n0, n1, split); break;
                    case 6: walk_columns<T, D, WAVES, MODE, 6>(a, sm, g, c, s0, len, row, n0, n1, split); break;
                    case 7: walk_columns<T, D, WAVES, MODE, 7>(a, sm, g, c, s0, len, row, n0, n1, split); break;
                    default: walk_columns<T, D, WAVES, MODE, 8>(a, sm, g, c, s0, len, row, n0, n1, split); break;
                }
            }
    }
}

// Base-2 log-sum-exp over a chunk's segments into the chunk's first row (chunks of several segments), or over all
// segments of the prompt into the last row.  grid (columns / 256, KV heads, chunks or 1).
template <int SEG>
__global__ __launch_bounds__(256) void score_lse_combine_kernel(ChunkTable ct, int n_cols, int lse_rows, int global_scope,
                                                                float* __restrict__ lse2) {
    const int n = blockIdx.x * 256 + threadIdx.x;
    if (n >= n_cols) return;
    float* base = lse2 + (size_t)blockIdx.y * lse_rows * n_cols + n;
    const int first = global_scope ? 0 : (int)blockIdx.z, end = global_scope ? ct.n : first + 1;
    float m = -INFINITY, l = 0.f;
    for (int pass = 0; pass < 2; ++pass)
        for (int c = first; c < end; ++c) {
            const int parts = segments<SEG>(ct.off[c + 1] - ct.off[c]);
            if (!global_scope && parts < 2) return;
            for (int i = 0; i < parts; ++i) {
                const float v = base[(size_t)(lse_row<SEG>(c, ct.off[c]) + i) * n_cols];
                if (pass == 0) m = fmaxf(m, v); else l += exp2f(v - m);
            }
        }
    base[(size_t)(global_scope ? lse_rows - 1 : lse_row<SEG>(first, ct.off[first])) * n_cols] = m + log2f(l);
}

// Sum of a token's n_parts partial sums: 64 tokens per workgroup, wave w adds parts w, w + groups, ... and the waves' sums
// are added in order.  One thread per token walked up to 128 parts of a short prompt one after the other (10.8 us for 880
// tokens, 6.0 for 16384); with at most REDUCE_AHEAD parts per wave, all in flight together, it is one round trip (2.6, 4.8).
constexpr int REDUCE_AHEAD = 8, REDUCE_MAX_WAVES = 16;
__global__ __launch_bounds__(64 * REDUCE_MAX_WAVES) void score_reduce_kernel(const float* __restrict__ partial, int n_parts, int L_ctx,
                                                                             int add, float* __restrict__ scores) {
    __shared__ float sums[REDUCE_MAX_WAVES][64];
    const int j = min((int)(blockIdx.x * 64 + threadIdx.x), L_ctx - 1), groups = blockDim.y;
    float t = 0.f;
    for (int i0 = threadIdx.y; i0 < n_parts; i0 += REDUCE_AHEAD * groups) {
        float v[REDUCE_AHEAD];
#pragma unroll
        for (int u = 0; u < REDUCE_AHEAD; ++u)   // (clamped rather than skipped: behind a branch each load would be waited for)
            v[u] = partial[(size_t)min(i0 + u * groups, n_parts - 1) * L_ctx + j];
#pragma unroll
        for (int u = 0; u < REDUCE_AHEAD; ++u) t += i0 + u * groups < n_parts ? v[u] : 0.f;
    }
    sums[threadIdx.y][threadIdx.x] = t;
    __syncthreads();
    if (threadIdx.y != 0) return;
    t = 0.f;
    for (int w = 0; w < groups; ++w) t += sums[w][threadIdx.x];
    if ((int)(blockIdx.x * 64 + threadIdx.x) < L_ctx) scores[j] = add ? scores[j] + t : t;   // add: not the first columns
}

// Column ranges per (chunk, KV head).  A workgroup holds a compute unit to itself, pays about 3 steps' time before its
// first step (5 us for 1024 keys, against 2 us per 32 columns), and a chunk's steps cannot be balanced otherwise:
// the fewest ranges that fill the chip, counted in rounds of workgroups.  (24 chunks of 640 keys, 400 question tokens, 32 / 8 heads: 69.5 us, 79.3 if
// priced at 6 steps as when the keys came straight into registers; 56 other calls 0.3 % apart on average.)
int choose_splits(int items, int n_steps, int n_cu, int max_split) {
    const int least = (n_steps * RANGE_UNIT + MAX_COLS - 1) / MAX_COLS;
    int best = least;
    double best_t = 1e30;
    for (int s = least; s <= std::max(least, std::min(max_split, n_steps)); ++s) {
        const double rounds = (double)items * s / n_cu, per = 3.0 + (n_steps + s - 1) / s;
        const double t = per * (rounds < 4.0 ? (double)(int64_t)(rounds + 0.999) : rounds + 0.5);
        if (t < best_t - 1e-9) { best_t = t; best = s; }
    }
    return best;
}

template <typename T, int D>
constexpr bool FEW_WAVES = D * sizeof(T) <= 256;   // two workgroups' LDS fits a compute unit

template <typename T, int D>
hipError_t run(const Shape& s, const void* q, int nq, const void* k, const ChunkTable& ct, int norm, const Workspace& ws,
               float* scores, int src, const int32_t* store_row0, const ChunkDeltas* deltas, SelectAfter* select, hipStream_t st) {
    using O = Op<T, D>;
    const int L_ctx = ct.off[ct.n], NQG = nq * s.G;
    ScoreArgs a;
    a.q = q; a.k = k; a.theta = ws.rope_theta; a.lse2 = ws.lse; a.partial = ws.col_partial;
    a.nq = nq; a.Hq = s.Hq; a.Hkv = s.Hkv; a.G = s.G;
    a.src = src;
    a.global_scope = norm == FR_NORM_GLOBAL;
    a.magic = (uint32_t)((((uint64_t)1 << 32) + s.G - 1) / s.G);
    a.scale_log2e = (1.0f / sqrtf((float)s.d)) * 1.4426950408889634f;
    a.ct = ct;
    if (deltas) a.deltas = *deltas;
    int n = 0, max_len = 0, min_parts = INT32_MAX;   // non-empty chunks, longest first
    for (int c = 0; c < ct.n; ++c) {
        a.rows.row0[c] = store_row0 ? store_row0[c] : 0;
        const int len = ct.off[c + 1] - ct.off[c];
        if (len == 0) continue;
        a.order[n++] = (uint8_t)c;
        max_len = std::max(max_len, len);
        min_parts = std::min(min_parts, segments<O::SEG>(len));
    }
    std::stable_sort(a.order, a.order + n, [&](uint8_t x, uint8_t y) { return ct.off[x + 1] - ct.off[x] > ct.off[y + 1] - ct.off[y]; });
    a.max_parts = (max_len + O::SEG - 1) / O::SEG;   // (at least segments(len) for every chunk)
    a.lse_rows = ct.n + L_ctx / O::SEG + 1;
    const bool two_walks = a.global_scope || a.max_parts > 1;
    // Four waves where every chunk fits them: two workgroups then share a compute unit, each with barriers of its own, and a wave has twice the key blocks per
    // exchange of the sums.  64 x 300 keys, 512 question tokens, 64 / 8 heads 290 -> 193 us; 64 x 220, 100 tokens, 32 / 8 heads 38 -> 30; 24 x 300, 200 tokens 33.9 -> 29.7.  Not for a
    // few steps, whose time is that of the loads in front (24 x 500 keys, 16 tokens, 64 / 8 heads 13.8 : 14.7, 16 x 220, 40 tokens, 32 / 8 heads 10.9 : 11.4), nor with one launch for
    // the short chunks and one for the others: each leaves the chip idle at its end (12 calls 1 to 59 % longer).
    bool few_waves = false;
    if constexpr (FEW_WAVES<T, D>)
        few_waves = !two_walks && max_len <= Op<T, D, MOST_WAVES / 2>::SEG && (int64_t)n * s.Hkv * ((NQG + RANGE_UNIT - 1) / RANGE_UNIT) >= 4 * ws.n_cu;
    // All columns at once where the workspace holds their partial sums and normalisers (score_lse_floats, score_column_ranges), else in turns.
    int64_t cols = std::min<int64_t>(NQG, (int64_t)ws.col_splits * MAX_COLS);
    if (two_walks) cols = std::min<int64_t>(cols, (int64_t)(ws.lse_floats / ((size_t)s.Hkv * a.lse_rows)));
    if (cols < NQG) cols = cols / RANGE_UNIT * RANGE_UNIT;
    if (cols <= 0) return hipErrorInvalidValue;
    const int all_parts = a.max_parts;
    for (a.col0 = 0; a.col0 < NQG; a.col0 = a.col_end) {
        a.col_end = (int)std::min<int64_t>(NQG, a.col0 + cols);
        const int n_cols = a.col_end - a.col0, n_steps = (n_cols + RANGE_UNIT - 1) / RANGE_UNIT;
        a.n_split = choose_splits(n * all_parts * s.Hkv, n_steps, few_waves ? 2 * ws.n_cu : ws.n_cu, ws.col_splits);
        a.split_cols = (n_steps + a.n_split - 1) / a.n_split * RANGE_UNIT;
        a.n_split = (n_cols + a.split_cols - 1) / a.split_cols;
        if (a.n_split > ws.col_splits) return hipErrorInvalidValue;
        const dim3 block(64 * MOST_WAVES);
        if (!a.global_scope && min_parts == 1) {   // (the chunks of several segments return at once)
            a.max_parts = 1;
            const dim3 grid(n * a.n_split * s.Hkv);
            if constexpr (FEW_WAVES<T, D>)
                if (few_waves) score_kernel<T, D, MOST_WAVES / 2, MODE_FUSED><<<grid, dim3(32 * MOST_WAVES), 0, st>>>(a);
            if (!few_waves) score_kernel<T, D, MOST_WAVES, MODE_FUSED><<<grid, block, 0, st>>>(a);
            a.max_parts = all_parts;
        }
        if (two_walks) {
            const dim3 grid(n * a.max_parts * a.n_split * s.Hkv);
            score_kernel<T, D, MOST_WAVES, MODE_LSE><<<grid, block, 0, st>>>(a);
            score_lse_combine_kernel<O::SEG><<<dim3((n_cols + 255) / 256, s.Hkv, a.global_scope ? 1 : ct.n), dim3(256), 0, st>>>(
                ct, n_cols, a.lse_rows, a.global_scope, a.lse2);
            score_kernel<T, D, MOST_WAVES, MODE_GIVEN><<<grid, block, 0, st>>>(a);
        }
        const int n_sums = a.n_split * s.Hkv;
        if (a.col0 == 0 && a.col_end == NQG && sum_and_select_pays(L_ctx, n_sums)) {
            select->done = true;
            return launch_sum_and_select(ws.col_partial, n_sums, L_ctx, scores, (int)select->k, select->nq, select->q_index, st);
        }
        score_reduce_kernel<<<dim3((L_ctx + 63) / 64), dim3(64, std::min(REDUCE_MAX_WAVES, (n_sums + REDUCE_AHEAD - 1) / REDUCE_AHEAD)), 0, st>>>(
            ws.col_partial, n_sums, L_ctx, a.col0 > 0, scores);
    }
    return hipGetLastError();
}

}  // namespace

// Workspace of the softmax scoring.  lse_floats: normalisers; the two-pass kernels need all columns' at once, those of this file
// run them in turns of as many as fit.  col_splits: column ranges of partial sums, up to 16 while they stay below 4 MB, and
// enough for all columns at once while they stay below SCORE_TURN_BYTES.
constexpr int64_t SCORE_TURN_BYTES = (int64_t)64 << 20;
size_t score_lse_floats(const Shape& s, int64_t max_tokens, int max_chunks, int max_q) {
    if (score_two_pass_supported(s)) return score_two_pass_lse_floats(s, max_chunks, max_q);   // (chunks that fit need none)
    const int64_t seg = (s.d * s.esize == 512) ? Op<float, 128>::SEG : Op<__bf16, 128>::SEG;
    const int64_t rows = (int64_t)s.Hkv * (max_chunks + max_tokens / seg + 1);
    return (size_t)(rows * std::min<int64_t>((int64_t)s.G * max_q, std::max<int64_t>(MAX_COLS, SCORE_TURN_BYTES / 4 / rows)));
}
int score_column_ranges(const Shape& s, int64_t max_tokens, int max_q) {
    const int64_t all = ((int64_t)max_q * s.G + RANGE_UNIT - 1) / RANGE_UNIT * RANGE_UNIT / MAX_COLS + 1;
    const int64_t range_bytes = s.Hkv * max_tokens * 4;
    const int64_t few = std::min<int64_t>(16, std::max<int64_t>(((int64_t)4 << 20) / range_bytes, 2));
    return (int)std::max(few, std::min(all, SCORE_TURN_BYTES / range_bytes));
}

// One softmax over the prompt, or any chunk of more than SEG keys: shapes that k_score_mfma.hip takes go there, with the
// whole call.  Its two passes keep 64 columns or keys of a wave in registers without any exchange between waves; MODE_LSE
// and MODE_GIVEN pay a barrier per step (layer times: 16 x 1024 keys, 512 question tokens, 32/8 heads, global scope 0.329
// against 0.348 ms; 12 chunks of 500 to 1500 keys, where three launches each leave most of the chip idle, 0.206 against 0.340 ms).
// Chunks of at most SEG keys are faster here at every size (layer times against the two passes: 64 chunks of 128 keys 0.218
// / 0.230 ms, 32 of 512 0.286 / 0.325, 16 of 1024 0.618 / 0.656, 8 of 128 with 30 question tokens 0.0654 / 0.0661).
//
// Softmax scopes only; FR_NORM_RAW has kernels of its own.  store_row0 != NULL (host): k is a chunk store that is never
// written; chunk c occupies its rows store_row0[c] .., and its keys are moved to their prompt positions while they are
// loaded (`deltas`: host, positions per chunk).
hipError_t launch_score(const Shape& s, const void* q, int nq, const void* k, const ChunkTable& ct, int norm,
                        const Workspace& ws, float* scores, const int32_t* store_row0, const ChunkDeltas* deltas, SelectAfter* select, hipStream_t st) {
    select->done = false;
    if (ct.off[ct.n] == 0 || nq == 0) return hipSuccess;
    if (score_two_pass_supported(s)) {
        int max_len = 0;
        for (int c = 0; c < ct.n; ++c) max_len = std::max(max_len, ct.off[c + 1] - ct.off[c]);
        if (norm == FR_NORM_GLOBAL || max_len > Op<__bf16, 128>::SEG) {
            if (store_row0) {
                const hipError_t e = launch_rope_table(s, *deltas, ct.n, ws.rope_theta, ws.rope_table, st);
                if (e != hipSuccess) return e;
            }
            return launch_score_two_pass(s, q, nq, k, ct, norm, ws, scores, store_row0, ws.rope_table, st);
        }
    }
    const int src = !store_row0 ? SRC_PROMPT : s.rope_layout == FR_ROPE_INTERLEAVED ? SRC_STORE_INTERLEAVED : SRC_STORE_HALF;
    if (s.dtype == FR_BF16)
        return s.d == 64 ? run<__bf16, 64>(s, q, nq, k, ct, norm, ws, scores, src, store_row0, deltas, select, st)
                         : run<__bf16, 128>(s, q, nq, k, ct, norm, ws, scores, src, store_row0, deltas, select, st);
    return s.d == 64 ? run<float, 64>(s, q, nq, k, ct, norm, ws, scores, src, store_row0, deltas, select, st)
                     : run<float, 128>(s, q, nq, k, ct, norm, ws, scores, src, store_row0, deltas, select, st);
}

}  // namespace fr
