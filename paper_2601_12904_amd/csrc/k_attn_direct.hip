// Sparse prefill attention (eq. 9, Sec. 4.3) of short prompts on the gfx950 matrix cores: bf16, head_dim 64 or 128, up to 64 query
// heads per KV head; keys and values come straight from the cache and the fresh rows, in one launch.
//
// What bounds a short prompt is latency, not work: the tiled path (k_attn_mfma.hip) packs its images, walks a handful of tiles with eight
// waves in step and adds up the parts of its items, three dependent launches of which the middle one spends most of its time on
// prologue, exchange and epilogue.  Here one workgroup = one KV head x 16 NC query columns ((row, query head) pairs, the heads of the
// group fastest), whose eight waves deal the blocks of 32 keys among themselves, each with accumulators of its own, and are merged
// through LDS once at the end: nothing in the loop waits for another wave.
//
// S^T = K Q^T and O^T = V^T P^T with v_mfma_f32_16x16x32_bf16, keys on the register dimension of S^T and columns on lanes: the
// accumulators of two 16-key blocks are, after conversion, the B operand of the second product, as in the tiled kernel.  Row m of value product md is
// dim D / 16 m + md, so that a lane needs 16 (8) neighbouring bytes of each of its eight value rows and transposes them itself with byte
// permutes, and holds neighbouring dims of the output.  Weights as in the tiled kernel: bf16 where the shape has an instance of its own
// there, else (SPLIT) as the sum of three bf16 numbers, together the 24 bits of the fp32 weight.
//
// A wave copies its block global -> LDS (no registers, no wait) while it works on the one before.  Not straight into fragment registers: a
// fragment wants 16 rows x 64 bytes per instruction with neighbouring lanes in different rows, which the vector cache serves at 16 bytes
// a cycle (40 accesses per KB measured over keys and values, 16 with rows side by side): 45 rows of 920 positions 13.6 us, through LDS 9.4.
//
// us a call, three launches : this kernel.  32 / 8 heads, head_dim 128: 54 rows of 272 positions 19.8 : 7.0, 84 of 450 22.4 : 7.5, 172 of 920
// 26.0 : 13.5, 244 of 1300 29.2 : 16.0, 167 of 3400 37.7 : 27.0; 28 / 4 heads: 172 of 920 31.4 : 15.3; 16 / 8 heads, head_dim 64: 172 of 920 21.7 : 7.6.
// A round of eight blocks takes 1.1 us with 16 columns, 1.5 with 32 (issue of the vector instructions: addresses, softmax, permutes).
//
// Softmax.  As in the tiled kernel the exponent reference of a column is the maximum over its visible ones of keys 0..31; wave 0 passes it on before the
// first weights.  Weights that leave it far behind raise the wave's own reference by a whole number and scale its sums by that power of two, so
// a weight has the same bits (and its rounding the same error) as in the tiled kernel.
//
// What a column does not see stays out of it by hand, as a weight of 0 does not take a NaN or an infinity out of a product: keys behind the
// tile's last row (they may be stale or hold nothing) repeat that one, and values that are not finite leave a block that only some
// columns see whole and reach those columns when the loop is over.
#include "fr_internal.hpp"

#include <hip/hip_ext.h>

#include <algorithm>

namespace fr {

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(4))) int32_t i32x4;
typedef __attribute__((ext_vector_type(2))) uint16_t u16x2;
constexpr float NEG_BIG = -1.0e30f;
constexpr float LARGE = 1024.f;   // a lane's weights of a block: beyond it the reference goes up
constexpr int W = 8;              // waves per workgroup
constexpr int MAP_MAX_L = 6144;   // positions whose map fits LDS beside the rest

struct DirectArgs {
    const __bf16* q_rows;
    const int32_t* q_index;
    const __bf16 *k_cache, *v_cache, *k_new, *v_new;
    __bf16* out;
    float* lse;
    int R, L, Hq, Hkv, G, n_tiles, writeback;
    uint32_t magic;           // ceil(2^32 / G): n / G = mulhi(n, magic) for G > 1
    float scale_log2e;
};

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

// The two bf16 numbers of a word, 0 in the place of one that is not finite.
__device__ __forceinline__ uint32_t finite_or_zero(uint32_t w) {
    if ((w & 0x00007F80u) == 0x00007F80u) w &= 0xFFFF0000u;
    if ((w & 0x7F800000u) == 0x7F800000u) w &= 0x0000FFFFu;
    return w;
}

template <int D, int NC>
struct DirectLds {
    static constexpr int PITCH = D + 4;
    static constexpr int TILE = 32 * D * 2;   // bytes of a block of 32 keys or values
    int32_t source[MAP_MAX_L + 32];           // where position j is read: byte offset of its head row, + FRESH in the fresh rows
    float ref[16 * NC];                       // the columns' exponent references
    union {
        struct { unsigned char k[W][TILE], v[W][TILE]; };
        struct {
            float o[W][16 * NC][PITCH];
            float m[16 * NC][W], l[16 * NC][W];
        };
    };
};
constexpr uint32_t FRESH = 0x80000000u;

__device__ __forceinline__ uint32_t lds_address(const void* p) {
    return __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) const unsigned char*)p);
}
// 16 bytes per lane, global -> LDS (lane i at lds_dst + 16 i), no registers involved.  Completion: the issuing wave's vmcnt.
__device__ __forceinline__ void dma(const unsigned char* src, uint32_t lds_dst) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(src), "s"(lds_dst) : "memory");
}
template <int N>
__device__ __forceinline__ void wait_dma_but() {   // until all but the wave's last N copies have landed
    static_assert(N < 16, "one field of the counter");
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0f70 | N);
    asm volatile("" ::: "memory");
}

__device__ __forceinline__ void wave_barrier() {   // without the fences of __syncthreads(), which would wait for the copies
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

template <int D, bool SPLIT, int NC>
__global__ __launch_bounds__(64 * W) void attn_direct_kernel(const DirectArgs a) {
    constexpr int NJ = D / 16, NK = D / 32, VW = D / 32;   // dims per lane of a value row, matrix steps of a logit, words of a lane's values
    constexpr int PARTS = SPLIT ? 3 : 1;
    using Lds = DirectLds<D, NC>;
    typedef __attribute__((ext_vector_type(VW))) uint32_t VVec;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    Lds& sm = *reinterpret_cast<Lds*>(smem_raw);
    const int tid = threadIdx.x, lane = tid & 63, x = lane & 15, kg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = blockIdx.x % a.Hkv, tile = a.n_tiles - 1 - blockIdx.x / a.Hkv;   // longest tiles first
    const int G = a.G, cols = a.R * G, col0 = 16 * NC * tile;
    auto row_of_column = [&](int n) { return G > 1 ? (int)__umulhi((uint32_t)n, a.magic) : n; };
    const int r_first = row_of_column(col0), r_last = row_of_column(min(col0 + 16 * NC, cols) - 1);
    const bool have_new = a.k_new != nullptr;

    bf16x8 qf[NC][NK];   // B operand of S^T = K Q^T
    int pos[NC];
#pragma unroll
    for (int nb = 0; nb < NC; ++nb) {   // columns past the end: a copy of the last
        const int n = min(col0 + 16 * nb + x, cols - 1), r = row_of_column(n);
        const __bf16* p = a.q_rows + ((size_t)r * a.Hq + g * G + (n - r * G)) * D + 8 * kg;
        pos[nb] = a.q_index[r];
#pragma unroll
        for (int ks = 0; ks < NK; ++ks) qf[nb][ks] = *reinterpret_cast<const bf16x8*>(p + 32 * ks);
    }
    const int p_first = a.q_index[r_first];   // rows ascend: keys up to here are visible to every column
    const int p_last = max(min(a.q_index[r_last], a.L - 1), 0), n_blocks = p_last / 32 + 1;   // (in bounds whatever the Q index holds)
    // Where each key is read.  Keys behind the tile's last row repeat that one (they may be stale or hold nothing).
    const uint32_t row_bytes = (uint32_t)(a.Hkv * D * 2), head_bytes = (uint32_t)(g * D * 2);
    auto source_of = [&](int row) { return (uint32_t)row * row_bytes + head_bytes; };
    for (int j = tid; j < 32 * n_blocks; j += 64 * W)
        sm.source[j] = (int32_t)(j <= p_last ? source_of(j) : have_new ? source_of(r_last) | FRESH : source_of(p_last));
    __syncthreads();
    if (have_new) {   // rows up to the tile's last one, the others' positions are not visible
        for (int i = tid; i <= r_last; i += 64 * W) {
            const int p = a.q_index[i];
            if (p >= 0 && p <= p_last) sm.source[p] = (int32_t)(source_of(i) | FRESH);
        }
        __syncthreads();
    }
    // (the fresh rows' base takes FRESH off again)
    auto address = [&](uint32_t source, const __bf16* cache, const __bf16* fresh) -> const unsigned char* {
        return reinterpret_cast<const unsigned char*>((int32_t)source < 0 ? reinterpret_cast<uintptr_t>(fresh) - FRESH : reinterpret_cast<uintptr_t>(cache)) + source;
    };
    // A wave's block of 32 keys, and of their values, in LDS.  A copy brings 64 / RV rows, RV lanes side by side to a row; copy i the rows COPIES q + i of
    // the lanes' groups q, so that a lane's sources are neighbours.  Vector c of key row r sits in place c ^ swz(r), so that the 16 rows of a fragment read
    // meet in no bank.
    constexpr int RV = D / 8, COPIES = 32 * RV / 64;
    auto swz = [](int r) { return D == 128 ? r & 15 : (r & 3) | (r >> 1 & 4); };
    auto row_at = [](int r) { return 1024 * (r % COPIES) + 16 * RV * (r / COPIES); };
    const uint32_t k_lds = lds_address(sm.k[wave]), v_lds = lds_address(sm.v[wave]);
    const int q = lane / RV, vec = lane % RV, k_place = 16 * (vec ^ swz(COPIES * q));   // swz(COPIES q + i) = swz(COPIES q) ^ swz(i)
    i32x4 source[COPIES / 4];   // of the block on its way
    auto copy_k = [&](int b) {
#pragma unroll
        for (int i = 0; i < COPIES / 4; ++i) source[i] = *reinterpret_cast<const i32x4*>(&sm.source[32 * b + COPIES * q + 4 * i]);
#pragma unroll
        for (int i = 0; i < COPIES; ++i)
            dma(address((uint32_t)source[i / 4][i % 4] + ((uint32_t)k_place ^ swz(i) * 16u), a.k_cache, a.k_new), k_lds + 1024 * i);
    };
    auto copy_v = [&] {   // of the same block
#pragma unroll
        for (int i = 0; i < COPIES; ++i) dma(address((uint32_t)source[i / 4][i % 4] + 16u * vec, a.v_cache, a.v_new), v_lds + 1024 * i);
    };
    f32x4 o[NJ][NC];   // O^T: row m of product md is dim NJ m + md
    float m[NC], l[NC];
#pragma unroll
    for (int nb = 0; nb < NC; ++nb) {
        m[nb] = NEG_BIG;   // (of a wave without a block)
        l[nb] = 0.f;
#pragma unroll
        for (int md = 0; md < NJ; ++md) o[md][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    wait_dma_but<0>();   // (nothing that the compiler counts is in flight from here on)
    copy_k(min(wave, n_blocks - 1));   // (past the last block: that one again, nobody uses it; the counts of the waits stay the same)
    copy_v();
    auto block_max = [&](const f32x4 (&s)[2][NC], int nb) {   // of a column's scaled logits
        float t = NEG_BIG;
#pragma unroll
        for (int bb = 0; bb < 2; ++bb)
#pragma unroll
            for (int v = 0; v < 4; ++v) t = fmaxf(t, s[bb][nb][v]);
        return column_max(t) * a.scale_log2e;
    };
    bool apart = false;
#pragma unroll 1
    for (int b = wave; b < n_blocks; b += W) {
        f32x4 s[2][NC];
        wait_dma_but<COPIES>();
        {
            bf16x8 kf[2][NK];   // keys 32 b + 16 bb + x: dims 32 ks + 8 kg ..
#pragma unroll
            for (int ks = 0; ks < NK; ++ks)
#pragma unroll
                for (int bb = 0; bb < 2; ++bb)
                    kf[bb][ks] = *reinterpret_cast<const bf16x8*>(sm.k[wave] + row_at(16 * bb + x) + 16 * ((4 * ks + kg) ^ swz(x)));
            // (the tiled kernel's order of the dims, which the query fragments' places give it: the same logits to the bit)
            constexpr int FIRST = D == 64 ? 0 : SPLIT ? 1 : 3;
#pragma unroll
            for (int j = 0; j < NK; ++j) {
                const int ks = j == 0 ? FIRST : j <= FIRST ? j - 1 : j;
#pragma unroll
                for (int bb = 0; bb < 2; ++bb)
#pragma unroll
                    for (int nb = 0; nb < NC; ++nb)
                        s[bb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[bb][ks], qf[nb][ks], j == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : s[bb][nb], 0, 0, 0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        copy_k(min(b + W, n_blocks - 1));
        const bool partial = 32 * b + 31 > p_first;   // not every column sees all of these keys
        if (partial) {
#pragma unroll
            for (int bb = 0; bb < 2; ++bb)
#pragma unroll
                for (int v = 0; v < 4; ++v)
#pragma unroll
                    for (int nb = 0; nb < NC; ++nb)
                        if (32 * b + 16 * bb + 4 * kg + v > pos[nb]) s[bb][nb][v] = -INFINITY;
        }
        if (b == wave) {   // the exponent references: maxima over the visible ones of keys 0..31, which wave 0 has now
            if (wave == 0) {
#pragma unroll
                for (int nb = 0; nb < NC; ++nb) sm.ref[16 * nb + x] = block_max(s, nb);
            }
            wave_barrier();
#pragma unroll
            for (int nb = 0; nb < NC; ++nb) m[nb] = sm.ref[16 * nb + x];
        }
        u32x4 p[PARTS][NC];   // weights as the B operand of the second product: slot 4 bb + v of quarter kg is key 16 bb + 4 kg + v
        float sum[NC];
#pragma unroll 1
        for (bool again = false;; again = true) {
            bool large = false;
#pragma unroll
            for (int nb = 0; nb < NC; ++nb) {
                sum[nb] = 0.f;
#pragma unroll
                for (int bb = 0; bb < 2; ++bb)
#pragma unroll
                    for (int v = 0; v < 4; v += 2) {
                        float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[bb][nb][v], a.scale_log2e, -m[nb]));
                        float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[bb][nb][v + 1], a.scale_log2e, -m[nb]));
                        sum[nb] += p0 + p1;
                        if constexpr (SPLIT) {   // three bf16 numbers that together are the fp32 weight
#pragma unroll
                            for (int u = 0; u < PARTS; ++u) {
                                p[u][nb][2 * bb + v / 2] = __builtin_amdgcn_perm(__float_as_uint(p1), __float_as_uint(p0), 0x07060302u);
                                p0 -= __uint_as_float(__float_as_uint(p0) & 0xFFFF0000u);
                                p1 -= __uint_as_float(__float_as_uint(p1) & 0xFFFF0000u);
                            }
                        } else {
                            bf16x2 t;
                            t[0] = (__bf16)p0;
                            t[1] = (__bf16)p1;
                            p[0][nb][2 * bb + v / 2] = __builtin_bit_cast(uint32_t, t);
                        }
                    }
                large = large || sum[nb] > LARGE;
            }
            if (again || !__any(large)) break;
#pragma unroll
            for (int nb = 0; nb < NC; ++nb) {   // by whole numbers: the weights keep their bits
                const float up = fmaxf(__builtin_ceilf(block_max(s, nb) - m[nb]), 0.f), down = __builtin_amdgcn_exp2f(-up);
                m[nb] += up;
                l[nb] *= down;
#pragma unroll
                for (int md = 0; md < NJ; ++md) o[md][nb] *= down;
            }
        }
#pragma unroll
        for (int nb = 0; nb < NC; ++nb) l[nb] += sum[nb];
        wait_dma_but<COPIES>();
        VVec vf[8];   // values of keys 32 b + 16 (i / 4) + 4 kg + i % 4, dims NJ x ..
#pragma unroll
        for (int i = 0; i < 8; ++i) vf[i] = *reinterpret_cast<const VVec*>(sm.v[wave] + row_at(16 * (i >> 2) + 4 * kg + (i & 3)) + 2 * NJ * x);
        if (partial) {
            u16x2 most = {0, 0};   // the largest exponent and mantissa
#pragma unroll
            for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int e = 0; e < VW; ++e) most = __builtin_elementwise_max(most, __builtin_bit_cast(u16x2, vf[i][e] & 0x7FFF7FFFu));
            if (__builtin_expect(__any(max(most[0], most[1]) >= 0x7F80), 0)) {   // values that are not finite: not into the product
                apart = true;
#pragma unroll
                for (int i = 0; i < 8; ++i)
#pragma unroll
                    for (int e = 0; e < VW; ++e) vf[i][e] = finite_or_zero(vf[i][e]);
            }
        }
#pragma unroll
        for (int md = 0; md < NJ; ++md) {
            u32x4 vt;   // dim NJ x + md of the eight keys
#pragma unroll
            for (int j = 0; j < 4; ++j)
                vt[j] = __builtin_amdgcn_perm(vf[2 * j + 1][md / 2], vf[2 * j][md / 2], md % 2 == 0 ? 0x05040100u : 0x07060302u);
#pragma unroll
            for (int u = 0; u < PARTS; ++u)
#pragma unroll
                for (int nb = 0; nb < NC; ++nb)
                    o[md][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vt), __builtin_bit_cast(bf16x8, p[u][nb]), o[md][nb], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        copy_v();
    }
    if (wave >= n_blocks) wave_barrier();   // (the references)
    if (__builtin_expect(apart, 0)) {   // the values that were left out reach the columns that see them
#pragma unroll 1
        for (int b = wave; b < n_blocks; b += W)
#pragma unroll 1
            for (int t = 0; t < 32; ++t) {
                if (32 * b + 31 <= p_first || 32 * b + t > p_last) continue;
                const uint16_t* key = reinterpret_cast<const uint16_t*>(address((uint32_t)sm.source[32 * b + t], a.v_cache, a.v_new));
#pragma unroll
                for (int v = 0; v < 4; ++v)
#pragma unroll
                    for (int md = 0; md < NJ; ++md) {
                        const uint32_t w = key[NJ * (4 * kg + v) + md];
                        const float add = (w & 0x7F80u) == 0x7F80u ? __uint_as_float(w << 16) : 0.f;
#pragma unroll
                        for (int nb = 0; nb < NC; ++nb) o[md][nb][v] += 32 * b + t <= pos[nb] ? add : 0.f;
                    }
            }
    }
    wait_dma_but<0>();
    __syncthreads();   // everyone is done with the copies
    // ---- merge the waves ---------------------------------------------------------------------------------------------
#pragma unroll
    for (int nb = 0; nb < NC; ++nb) {
        const float sum = column_sum(l[nb]);
        if (kg == 0) { sm.m[16 * nb + x][wave] = m[nb]; sm.l[16 * nb + x][wave] = sum; }
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int h = 0; h < NJ / 4; ++h)
                *reinterpret_cast<f32x4*>(&sm.o[wave][16 * nb + x][NJ * (4 * kg + v) + 4 * h]) =
                    f32x4{o[4 * h][nb][v], o[4 * h + 1][nb][v], o[4 * h + 2][nb][v], o[4 * h + 3][nb][v]};
    }
    __syncthreads();
    constexpr int NV = D / 8;
    for (int i = tid; i < 16 * NC * NV; i += 64 * W) {
        const int c = i / NV, vec = i % NV, n = col0 + c;
        if (n >= cols) break;
        float mw[W], lsum = 0.f, M = NEG_BIG;
#pragma unroll
        for (int w = 0; w < W; ++w) { mw[w] = sm.m[c][w]; M = fmaxf(M, mw[w]); }
        f32x4 lo = {0.f, 0.f, 0.f, 0.f}, hi = lo;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const float f = __builtin_amdgcn_exp2f(mw[w] - M);   // (a wave without a block: m = NEG_BIG, factor 0)
            lsum = __builtin_fmaf(sm.l[c][w], f, lsum);
            lo += *reinterpret_cast<const f32x4*>(&sm.o[w][c][8 * vec]) * f;
            hi += *reinterpret_cast<const f32x4*>(&sm.o[w][c][8 * vec + 4]) * f;
        }
        const float inv_l = 1.0f / lsum;
        struct alignas(16) { __bf16 v[8]; } y;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            y.v[e] = (__bf16)(lo[e] * inv_l);
            y.v[4 + e] = (__bf16)(hi[e] * inv_l);
        }
        const int r = row_of_column(n);
        const size_t oc = (size_t)r * a.Hq + g * G + (n - r * G);
        *reinterpret_cast<u32x4*>(a.out + oc * D + 8 * vec) = __builtin_bit_cast(u32x4, y);
        if (vec == 0 && a.lse != nullptr) a.lse[oc] = (M + __builtin_amdgcn_logf(lsum)) * 0.6931471805599453f;
    }
    if (a.writeback) {   // this tile's fresh rows (a position with a fresh row is never read from the cache)
        for (int i = tid; i < (r_last - r_first + 1) * NV; i += 64 * W) {
            const int r = r_first + i / NV, p = a.q_index[r];
            const size_t src = ((size_t)r * a.Hkv + g) * D + 8 * (i % NV), dst = ((size_t)p * a.Hkv + g) * D + 8 * (i % NV);
            if (p >= 0 && p < a.L) {
                *reinterpret_cast<u32x4*>(const_cast<__bf16*>(a.k_cache) + dst) = *reinterpret_cast<const u32x4*>(a.k_new + src);
                *reinterpret_cast<u32x4*>(const_cast<__bf16*>(a.v_cache) + dst) = *reinterpret_cast<const u32x4*>(a.v_new + src);
            }
        }
    }
}

template <int D, bool SPLIT, int NC>
hipError_t launch(const DirectArgs& args, KernelTimer* timer, hipStream_t st) {
    using Lds = DirectLds<D, NC>;
    static_assert(sizeof(Lds) <= 160 * 1024, "LDS of a compute unit");
    // Raises the kernel's dynamic LDS limit, once per process.
    static const hipError_t once = hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_direct_kernel<D, SPLIT, NC>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(Lds));
    if (once != hipSuccess) return once;
    DirectArgs a = args;
    a.n_tiles = (a.R * a.G + 16 * NC - 1) / (16 * NC);
    const dim3 grid((unsigned)(a.n_tiles * a.Hkv)), block(64 * W);
    if (timer != nullptr && timer->n_slots > 0) {
        const int slot = (int)(timer->n_recorded % timer->n_slots);
        hipExtLaunchKernelGGL((attn_direct_kernel<D, SPLIT, NC>), grid, block, (uint32_t)sizeof(Lds), st, timer->start[slot], timer->stop[slot], 0u, a);
        ++timer->n_recorded;
    } else {
        attn_direct_kernel<D, SPLIT, NC><<<grid, block, sizeof(Lds), st>>>(a);
    }
    return hipGetLastError();
}

}  // namespace

// 32-column tiles of a call, all KV heads.
static int64_t column_tiles(const Shape& s, int R) { return ((int64_t)R * s.G + 31) / 32 * s.Hkv; }

// Where one launch is faster than the tiled path: 300 calls of 272 to 6000 positions, five head layouts, rows spread over the prompt and rows at its end
// (all of them long).  As long as every compute unit has at most one workgroup it is at every length (tiled : here 42 : 30 us for 201 of 4096 rows,
// 44.3 : 36.3 for 200 at the end of 5000, 47.9 : 42.3 for 240 at the end of 6000, 32 / 8 heads); a second generation of workgroups pays while the walk is short, at head_dim
// 64, half the bytes and products per key, for longer: spread and at the end, 1.5 per unit of 1800 positions 34 : 22 and 33.8 : 32.1, of 2500 37 : 32
// and 38 : 41, of 3400 43 : 36 and 40 : 51; head_dim 64 of 4096 49 : 32 and 49.7 : 47.1; two per unit of 920 positions 29 : 19 and 28.4 : 22.1 (1.5).
bool attn_direct_pays(const Shape& s, int R, int64_t L, int n_cu) {
    if (s.dtype != FR_BF16 || s.G > 64 || L > MAP_MAX_L) return false;
    const int64_t most = L <= 1024 ? 2 * n_cu : L <= (s.d == 64 ? 4096 : 1792) ? 3 * n_cu / 2 : n_cu;
    return column_tiles(s, R) <= most;
}

hipError_t launch_attn_direct(const Shape& s, const void* q_rows, const int32_t* q_index, int R, const void* k_cache,
                              const void* v_cache, int64_t L, const void* k_new, const void* v_new, void* out, float* lse,
                              int n_cu, KernelTimer* timer, bool writeback, hipStream_t st) {
    if (R == 0) return hipSuccess;
    DirectArgs a;
    a.q_rows = (const __bf16*)q_rows; a.q_index = q_index;
    a.k_cache = (const __bf16*)k_cache; a.v_cache = (const __bf16*)v_cache;
    a.k_new = (const __bf16*)k_new; a.v_new = (const __bf16*)v_new;
    a.out = (__bf16*)out; a.lse = lse;
    a.R = R; a.L = (int)L; a.Hq = s.Hq; a.Hkv = s.Hkv; a.G = s.G; a.n_tiles = 0; a.writeback = writeback && k_new != nullptr;
    a.magic = (uint32_t)((((uint64_t)1 << 32) + s.G - 1) / s.G);
    a.scale_log2e = (1.0f / sqrtf((float)s.d)) * 1.4426950408889634f;
    const bool split = !(s.d == 128 && (s.G == 1 || s.G == 2 || s.G == 4 || s.G == 8));
    // 16 columns per workgroup while that leaves at most one workgroup per compute unit: 131 rows of 700 positions (262 workgroups) 10.4 : 11.0 us with 16
    // and 32 columns, 45 of 920 (90) 9.4 : 12.3, 184 at the end of 920 (368) 16.0 : 12.6.
    const bool narrow = 2 * column_tiles(s, R) <= n_cu;
    if (s.d == 64) return narrow ? launch<64, true, 1>(a, timer, st) : launch<64, true, 2>(a, timer, st);
    if (split) return narrow ? launch<128, true, 1>(a, timer, st) : launch<128, true, 2>(a, timer, st);
    return narrow ? launch<128, false, 1>(a, timer, st) : launch<128, false, 2>(a, timer, st);
}

}  // namespace fr
