// Sparse prefill attention (eq. 9, Sec. 4.3) with fp32 products on the matrix cores: fp32 contexts, and bf16 contexts with
// more query heads per KV head than the tiled kernel takes.
//
// One workgroup = one KV head x 16 query columns ((row, query head) pairs, the heads of the group fastest), its waves deal
// the key blocks of 16 among themselves (wave w takes blocks w, w + W, ...), each with a running softmax of its own, and are
// merged through LDS once at the end.  The shapes served here are small (verification runs of a few hundred tokens), so what
// bounds the kernel is latency: with one wave per column tile the chip would hold a few dozen waves that walk dozens of
// blocks each; dealt to eight waves every wave has four or five.  S^T = K Q^T and O^T = V^T P^T with
// v_mfma_f32_16x16x4_f32: keys on the register dimension of S^T, columns on lanes, and register i of the weights is
// exactly the B operand of step i of the second product (its contraction index kg is key 4 kg + i), so the weights never
// leave their registers.  Fresh rows are found through a position -> row map in LDS, built by the workgroup itself.
// A weight of 0 does not take a NaN or an infinity out of a matrix product, so what a column does not see is kept out by hand:
// keys behind the tile's last row (they may be stale or hold nothing) repeat that one, and a block that only some of the columns
// see whole is searched for values that are not finite.
// A block's product is formed from zero and added to the running sum with one rounding: onto the running sum the product rounds that several
// times a block, which the longer chains of eight waves had made 1 to 3 % worse against float64 than 16 (head_dim 64: 1.652e-7 with 16
// waves, 1.670e-7 with eight, now 1.610e-7 at 109 of 544 positions; 1 % of the call).
// 4 heads, head_dim 64, us a call, keys and values straight into fragment registers : through LDS: 42 rows of 272 positions 9.3 : 7.9, 109 of 544 13.2 : 11.3, 310 of 800
// 17.3 : 14.9, 768 of 1280 25.4 : 21.2; bf16, 80 heads over one KV head, 172 of 920 46 : 31; with copies of a block past the end, which the waves then wait for, 8.3, 11.6, 15.1,
// 21.5, 32, and few keys slower than from registers: 1 row of 36 positions 4.5 : 4.3 (4.8), 12 of 40, 8 / 2 heads of 128, 8.4 : 8.1 (8.9).  A round of eight blocks takes about a microsecond of the matrix pipes, on as
// many compute units as there are column tiles.  Four waves are slower, 16 waves too (11.1 and 15.2 where eight took 9.0 and 12.9).
#include "fr_internal.hpp"

#include <algorithm>
#include <type_traits>

namespace fr {

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;
constexpr float NEG_BIG = -1.0e30f;
constexpr int MAP_MAX_L = 8192;   // positions whose map fits LDS beside the rest (16-bit row numbers: 16 KB)

template <typename T>
__device__ __forceinline__ f32x4 load4(const T* p) {
    struct alignas(4 * sizeof(T)) V { T v[4]; };
    const V t = *reinterpret_cast<const V*>(p);
    return f32x4{Elem<T>::to_f32(t.v[0]), Elem<T>::to_f32(t.v[1]), Elem<T>::to_f32(t.v[2]), Elem<T>::to_f32(t.v[3])};
}
__device__ __forceinline__ float column_max(float v) { v = fmaxf(v, __shfl_xor(v, 16)); return fmaxf(v, __shfl_xor(v, 32)); }
__device__ __forceinline__ float column_sum(float v) { v += __shfl_xor(v, 16); return v + __shfl_xor(v, 32); }

template <typename T, int D, int W>
__global__ __launch_bounds__(64 * W) void attn_f32_kernel(const T* __restrict__ q_rows, const int32_t* __restrict__ q_index, int R,
                                                          const T* __restrict__ k_cache, const T* __restrict__ v_cache, int L,
                                                          const T* __restrict__ k_new, const T* __restrict__ v_new,
                                                          const int32_t* __restrict__ inv, T* __restrict__ out,
                                                          float* __restrict__ lse, int Hq, int Hkv, int n_tiles, float scale_log2e) {
    constexpr int NJ = D / 16, PITCH = D + 4;
    constexpr int RB = D * (int)sizeof(T), RV = RB / 16, COPIES = 16 * RB / 1024, RC = 1024 / RB;   // bytes of a head row, its 16-byte vectors; copies of a block of 16, rows of a copy
    struct Blocks { unsigned char k[W][16 * RB], v[W][16 * RB]; };
    struct Merge { float o[W][16][PITCH]; };
    __shared__ __attribute__((aligned(1024))) unsigned char smem[sizeof(Blocks) > sizeof(Merge) ? sizeof(Blocks) : sizeof(Merge)];
    Blocks& blocks = *reinterpret_cast<Blocks*>(smem);
    auto& o_lds = reinterpret_cast<Merge*>(smem)->o;
    __shared__ float m_lds[W][16], l_lds[W][16];
    __shared__ uint16_t row_of[MAP_MAX_L];   // fresh row + 1 of a position, 0 = none (only where `inv` is not given)
    const int tid = threadIdx.x, lane = tid & 63, x = lane & 15, kg = lane >> 4, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = blockIdx.x % Hkv, tile = n_tiles - 1 - blockIdx.x / Hkv;   // longest tiles first
    const int G = Hq / Hkv, cols = R * G;
    const int n = min(16 * tile + x, cols - 1), r = n / G, head = g * G + n % G;   // columns past the end: a copy of the last
    f32x4 qv[NJ];   // dims 16 j + 4 kg + e of this lane's column
#pragma unroll
    for (int j = 0; j < NJ; ++j) qv[j] = load4(q_rows + ((size_t)r * Hq + head) * D + 16 * j + 4 * kg);
    const int pos = q_index[r];
    const int p_max = q_index[min(16 * tile + 15, cols - 1) / G];   // rows ascend
    const int p_last = max(min(p_max, L - 1), 0), n_blocks = p_last / 16 + 1;   // (in bounds whatever the Q index holds)
    const int p_first = q_index[16 * tile / G];   // keys up to here are visible to every column of the tile

    const bool have_new = k_new != nullptr, own_map = have_new && inv == nullptr;
    if (own_map) {   // rows up to the tile's last one, the others' positions are not visible
        for (int j = tid; j < 16 * n_blocks; j += 64 * W) row_of[j] = 0;
        __syncthreads();
        const int last = min(16 * tile + 15, cols - 1) / G;
        for (int i = tid; i <= last; i += 64 * W) {
            const int p = q_index[i];
            if (p >= 0 && p < 16 * n_blocks) row_of[p] = (uint16_t)(i + 1);
        }
        __syncthreads();
    }
    // A wave's block of 16 keys, and of their values, in LDS: copied global -> LDS (no registers, no wait) while the wave works on the one before, rows side by side: a
    // fragment's 16 rows x 64 bytes per instruction, neighbouring lanes in different rows, take the vector cache four times the accesses.
    // Vector c of key row r sits in place c ^ swz(r): the 16 rows of a fragment read meet in no bank.
    const int q = lane / RV, vec = lane % RV;
    auto swz = [](int r) { return RB == 128 ? (r >> 1) & 7 : r & 15; };
    auto lds_address = [](const void* p) { return __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) const unsigned char*)p); };
    auto dma = [](const unsigned char* src, uint32_t dst) { asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(src), "s"(dst) : "memory"); };
    auto wait_but = [](auto n) {   // until all but the wave's last n copies have landed
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0x0f70 | decltype(n)::value);
        asm volatile("" ::: "memory");
    };
    const uint32_t k_lds = lds_address(blocks.k[wave]), v_lds = lds_address(blocks.v[wave]);
    size_t source[COPIES];   // byte offset of the lane's rows of the block on its way
    bool fresh[COPIES];
    auto locate = [&](int b) {
        int f[COPIES];   // fresh rows
        auto key = [&](int i) { return min(16 * b + RC * i + q, p_last); };   // keys behind the tile's last row repeat that one
        if (own_map) {
#pragma unroll
            for (int i = 0; i < COPIES; ++i) f[i] = (int)row_of[key(i)] - 1;
        } else if (have_new) {
#pragma unroll
            for (int i = 0; i < COPIES; ++i) f[i] = inv[key(i)];
#pragma unroll
            for (int i = 0; i < COPIES; ++i) asm volatile("" : "+v"(f[i]));   // (waited for here: behind the branch the other calls would wait for their values' copies)
        } else {
#pragma unroll
            for (int i = 0; i < COPIES; ++i) f[i] = -1;
        }
#pragma unroll
        for (int i = 0; i < COPIES; ++i) {
            fresh[i] = f[i] >= 0;
            source[i] = ((size_t)(fresh[i] ? f[i] : key(i)) * Hkv + g) * RB;
        }
    };
    auto copy_k = [&] {   // of the block that has been located
#pragma unroll
        for (int i = 0; i < COPIES; ++i)
            dma(reinterpret_cast<const unsigned char*>(fresh[i] ? k_new : k_cache) + source[i] + 16 * (vec ^ swz(RC * i + q)), k_lds + 1024 * i);
    };
    auto copy_v = [&] {   // of the same block
#pragma unroll
        for (int i = 0; i < COPIES; ++i) dma(reinterpret_cast<const unsigned char*>(fresh[i] ? v_new : v_cache) + source[i] + 16 * vec, v_lds + 1024 * i);
    };

    f32x4 o[NJ];    // O^T: row m of product md is dim NJ m + md, so a lane's values of a key are neighbours in memory; o[md][i]: m = 4 kg + i
#pragma unroll
    for (int md = 0; md < NJ; ++md) o[md] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m = NEG_BIG, l = 0.f;
    wait_but(std::integral_constant<int, 0>{});   // (nothing that the compiler counts is in flight from here on)
    if (wave < n_blocks) {
        locate(wave);
        copy_k();
        copy_v();
    }
    for (int b = wave; b < n_blocks; b += W) {
        // (nothing is copied past the end: of few keys a wave has a block or two, and would wait for one more)
        const bool more = b + W < n_blocks;
        wait_but(std::integral_constant<int, COPIES>{});
        f32x4 kv[NJ], vv[4][NJ / 4];   // key 16 b + x, dims 16 j + 4 kg + e; values of keys 4 kg + i, dims NJ x ..
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const int at = (16 * j + 4 * kg) * (int)sizeof(T);
            kv[j] = load4(reinterpret_cast<const T*>(blocks.k[wave] + x * RB + ((at / 16) ^ swz(x)) * 16 + at % 16));
        }
        auto value = [&](int i, int md) -> float { return vv[i][md >> 2][md & 3]; };
        f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < NJ; ++j) {   // two chains
            s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(kv[j][0], qv[j][0], s0, 0, 0, 0);
            s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(kv[j][1], qv[j][1], s1, 0, 0, 0);
            s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(kv[j][2], qv[j][2], s0, 0, 0, 0);
            s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(kv[j][3], qv[j][3], s1, 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        locate(min(b + W, n_blocks - 1));
        f32x4 s = s0 + s1;
        float mx = NEG_BIG;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (16 * b + 4 * kg + i > pos) s[i] = -INFINITY;
            mx = fmaxf(mx, s[i] * scale_log2e);
        }
        const float m_new = fmaxf(m, column_max(mx)), alpha = __builtin_amdgcn_exp2f(m - m_new);
        m = m_new;
        float p[4], psum = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            p[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[i], scale_log2e, -m_new));
            psum += p[i];
        }
        l = l * alpha + psum;
        float scale_o = alpha;
        if (more) {
            copy_k();
            wait_but(std::integral_constant<int, COPIES>{});
        } else {
            wait_but(std::integral_constant<int, 0>{});
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int h = 0; h < NJ / 4; ++h) vv[i][h] = load4(reinterpret_cast<const T*>(blocks.v[wave] + (4 * kg + i) * RB) + NJ * x + 4 * h);
        if (16 * b + 15 > p_first) {   // values that are not finite: out of the product, into the columns that see them
            float z = 0.f;   // NaN if one of them is not finite
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int md = 0; md < NJ; ++md) z = __builtin_fmaf(value(i, md), 0.f, z);
            const bool odd = !(z == 0.f);
            if (__builtin_expect(__any(odd), 0)) {
#pragma unroll
                for (int md = 0; md < NJ; ++md) o[md] *= alpha;
                scale_o = 1.f;
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int md = 0; md < NJ; ++md) {
                        const bool finite = fabsf(value(i, md)) < INFINITY;
                        const float apart = finite ? 0.f : value(i, md);
                        if (!finite) vv[i][md >> 2][md & 3] = 0.f;
                        for (int src = 0; src < 4; ++src) {   // key 4 src + i of the block
                            const bool seen = 16 * b + 4 * src + i <= pos;
                            const float weight = __shfl(p[i], 16 * src + x);
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                const float v = __shfl(apart, 16 * src + 4 * kg + e);   // row 4 kg + e of the product
                                if (seen && v != 0.f) o[md][e] += weight * v;
                            }
                        }
                    }
            }
        }
        f32x4 pv[NJ];   // of this block alone: added to o with one rounding, so the number of blocks a wave walks counts for little
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int md = 0; md < NJ; ++md)
                pv[md] = __builtin_amdgcn_mfma_f32_16x16x4f32(value(i, md), p[i], i == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : pv[md], 0, 0, 0);
#pragma unroll
        for (int md = 0; md < NJ; ++md)
#pragma unroll
            for (int e = 0; e < 4; ++e) o[md][e] = __builtin_fmaf(o[md][e], scale_o, pv[md][e]);
        __builtin_amdgcn_sched_barrier(0);
        if (more) copy_v();
    }
    __syncthreads();   // everyone is done with the copies
    // ---- merge the waves ---------------------------------------------------------------------------------------------
    l = column_sum(l);
    if (kg == 0) { m_lds[wave][x] = m; l_lds[wave][x] = l; }
    __syncthreads();
    float M = NEG_BIG;
    for (int w = 0; w < W; ++w) M = fmaxf(M, m_lds[w][x]);
    const float f = __builtin_amdgcn_exp2f(m - M);   // (a wave without a visible key: m = NEG_BIG, factor 0)
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int h = 0; h < NJ / 4; ++h)
            *reinterpret_cast<f32x4*>(&o_lds[wave][x][NJ * (4 * kg + i) + 4 * h]) = f32x4{o[4 * h][i], o[4 * h + 1][i], o[4 * h + 2][i], o[4 * h + 3][i]} * f;
    __syncthreads();
    for (int i = tid; i < 16 * D; i += 64 * W) {
        const int c = i / D, e = i % D, nc = 16 * tile + c;
        if (nc >= cols) continue;
        float mc = NEG_BIG, lc = 0.f, v = 0.f;
        for (int w = 0; w < W; ++w) mc = fmaxf(mc, m_lds[w][c]);
        for (int w = 0; w < W; ++w) {
            lc += l_lds[w][c] * __builtin_amdgcn_exp2f(m_lds[w][c] - mc);
            v += o_lds[w][c][e];
        }
        const size_t oc = (size_t)(nc / G) * Hq + g * G + nc % G;
        out[oc * D + e] = Elem<T>::from_f32(v / lc);
        if (e == 0 && lse != nullptr) lse[oc] = (mc + __builtin_amdgcn_logf(lc)) * 0.6931471805599453f;
    }
}

// inv[j] = row r of k_new / v_new that holds the recomputed entry of position j, else -1: prompts whose map does not fit LDS.
__global__ __launch_bounds__(256) void inv_index_kernel(const int32_t* __restrict__ q_index, int R, int64_t L, int32_t* __restrict__ inv) {
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= L) return;
    int lo = 0, hi = R;   // first r with q_index[r] >= j
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (q_index[mid] < j) lo = mid + 1; else hi = mid;
    }
    inv[j] = (lo < R && q_index[lo] == j) ? lo : -1;
}

}  // namespace

// `inv`: device scratch of L ints.
hipError_t launch_attn_f32(const Shape& s, const void* q_rows, const int32_t* q_index, int R, const void* k_cache,
                           const void* v_cache, int64_t L, const void* k_new, const void* v_new, int32_t* inv, void* out,
                           float* lse, hipStream_t st) {
    if (R == 0) return hipSuccess;
    if (k_new == nullptr || L <= MAP_MAX_L)
        inv = nullptr;
    else
        inv_index_kernel<<<dim3((unsigned)((L + 255) / 256)), dim3(256), 0, st>>>(q_index, R, L, inv);
    const int n_tiles = (int)(((int64_t)R * s.G + 15) / 16);
    const dim3 grid((unsigned)(n_tiles * s.Hkv));
    const float scale_log2e = (1.0f / sqrtf((float)s.d)) * 1.4426950408889634f;
#define FR_ATTN_LAUNCH(T, D, W)                                                                                             \
    attn_f32_kernel<T, D, W><<<grid, dim3(64 * W), 0, st>>>((const T*)q_rows, q_index, R, (const T*)k_cache, (const T*)v_cache, \
                                                            (int)L, (const T*)k_new, (const T*)v_new, inv, (T*)out, lse, s.Hq, \
                                                            s.Hkv, n_tiles, scale_log2e)
    if (s.dtype == FR_BF16) {
        if (s.d == 64) FR_ATTN_LAUNCH(__bf16, 64, 8); else FR_ATTN_LAUNCH(__bf16, 128, 8);
    } else {
        if (s.d == 64) FR_ATTN_LAUNCH(float, 64, 8); else FR_ATTN_LAUNCH(float, 128, 8);
    }
#undef FR_ATTN_LAUNCH
    return hipGetLastError();
}

}  // namespace fr
