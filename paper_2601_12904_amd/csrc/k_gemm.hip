// The model steps around the selective-prefill path for the recomputed rows (the per-layer work of the
// full-stack configuration): y = x W^T on the gfx950 matrix cores with fused epilogues, RMSNorm, and the
// rotary table of the rows' positions.
//
// GEMM.  out[M, N] = a[M, K] . w[N, K]^T, bf16 in, fp32 accumulate.  Both operands are K-contiguous, so the
// kernel computes the transposed tile C^T = W A^T with v_mfma_f32_32x32x16_bf16 (16 x 16 x 32 in the 256 x 256 kernel): output features run along the
// accumulator's register dimension and activation rows along lanes, which puts four consecutive features of one
// row into one lane -- rotary pairs and (gate, up) pairs are then combined without any lane exchange.
// Large launches run the 256 x 256 kernel further down; in the others
// one workgroup computes (64 WF) features x 128 rows with WF x 2 waves of 64 x 64 each: WF = 4 (8 waves, two per
// SIMD, so one wave's LDS reads and barriers hide behind the other's matrix instructions; 48 KB per K tile, ring
// of 3) where the feature count allows, else WF = 2 (4 waves, 32 KB per K tile, ring of 4).  K is walked in tiles
// of 64: both operand tiles (rows of 128 bytes) are copied straight into an LDS ring with direct-to-LDS loads
// (no staging registers); each lane chooses which 16-byte chunk of its row it fetches so that chunk c of row r
// lands at chunk position c ^ swz(r), swz(r) = (r ^ (r >> 3)) & 7: the 16-byte fragment reads (one lane per row)
// of any 16 consecutive rows then fall into 16 distinct bank groups.
#include "fr_internal.hpp"

#include <type_traits>

#include <algorithm>

namespace fr {

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

constexpr int BR = 128;   // activation rows per workgroup (MFMA N side)
constexpr int BK = 64;    // K elements per tile: 128 bytes per row
constexpr int EPI_PITCH = 64 + 4;                   // fp32 elements per row of a wave's epilogue staging

// Accumulators of a wave's 64 features x 64 rows, as 32 x 32 tiles [features + 32][rows + 32] or as 16 x 16 tiles.
typedef f32x16 Acc32[2][2];
typedef f32x4 Acc16[4][4];

enum { EPI_STORE = 0, EPI_RESIDUAL = 1, EPI_QKV_ROPE = 2, EPI_SWIGLU = 3 };

struct GemmArgs {
    const __bf16* a;        // [M, K]
    const __bf16* w;        // [N, K]
    int M, N, K;
    __bf16* out;            // EPI_STORE / EPI_RESIDUAL: [M, N];  EPI_SWIGLU: [M, N / 2]
    const __bf16* residual; // EPI_RESIDUAL: [M, N]
    // EPI_QKV_ROPE: features [0, Hq d) -> q_out[M, Hq, d] rotated, [Hq d, (Hq + Hkv) d) -> k_out rotated, rest -> v_out
    __bf16 *q_out, *k_out, *v_out;
    const float2* rope;     // [M][d / 2] (cos, sin) of each row's position
    int Hq, Hkv, d;
    // Tail split.  Tiles [0, n_whole) are computed by one workgroup each; every later tile by n_parts workgroups that
    // walk 1 / n_parts of K each and leave their fp32 accumulators in `partials` (gemm_fixup_kernel adds them and
    // runs the epilogue).  n_parts = 1: no tile is split.
    int n_whole, n_parts;
    float* partials;        // [(tile - n_whole) * n_parts + part][wave][64 registers][64 lanes]
    size_t partials_bytes;  // (host side: what the buffer holds)
};

template <int WF>
struct Tiling {
    typedef Acc32 Acc;
    static constexpr int NW = 2 * WF;                    // waves per workgroup
    static constexpr int BF = 64 * WF;                   // output features per workgroup (MFMA M side)
    static constexpr int BRT = BR;                       // and rows
    static constexpr int WAVE_TILES = NW;                // 64 x 64 pieces of the output tile
    // What a launch takes (plan_tiling): time per K tile of a full round, the share of it that a nearly empty round still
    // takes (a full round is held back by the chip's power limit), the same where that round is the launch's only one, its tiles whole or split,
    // launch, pipeline fill and epilogue, a split last round.
    // Chosen so that the better of the two tilings is taken, at first over 742 products (N 256 .. 28672, K 128 .. 14336, 1 .. 4096 rows).  With the 256 x 256
    // tiling's 16 x 16 x 32 instructions: over 352 products (32 row counts of 11 shapes) the choice is 0.3 % off the faster one on average, 18 % at worst (384 rows,
    // 28672 x 4096, 101 us in 256 x 128, 86 in 256 x 256); over 130 more, picked because estimates disagree there, 4.5 %, 37 % at worst (877 rows, 18944 x 4096,
    // 175 us, 128 in 256 x 256).  1100 rows of 4096 x 8192, 144 whole tiles of 256 x 128 or 80 of 256 x 256 in three parts: 82 and 88 us.
    static constexpr float US_PER_K_TILE = 0.9f, ROUND_BASE = 0.33f, ONLY_BASE = 0.24f, ONLY_BASE_SPLIT = 0.33f, US_LAUNCH = 8.0f, US_SPLIT = 6.0f;
    static __host__ __device__ constexpr int feature0(int v) { return 64 * (v % WF); }
    static __host__ __device__ constexpr int row_0(int v) { return 64 * (v / WF); }
    // feature tiles fastest, so that workgroups that share an activation tile are neighbours
    static __device__ __forceinline__ void origin(const GemmArgs& g, int tile, int& f0, int& r0) {
        const int n_f = (g.N + BF - 1) / BF;
        f0 = (tile % n_f) * BF;
        r0 = (tile / n_f) * BRT;
    }
    static constexpr int W_TILE_BYTES = BF * BK * 2;     // 16 or 32 KB
    static constexpr int A_TILE_BYTES = BR * BK * 2;     // 16 KB
    static constexpr int STAGE_BYTES = W_TILE_BYTES + A_TILE_BYTES;
    static constexpr int N_STAGE = (WF == 4) ? 3 : 4;
    static constexpr int W_ROUNDS = BF * 8 / (NW * 64);  // direct-to-LDS instructions per lane and W tile
    static constexpr int A_ROUNDS = BR * 8 / (NW * 64);
    static constexpr int LDS_BYTES = N_STAGE * STAGE_BYTES;
    static_assert(NW * 64 * EPI_PITCH * 4 <= LDS_BYTES, "epilogue staging must fit into the ring");
};

__device__ __forceinline__ int swz(int r) { return (r ^ (r >> 3)) & 7; }

// Copy one operand tile (rows of 128 bytes) into LDS.  Chunk u (16 bytes) of the tile sits at byte 16 u; every wave
// moves 1 KB per round.  The per-lane part of a copy's source address does not change from K tile to K tile (which
// row, which 16-byte chunk of its 128 bytes: `lane_off`, set up once by dma_offsets; rows past the end of the operand
// are clamped and never stored), the rest is the same for the whole workgroup and travels in scalar registers, as
// does the LDS address: a copy costs the vector ALU nothing.
// (The copies are written out rather than left to the builtin: with it the compiler takes the pending copy for an
// access that may complete out of order with the LDS reads, and waits for all outstanding fragment reads before
// every matrix instruction.)
template <int ROUNDS, int NW>
__device__ __forceinline__ void dma_offsets(int64_t ld, int row0, int rows, int wave, int lane, uint32_t (&lane_off)[ROUNDS]) {
#pragma unroll
    for (int j = 0; j < ROUNDS; ++j) {
        const int u = (j * NW + wave) * 64 + lane;
        const int r = u >> 3, cpos = u & 7;
        const int c = cpos ^ swz(r);
        // relative to the operand's row row0 and the current K tile; fits 32 bits: at most 256 rows of at most 2^22
        // elements (checked by the caller)
        lane_off[j] = (uint32_t)(((int64_t)(min(row0 + r, rows - 1) - row0) * ld + 8 * c) * 2);
    }
}
template <int ROUNDS, int NW>
__device__ __forceinline__ void dma_tile(const unsigned char* tile_src /* uniform: row row0, current K tile */,
                                         const uint32_t (&lane_off)[ROUNDS], uint32_t lds_tile /* uniform */, int wave_u) {
#pragma unroll
    for (int j = 0; j < ROUNDS; ++j) {
        const uint32_t l = lds_tile + (uint32_t)(j * NW + wave_u) * 1024u;
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(lane_off[j]), "s"(tile_src), "s"(l) : "memory");
    }
}

// Workgroup barrier without the fences of __syncthreads(): those make the compiler wait for *all* outstanding
// memory operations (vmcnt(0)), which would drain the direct-to-LDS copies and register prefetches that are meant
// to stay in flight across the barrier.  The callers wait by hand for exactly the copies the next phase needs; the
// empty asm statements keep the compiler from moving LDS accesses across the barrier.
__device__ __forceinline__ void barrier_keep_loads_in_flight() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

constexpr int PARTIAL_FLOATS_PER_WAVE = 64 * 64;
constexpr int MIN_K_TILES_PER_PART = 16;

// Epilogue shared by the kernels: this wave's fp32 64 x 64 tile goes through LDS ([row][feature]), then every lane
// handles 8 consecutive features of a row.  fw0 / rw0 = first feature / row of the wave's tile.
__device__ __forceinline__ void stage_tile(const Acc32& acc, float* ep, int lane) {   // -> [row][feature]
    const int x = lane & 31, h = lane >> 5;
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                f32x4 t;
#pragma unroll
                for (int e = 0; e < 4; ++e) t[e] = acc[mb][nb][4 * q4 + e];
                *reinterpret_cast<f32x4*>(&ep[(32 * nb + x) * EPI_PITCH + 32 * mb + 8 * q4 + 4 * h]) = t;
            }
}
__device__ __forceinline__ void stage_tile(const Acc16& acc, float* ep, int lane) {
    const int x = lane & 15, kg = lane >> 4;
#pragma unroll
    for (int fb = 0; fb < 4; ++fb)
#pragma unroll
        for (int rb = 0; rb < 4; ++rb)
            *reinterpret_cast<f32x4*>(&ep[(16 * rb + x) * EPI_PITCH + 16 * fb + 4 * kg]) = acc[fb][rb];
}
template <int EPI, class Acc>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs& g, const Acc& acc, unsigned char* smem, int wave, int lane,
                                              int fw0, int rw0) {
    // ---- epilogue: fp32 tile through LDS ([row][feature] per wave), then 8 consecutive features per lane ----
    __syncthreads();
    float* ep = reinterpret_cast<float*>(smem) + wave * 64 * EPI_PITCH;
    stage_tile(acc, ep, lane);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int rl = 8 * i + (lane >> 3), seg = lane & 7;     // local row, group of 8 features
        const int r = rw0 + rl;
        const int f = fw0 + 8 * seg;
        if (r >= g.M || f >= g.N) continue;
        float v[8];
        {
            const f32x4 lo = *reinterpret_cast<const f32x4*>(&ep[rl * EPI_PITCH + 8 * seg]);
            const f32x4 hi = *reinterpret_cast<const f32x4*>(&ep[rl * EPI_PITCH + 8 * seg + 4]);
#pragma unroll
            for (int e = 0; e < 4; ++e) { v[e] = lo[e]; v[4 + e] = hi[e]; }
        }
        if (EPI == EPI_STORE || EPI == EPI_RESIDUAL) {
            if (EPI == EPI_RESIDUAL) {
                const bf16x8 res = *reinterpret_cast<const bf16x8*>(g.residual + (int64_t)r * g.N + f);
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] += (float)res[e];
            }
            bf16x8 o;
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = (__bf16)v[e];
            *reinterpret_cast<bf16x8*>(g.out + (int64_t)r * g.N + f) = o;
        } else if (EPI == EPI_SWIGLU) {   // features interleaved (gate_j, up_j): out_j = silu(gate_j) * up_j
            bf16x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float gt = v[2 * e], up = v[2 * e + 1];
                o[e] = (__bf16)(gt / (1.0f + __expf(-gt)) * up);
            }
            *reinterpret_cast<bf16x4*>(g.out + (int64_t)r * (g.N / 2) + f / 2) = o;
        } else {                          // EPI_QKV_ROPE
            const int qf_end = g.Hq * g.d, kf_end = qf_end + g.Hkv * g.d;
            __bf16* dst;
            bool rotate = true;
            if (f < qf_end) dst = g.q_out + (int64_t)r * qf_end + f;
            else if (f < kf_end) dst = g.k_out + (int64_t)r * (g.Hkv * g.d) + (f - qf_end);
            else { dst = g.v_out + (int64_t)r * (g.Hkv * g.d) + (f - kf_end); rotate = false; }
            if (rotate) {
                const int p0 = (f % g.d) >> 1;   // first rotary pair of this group (interleaved pairs)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float2 cs = g.rope[(int64_t)r * (g.d / 2) + p0 + e];
                    const float a = v[2 * e], b = v[2 * e + 1];
                    v[2 * e] = a * cs.x - b * cs.y;
                    v[2 * e + 1] = b * cs.x + a * cs.y;
                }
            }
            bf16x8 o;
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = (__bf16)v[e];
            *reinterpret_cast<bf16x8*>(dst) = o;
        }
    }
}

template <int EPI, int WF>
__global__ __launch_bounds__(128 * WF) void gemm_bf16_kernel(GemmArgs g) {
    using TL = Tiling<WF>;
    constexpr int NW = TL::NW, STAGE_BYTES = TL::STAGE_BYTES, N_STAGE = TL::N_STAGE;
    constexpr int DMA_PER_TILE = TL::W_ROUNDS + TL::A_ROUNDS;   // outstanding copies per lane and K tile
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, x = lane & 31, h = lane >> 5;
    const int wf = wave % WF, wr = wave / WF;          // wave position: features x rows
    int tile = (int)blockIdx.x, part = 0;
    if (tile >= g.n_whole) {
        const int j = tile - g.n_whole;
        tile = g.n_whole + j / g.n_parts;
        part = j % g.n_parts;
    }
    const bool split_tile = (int)blockIdx.x >= g.n_whole && g.n_parts > 1;
    int f0, r0;
    TL::origin(g, tile, f0, r0);
    const int n_kt_all = g.K / BK;
    const int kt_begin = split_tile ? (int)((int64_t)n_kt_all * part / g.n_parts) : 0;
    const int kt_end = split_tile ? (int)((int64_t)n_kt_all * (part + 1) / g.n_parts) : n_kt_all;
    const int n_kt = kt_end - kt_begin;   // K tiles of this workgroup: kt below counts from kt_begin

    // fragment byte offsets inside a tile: row (32 blk + x) of this wave's half, k step ks -> chunk (2 ks + h)
    int frag[4][2];   // [ks][blk & 1]
    {
        const int keyx = (x ^ (x >> 3)) & 7;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
            for (int par = 0; par < 2; ++par) frag[ks][par] = x * 128 + (((2 * ks + h) ^ keyx ^ (4 * par)) << 4);
    }
    f32x16 acc[2][2];
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[mb][nb][v] = 0.f;

    uint32_t w_off[TL::W_ROUNDS], a_off[TL::A_ROUNDS];
    dma_offsets<TL::W_ROUNDS, NW>(g.K, f0, g.N, wave, lane, w_off);
    dma_offsets<TL::A_ROUNDS, NW>(g.K, r0, g.M, wave, lane, a_off);
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem);
    const unsigned char* w_row0 = reinterpret_cast<const unsigned char*>(g.w + (int64_t)f0 * g.K);
    const unsigned char* a_row0 = reinterpret_cast<const unsigned char*>(g.a + (int64_t)r0 * g.K);
    auto issue = [&](int kt) {
        const uint32_t st = lds0 + (uint32_t)(kt % N_STAGE) * STAGE_BYTES;
        const int64_t k_bytes = (int64_t)(kt_begin + kt) * BK * 2;
        dma_tile<TL::W_ROUNDS, NW>(w_row0 + k_bytes, w_off, st, wave_u);
        dma_tile<TL::A_ROUNDS, NW>(a_row0 + k_bytes, a_off, st + TL::W_TILE_BYTES, wave_u);
    };
#pragma unroll
    for (int p = 0; p < N_STAGE - 1; ++p)
        if (p < n_kt) issue(p);

    // One K tile.  The ring slot is a compile-time constant (the loop below is unrolled by the ring's length) and the
    // LDS address of every fragment read sits in a register of its own, set up once (the ring is larger than the 64 KB
    // an instruction's offset field reaches, and the compiler, left to itself, adds the slot's offset before every
    // read): no address arithmetic between the matrix instructions.
    uint32_t rd_w[N_STAGE][4][2], rd_a[N_STAGE][4][2];   // [slot][k step][row block parity]
    {
        const uint32_t lds_v = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
#pragma unroll
        for (int sl = 0; sl < N_STAGE; ++sl)
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                for (int par = 0; par < 2; ++par) {
                    rd_w[sl][ks][par] = lds_v + sl * STAGE_BYTES + (64 * wf) * 128 + frag[ks][par];
                    rd_a[sl][ks][par] = lds_v + sl * STAGE_BYTES + TL::W_TILE_BYTES + (64 * wr) * 128 + frag[ks][par];
                    asm volatile("" : "+v"(rd_w[sl][ks][par]), "+v"(rd_a[sl][ks][par]));   // keep them: no re-derivation in the loop
                }
    }
    auto step = [&](auto slot_c, int kt) {
        constexpr int slot = decltype(slot_c)::value;
        // own copies of tile kt are the oldest outstanding: wait until at most the (N_STAGE - 2) newer tiles remain
        if (kt + N_STAGE - 2 < n_kt) {
            constexpr int newer = DMA_PER_TILE * (N_STAGE - 2);
            __builtin_amdgcn_s_waitcnt(0x0f70 | (newer & 15) | ((newer >> 4) << 14));
        } else {
            __builtin_amdgcn_s_waitcnt(0x0f70);
        }
        barrier_keep_loads_in_flight();   // tile kt complete and visible; everyone is done with tile kt-1, whose stage is refilled next
        // fragments of K step ks + 1 are requested before the matrix instructions of step ks are issued
        typedef const bf16x8 __attribute__((address_space(3))) * lds_frag_ptr;
        bf16x8 wfrag[2][2], afrag[2][2];
        auto request = [&](int ks, int buf) {
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                wfrag[buf][b] = *reinterpret_cast<lds_frag_ptr>((uintptr_t)(rd_w[slot][ks][b] + b * (32 * 128)));
                afrag[buf][b] = *reinterpret_cast<lds_frag_ptr>((uintptr_t)(rd_a[slot][ks][b] + b * (32 * 128)));
            }
        };
        request(0, 0);
        // the refill of the freed stage is issued behind the first fragment requests: its issue time passes while they
        // are on their way, instead of in front of them
        if (kt + N_STAGE - 1 < n_kt) issue(kt + N_STAGE - 1);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            if (ks + 1 < 4) request(ks + 1, (ks + 1) & 1);
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                for (int nb = 0; nb < 2; ++nb)
                    acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wfrag[ks & 1][mb], afrag[ks & 1][nb], acc[mb][nb], 0, 0, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);   // LDS reads of step 0
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            if (ks + 1 < 4) __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);   // matrix
        }
    };
    using S0 = std::integral_constant<int, 0>;
    using S1 = std::integral_constant<int, 1>;
    using S2 = std::integral_constant<int, 2>;
    using S3 = std::integral_constant<int, 3>;
    int kt = 0;
    for (; kt + N_STAGE <= n_kt; kt += N_STAGE) {
        step(S0{}, kt);
        step(S1{}, kt + 1);
        step(S2{}, kt + 2);
        if constexpr (N_STAGE == 4) step(S3{}, kt + 3);
    }
    if (kt < n_kt) step(S0{}, kt);
    if (kt + 1 < n_kt) step(S1{}, kt + 1);
    if constexpr (N_STAGE == 4) {
        if (kt + 2 < n_kt) step(S2{}, kt + 2);
    }

    if (split_tile) {   // leave the partial sums: register-major, one coalesced 256-byte line per wave and register
        float* dst = g.partials + ((size_t)(((int)blockIdx.x - g.n_whole) * NW + wave)) * PARTIAL_FLOATS_PER_WAVE + lane;
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
            for (int nb = 0; nb < 2; ++nb)
#pragma unroll
                for (int v = 0; v < 16; ++v) dst[((2 * mb + nb) * 16 + v) * 64] = acc[mb][nb][v];
        return;
    }
    gemm_epilogue<EPI>(g, acc, smem, wave, lane, f0 + 64 * wf, r0 + 64 * wr);
}

// The 256 x 256 kernel: eight waves (two per SIMD) of 128 features x 64 rows, K tiles of 64 in two stages of LDS.
//
// What bounds the 256 x 128 kernel is the vector-memory path that feeds the ring (48 KB per K tile and 16 matrix
// instructions of a wave; 64 KB per 32 here), and the fragment reads, one per matrix instruction (24 per 32 here).
// The eight waves run as two groups half a phase apart: while one wave of a SIMD multiplies (16 matrix instructions, a
// quarter of its tile, at raised priority), the other one reads fragments and issues copies; a barrier separates any
// two half phases.  Per K tile and wave (w = its 4 blocks of 32 features, a = its 2 blocks of 32 rows):
//
//   phase   reads for this phase and the next ones    copies of tile k + 2    products
//     0     a0, first half of w2                       w0, w1                  (w0, w1) x a0
//     1     a1, second half of w2                      a0                      (w0, w1) x a1
//     2     w3; first quarter of the next w0, w1       a1                      (w2, w3) x a1
//     3     the rest of the next w0, w1                w2, w3                  (w2, w3) x a0
//
// Six reads (one in 16 cycles) per phase of 256 cycles of the matrix pipe.  A stage consists of four 16 KB pieces (w0 w1
// of all waves, w2 w3, a0, a1).  A wave waits for its own reads before the barrier that ends its half phase, so a piece is
// free one phase after it was last read, which is when its copy for tile k + 2 goes out; that copy is waited for (by
// count, never to zero before the last two tiles) five to seven phases later, at the end of the phase in front of its
// first read.
// At 4096 rows of the gate / up projection (N = 28672, K = 4096) with 32 x 32 x 16 matrix instructions: 882 -> 707 us, 1360 TFLOP/s on
// normally distributed operands, 1830 on zeros (1054 before): with real data the chip's power limit is the bound, no longer the schedule.
// Hence 16 x 16 x 32 instructions, which touch their accumulators half as often (1.98 instead of 1.78 PFLOP/s from registers alone), each sharing an
// operand with its neighbours: 712 -> 656 us, 1467 TFLOP/s; 2970 rows: gate / up 550 -> 512, down 275 -> 257, O 89 -> 84, Q / K / V 142 -> 131 us.
// Waiting only for the reads that the coming products need, with the copies one phase later: no difference.
struct Tiling256 {
    typedef Acc16 Acc;
    static constexpr int NW = 8;
    static constexpr int BF = 256, BRT = 256;
    // Chunk c of row r of a piece lies at c ^ swz16(r): the 16 rows of a fragment, chunks 4 ks .. 4 ks + 3 by quarters of the wave, fall
    // into 16 different 16-byte bank groups whether the LDS serves lanes 0 .. 15 together or 0 .. 3, 12 .. 15 and 20 .. 27.
    static __host__ __device__ constexpr int swz16(int r) { return ((r >> 1) & 1) | ((r >> 3) & 1) << 1 | (((r >> 2) ^ (r >> 3)) & 1) << 2; }
    static constexpr int PIECE = 128 * BK * 2;             // 16 KB
    static constexpr int STAGE = 4 * PIECE;                // [w0 w1][w2 w3][a0][a1]
    static constexpr int WAVE_TILES = 16;                  // 64 x 64 pieces of the output tile, two per wave
    static constexpr int LDS_BYTES = NW * 64 * EPI_PITCH * 4;
    static constexpr float US_PER_K_TILE = 1.47f, ROUND_BASE = 0.30f, ONLY_BASE = 0.20f, ONLY_BASE_SPLIT = 0.15f, US_LAUNCH = 9.5f, US_SPLIT = 17.0f;   // see Tiling
    static_assert(2 * STAGE <= LDS_BYTES, "the epilogue staging is the larger one");
    static __host__ __device__ constexpr int feature0(int v) { return 128 * (v >> 3) + 64 * (v & 1); }   // v = 2 wave + half
    static __host__ __device__ constexpr int row_0(int v) { return 64 * ((v >> 1) & 3); }
    static __device__ __forceinline__ void origin(const GemmArgs& g, int tile, int& f0, int& r0) {
        // rows fastest inside groups of 8 row tiles: the 32 workgroups of an XCD walk about 8 x 4 tiles, so its L2 takes 12
        // operand slices instead of up to 35 (gate / up, 2970 rows: 567 -> 551 us; the other projections unchanged)
        constexpr int GR = 8;
        const int n_f = (g.N + BF - 1) / BF, n_r = (g.M + BRT - 1) / BRT;
        const int grp = tile / (GR * n_f), in = tile % (GR * n_f), gr = min(GR, n_r - grp * GR);
        f0 = in / gr * BF;
        r0 = (grp * GR + in % gr) * BRT;
    }
};

template <int EPI>
__global__ __launch_bounds__(512) void gemm_bf16_256_kernel(GemmArgs g) {
    using TL = Tiling256;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, x = lane & 15, kg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wf = wave >> 2, wr = wave & 3;           // 2 x 4 waves; waves w and w + 4 share a SIMD
    int tile = (int)blockIdx.x, part = 0;
    const bool split_tile = tile >= g.n_whole && g.n_parts > 1;
    if (split_tile) {
        const int j = tile - g.n_whole;
        tile = g.n_whole + j / g.n_parts;
        part = j % g.n_parts;
    } else {   // workgroups go to the XCDs in turn: XCD x takes the x-th run of whole tiles
        const int q = g.n_whole >> 3, extra = g.n_whole & 7, xcd = tile & 7;
        tile = xcd * q + min(xcd, extra) + (tile >> 3);
    }
    int f0, r0;
    TL::origin(g, tile, f0, r0);
    const int n_kt_all = g.K / BK;
    const int kt_begin = split_tile ? (int)((int64_t)n_kt_all * part / g.n_parts) : 0;
    const int kt_end = split_tile ? (int)((int64_t)n_kt_all * (part + 1) / g.n_parts) : n_kt_all;
    const int n_kt = kt_end - kt_begin;

    // Copies: 16-byte chunk u of a piece lies at byte 16 u; row r of a w piece is feature 128 (r / 64) + r % 64 of the
    // tile (+ 64 in the second one), row r of an a piece is row 64 (r / 32) + r % 32 (+ 32).  Rows past the end are
    // clamped and never stored.
    uint32_t w_off[2], a_off[2][2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int u = (j * TL::NW + wave) * 64 + lane;
        const int r = u >> 3, c = (u & 7) ^ TL::swz16(r);
        w_off[j] = (uint32_t)(((int64_t)(128 * (r >> 6) + (r & 63)) * g.K + 8 * c) * 2);
#pragma unroll
        for (int hf = 0; hf < 2; ++hf)
            a_off[hf][j] = (uint32_t)(((int64_t)(min(r0 + 64 * (r >> 5) + (r & 31) + 32 * hf, g.M - 1) - r0) * g.K + 8 * c) * 2);
    }
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem);
    const unsigned char* w_src = reinterpret_cast<const unsigned char*>(g.w + (int64_t)f0 * g.K + (int64_t)kt_begin * BK);
    const unsigned char* a_src = reinterpret_cast<const unsigned char*>(g.a + (int64_t)r0 * g.K + (int64_t)kt_begin * BK);
    const int64_t w_half = (int64_t)64 * g.K * 2;
    enum { W01 = 0, W23 = 1, A0 = 2, A1 = 3 };
    auto copy = [&](auto piece_c, int kt) {
        constexpr int piece = decltype(piece_c)::value;
        const uint32_t dst = lds0 + (uint32_t)(kt & 1) * TL::STAGE + piece * TL::PIECE;
        const int64_t k_bytes = (int64_t)kt * BK * 2;
        if constexpr (piece == W01) dma_tile<2, TL::NW>(w_src + k_bytes, w_off, dst, wave);
        if constexpr (piece == W23) dma_tile<2, TL::NW>(w_src + w_half + k_bytes, w_off, dst, wave);
        if constexpr (piece == A0) dma_tile<2, TL::NW>(a_src + k_bytes, a_off[0], dst, wave);
        if constexpr (piece == A1) dma_tile<2, TL::NW>(a_src + k_bytes, a_off[1], dst, wave);
    };
    using CW01 = std::integral_constant<int, W01>;
    using CW23 = std::integral_constant<int, W23>;
    using CA0 = std::integral_constant<int, A0>;
    using CA1 = std::integral_constant<int, A1>;

    // Fragment reads: row 64 wf + 16 b + x of a w piece (b = 0 .. 3), row 32 wr + 16 b + x of an a piece (b = 0, 1); k step ks -> chunk
    // (4 ks + kg) ^ swz16(row).  Block i >> 1 of a 32-row group, k step i & 1: the four fragments of a group are i = 0 .. 3.
    typedef const bf16x8 __attribute__((address_space(3))) * lds_frag_ptr;
    uint32_t rd_w[2], rd_a[2];
    {
        const uint32_t lds_v = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            rd_w[ks] = lds_v + (64 * wf + x) * 128 + (((4 * ks + kg) ^ TL::swz16(x)) << 4);
            rd_a[ks] = lds_v + A0 * TL::PIECE + (32 * wr + x) * 128 + (((4 * ks + kg) ^ TL::swz16(x)) << 4);
        }
    }
    // (the other stage is reached by adding its offset with one vector instruction per address and tile: it lies beyond the
    // 64 KB of an instruction's offset field)
    int stage_step = TL::STAGE;
    auto frag_w = [&](int blk, int i) {   // (indexed from a pointer: the constants go into the instructions' offsets)
        return reinterpret_cast<lds_frag_ptr>((uintptr_t)rd_w[i & 1])[((blk >> 1) * TL::PIECE + (32 * (blk & 1) + 16 * (i >> 1)) * 128) / 16];
    };
    auto frag_a = [&](int hf, int i) { return reinterpret_cast<lds_frag_ptr>((uintptr_t)rd_a[i & 1])[(hf * TL::PIECE + 16 * (i >> 1) * 128) / 16]; };

    Acc16 acc[2];   // [features + 64][features + 16][rows + 16]
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int fb = 0; fb < 4; ++fb)
#pragma unroll
            for (int rb = 0; rb < 4; ++rb) acc[q][fb][rb] = f32x4{0.f, 0.f, 0.f, 0.f};

    bf16x8 w[4][4], a[2][4];   // [block of 32][block of 16, k step]
    auto end_of_reads = [&] {  // own reads complete; then both groups change places
        __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
        __builtin_amdgcn_sched_barrier(0);
        barrier_keep_loads_in_flight();
        __builtin_amdgcn_sched_barrier(0);
    };
    auto multiply = [&](auto q_c, auto hf_c) {
        constexpr int q = decltype(q_c)::value, hf = decltype(hf_c)::value;
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int fb = 0; fb < 4; ++fb)
#pragma unroll
                for (int t = 0; t < 2; ++t) {   // (back and forth: neighbours in time share an operand, which saves power)
                    const int rb = (fb & 1) ? 1 - t : t;
                    f32x4& c = acc[q][fb][2 * hf + rb];
                    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[2 * q + (fb >> 1)][2 * (fb & 1) + ks], a[hf][2 * rb + ks], c, 0, 0, 0);
                }
        __builtin_amdgcn_s_setprio(0);
        __builtin_amdgcn_sched_barrier(0);
        barrier_keep_loads_in_flight();
        __builtin_amdgcn_sched_barrier(0);
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;

    copy(CW01{}, 0); copy(CA0{}, 0); copy(CA1{}, 0); copy(CW23{}, 0);
    if (n_kt > 1) {
        copy(CW01{}, 1); copy(CA0{}, 1); copy(CA1{}, 1); copy(CW23{}, 1);
        __builtin_amdgcn_s_waitcnt(0x0f70 | 8);
    } else {
        __builtin_amdgcn_s_waitcnt(0x0f70);
    }
    barrier_keep_loads_in_flight();
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) { w[0][ks] = frag_w(0, ks); w[1][ks] = frag_w(1, ks); }
    end_of_reads();
    if (wave >= 4) barrier_keep_loads_in_flight();   // the second group starts half a phase later

    for (int kt = 0; kt < n_kt; ++kt) {
        const bool more = kt + 2 < n_kt;
        // phase 0
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) a[0][ks] = frag_a(0, ks);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) w[2][ks] = frag_w(2, ks);
        if (more) copy(CW01{}, kt + 2);
        end_of_reads();
        multiply(I0{}, I0{});
        // phase 1
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) a[1][ks] = frag_a(1, ks);
#pragma unroll
        for (int ks = 2; ks < 4; ++ks) w[2][ks] = frag_w(2, ks);
        if (more) {
            copy(CA0{}, kt + 2);
            __builtin_amdgcn_s_waitcnt(0x0f70 | 10);   // w0, w1 of the next tile are there
        } else {
            __builtin_amdgcn_s_waitcnt(0x0f70 | 6);
        }
        end_of_reads();
        multiply(I0{}, I1{});
        // phase 2
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) w[3][ks] = frag_w(3, ks);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {   // on to the other stage (behind the last tile: stale data, never used)
            rd_w[ks] += stage_step;
            rd_a[ks] += stage_step;
        }
        stage_step = -stage_step;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) w[0][ks] = frag_w(0, ks);
        if (more) copy(CA1{}, kt + 2);
        end_of_reads();
        multiply(I1{}, I1{});
        // phase 3
#pragma unroll
        for (int ks = 2; ks < 4; ++ks) w[0][ks] = frag_w(0, ks);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) w[1][ks] = frag_w(1, ks);
        if (more) {
            copy(CW23{}, kt + 2);
            __builtin_amdgcn_s_waitcnt(0x0f70 | 8);    // everything of the next tile is there
        } else {
            __builtin_amdgcn_s_waitcnt(0x0f70);
        }
        end_of_reads();
        multiply(I1{}, I0{});
    }
    if (wave < 4) barrier_keep_loads_in_flight();

    if (split_tile) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            float* dst = g.partials + ((size_t)(((int)blockIdx.x - g.n_whole) * TL::WAVE_TILES + 2 * wave + q)) * PARTIAL_FLOATS_PER_WAVE + lane;
#pragma unroll
            for (int i = 0; i < 64; ++i) dst[i * 64] = acc[q][i >> 4][(i >> 2) & 3][i & 3];
        }
        return;
    }
#pragma unroll
    for (int q = 0; q < 2; ++q)
        gemm_epilogue<EPI>(g, acc[q], smem, wave, lane, f0 + TL::feature0(2 * wave + q), r0 + TL::row_0(2 * wave + q));
}

// Adds the n_parts partial sums of every split tile and runs the epilogue on the result.  One wave per workgroup and
// grid.x = split tiles * NW: the work is a stream of partial sums, and with a 17 KB staging area instead of the
// ring's LDS many of these small workgroups share a CU and keep enough loads in flight.
template <int EPI, class TL>
__global__ __launch_bounds__(64) void gemm_fixup_kernel(GemmArgs g) {
    constexpr int NW = TL::WAVE_TILES;
    __shared__ __attribute__((aligned(16))) unsigned char smem[64 * EPI_PITCH * 4];
    const int lane = threadIdx.x;
    const int split = (int)blockIdx.x / NW, wave = (int)blockIdx.x % NW;
    int f0, r0;
    TL::origin(g, g.n_whole + split, f0, r0);
    typename TL::Acc acc;
    constexpr int V = sizeof(acc[0][0]) / sizeof(float), B = sizeof(acc[0]) / sizeof(acc[0][0]);   // accumulators of a tile, tiles along the rows
#pragma unroll
    for (int i = 0; i < 64; ++i) acc[i / V / B][i / V % B][i % V] = 0.f;
    for (int p = 0; p < g.n_parts; ++p) {
        const float* src = g.partials + ((size_t)((split * g.n_parts + p) * NW + wave)) * PARTIAL_FLOATS_PER_WAVE + lane;
#pragma unroll
        for (int i = 0; i < 64; ++i) acc[i / V / B][i / V % B][i % V] += src[i * 64];
    }
    gemm_epilogue<EPI>(g, acc, smem, /*staging slot*/ 0, lane, f0 + TL::feature0(wave), r0 + TL::row_0(wave));
}

// y = x * rsqrt(mean(x^2) + eps) * gain, one wave per row, fp32 statistics.
__global__ __launch_bounds__(256) void rmsnorm_kernel(const __bf16* __restrict__ x, const __bf16* __restrict__ gain, int R,
                                                      int hidden, float eps, __bf16* __restrict__ out) {
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (row >= R) return;
    const __bf16* xr = x + (int64_t)row * hidden;
    float ss = 0.f;
    for (int c = lane * 8; c < hidden; c += 512) {
        const bf16x8 v = *reinterpret_cast<const bf16x8*>(xr + c);
#pragma unroll
        for (int e = 0; e < 8; ++e) ss += (float)v[e] * (float)v[e];
    }
    for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
    const float inv = 1.0f / sqrtf(ss / (float)hidden + eps);
    __bf16* orow = out + (int64_t)row * hidden;
    for (int c = lane * 8; c < hidden; c += 512) {
        const bf16x8 v = *reinterpret_cast<const bf16x8*>(xr + c);
        const bf16x8 gn = *reinterpret_cast<const bf16x8*>(gain + c);
        bf16x8 o;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = (__bf16)((float)v[e] * inv * (float)gn[e]);
        *reinterpret_cast<bf16x8*>(orow + c) = o;
    }
}

// rope[r][p] = (cos, sin)(positions[r] * theta_p) in fp64, rounded once.
__global__ void rope_rows_table_kernel(const int32_t* __restrict__ positions, int R, int half_d, int d, double base,
                                       int index_base, float2* __restrict__ table) {
    const int r = blockIdx.x, p = threadIdx.x;
    if (r >= R || p >= half_d) return;
    const double theta = pow(base, -2.0 * (double)(p + index_base) / (double)d);
    double sn, cs;
    sincos((double)positions[r] * theta, &sn, &cs);
    table[(size_t)r * half_d + p] = make_float2((float)cs, (float)sn);
}

// How a launch of one tiling is laid out, and what it takes.
// One workgroup per CU at a time (the LDS ring fills it), so a launch runs in rounds of n_cu tiles and a last round
// of `rest` tiles leaves CUs idle.  The tiles of that round are split along K over n_cu / rest workgroups each: the
// round then takes 1 / n_parts of a tile's time, and the launch rest / n_cu rounds less.
// A part pays its own pipeline fill, a dump of partial sums (128 or 256 KB) and its share of the second kernel (13 us for
// 128 tiles of 256 x 128 in two parts).  Measured at 2970 rows with 256 x 128 tiles: K = 14336, 384 tiles, two parts of
// 112 K tiles: 9 % less time; K = 4096, 576 tiles, four parts of 16: 8 % less; K = 4096, 384 tiles, two parts of 32: 4 %
// less; K = 4096, 2688 tiles (a tenth of them in the last round): no change.
struct Plan {
    int n_tiles, n_whole, n_parts;
    float us;
};
template <class TL>
Plan plan_tiling(const GemmArgs& g, int n_cu, const GemmTuning& tune) {
    Plan p;
    p.n_tiles = ((g.N + TL::BF - 1) / TL::BF) * ((g.M + TL::BRT - 1) / TL::BRT);
    const int rest = p.n_tiles % n_cu, n_kt = g.K / BK;
    int n_parts = (rest == 0 || tune.tail_split == 0) ? 1 : std::min(n_cu / rest, 8);
    n_parts = std::min(n_parts, n_kt / MIN_K_TILES_PER_PART);
    if (n_parts > 1 &&
        (g.partials == nullptr || (size_t)rest * n_parts * TL::WAVE_TILES * PARTIAL_FLOATS_PER_WAVE * sizeof(float) > g.partials_bytes))
        n_parts = 1;
    p.n_parts = std::max(n_parts, 1);
    p.n_whole = p.n_parts > 1 ? p.n_tiles - rest : p.n_tiles;
    const float last = (float)(rest * p.n_parts) / (float)n_cu;   // share of the CUs that the last round keeps busy
    const float base = p.n_tiles > n_cu ? TL::ROUND_BASE : p.n_parts > 1 ? TL::ONLY_BASE_SPLIT : TL::ONLY_BASE;
    const float last_round = rest ? base + (1.0f - base) * last : 0.0f;
    p.us = TL::US_PER_K_TILE * n_kt * ((float)(p.n_tiles / n_cu) + last_round / (float)p.n_parts) + TL::US_LAUNCH +
           (p.n_parts > 1 ? TL::US_SPLIT : 0.0f);
    return p;
}

template <int EPI, class TL>
hipError_t launch_tiling(GemmArgs g, void (*kernel)(GemmArgs), const Plan& p, hipStream_t st) {
    // once per process (a function-local static is initialised exactly once, also under concurrent first calls)
    static const hipError_t setup = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, TL::LDS_BYTES);
    if (setup != hipSuccess) return setup;
    g.n_whole = p.n_whole;
    g.n_parts = p.n_parts;
    kernel<<<dim3(p.n_whole + (p.n_tiles - p.n_whole) * p.n_parts), dim3(64 * TL::NW), TL::LDS_BYTES, st>>>(g);
    if (p.n_parts > 1) gemm_fixup_kernel<EPI, TL><<<dim3((p.n_tiles - p.n_whole) * TL::WAVE_TILES), dim3(64), 0, st>>>(g);
    return hipGetLastError();
}

template <int EPI>
hipError_t launch_gemm(const GemmArgs& g, const GemmTuning& tune, hipStream_t st) {
    static const int n_cu = [] {
        int dev = 0, n = 0;
        return hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess ? n : 0;
    }();
    if (n_cu <= 0) return hipErrorInvalidDevice;
    // (Feeding the weight fragments from memory straight into registers, to halve the LDS traffic, was tried: 16-byte
    // pieces of 32 rows per load instruction cost far more in the memory pipeline than they save: 400-500 TFLOP/s.)
    const bool wide = (tune.tile == 256) || (tune.tile == 0 && g.N % 256 == 0);
    if (!wide) return launch_tiling<EPI, Tiling<2>>(g, &gemm_bf16_kernel<EPI, 2>, plan_tiling<Tiling<2>>(g, n_cu, tune), st);
    const Plan narrow = plan_tiling<Tiling<4>>(g, n_cu, tune);
    // 256 rows per workgroup where that is the shorter launch by the estimate above: a tile of twice the area takes 1.6
    // times as long, but it comes in rounds twice as coarse and its partial sums cost more.  256 x 128 -> 256 x 256, us:
    //   28672 x 4096 (gate / up): 1100 rows 235 stays, 2048 rows 425 -> 351, 2970 rows 650 -> 512, 4096 rows 895 -> 656
    //   4096 x 14336 (down):      1100 rows 145 -> 138, 2048 rows 193 -> 181, 2970 rows 305 -> 257, 4096 rows 397 -> 314
    //   4096 x 4096 (output):     1100 rows  46 stays, 2048 rows 63 stays, 2970 rows 103 -> 84, 4096 rows 125 -> 99
    //   6144 x 4096 (Q / K / V):  1100 rows  58 stays, 2048 rows 105 -> 87, 2970 rows 149 -> 131, 4096 rows 183 -> 166
    //   256 x 1792:               1 row      19 stays (30)
    if (tune.tile == 0) {
        const Plan square = plan_tiling<Tiling256>(g, n_cu, tune);
        if (square.us < narrow.us) return launch_tiling<EPI, Tiling256>(g, &gemm_bf16_256_kernel<EPI>, square, st);
    }
    return launch_tiling<EPI, Tiling<4>>(g, &gemm_bf16_kernel<EPI, 4>, narrow, st);
}

}  // namespace

size_t gemm_partials_bytes() { return (size_t)256 * 16 * PARTIAL_FLOATS_PER_WAVE * sizeof(float); }   // 256 parts of a 256 x 256 tile

hipError_t launch_linear(const void* a, const void* w, int M, int N, int K, const void* residual, void* out,
                         float* partials, size_t partials_bytes, const GemmTuning& tune, hipStream_t st) {
    GemmArgs g{};
    g.partials = partials; g.partials_bytes = partials_bytes;
    g.a = (const __bf16*)a; g.w = (const __bf16*)w; g.M = M; g.N = N; g.K = K;
    g.out = (__bf16*)out; g.residual = (const __bf16*)residual;
    return residual ? launch_gemm<EPI_RESIDUAL>(g, tune, st) : launch_gemm<EPI_STORE>(g, tune, st);
}

hipError_t launch_linear_swiglu(const void* a, const void* w_gate_up, int M, int F, int K, void* out, float* partials,
                                size_t partials_bytes, const GemmTuning& tune, hipStream_t st) {
    GemmArgs g{};
    g.partials = partials; g.partials_bytes = partials_bytes;
    g.a = (const __bf16*)a; g.w = (const __bf16*)w_gate_up; g.M = M; g.N = 2 * F; g.K = K; g.out = (__bf16*)out;
    return launch_gemm<EPI_SWIGLU>(g, tune, st);
}

hipError_t launch_qkv_rope(const Shape& s, const void* a, const void* w_qkv, int M, int K, const int32_t* positions,
                           float2* rope_rows, void* q_out, void* k_out, void* v_out, float* partials,
                           size_t partials_bytes, const GemmTuning& tune, hipStream_t st) {
    rope_rows_table_kernel<<<dim3(M), dim3(64), 0, st>>>(positions, M, s.d / 2, s.d, s.rope_base, s.rope_index_base,
                                                          rope_rows);
    GemmArgs g{};
    g.partials = partials; g.partials_bytes = partials_bytes;
    g.a = (const __bf16*)a; g.w = (const __bf16*)w_qkv; g.M = M; g.N = (s.Hq + 2 * s.Hkv) * s.d; g.K = K;
    g.q_out = (__bf16*)q_out; g.k_out = (__bf16*)k_out; g.v_out = (__bf16*)v_out; g.rope = rope_rows;
    g.Hq = s.Hq; g.Hkv = s.Hkv; g.d = s.d;
    return launch_gemm<EPI_QKV_ROPE>(g, tune, st);
}

hipError_t launch_rmsnorm(const void* x, const void* gain, int R, int hidden, float eps, void* out, hipStream_t st) {
    if (R == 0) return hipSuccess;
    rmsnorm_kernel<<<dim3((R + 3) / 4), dim3(256), 0, st>>>((const __bf16*)x, (const __bf16*)gain, R, hidden, eps,
                                                           (__bf16*)out);
    return hipGetLastError();
}

}  // namespace fr
