// Sparse prefill attention (eq. 9, Sec. 4.3) on the gfx950 matrix cores: bf16, head_dim 64 or 128, up to 64 query heads
// per KV head.
//
// Work split.  One workgroup (4 waves) owns one KV head and a tile of consecutive Q-index rows;
// each wave owns 64 "query columns" = floor(64 / G) token rows x the G query heads that share the KV
// head (a group size that does not divide 64 leaves a few columns idle: one of 64 at 7, four at 5), so every K/V tile staged in LDS is reused by the whole grouped-query group and by all
// four waves.  Rows are sorted by position, so a tile needs keys 0 .. (position of its last row);
// tiles are issued longest first.
//
// Orientation.  The kernel computes the transposed products S^T = K Q^T and O^T = V^T P^T with
// v_mfma_f32_32x32x16_bf16:
//   * keys run along the M (register) dimension of S^T and query columns along N (lanes), so the
//     softmax statistics of a query column live in one lane (plus its partner lane + 32);
//   * the fp32 accumulator layout of S^T is, after conversion to bf16, exactly the B-operand
//     layout of the second product (contraction over keys), so P never leaves registers;
//   * V is transposed once per (KV head, key tile) by the packing pre-pass (4 keys x 8 dims per lane,
//     repacked with byte permutes), so the A operand of the second product is a 16-byte LDS read.
// The key order inside every block of 16 keys is permuted identically in P^T and V^T
// ([0-3, 8-11, 4-7, 12-15]); a contraction does not care about the order of its terms.
//
// Softmax.  exp(s - m) / sum exp(s - m) does not depend on m, and fp32 / bf16 leave about 2^127 of
// headroom, so the fast kernel fixes each query column's reference m once (the maximum over the
// column's first 32 visible keys) and never rescales: the tile loop holds no maximum, no
// comparison and no branch.  If a later logit exceeds the reference by more than that headroom
// the sums overflow to inf; the workgroup then recomputes its item with the classic online softmax
// (running maximum).
//
// K/V tile images.  Every row tile of a KV head walks the same K/V stream (47 row tiles per head at 17k
// tokens / 15 %), so the work that does not depend on the rows is done once, by a packing pre-pass: for each
// (KV head, 64-key tile) it resolves stale / fresh rows (key j comes from k_new/v_new when inv[j] >= 0, i.e.
// its token is in the Q index, and from the cache otherwise: the cache is never written and stale rows are
// never read), transposes V, pads the rows against LDS bank conflicts and writes an image (35 KB at head_dim 128) that is byte
// for byte what the attention kernels want in LDS.  The fast kernel's tile loop then stages a tile with direct-to-LDS
// copies: no lookups, no pointer selects, no permutes, no address arithmetic, no staging registers.
//
// What a row does not see.  A weight of 0 does not take a NaN or an infinity out of a matrix product.  Positions behind the last
// row of the Q index may hold anything: they are not read.  A value that is not finite and that only some rows of a tile see makes the
// sums of the others NaN, which the overflow check finds; in the instances with split weights running_max_item then keeps such values apart.  (In
// the others the code for it would cost the tile loop 0.6 % through its registers; there a row is NaN too if one of the at most 63
// positions behind it in its last key tile is.)
#include "fr_internal.hpp"
#include "k_rotate.hpp"

#include <hip/hip_ext.h>

#include <algorithm>
#include <type_traits>

namespace fr {

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

constexpr int KT = 64;           // keys per tile
constexpr float NEG_BIG = -1.0e30f;

// Tile image = [K image][V^T image] (17 and 18 KB at head_dim 128, 9 KB each at 64), padded so that 16-byte operand reads (one
// lane per row, 16 lanes per LDS pass) fall into 16 distinct bank groups and every fragment address is base + constant:
//   K image:   64 rows (keys) of 2 D bytes of data + 16 B pad, rounded up to whole KB;
//   V^T image: D rows (dims) of 144 B (64 key slots = 128 B of data + 16 B pad), slot order see key_slot.
constexpr int V_ROW = 144;
template <int D>
struct Img {
    static constexpr int K_ROW = 2 * D + 16;
    static constexpr int K_BYTES = (KT * K_ROW + 1023) / 1024 * 1024;
    static constexpr int V_BYTES = D * V_ROW;
    static constexpr int BYTES = K_BYTES + V_BYTES;
    static constexpr int NK = D / 16;        // matrix steps of a 32-key half's logits, and of its share of the output
    static constexpr int MD = D / 32;        // 32-dim blocks of the output
    static constexpr int O_PITCH = D + 8;    // bf16 elements per output row in the epilogue's LDS staging
    static constexpr size_t EPILOGUE_LDS = 4 * 64 * O_PITCH * sizeof(__bf16);   // four waves x [64 columns][d] bf16
    static_assert(V_BYTES % 1024 == 0 && BYTES % 1024 == 0, "image layout");
};
// Inside every block of 16 keys the order is [0-3, 8-11, 4-7, 12-15]: the order in which the accumulator
// layout of S^T hands the keys to the second product.  Slot of key t (0..63) of a tile:
__device__ __forceinline__ int key_slot(int t) { return 16 * (t >> 4) + 4 * ((0x3120 >> (4 * ((t >> 2) & 3))) & 3) + (t & 3); }

// The fast kernel keeps separate rings of three K images and three V^T images (see its tile loop).
template <int D>
struct __attribute__((aligned(16))) Rings {
    unsigned char k[3][Img<D>::K_BYTES];
    unsigned char vt[3][Img<D>::V_BYTES];
};

__device__ __forceinline__ uint32_t perm_lo(uint32_t a, uint32_t b) {  // (a.lo16, b.lo16) -> a in low half
    return __builtin_amdgcn_perm(b, a, 0x05040100u);
}
__device__ __forceinline__ uint32_t perm_hi(uint32_t a, uint32_t b) {  // (a.hi16, b.hi16)
    return __builtin_amdgcn_perm(b, a, 0x07060302u);
}

// ---- what a lane knows about its workgroup, wave and two query columns ---------------------------
// G: query heads per KV head; 0 = known at run time only (group sizes without an instance of their own).
template <int G>
struct Geometry {
    int heads, trw;                      // query heads per KV head, token rows per wave
    int g, tile, row0;
    int x, h, wave;
    int col_row[2], col_head[2], col_pos[2];
    int wp_max;    // no key beyond it is visible to any row of this wave
    int n_kt;      // key tiles the workgroup walks
    int n_plain;   // leading tiles whose keys are visible to every row of the workgroup

    // ordinal counts the row tiles of a query from the longest one; ordinal < n_row_tiles
    __device__ __forceinline__ void init(const int32_t* __restrict__ q_index, int R, int Hq, int Hkv, int n_row_tiles,
                                         int n_img_tiles, int g_, int ordinal) {
        init_rows(Hq, Hkv, n_row_tiles, g_, ordinal);
        init_positions(q_index, R, n_img_tiles);
    }
    // The part that does not read the Q index: which rows and heads the lane's two columns are.
    __device__ __forceinline__ void init_rows(int Hq, int Hkv, int n_row_tiles, int g_, int ordinal) {
        const int tid = threadIdx.x, lane = tid & 63;
        heads = G > 0 ? G : Hq / Hkv;
        trw = G > 0 ? 64 / (G > 0 ? G : 1) : 64 / heads;
        wave = tid >> 6;
        x = lane & 31;
        h = lane >> 5;
        g = g_;
        tile = n_row_tiles - 1 - ordinal;                   // longest tiles first
        row0 = tile * 4 * trw;
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) {
            const int col = 32 * nb + x;
            const int head = min(col / trw, heads - 1);      // columns past trw x heads compute a copy of an earlier one
            const int r = row0 + wave * trw + (col % trw);
            col_row[nb] = r;                                 // rows past the end compute a copy of the last
            col_head[nb] = g * heads + head;                 // row; neither is ever stored
        }
    }
    // The positions of the rows, from the Q index.
    // (a position beyond the prompt breaks the caller's contract; the walk then ends with the last image that exists)
    __device__ __forceinline__ void init_positions(const int32_t* __restrict__ q_index, int R, int n_img_tiles) {
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) col_pos[nb] = q_index[min(col_row[nb], R - 1)];
        const int p_first = q_index[row0];                   // rows ascend: every key <= p_first is visible to all
        const int p_max = q_index[min(R, row0 + 4 * trw) - 1];    // the workgroup's furthest key
        wp_max = q_index[min(row0 + wave * trw + trw, R) - 1];   // a wave past the end copies the last row
        n_kt = min(p_max / KT + 1, n_img_tiles);
        n_plain = min((p_first + 1) / KT, n_kt - 1);
    }
};

// ---- which keys of a 64-key tile are fresh ---------------------------------------------------------------
// fresh[t] = row r of k_new / v_new that holds the recomputed entry of position 64 kt + t (q_index[r] == that
// position), else -1.  The Q index is strictly ascending: wave 0 finds the first row at or behind the tile's first
// position by a 64-ary search (every round probes 64 evenly spaced rows at once: two dependent loads for up to 4096
// rows, where a binary search needs twelve), then the at most 64 rows that can fall into the tile are read in one go.
// All 256 threads call it; `fresh` is LDS, valid after the call's closing barrier.
__device__ __forceinline__ void tile_fresh_rows(const int32_t* __restrict__ q_index, int R, int kt, int32_t* fresh) {
    const int tid = threadIdx.x;
    if (tid < KT) fresh[tid] = -1;
    __syncthreads();
    if (tid < 64) {
        const int target = kt * KT;
        int lo = 0, hi = R;   // the first row with q_index[row] >= target lies in [lo, hi]
        while (lo < hi) {
            const int step = (hi - lo + 63) >> 6;
            const int probe = lo + tid * step;
            const bool below = probe < hi && q_index[probe] < target;
            const int cnt = __popcll(__ballot(below));   // probes are ascending, so the ones below the target come first
            if (cnt == 0) { hi = lo; break; }
            const int last_below = lo + (cnt - 1) * step;
            hi = min(hi, last_below + step);
            lo = last_below + 1;
        }
        const int row = lo + tid;
        if (row < R) {
            const int pos = q_index[row];
            if (pos >= target && pos < target + KT) fresh[pos - target] = row;   // (pos < target only for an index that is not ascending)
        }
    }
    __syncthreads();
}

// ---- packing pre-pass: grid (key tiles, KV heads) ---------------------------------------------------------
// A thread's share of a tile in the packing kernels: 16-byte vector `vec` of the head rows of keys key + (256 / NV) i
// (K), and of the four consecutive keys 4 key + i (V, whose first 16 NV threads have a share).
template <int D>
struct PackShare {
    static constexpr int NV = D / 8;              // 16-byte vectors of a head row
    static constexpr int KI = KT * NV / 256;      // key vectors per thread: 4 at head_dim 128, 2 at 64
    int vec, key;
    bool has_v;
    __device__ __forceinline__ PackShare() {
        vec = threadIdx.x % NV;
        key = threadIdx.x / NV;
        has_v = threadIdx.x < 16 * NV;
    }
};
// Second half of both packing kernels: the thread's key vectors and 4 value vectors go into the LDS image, which is
// then written out as it is.
template <int D>
__device__ __forceinline__ void write_image(const PackShare<D>& ps, const u32x4 (&kreg)[PackShare<D>::KI],
                                            const u32x4 (&vreg)[4], unsigned char* img, unsigned char* __restrict__ dst) {
    using I = Img<D>;
    const int tid = threadIdx.x;
#pragma unroll
    for (int i = 0; i < PackShare<D>::KI; ++i)
        *reinterpret_cast<u32x4*>(&img[(ps.key + (256 / PackShare<D>::NV) * i) * I::K_ROW + 16 * ps.vec]) = kreg[i];
    {   // pads: K row tails, K image tail, V^T row tails (never read by the matrix operands; kept zero)
        const u32x4 z = {0u, 0u, 0u, 0u};
        if (tid < KT) *reinterpret_cast<u32x4*>(&img[tid * I::K_ROW + 2 * D]) = z;
        if (tid < (I::K_BYTES - KT * I::K_ROW) / 16) *reinterpret_cast<u32x4*>(&img[KT * I::K_ROW + 16 * tid]) = z;
        if (tid < D) *reinterpret_cast<u32x4*>(&img[I::K_BYTES + tid * V_ROW + 128]) = z;
    }
    if (ps.has_v) {
        const int slot = key_slot(4 * ps.key);   // the 4 keys of this lane occupy slots slot .. slot + 3
#pragma unroll
        for (int c = 0; c < 4; ++c) {   // dims 8 vec + 2c and + 2c + 1: gather the 4 keys of each
            u32x2 lo, hi;
            lo[0] = perm_lo(vreg[0][c], vreg[1][c]);
            lo[1] = perm_lo(vreg[2][c], vreg[3][c]);
            hi[0] = perm_hi(vreg[0][c], vreg[1][c]);
            hi[1] = perm_hi(vreg[2][c], vreg[3][c]);
            const int d0 = 8 * ps.vec + 2 * c, d1 = d0 + 1;
            *reinterpret_cast<u32x2*>(&img[I::K_BYTES + d0 * V_ROW + 2 * slot]) = lo;
            *reinterpret_cast<u32x2*>(&img[I::K_BYTES + d1 * V_ROW + 2 * slot]) = hi;
        }
    }
    __syncthreads();
    for (int i = tid * 16; i < I::BYTES; i += 4096)
        *reinterpret_cast<u32x4*>(dst + i) = *reinterpret_cast<const u32x4*>(&img[i]);
}

// WRITEBACK: the fresh rows are also stored at their positions of the cache (the write-back of Sec. 4.3 fused into
// this pass: the row is in registers anyway).  No workgroup reads a cache row that another one writes: a position
// with a fresh row is never read from the cache.
template <int D, bool WRITEBACK>
__global__ __launch_bounds__(256) void pack_kv_images_kernel(const __bf16* k_cache, const __bf16* v_cache, int L,
                                                             const __bf16* __restrict__ k_new,
                                                             const __bf16* __restrict__ v_new,
                                                             const int32_t* __restrict__ q_index, int R, int Hkv,
                                                             int n_img_tiles, unsigned char* __restrict__ images) {
    __shared__ __attribute__((aligned(16))) unsigned char img[Img<D>::BYTES];
    __shared__ int32_t fresh[KT];
    const int kt = blockIdx.x, g = blockIdx.y;
    const PackShare<D> ps;
    const bool have_new = k_new != nullptr;   // else the cache already holds the fresh rows
    // no row sees a position behind `last`: such keys of the tile repeat the one there (they may hold anything)
    const int last = max(min(q_index[R - 1], L - 1), kt * KT);
    if (have_new) tile_fresh_rows(q_index, R, kt, fresh);
    // key `t` of the tile, from k_new / v_new where it is fresh (with the write-back a repeated one: the same bytes again)
    auto fetch = [&](int t, const __bf16* cache, const __bf16* fresh_rows) -> u32x4 {
        const int j = min(kt * KT + t, last);
        const int r = have_new ? fresh[j - kt * KT] : -1;
        const __bf16* src = r >= 0 ? fresh_rows + ((size_t)r * Hkv + g) * D : cache + ((size_t)j * Hkv + g) * D;
        const u32x4 x = *reinterpret_cast<const u32x4*>(src + 8 * ps.vec);
        if (WRITEBACK && r >= 0)
            *reinterpret_cast<u32x4*>(const_cast<__bf16*>(cache) + ((size_t)j * Hkv + g) * D + 8 * ps.vec) = x;
        return x;
    };
    u32x4 kreg[PackShare<D>::KI], vreg[4];
#pragma unroll
    for (int i = 0; i < PackShare<D>::KI; ++i) kreg[i] = fetch(ps.key + (256 / PackShare<D>::NV) * i, k_cache, k_new);
    if (ps.has_v) {
#pragma unroll
        for (int i = 0; i < 4; ++i) vreg[i] = fetch(4 * ps.key + i, v_cache, v_new);
    }
    write_image<D>(ps, kreg, vreg, img, images + ((size_t)g * n_img_tiles + kt) * Img<D>::BYTES);
}

// The same images built from a chunk store that is shared between queries and never written (Sec. 4.3): position
// j < L_ctx of the prompt belongs to chunk c = (the chunk whose offsets contain j) and reads store row
// row0[c] + j - off[c]; its key is moved to the prompt position on the way (Appendix A: one more rotation by
// Delta_c, from the (cos, sin) rows of `table`, same arithmetic as the stand-alone position shift).  Positions
// listed in the Q index (inv[j] >= 0: recomputed context tokens and all question tokens) read the query's own
// fresh rows instead, so the store's stale entries of those tokens are never read and no per-query copy of the
// cache exists.  Positions >= L_ctx that are not in the Q index have no data: they read as zero.

// Prompt position -> (store row, chunk) for the packing kernel, so that it needs no search and no dependent loads:
// grid (position tiles of the longest chunk, chunks + 1); the extra y index covers the positions behind the context
// (no store row: -1).
__global__ __launch_bounds__(256) void prompt_map_kernel(ChunkTable ct, ChunkRows rows, int L,
                                                         int32_t* __restrict__ store_row, int32_t* __restrict__ chunk_id) {
    const int c = blockIdx.y;
    const int begin = (c < ct.n) ? ct.off[c] : ct.off[ct.n];
    const int end = (c < ct.n) ? ct.off[c + 1] : L;
    for (int j = begin + blockIdx.x * 256 + threadIdx.x; j < end; j += gridDim.x * 256) {
        store_row[j] = (c < ct.n) ? rows.row0[c] + (j - begin) : -1;
        chunk_id[j] = (c < ct.n) ? c : 0;
    }
}

template <int LAYOUT>
__global__ __launch_bounds__(256) void pack_kv_images_shared_kernel(const __bf16* __restrict__ k_store,
                                                                    const __bf16* __restrict__ v_store,
                                                                    const int32_t* __restrict__ store_row,
                                                                    const int32_t* __restrict__ chunk_id,
                                                                    const float2* __restrict__ table,
                                                                    int L, const __bf16* __restrict__ k_new,
                                                                    const __bf16* __restrict__ v_new,
                                                                    const int32_t* __restrict__ q_index, int R, int Hkv,
                                                                    int n_img_tiles, unsigned char* __restrict__ images) {
    constexpr int D = 128;
    __shared__ __attribute__((aligned(16))) unsigned char img[Img<D>::BYTES];
    __shared__ int32_t fresh[KT];
    const int kt = blockIdx.x, g = blockIdx.y;
    const PackShare<D> ps;
    const int st_vec = ps.vec, st_key = ps.key;
    const u32x4 zero = {0u, 0u, 0u, 0u};
    tile_fresh_rows(q_index, R, kt, fresh);
    int jk[4], jv[4], rk[4], rv[4], sk[4], sv[4], ck[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {   // the maps first, all at once: no load below depends on more than one of them
        jk[i] = min(kt * KT + st_key + 16 * i, L - 1);
        jv[i] = min(kt * KT + 4 * st_key + i, L - 1);
        rk[i] = fresh[jk[i] - kt * KT];
        rv[i] = fresh[jv[i] - kt * KT];
        sk[i] = store_row[jk[i]];
        sv[i] = store_row[jv[i]];
        ck[i] = chunk_id[jk[i]];
    }
    u32x4 kreg[4], vreg[4], kpart[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {   // positions that are neither fresh nor in a chunk read row 0 of the page and become zero
        const __bf16* pk = (rk[i] >= 0 || sk[i] < 0) ? k_new + ((size_t)max(rk[i], 0) * Hkv + g) * D
                                                      : k_store + ((size_t)sk[i] * Hkv + g) * D;
        const __bf16* pv = (rv[i] >= 0 || sv[i] < 0) ? v_new + ((size_t)max(rv[i], 0) * Hkv + g) * D
                                                      : v_store + ((size_t)sv[i] * Hkv + g) * D;
        kreg[i] = *reinterpret_cast<const u32x4*>(pk + 8 * st_vec);
        if (LAYOUT != FR_ROPE_INTERLEAVED) kpart[i] = *reinterpret_cast<const u32x4*>(pk + 8 * (st_vec ^ 8));
        vreg[i] = *reinterpret_cast<const u32x4*>(pv + 8 * st_vec);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (rk[i] < 0) {
            if (sk[i] >= 0)
                kreg[i] = rotate_key_vector<__bf16, D, LAYOUT>(kreg[i], LAYOUT != FR_ROPE_INTERLEAVED ? kpart[i] : kreg[i],
                                                    table + (size_t)ck[i] * (D / 2), st_vec);
            else
                kreg[i] = zero;
        }
        if (rv[i] < 0 && sv[i] < 0) vreg[i] = zero;
    }
    write_image<D>(ps, kreg, vreg, img, images + ((size_t)g * n_img_tiles + kt) * Img<D>::BYTES);
}

// ---- staging in the fast kernel: image -> LDS directly (global_load_lds_dwordx4: lane i of a wave deposits its
//      16 bytes at the wave's LDS base + 16 i), no registers involved.  An image is N = 18 (9 at head_dim 64) chunks
//      of 1 KB; wave w moves chunks w, w + 4, ...  Completion: the issuing wave's vmcnt, then a workgroup barrier. ----------
template <int N>
__device__ __forceinline__ void dma_image(const unsigned char* src, unsigned char* lds_dst, int wave, int lane) {
    // Written out rather than left to the builtin: the compiler treats a pending direct-to-LDS load as an access
    // that may complete out of order with the LDS reads, and from then on waits for *all* outstanding fragment
    // reads before every use (lgkmcnt(0)), which puts a full LDS round trip in front of the matrix pipe every few
    // fragments.  Completion is waited for explicitly anyway (wait_dma + workgroup barrier), so nothing is lost.
    // The image address is the same for the whole workgroup, so it travels in scalar registers (base + 16 lane):
    // the copies cost the vector ALU nothing.  `wave` must be wave-uniform in the compiler's eyes (readfirstlane).
    const uint32_t lds_base = __builtin_amdgcn_readfirstlane(
        (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds_dst);
    const uint32_t lane_off = (uint32_t)lane * 16u;
#pragma unroll
    for (int c = 0; c < (N + 3) / 4; ++c) {
        const int chunk = wave + 4 * c;
        if (4 * c + 3 < N || wave < N - 4 * c) {
            const unsigned char* g = src + chunk * 1024;
            const uint32_t l = lds_base + (uint32_t)chunk * 1024u;
            asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(lane_off), "s"(g), "s"(l) : "memory");
        }
    }
}
__device__ __forceinline__ void wait_dma() { __builtin_amdgcn_s_waitcnt(0x0f70); }   // vmcnt(0)

// ---- staging in the safe kernel: image -> registers -> LDS, 16 bytes per lane and copy -------------------
template <int D>
struct ImageStager {
    static constexpr int BYTES = Img<D>::BYTES;
    static constexpr int N = (BYTES + 4095) / 4096;   // the last copy may be a part of the workgroup's
    const unsigned char* head_images;   // images of this KV head
    int lane_off;                       // threadIdx.x * 16
    u32x4 reg[N];
    __device__ __forceinline__ void init(const unsigned char* images, int g, int n_img_tiles) {
        head_images = images + (size_t)g * n_img_tiles * BYTES;
        lane_off = threadIdx.x * 16;
    }
    __device__ __forceinline__ void load(int kt) {
        const unsigned char* p = head_images + (size_t)kt * BYTES;
#pragma unroll
        for (int i = 0; i < N; ++i)
            reg[i] = *reinterpret_cast<const u32x4*>(p + min(i * 4096 + lane_off, BYTES - 16));
    }
    __device__ __forceinline__ void write(unsigned char* img) const {
#pragma unroll
        for (int i = 0; i < N; ++i)
            if (i * 4096 + lane_off < BYTES) *reinterpret_cast<u32x4*>(img + i * 4096 + lane_off) = reg[i];
    }
};

// Per-lane byte offsets of the operand fragments inside an image: row x, 16-byte half h.
template <int D>
struct FragOffsets {
    int k;   // K fragment: + 32 ks (16 dims per step) + 32 * Img<D>::K_ROW for the second half of the tile
    int v;   // V^T fragment: + 32 kb (16 key slots per block) + 32 * V_ROW * md for dim block md
    __device__ __forceinline__ void init(int x, int h) {
        k = x * Img<D>::K_ROW + 16 * h;
        v = x * V_ROW + 16 * h;
    }
};

// The weights of 32 keys x 64 columns as operands of the second product.  SPLIT: every weight as the sum of three bf16
// numbers, each the rounding of what the ones before leave (8 bits each, the differences are exact): all 24 bits of an fp32 weight, for
// the shapes whose weights have always been kept in fp32; the second product then takes three instructions per fragment.
// (Error of the output beyond its own rounding, 17k tokens: two numbers 2.0e-6, three 0.4e-6, the vector ALU's fp32 0.2e-6.  Two
// take 0.62 ms for the tile loop of 28 / 4 heads and 2970 rows, three 0.80.)
template <bool SPLIT>
struct Weights {
    static constexpr int PARTS = SPLIT ? 3 : 1;
    bf16x8 part[PARTS][2][2];
    __device__ __forceinline__ void set(int nb, int v, float p) {
#pragma unroll
        for (int i = 0; i < PARTS; ++i) {
            const __bf16 t = (__bf16)p;
            part[i][nb][v >> 3][v & 7] = t;
            p -= (float)t;
        }
    }
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
            for (int v = 0; v < 16; ++v) set(nb, v, 0.f);
    }
    __device__ __forceinline__ void multiply(const bf16x8& a, int nb, int kk, f32x16& acc) const {
#pragma unroll
        for (int i = 0; i < PARTS; ++i) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, part[i][nb][kk], acc, 0, 0, 0);
    }
};

// S^T for 32 keys (half mb of a staged tile) against this wave's 64 query columns.
template <int D>
__device__ __forceinline__ void qk_half(const unsigned char* k, int mb, const bf16x8 (&qf)[2][D / 16], const FragOffsets<D>& fo,
                                        f32x16 (&s)[2]) {
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int v = 0; v < 16; ++v) s[nb][v] = 0.f;
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) {
        const bf16x8 a = *reinterpret_cast<const bf16x8*>(k + fo.k + 32 * ks + mb * (32 * Img<D>::K_ROW));
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) s[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[nb][ks], s[nb], 0, 0, 0);
    }
}

template <bool MASK>
__device__ __forceinline__ void mask_half(f32x16 (&s)[2], const int (&col_pos)[2], int key_base, int h) {
    if (!MASK) return;
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int key = key_base + 8 * (v >> 2) + 4 * h + (v & 3);
            if (key > col_pos[nb]) s[nb][v] = -INFINITY;
        }
}

// The two bf16 numbers of a word, 0 in the place of one that is not finite.
__device__ __forceinline__ uint32_t finite_or_zero(uint32_t w) {
    if ((w & 0x00007F80u) == 0x00007F80u) w &= 0xFFFF0000u;
    if ((w & 0x7F800000u) == 0x7F800000u) w &= 0x0000FFFFu;
    return w;
}

// O^T += V^T P^T for the 32 keys of half mb.  FINITE_ONLY: without the values that are not finite.
template <int D, bool SPLIT, bool FINITE_ONLY = false>
__device__ __forceinline__ void pv_half(const unsigned char* vt, int mb, const Weights<SPLIT>& pf, const FragOffsets<D>& fo,
                                        f32x16 (&o)[D / 32][2]) {
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
        const int kb = 2 * mb + kk;
#pragma unroll
        for (int md = 0; md < D / 32; ++md) {
            bf16x8 a = *reinterpret_cast<const bf16x8*>(vt + fo.v + 32 * kb + md * (32 * V_ROW));
            if constexpr (FINITE_ONLY) {
                u32x4 bits = __builtin_bit_cast(u32x4, a);
#pragma unroll
                for (int e = 0; e < 4; ++e) bits[e] = finite_or_zero(bits[e]);
                a = __builtin_bit_cast(bf16x8, bits);
            }
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) pf.multiply(a, nb, kk, o[md][nb]);
        }
    }
}

// Does the V^T image of a tile hold a value that is not finite?  The same answer in every lane of the wave.
template <int D>
__device__ __forceinline__ bool holds_not_finite(const unsigned char* vt) {
    bool found = false;
    for (int i = (threadIdx.x & 63) * 16; i < Img<D>::V_BYTES; i += 1024) {
        const u32x4 w = *reinterpret_cast<const u32x4*>(vt + i);
#pragma unroll
        for (int e = 0; e < 4; ++e) found = found || finite_or_zero(w[e]) != w[e];
    }
    return __any(found);
}
// O^T += those values, for the columns that see them.  Their weights are positive: an infinity stays what it is, a NaN too.
template <int D>
__device__ __forceinline__ void add_not_finite(const unsigned char* vt, int key_base, const int (&col_pos)[2], int h,
                                               f32x16 (&o)[D / 32][2]) {
    for (int t = 0; t < KT; ++t) {
        const unsigned char* key = vt + 2 * key_slot(t) + 4 * h * V_ROW;
#pragma unroll
        for (int md = 0; md < D / 32; ++md)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const uint32_t w = *reinterpret_cast<const uint16_t*>(key + (32 * md + 8 * (v >> 2) + (v & 3)) * V_ROW);
                if ((w & 0x7F80u) != 0x7F80u) continue;
#pragma unroll
                for (int nb = 0; nb < 2; ++nb)
                    if (key_base + t <= col_pos[nb]) o[md][nb][v] += __uint_as_float(w << 16);
            }
    }
}

// One step of the fast kernel's software pipeline, at the granularity of 32 keys ("a half").  It turns the
// logits of half j (s_cur) into bf16 weights (pf_cur), while the matrix cores form the logits of half j+1
// (s_nxt = K Q^T, 16 instructions at head_dim 128) and add half j-1 to the output (O^T += V^T P^T with pf_prev, 16
// instructions, 48 with split weights).  The three strands are independent, so the vector ALU's exp work runs in the shadow of the
// matrix instructions.  The exponent reference is fixed per column: no maximum, no rescale, no branch.
template <int D, bool SPLIT, bool MASK, bool DO_QK>
__device__ __forceinline__ void pipeline_step(const unsigned char* k_next, int mb_next, const unsigned char* vt_prev,
                                              int mb_prev, const FragOffsets<D>& fo, const bf16x8 (&qf)[2][D / 16],
                                              f32x16 (&s_cur)[2], f32x16 (&s_nxt)[2], const Weights<SPLIT>& pf_prev,
                                              Weights<SPLIT>& pf_cur, f32x16 (&o)[D / 32][2],
                                              float (&lsum)[2], const float (&mref)[2], const int (&col_pos)[2],
                                              int key_base, int h, float scale_log2e) {
    mask_half<MASK>(s_cur, col_pos, key_base, h);
    if (DO_QK) {
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
            for (int v = 0; v < 16; ++v) s_nxt[nb][v] = 0.f;
    }
    // Operand fragments are requested from LDS PF matrix steps before their use (rotating register buffer), so the
    // LDS latency overlaps the matrix and vector work already in flight.
    constexpr int PF = 4;
    constexpr int NK = Img<D>::NK, MD = Img<D>::MD;   // steps 0 .. NK - 1: logits, NK .. 2 NK - 1: output
    bf16x8 fr[PF + 1];
    auto frag = [&](int i) -> bf16x8 {   // i < NK: K fragment ks = i of the next half;  else: V fragment (kk, md)
        if (i < NK) return *reinterpret_cast<const bf16x8*>(k_next + fo.k + 32 * i + mb_next * (32 * Img<D>::K_ROW));
        const int j = i - NK, kk = j / MD, md = j % MD;
        return *reinterpret_cast<const bf16x8*>(vt_prev + fo.v + 32 * (2 * mb_prev + kk) + md * (32 * V_ROW));
    };
    constexpr int first = DO_QK ? 0 : NK;
#pragma unroll
    for (int i = 0; i < PF; ++i) fr[i] = frag(first + i);
    float psum0 = 0.f, psum1 = 0.f;
    constexpr int EW = 16 / NK;   // weights per matrix step: column block 0 during the logits, block 1 during the output
#pragma unroll
    for (int i = first; i < 2 * NK; ++i) {
        if (i + PF < 2 * NK) fr[(i - first + PF) % (PF + 1)] = frag(i + PF);
        const bf16x8 a = fr[(i - first) % (PF + 1)];
        if (i < NK) {
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) s_nxt[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[nb][i], s_nxt[nb], 0, 0, 0);
        } else {
            const int j = i - NK, kk = j / MD, md = j % MD;
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) pf_prev.multiply(a, nb, kk, o[md][nb]);
        }
        if (DO_QK || i >= NK) {
            const int nb = (i < NK) ? 0 : 1;
#pragma unroll
            for (int e = 0; e < EW; ++e) {
                const int v = EW * (i % NK) + e;
                const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s_cur[nb][v], scale_log2e, -mref[nb]));
                if (nb == 0) psum0 += p; else psum1 += p;
                pf_cur.set(nb, v, p);
            }
        }
    }
    if (!DO_QK) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s_cur[0][v], scale_log2e, -mref[0]));
            psum0 += p;
            pf_cur.set(0, v, p);
        }
    }
    lsum[0] += psum0;
    lsum[1] += psum1;
    // Ask the scheduler for: every fragment read PF matrix steps ahead of its use, and matrix and transcendental
    // instructions (the two long-latency strands) alternating.  Measured: several per cent over its own order;
    // patterns that also place the remaining vector work lose.
    __builtin_amdgcn_sched_group_barrier(0x100, PF, 0);       // the first PF fragment reads
#pragma unroll
    for (int i = first; i < 2 * NK; ++i) {
        if (i + PF < 2 * NK) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // fragment i + PF
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (SPLIT && i >= NK) __builtin_amdgcn_sched_group_barrier(0x008, Weights<SPLIT>::PARTS, 0); else __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // matrix
            __builtin_amdgcn_sched_group_barrier(0x400, EW / 2, 0);   // transcendental
        }
    }
}

// Normalise, transpose through LDS and store 16 bytes per lane; lse = (m + log2 l) ln 2.
template <int G, int D>
__device__ __forceinline__ void store_output(const Geometry<G>& ge, f32x16 (&o)[D / 32][2], const float (&l)[2],
                                             const float (&mref)[2], int R, int Hq, unsigned char* smem,
                                             __bf16* __restrict__ out, float* __restrict__ lse_out) {
    constexpr int O_PITCH = Img<D>::O_PITCH, NV = D / 8;
    __bf16* ob = reinterpret_cast<__bf16*>(smem) + ge.wave * 64 * O_PITCH;   // this wave's [64 columns][d]
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
        const float inv_l = 1.0f / l[nb];
#pragma unroll
        for (int md = 0; md < D / 32; ++md)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                bf16x4 w;
#pragma unroll
                for (int e = 0; e < 4; ++e) w[e] = (__bf16)(o[md][nb][4 * q4 + e] * inv_l);
                *reinterpret_cast<bf16x4*>(&ob[(32 * nb + ge.x) * O_PITCH + 32 * md + 8 * q4 + 4 * ge.h]) = w;
            }
        if (lse_out != nullptr && ge.h == 0 && ge.col_row[nb] < R && 32 * nb + ge.x < ge.trw * ge.heads)
            lse_out[(size_t)ge.col_row[nb] * Hq + ge.col_head[nb]] =
                (mref[nb] + __builtin_amdgcn_logf(l[nb])) * 0.6931471805599453f;
    }
    __syncthreads();   // (each wave reads back only its own region; the barrier orders its LDS writes and reads)
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int col = (64 / NV) * i + lane / NV, vec = lane % NV;
        const int r = ge.row0 + ge.wave * ge.trw + (col % ge.trw), head = col / ge.trw;
        if (r < R && head < ge.heads) {
            const u32x4 w = *reinterpret_cast<const u32x4*>(&ob[col * O_PITCH + 8 * vec]);
            *reinterpret_cast<u32x4*>(out + ((size_t)r * Hq + ge.g * ge.heads + head) * D + 8 * vec) = w;
        }
    }
}

// The same for dims 32 md .. 32 md + 31 only (a workgroup of the combine pass).
template <int G, int D>
__device__ __forceinline__ void store_slice(const Geometry<G>& ge, const f32x16 (&acc)[2], int md, const float (&l)[2],
                                            const float (&mref)[2], int R, int Hq, unsigned char* smem,
                                            __bf16* __restrict__ out, float* __restrict__ lse_out) {
    constexpr int PITCH = 40;   // 32 dims + 16 bytes
    __bf16* ob = reinterpret_cast<__bf16*>(smem) + ge.wave * 64 * PITCH;
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
        const float inv_l = 1.0f / l[nb];
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            bf16x4 w;
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e] = (__bf16)(acc[nb][4 * q4 + e] * inv_l);
            *reinterpret_cast<bf16x4*>(&ob[(32 * nb + ge.x) * PITCH + 8 * q4 + 4 * ge.h]) = w;
        }
        if (md == 0 && lse_out != nullptr && ge.h == 0 && ge.col_row[nb] < R && 32 * nb + ge.x < ge.trw * ge.heads)
            lse_out[(size_t)ge.col_row[nb] * Hq + ge.col_head[nb]] =
                (mref[nb] + __builtin_amdgcn_logf(l[nb])) * 0.6931471805599453f;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int col = 16 * i + lane / 4, vec = lane % 4;
        const int r = ge.row0 + ge.wave * ge.trw + (col % ge.trw), head = col / ge.trw;
        if (r < R && head < ge.heads) {
            const u32x4 w = *reinterpret_cast<const u32x4*>(&ob[col * PITCH + 8 * vec]);
            *reinterpret_cast<u32x4*>(out + ((size_t)r * Hq + ge.g * ge.heads + head) * D + 32 * md + 8 * vec) = w;
        }
    }
}

// Partial result of one part of an item, per lane: its 2 x D / 2 output accumulators, the two sums, the two exponent
// references and two scale exponents as 32-bit words.  Register-major (word r of thread t at [r * 256 + t]: every store
// and load is one coalesced 1 KB line per wave).  Part p of item (ordinal, KV head g) lives at
// (((query * max_row_tiles + ordinal) * n_parts + p) * Hkv + g) * WORDS.  Infinities and NaNs survive the packing (the
// combine pass must still see an overflow).
// F32: the accumulators as they are.  Otherwise as half-precision pairs, the 64 of a column block scaled by a power of two
// that brings the largest of them into [0.5, 1) (11 significant bits of that column's largest value): 70 words instead of
// 134.  Which one: half_parts.
template <int D, bool F32>
struct Part {
    static constexpr int O_WORDS = F32 ? D : D / 2;   // per lane, both column blocks
    static constexpr int REGS = O_WORDS + 6;
    static constexpr int WORDS = REGS * 256;          // 32-bit words of a part
};
typedef _Float16 __attribute__((ext_vector_type(2))) f16x2;

template <int D, bool F32>
__device__ __forceinline__ void store_partial(float* __restrict__ dst_f, const f32x16 (&o)[D / 32][2], const float (&lsum)[2],
                                              const float (&mref)[2]) {
    constexpr int OW = Part<D, F32>::O_WORDS;
    uint32_t* dst = reinterpret_cast<uint32_t*>(dst_f);
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
        int e = 0;
        if constexpr (F32) {
#pragma unroll
            for (int md = 0; md < D / 32; ++md)
#pragma unroll
                for (int v = 0; v < 16; ++v) dst[(nb * (OW / 2) + md * 16 + v) * 256] = __float_as_uint(o[md][nb][v]);
        } else {
            float m = 0.f;
#pragma unroll
            for (int md = 0; md < D / 32; ++md)
#pragma unroll
                for (int v = 0; v < 16; ++v) m = fmaxf(m, fabsf(o[md][nb][v]));
            // m = f 2^e with f in [0.5, 1); an infinite m keeps e = 0: the infinity is stored as it is
            e = (m < INFINITY) ? __builtin_amdgcn_frexp_expf(m) : 0;
#pragma unroll
            for (int md = 0; md < D / 32; ++md)
#pragma unroll
                for (int v = 0; v < 16; v += 2) {
                    f16x2 h;
                    h[0] = (_Float16)__builtin_ldexpf(o[md][nb][v], -e);
                    h[1] = (_Float16)__builtin_ldexpf(o[md][nb][v + 1], -e);
                    dst[(nb * (OW / 2) + md * 8 + v / 2) * 256] = __builtin_bit_cast(uint32_t, h);
                }
        }
        dst[(OW + nb) * 256] = __float_as_uint(lsum[nb]);
        dst[(OW + 2 + nb) * 256] = __float_as_uint(mref[nb]);
        dst[(OW + 4 + nb) * 256] = (uint32_t)e;
    }
}

// One launch serves up to ATTN_MAX_BATCH queries with their own rows, index sets, tile images and outputs (Sec. 4.3:
// queries of a batch share nothing but the chunk store the images were built from).  The table travels as a kernel
// argument.  blockIdx.x = (query * max_row_tiles + ordinal) * Hkv + KV head (launches without parts): consecutive blocks land
// on different XCDs, so with 8 KV heads each XCD's L2 serves the images of one head; the queries follow one another,
// each with its row tiles longest first, so that the short tiles at the end of one query run beside the long ones of
// the next and no more than about two queries' images are in use at a time (interleaving the queries was measured:
// their images then compete for the caches and the batch gains nothing over one launch per query).  A query with fewer
// row tiles than the longest one leaves its surplus blocks empty.
struct AttnQuery {
    const __bf16* q_rows;
    const int32_t* q_index;
    const unsigned char* images;
    __bf16* out;
    float* lse;
    int R, n_row_tiles, n_img_tiles, pad;
};
struct AttnBatch {
    AttnQuery q[ATTN_MAX_BATCH];
    int n, max_row_tiles;
};
struct BlockWork {
    int g, ordinal, query;
    __device__ __forceinline__ void init(int max_row_tiles, int Hkv) {
        int t = (int)blockIdx.x;
        g = t % Hkv; t /= Hkv;
        ordinal = t % max_row_tiles;
        query = t / max_row_tiles;
    }
};

// ---- classic online softmax (running maximum) for one (row tile, KV head): the whole key range, one workgroup.
//      Runs where the fixed exponent reference overflowed, and everywhere under FR_ATTN_SOFTMAX_RUNNING_MAX.
//      `smem` holds one image or the epilogue's staging; every thread of the workgroup calls it.  slice >= 0: only the
//      dims of that block of 32 are stored (a workgroup of the combine pass).  -------------------------------------------
template <int G, int D, bool SPLIT>
__device__ __forceinline__ void running_max_item(const AttnQuery& aq, int g, int ordinal, int Hq, int Hkv,
                                                 float scale_log2e, unsigned char* smem, int slice = -1) {
    const __bf16* __restrict__ q_rows = aq.q_rows;
    const int R = aq.R, n_img_tiles = aq.n_img_tiles;
    unsigned char* k_img = smem;
    unsigned char* v_img = smem + Img<D>::K_BYTES;
    Geometry<G> ge;
    ge.init(aq.q_index, R, Hq, Hkv, aq.n_row_tiles, n_img_tiles, g, ordinal);
    const int h = ge.h;
    FragOffsets<D> fo;
    fo.init(ge.x, h);
    bf16x8 qf[2][D / 16];
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
        const __bf16* qp = q_rows + ((size_t)min(ge.col_row[nb], R - 1) * Hq + ge.col_head[nb]) * D + 8 * h;
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) qf[nb][ks] = *reinterpret_cast<const bf16x8*>(qp + 16 * ks);
    }
    f32x16 o[D / 32][2];
#pragma unroll
    for (int md = 0; md < D / 32; ++md)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
            for (int v = 0; v < 16; ++v) o[md][nb][v] = 0.f;
    float lsum[2] = {0.f, 0.f};
    float m2[2] = {NEG_BIG, NEG_BIG};
    ImageStager<D> sg;
    sg.init(aq.images, ge.g, n_img_tiles);
    for (int kt = 0; kt < ge.n_kt; ++kt) {
        sg.load(kt);
        __syncthreads();
        sg.write(k_img);
        __syncthreads();
        if (kt * KT > ge.wp_max) continue;   // wave-uniform; the barriers stay outside
        const bool apart = SPLIT && kt >= ge.n_plain && holds_not_finite<D>(v_img);   // some rows may not see them
#pragma unroll
        for (int mb = 0; mb < 2; ++mb) {
            f32x16 s[2];
            qk_half<D>(k_img, mb, qf, fo, s);
            mask_half<true>(s, ge.col_pos, kt * KT + 32 * mb, h);
            Weights<SPLIT> pf;
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) {
                float t = s[nb][0];
#pragma unroll
                for (int v = 1; v < 16; ++v) t = fmaxf(t, s[nb][v]);
                t = fmaxf(t, __shfl_xor(t, 32));
                const float m_new = fmaxf(m2[nb], t * scale_log2e);
                const float alpha = __builtin_amdgcn_exp2f(m2[nb] - m_new);
                m2[nb] = m_new;
                float psum = 0.f;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[nb][v], scale_log2e, -m_new));
                    psum += p;
                    pf.set(nb, v, p);
                }
                lsum[nb] = lsum[nb] * alpha + psum;
#pragma unroll
                for (int md = 0; md < D / 32; ++md)
#pragma unroll
                    for (int v = 0; v < 16; ++v) o[md][nb][v] *= alpha;
            }
            if constexpr (SPLIT) {
                if (apart) pv_half<D, SPLIT, true>(v_img, mb, pf, fo, o); else pv_half<D, SPLIT>(v_img, mb, pf, fo, o);
            } else {
                pv_half<D, SPLIT>(v_img, mb, pf, fo, o);
            }
        }
        if constexpr (SPLIT) { if (apart) add_not_finite<D>(v_img, kt * KT, ge.col_pos, h, o); }
    }
    float l[2];
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) l[nb] = lsum[nb] + __shfl_xor(lsum[nb], 32);
    __syncthreads();
    if (slice < 0) {
        store_output<G, D>(ge, o, l, m2, R, Hq, smem, aq.out, aq.lse);
        return;
    }
    f32x16 acc[2] = {o[0][0], o[0][1]};
#pragma unroll
    for (int md = 1; md < D / 32; ++md)
        if (md == slice) { acc[0] = o[md][0]; acc[1] = o[md][1]; }
    store_slice<G, D>(ge, acc, slice, l, m2, R, Hq, smem, aq.out, aq.lse);
}

// Overflow check of a finished item: with a fixed reference a runaway logit shows up as inf / nan in the sums.
// Returns (workgroup-uniform) whether any column of the workgroup is affected; l = the columns' softmax sums.
template <int D>
__device__ __forceinline__ int sums_overflowed(const f32x16 (&o)[D / 32][2], const float (&lsum)[2], float (&l)[2]) {
    bool bad = false;
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
        l[nb] = lsum[nb] + __shfl_xor(lsum[nb], 32);
        float chk = l[nb];
#pragma unroll
        for (int md = 0; md < D / 32; ++md)
#pragma unroll
            for (int v = 0; v < 16; ++v) chk += fabsf(o[md][nb][v]);
        bad = bad || !(chk < INFINITY) || !(l[nb] > 0.f);
    }
    return __syncthreads_or(bad ? 1 : 0);   // also: every wave is done with the rings
}

// ---- fast path: key tiles [kb, ke) of one (row tile, KV head) ---------------------------------------------
// part < 0: the piece is the whole item; the workgroup finishes it: overflow check, then the output, or the item again with
// a running maximum (in this kernel: a second one that looked for flagged items cost 4 us per call and found none).
// part >= 0: the piece is
// share `part` of `n_parts` of the item's key tiles; it leaves its partial sums, and attn_combine_kernel finishes
// the item.  Every part uses the same exponent reference (each derives it from keys 0..31), so the parts simply add up.
template <int G, int D, bool SPLIT>
__device__ __forceinline__ void process_piece(const AttnQuery& aq, int g, int ordinal, int part, int n_parts, int item,
                                              float* __restrict__ partials, bool half, int Hq, int Hkv, float scale_log2e,
                                              unsigned char* smem_raw) {
    using I = Img<D>;
    Rings<D>& rg = *reinterpret_cast<Rings<D>*>(smem_raw);
    const __bf16* __restrict__ q_rows = aq.q_rows;
    const int R = aq.R, n_img_tiles = aq.n_img_tiles;
    // ---- prologue.  Everything that does not depend on the Q index is requested first (the query fragments, and K
    //      image 0 for the exponent reference), then the Q index itself, so that the three memory round trips of the
    //      prologue overlap instead of following one another. ------------------------------------------------------
    Geometry<G> ge;
    ge.init_rows(Hq, Hkv, aq.n_row_tiles, g, ordinal);
    const int x = ge.x, h = ge.h;
    FragOffsets<D> fo;
    fo.init(x, h);
    const unsigned char* head_images = aq.images + (size_t)ge.g * n_img_tiles * I::BYTES;
    const int wave = __builtin_amdgcn_readfirstlane(ge.wave), lane = threadIdx.x & 63;
    dma_image<I::K_BYTES / 1024>(head_images, rg.k[2], wave, lane);   // K image 0 into ring slot 2: the exponent reference comes from it

    // Q fragments: B operand of S^T = K Q^T, kept in registers for the whole loop
    bf16x8 qf[2][D / 16];
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
        const __bf16* qp = q_rows + ((size_t)min(ge.col_row[nb], R - 1) * Hq + ge.col_head[nb]) * D + 8 * h;
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) qf[nb][ks] = *reinterpret_cast<const bf16x8*>(qp + 16 * ks);
    }
    ge.init_positions(aq.q_index, R, n_img_tiles);
    const int n_kt = ge.n_kt;
    // this piece's key tiles [kb, ke): shares of ceil(n_kt / n_parts) tiles, so part 0 is never empty
    const int per_part = part < 0 ? n_kt : (n_kt + n_parts - 1) / n_parts;
    const int kb = part < 0 ? 0 : part * per_part, ke = min(n_kt, kb + per_part);
    const int part_words = half ? Part<D, false>::WORDS : Part<D, true>::WORDS;
    float* part_dst = part < 0 ? nullptr : partials + (((size_t)item * n_parts + part) * Hkv + g) * part_words + threadIdx.x;
    if (kb >= ke) {   // fewer key tiles than parts: this one adds nothing
        for (int r = 0; r < part_words; r += 256) part_dst[r] = 0.f;
        return;       // (the hardware waits for the outstanding copy before it retires the wave)
    }
    f32x16 o[D / 32][2];
#pragma unroll
    for (int md = 0; md < D / 32; ++md)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
            for (int v = 0; v < 16; ++v) o[md][nb][v] = 0.f;
    float lsum[2] = {0.f, 0.f};

    // K images kb and kb + 1 and V image kb land in LDS
    const unsigned char* first_image = head_images + (size_t)kb * I::BYTES;
    dma_image<I::K_BYTES / 1024>(first_image, rg.k[0], wave, lane);
    dma_image<I::V_BYTES / 1024>(first_image + I::K_BYTES, rg.vt[0], wave, lane);
    if (kb + 1 < n_kt) dma_image<I::K_BYTES / 1024>(first_image + I::BYTES, rg.k[1], wave, lane);
    {   // V ring slot 2 is read (against all-zero weights) by the very first step: it must hold finite numbers
        const u32x4 z = {0u, 0u, 0u, 0u};
        for (int i = threadIdx.x; i < I::V_BYTES / 16; i += 256) *reinterpret_cast<u32x4*>(&rg.vt[2][16 * i]) = z;
    }
    wait_dma();
    __syncthreads();

    // exponent reference of each column = the maximum of its logits over the visible ones of keys 0..31
    f32x16 s_a[2], s_b[2];
    qk_half<D>(rg.k[2], 0, qf, fo, s_a);
    float mref[2];
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
        float t = NEG_BIG;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int key = 8 * (v >> 2) + 4 * h + (v & 3);
            t = fmaxf(t, key <= ge.col_pos[nb] ? s_a[nb][v] : NEG_BIG);
        }
        t = fmaxf(t, __shfl_xor(t, 32));   // key 0 (held by the h = 0 lane) is visible to every row
        mref[nb] = t * scale_log2e;
    }
    __syncthreads();                                // ring slot 2 is free again before the loop copies into it
    if (kb > 0) qk_half<D>(rg.k[0], 0, qf, fo, s_a);   // logits of this part's first 32 keys (else: those above)
    Weights<SPLIT> pf_a, pf_b;
    pf_b.clear();

    // ---- tile loop ------------------------------------------------------------------------------------
    // Iteration kt: wait for the own direct-to-LDS copies issued one iteration ago, barrier (now K image kt+1
    // and V image kt are complete and visible, and nobody reads the slots of K image kt-1 / V image kt-2 any
    // more), issue the copies of K image kt+2 and V image kt+1 into those slots, and run two pipeline steps:
    //   step (kt, 0): weights of keys [64kt, 64kt+32)    | logits of (kt, 1) from K[kt]     | O += half (kt-1, 1), V[kt-1]
    //   step (kt, 1): weights of keys [64kt+32, 64kt+64) | logits of (kt+1, 0) from K[kt+1] | O += half (kt, 0),   V[kt]
    int k0 = 0, k1 = 1, k2 = 2;   // ring slots of K images kt, kt+1, kt+2; V images kt-1, kt, kt+1 sit in k2, k0, k1
    int kt = kb;
    const int plain_end = min(ge.n_plain, ke);
    for (; kt < plain_end; ++kt) {   // plain tiles: every key visible to every row; image kt+1 always exists
        if (kt > kb) {
            wait_dma();
            __syncthreads();
        }
        const unsigned char* nxt = head_images + (size_t)(kt + 1) * I::BYTES;
        if (kt + 2 < n_kt) dma_image<I::K_BYTES / 1024>(nxt + I::BYTES, rg.k[k2], wave, lane);
        dma_image<I::V_BYTES / 1024>(nxt + I::K_BYTES, rg.vt[k1], wave, lane);
        pipeline_step<D, SPLIT, false, true>(rg.k[k0], 1, rg.vt[k2], 1, fo, qf, s_a, s_b, pf_b, pf_a, o, lsum, mref, ge.col_pos,
                                   kt * KT, h, scale_log2e);
        pipeline_step<D, SPLIT, false, true>(rg.k[k1], 0, rg.vt[k0], 0, fo, qf, s_b, s_a, pf_a, pf_b, o, lsum, mref, ge.col_pos,
                                   kt * KT + 32, h, scale_log2e);
        const int t = k0; k0 = k1; k1 = k2; k2 = t;
    }
    for (; kt < ke; ++kt) {           // tiles that cross some row's own position
        if (kt > kb) {
            wait_dma();
            __syncthreads();
        }
        const unsigned char* nxt = head_images + (size_t)(kt + 1) * I::BYTES;
        if (kt + 2 < ke) dma_image<I::K_BYTES / 1024>(nxt + I::BYTES, rg.k[k2], wave, lane);
        if (kt + 1 < ke) dma_image<I::V_BYTES / 1024>(nxt + I::K_BYTES, rg.vt[k1], wave, lane);
        pipeline_step<D, SPLIT, true, true>(rg.k[k0], 1, rg.vt[k2], 1, fo, qf, s_a, s_b, pf_b, pf_a, o, lsum, mref, ge.col_pos,
                                  kt * KT, h, scale_log2e);
        if (kt + 1 < ke)
            pipeline_step<D, SPLIT, true, true>(rg.k[k1], 0, rg.vt[k0], 0, fo, qf, s_b, s_a, pf_a, pf_b, o, lsum, mref,
                                      ge.col_pos, kt * KT + 32, h, scale_log2e);
        else
            pipeline_step<D, SPLIT, true, false>(rg.k[k1], 0, rg.vt[k0], 0, fo, qf, s_b, s_a, pf_a, pf_b, o, lsum, mref,
                                       ge.col_pos, kt * KT + 32, h, scale_log2e);
        const int t = k0; k0 = k1; k1 = k2; k2 = t;
    }
    pv_half<D, SPLIT>(rg.vt[k2], 1, pf_b, fo, o);   // the last half: V image ke-1 now sits in slot k2

    if (part >= 0) {   // leave the partial result; attn_combine_kernel adds the parts, checks and stores
        if (!SPLIT && half) store_partial<D, false>(part_dst, o, lsum, mref); else store_partial<D, true>(part_dst, o, lsum, mref);
        return;
    }
    float l[2];
    if (!sums_overflowed<D>(o, lsum, l)) {
        store_output<G, D>(ge, o, l, mref, R, Hq, smem_raw, aq.out, aq.lse);
        return;
    }
    // the sums overflowed the fixed exponent reference (rare): the item again, with a running maximum
    __syncthreads();
    running_max_item<G, D, SPLIT>(aq, g, ordinal, Hq, Hkv, scale_log2e, smem_raw);
}

// blockIdx.x = ((query * max_row_tiles + ordinal) * n_parts + part) * Hkv + KV head.  n_parts = 1: every item whole.
// n_parts > 1 (few items: the chip would idle behind the longest ones): the key tiles of every item are
// dealt to n_parts workgroups in equal consecutive shares; items are launched longest first, so the pieces are too.
// Dynamic LDS: the larger of the K/V rings and the epilogue's staging.
template <int G, int D, bool SPLIT>
__global__ __launch_bounds__(256) void attn_fixed_ref_kernel(const AttnBatch batch, float* __restrict__ partials, int n_parts,
                                                             int half, int Hq, int Hkv, float scale_log2e) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    int t = (int)blockIdx.x;
    const int g = t % Hkv; t /= Hkv;
    const int part = t % n_parts; t /= n_parts;
    const int ordinal = t % batch.max_row_tiles, query = t / batch.max_row_tiles;
    const AttnQuery& aq = batch.q[query];
    if (ordinal >= aq.n_row_tiles) return;
    process_piece<G, D, SPLIT>(aq, g, ordinal, n_parts > 1 ? part : -1, n_parts, t, partials, half != 0, Hq, Hkv, scale_log2e, smem_raw);
}

// ---- combine: adds the parts of every item, then checks and stores like the fast path's own epilogue; on overflow
//      the item is recomputed with a running maximum.  One workgroup per (item, 32 dims of the output): the pass is bound by
//      the latency of its loads, and a workgroup per item left a short prompt's 24 items in eight parts to 24 compute units
//      (24 us; now 7.5; the offline stage's 128 items in two parts 13.6 -> 7.6).  A column's sum is added up by every slice; a slice that sees an overflow computes and stores its own dims.
//      grid.x = ((query * max_row_tiles + ordinal) * D / 32 + slice) * Hkv + KV head, LDS = max(epilogue staging, one image).
template <int G, int D, bool SPLIT, bool F32>
__global__ __launch_bounds__(256, 2) void attn_combine_kernel(const AttnBatch batch, const float* __restrict__ partials,
                                                              int n_parts, int Hq, int Hkv, float scale_log2e) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    int t = (int)blockIdx.x;
    const int g = t % Hkv; t /= Hkv;
    const int md = t % (D / 32);
    const int item = t / (D / 32);
    const int ordinal = item % batch.max_row_tiles;
    const AttnQuery& aq = batch.q[item / batch.max_row_tiles];
    if (ordinal >= aq.n_row_tiles) return;
    {
        using P = Part<D, F32>;
        constexpr int OW = P::O_WORDS, SW = F32 ? 16 : 8;   // words of a part, of a slice of a column block
        constexpr int AHEAD = 4;                            // parts whose loads are in flight together
        const uint32_t* p0 = reinterpret_cast<const uint32_t*>(partials + ((size_t)item * n_parts * Hkv + g) * P::WORDS) + threadIdx.x;
        const size_t part_stride = (size_t)Hkv * P::WORDS;
        f32x16 acc[2];
        float lsum[2] = {0.f, 0.f}, mref[2];
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) {
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[nb][v] = 0.f;
            mref[nb] = __uint_as_float(p0[(OW + 2 + nb) * 256]);   // part 0 is never empty; every part derives the same reference
        }
        auto add = [&](int first, auto count) {
            constexpr int N = decltype(count)::value;
            uint32_t w[N][2][SW], tail[N][2][2];
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const uint32_t* pp = p0 + (first + i) * part_stride;
#pragma unroll
                for (int nb = 0; nb < 2; ++nb) {
#pragma unroll
                    for (int j = 0; j < SW; ++j) w[i][nb][j] = pp[(nb * (OW / 2) + md * SW + j) * 256];
                    tail[i][nb][0] = pp[(OW + nb) * 256];
                    tail[i][nb][1] = F32 ? 0u : pp[(OW + 4 + nb) * 256];
                }
            }
#pragma unroll
            for (int i = 0; i < N; ++i)
#pragma unroll
                for (int nb = 0; nb < 2; ++nb) {
                    const int e = (int)tail[i][nb][1];
#pragma unroll
                    for (int v = 0; v < 16; v += 2) {
                        if constexpr (F32) {
                            acc[nb][v] += __uint_as_float(w[i][nb][v]);
                            acc[nb][v + 1] += __uint_as_float(w[i][nb][v + 1]);
                        } else {
                            const f16x2 h = __builtin_bit_cast(f16x2, w[i][nb][v / 2]);
                            acc[nb][v] += __builtin_ldexpf((float)h[0], e);
                            acc[nb][v + 1] += __builtin_ldexpf((float)h[1], e);
                        }
                    }
                    lsum[nb] += __uint_as_float(tail[i][nb][0]);
                }
        };
        int part = 0;
        for (; part + AHEAD <= n_parts; part += AHEAD) add(part, std::integral_constant<int, AHEAD>{});
        if (part + 2 <= n_parts) { add(part, std::integral_constant<int, 2>{}); part += 2; }
        if (part < n_parts) add(part, std::integral_constant<int, 1>{});
        Geometry<G> ge;
        ge.init(aq.q_index, aq.R, Hq, Hkv, aq.n_row_tiles, aq.n_img_tiles, g, ordinal);
        float l[2];
        bool bad = false;
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) {
            l[nb] = lsum[nb] + __shfl_xor(lsum[nb], 32);
            float chk = l[nb];
#pragma unroll
            for (int v = 0; v < 16; ++v) chk += fabsf(acc[nb][v]);
            bad = bad || !(chk < INFINITY) || !(l[nb] > 0.f);
        }
        if (!__syncthreads_or(bad ? 1 : 0)) {
            store_slice<G, D>(ge, acc, md, l, mref, aq.R, Hq, smem_raw, aq.out, aq.lse);
            return;
        }
    }
    // the sums overflowed the fixed exponent reference (rare): the item again, with a running maximum
    __syncthreads();
    running_max_item<G, D, SPLIT>(aq, g, ordinal, Hq, Hkv, scale_log2e, smem_raw, md);
}

// ---- all items with the running maximum (FR_ATTN_SOFTMAX_RUNNING_MAX) -------------------------------------
template <int G, int D, bool SPLIT>
__global__ __launch_bounds__(256) void attn_running_max_kernel(const AttnBatch batch, int Hq, int Hkv,
                                                               float scale_log2e) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    BlockWork bw;
    bw.init(batch.max_row_tiles, Hkv);
    const AttnQuery& aq = batch.q[bw.query];
    if (bw.ordinal >= aq.n_row_tiles) return;
    running_max_item<G, D, SPLIT>(aq, bw.g, bw.ordinal, Hq, Hkv, scale_log2e, smem_raw);
}

// Where one query's packing pass leaves its results.
struct QueryScratch {
    int32_t* store_row_map;   // [L], shared-store queries only
    int32_t* chunk_id_map;    // [L], shared-store queries only
    unsigned char* images;
    size_t images_bytes;
};

template <int D>
constexpr size_t LDS_FAST = std::max(sizeof(Rings<D>), Img<D>::EPILOGUE_LDS);
template <int D>
constexpr size_t LDS_SAFE = std::max((size_t)Img<D>::BYTES, Img<D>::EPILOGUE_LDS);

// Raises the kernels' dynamic LDS limit, once per process (C++ initialises a function-local static exactly once,
// also when several host threads arrive together).
template <int G, int D, bool SPLIT>
hipError_t set_kernel_attributes() {
    static const hipError_t once = [] {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_fixed_ref_kernel<G, D, SPLIT>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS_FAST<D>);
        if (e != hipSuccess) return e;
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_combine_kernel<G, D, SPLIT, true>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS_SAFE<D>);
        if (e != hipSuccess) return e;
        if constexpr (!SPLIT) {
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_combine_kernel<G, D, SPLIT, false>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS_SAFE<D>);
            if (e != hipSuccess) return e;
        }
        return hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_running_max_kernel<G, D, SPLIT>),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS_SAFE<D>);
    }();
    return once;
}

// Packing pass of one query: tile images of its effective K/V into sc.images; fills the query's line of the table.
template <int D>
hipError_t pack_query(const Shape& s, const void* q_rows, const int32_t* q_index, int R, const void* k_cache,
                      const void* v_cache, int64_t L, const void* k_new, const void* v_new, void* out, float* lse,
                      const QueryScratch& sc, const SharedStoreArgs* shared, bool writeback, AttnQuery* aq, hipStream_t st) {
    const int TR = 4 * (64 / s.G);   // token rows per workgroup
    const int n_row_tiles = (R + TR - 1) / TR;
    const int n_img_tiles = (int)((L + KT - 1) / KT);
    const dim3 block(256);
    if ((size_t)n_img_tiles * s.Hkv * Img<D>::BYTES > sc.images_bytes) return hipErrorInvalidValue;
    if (shared == nullptr) {
        if (writeback)
            pack_kv_images_kernel<D, true><<<dim3(n_img_tiles, s.Hkv), block, 0, st>>>(
                (const __bf16*)k_cache, (const __bf16*)v_cache, (int)L, (const __bf16*)k_new, (const __bf16*)v_new, q_index, R,
                s.Hkv, n_img_tiles, sc.images);
        else
            pack_kv_images_kernel<D, false><<<dim3(n_img_tiles, s.Hkv), block, 0, st>>>(
                (const __bf16*)k_cache, (const __bf16*)v_cache, (int)L, (const __bf16*)k_new, (const __bf16*)v_new, q_index, R,
                s.Hkv, n_img_tiles, sc.images);
    } else if constexpr (D == 128) {   // k_cache / v_cache are the shared chunk store
        ChunkRows rows;
        int max_len = (int)L - shared->ct.off[shared->ct.n];
        for (int c = 0; c < shared->ct.n; ++c) {
            rows.row0[c] = shared->store_row0[c];
            max_len = std::max(max_len, shared->ct.off[c + 1] - shared->ct.off[c]);
        }
        prompt_map_kernel<<<dim3(std::max(1, (max_len + 255) / 256), shared->ct.n + 1), block, 0, st>>>(
            shared->ct, rows, (int)L, sc.store_row_map, sc.chunk_id_map);
        if (s.rope_layout == FR_ROPE_INTERLEAVED)
            pack_kv_images_shared_kernel<FR_ROPE_INTERLEAVED><<<dim3(n_img_tiles, s.Hkv), block, 0, st>>>(
                (const __bf16*)k_cache, (const __bf16*)v_cache, sc.store_row_map, sc.chunk_id_map, shared->table, (int)L,
                (const __bf16*)k_new, (const __bf16*)v_new, q_index, R, s.Hkv, n_img_tiles, sc.images);
        else
            pack_kv_images_shared_kernel<FR_ROPE_HALF><<<dim3(n_img_tiles, s.Hkv), block, 0, st>>>(
                (const __bf16*)k_cache, (const __bf16*)v_cache, sc.store_row_map, sc.chunk_id_map, shared->table, (int)L,
                (const __bf16*)k_new, (const __bf16*)v_new, q_index, R, s.Hkv, n_img_tiles, sc.images);
    } else {
        return hipErrorInvalidValue;   // (such shapes gather the query's keys and values first)
    }
    aq->q_rows = (const __bf16*)q_rows;
    aq->q_index = q_index;
    aq->images = sc.images;
    aq->out = (__bf16*)out;
    aq->lse = lse;
    aq->R = R;
    aq->n_row_tiles = n_row_tiles;
    aq->n_img_tiles = n_img_tiles;
    aq->pad = 0;
    return hipGetLastError();
}

// Launches the key-tile loop; with a live timer its event pair rides on the kernel's own dispatch (start and end of its
// execution), so the stream carries no extra marker packets and the kernels before and after it are not held up.
template <int G, int D, bool SPLIT>
void launch_tile_loop(const AttnBatch& batch, dim3 grid, float* partials, int n_parts, bool half, const Shape& s, float scale_log2e,
                      KernelTimer* timer, bool timed, hipStream_t st) {
    if (timed) {
        const int slot = (int)(timer->n_recorded % timer->n_slots);
        hipExtLaunchKernelGGL((attn_fixed_ref_kernel<G, D, SPLIT>), grid, dim3(256), (uint32_t)LDS_FAST<D>, st, timer->start[slot],
                              timer->stop[slot], 0u, batch, partials, n_parts, (int)half, s.Hq, s.Hkv, scale_log2e);
        ++timer->n_recorded;
    } else {
        attn_fixed_ref_kernel<G, D, SPLIT><<<grid, dim3(256), LDS_FAST<D>, st>>>(batch, partials, n_parts, (int)half, s.Hq, s.Hkv, scale_log2e);
    }
}

// Parts per item of a one-query launch of `items` (row tile, KV head) items over n_img_tiles key tiles.  With few items
// the chip would idle behind the longest ones (rows ascend by position: the question rows' tiles walk the whole prompt),
// so every item's key tiles are dealt to several workgroups.  Measured on a 17k-token prompt (256 compute units, one
// workgroup each): two parts pay up to about 400 items (recompute ratios up to 15 %; at 30 %, 680 items, the partial
// results' traffic and the combine pass cost more than the balance gains); below half a workgroup per compute unit more
// parts pay until there is about one piece per compute unit (question-only prefill, 64 items: 4 parts, 0.24 -> 0.17 ms);
// in between two parts stay best (168 items at 5 %, 128 items of the offline stage: three or four parts lose 3-15 %).
// Short prompts (under 32 key tiles) are cut only below half a workgroup per compute unit, down to two tiles a part: a tile
// is 1.8 us of a workgroup, the combine pass 7.5 us (920 tokens, 24 items of up to 15 tiles: 31 us whole, 14 + 7.5 in eight parts).
int choose_parts(int split_mode, int items, int n_img_tiles, int n_cu, size_t part_bytes, size_t partials_bytes) {
    int parts = 1;
    if (split_mode == FR_ATTN_SPLIT_ON) parts = 2;
    if (split_mode == FR_ATTN_SPLIT_AUTO) {
        if (2 * items <= n_cu) parts = std::min({ATTN_MAX_PARTS, n_cu / std::max(items, 1), (n_img_tiles + 1) / 2});
        if (n_img_tiles >= 32 && items <= ATTN_SPLIT_AUTO_ITEMS) parts = std::max(parts, 2);
    }
    while (parts > 1 && (size_t)items * parts * part_bytes > partials_bytes) --parts;
    return parts;
}

// Half-precision partial results: only for a single query of a long prompt (32 key tiles and more) whose weights are plain
// bf16, where 400 items in two parts would otherwise move 2 x 108 MB of partial sums (combine pass 21.1 us, 15.5 us in half
// precision).  Short prompts, batches and more than four parts, a few hundred pieces at most, keep all 32 bits
// (6730 tokens, 32 items: 2.174e-3 off float64 in eight parts, 2.184e-3 in four of half precision; the layer takes 163 us, 159 in
// eight of half precision, 183 in four).
constexpr int HALF_MAX_PARTS = 4;
template <bool SPLIT>
bool half_parts(int n_img_tiles) { return !SPLIT && n_img_tiles >= 32; }
template <int D>
size_t part_bytes(bool half) { return (half ? Part<D, false>::WORDS : Part<D, true>::WORDS) * sizeof(float); }

// Packed queries -> attention launches: tile loop (+ combine pass), or the running-maximum kernel.
template <int G, int D, bool SPLIT>
hipError_t launch_packed(const Shape& s, const AttnBatch& batch, int n_parts, bool half, const Workspace& ws, int mode,
                         KernelTimer* timer, hipStream_t st) {
    const float scale_log2e = (1.0f / sqrtf((float)s.d)) * 1.4426950408889634f;
    const dim3 grid(batch.max_row_tiles * batch.n * s.Hkv);
    if (mode == FR_ATTN_SOFTMAX_RUNNING_MAX) {   // every item with the running maximum
        attn_running_max_kernel<G, D, SPLIT><<<grid, dim3(256), LDS_SAFE<D>, st>>>(batch, s.Hq, s.Hkv, scale_log2e);
        return hipGetLastError();
    }
    const bool timed = timer != nullptr && timer->n_slots > 0;
    launch_tile_loop<G, D, SPLIT>(batch, dim3(grid.x * n_parts), ws.attn_partials, n_parts, half, s, scale_log2e, timer, timed, st);
    if (n_parts > 1) {   // adds the parts, stores, and recomputes the items whose sums overflowed
        if constexpr (!SPLIT) {
            if (half) {
                attn_combine_kernel<G, D, SPLIT, false><<<dim3(grid.x * (D / 32)), dim3(256), LDS_SAFE<D>, st>>>(batch, ws.attn_partials, n_parts, s.Hq, s.Hkv, scale_log2e);
                return hipGetLastError();
            }
        }
        attn_combine_kernel<G, D, SPLIT, true><<<dim3(grid.x * (D / 32)), dim3(256), LDS_SAFE<D>, st>>>(batch, ws.attn_partials, n_parts, s.Hq, s.Hkv, scale_log2e);
    }
    return hipGetLastError();
}

template <int G, int D, bool SPLIT>
hipError_t launch(const Shape& s, const void* q_rows, const int32_t* q_index, int R, const void* k_cache,
                  const void* v_cache, int64_t L, const void* k_new, const void* v_new, void* out, float* lse,
                  const Workspace& ws, int mode, int split_mode, const SharedStoreArgs* shared, KernelTimer* timer,
                  bool writeback, hipStream_t st) {
    hipError_t e = set_kernel_attributes<G, D, SPLIT>();
    if (e != hipSuccess) return e;
    const QueryScratch sc{ws.store_row_map, ws.chunk_id_map, ws.kv_images, ws.kv_images_bytes};
    AttnBatch batch;
    batch.n = 1;
    e = pack_query<D>(s, q_rows, q_index, R, k_cache, v_cache, L, k_new, v_new, out, lse, sc, shared, writeback, &batch.q[0], st);
    if (e != hipSuccess) return e;
    batch.max_row_tiles = batch.q[0].n_row_tiles;
    bool half = half_parts<SPLIT>(batch.q[0].n_img_tiles);
    auto parts_of = [&](bool h) {
        return choose_parts(split_mode, batch.q[0].n_row_tiles * s.Hkv, batch.q[0].n_img_tiles, ws.n_cu, part_bytes<D>(h),
                            ws.attn_partials_bytes);
    };
    int n_parts = parts_of(half);
    if (half && n_parts > HALF_MAX_PARTS) {   // 32 bits, or as many parts as half precision may have
        const int full = parts_of(false);
        half = full <= HALF_MAX_PARTS;
        n_parts = half ? HALF_MAX_PARTS : full;
    }
    return launch_packed<G, D, SPLIT>(s, batch, n_parts, half, ws, mode, timer, st);
}

template <int G, int D, bool SPLIT>
hipError_t launch_shared_batch(const Shape& s, int n, const SharedBatchQuery* qs, const void* k_store, const void* v_store,
                               const Workspace& ws, int mode, int split_mode, KernelTimer* timer, hipStream_t st) {
    hipError_t e = set_kernel_attributes<G, D, SPLIT>();
    if (e != hipSuccess) return e;
    AttnBatch batch;
    batch.n = n;
    batch.max_row_tiles = 0;
    const size_t slot = part_bytes<D>(false);   // partial results of a batch stay fp32
    int n_parts = 1;
    for (int i = 0; i < n; ++i) {
        const SharedBatchQuery& q = qs[i];
        const QueryScratch sc{q.store_row_map, q.chunk_id_map, q.images, q.images_bytes};
        e = pack_query<D>(s, q.q_rows, q.q_index, q.R, k_store, v_store, q.L, q.k_new, q.v_new, q.out, q.lse, sc, &q.shared,
                          false, &batch.q[i], st);
        if (e != hipSuccess) return e;
        batch.max_row_tiles = std::max(batch.max_row_tiles, batch.q[i].n_row_tiles);
        n_parts = std::max(n_parts, choose_parts(split_mode, batch.q[i].n_row_tiles * s.Hkv, batch.q[i].n_img_tiles, ws.n_cu,
                                                 slot, ws.attn_partials_bytes));
    }
    // A batch of queries usually fills the chip by itself: every item whole, one workgroup each.  Up to a quarter of a
    // workgroup per compute unit it is cut like its queries would be alone; in between like one query of as many items.
    const int items = batch.max_row_tiles * n * s.Hkv;
    int tiles = 0;
    for (int i = 0; i < n; ++i) tiles = std::max(tiles, batch.q[i].n_img_tiles);
    if (4 * items > ws.n_cu) n_parts = choose_parts(split_mode, items, tiles, ws.n_cu, slot, ws.attn_partials_bytes);
    while (n_parts > 1 && (size_t)items * n_parts * slot > ws.attn_partials_bytes) --n_parts;
    return launch_packed<G, D, SPLIT>(s, batch, n_parts, false, ws, mode, timer, st);
}

}  // namespace

// Shapes with an instance of their own; the others (any group size up to 64, head_dim 64 too) run the kernels whose group
// size is an argument and whose weights are split (Weights).  The group size enters the prologue and the epilogue only.
// 28 query / 4 KV heads over a 17k-token prompt, 2970 rows: 0.80 ms for the tile loop (387 GFLOP as 774 GFLOP of matrix
// instructions: 0.97 PFLOP/s) + 0.022 + 0.018 ms; one wave per (row, head) on the vector ALU took 50.5 ms.
static bool own_instance(const Shape& s) { return s.d == 128 && (s.G == 1 || s.G == 2 || s.G == 4 || s.G == 8); }

// Partial results of a launch in parts: one slot per piece.
size_t attn_mfma_partials_bytes(const Shape& s, int64_t max_tokens) {
    const int64_t tr = 4 * (64 / s.G);   // token rows per workgroup
    const int64_t items = std::min<int64_t>(((max_tokens + tr - 1) / tr) * s.Hkv, ATTN_SPLIT_AUTO_ITEMS);
    // two parts of the most items that are split without being asked (32-bit words unless they may be half_parts), and up
    // to eight parts of few items (about one piece per compute unit), always in 32 bits
    const size_t full = (s.d == 128 ? Part<128, true>::WORDS : Part<64, true>::WORDS) * sizeof(float);
    const size_t half = own_instance(s) ? Part<128, false>::WORDS * sizeof(float) : full;
    return std::max((size_t)(2 * items) * half, (size_t)std::min<int64_t>(ATTN_MAX_PARTS * items, 256) * full);
}

bool attn_mfma_supported(const Shape& s) { return s.dtype == FR_BF16 && s.G <= 64; }
bool attn_mfma_store_supported(const Shape& s) { return s.dtype == FR_BF16 && own_instance(s); }

hipError_t launch_attn_mfma(const Shape& s, const void* q_rows, const int32_t* q_index, int R, const void* k_cache,
                            const void* v_cache, int64_t L, const void* k_new, const void* v_new, void* out, float* lse,
                            const Workspace& ws, int mode, int split_mode, const SharedStoreArgs* shared,
                            KernelTimer* timer, bool writeback, hipStream_t st) {
    if (R == 0) return hipSuccess;
    if (!own_instance(s)) {
        if (s.d == 64)
            return launch<0, 64, true>(s, q_rows, q_index, R, k_cache, v_cache, L, k_new, v_new, out, lse, ws, mode, split_mode, shared, timer, writeback, st);
        return launch<0, 128, true>(s, q_rows, q_index, R, k_cache, v_cache, L, k_new, v_new, out, lse, ws, mode, split_mode, shared, timer, writeback, st);
    }
    switch (s.G) {
        case 1: return launch<1, 128, false>(s, q_rows, q_index, R, k_cache, v_cache, L, k_new, v_new, out, lse, ws, mode, split_mode, shared, timer, writeback, st);
        case 2: return launch<2, 128, false>(s, q_rows, q_index, R, k_cache, v_cache, L, k_new, v_new, out, lse, ws, mode, split_mode, shared, timer, writeback, st);
        case 4: return launch<4, 128, false>(s, q_rows, q_index, R, k_cache, v_cache, L, k_new, v_new, out, lse, ws, mode, split_mode, shared, timer, writeback, st);
        default: return launch<8, 128, false>(s, q_rows, q_index, R, k_cache, v_cache, L, k_new, v_new, out, lse, ws, mode, split_mode, shared, timer, writeback, st);
    }
}

size_t attn_mfma_images_bytes(const Shape& s, int64_t L) {
    return (size_t)((L + KT - 1) / KT) * s.Hkv * (s.d == 128 ? Img<128>::BYTES : Img<64>::BYTES);
}

hipError_t launch_attn_mfma_shared_batch(const Shape& s, int n, const SharedBatchQuery* qs, const void* k_store,
                                         const void* v_store, const Workspace& ws, int mode, int split_mode, KernelTimer* timer,
                                         hipStream_t st) {
    if (n <= 0) return hipSuccess;
    if (n > ATTN_MAX_BATCH) return hipErrorInvalidValue;
    switch (s.G) {
        case 1: return launch_shared_batch<1, 128, false>(s, n, qs, k_store, v_store, ws, mode, split_mode, timer, st);
        case 2: return launch_shared_batch<2, 128, false>(s, n, qs, k_store, v_store, ws, mode, split_mode, timer, st);
        case 4: return launch_shared_batch<4, 128, false>(s, n, qs, k_store, v_store, ws, mode, split_mode, timer, st);
        default: return launch_shared_batch<8, 128, false>(s, n, qs, k_store, v_store, ws, mode, split_mode, timer, st);
    }
}

}  // namespace fr
