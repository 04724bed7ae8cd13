// Sparse prefill attention (eq. 9, Sec. 4.3) on the gfx950 matrix cores: bf16, head_dim 64 or 128, up to 64 query heads
// per KV head.
//
// Work split.  One workgroup owns one KV head and a tile of consecutive Q-index rows in four row groups of 64 "query columns" =
// floor(64 / G) token rows x the G query heads that share the KV
// head (a group size that does not divide 64 leaves a few columns idle: one of 64 at 7, four at 5), so every K/V tile staged in LDS is reused by the whole grouped-query group and by all
// row groups.  The fast kernel has two waves per row group (and per SIMD), each with half of the keys of every tile.  Rows are sorted by
// position, so a tile needs keys 0 .. (position of its last row); tiles are issued longest first.
//
// Orientation.  The kernel computes the transposed products S^T = K Q^T and O^T = V^T P^T with
// v_mfma_f32_16x16x32_bf16:
//   * keys run along the M (register) dimension of S^T and query columns along N (lanes), so the
//     softmax statistics of a query column live in four lanes (x, x + 16, x + 32, x + 48), and in-lane during the loop;
//   * the fp32 accumulators of two S^T blocks (32 keys) are, after conversion to bf16, exactly the B-operand
//     layout of the second product (contraction over keys), so P never leaves registers;
//   * V is transposed once per (KV head, key tile) by the packing pre-pass (4 keys x 8 dims per lane,
//     repacked with byte permutes), so the A operand of the second product is a 16-byte LDS read.
// The key order inside every block of 32 keys is permuted identically in P^T and V^T (key_slot); a contraction does not care
// about the order of its terms.
//
// What bounds it.  The chip's power: matrix instructions alone, on normally distributed operands in registers, sustain 1.78 PFLOP/s as
// 32 x 32 x 16 and 1.98 as 16 x 16 x 32 (2.45 either on zeros), because a contraction of 32 reads and writes its accumulators half as often; and 2 - 3 % more where
// neighbouring instructions share an operand.  With one wave per SIMD and 32 x 32 tiles (four waves, vector work between the matrix
// instructions of the same wave) the loop took 20 % more cycles at a higher clock; two waves per SIMD with 32 x 32 tiles needed the fewest
// cycles (matrix pipe busy 73 %) at 1.63 GHz and were 4 % faster; with 16 x 16 tiles 71 % at 1.93 GHz.  Measured on one box, 32 / 8 heads:
// 2970 of 16896 rows 432 -> 371 us, all rows 1974 -> 1661 us (1.18 -> 1.41 PFLOP/s); 28 / 4 heads with split weights 709 -> 581 us.
// Raising the priority of either phase changes nothing; query fragments from LDS instead of registers cost 1 % for each
// quarter of them (power again), so as many stay in registers as the loop has room for.
//
// Softmax.  exp(s - m) / sum exp(s - m) does not depend on m, and fp32 / bf16 leave about 2^127 of
// headroom, so the fast kernel fixes each query column's reference m once (the maximum over the
// column's first 32 visible keys) and never rescales: the tile loop holds no maximum, no
// comparison and no branch on values.  If a later logit exceeds the reference by more than that headroom
// the sums overflow to inf; the workgroup then finds the largest logit of its keys in a pass of its own and does the piece again.
//
// K/V tile images.  Every row tile of a KV head walks the same K/V stream (47 row tiles per head at 17k
// tokens / 15 %), so the work that does not depend on the rows is done once, by a packing pre-pass: for each
// (KV head, 64-key tile) it resolves stale / fresh rows (key j comes from k_new/v_new when its token is in the Q index, and
// from the cache otherwise: the cache is never written and stale rows are
// never read), transposes V and writes an image (32 KB at head_dim 128) that is byte
// for byte what the attention kernels want in LDS.  The fast kernel's tile loop then stages a tile with direct-to-LDS
// copies: no lookups, no pointer selects, no permutes, no address arithmetic, no staging registers.
//
// What a row does not see.  A weight of 0 does not take a NaN or an infinity out of a matrix product.  Positions behind the last
// row of the Q index may hold anything: they are not read.  A value that is not finite and that only some rows of an item see makes the
// sums of the others NaN, which the overflow check finds; the second go then keeps such values apart.
#include "fr_internal.hpp"
#include "k_rotate.hpp"

#include <hip/hip_ext.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace fr {

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

constexpr int KT = 64;           // keys per tile
constexpr float NEG_BIG = -1.0e30f;
constexpr float ITEM_DONE = INFINITY;   // in the place of a half-precision part's reference: its item has been stored

// Tile image = [K image][V^T image], 16 KB each at head_dim 128, 8 KB at 64.  Both are stored as the matrix operands read them: in
// planes of 16 bytes per row,
//   K image:   plane = 16-byte vector (8 dims) of the head row, row = key;
//   V^T image: plane = eight key slots (slot order see key_slot), row = dim.
// A fragment (lane = row x, quarter kg) is 16 bytes of plane 4 ks + kg (K) or 4 half + kg (V^T).  Planes are multiples of 256 bytes: any
// 16 lanes that the LDS serves together hold 16 different rows mod 16, so 16 different 16-byte bank groups, whichever quarters they are.
// Every fragment address is base + constant.
template <int D>
struct Img {
    static constexpr int K_PLANE = KT * 16, V_PLANE = D * 16;
    static constexpr int BLOCK = 16 * 16;                             // from one block of 16 rows to the next
    static constexpr int K_BYTES = D / 8 * K_PLANE, V_BYTES = KT / 8 * V_PLANE;
    static constexpr int BYTES = K_BYTES + V_BYTES;
    static constexpr int NK = D / 32;        // matrix steps over the dims of a logit
    static constexpr int MD = D / 16;        // 16-dim blocks of the output
    static constexpr int O_PITCH = D + 8;    // bf16 elements per output row in the epilogue's LDS staging
    static constexpr size_t EPILOGUE_LDS = 4 * 64 * O_PITCH * sizeof(__bf16);   // four waves x [64 columns][d] bf16
    static_assert(K_BYTES == V_BYTES && K_BYTES % (8 * 1024) == 0, "the fast kernel's copies");
};
// Inside every block of 32 keys the order is [0-3, 16-19, 4-7, 20-23, 8-11, 24-27, 12-15, 28-31]: the order in which the accumulator
// layout of S^T hands the keys to the second product.  Slot of key t (0..63) of a tile:
__device__ __forceinline__ int key_slot(int t) { return (t & 32) + 8 * ((t >> 2) & 3) + 4 * ((t >> 4) & 1) + (t & 3); }
constexpr int NC = 4;            // blocks of 16 query columns per wave
constexpr int FAST_WAVES = 8;    // of the fast kernel

// LDS of the fast kernel: rings of K and V^T images (see its tile loop) and the part of the query fragments that does not stay in
// registers, as [row group][column block][matrix step][lane]: both waves of a row group read the same 16 bytes per lane.
template <int D, bool SPLIT>
struct __attribute__((aligned(16))) FastLds {
    static constexpr int NK = Img<D>::NK;
    static constexpr int QR = D == 64 ? NK : SPLIT ? 1 : 3;   // matrix steps whose query fragments stay in registers
    static constexpr int QL = NK - QR;                        // and those that come from LDS
    unsigned char k[3][Img<D>::K_BYTES];
    unsigned char vt[3][Img<D>::V_BYTES];
    unsigned char q[QL > 0 ? 4 * QL * NC * 1024 : 16];
    int pos[4][64];                                           // positions of the row groups' columns (masked tiles)
    float ref[FAST_WAVES][64];                                // the waves' largest logits (EXACT)
};

__device__ __forceinline__ uint32_t perm_lo(uint32_t a, uint32_t b) {  // (a.lo16, b.lo16) -> a in low half
    return __builtin_amdgcn_perm(b, a, 0x05040100u);
}
__device__ __forceinline__ uint32_t perm_hi(uint32_t a, uint32_t b) {  // (a.hi16, b.hi16)
    return __builtin_amdgcn_perm(b, a, 0x07060302u);
}

// ---- what a lane knows about its workgroup, wave and four query columns ---------------------------
// G: query heads per KV head; 0 = known at run time only (group sizes without an instance of their own).
template <int G>
struct Geometry {
    int heads, trw;                      // query heads per KV head, token rows per wave
    int g, tile, row0;
    int x, kg, wave;                     // column inside a block, quarter of the keys (of the dims), row group
    int col_row[NC], col_head[NC], col_pos[NC];
    int wp_max;    // no key beyond it is visible to any row of this wave
    int n_kt;      // key tiles the workgroup walks
    int n_plain;   // leading tiles whose keys are visible to every row of the workgroup

    // ordinal counts the row tiles of a query from the longest one; ordinal < n_row_tiles
    __device__ __forceinline__ void init(const int32_t* __restrict__ q_index, int R, int Hq, int Hkv, int n_row_tiles,
                                         int n_img_tiles, int g_, int ordinal) {
        init_rows(Hq, Hkv, n_row_tiles, g_, ordinal);
        init_positions(q_index, R, n_img_tiles);
    }
    // The part that does not read the Q index: which rows and heads the lane's columns are.
    __device__ __forceinline__ void init_rows(int Hq, int Hkv, int n_row_tiles, int g_, int ordinal) {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));   // (opaque: what is formed from it again later need not be kept meanwhile)
        const int lane = tid & 63;
        heads = G > 0 ? G : Hq / Hkv;
        trw = G > 0 ? 64 / (G > 0 ? G : 1) : 64 / heads;
        wave = (tid >> 6) & 3;                               // (the fast kernel has two waves per row group)
        x = lane & 15;
        kg = lane >> 4;
        g = g_;
        tile = n_row_tiles - 1 - ordinal;                   // longest tiles first
        row0 = tile * 4 * trw;
#pragma unroll
        for (int nb = 0; nb < NC; ++nb) {
            const int col = 16 * nb + x;
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
        for (int nb = 0; nb < NC; ++nb) col_pos[nb] = q_index[min(col_row[nb], R - 1)];
        const int p_first = q_index[row0];                   // rows ascend: every key <= p_first is visible to all
        const int p_max = q_index[min(R, row0 + 4 * trw) - 1];    // the workgroup's furthest key
        wp_max = q_index[min(row0 + wave * trw + trw, R) - 1];   // a wave past the end copies the last row
        n_kt = __builtin_amdgcn_readfirstlane(min(p_max / KT + 1, n_img_tiles));
        n_plain = __builtin_amdgcn_readfirstlane(min((p_first + 1) / KT, n_kt - 1));
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

// ---- packing pre-pass: grid (key tiles x KV heads) ---------------------------------------------------------
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
    // Staged in LDS with the rows of a plane permuted, so that neither the writes (a key row's vectors, the dims of eight-dim
    // groups) nor the reads (a plane's rows) meet in one bank group: row r of K plane v at r ^ (v & 15), of V^T planes at r ^ ((r >> 3) & 7).
    using I = Img<D>;
    const int tid = threadIdx.x;
#pragma unroll
    for (int i = 0; i < PackShare<D>::KI; ++i)
        *reinterpret_cast<u32x4*>(&img[ps.vec * I::K_PLANE + 16 * ((ps.key + (256 / PackShare<D>::NV) * i) ^ ps.vec)]) = kreg[i];
    if (ps.has_v) {
        const int slot = key_slot(4 * ps.key);   // the 4 keys of this lane occupy slots slot .. slot + 3
        unsigned char* vt = img + I::K_BYTES + (slot >> 3) * I::V_PLANE + 2 * (slot & 7);
#pragma unroll
        for (int c = 0; c < 4; ++c) {   // dims 8 vec + 2c and + 2c + 1: gather the 4 keys of each
            u32x2 lo, hi;
            lo[0] = perm_lo(vreg[0][c], vreg[1][c]);
            lo[1] = perm_lo(vreg[2][c], vreg[3][c]);
            hi[0] = perm_hi(vreg[0][c], vreg[1][c]);
            hi[1] = perm_hi(vreg[2][c], vreg[3][c]);
            const int d0 = 8 * ps.vec + 2 * c, d1 = d0 + 1;
            *reinterpret_cast<u32x2*>(vt + 16 * (d0 ^ (ps.vec & 7))) = lo;
            *reinterpret_cast<u32x2*>(vt + 16 * (d1 ^ (ps.vec & 7))) = hi;
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < I::BYTES / 4096; ++i) {
        const int at = i * 4096 + tid * 16, r = at >> 4;
        const int perm = at < I::K_BYTES ? (at / I::K_PLANE) & 15 : (r >> 3) & 7;
        *reinterpret_cast<u32x4*>(dst + at) = *reinterpret_cast<const u32x4*>(&img[at ^ (16 * perm)]);
    }
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
    const int kt = blockIdx.x / Hkv, g = blockIdx.x % Hkv;   // as in the attention kernels: the workgroups of a KV head on one XCD
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

// Prompt position -> (store row, chunk) for the packing kernel, so that it needs no search and no dependent loads, and
// the chunks' (cos, sin) rows, in one launch: grid (position tiles of the longest chunk, chunks + 1); the extra y index
// covers the positions behind the context (no store row: -1).  A query's chunk tables fill most of the 4 KB of kernel
// arguments, so a batch launches this once per query
// (a kernel for the rotations and one for the maps: 3 + 2 us and a gap more per query; one launch 3 us).
__global__ __launch_bounds__(256) void prompt_tables_kernel(ChunkTable ct, ChunkRows rows, ChunkDeltas deltas, int L, int half_d,
                                                            const double* __restrict__ theta, float2* __restrict__ table,
                                                            int32_t* __restrict__ store_row, int32_t* __restrict__ chunk_id) {
    const int c = blockIdx.y;
    if (blockIdx.x == 0 && c < ct.n && (int)threadIdx.x < half_d)
        table[(size_t)c * half_d + threadIdx.x] = chunk_rotation(deltas.delta[c], theta[threadIdx.x]);
    const int begin = (c < ct.n) ? ct.off[c] : ct.off[ct.n];
    const int end = (c < ct.n) ? ct.off[c + 1] : L;
    for (int j = begin + blockIdx.x * 256 + threadIdx.x; j < end; j += gridDim.x * 256) {
        store_row[j] = (c < ct.n) ? rows.row0[c] + (j - begin) : -1;
        chunk_id[j] = (c < ct.n) ? c : 0;
    }
}

// Every query of a batch in one launch: grid (key tiles of the longest prompt x KV heads, queries).  One
// query's images are a few hundred workgroups, less than the chip holds: 4 queries of 1264 positions, selections and
// attention, 178 us with a launch each, 155 with one; 8 of 4064 positions 523 -> 481; 8 of 16896 4425 -> 4350.
struct SharedPackQuery {
    const __bf16 *k_new, *v_new;
    const int32_t *q_index, *store_row, *chunk_id;
    const float2* table;
    unsigned char* images;
    int32_t R, L, n_img_tiles, pad;
};
struct SharedPackBatch { SharedPackQuery q[ATTN_MAX_BATCH]; };
template <int LAYOUT>
__global__ __launch_bounds__(256) void pack_kv_images_shared_kernel(const SharedPackBatch batch, const __bf16* __restrict__ k_store,
                                                                    const __bf16* __restrict__ v_store, int Hkv) {
    constexpr int D = 128;
    __shared__ __attribute__((aligned(16))) unsigned char img[Img<D>::BYTES];
    __shared__ int32_t fresh[KT];
    const SharedPackQuery& pq = batch.q[blockIdx.y];
    const int kt = blockIdx.x / Hkv, g = blockIdx.x % Hkv;   // as in the attention kernels: the workgroups of a KV head on one XCD
    const int L = pq.L, R = pq.R, n_img_tiles = pq.n_img_tiles;
    if (kt >= n_img_tiles) return;   // a shorter prompt
    const __bf16 *__restrict__ k_new = pq.k_new, *__restrict__ v_new = pq.v_new;
    const int32_t *__restrict__ q_index = pq.q_index, *__restrict__ store_row = pq.store_row, *__restrict__ chunk_id = pq.chunk_id;
    const float2* __restrict__ table = pq.table;
    unsigned char* __restrict__ images = pq.images;
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
//      16 bytes at the wave's LDS base + 16 i), no registers involved, 1 KB per wave instruction.  Completion: the issuing
//      wave's vmcnt, then a workgroup barrier. ----------
__device__ __forceinline__ uint32_t lds_address(const unsigned char* p) {
    return __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) const unsigned char*)p);
}
// Written out rather than left to the builtin: the compiler treats a pending direct-to-LDS load as an access
// that may complete out of order with the LDS reads, and from then on waits for *all* outstanding fragment
// reads before every use (lgkmcnt(0)), which puts a full LDS round trip in front of the matrix pipe every few
// fragments.  Completion is waited for explicitly anyway, so nothing is lost.  The address is the same for the whole
// wave (scalar registers, + 16 lane): the copies cost the vector ALU nothing.
__device__ __forceinline__ void dma_chunk(const unsigned char* src, uint32_t lds_dst, uint32_t lane_off) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(lane_off), "s"(src), "s"(lds_dst) : "memory");
}
typedef const bf16x8 __attribute__((address_space(3)))* lds_frag_ptr;
// A wave's share of an image: chunks w, w + 8, ... of its N.  `wave` must be wave-uniform in the compiler's eyes (readfirstlane).
template <int N>
__device__ __forceinline__ void dma_image(const unsigned char* src, uint32_t lds_dst, int wave, uint32_t lane_off) {
    static_assert(N % FAST_WAVES == 0, "the same for every wave");
#pragma unroll
    for (int c = 0; c < N / FAST_WAVES; ++c)
        dma_chunk(src + (wave + FAST_WAVES * c) * 1024, lds_dst + (uint32_t)(wave + FAST_WAVES * c) * 1024u, lane_off);
}
__device__ __forceinline__ void wait_dma() { __builtin_amdgcn_s_waitcnt(0x0f70); }   // vmcnt(0)
template <int N>
__device__ __forceinline__ void wait_dma_but() {   // until all but the wave's last N copies have landed
    static_assert(N < 16, "one field of the counter");
    __builtin_amdgcn_s_waitcnt(0x0f70 | N);
}
__device__ __forceinline__ void plain_barrier() {   // without the fences of __syncthreads(): the waits are explicit
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Per-lane byte offsets of the operand fragments inside an image: row x, 16-byte quarter kg.
template <int D>
struct FragOffsets {
    int k;   // K fragment: + 4 planes per step of 32 dims + Img<D>::BLOCK per block of 16 keys
    int v;   // V^T fragment: + 4 planes for the second half of the key slots + Img<D>::BLOCK per block of 16 dims
    __device__ __forceinline__ void init(int x, int kg) {
        k = kg * Img<D>::K_PLANE + 16 * x;
        v = kg * Img<D>::V_PLANE + 16 * x;
    }
};
__device__ __forceinline__ f32x4 mfma(const bf16x8& a, const bf16x8& b, const f32x4& c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
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

// The weights of 32 keys x 64 columns as operands of the second product: weight (b, v) of a column is that of key 16 b + 4 kg + v.
// SPLIT: every weight as the sum of three bf16
// numbers, each the leading 8 bits of what the ones before leave: together exactly the 24 bits of an fp32 weight, for
// the shapes whose weights have always been kept in fp32; the second product then takes three instructions per fragment.
// (Cut off rather than rounded: a pair of leading parts is then one byte permute of the two weights.)
template <bool SPLIT>
struct Weights {
    static constexpr int PARTS = SPLIT ? 3 : 1;
    u32x4 part[PARTS][NC];
    __device__ __forceinline__ void set_pair(int nb, int b, int v, float p0, float p1) {   // weights (b, v) and (b, v + 1); v is 0 or 2
        const int at = 2 * b + v / 2;
        if constexpr (SPLIT) {
#pragma unroll
            for (int i = 0; i < PARTS; ++i) {
                part[i][nb][at] = __builtin_amdgcn_perm(__float_as_uint(p1), __float_as_uint(p0), 0x07060302u);   // the upper halves
                if (i + 1 < PARTS) {
                    p0 -= __uint_as_float(__float_as_uint(p0) & 0xFFFF0000u);
                    p1 -= __uint_as_float(__float_as_uint(p1) & 0xFFFF0000u);
                }
            }
        } else {
            bf16x2 t;
            t[0] = (__bf16)p0;
            t[1] = (__bf16)p1;
            part[0][nb][at] = __builtin_bit_cast(uint32_t, t);
        }
    }
    __device__ __forceinline__ bf16x8 operand(int i, int nb) const { return __builtin_bit_cast(bf16x8, part[i][nb]); }
};

__device__ __forceinline__ void mask_half(f32x4 (&s)[2][NC], const int (&col_pos)[NC], int key_base, int kg) {
#pragma unroll
    for (int nb = 0; nb < NC; ++nb) {
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (key_base + 16 * b + 4 * kg + v > col_pos[nb]) s[b][nb][v] = -INFINITY;
        __builtin_amdgcn_sched_barrier(0);   // (block by block: the results of all comparisons at once take scalar registers that the loop needs)
    }
}

// The two bf16 numbers of a word, 0 in the place of one that is not finite.
__device__ __forceinline__ uint32_t finite_or_zero(uint32_t w) {
    if ((w & 0x00007F80u) == 0x00007F80u) w &= 0xFFFF0000u;
    if ((w & 0x7F800000u) == 0x7F800000u) w &= 0x0000FFFFu;
    return w;
}

// Behind a barrier; uniform in the compiler's eyes too (what lies behind a divergent branch keeps its registers through the other side).
__device__ __forceinline__ bool any_of_workgroup(bool v) { return __builtin_amdgcn_readfirstlane(__syncthreads_or(v ? 1 : 0)) != 0; }

// Takes the values that are not finite out of half of a V^T image, for this wave a quarter of it.  Were there any?
template <int D>
__device__ __forceinline__ bool drop_not_finite(unsigned char* half, int quarter) {
    constexpr int QUARTER = Img<D>::V_BYTES / 8;
    bool found = false;
    for (int i = quarter * QUARTER + (threadIdx.x & 63) * 16; i < (quarter + 1) * QUARTER; i += 1024) {
        u32x4 w = *reinterpret_cast<const u32x4*>(half + i);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t kept = finite_or_zero(w[e]);
            found = found || kept != w[e];
            w[e] = kept;
        }
        *reinterpret_cast<u32x4*>(half + i) = w;
    }
    return found;
}
// O^T += those values of an image in memory, for the columns that see them: their weights are positive, so an infinity stays what it is, a
// NaN too.  M of the columns' 16-dim blocks, from block md0 on.
template <int D, int M>
__device__ __forceinline__ void add_not_finite(const unsigned char* vt, int key_base, const int (&col_pos)[NC], int kg, int md0, f32x4 (&o)[M][NC]) {
#pragma unroll 1
    for (int t = 0; t < KT; ++t) {
        const int slot = key_slot(t);
        const unsigned char* key = vt + (slot >> 3) * Img<D>::V_PLANE + 2 * (slot & 7) + 16 * (16 * md0 + 4 * kg);
#pragma unroll
        for (int md = 0; md < M; ++md)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const uint32_t w = *reinterpret_cast<const uint16_t*>(key + 16 * (16 * md + v));
                const float add = (w & 0x7F80u) == 0x7F80u ? __uint_as_float(w << 16) : 0.f;
#pragma unroll
                for (int nb = 0; nb < NC; ++nb) o[md][nb][v] += key_base + t <= col_pos[nb] ? add : 0.f;
            }
    }
}

// Normalise, transpose through LDS and store 16 bytes per lane; lse = (m + log2 l) ln 2.  A wave brings M of its columns' 16-dim
// blocks, from block md0 on: all of them, or half of them beside another wave of its rows (then each stores half of the columns).
template <int G, int D, int M>
__device__ __forceinline__ void store_output(const Geometry<G>& ge, const f32x4 (&o)[M][NC], int md0, const float (&l)[NC],
                                             const float (&mref)[NC], int R, int Hq, unsigned char* smem,
                                             __bf16* __restrict__ out, float* __restrict__ lse_out) {
    constexpr int O_PITCH = Img<D>::O_PITCH, NV = D / 8, MD = Img<D>::MD;
    __bf16* ob = reinterpret_cast<__bf16*>(smem) + ge.wave * 64 * O_PITCH;   // this wave's [64 columns][d]
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int nb = 0; nb < NC; ++nb) {
        const float inv_l = 1.0f / l[nb];
#pragma unroll
        for (int md = 0; md < M; ++md) {
            bf16x4 w;
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e] = (__bf16)(o[md][nb][e] * inv_l);
            *reinterpret_cast<bf16x4*>(&ob[(16 * nb + ge.x) * O_PITCH + 16 * (md0 + md) + 4 * ge.kg]) = w;
        }
        if (md0 == 0 && lse_out != nullptr && ge.kg == 0 && ge.col_row[nb] < R && 16 * nb + ge.x < ge.trw * ge.heads)
            lse_out[(size_t)ge.col_row[nb] * Hq + ge.col_head[nb]] =
                (mref[nb] + __builtin_amdgcn_logf(l[nb])) * 0.6931471805599453f;
    }
    __syncthreads();   // (the barrier orders the LDS writes and reads of the waves of a row group)
#pragma unroll
    for (int i = 0; i < NV * M / MD; ++i) {
        const int col = (64 / NV) * (i + (md0 > 0 ? NV * M / MD : 0)) + lane / NV, vec = lane % NV;
        const int r = ge.row0 + ge.wave * ge.trw + (col % ge.trw), head = col / ge.trw;
        if (r < R && head < ge.heads) {
            const u32x4 w = *reinterpret_cast<const u32x4*>(&ob[col * O_PITCH + 8 * vec]);
            *reinterpret_cast<u32x4*>(out + ((size_t)r * Hq + ge.g * ge.heads + head) * D + 8 * vec) = w;
        }
    }
}

// The same for dims 32 sl .. 32 sl + 31 only (a workgroup of the combine pass).
constexpr int SLICE_PITCH = 40;   // 32 dims + 16 bytes
constexpr int SLICE_LDS = 4 * 64 * SLICE_PITCH * (int)sizeof(__bf16);
template <int G, int D>
__device__ __forceinline__ void store_slice(const Geometry<G>& ge, const f32x4 (&acc)[2][NC], int sl, const float (&l)[NC],
                                            const float (&mref)[NC], int R, int Hq, unsigned char* smem,
                                            __bf16* __restrict__ out, float* __restrict__ lse_out) {
    constexpr int PITCH = SLICE_PITCH;
    __bf16* ob = reinterpret_cast<__bf16*>(smem) + ge.wave * 64 * PITCH;
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int nb = 0; nb < NC; ++nb) {
        const float inv_l = 1.0f / l[nb];
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            bf16x4 w;
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e] = (__bf16)(acc[b][nb][e] * inv_l);
            *reinterpret_cast<bf16x4*>(&ob[(16 * nb + ge.x) * PITCH + 16 * b + 4 * ge.kg]) = w;
        }
        if (sl == 0 && lse_out != nullptr && ge.kg == 0 && ge.col_row[nb] < R && 16 * nb + ge.x < ge.trw * ge.heads)
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
            *reinterpret_cast<u32x4*>(out + ((size_t)r * Hq + ge.g * ge.heads + head) * D + 32 * sl + 8 * vec) = w;
        }
    }
}

// The value of column block kg in lane (x, kg): one word per lane carries what a wave's 64 columns have once each.
__device__ __forceinline__ float own_block(const float (&v)[NC], int kg) {
    const float v0 = v[0], v1 = v[1], v2 = v[2], v3 = v[3];   // (a choice between places of the array would put it into memory)
    const float lo = (kg & 1) ? v1 : v0, hi = (kg & 1) ? v3 : v2;
    return (kg & 2) ? hi : lo;
}
__device__ __forceinline__ uint32_t of_block(uint32_t word, int nb, int x) {   // and back
    return (uint32_t)__builtin_amdgcn_ds_bpermute(4 * (16 * nb + x), (int)word);
}

// Partial result of one part of an item, per lane of a row group's wave: its D output accumulators (D / 4 of each of its four
// columns) and one word each of its wave's column sums, exponent references and two scale exponents (own_block).  Four words of a
// thread side by side (words 4 r .. 4 r + 3 of thread t at [4 (r * 256 + t)]: every store and load of a wave is one line of 1 KB).  Part p of item (ordinal, KV head g) lives at
// (((query * max_row_tiles + ordinal) * n_parts + p) * Hkv + g) * WORDS.  Infinities and NaNs survive the packing (the
// output shows what the values held).
// F32: the accumulators as they are.  Otherwise as half-precision pairs, the D / 2 of a column in half of the dims scaled by a power of two
// that brings the largest of them into [0.5, 1) (11 significant bits of that column's largest value): 68 words instead of
// 132.  Which one: half_parts.
template <int D, bool F32>
struct Part {
    static constexpr int O_WORDS = F32 ? D : D / 2;   // per lane, all column blocks
    static constexpr int COL_WORDS = O_WORDS / NC;    // of a column block; block md of 16 dims has COL_WORDS / (D / 16) of them
    static constexpr int SUM = O_WORDS, REFERENCE = O_WORDS + 1;   // and the exponents: four words side by side
    static constexpr int REGS = O_WORDS + 4;
    static constexpr int WORDS = REGS * 256;          // 32-bit words of a part
    static __device__ __forceinline__ int exponent(int md) { return O_WORDS + 2 + md / (D / 32); }
    static __device__ __forceinline__ int at(int word) { return (word >> 2) * 1024 + (word & 3); }   // place of a word, + 4 t
};
typedef _Float16 __attribute__((ext_vector_type(2))) f16x2;

// The half of a row group's dims that a wave holds: blocks md0 .. md0 + D / 32 - 1.
template <int D, bool F32>
__device__ __forceinline__ void store_partial(float* __restrict__ dst_f, const f32x4 (&o)[D / 32][NC], int md0, const float (&l)[NC],
                                              const float (&mref)[NC], int kg) {
    using P = Part<D, F32>;
    uint32_t* dst = reinterpret_cast<uint32_t*>(dst_f);
    float e[NC];
#pragma unroll
    for (int nb = 0; nb < NC; ++nb) {
        if constexpr (F32) {
#pragma unroll
            for (int md = 0; md < D / 32; ++md)
                *reinterpret_cast<f32x4*>(dst + P::at(nb * P::COL_WORDS + (md0 + md) * 4)) = o[md][nb];
        } else {
            float m = 0.f;
#pragma unroll
            for (int md = 0; md < D / 32; ++md)
#pragma unroll
                for (int v = 0; v < 4; ++v) m = fmaxf(m, fabsf(o[md][nb][v]));
            m = column_max(m);
            // m = f 2^e with f in [0.5, 1); an infinite m keeps e = 0: the infinity is stored as it is
            const int ex = (m < INFINITY) ? __builtin_amdgcn_frexp_expf(m) : 0;
            e[nb] = __uint_as_float((uint32_t)ex);
#pragma unroll
            for (int md = 0; md < D / 32; md += 2) {
                u32x4 w;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    f16x2 h;
                    h[0] = (_Float16)__builtin_ldexpf(o[md + (j >> 1)][nb][2 * (j & 1)], -ex);
                    h[1] = (_Float16)__builtin_ldexpf(o[md + (j >> 1)][nb][2 * (j & 1) + 1], -ex);
                    w[j] = __builtin_bit_cast(uint32_t, h);
                }
                *reinterpret_cast<u32x4*>(dst + P::at(nb * P::COL_WORDS + (md0 + md) * 2)) = w;
            }
        }
    }
    if (md0 == 0) {
        dst[P::at(P::SUM)] = __float_as_uint(own_block(l, kg));
        dst[P::at(P::REFERENCE)] = __float_as_uint(own_block(mref, kg));
    }
    if constexpr (!F32) dst[P::at(P::exponent(md0))] = __float_as_uint(own_block(e, kg));
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
// ---- fast path: key tiles [kb, ke) of one (row tile, KV head) ---------------------------------------------
// Eight waves, two per SIMD.  Waves w and w + 4 own the same 64 query columns; the first takes keys 0..31 of every tile, the second
// keys 32..63, each with output accumulators of its own, which are added up at the end.

// One matrix phase of a wave: O^T += V^T P^T for its half of one tile, S^T = K Q^T for its half of another one.  `vt` and `k` are the LDS
// addresses of the halves.  Operand fragments are
// requested from LDS PF steps of four matrix instructions ahead of their use (rotating register buffer), those of the query a
// step of its dims ahead; the steps whose query fragments come from LDS alternate with those that have theirs in registers.
template <int D, bool SPLIT, bool PV>
__device__ __forceinline__ void matrix_phase(uint32_t vt, uint32_t k, const FragOffsets<D>& fo,
                                             const bf16x8 (&qf)[NC][FastLds<D, SPLIT>::QR > 0 ? FastLds<D, SPLIT>::QR : 1], uint32_t q_lds,
                                             const Weights<SPLIT>& p, f32x4 (&o)[D / 16][NC], f32x4 (&s)[2][NC]) {
    using F = FastLds<D, SPLIT>;
    constexpr int NK = F::NK, MD = Img<D>::MD, PF = 4, QR = F::QR, QL = F::QL;
    constexpr int FIRST = PV ? 0 : MD, STEPS = MD + 2 * NK;   // steps 0 .. MD - 1: output; then logits: (dims ks, key block b)
    // order of the dims: LDS, registers, LDS, ...; the longer kind's surplus last
    auto dims = [&](int j) {   // j-th step of the dims -> ks; ks < QR: registers
        constexpr int M = QR < QL ? QR : QL;
        if (j < 2 * M) return (j & 1) ? j / 2 : QR + j / 2;
        return QL > QR ? QR + j - M : j - M;
    };
    bf16x8 fr[PF + 1], qb[2][NC];
    // (indexed from pointers: the constants then go into the instructions' offsets)
    const lds_frag_ptr v_frag = reinterpret_cast<lds_frag_ptr>((uintptr_t)(vt + fo.v)), k_frag = reinterpret_cast<lds_frag_ptr>((uintptr_t)(k + fo.k));
    const lds_frag_ptr q_frag = reinterpret_cast<lds_frag_ptr>((uintptr_t)q_lds);
    auto frag = [&](int i) -> bf16x8 {
        if (i < MD) return v_frag[i * Img<D>::BLOCK / 16];
        return k_frag[(4 * dims((i - MD) / 2) * Img<D>::K_PLANE + (i & 1) * Img<D>::BLOCK) / 16];
    };
    static_assert(MD % 2 == 0, "key block of step i is i & 1");
    auto load_q = [&](int j) {   // query fragments of the j-th step of the dims, if they are in LDS
        const int ks = dims(j);
        if (ks < QR) return 0;
#pragma unroll
        for (int nb = 0; nb < NC; ++nb) qb[j & 1][nb] = q_frag[((ks - QR) * NC + nb) * 64];
        return NC;
    };
    int reads[STEPS] = {};   // LDS reads issued in front of step i's products
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = FIRST; i < FIRST + PF; ++i) fr[i % (PF + 1)] = frag(i);
    if (!PV) reads[FIRST] += load_q(0);
#pragma unroll
    for (int i = FIRST; i < STEPS; ++i) {
        if (i + PF < STEPS) {
            fr[(i + PF) % (PF + 1)] = frag(i + PF);
            ++reads[i];
        }
        if (PV && i == MD - 2) reads[i] += load_q(0);   // two steps ahead
        if (i >= MD && (i - MD) % 2 == 0 && (i - MD) / 2 + 1 < NK) reads[i] += load_q((i - MD) / 2 + 1);
        const bf16x8 a = fr[i % (PF + 1)];
        if (i < MD) {
#pragma unroll
            for (int u = 0; u < Weights<SPLIT>::PARTS; ++u)
#pragma unroll
                for (int c = 0; c < NC; ++c) {   // (back and forth: neighbours in time share an operand, which saves power)
                    const int nb = (i * Weights<SPLIT>::PARTS + u) & 1 ? NC - 1 - c : c;
                    o[i][nb] = mfma(a, p.operand(u, nb), o[i][nb]);
                }
        } else {
            const int j = (i - MD) / 2, ks = dims(j), b = i & 1;
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const int nb = b ? NC - 1 - c : c;
                s[b][nb] = mfma(a, ks < QR ? qf[nb][ks < QR ? ks : 0] : qb[j & 1][nb], j == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : s[b][nb]);
            }
        }
    }
    __builtin_amdgcn_sched_group_barrier(0x100, PF, 0);
#pragma unroll
    for (int i = FIRST; i < STEPS; ++i) {
        if (reads[i] == 1) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        if (reads[i] == NC) __builtin_amdgcn_sched_group_barrier(0x100, NC, 0);
        if (reads[i] > NC + 1) __builtin_amdgcn_sched_group_barrier(0x100, 2 * NC + 1, 0);
        if (reads[i] == NC + 1) __builtin_amdgcn_sched_group_barrier(0x100, NC + 1, 0);
        if (i < MD) __builtin_amdgcn_sched_group_barrier(0x008, NC * Weights<SPLIT>::PARTS, 0); else __builtin_amdgcn_sched_group_barrier(0x008, NC, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
}

// Logits -> weights: exp2(s scale - reference), their sums.
template <bool SPLIT>
__device__ __forceinline__ void softmax_phase(const f32x4 (&s)[2][NC], Weights<SPLIT>& p, float (&lsum)[NC], const float (&mref)[NC],
                                              float scale_log2e) {
#pragma unroll
    for (int nb = 0; nb < NC; ++nb) {
        float sum[2];
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int v = 0; v < 4; v += 2) {
                const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[b][nb][v], scale_log2e, -mref[nb]));
                const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[b][nb][v + 1], scale_log2e, -mref[nb]));
                if (b == 0 && v == 0) {
                    sum[0] = p0;
                    sum[1] = p1;
                } else {
                    sum[0] += p0;
                    sum[1] += p1;
                }
                p.set_pair(nb, b, v, p0, p1);
            }
        lsum[nb] += sum[0] + sum[1];
    }
    __builtin_amdgcn_sched_barrier(0);
}

// Halves of the accumulators that the two waves of a row group exchange at the end, and their sums.
template <int D>
constexpr int EXCHANGE_WAVE = Img<D>::MD / 2 * NC * 1024 + 1024;
template <int D>
constexpr size_t EXCHANGE_LDS = (size_t)FAST_WAVES * EXCHANGE_WAVE<D>;

// part < 0: the piece is the whole item; the workgroup finishes it.  part >= 0: the piece is share `part` of `n_parts` of the
// item's key tiles; it leaves its partial sums and their exponent reference, and attn_combine_kernel finishes the item.  Every part derives
// the same reference from keys 0..31, so as a rule the parts simply add up.
// EXACT = false: returns false where the sums overflowed that reference, and what it stored is worth nothing; the caller then does the piece
// again with EXACT = true, whose reference is the largest logit of the piece's own keys, found in a pass over them that forms nothing but
// logits (a part then leaves it as its reference).  So both run the same loop in the same kernel.  A second kernel that looked for flagged items
// cost 4 us per call and found none; a loop that rescales its accumulators to a running maximum spills registers, and one of four waves beside
// this one took, with every item of 2970 of 16896 rows overflowing, 2190 us a call whole and 6180 in two parts, now 913 and 1190 (397 and 407
// without overflow); without a fixed reference to begin with 1310 us, now 590.
template <int G, int D, bool SPLIT, bool EXACT>
__device__ __forceinline__ bool process_piece(const AttnQuery& aq, int g, int ordinal, int part, int n_parts, int item,
                                              float* __restrict__ partials, bool half, int Hq, int Hkv, float scale_log2e,
                                              unsigned char* smem_raw) {
    using I = Img<D>;
    using F = FastLds<D, SPLIT>;
    constexpr int MD = I::MD, CH = I::K_BYTES / 1024;      // chunks of a K image, and of a V^T image
    F& sm = *reinterpret_cast<F*>(smem_raw);
    const __bf16* __restrict__ q_rows = aq.q_rows;
    const int R = aq.R, n_img_tiles = aq.n_img_tiles;
    // ---- prologue.  Everything that does not depend on the Q index is requested first (the query fragments, and K
    //      image 0 for the exponent reference), then the Q index itself, so that the three memory round trips of the
    //      prologue overlap instead of following one another. ------------------------------------------------------
    Geometry<G> ge;
    ge.init_rows(Hq, Hkv, aq.n_row_tiles, g, ordinal);
    FragOffsets<D> fo;
    fo.init(ge.x, ge.kg);
    const unsigned char* head_images = aq.images + (size_t)ge.g * n_img_tiles * I::BYTES;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int second = wave >> 2;                          // which half of every tile
    const uint32_t lane_off = (uint32_t)lane * 16u;
    const uint32_t k_base = lds_address(sm.k[0]), v_base = lds_address(sm.vt[0]);
    if constexpr (!EXACT) dma_image<CH>(head_images, k_base + 2 * I::K_BYTES, wave, lane_off);   // K image 0 into ring slot 2: the exponent reference comes from it

    // Q fragments: B operand of S^T = K Q^T, for the whole loop; the two waves of a row group bring two column blocks' each to LDS
    bf16x8 qf[NC][F::QR > 0 ? F::QR : 1], ql[2][F::QL > 0 ? F::QL : 1];
    const uint32_t q_lds = lds_address(sm.q) + (wave & 3) * (F::QL * NC * 1024) + lane_off;
    auto q_row = [&](int row, int head) { return q_rows + ((size_t)min(row, R - 1) * Hq + head) * D + 8 * ge.kg; };
#pragma unroll
    for (int nb = 0; nb < NC; ++nb)
#pragma unroll
        for (int ks = 0; ks < F::QR; ++ks) qf[nb][ks] = *reinterpret_cast<const bf16x8*>(q_row(ge.col_row[nb], ge.col_head[nb]) + 32 * ks);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const __bf16* qp = q_row(second ? ge.col_row[2 + i] : ge.col_row[i], second ? ge.col_head[2 + i] : ge.col_head[i]);
#pragma unroll
        for (int ks = 0; ks < F::QL; ++ks) ql[i][ks] = *reinterpret_cast<const bf16x8*>(qp + 32 * (F::QR + ks));
    }
    ge.init_positions(aq.q_index, R, n_img_tiles);
    const int n_kt = ge.n_kt;
    // this piece's key tiles [kb, ke): shares of ceil(n_kt / n_parts) tiles, so part 0 is never empty
    const int per_part = part < 0 ? n_kt : (n_kt + n_parts - 1) / n_parts;
    const int kb = part < 0 ? 0 : part * per_part, ke = min(n_kt, kb + per_part);
    const int part_words = half ? Part<D, false>::WORDS : Part<D, true>::WORDS;
    float* part_dst = part < 0 ? nullptr : partials + (((size_t)item * n_parts + part) * Hkv + g) * part_words;
    if (kb >= ke) {   // fewer key tiles than parts: this one adds nothing
        const int ref_word = half ? Part<D, false>::at(Part<D, false>::REFERENCE) : Part<D, true>::at(Part<D, true>::REFERENCE);
        for (int r = threadIdx.x; r < part_words; r += 64 * FAST_WAVES) part_dst[r] = r >= ref_word && (r - ref_word) % 4 == 0 ? NEG_BIG : 0.f;
        return true;  // (the hardware waits for the outstanding copy before it retires the wave)
    }

    // K images kb and kb + 1 and V image kb land in LDS.  (Past the piece's last tile the copies repeat that one, here and in
    // the loop: the counts of the waits stay the same, and nobody reads them.)
    auto tile_image = [&](int kt) { return head_images + (size_t)min(kt, ke - 1) * I::BYTES; };
    dma_image<CH>(tile_image(kb), k_base, wave, lane_off);
    dma_image<CH>(tile_image(kb) + I::K_BYTES, v_base, wave, lane_off);
    dma_image<CH>(tile_image(kb + 1), k_base + I::K_BYTES, wave, lane_off);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int ks = 0; ks < F::QL; ++ks)
            *reinterpret_cast<bf16x8 __attribute__((address_space(3)))*>((uintptr_t)(q_lds + (ks * NC + 2 * second + i) * 1024)) = ql[i][ks];
    if (!second && ge.kg == 0) {
#pragma unroll
        for (int nb = 0; nb < NC; ++nb) sm.pos[wave & 3][16 * nb + ge.x] = ge.col_pos[nb];
    }
    if constexpr (EXACT) {   // V ring slot 2 holds zeros for the matrix phase in front
#pragma unroll
        for (int i = 0; i < I::V_BYTES / (64 * FAST_WAVES * 16); ++i)
            *reinterpret_cast<u32x4*>(sm.vt[2] + (i * 64 * FAST_WAVES + threadIdx.x) * 16) = u32x4{0u, 0u, 0u, 0u};
    }
    wait_dma();
    __syncthreads();

    // ---- tile loop ------------------------------------------------------------------------------------
    // A wave alternates between a matrix phase (O += its half of tile kt - 1, logits of its half of tile kt: 64 matrix instructions at
    // head_dim 128, 128 with split weights) and a softmax phase (exponentials of its logits).  The two waves of a SIMD do so in turn:
    //   waves 0..3   barrier kt | matrix (kt - 1, kt) | copies kt | softmax kt
    //   waves 4..7   barrier kt | copies kt | softmax kt - 1 | matrix (kt - 1, kt)
    // so that the vector work of one runs beside the matrix instructions of the other.  (A barrier behind every phase, which holds the
    // waves to it strictly, lets the matrix pipe idle whenever the one wave that feeds it waits for its operands: 17 % more cycles.)
    // Barrier kt says that K image kt and V image kt - 1 have landed and that nobody reads K image kt - 1 and V image kt - 2 any
    // more; the copies behind it refill those slots: K image kt + 2 and V image kt + 1.
    // The matrix phase in front (logits of tile kb) adds V image kb with weights of 0 (zeros, if its values may not be finite), the one behind the last tile forms logits that
    // nobody reads: the loop's code is the only copy of it, which the pieces of a short prompt gain from (their time is that of
    // instructions that arrive for the first time).
    int c0 = 0, c1 = I::K_BYTES, c2 = 2 * I::K_BYTES;   // ring slots (their bytes) of K and V images kt, kt + 1, kt + 2
    const int n_plain = ge.n_plain;
    f32x4 s[2][NC], o[MD][NC];
    Weights<SPLIT> p;
    float lsum[NC], mref[NC];
    if constexpr (EXACT) {   // the maximum of its logits over the piece's visible keys
        float t[NC] = {NEG_BIG, NEG_BIG, NEG_BIG, NEG_BIG};
        for (int kt = kb; kt < ke; ++kt) {   // K images kt and kt + 1 are in ring slots, kt + 2 follows
            dma_image<CH>(tile_image(kt + 2), k_base + c2, wave, lane_off);
            matrix_phase<D, SPLIT, false>(0, k_base + second * (2 * I::BLOCK) + c0, fo, qf, q_lds, p, o, s);
            if (kt >= ge.n_plain) mask_half(s, ge.col_pos, kt * KT + 32 * second, ge.kg);
#pragma unroll
            for (int nb = 0; nb < NC; ++nb)
#pragma unroll
                for (int v = 0; v < 4; ++v) t[nb] = fmaxf(t[nb], fmaxf(s[0][nb][v], s[1][nb][v]));
            wait_dma_but<CH / FAST_WAVES>();       // all but the newest image
            __builtin_amdgcn_s_waitcnt(0xc07f);    // lgkmcnt(0): the wave's own fragment reads
            plain_barrier();
            const int c = c0;
            c0 = c1; c1 = c2; c2 = c;
        }
#pragma unroll
        for (int nb = 0; nb < NC; ++nb) {
            t[nb] = column_max(t[nb]);
            if (ge.kg == 0) sm.ref[wave][16 * nb + ge.x] = t[nb];
        }
        wait_dma();
        __syncthreads();
#pragma unroll
        for (int nb = 0; nb < NC; ++nb) mref[nb] = fmaxf(t[nb], sm.ref[wave ^ 4][16 * nb + ge.x]) * scale_log2e;
        c0 = 0; c1 = I::K_BYTES; c2 = 2 * I::K_BYTES;
        dma_image<CH>(tile_image(kb), k_base, wave, lane_off);   // and once more from the start
        dma_image<CH>(tile_image(kb + 1), k_base + I::K_BYTES, wave, lane_off);
        wait_dma();
        __syncthreads();
    } else {
    // exponent reference of each column = the maximum of its logits over the visible ones of keys 0..31
        matrix_phase<D, SPLIT, false>(0, k_base + 2 * I::K_BYTES, fo, qf, q_lds, p, o, s);
#pragma unroll
        for (int nb = 0; nb < NC; ++nb) {
            float t = NEG_BIG;
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int v = 0; v < 4; ++v) t = fmaxf(t, 16 * b + 4 * ge.kg + v <= ge.col_pos[nb] ? s[b][nb][v] : NEG_BIG);
            mref[nb] = column_max(t) * scale_log2e;   // key 0 is visible to every row
        }
    }
#pragma unroll
    for (int nb = 0; nb < NC; ++nb) {
        lsum[nb] = 0.f;
#pragma unroll
        for (int md = 0; md < MD; ++md) o[md][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < Weights<SPLIT>::PARTS; ++u) p.part[u][nb] = u32x4{0u, 0u, 0u, 0u};
    }
    if constexpr (!EXACT) __syncthreads();   // K image 0 has been read: ring slot 2 is free
    auto copies = [&](int kt) {
        dma_image<CH>(tile_image(kt + 2), k_base + c2, wave, lane_off);
        dma_image<CH>(tile_image(kt + 1) + I::K_BYTES, v_base + c1, wave, lane_off);
    };
    int vp = EXACT ? 2 * I::V_BYTES : 0;   // ring slot of V image kt - 1
    auto barrier = [&] {
        __builtin_amdgcn_sched_barrier(0);
        wait_dma_but<2 * CH / FAST_WAVES>();   // all but the newest tile's copies
        __builtin_amdgcn_s_waitcnt(0xc07f);    // lgkmcnt(0): the wave's own fragment reads
        plain_barrier();
        vp = c0;
        c0 = c1; c1 = c2; c2 = vp;
        __builtin_amdgcn_sched_barrier(0);
    };
    const uint32_t k_half = k_base + second * (2 * I::BLOCK), v_half = v_base + second * (4 * I::V_PLANE);
    auto positions = [&](int (&pos)[NC]) {   // of the lane's columns; returns kg
        uint32_t ln = lane_off;
        asm volatile("" : "+v"(ln));   // (opaque: nothing that follows from it is kept over the loop)
        ln >>= 4;
#pragma unroll
        for (int nb = 0; nb < NC; ++nb) pos[nb] = sm.pos[wave & 3][16 * nb + (ln & 15)];
        return (int)(ln >> 4);
    };
    auto softmax = [&](int kt) {
        if (__builtin_expect(kt >= n_plain, 0)) {   // weight 0 behind a column's own position
            int pos[NC];
            const int kg = positions(pos);
            mask_half(s, pos, kt * KT + 32 * second, kg);
        }
        softmax_phase<SPLIT>(s, p, lsum, mref, scale_log2e);
    };
    // Values of tile kt that are not finite leave the image; the columns that see them get them at the end.  Called between barrier kt + 1
    // and the matrix phase behind it, by all waves for the same tiles.
    bool apart = false;
    auto keep_apart = [&](int kt) {
        if constexpr (EXACT) {
            if (kt < n_plain) return;
            const bool found = drop_not_finite<D>(sm.vt[0] + vp + second * (4 * I::V_PLANE), wave & 3);
            apart = any_of_workgroup(found) || apart;
        }
    };
    if (!second) {
        for (int kt = kb;; ++kt) {
            matrix_phase<D, SPLIT, true>(v_half + vp, k_half + c0, fo, qf, q_lds, p, o, s);
            if (kt == ke) break;
            copies(kt);
            softmax(kt);
            barrier();
            keep_apart(kt);
        }
    } else {
        copies(kb);
        for (int kt = kb;; ++kt) {
            matrix_phase<D, SPLIT, true>(v_half + vp, k_half + c0, fo, qf, q_lds, p, o, s);
            if (kt == ke) break;
            barrier();
            copies(kt + 1);
            softmax(kt);
            keep_apart(kt);
        }
    }
    wait_dma();

    // ---- the two waves of a row group add up: each keeps half of the dims --------------------------------------
    __syncthreads();   // (also: everyone is done with the rings)
    ge.init_rows(Hq, Hkv, aq.n_row_tiles, g, ordinal);   // (formed anew: the loop has no registers to spare)
    constexpr int MH = MD / 2;
    f32x4 oh[MH][NC];
    const int md0 = second * MH;
    {
        unsigned char* mine = smem_raw + (size_t)wave * EXCHANGE_WAVE<D> + lane_off;
        const unsigned char* other = smem_raw + (size_t)(wave ^ 4) * EXCHANGE_WAVE<D> + lane_off;
#pragma unroll
        for (int md = 0; md < MH; ++md)
#pragma unroll
            for (int nb = 0; nb < NC; ++nb) {
                f32x4 w;
#pragma unroll
                for (int e = 0; e < 4; ++e) {   // (element by element: a choice between the arrays' places would put them into memory)
                    const float lo = o[md][nb][e], hi = o[MH + md][nb][e];
                    w[e] = second ? lo : hi;
                    oh[md][nb][e] = second ? hi : lo;
                }
                *reinterpret_cast<f32x4*>(mine + (md * NC + nb) * 1024) = w;
            }
        *reinterpret_cast<f32x4*>(mine + MH * NC * 1024) = f32x4{lsum[0], lsum[1], lsum[2], lsum[3]};
        __syncthreads();
#pragma unroll
        for (int md = 0; md < MH; ++md)
#pragma unroll
            for (int nb = 0; nb < NC; ++nb) {
                const f32x4 w = *reinterpret_cast<const f32x4*>(other + (md * NC + nb) * 1024);
#pragma unroll
                for (int e = 0; e < 4; ++e) oh[md][nb][e] += w[e];
            }
        const f32x4 l2 = *reinterpret_cast<const f32x4*>(other + MH * NC * 1024);
#pragma unroll
        for (int nb = 0; nb < NC; ++nb) lsum[nb] += l2[nb];
    }
    if constexpr (EXACT) {
        if (apart) {
            ge.init_positions(aq.q_index, R, n_img_tiles);
            for (int kt = max(kb, n_plain); kt < ke; ++kt)
                add_not_finite<D, MH>(head_images + (size_t)kt * I::BYTES + I::K_BYTES, kt * KT, ge.col_pos, ge.kg, md0, oh);
        }
    }
    // Overflow check: with a fixed reference a runaway logit shows up as inf / nan in the sums.  The sums of a part stay so far below
    // that up to eight of them add up.
    float l[NC];
    bool bad = false;
    const float limit = part < 0 ? INFINITY : 0x1p123f;
#pragma unroll
    for (int nb = 0; nb < NC; ++nb) {
        l[nb] = column_sum(lsum[nb]);
        if constexpr (!EXACT) {
            float chk = l[nb];
#pragma unroll
            for (int md = 0; md < MH; ++md)
#pragma unroll
                for (int v = 0; v < 4; ++v) chk += fabsf(oh[md][nb][v]);
            bad = bad || !(chk < limit);
        }
    }
    if (part >= 0) {   // leave the partial result; attn_combine_kernel adds the parts and stores
        float* dst = part_dst + 4 * (threadIdx.x & 255);
        if (!SPLIT && half) store_partial<D, false>(dst, oh, md0, l, mref, ge.kg); else store_partial<D, true>(dst, oh, md0, l, mref, ge.kg);
        if constexpr (!EXACT) bad = any_of_workgroup(bad);
    } else {
        if constexpr (EXACT) __syncthreads(); else bad = any_of_workgroup(bad);   // (also: the exchange has been read)
        store_output<G, D, MH>(ge, oh, md0, l, mref, R, Hq, smem_raw, aq.out, aq.lse);
    }
    return !bad;   // (stored all the same: the second go writes the same places, each from the same thread)
}

// blockIdx.x = ((query * max_row_tiles + ordinal) * n_parts + part) * Hkv + KV head.  n_parts = 1: every item whole.
// n_parts > 1 (few items: the chip would idle behind the longest ones): the key tiles of every item are
// dealt to n_parts workgroups in equal consecutive shares; items are launched longest first, so the pieces are too.
// exact: no fixed reference to begin with (FR_ATTN_SOFTMAX_RUNNING_MAX).
// Dynamic LDS: the larger of the K/V rings and the epilogue's staging.
template <int G, int D, bool SPLIT>
__global__ __launch_bounds__(64 * FAST_WAVES) void attn_fixed_ref_kernel(const AttnBatch batch, float* __restrict__ partials, int n_parts,
                                                             int half, int exact, int Hq, int Hkv, float scale_log2e) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    int t = (int)blockIdx.x;
    const int g = t % Hkv; t /= Hkv;
    const int part = t % n_parts; t /= n_parts;
    const int ordinal = t % batch.max_row_tiles, query = t / batch.max_row_tiles;
    const AttnQuery& aq = batch.q[query];
    if (ordinal >= aq.n_row_tiles) return;
    const int share = n_parts > 1 ? part : -1;
    bool redo = exact != 0;
    if (!redo) {
        redo = !process_piece<G, D, SPLIT, false>(aq, g, ordinal, share, n_parts, t, partials, half != 0, Hq, Hkv, scale_log2e, smem_raw);
        if (redo) __syncthreads();   // (the epilogue's staging has been read)
    }
    if (!redo) return;
    // Parts in half precision: the whole item, whose sums then stay in 32 bits; every part that overflowed does so and stores the same.
    const bool whole = !SPLIT && half && share >= 0;
    process_piece<G, D, SPLIT, true>(aq, g, ordinal, whole ? -1 : share, n_parts, t, partials, half != 0, Hq, Hkv, scale_log2e, smem_raw);
    if (whole && threadIdx.x < 256) {
        using P = Part<D, false>;
        partials[(((size_t)t * n_parts + part) * Hkv + g) * P::WORDS + 4 * threadIdx.x + P::at(P::REFERENCE)] = ITEM_DONE;
    }
}

// ---- combine: adds the parts of every item and stores like the fast path's own epilogue.  One workgroup per (item, 32 dims of the output):
//      the pass is bound by the latency of its loads, and a workgroup per item left a short prompt's 24 items in eight parts to 24 compute units
//      (24 us; with one per 32 dims 7.5, in four parts 4.2).  A column's sum is added up by every slice.
//      grid.x = ((query * max_row_tiles + ordinal) * D / 32 + slice) * Hkv + KV head.
template <int G, int D, bool SPLIT, bool F32>
__global__ __launch_bounds__(256, 2) void attn_combine_kernel(const AttnBatch batch, const float* __restrict__ partials,
                                                              int n_parts, int Hq, int Hkv) {
    __shared__ __attribute__((aligned(16))) unsigned char staging[SLICE_LDS];
    int t = (int)blockIdx.x;
    const int g = t % Hkv; t /= Hkv;
    const int sl = t % (D / 32);
    const int item = t / (D / 32);
    const int ordinal = item % batch.max_row_tiles;
    const AttnQuery& aq = batch.q[item / batch.max_row_tiles];
    if (ordinal >= aq.n_row_tiles) return;
    using P = Part<D, F32>;
    constexpr int SW = F32 ? 8 : 4;                     // words of a slice of a column block
    constexpr int AHEAD = 4;                            // parts whose loads are in flight together
    typedef std::conditional_t<F32, u32x2, u32x4> Tail; // sum, reference (and exponents; words that nobody reads would be waited for)
    const uint32_t* p0 = reinterpret_cast<const uint32_t*>(partials + ((size_t)item * n_parts * Hkv + g) * P::WORDS) + 4 * threadIdx.x;
    const size_t part_stride = (size_t)Hkv * P::WORDS;
    f32x4 acc[2][NC];
#pragma unroll
    for (int nb = 0; nb < NC; ++nb) acc[0][nb] = acc[1][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
    float sum = 0.f, ref = NEG_BIG;
    bool done = false;
    const int x = threadIdx.x & 15;
    auto add = [&](int first, auto count) {
        constexpr int N = decltype(count)::value;
        u32x4 w[N][NC][SW / 4];
        Tail tail[N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const uint32_t* pp = p0 + (first + i) * part_stride;
#pragma unroll
            for (int nb = 0; nb < NC; ++nb)
#pragma unroll
                for (int j = 0; j < SW; j += 4) w[i][nb][j / 4] = *reinterpret_cast<const u32x4*>(pp + P::at(nb * P::COL_WORDS + sl * SW + j));
            tail[i] = *reinterpret_cast<const Tail*>(pp + P::at(P::SUM));
        }
        __builtin_amdgcn_sched_barrier(0);   // (all loads before the first wait)
        auto reference = [&](int i) { return __uint_as_float(tail[i][1]); };
        if (first == 0) ref = reference(0);   // part 0 is never empty; an empty part brings NEG_BIG and zeros
        if constexpr (F32) {   // equal references as a rule; another one where a part overflowed it
            bool other = false;
            float m = ref;
#pragma unroll
            for (int i = 0; i < N; ++i) {
                other |= (reference(i) != ref) & (reference(i) != NEG_BIG);
                m = fmaxf(m, reference(i));
            }
            if (__builtin_expect(__any(other), 0)) {
                const float f = __builtin_amdgcn_exp2f(ref - m);
                ref = m;
                sum *= f;
#pragma unroll
                for (int nb = 0; nb < NC; ++nb) {
                    const float fb = __uint_as_float(of_block(__float_as_uint(f), nb, x));
                    acc[0][nb] *= fb;
                    acc[1][nb] *= fb;
                }
#pragma unroll
                for (int i = 0; i < N; ++i) {
                    const float fi = __builtin_amdgcn_exp2f(reference(i) - m);
                    tail[i][0] = __float_as_uint(__uint_as_float(tail[i][0]) * fi);
#pragma unroll
                    for (int nb = 0; nb < NC; ++nb) {
                        const float fb = __uint_as_float(of_block(__float_as_uint(fi), nb, x));
#pragma unroll
                        for (int j = 0; j < SW; ++j) w[i][nb][j / 4][j & 3] = __float_as_uint(__uint_as_float(w[i][nb][j / 4][j & 3]) * fb);
                    }
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < N; ++i) done |= reference(i) == ITEM_DONE;
        }
#pragma unroll
        for (int i = 0; i < N; ++i) {
#pragma unroll
            for (int nb = 0; nb < NC; ++nb) {
                int e = 0;
                if constexpr (!F32) e = (int)of_block(tail[i][P::exponent(2 * sl) - P::SUM], nb, x);
#pragma unroll
                for (int j = 0; j < 8; j += 2) {   // accumulators j and j + 1 of the slice's eight
                    if constexpr (F32) {
                        acc[j >> 2][nb][j & 3] += __uint_as_float(w[i][nb][j >> 2][j & 3]);
                        acc[j >> 2][nb][(j & 3) + 1] += __uint_as_float(w[i][nb][j >> 2][(j & 3) + 1]);
                    } else {
                        const f16x2 h = __builtin_bit_cast(f16x2, (uint32_t)w[i][nb][0][j / 2]);
                        acc[j >> 2][nb][j & 3] += __builtin_ldexpf((float)h[0], e);
                        acc[j >> 2][nb][(j & 3) + 1] += __builtin_ldexpf((float)h[1], e);
                    }
                }
            }
            sum += __uint_as_float(tail[i][0]);
        }
    };
    int part = 0;
    for (; part + AHEAD <= n_parts; part += AHEAD) add(part, std::integral_constant<int, AHEAD>{});
    if (part + 2 <= n_parts) { add(part, std::integral_constant<int, 2>{}); part += 2; }
    if (part < n_parts) add(part, std::integral_constant<int, 1>{});
    if (__any(done)) return;   // the same in every wave
    Geometry<G> ge;
    ge.init_rows(Hq, Hkv, aq.n_row_tiles, g, ordinal);
    float l[NC], mref[NC];
#pragma unroll
    for (int nb = 0; nb < NC; ++nb) {
        l[nb] = __uint_as_float(of_block(__float_as_uint(sum), nb, x));
        mref[nb] = __uint_as_float(of_block(__float_as_uint(ref), nb, x));
    }
    store_slice<G, D>(ge, acc, sl, l, mref, aq.R, Hq, staging, aq.out, aq.lse);
}

// Where one query's packing pass leaves its results.
struct QueryScratch {
    int32_t* store_row_map;   // [L], shared-store queries only
    int32_t* chunk_id_map;    // [L], shared-store queries only
    unsigned char* images;
    size_t images_bytes;
};

template <int D, bool SPLIT>
constexpr size_t LDS_FAST = std::max({sizeof(FastLds<D, SPLIT>), Img<D>::EPILOGUE_LDS, EXCHANGE_LDS<D>});

// Raises the kernel's dynamic LDS limit, once per process (C++ initialises a function-local static exactly once,
// also when several host threads arrive together).
template <int G, int D, bool SPLIT>
hipError_t set_kernel_attributes() {
    static const hipError_t once = [] {
        return hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_fixed_ref_kernel<G, D, SPLIT>),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS_FAST<D, SPLIT>);
    }();
    return once;
}

// Packing pass of one query: tile images of its effective K/V into sc.images; fills the query's line of the table.  With
// `shared` it only makes the query's maps and its line of the packing launch (`pq`), which pack_shared sends for all.
template <int D>
hipError_t pack_query(const Shape& s, const void* q_rows, const int32_t* q_index, int R, const void* k_cache,
                      const void* v_cache, int64_t L, const void* k_new, const void* v_new, void* out, float* lse,
                      const QueryScratch& sc, const SharedStoreArgs* shared, const double* theta, bool writeback, AttnQuery* aq,
                      SharedPackQuery* pq, hipStream_t st) {
    const int TR = 4 * (64 / s.G);   // token rows per workgroup
    const int n_row_tiles = (R + TR - 1) / TR;
    const int n_img_tiles = (int)((L + KT - 1) / KT);
    const dim3 block(256);
    if ((size_t)n_img_tiles * s.Hkv * Img<D>::BYTES > sc.images_bytes) return hipErrorInvalidValue;
    if (shared == nullptr) {
        if (writeback)
            pack_kv_images_kernel<D, true><<<dim3(n_img_tiles * s.Hkv), block, 0, st>>>(
                (const __bf16*)k_cache, (const __bf16*)v_cache, (int)L, (const __bf16*)k_new, (const __bf16*)v_new, q_index, R,
                s.Hkv, n_img_tiles, sc.images);
        else
            pack_kv_images_kernel<D, false><<<dim3(n_img_tiles * s.Hkv), block, 0, st>>>(
                (const __bf16*)k_cache, (const __bf16*)v_cache, (int)L, (const __bf16*)k_new, (const __bf16*)v_new, q_index, R,
                s.Hkv, n_img_tiles, sc.images);
    } else if constexpr (D == 128) {   // k_cache / v_cache are the shared chunk store
        ChunkRows rows;
        int max_len = (int)L - shared->ct.off[shared->ct.n];
        for (int c = 0; c < shared->ct.n; ++c) {
            rows.row0[c] = shared->store_row0[c];
            max_len = std::max(max_len, shared->ct.off[c + 1] - shared->ct.off[c]);
        }
        prompt_tables_kernel<<<dim3(std::max(1, (max_len + 255) / 256), shared->ct.n + 1), block, 0, st>>>(
            shared->ct, rows, *shared->deltas, (int)L, D / 2, theta, shared->table, sc.store_row_map, sc.chunk_id_map);
        *pq = {(const __bf16*)k_new, (const __bf16*)v_new, q_index, sc.store_row_map, sc.chunk_id_map, shared->table, sc.images,
               R, (int)L, n_img_tiles, 0};
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

// The packing launch of n queries over a shared chunk store.
hipError_t pack_shared(const Shape& s, int n, const SharedPackBatch& pb, const void* k_store, const void* v_store, hipStream_t st) {
    int tiles = 0;
    for (int i = 0; i < n; ++i) tiles = std::max(tiles, pb.q[i].n_img_tiles);
    const dim3 grid(tiles * s.Hkv, n), block(256);
    if (s.rope_layout == FR_ROPE_INTERLEAVED)
        pack_kv_images_shared_kernel<FR_ROPE_INTERLEAVED><<<grid, block, 0, st>>>(pb, (const __bf16*)k_store, (const __bf16*)v_store, s.Hkv);
    else
        pack_kv_images_shared_kernel<FR_ROPE_HALF><<<grid, block, 0, st>>>(pb, (const __bf16*)k_store, (const __bf16*)v_store, s.Hkv);
    return hipGetLastError();
}

// Launches the key-tile loop; with a live timer its event pair rides on the kernel's own dispatch (start and end of its
// execution), so the stream carries no extra marker packets and the kernels before and after it are not held up.
template <int G, int D, bool SPLIT>
void launch_tile_loop(const AttnBatch& batch, dim3 grid, float* partials, int n_parts, bool half, bool exact, const Shape& s,
                      float scale_log2e, KernelTimer* timer, bool timed, hipStream_t st) {
    if (timed) {
        const int slot = (int)(timer->n_recorded % timer->n_slots);
        hipExtLaunchKernelGGL((attn_fixed_ref_kernel<G, D, SPLIT>), grid, dim3(64 * FAST_WAVES), (uint32_t)LDS_FAST<D, SPLIT>, st, timer->start[slot],
                              timer->stop[slot], 0u, batch, partials, n_parts, (int)half, (int)exact, s.Hq, s.Hkv, scale_log2e);
        ++timer->n_recorded;
    } else {
        attn_fixed_ref_kernel<G, D, SPLIT><<<grid, dim3(64 * FAST_WAVES), LDS_FAST<D, SPLIT>, st>>>(batch, partials, n_parts, (int)half, (int)exact, s.Hq, s.Hkv, scale_log2e);
    }
}

// Parts per item of a one-query launch of `items` (row tile, KV head) items over n_img_tiles key tiles.  With few items
// the chip would idle behind the longest ones (rows ascend by position: the question rows' tiles walk the whole prompt),
// so every item's key tiles are dealt to several workgroups, at the price of the partial results' traffic, the combine pass, and a
// prologue, an exchange between the waves and one matrix phase more per piece.  738 calls measured with one to eight parts, 100 to 17k tokens,
// row sets spread over the prompt and at its end (their items are all long); the host cannot tell the two apart, so a line lies where what one
// of them loses the other gains.  us a call, whole : two parts, 32 / 8 heads, spread : at the end:
//   2600 tokens, 264 items   69 :  80 and  70 :  89      6000, 304 items  142 : 143 and 200 : 199     11600, 352 items  270 : 268 and 435 : 389
//   4000 tokens, 264 items   97 :  98 and 117 : 134      8192, 328 items  190 : 191 and 293 : 272     16896, 352 items  384 : 381
// 376 items of 16896 tokens, the ordinary request, are 391 : 403 spread and 657 : 589 at the end; above 1.5 items per compute unit the parts make a
// fourth half round anyway (400 items at the end of 11600 tokens 434 : 484).  So: two parts from 32 key tiles on, up to a quarter of the compute
// units in items for each doubling of the prompt beyond four key tiles, at most 11 / 8 of their number; split weights, twice the matrix work
// on a tile of the same partial results, an eighth more, at most 1.5 times, and at head_dim 64, half the partial results, 1.5 times in any case.
// Below half a workgroup per compute unit more parts pay until there is about one piece per compute unit (question-only prefill, 64
// items: 446 us whole, 302, 253, 244, 277, 268 in two, three, four, six, eight parts, with the loop of four waves); in between two parts stay best.
// The smallest piece: four tiles (32 / 8 heads, 24 items of 8 tiles 24.4 us whole, 23.6, 22.8, 23.2, 24.1 in two to five parts; 40 of 5 tiles 20.4 whole,
// 23.0 in two), two where there are next to no items or the weights are split; more than a quarter of a workgroup per compute unit and fewer than 16 tiles stay whole (64
// items of 8 tiles 23.7 whole, 25.3 and 27.1 in two and four parts).  Of short prompts those over a chunk store come here, and over caches of their own those with too many
// columns for one launch (attn_direct_pays).  Split weights, which read no store, have 65 items and more then, and stay whole up to seven tiles (whole : as many parts as
// there are units for, 55 calls: 100 items of 4 tiles 25.6 : 33.0, 67 of 6 29.4 : 33.8, 80 of 6 tiles of head_dim 64 23.7 : 25.8, 85 of 7 31.6 : 35.0, 96 of 8 33.9 : 34.0,
// 80 of 9 36.4 : 34.1, 76 of 12 42.4 : 36.6).
template <int D, bool SPLIT>
int choose_parts(int split_mode, int items, int n_img_tiles, int n_cu, size_t part_bytes, size_t partials_bytes) {
    int parts = 1;
    if (split_mode == FR_ATTN_SPLIT_ON) parts = 2;
    if (split_mode == FR_ATTN_SPLIT_AUTO) {
        const int tiles = n_img_tiles;
        if (2 * items <= n_cu) {
            int pieces;
            if (SPLIT)
                pieces = tiles < 8 ? 1 : (tiles + 1) / 2;
            else if (32 * items <= n_cu)
                pieces = tiles < 5 ? 1 : (tiles + 1) / 2;
            else if (tiles < 6 || (tiles < 16 && 4 * items > n_cu))
                pieces = 1;
            else
                pieces = tiles < 10 ? (tiles + 2) / 3 : (tiles + 2) / 4;
            parts = std::max(1, std::min({ATTN_MAX_PARTS, n_cu / std::max(items, 1), pieces}));
        }
        const int most = n_cu + (SPLIT ? n_cu / 2 : 3 * n_cu / 8);
        const float line = n_cu / 4 * std::log2(tiles / 4.f) + (SPLIT ? n_cu / 8 : 0);
        if (tiles >= 32 && items <= most && (D == 64 || items <= line)) parts = std::max(parts, 2);
    }
    while (parts > 1 && (size_t)items * parts * part_bytes > partials_bytes) --parts;
    return parts;
}

// Half-precision partial results: only for a single query of a long prompt (32 key tiles and more) whose weights are plain
// bf16, where the most items that are cut on their own, 352 in two parts, would otherwise move 2 x 95.2 MB of partial sums, as they are 2 x 49.0
// (combine pass 12.8 us; 332 items in 32 bits, split weights, 18.8).
// Short prompts, batches and more than four parts, a few hundred pieces at most, keep all 32 bits
// (6730 tokens, 32 items: 2.174e-3 off float64 in eight parts, 2.184e-3 in four of half precision; the layer takes 163 us, 159 in
// eight of half precision, 183 in four).
constexpr int HALF_MAX_PARTS = 4;
template <bool SPLIT>
bool half_parts(int n_img_tiles) { return !SPLIT && n_img_tiles >= 32; }
template <int D>
size_t part_bytes(bool half) { return (half ? Part<D, false>::WORDS : Part<D, true>::WORDS) * sizeof(float); }

// Packed queries -> attention launches: tile loop (+ combine pass).
template <int G, int D, bool SPLIT>
hipError_t launch_packed(const Shape& s, const AttnBatch& batch, int n_parts, bool half, const Workspace& ws, int mode,
                         KernelTimer* timer, hipStream_t st) {
    const float scale_log2e = (1.0f / sqrtf((float)s.d)) * 1.4426950408889634f;
    const dim3 grid(batch.max_row_tiles * batch.n * s.Hkv);
    if (mode == FR_ATTN_SOFTMAX_RUNNING_MAX) {   // every item whole
        launch_tile_loop<G, D, SPLIT>(batch, grid, nullptr, 1, false, true, s, scale_log2e, nullptr, false, st);
        return hipGetLastError();
    }
    const bool timed = timer != nullptr && timer->n_slots > 0;
    launch_tile_loop<G, D, SPLIT>(batch, dim3(grid.x * n_parts), ws.attn_partials, n_parts, half, false, s, scale_log2e, timer, timed, st);
    if (n_parts > 1) {
        if constexpr (!SPLIT) {
            if (half) {
                attn_combine_kernel<G, D, SPLIT, false><<<dim3(grid.x * (D / 32)), dim3(256), 0, st>>>(batch, ws.attn_partials, n_parts, s.Hq, s.Hkv);
                return hipGetLastError();
            }
        }
        attn_combine_kernel<G, D, SPLIT, true><<<dim3(grid.x * (D / 32)), dim3(256), 0, st>>>(batch, ws.attn_partials, n_parts, s.Hq, s.Hkv);
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
    SharedPackBatch pb;
    e = pack_query<D>(s, q_rows, q_index, R, k_cache, v_cache, L, k_new, v_new, out, lse, sc, shared, ws.rope_theta, writeback,
                      &batch.q[0], &pb.q[0], st);
    if (e == hipSuccess && shared != nullptr) e = pack_shared(s, 1, pb, k_cache, v_cache, st);
    if (e != hipSuccess) return e;
    batch.max_row_tiles = batch.q[0].n_row_tiles;
    bool half = half_parts<SPLIT>(batch.q[0].n_img_tiles);
    auto parts_of = [&](bool h) {
        return choose_parts<D, SPLIT>(split_mode, batch.q[0].n_row_tiles * s.Hkv, batch.q[0].n_img_tiles, ws.n_cu, part_bytes<D>(h),
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
    SharedPackBatch pb;
    for (int i = 0; i < n; ++i) {
        const SharedBatchQuery& q = qs[i];
        const QueryScratch sc{q.store_row_map, q.chunk_id_map, q.images, q.images_bytes};
        e = pack_query<D>(s, q.q_rows, q.q_index, q.R, k_store, v_store, q.L, q.k_new, q.v_new, q.out, q.lse, sc, &q.shared,
                          ws.rope_theta, false, &batch.q[i], &pb.q[i], st);
        if (e != hipSuccess) return e;
        batch.max_row_tiles = std::max(batch.max_row_tiles, batch.q[i].n_row_tiles);
        n_parts = std::max(n_parts, choose_parts<D, SPLIT>(split_mode, batch.q[i].n_row_tiles * s.Hkv, batch.q[i].n_img_tiles,
                                                        ws.n_cu, slot, ws.attn_partials_bytes));
    }
    e = pack_shared(s, n, pb, k_store, v_store, st);
    if (e != hipSuccess) return e;
    // A batch of queries usually fills the chip by itself: every item whole, one workgroup each.  Up to a quarter of a
    // workgroup per compute unit it is cut like its queries would be alone; in between like one query of as many items.
    const int items = batch.max_row_tiles * n * s.Hkv;
    int tiles = 0;
    for (int i = 0; i < n; ++i) tiles = std::max(tiles, batch.q[i].n_img_tiles);
    if (4 * items > ws.n_cu) n_parts = choose_parts<D, SPLIT>(split_mode, items, tiles, ws.n_cu, slot, ws.attn_partials_bytes);
    while (n_parts > 1 && (size_t)items * n_parts * slot > ws.attn_partials_bytes) --n_parts;
    return launch_packed<G, D, SPLIT>(s, batch, n_parts, false, ws, mode, timer, st);
}

}  // namespace

// Shapes with an instance of their own; the others (any group size up to 64, head_dim 64 too) run the kernels whose group
// size is an argument and whose weights are split (Weights).  The group size enters the prologue and the epilogue only.
// 28 query / 4 KV heads over a 17k-token prompt, 2970 rows: 0.58 ms for the tile loop (410 GFLOP as 820 GFLOP of matrix
// instructions: 1.41 PFLOP/s) + 0.022 + 0.015 ms; one wave per (row, head) on the vector ALU took 50.5 ms.
static bool own_instance(const Shape& s) { return s.d == 128 && (s.G == 1 || s.G == 2 || s.G == 4 || s.G == 8); }

// Partial results of a launch in parts: one slot per piece.
size_t attn_mfma_partials_bytes(const Shape& s, int64_t max_tokens) {
    const int64_t tr = 4 * (64 / s.G);   // token rows per workgroup
    const int64_t items = std::min<int64_t>(((max_tokens + tr - 1) / tr) * s.Hkv, ATTN_SPLIT_ITEMS);
    // two parts of ATTN_SPLIT_ITEMS items (32-bit words unless they may be half_parts), and up
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
