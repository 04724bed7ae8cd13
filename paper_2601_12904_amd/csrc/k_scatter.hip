// Write-back of the recomputed K/V rows (Sec. 4.3): cache[q_index[r]] = new[r], bit-exact.
// Pure data movement: 16-byte vectors, K and V in the same launch.  A call moves 24 MB on the headline layer, so the
// kernel is sized by latency, not by bandwidth: every thread has four independent vectors in flight and the grid holds
// a thread for every four vectors (about 750 workgroups), rather than a few workgroups that loop.
#include "fr_internal.hpp"

namespace fr {

// grid: x = blocks of 1024 vectors, y = 0 (K) / 1 (V).  row_vecs = 16-byte vectors per token row, row_shift its logarithm where
// it is a power of two, else -1.  Index = uint32_t while all vectors can be counted in it: a division of 64 bits is over a hundred
// instructions, eight of which were a fifth of a short call (158 rows of 2 KB 3.07 us back to back, with shifts 2.41; 2949 rows 4.90 : 4.14).
template <typename Index>
__global__ __launch_bounds__(256) void kv_scatter_kernel(const uint4* __restrict__ k_new, const uint4* __restrict__ v_new,
                                                         const int32_t* __restrict__ q_index, Index n_vec,
                                                         uint4* __restrict__ k_cache, uint4* __restrict__ v_cache,
                                                         int64_t L, Index row_vecs, int row_shift) {
    constexpr int U = 4;
    const uint4* src = blockIdx.y ? v_new : k_new;
    uint4* dst = blockIdx.y ? v_cache : k_cache;
    const Index base = (Index)blockIdx.x * (256 * U) + threadIdx.x;
    uint4 val[U];
    int32_t pos[U];
    Index row[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {   // all loads first: the four vectors and their rows' positions travel together
        const Index at = base + 256 * u, i = at < n_vec ? at : n_vec - 1;
        row[u] = row_shift >= 0 ? i >> row_shift : i / row_vecs;
        pos[u] = q_index[row[u]];
        val[u] = src[i];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const Index i = base + 256 * u;
        // (an entry outside the cache breaks the caller's contract; its row is dropped rather than written out of bounds)
        if (i < n_vec && pos[u] >= 0 && pos[u] < L) dst[(size_t)pos[u] * row_vecs + (i - row[u] * row_vecs)] = val[u];
    }
}

hipError_t launch_kv_scatter(const Shape& s, const void* k_new, const void* v_new, const int32_t* q_index,
                             int R, void* k_cache, void* v_cache, int64_t L, hipStream_t st) {
    if (R == 0) return hipSuccess;
    const int row_vecs = s.Hkv * s.d * s.esize / 16;
    const int row_shift = (row_vecs & (row_vecs - 1)) == 0 ? __builtin_ctz(row_vecs) : -1;
    const int64_t n_vec = (int64_t)R * row_vecs;
    const dim3 grid((unsigned)((n_vec + 1023) / 1024), 2), block(256);
#define FR_SCATTER_LAUNCH(Index)                                                                                                 \
    kv_scatter_kernel<Index><<<grid, block, 0, st>>>((const uint4*)k_new, (const uint4*)v_new, q_index, (Index)n_vec, (uint4*)k_cache, \
                                                     (uint4*)v_cache, L, (Index)row_vecs, row_shift)
    if (n_vec <= INT32_MAX) FR_SCATTER_LAUNCH(uint32_t); else FR_SCATTER_LAUNCH(uint64_t);
#undef FR_SCATTER_LAUNCH
    return hipGetLastError();
}

}  // namespace fr
