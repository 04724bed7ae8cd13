// Position recovery of cached chunk keys (Sec. 2.2.1 footnote, Appendix A): every key of chunk c is
// rotated by Delta_c positions.  HBM-bound streaming: 16-byte loads and stores; a workgroup forms its chunk's (cos, sin)
// row in fp64 itself.  880 tokens of 2 KB: 2.8 us back to back (4.2 with 32 tokens per workgroup, which leaves two thirds of the chip without one; 4800 tokens 4.6 : 5.2,
// of 1 KB 3.6 either way); 16384 tokens: 12.5 us; 32 layers of them 0.39 ms = 5.5 TB/s.
#include "k_rotate.hpp"

namespace fr {

// table[c][p], theta: [half_d] rotary frequencies
__global__ void rope_table_kernel(ChunkDeltas deltas, int half_d, const double* __restrict__ theta, float2* __restrict__ table) {
    const int c = blockIdx.x, p = threadIdx.x;
    if (p < half_d) table[(size_t)c * half_d + p] = chunk_rotation(deltas.delta[c], theta[p]);
}

template <typename T>
struct Vec16 {
    static constexpr int N = 16 / sizeof(T);
    T v[N];
};

// grid: x = token tiles inside a chunk, y = chunk, z = batch.  TOK tokens per block.
template <typename T, int LAYOUT, int TOK>
__global__ __launch_bounds__(256) void rope_shift_kernel(const T* __restrict__ src, T* __restrict__ dst,
                                                         ChunkTable ct, ChunkDeltas deltas, const double* __restrict__ theta,
                                                         int Hkv, int d, int64_t src_stride,
                                                         int64_t dst_stride, ChunkRows src_rows, int from_store) {
    constexpr int N = 16 / sizeof(T);  // elements per 16-byte vector
    __shared__ float2 cs[64];          // d/2 <= 64 (cos, sin) pairs of this chunk
    const int c = blockIdx.y;
    const int c0 = ct.off[c], c1 = ct.off[c + 1];
    const int tok0 = c0 + blockIdx.x * TOK;
    if (tok0 >= c1) return;
    const int half_d = d >> 1;
    const int ntok = min(TOK, c1 - tok0);
    const size_t row = (size_t)Hkv * d;  // elements per token
    // source row of the block's first token: its prompt position, or its row in a chunk store
    const size_t src_tok0 = from_store ? (size_t)src_rows.row0[c] + (size_t)(tok0 - c0) : (size_t)tok0;
    const T* s = src + (size_t)blockIdx.z * src_stride + src_tok0 * row;
    T* o = dst + (size_t)blockIdx.z * dst_stride + (size_t)tok0 * row;
    // (half_d is 32 or 64; every thread forms one rotation, the copies are equal)
    const int32_t delta = deltas.delta[c];
    const int my_p = threadIdx.x & (half_d - 1);
    const double my_theta = theta[my_p];
    auto rotations = [&] {
        cs[my_p] = chunk_rotation(delta, my_theta);
        __syncthreads();
    };

    if (LAYOUT == FR_ROPE_INTERLEAVED) {
        constexpr int AHEAD = 8;   // vectors of a thread in flight
        const int vec_per_head = d / N;
        const int nvec = ntok * Hkv * vec_per_head;
        Vec16<T> x[AHEAD];
        auto load = [&](int i0) {   // past the end: the last vector, not stored (a branch would wait for each load)
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) x[u] = *reinterpret_cast<const Vec16<T>*>(s + (size_t)min(i0 + 256 * u, nvec - 1) * N);
        };
        load(threadIdx.x);
        rotations();
        // vec_per_head divides 256 (d is 64 or 128), so a thread meets the same slice of the head row in every step:
        // its (cos, sin) values stay in registers
        const int p0 = (threadIdx.x % vec_per_head) * (N / 2);  // first rotary pair of this thread's vectors
        float2 tw[N / 2];
#pragma unroll
        for (int e = 0; e < N / 2; ++e) tw[e] = cs[p0 + e];
        for (int i0 = threadIdx.x; i0 < nvec; i0 += 256 * AHEAD) {
            if (i0 != (int)threadIdx.x) load(i0);
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) {
                if (i0 + 256 * u >= nvec) continue;
                Vec16<T> y;
#pragma unroll
                for (int e = 0; e < N / 2; ++e) {
                    const float2 t = tw[e];
                    const float a = Elem<T>::to_f32(x[u].v[2 * e]), b = Elem<T>::to_f32(x[u].v[2 * e + 1]);
                    y.v[2 * e] = Elem<T>::from_f32(a * t.x - b * t.y);
                    y.v[2 * e + 1] = Elem<T>::from_f32(b * t.x + a * t.y);
                }
                *reinterpret_cast<Vec16<T>*>(o + (size_t)(i0 + 256 * u) * N) = y;
            }
        }
    } else {  // pairs (p, p + d/2): one lane moves the low and the high vector of a head together
        constexpr int AHEAD = 4;
        const int vec_per_half = half_d / N;   // a power of two
        const int nvec = ntok * Hkv * vec_per_half;
        Vec16<T> xa[AHEAD], xb[AHEAD];
        auto place = [&](int i) -> size_t { return (size_t)(i / vec_per_half) * d + (i % vec_per_half) * N; };   // of the low vector
        auto load = [&](int i0) {
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) {
                const size_t lo = place(min(i0 + 256 * u, nvec - 1));
                xa[u] = *reinterpret_cast<const Vec16<T>*>(s + lo);
                xb[u] = *reinterpret_cast<const Vec16<T>*>(s + lo + half_d);
            }
        };
        load(threadIdx.x);
        rotations();
        float2 tw[N];   // (vec_per_half divides 256: the same pairs in every step)
#pragma unroll
        for (int e = 0; e < N; ++e) tw[e] = cs[(threadIdx.x % vec_per_half) * N + e];
        for (int i0 = threadIdx.x; i0 < nvec; i0 += 256 * AHEAD) {
            if (i0 != (int)threadIdx.x) load(i0);
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) {
                if (i0 + 256 * u >= nvec) continue;
                const size_t lo = place(i0 + 256 * u);
                Vec16<T> ya, yb;
#pragma unroll
                for (int e = 0; e < N; ++e) {
                    const float a = Elem<T>::to_f32(xa[u].v[e]), b = Elem<T>::to_f32(xb[u].v[e]);
                    ya.v[e] = Elem<T>::from_f32(a * tw[e].x - b * tw[e].y);
                    yb.v[e] = Elem<T>::from_f32(b * tw[e].x + a * tw[e].y);
                }
                *reinterpret_cast<Vec16<T>*>(o + lo) = ya;
                *reinterpret_cast<Vec16<T>*>(o + lo + half_d) = yb;
            }
        }
    }
}

hipError_t launch_rope_table(const Shape& s, const ChunkDeltas& deltas, int n_chunks, const double* theta, float2* table,
                             hipStream_t st) {
    if (n_chunks == 0) return hipSuccess;
    rope_table_kernel<<<dim3(n_chunks), dim3(64), 0, st>>>(deltas, s.d / 2, theta, table);
    return hipGetLastError();
}

hipError_t launch_rope_shift(const Shape& s, const void* src, void* dst, const ChunkTable& ct, const ChunkDeltas& deltas,
                             int max_chunk_len, const double* theta, int n_batch, int64_t src_stride,
                             int64_t dst_stride, const ChunkRows* src_rows, int n_cu, hipStream_t st) {
    if (ct.n == 0 || max_chunk_len == 0 || n_batch == 0) return hipSuccess;
    const ChunkRows none{};
    const ChunkRows& rows = src_rows ? *src_rows : none;
    const int from_store = src_rows ? 1 : 0;
    // Tokens per workgroup: 32, eight vectors of a thread in flight twice over; while that would leave compute units without a workgroup, 8 (see the head).  Four times the
    // workgroups cost more than they bring where a row is short: from half the units on below 1536 bytes (32 : 8 tokens, us, 128 and 250 tiles: rows of 1024 bytes 3.5 : 3.3 and 4.2 : 4.5, of
    // 1536 4.0 : 3.4 and 5.3 : 5.0, of 2048 5.4 : 4.3 and 6.5 : 6.0), and where 32 tokens are but a vector (two in the half-split layout) of a thread (128 tiles 2.8 : 2.9).
    const int64_t tiles = (int64_t)((max_chunk_len + 31) / 32) * ct.n * n_batch;
    const int row = s.Hkv * s.d * s.esize, short_row = s.rope_layout == FR_ROPE_HALF ? 512 : 256;
    const bool few = row >= 1536 ? tiles < n_cu : row >= short_row && 2 * tiles <= n_cu;
    const int tok = few ? 8 : 32;
    dim3 grid((max_chunk_len + tok - 1) / tok, ct.n, n_batch);
#define FR_ROPE_LAUNCH_TOK(T, LAY, TOK)                                                             \
    rope_shift_kernel<T, LAY, TOK><<<grid, dim3(256), 0, st>>>((const T*)src, (T*)dst, ct, deltas, theta, \
                                                               s.Hkv, s.d, src_stride, dst_stride, rows, from_store)
#define FR_ROPE_LAUNCH(T, LAY) do { if (few) FR_ROPE_LAUNCH_TOK(T, LAY, 8); else FR_ROPE_LAUNCH_TOK(T, LAY, 32); } while (0)
    if (s.dtype == FR_BF16) {
        if (s.rope_layout == FR_ROPE_INTERLEAVED)
            FR_ROPE_LAUNCH(__bf16, FR_ROPE_INTERLEAVED);
        else
            FR_ROPE_LAUNCH(__bf16, FR_ROPE_HALF);
    } else {
        if (s.rope_layout == FR_ROPE_INTERLEAVED)
            FR_ROPE_LAUNCH(float, FR_ROPE_INTERLEAVED);
        else
            FR_ROPE_LAUNCH(float, FR_ROPE_HALF);
    }
#undef FR_ROPE_LAUNCH_TOK
#undef FR_ROPE_LAUNCH
    return hipGetLastError();
}

}  // namespace fr
