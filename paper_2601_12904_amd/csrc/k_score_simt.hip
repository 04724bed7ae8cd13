// Critical scores without the softmax (FR_NORM_RAW) -- generic kernel for the shapes whose key rows are too long for the
// streaming kernel, and the zeros of a selection without question tokens.  Fixed summation order.
#include "fr_internal.hpp"

namespace fr {

// One thread per context key j: score[j] = sum_h sum_i q[i, h] . k[j, g(h)] / sqrt(d), heads outer, question tokens inner.
template <typename T>
__global__ __launch_bounds__(64) void score_raw_generic_kernel(const T* __restrict__ q, const T* __restrict__ k, int64_t L_ctx,
                                                               int nq, int Hq, int Hkv, int d, float scale,
                                                               float* __restrict__ scores) {
    const int64_t j = (int64_t)blockIdx.x * 64 + threadIdx.x;
    if (j >= L_ctx) return;
    const int G = Hq / Hkv;
    float total = 0.f;
    for (int h = 0; h < Hq; ++h) {
        const T* kv = k + ((size_t)j * Hkv + h / G) * d;
        float acc = 0.f;
        for (int i = 0; i < nq; ++i) {
            const T* qv = q + ((size_t)i * Hq + h) * d;
            float s = 0.f;
            for (int t = 0; t < d; ++t) s += Elem<T>::to_f32(qv[t]) * Elem<T>::to_f32(kv[t]);
            acc += s * scale;
        }
        total += acc;
    }
    scores[j] = total;
}

hipError_t launch_score_simt(const Shape& s, const void* q, int nq, const void* k_ctx, int64_t L_ctx, float* scores,
                             hipStream_t st) {
    if (L_ctx == 0) return hipSuccess;
    const float scale = 1.0f / sqrtf((float)s.d);
    const dim3 grid((unsigned)((L_ctx + 63) / 64)), block(64);
    if (s.dtype == FR_BF16)
        score_raw_generic_kernel<__bf16><<<grid, block, 0, st>>>((const __bf16*)q, (const __bf16*)k_ctx, L_ctx, nq, s.Hq, s.Hkv, s.d, scale, scores);
    else
        score_raw_generic_kernel<float><<<grid, block, 0, st>>>((const float*)q, (const float*)k_ctx, L_ctx, nq, s.Hq, s.Hkv, s.d, scale, scores);
    return hipGetLastError();
}

}  // namespace fr
