// Position shift of Appendix A applied to one 16-byte vector of a key on its way from a shared chunk store into a kernel
// (the store itself is never written): rotation of every (even, odd) or (p, p + d/2) pair by the chunk's angle, fp32
// arithmetic, rounded to the storage type -- the same arithmetic as the stand-alone shift.
#pragma once

#include "fr_internal.hpp"

namespace fr {

// (cos, sin)(Delta * theta_p), in fp64, rounded once to fp32.  Delta reaches tens of thousands of positions, so the angle
// is formed and reduced in double precision.
__device__ __forceinline__ float2 chunk_rotation(int32_t delta, double theta) {
    double sn, cs;
    sincos_reduced((double)delta * theta, &sn, &cs);
    return make_float2((float)cs, (float)sn);
}

typedef __attribute__((ext_vector_type(4))) uint32_t rot_u32x4;

// own = elements N vec .. N vec + N - 1 of the head row (N = 16 / sizeof(T)), `t` their rotations: interleaved pairs (2p, 2p + 1) inside the
// vector have N / 2, half-split pairs (p, p + D/2), whose `partner` is the vector D/2 elements away, N; low: own holds the first elements of its pairs.
template <typename T, int LAYOUT>
__device__ __forceinline__ rot_u32x4 rotate_vector(rot_u32x4 own, rot_u32x4 partner, const float2* t, bool low) {
    constexpr int N = 16 / sizeof(T);
    struct alignas(16) V { T v[N]; };
    const V mine = __builtin_bit_cast(V, own), other = __builtin_bit_cast(V, partner);
    V y;
    if (LAYOUT == FR_ROPE_INTERLEAVED) {
#pragma unroll
        for (int e = 0; e < N / 2; ++e) {
            const float a = Elem<T>::to_f32(mine.v[2 * e]), b = Elem<T>::to_f32(mine.v[2 * e + 1]);
            y.v[2 * e] = Elem<T>::from_f32(a * t[e].x - b * t[e].y);
            y.v[2 * e + 1] = Elem<T>::from_f32(b * t[e].x + a * t[e].y);
        }
    } else {
#pragma unroll
        for (int e = 0; e < N; ++e) {
            const float m = Elem<T>::to_f32(mine.v[e]), o = Elem<T>::to_f32(other.v[e]);
            const float a = low ? m : o, b = low ? o : m;
            y.v[e] = low ? Elem<T>::from_f32(a * t[e].x - b * t[e].y) : Elem<T>::from_f32(b * t[e].x + a * t[e].y);
        }
    }
    return __builtin_bit_cast(rot_u32x4, y);
}
// The same with the rotations of the head row in memory.
template <typename T, int D, int LAYOUT>
__device__ __forceinline__ rot_u32x4 rotate_key_vector(rot_u32x4 own, rot_u32x4 partner, const float2* __restrict__ trow, int vec) {
    constexpr int N = 16 / sizeof(T), M = LAYOUT == FR_ROPE_INTERLEAVED ? N / 2 : N;
    float2 t[M];
#pragma unroll
    for (int e = 0; e < M; ++e) t[e] = trow[(M * vec + e) & (D / 2 - 1)];
    return rotate_vector<T, LAYOUT>(own, partner, t, vec < D / (2 * N));
}

}  // namespace fr
