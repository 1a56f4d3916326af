// pk_winograd.hpp -- the 1-D transforms of the Winograd convolutions, shared by
// the three-kernel form (pk_winograd.hip) and the one-kernel form
// (pk_winograd_fused.hip).
#pragma once

#include <hip/hip_runtime.h>

namespace pk {

// The 1-D transforms along one axis of a tile (elementwise on vectors):
// e = B^T d (input), r = A^T mm (output), u = G g (filter).
template <int MT>
struct Wino;

template <>
struct Wino<2> {
    static constexpr int A = 4;
    template <typename T>
    __device__ static __forceinline__ void input_1d(const T *d, T *e)
    {
        e[0] = d[0] - d[2];
        e[1] = d[1] + d[2];
        e[2] = d[2] - d[1];
        e[3] = d[1] - d[3];
    }
    template <typename T>
    __device__ static __forceinline__ void output_1d(const T *mm, T *r)
    {
        r[0] = mm[0] + mm[1] + mm[2];
        r[1] = mm[1] - mm[2] - mm[3];
    }
    __device__ static __forceinline__ void filter_1d(const float *g, float *u)
    {
        u[0] = g[0];
        u[1] = 0.5f * (g[0] + g[1] + g[2]);
        u[2] = 0.5f * (g[0] - g[1] + g[2]);
        u[3] = g[2];
    }
};

template <>
struct Wino<4> {
    static constexpr int A = 6;
    template <typename T>
    __device__ static __forceinline__ void input_1d(const T *d, T *e)
    {
        const T a = d[4] - 4.f * d[2];  // shared by rows 1 and 2
        const T b = d[3] - 4.f * d[1];
        const T c = d[4] - d[2];         // shared by rows 3 and 4
        const T s = 2.f * (d[3] - d[1]);
        e[0] = 4.f * d[0] - 5.f * d[2] + d[4];
        e[1] = a + b;
        e[2] = a - b;
        e[3] = c + s;
        e[4] = c - s;
        e[5] = 4.f * d[1] - 5.f * d[3] + d[5];
    }
    template <typename T>
    __device__ static __forceinline__ void output_1d(const T *mm, T *r)
    {
        const T p12 = mm[1] + mm[2], m12 = mm[1] - mm[2];
        const T p34 = mm[3] + mm[4], m34 = mm[3] - mm[4];
        r[0] = mm[0] + p12 + p34;
        r[1] = m12 + 2.f * m34;
        r[2] = p12 + 4.f * p34;
        r[3] = m12 + 8.f * m34 + mm[5];
    }
    __device__ static __forceinline__ void filter_1d(const float *g, float *u)
    {
        const float s = g[0] + g[2];
        u[0] = 0.25f * g[0];
        u[1] = (-1.f / 6.f) * (s + g[1]);
        u[2] = (-1.f / 6.f) * (s - g[1]);
        const float q = (1.f / 24.f) * g[0] + (1.f / 6.f) * g[2];
        u[3] = q + (1.f / 12.f) * g[1];
        u[4] = q - (1.f / 12.f) * g[1];
        u[5] = g[2];
    }
};

}  // namespace pk
