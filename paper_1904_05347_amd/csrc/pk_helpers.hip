// pk_helpers.hip -- the split-K reduction and the beta-scaling launches.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "pk_configs.hpp"

namespace pk {

// Fixed-order reduction of split-K partials: C = sum_z ws[z] (+ beta * C).
// Element e of the M x N result is summed over z = 0, 1, ... in that order,
// so the result does not depend on scheduling.  A partial sum is packed, so
// each work-item takes the next four of its M * N elements, whatever rows they
// lie in, and issues the loads of up to eight partials before the first
// addition, so a split of S costs about S/8 memory round trips instead of S.
// ALIGNED: rows and both buffers allow 16-byte accesses; otherwise (of at least
// four elements) the four are accessed at their own 4-byte alignment (one
// instruction all the same), in C one by one where they cross the end of a row.
// The last work-item goes back to the last four elements and stores those left
// over.  Bound by memory: 1021 x 1531, two partials 4.5 us (beta = 0) and 4.8
// (0.5), 7.9 and 8.0 with one element per work-item.
template <bool ALIGNED>
__global__ void __launch_bounds__(256) splitk_reduce_kernel(const float *ws, float *C, int M, int N,
                                                            int64_t ldc, int splits, float beta)
{
    typedef float V4 __attribute__((ext_vector_type(4)));
    typedef V4 U4 __attribute__((aligned(4)));
    typedef typename std::conditional<ALIGNED, V4, U4>::type VT;
    constexpr int B = 8;  // partials in flight per work-item
    const int64_t total = (int64_t)M * N;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t it = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; 4 * it < total; it += stride) {
        const int64_t e = ALIGNED || 4 * it + 4 <= total ? 4 * it : total - 4;
        const int skip = (int)(4 * it - e);  // of the last work-item: elements that the one before it stores
        const int64_t row = e / N;
        int col = (int)(e - row * N);
        const float *p = ws + e;
        float *c = C + row * ldc + col;
        V4 s = *reinterpret_cast<const VT *>(p);
        for (int z = 1; z < splits; z += B) {
            V4 v[B];
#pragma unroll
            for (int u = 0; u < B; ++u)
                if (z + u < splits) v[u] = *reinterpret_cast<const VT *>(p + (int64_t)(z + u) * total);
#pragma unroll
            for (int u = 0; u < B; ++u)
                if (z + u < splits) s += v[u];
        }
        if (ALIGNED || (skip == 0 && col + 4 <= N)) {
            if (beta != 0.f) {
                const V4 old = *reinterpret_cast<const VT *>(c);
#pragma unroll
                for (int j = 0; j < 4; ++j) s[j] = fmaf(beta, old[j], s[j]);
            }
            *reinterpret_cast<VT *>(c) = s;
            continue;
        }
        float *at[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (col == N) {
                col = 0;
                c += ldc - N;
            }
            at[j] = c++;
            ++col;
        }
        if (beta != 0.f) {
            float old[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) old[j] = j >= skip ? *at[j] : 0.f;
#pragma unroll
            for (int j = 0; j < 4; ++j) s[j] = fmaf(beta, old[j], s[j]);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (j >= skip) *at[j] = s[j];
    }
}

// C <- beta * C (alpha == 0 or K == 0).  beta == 0 writes zeros without reading.
__global__ void __launch_bounds__(256) scale_kernel(float *C, int M, int N, int64_t ldc, float beta)
{
    const int64_t total = (int64_t)M * N;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += stride) {
        const int64_t row = e / N, col = e - row * N;
        float *c = C + row * ldc + col;
        *c = beta != 0.f ? beta * *c : 0.f;
    }
}

// The same for unaligned results of at most kShortReduce elements, one element
// per work-item: there a launch and a round trip to memory are all, and four
// times the work-items with nothing to sort out by rows take 2.1 us instead of
// 2.7 (160 x 98, two partials; 2.8 and 2.8 at 600 x 407, 3.7 and 2.9 at
// 800 x 611; eight and sixteen partials cross at the same size).
constexpr int kShortReduce = 1 << 18;

__global__ void __launch_bounds__(256) splitk_reduce_short_kernel(const float *ws, float *C, int M, int N, int64_t ldc,
                                                                  int splits, float beta)
{
    constexpr int B = 8;  // partials in flight per work-item
    const int total = M * N;
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= total) return;
    const int row = e / N;
    float *c = C + row * ldc + (e - row * N);
    float s = ws[e];
    for (int z = 1; z < splits; z += B) {
        float v[B];
#pragma unroll
        for (int u = 0; u < B; ++u)
            if (z + u < splits) v[u] = ws[(int64_t)(z + u) * total + e];
#pragma unroll
        for (int u = 0; u < B; ++u)
            if (z + u < splits) s += v[u];
    }
    *c = beta != 0.f ? fmaf(beta, *c, s) : s;
}

// Arrival counters of a stream-K launch start at zero.
__global__ void __launch_bounds__(256) zero_ints_kernel(int *p, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

// ---------------------------------------------------------------- helpers

int device_cu_count()
{
    static int counts[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
    if (counts[dev] == 0) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1) n = 256;
        counts[dev] = n;
    }
    return counts[dev];
}

hipError_t launch_splitk_reduce(const float *ws, float *C, int M, int N, int64_t ldc, int splits,
                                float beta, hipStream_t stream)
{
    const bool v4 = N % 4 == 0 && ldc % 4 == 0 && reinterpret_cast<uintptr_t>(C) % 16 == 0 &&
                    reinterpret_cast<uintptr_t>(ws) % 16 == 0;
    const int64_t total = (int64_t)M * N, blocks = ((total + 3) / 4 + 255) / 256;
    const unsigned grid = (unsigned)(blocks < 8192 ? blocks : 8192);
    if (!v4 && total <= kShortReduce)
        hipLaunchKernelGGL(splitk_reduce_short_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream, ws, C,
                           M, N, ldc, splits, beta);
    else if (v4)
        hipLaunchKernelGGL(splitk_reduce_kernel<true>, dim3(grid), dim3(256), 0, stream, ws, C, M, N, ldc, splits, beta);
    else
        hipLaunchKernelGGL(splitk_reduce_kernel<false>, dim3(grid), dim3(256), 0, stream, ws, C, M, N, ldc, splits, beta);
    return hipGetLastError();
}

hipError_t launch_scale(float *C, int M, int N, int64_t ldc, float beta, hipStream_t stream)
{
    const int64_t total = (int64_t)M * N;
    const int64_t blocks = (total + 255) / 256;
    const unsigned grid = (unsigned)(blocks < 8192 ? blocks : 8192);
    hipLaunchKernelGGL(scale_kernel, dim3(grid), dim3(256), 0, stream, C, M, N, ldc, beta);
    return hipGetLastError();
}

hipError_t launch_zero_ints(int *p, int n, hipStream_t stream)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(zero_ints_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, p, n);
    return hipGetLastError();
}

}  // namespace pk
