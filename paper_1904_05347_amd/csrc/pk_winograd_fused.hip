// pk_winograd_fused.hip -- Winograd F(m x m, 3x3) convolution with the input
// transform, the products and the output transform in one kernel.
//
// The three-kernel form (pk_winograd.hip) writes the transformed input V
// ((m+2)^2 / m^2 times the image: 4x for m = 2) and the products M (4x the
// output) to memory and reads them back.  Here a work-group keeps a block of BT
// tiles x BC output channels through all A*A transformed positions (A = m + 2):
//   - the A x A input pixels of its tiles, 16 channels at a time, are copied
//     straight into LDS (two stages, buffer_load ... lds);
//   - wave (a, ...) owns row a of the transformed tile: each lane combines the
//     input rows that row needs, then transforms along the columns, in
//     registers.  With tile l32 and channels 4h .. 4h+3 of an 8-channel chunk
//     in lane (l32, h), the transformed values are the A operands of
//     v_mfma_f32_32x32x2_f32 as they stand, so V never touches LDS or memory;
//   - the transformed filter comes from the workspace in operand order (one
//     16-byte load per lane, position and 32 channels), fetched two positions
//     ahead;
//   - after the last channel each wave transforms its positions along the
//     columns, the rows meet in LDS, and y is written.
// Bound: the matrix cores and the latency of what feeds them (a stage of 16
// channels takes 1.40 us on 32 x 32 and 2.33 us on 32 x 64 for m = 2, 4.8 and
// 6.7 us for m = 4; the products alone 0.85, 1.71, 1.92 and 3.84).  m = 2: two
// work-groups of four waves share a CU.  m = 4: six waves leave two SIMDs half
// idle, so the wide form splits its channels over twelve.
// Measured against the three kernels (whole call, graph-timed): 32 x 56 x 56 x
// 64 -> 64 97 -> 53 us, 4 x 56 x 56 x 64 -> 64 25.8 -> 13.6 us, 32 x 56 x 56 x 256
// -> 256 650 -> 476 us (m = 2); 32 x 56 x 56 x 64 -> 64 60.5 -> 41.1 us (m = 4).
// Deep channels on few tiles stay with the three kernels: a work-group walks all
// of Cin (1 x 14 x 14 x 512 -> 512: 61 us here, 29 there).
// Tried and dropped: two groups of waves splitting the channels (1-8 %, on few
// tiles only), copies and fetches two stages ahead (none: not the latency of
// memory), 64 tiles x 64 channels on eight waves (slower throughout).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "pk_configs.hpp"
#include "pk_winograd.hpp"

namespace pk {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int KC = 16;  // channels per LDS stage

struct FusedArgs {
    const float *x, *U;
    float *y;
    int H, W, Cin, Cout, pt, pl, TH, TW, T, Ho, Wo;
    int ks;    // stages of KC channels
    int cb;    // blocks of 32 output channels in U (Cout rounded up to 64)
    int vec4;  // y takes 16-byte stores
};

// Row a of B^T d as a sum of up to four input rows (the rows and factors of
// Wino<MT>::input_1d's output a).
template <int MT>
struct RowSum;
template <>
struct RowSum<2> {
    static constexpr int N = 2;  // rows in every sum
    static constexpr bool FOUR = false;
};
template <>
struct RowSum<4> {
    static constexpr int N = 3;
    static constexpr bool FOUR = true;  // rows 1 .. 4 of B^T have a fourth
};
__device__ constexpr int kRow2[4][2] = {{0, 2}, {1, 2}, {2, 1}, {1, 3}};
__device__ constexpr float kFac2[4][2] = {{1.f, -1.f}, {1.f, 1.f}, {1.f, -1.f}, {1.f, -1.f}};
__device__ constexpr int kRow4[6][4] = {{0, 2, 4, 4}, {1, 2, 3, 4}, {1, 2, 3, 4}, {1, 2, 3, 4}, {1, 2, 3, 4}, {1, 3, 5, 5}};
__device__ constexpr float kFac4[6][4] = {{4.f, -5.f, 1.f, 0.f},  {-4.f, -4.f, 1.f, 1.f}, {4.f, -4.f, -1.f, 1.f},
                                          {-2.f, -1.f, 2.f, 1.f}, {2.f, -1.f, -2.f, 1.f}, {4.f, -5.f, 1.f, 0.f}};

// The transformed filter in operand order: for chunk 2s + u of 8 channels,
// block j of 32 output channels and position p, lane (l32, h)'s channels
// 16s + 8u + 4h .. +3 of output channel 32j + l32, zero past Cin and Cout.
// (The positions of a chunk and block lie together: with the positions
// outermost, a power of two apart, a wave's loads fell on the same channels.)
template <int MT>
__global__ void __launch_bounds__(256) wino_filter_operand_kernel(const float *__restrict__ f, float *__restrict__ U,
                                                                  int Cin, int Cout, int ks, int cb)
{
    constexpr int A = Wino<MT>::A;
    const int ncout = cb * 32;
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;  // four channels x one output channel
    if (e >= (int64_t)ks * 4 * ncout) return;
    const int c4 = (int)(e / ncout), co = (int)(e - (int64_t)c4 * ncout);
    const int64_t pairs = (int64_t)Cin * Cout;
    float t[4][A][3];  // G g, per channel
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int ci = 4 * c4 + q;
        const bool ok = ci < Cin && co < Cout;
        const float *src = f + (ok ? (int64_t)ci * Cout + co : 0);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            float col[3], out[A];
#pragma unroll
            for (int r = 0; r < 3; ++r) {
                const float v = src[(int64_t)(r * 3 + c) * pairs];
                col[r] = ok ? v : 0.f;
            }
            Wino<MT>::filter_1d(col, out);
#pragma unroll
            for (int a = 0; a < A; ++a) t[q][a][c] = out[a];
        }
    }
    // c4 = 4s + 2u + h
    float *dst = U + ((int64_t)(c4 >> 1) * cb + (co >> 5)) * (A * A * 256) + ((c4 & 1) * 32 + (co & 31)) * 4;
#pragma unroll
    for (int a = 0; a < A; ++a) {
        float u[4][A];
#pragma unroll
        for (int q = 0; q < 4; ++q) Wino<MT>::filter_1d(t[q][a], u[q]);
#pragma unroll
        for (int b = 0; b < A; ++b)
            *(f32x4 *)(dst + (A * a + b) * 256) = f32x4{u[0][b], u[1][b], u[2][b], u[3][b]};
    }
}

// One instruction's 1 KiB copied straight into LDS: lane i's 16 bytes at
// base + off (bytes; zeros for an offset past the range) to dst + 16 i.
__device__ __forceinline__ void copy_1k(const float *base, float *dst, int off)
{
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, 0x7fffffff, 0x00020000);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void *)dst, 16, off, 0, 0, 0);
}

// BT tiles x BC output channels; CW waves share a row's BC channels.
template <int MT, int BT, int BC, int CW, int D, int OCC>
__global__ void __launch_bounds__(64 * Wino<MT>::A * (BT / 32) * CW) __attribute__((amdgpu_waves_per_eu(OCC, 8)))
wino_fused_kernel(FusedArgs p)
{
    constexpr int A = Wino<MT>::A, P = A * A;
    constexpr int NW = A * (BT / 32) * CW;  // waves
    constexpr int NJ = BC / 32 / CW;        // 32-channel blocks of one wave
    constexpr int G = BT / 16;              // 16-tile groups: one copy each per pixel plane
    constexpr int PL = P / NW;              // pixel planes a wave copies
    static_assert(P % NW == 0 && BT % 32 == 0 && BC % (32 * CW) == 0, "whole planes and blocks per wave");
    constexpr int STAGE = P * BT * KC;      // floats
    static_assert((2 * A) % D == 0 && D * NJ <= 63, "the filter's ring divides a stage's positions; vmcnt range");
    constexpr int JP = 2;                   // output columns exchanged at a time
    constexpr int EXCH = A * JP * BT * BC;
    __shared__ __attribute__((aligned(16))) float smem[2 * STAGE > EXCH ? 2 * STAGE : EXCH];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, h = lane >> 5;
    const int a = wave % A;                 // row of the transformed tile
    const int th32 = wave / A % (BT / 32);  // 32-tile half
    const int cw = wave / A / (BT / 32);    // channel share
    const int t0 = blockIdx.x * BT, c0 = blockIdx.y * BC;

    // the lane's share of the copies: tile t0 + 16g + lane/4, channels 4 * chunk
    const int chunk = (lane & 3) ^ ((lane >> 4) & 3);
    int off[G][PL];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const int t = t0 + 16 * g + (lane >> 2);
        const int tt = t < p.T ? t : 0;
        const int n = tt / (p.TH * p.TW), r = tt - n * (p.TH * p.TW);
        const int ty = r / p.TW, tx = r - ty * p.TW;
        const int ih0 = MT * ty - p.pt, iw0 = MT * tx - p.pl;
#pragma unroll
        for (int q = 0; q < PL; ++q) {
            const int pix = wave * PL + q;
            const int ih = ih0 + pix / A, iw = iw0 + pix % A;
            const bool ok = t < p.T && (unsigned)ih < (unsigned)p.H && (unsigned)iw < (unsigned)p.W;
            off[g][q] = ok ? (((n * p.H + ih) * p.W + iw) * p.Cin + 4 * chunk) * 4 : (int)0x80000000;
        }
    }
    auto copy_stage = [&](int s, int buf) {
        const bool k_ok = s * KC + 4 * chunk < p.Cin;
        float *st = smem + buf * STAGE + wave * (PL * G * 256);
#pragma unroll
        for (int q = 0; q < PL; ++q)
#pragma unroll
            for (int g = 0; g < G; ++g) copy_1k(p.x + s * KC, st + (q * G + g) * 256, k_ok ? off[g][q] : (int)0x80000000);
    };

    // the wave's filter operands: position f of stage s is (u = f / A, b = f % A)
    const int64_t step_u = (int64_t)p.cb * (P * 256);
    const float *ubase = p.U + ((int64_t)(c0 / 32 + cw * NJ) * P + a * A) * 256 + lane * 4;
    f32x4 uf[D][NJ];
    auto fetch = [&](int s, int f, f32x4(&dst)[NJ]) {
        const float *src = ubase + (s * 2 + f / A) * step_u + (f % A) * 256;
#pragma unroll
        for (int j = 0; j < NJ; ++j) dst[j] = *(const f32x4 *)(src + j * (P * 256));
    };

    // row a as a sum of input rows
    constexpr int NR = RowSum<MT>::FOUR ? 4 : RowSum<MT>::N;
    int rplane[NR];
    float rfac[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        rplane[i] = (MT == 2 ? kRow2[a & 3][i & 1] : kRow4[a][i]) * A * (BT * KC);
        rfac[i] = MT == 2 ? kFac2[a & 3][i & 1] : kFac4[a][i];
    }
    const bool four = RowSum<MT>::FOUR && a > 0 && a < A - 1;

    f32x16 acc[A][NJ];
#pragma unroll
    for (int b = 0; b < A; ++b)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[b][j][r] = 0.f;

    copy_stage(0, 0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int f = 0; f < D; ++f) fetch(0, f, uf[f]);

    const int row = th32 * 32 + l32;
    const int swz = (row >> 2) & 3;
    int buf = 0;
    for (int s = 0; s < p.ks; ++s) {
        // this stage's copies are older than the last D fetches; after the
        // barrier every wave's have landed and the other stage is free
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(D * NJ) : "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (s + 1 < p.ks) copy_stage(s + 1, buf ^ 1);
        __builtin_amdgcn_sched_barrier(0);  // the fetches below stay behind the copies (the count above)
        const float *st = smem + buf * STAGE + row * KC;
        buf ^= 1;
        // the input rows that row a needs, summed per column
        auto row_sums = [&](int u, f32x4(&sum)[A]) {
            const float *src = st + 4 * ((2 * u + h) ^ swz);
#pragma unroll
            for (int c = 0; c < A; ++c) {
                const float *px = src + c * (BT * KC);
                f32x4 v = *(const f32x4 *)(px + rplane[0]);
                if constexpr (MT == 4) v *= rfac[0];
#pragma unroll
                for (int i = 1; i < RowSum<MT>::N; ++i) {
                    const f32x4 d = *(const f32x4 *)(px + rplane[i]);
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = fmaf(rfac[i], d[e], v[e]);
                }
                sum[c] = v;
            }
            if constexpr (RowSum<MT>::FOUR) {
                if (four) {
#pragma unroll
                    for (int c = 0; c < A; ++c) {
                        const f32x4 d = *(const f32x4 *)(src + c * (BT * KC) + rplane[NR - 1]);
#pragma unroll
                        for (int e = 0; e < 4; ++e) sum[c][e] = fmaf(rfac[NR - 1], d[e], sum[c][e]);
                    }
                }
            }
        };
        // m = 2: the same in two steps, so that chunk 1's reads are behind it
        // when chunk 0's products end
        auto read_rows = [&](int u, f32x4(&raw)[2][A]) {
            const float *src = st + 4 * ((2 * u + h) ^ swz);
#pragma unroll
            for (int c = 0; c < A; ++c)
#pragma unroll
                for (int i = 0; i < 2; ++i) raw[i][c] = *(const f32x4 *)(src + c * (BT * KC) + rplane[i]);
            __builtin_amdgcn_sched_barrier(0);
        };
        auto sum_rows = [&](const f32x4(&raw)[2][A], f32x4(&sum)[A]) {
#pragma unroll
            for (int c = 0; c < A; ++c)
#pragma unroll
                for (int e = 0; e < 4; ++e) sum[c][e] = fmaf(rfac[1], raw[1][c][e], raw[0][c][e]);
        };
        f32x4 sums[2][A], raw[2][A];
        row_sums(0, sums[0]);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (MT == 2 && u == 0) read_rows(1, raw);  // arrives while chunk 0 multiplies
            if (MT == 2 && u == 1) sum_rows(raw, sums[1]);
            if (MT == 4 && u == 1) row_sums(1, sums[1]);  // (no registers for that)
            f32x4(&sum)[A] = sums[u];
            f32x4 v[A];
            Wino<MT>::input_1d(sum, v);
#pragma unroll
            for (int b = 0; b < A; ++b) {
                const int f = u * A + b;
                f32x4(&w)[NJ] = uf[f % D];
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int j = 0; j < NJ; ++j)
                        acc[b][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(v[b][e], w[j][e], acc[b][j], 0, 0, 0);
                // (past the end the last stage again, never used)
                fetch(min(s + (f + D) / (2 * A), p.ks - 1), (f + D) % (2 * A), w);
                // (left alone, the compiler gathers a stage's fetches at its end,
                // where the next stage waits for them at once; m = 4 has no
                // registers to keep them apart)
                if (MT == 2) __builtin_amdgcn_sched_barrier(0);
            }
        }
    }

    // columns in registers: q[j] = sum_b AT[j][b] acc[b], kept in acc[j]
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            float m[A], q[MT];
#pragma unroll
            for (int b = 0; b < A; ++b) m[b] = acc[b][j][r];
            Wino<MT>::output_1d(m, q);
#pragma unroll
            for (int i = 0; i < MT; ++i) acc[i][j][r] = q[i];
        }
    // rows through LDS, JP output columns at a time: [a][column][tile][channel]
    constexpr int NT = 64 * NW;
#pragma unroll
    for (int jp = 0; jp < MT; jp += JP) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // no copy or fetch lands in what follows
        __syncthreads();
#pragma unroll
        for (int jj = 0; jj < JP; ++jj)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    smem[((a * JP + jj) * BT + th32 * 32 + 8 * (r >> 2) + (r & 3) + 4 * h) * BC + (cw * NJ + j) * 32 +
                         l32] = acc[jp + jj][j][r];
        __syncthreads();
        for (int e = tid; e < JP * BT * (BC / 4); e += NT) {
            const int co = c0 + (e % (BC / 4)) * 4;
            const int tj = e / (BC / 4);
            const int t = t0 + tj / JP, j = jp + tj % JP;
            if (t >= p.T || co >= p.Cout) continue;
            const int n = t / (p.TH * p.TW), rr = t - n * (p.TH * p.TW);
            const int ty = rr / p.TW, tx = rr - ty * p.TW;
            const int wo = MT * tx + j;
            if (wo >= p.Wo) continue;
            f32x4 m[A], o[MT];
#pragma unroll
            for (int i = 0; i < A; ++i)
                m[i] = *(const f32x4 *)(smem + ((i * JP + tj % JP) * BT + tj / JP) * BC + (e % (BC / 4)) * 4);
            Wino<MT>::output_1d(m, o);
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                const int ho = MT * ty + i;
                if (ho >= p.Ho) continue;
                float *dst = p.y + (((int64_t)n * p.Ho + ho) * p.Wo + wo) * p.Cout + co;
                if (p.vec4) {
                    *(f32x4 *)dst = o[i];
                } else {
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (co + q < p.Cout) dst[q] = o[i][q];
                }
            }
        }
    }
}

template <int MT, int BT, int BC, int CW, int D, int OCC>
hipError_t fused_launch(const FusedArgs &p, hipStream_t stream)
{
    const dim3 grid((unsigned)((p.T + BT - 1) / BT), (unsigned)((p.Cout + BC - 1) / BC));
    hipLaunchKernelGGL((wino_fused_kernel<MT, BT, BC, CW, D, OCC>), grid, dim3(64 * Wino<MT>::A * (BT / 32) * CW), 0,
                       stream, p);
    return hipGetLastError();
}

}  // namespace

size_t wino_operand_floats(int m, int64_t Cin, int64_t Cout)
{
    const int64_t ks = (Cin + KC - 1) / KC, cb = (Cout + 63) / 64 * 2;
    return (size_t)((m + 2) * (m + 2)) * (size_t)ks * 2 * (size_t)cb * 256;
}

bool wino_fused_fits(int m, int form, int64_t T, int64_t Cout)
{
    const int64_t threads = 64 * (m + 2) * (m == 4 && form == 1 ? 2 : 1), bc = form == 0 ? 32 : 64;
    return (T + 31) / 32 * threads < ((int64_t)1 << 32) && (Cout + bc - 1) / bc <= 65535;
}

hipError_t launch_wino_fused(int m, int form, const float *x, const float *f, float *U, float *y, int64_t H, int64_t W,
                             int64_t Cin, int64_t Cout, int64_t pt, int64_t pl, int64_t TH, int64_t TW, int64_t T,
                             int64_t Ho, int64_t Wo, bool vec4, hipStream_t stream)
{
    FusedArgs p;
    p.x = x;
    p.U = U;
    p.y = y;
    p.H = (int)H;
    p.W = (int)W;
    p.Cin = (int)Cin;
    p.Cout = (int)Cout;
    p.pt = (int)pt;
    p.pl = (int)pl;
    p.TH = (int)TH;
    p.TW = (int)TW;
    p.T = (int)T;
    p.Ho = (int)Ho;
    p.Wo = (int)Wo;
    p.ks = (int)((Cin + KC - 1) / KC);
    p.cb = (int)((Cout + 63) / 64 * 2);
    p.vec4 = vec4;
    const int64_t items = (int64_t)p.ks * 4 * p.cb * 32;
    const unsigned blocks = (unsigned)((items + 255) / 256);
    if (m == 4)
        hipLaunchKernelGGL(wino_filter_operand_kernel<4>, dim3(blocks), dim3(256), 0, stream, f, U, p.Cin, p.Cout,
                           p.ks, p.cb);
    else
        hipLaunchKernelGGL(wino_filter_operand_kernel<2>, dim3(blocks), dim3(256), 0, stream, f, U, p.Cin, p.Cout,
                           p.ks, p.cb);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (m == 4) {
        switch (form) {
        case 0: return fused_launch<4, 32, 32, 1, 6, 1>(p, stream);
        default: return fused_launch<4, 32, 64, 2, 3, 3>(p, stream);
        }
    }
    switch (form) {
    case 0: return fused_launch<2, 32, 32, 1, 8, 2>(p, stream);
    default: return fused_launch<2, 32, 64, 1, 4, 2>(p, stream);
    }
}

}  // namespace pk
