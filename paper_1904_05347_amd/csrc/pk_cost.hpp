// pk_cost.hpp -- the time of a product on each compiled tile, predicted from
// its sizes: the per-shape parameter choice of Section 5 for shapes that no
// table holds.
//
// A product on one tile configuration, its reduction split s ways across
// work-groups, runs items = tiles * s work-groups of `steps` K-blocks each,
// n = ceil(items / 256) of them on the fullest CU, which holds R at once:
//
//   t = t0 + sum over rounds of r <= R work-groups ( max(l, r * m) * steps + ov )
//          + (s > 1: c0 + c1 * (s + 1) * megabytes of one partial sum)
//
// m is a K-block's share of the CU when the matrix cores are busy (the tile's
// work over the rate it sustains), l its latency when nothing else runs there,
// ov a round's fill and epilogue, t0 a launch, c0 and c1 the second kernel
// that adds the partial sums (c0 is 1.6 to 2.6 in a graph; 4 stands here, what
// the second launch and the workspace cost a caller that launches each call).
// All in microseconds, fitted to graph-timed calls on MI355X: every tile and split of {1, 2, 3, 4, 6, 8, 12, 16} on 230
// random products (sides 16 to 4096, four layouts) and 220 random
// convolutions (1x1 to 7x7, stride 1 and 2, 8 to 1024 channels), 23 000 times
// in all, reproduced to 6-10 % (rms).  Taking the configuration and split of
// the least predicted time costs 2-4 % over the best of all of them
// (geometric mean per group of shapes; the limits on chains below add their
// 0.5 to 1.9 %); the rules that stood before cost
// 6-13 % on aligned products, 17-19 % on aligned convolutions, and the 4-byte
// kernels that served unaligned operands 21-36 % and 37-80 %.  Graph-timed
// against these rules over 6 000 random products and as many convolutions, the
// choices that differ (half of them) are 1.34 and 1.47 times as fast (geometric
// mean); 0.5 and 0.2 % of them are more than 3 % slower, the worst 11 %.
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace pk {

struct TileCost {
    const char *name;  // of the configuration; GEMM: "%s" stands for the layout
    int bm, bn, bk;
    int kg;       // groups of waves that split a tile's K-blocks inside the work-group
    int per_cu;   // R: work-groups a CU holds (LDS)
    int streamk;  // equal shares of the K-blocks: m * (all K-blocks) / CUs
    float l, m, ov;
};

struct CostFamily {
    float t0, c0, c1;
    int n;
    const TileCost *tiles;
};

// products whose operands allow 16-byte accesses (the 128 x 96 tile's m was
// fitted to 1.583: 5 of 24 products that took it were 2-10 % slower than the
// rule's; at 1.680 more others lost up to 22 %)
constexpr TileCost kCostGemm44Tiles[] = {
    {"gemm_256x256x32_w2x4_%s_v44_o2_dma2", 256, 256, 32, 1, 1, 0, 0.563f, 7.158f, 6.92f},
    {"gemm_128x128x32_w2x4_%s_v44_o2_dma2", 128, 128, 32, 1, 2, 0, 0.741f, 1.959f, 2.89f},
    {"gemm_128x96x32_w4x1_%s_v44_dma2", 128, 96, 32, 1, 2, 0, 0.156f, 1.610f, 3.49f},
    {"gemm_128x64x32_w2x2_%s_v44_dma2", 128, 64, 32, 1, 3, 0, 0.360f, 1.099f, 2.70f},
    {"gemm_128x32x32_w4x1_%s_v44_dma2", 128, 32, 32, 1, 4, 0, 0.489f, 0.668f, 2.10f},
    {"gemm_64x64x32_w2x2_%s_v44_dma2", 64, 64, 32, 1, 5, 0, 0.297f, 0.631f, 1.83f},
    {"gemm_64x64x16_w2x2_%s_v44_dma3", 64, 64, 16, 1, 6, 0, 0.375f, 0.307f, 1.74f},
    {"gemm_32x64x32_w1x2_%s_v44_dma3", 32, 64, 32, 1, 4, 0, 0.680f, 0.431f, 1.77f},
    {"gemm_64x64x32_w2x2_k4_%s_v44_dma2", 64, 64, 32, 4, 1, 0, 0.529f, 2.055f, 3.34f},
    {"gemm_64x64x32_w2x2_k2_%s_v44_dma3", 64, 64, 32, 2, 1, 0, 0.488f, 1.116f, 2.15f},
    {"gemm_32x64x32_w1x2_k4_%s_v44_dma3", 32, 64, 32, 4, 1, 0, 0.343f, 1.228f, 2.49f},
    {"gemm_64x64x16_w2x2_%s_v44", 64, 64, 16, 1, 8, 0, 0.424f, 0.324f, 1.75f},
};
constexpr CostFamily kCostGemm44 = {2.29f, 4.00f, 0.305f, 12, kCostGemm44Tiles};

// products of operands aligned to 4 bytes
constexpr TileCost kCostGemm11Tiles[] = {
    {"gemm_256x256x32_w2x4_%s_v11_o2_dma2", 256, 256, 32, 1, 1, 0, 0.138f, 7.236f, 6.98f},
    {"gemm_128x128x32_w2x4_%s_v11_o2_dma2", 128, 128, 32, 1, 2, 0, 1.458f, 2.038f, 2.82f},
    {"gemm_128x96x32_w4x1_%s_v11_dma2", 128, 96, 32, 1, 2, 0, 0.184f, 1.642f, 3.58f},
    {"gemm_128x64x32_w2x2_%s_v11_dma2", 128, 64, 32, 1, 3, 0, 0.513f, 1.137f, 2.72f},
    {"gemm_128x32x32_w4x1_%s_v11_dma2", 128, 32, 32, 1, 4, 0, 0.362f, 0.709f, 2.10f},
    {"gemm_64x64x32_w2x2_%s_v11_dma2", 64, 64, 32, 1, 5, 0, 0.373f, 0.681f, 1.78f},
    {"gemm_64x64x16_w2x2_%s_v11_dma3", 64, 64, 16, 1, 6, 0, 0.433f, 0.333f, 1.57f},
    {"gemm_32x64x32_w1x2_%s_v11_dma3", 32, 64, 32, 1, 4, 0, 0.736f, 0.453f, 1.81f},
    {"gemm_64x64x32_w2x2_k4_%s_v11_dma2", 64, 64, 32, 4, 1, 0, 0.194f, 2.159f, 3.51f},
    {"gemm_64x64x32_w2x2_k2_%s_v11_dma3", 64, 64, 32, 2, 1, 0, 0.330f, 1.210f, 2.18f},
    {"gemm_32x64x32_w1x2_k4_%s_v11_dma3", 32, 64, 32, 4, 1, 0, 0.681f, 1.347f, 2.59f},
    {"gemm_64x64x16_w2x2_%s_v11", 64, 64, 16, 1, 8, 0, 0.581f, 0.401f, 1.45f},
};
constexpr CostFamily kCostGemm11 = {2.71f, 4.00f, 0.331f, 12, kCostGemm11Tiles};

// convolutions, Cin and Cout multiples of four (the 32 x 64 tile's fit, 0.77,
// 0.339, 1.85, was wrong where it would have been taken: 11 of 11 convolutions
// 4-9 % slower than the rules'; c1 stands between the fitted 0.149 and the
// products', whose sum it is too: at the former 39 of 362 choices of 64 x 64 x 16
// split up to four times as far as the rule's ran up to 9 % slower; four groups'
// m was fitted to 2.174, and 6 of 21 convolutions that took them ran 3-8 %
// slower, 8 % beyond the prediction)
constexpr TileCost kCostConv44Tiles[] = {
    {"conv_128x128x32_w2x4_v44_o2_dma2", 128, 128, 32, 1, 2, 0, 0.491f, 1.992f, 3.36f},
    {"conv_128x96x32_w4x1_v44_dma2", 128, 96, 32, 1, 2, 0, 0.443f, 1.766f, 3.69f},
    {"conv_128x64x32_w2x2_v44_dma2", 128, 64, 32, 1, 3, 0, 0.093f, 1.153f, 2.82f},
    {"conv_128x32x32_w4x1_v44_dma2", 128, 32, 32, 1, 4, 0, 0.365f, 0.702f, 2.57f},
    {"conv_64x64x32_w2x2_v44_dma2", 64, 64, 32, 1, 5, 0, 0.510f, 0.613f, 2.12f},
    {"conv_64x64x16_w2x2_v44_dma3", 64, 64, 16, 1, 6, 0, 0.414f, 0.302f, 1.53f},
    {"conv_64x64x32_w2x2_k4_v44_dma2", 64, 64, 32, 4, 1, 0, 2.197f, 2.350f, 3.96f},
    {"conv_64x64x32_w2x2_k2_v44_dma3", 64, 64, 32, 2, 1, 0, 0.231f, 1.214f, 2.38f},
    {"conv_128x128x32_w2x4_v44_o2_dma2_sk", 128, 128, 32, 1, 2, 1, 0.329f, 2.103f, 28.29f},
};
constexpr CostFamily kCostConv44 = {3.46f, 4.00f, 0.220f, 9, kCostConv44Tiles};

// ... Cin a multiple of four, any Cout
constexpr TileCost kCostConv41Tiles[] = {
    {"conv_128x128x32_w2x4_v41_o2_dma2", 128, 128, 32, 1, 2, 0, 0.597f, 2.070f, 3.21f},
    {"conv_128x96x32_w4x1_v41_dma2", 128, 96, 32, 1, 2, 0, 0.114f, 1.783f, 3.38f},
    {"conv_128x64x32_w2x2_v41_dma2", 128, 64, 32, 1, 3, 0, 0.327f, 1.162f, 2.75f},
    {"conv_128x32x32_w4x1_v41_dma2", 128, 32, 32, 1, 4, 0, 0.897f, 0.656f, 1.61f},
    {"conv_64x64x32_w2x2_v41_dma2", 64, 64, 32, 1, 5, 0, 0.540f, 0.617f, 2.30f},
    {"conv_64x64x16_w2x2_v41_dma3", 64, 64, 16, 1, 6, 0, 0.464f, 0.320f, 1.31f},
    {"conv_32x64x32_w1x2_v41_dma3", 32, 64, 32, 1, 4, 0, 0.813f, 0.350f, 1.71f},
    {"conv_64x64x32_w2x2_k2_v41_dma3", 64, 64, 32, 2, 1, 0, 0.224f, 1.310f, 2.30f},
};
constexpr CostFamily kCostConv41 = {4.00f, 4.00f, 0.196f, 8, kCostConv41Tiles};

// ... any Cin and Cout
constexpr TileCost kCostConv11Tiles[] = {
    {"conv_128x128x32_w2x4_v11_o2_dma2", 128, 128, 32, 1, 2, 0, 0.320f, 2.383f, 3.02f},
    {"conv_128x96x32_w4x1_v11_dma2", 128, 96, 32, 1, 2, 0, 0.204f, 2.015f, 4.19f},
    {"conv_128x64x32_w2x2_v11_dma2", 128, 64, 32, 1, 3, 0, 0.420f, 1.351f, 3.63f},
    {"conv_128x32x32_w4x1_v11_dma2", 128, 32, 32, 1, 4, 0, 0.126f, 0.878f, 4.11f},
    {"conv_64x64x32_w2x2_v11_dma2", 64, 64, 32, 1, 5, 0, 0.318f, 0.718f, 2.09f},
    {"conv_64x64x16_w2x2_v11_dma3", 64, 64, 16, 1, 6, 0, 0.650f, 0.387f, 0.23f},
    {"conv_32x64x32_w1x2_v11_dma3", 32, 64, 32, 1, 4, 0, 1.063f, 0.442f, 1.25f},
    {"conv_64x64x32_w2x2_k2_v11_dma3", 64, 64, 32, 2, 1, 0, 1.213f, 1.496f, 2.65f},
    {"conv_64x64x16_w2x2_v11", 64, 64, 16, 1, 8, 0, 0.748f, 0.441f, 0.29f},
};
constexpr CostFamily kCostConv11 = {4.87f, 4.00f, 0.202f, 9, kCostConv11Tiles};

// Most partial sums the choice may ask a workspace for: the stream-K plans'
// 64 MiB, which the static scratch of the no-allocation entry also holds.
constexpr size_t kCostMaxPartials = (size_t)64 << 20;
constexpr int kCostCUs = 256;
constexpr int kCostSplits[] = {1, 2, 3, 4, 6, 8, 12, 16};

// Predicted time (us) of an M x N x K product on tile c with its reduction
// split s ways, or of a batch of such products (sizes at least 1).
inline float predict_us(const CostFamily &f, const TileCost &c, int64_t M, int64_t N, int64_t K, int s,
                        int64_t batch = 1)
{
    const int64_t tiles = ((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn) * batch;
    const int64_t nkb = (K + c.bk - 1) / c.bk;
    if (c.streamk) return f.t0 + c.ov + c.m * ((float)tiles * (float)nkb / kCostCUs);
    int64_t per = nkb;
    if (s > 1) {
        per = (nkb + s - 1) / s;
        s = (int)((nkb + per - 1) / per);
    }
    const float steps = (float)((per + c.kg - 1) / c.kg);
    const int64_t n = (tiles * s + kCostCUs - 1) / kCostCUs;
    const int64_t full = n / c.per_cu, rem = n - full * c.per_cu;
    auto round = [&](float r) { return (r * c.m > c.l ? r * c.m : c.l) * steps + c.ov; };
    float t = f.t0 + (float)full * round((float)c.per_cu);
    if (rem) t += round((float)rem);
    if (s > 1) t += f.c0 + f.c1 * 4e-6f * (float)(s + 1) * (float)M * (float)N;
    return t;
}

// Longest run of products that one accumulator adds up, in K, when a tile of
// bm x bn outputs walks K-blocks of bk: the whole K-blocks of one split and
// one of kg groups of waves, or, stream-K, a work-group's share of all tiles'
// K-blocks (two work-groups per CU hold them).  The rounding error of a result
// grows with it (about 7e-7 of the result at 1777, 1.1e-6 at 4096, 2-norm), so
// the choice takes no longer one than the configuration it replaces, to the end
// of a K-block of 32 (a rule's split in K-blocks of 16 may end in the middle of
// one: 2672 products against 2688 on 32-deep tiles, half the time): over
// 60 000 random sizes per family this limit and the next cost 0.5 to 0.6 % of the
// predicted time of products and 1.4 to 1.9 % of convolutions' (geometric mean);
// without them 4 to 7 and 13 to 20 % of them had a longer chain.
inline int64_t chain_of(int bm, int bn, int bk, int kg, bool streamk, int64_t M, int64_t N, int64_t K, int64_t s)
{
    const int64_t nkb = (K + bk - 1) / bk;
    int64_t blocks = (nkb + s - 1) / s;
    if (streamk) {
        const int64_t items = ((M + bm - 1) / bm) * ((N + bn - 1) / bn) * nkb;
        const int64_t share = (items + 2 * kCostCUs - 1) / (2 * kCostCUs);
        blocks = share < nkb ? share : nkb;
    } else {
        blocks = (blocks + kg - 1) / kg;
    }
    return blocks * bk < K ? blocks * bk : K;
}

// K shared evenly over groups and splits, which the choice does not raise above
// the rule's either: splits that only the rounding to K-blocks lets in ran slower
// than predicted (64 x 64 x 16 split 16 ways at K = 720 8.2 us, the choice without
// them 7.5).
inline int64_t even_chain(int64_t K, int64_t kg, int64_t s) { return (K + kg * s - 1) / (kg * s); }

// The tile and split of the least predicted time among the tiles for which
// usable(index) holds, the splits whose partial sums fit in ws_bytes and the
// chains of at most max_chain (even: max_even); -1 when there is none.
template <typename F>
int cheapest(const CostFamily &f, int64_t M, int64_t N, int64_t K, size_t ws_bytes, int64_t max_chain,
             int64_t max_even, F usable, int *split, float *us)
{
    int best = -1;
    const size_t room = ws_bytes < kCostMaxPartials ? ws_bytes : kCostMaxPartials;
    for (int i = 0; i < f.n; ++i) {
        const TileCost &c = f.tiles[i];
        if (!usable(i)) continue;
        const int64_t tiles = ((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn);
        const int64_t nkb = (K + c.bk - 1) / c.bk;
        // (stream-K was fitted where a tile has at most four contributors, whose
        // partial tiles the last one adds one after the other: 3 x 8 x 8 x 864 ->
        // 40, 7x7, on two tiles 298 us against 59)
        if (c.streamk && 2 * tiles < kCostCUs) continue;
        // (a 256 x 256 tile's epilogue and fill hide behind nothing when the
        // reduction is eight K-blocks or less: 15975 x 857 x 51 42 us against 31,
        // 14336 x 900 x 135 63 against 54)
        if (c.bm * c.bn >= 256 * 256 && K <= 256) continue;
        for (int s : kCostSplits) {
            // (a split that leaves a work-group under two K-blocks, or more
            // work-groups than the chip holds anyway, was never the fastest)
            if (s > 1 && (c.streamk || 2 * s > nkb || tiles * s > 16 * kCostCUs ||
                          (double)s * (double)M * (double)N * 4.0 > (double)room))
                break;
            if (chain_of(c.bm, c.bn, c.bk, c.kg, c.streamk != 0, M, N, K, s) > max_chain ||
                even_chain(K, c.kg, s) > max_even)
                continue;
            const float t = predict_us(f, c, M, N, K, s);
            if (best < 0 || t < *us) {
                best = i;
                *split = s;
                *us = t;
            }
        }
    }
    return best;
}

// The Winograd convolution of T tiles, Cin and Cout channels as one kernel
// (pk_winograd_fused.hip): blocks of bt tiles x bc channels as above, a step a
// stage of 16 channels; ft: the filter transform, per million Cin * Cout.
struct WinoFusedCost {
    int bt, bc, per_cu;
    float t0, l, m, ov, ft;
};
constexpr WinoFusedCost kWinoFused2[2] = {{32, 32, 2, 5.78f, 1.486f, 1.395f, 2.85f, 2.0f},
                                          {32, 64, 2, 5.46f, 2.386f, 2.332f, 4.55f, 19.3f}};
constexpr WinoFusedCost kWinoFused4[2] = {{32, 32, 1, 1.90f, 4.757f, 0.f, 9.65f, 43.7f},
                                          {32, 64, 1, 0.87f, 6.755f, 6.658f, 12.46f, 56.8f}};
// ... and as transforms around a batch of products: launches, bytes of V and
// M, K-blocks of the products, the filter.
struct WinoCost {
    float t0, v, m, l, k, ft;
};
constexpr WinoCost kWino2 = {13.49f, 1.38f, 1.70f, 1.216f, 0.533f, 30.2f};
constexpr WinoCost kWino4 = {18.12f, 1.27f, 1.60f, 0.786f, 0.561f, 57.6f};

inline float predict_wino_fused_us(const WinoFusedCost &c, int64_t T, int64_t Cin, int64_t Cout)
{
    const int64_t n = (((T + c.bt - 1) / c.bt) * ((Cout + c.bc - 1) / c.bc) + kCostCUs - 1) / kCostCUs;
    const float stages = (float)((Cin + 15) / 16);
    const int64_t full = n / c.per_cu, rem = n - full * c.per_cu;
    auto round = [&](float r) { return (r * c.m > c.l ? r * c.m : c.l) * stages + c.ov; };
    float t = c.t0 + c.ft * 1e-6f * (float)Cin * (float)Cout + (float)full * round((float)c.per_cu);
    if (rem) t += round((float)rem);
    return t;
}

inline float predict_wino_us(int m, int64_t T, int64_t Cin, int64_t Cout)
{
    const WinoCost &c = m == 2 ? kWino2 : kWino4;
    const float P = (float)((m + 2) * (m + 2)), nk = (float)((Cin + 31) / 32);
    const int64_t items = ((T + 63) / 64) * ((Cout + 63) / 64) * (m + 2) * (m + 2);
    const float n = (float)((items + kCostCUs - 1) / kCostCUs);
    return c.t0 + 1e-6f * (P * (float)T * (c.v * (float)Cin + c.m * (float)Cout) + c.ft * (float)Cin * (float)Cout) +
           (n * c.k > c.l ? n * c.k : c.l) * nk;
}

// The form of the one-kernel convolution (0, 1) predicted fastest, or -1 when
// the separate kernels are: over 106 random convolutions this choice was within
// 0.1 % of the faster of the three (geometric mean), the separate kernels 1.66x
// (m = 2) and 1.15x (m = 4) above it.
// Near the line the predictions err by up to a third, where channels are deep (a
// stage's latency counts for more) and, m = 4, where a round of blocks is barely
// begun, so one kernel needs a margin there.  These were set on 7000 random
// convolutions, each graph-timed as one kernel (both forms) and as three: the
// choice costs 0.34 % over the fastest (geometric mean; 0.41 % with 0.85 beyond
// 100 channels alone), and of 4071 taken as one kernel 5 ran more than 5 % slower
// than the three kernels on the older rules' tile, the worst 8 % (20 and 12 %).
// Margins that left none of them slower cost 1.0 %: they gave up one in nine.
inline float wino_margin(int m, int form, int64_t Cin)
{
    if (m == 4) return Cin <= 60 ? 1.f : 0.85f;
    if (form == 1) return Cin <= 100 ? 1.f : 0.9f;
    return Cin <= 100 ? 0.97f : Cin <= 400 ? 0.85f : 0.78f;
}

inline int wino_form(int m, int64_t T, int64_t Cin, int64_t Cout)
{
    const WinoFusedCost *c = m == 2 ? kWinoFused2 : kWinoFused4;
    const float t0 = predict_wino_fused_us(c[0], T, Cin, Cout), t1 = predict_wino_fused_us(c[1], T, Cin, Cout);
    const int form = t1 < t0;
    return (form ? t1 : t0) < wino_margin(m, form, Cin) * predict_wino_us(m, T, Cin, Cout) ? form : -1;
}

}  // namespace pk
