// Launches of the ascending-k fp32 sums on the matrix cores; the two translation units (weight bits, real weights) compile
// side by side.
#pragma once

#include "f32_chain_kernels.hpp"
#include "launch.hpp"

namespace bnn {
namespace {

template <int FM, int FN, int WR, int KC, int ACT, bool WREAL, bool VEC, bool SKIP = false>
void launch_chain_tile(const ChainArgs& a) {
    constexpr int TM = 16 * FM * WR, TN = 64 * FN / WR;
    constexpr unsigned lds = f32_chain_lds(TM, TN, KC);
    if constexpr (lds > 65536) {
        static std::atomic<uint64_t> allowed{0};
        (void)allow_lds(&f32_chain_kernel<FM, FN, WR, KC, ACT, WREAL, VEC, SKIP>, lds, allowed);   // (refused: the launch fails)
    }
    const int cols = ACT == ACT_SIGN ? a.yw32 * 32 : a.N;   // Sign: every word of a row of Y is written
    const dim3 grid((unsigned)((a.M + TM - 1) / TM), (unsigned)((cols + TN - 1) / TN));
    f32_chain_kernel<FM, FN, WR, KC, ACT, WREAL, VEC, SKIP><<<grid, 256, lds, a.st>>>(a.X, a.W, a.scale, a.bias, a.M, a.K, a.N, a.w32, a.Y, a.yw32, cleared_by(a.clear, grid));
}
// Workgroup tile: the one whose fullest CU has the least to multiply, counting what a tile of that size loses to its
// memory instructions (TFLOP/s: 132 with 256 x 128 tiles, 129 with 128 x 128 and 124 with 64 x 64, measured at 4096 x 2048 x 2048; 112
// with 32 x 64, 90 with 16 x 64, 70 with real weights, such that over 35000 sizes of 17 to 9000 frames, 68 to 4096 inputs and 200 to
// 4096 outputs, timed in every tile, the choice costs least: 1.1 % more than the best tile with weight bits, 0.4 % with real weights.  The
// rates these tiles had before their chunks of 64, 86 and 71, or 76, cost 2.7 and 2.0 %: 588 x 256 x 4096 with real weights 22.8 us in 64 x
// 64 tiles, 18.0 in 32 x 64; no size got slower by more than 2 %).
// Tiles of 32 x 64 take chunks of 64: with 128, half as many barriers but a first chunk that takes twice as long to arrive and a workgroup
// that shares its CU with no other, 256 x 2048 x 2048 took 25.0 us, 21.6 now (real weights 26.9 and 23.6), 256 x 440 x 2048 9.0 and
// 7.5, 256 x 3400 x 2048 40.0 and 34.2.
template <int ACT, bool WREAL>
void launch_chain_act(const ChainArgs& a) {
    // 32-bit byte offsets inside a workgroup's rows: 256 rows of at most 2^22 - 1 numbers
    const bool vec = (a.K & 3) == 0 && a.K < (1 << 22) && aligned(a.X, 16) && (!WREAL || aligned(a.W, 16));
    const bool wide = a.N > 65535 * 64 - 64;   // tiles of 64 outputs would not fit the second grid dimension
    auto tiles = [&](int tm, int tn) { return (int64_t)((a.M + tm - 1) / tm) * ((a.N + tn - 1) / tn); };
    // Tiles of 16 frames x 64 outputs, one fragment per wave: the time is the chain itself (K / 4 dependent MFMAs), the same
    // for 1 frame and for 64 as long as the grid fits the chip, 15 us for K = 2048 where 32 x 64 tiles take 21 (which is what
    // its rate in the model stands for).  Against the vector-ALU kernels: real weights 16 x 440 x 2048 12.1 -> 5.8 us,
    // 16 x 2048 x 2048 50 -> 14, 16 x 2047 x 2048 547 -> 16; weight bits 64 x 4096 x 4096 69 -> 33, 65 x 440 x 512
    // 6.2 -> 5.2, 256 x 2047 x 512 26 -> 15 (8.6 and 37 with the larger tiles).  Chunks of 64 for the weight bits (17.7 us
    // with 128 at K = 2048), of 128 for real weights, whose staging is spread over the chunk (13.9 us, 14.5 with 64).
    constexpr int kFewKC = WREAL ? 128 : 64;
    const double few_rate = WREAL ? (vec ? 70 : 60) : (vec ? 90 : 71);   // (84 KiB of LDS with real weights: one workgroup per CU)
    auto few = [&](auto v) { launch_chain_tile<1, 1, 1, kFewKC, ACT, WREAL, decltype(v)::value, true>(a); };
    const std::true_type yes;
    const std::false_type no;
    // Short sums in more tiles than the chip holds: what a workgroup does besides its products decides, so several of them
    // share a CU and no chunk is longer than the sum needs.  Real weights, 64 x 64 tiles with chunks of 32 (four workgroups per
    // CU): 1500 x 16 x 2048 7.2 us on the vector ALU, 10.6 in the tiles of the model, 6.5 here; 16384 x 64 x 2048 100, 73 and
    // 58.  Weight bits: 1500 x 16 x 2048 8.8, 10.7 and 8.1; 16384 x 48 x 2048 72, 73 and 64 in 64 x 128 tiles with chunks of
    // 32; 2500 x 48 x 2048 16.1 and 15.3 in 64 x 64 tiles that leave the unused part of their chunk out.
    // (A quarter of a gigabyte of fp32 outputs is written faster by the larger tiles, unless their chunks are half empty:
    // 16384 x 32 x 4096 weight bits 116 us and 128 here, x 48 151 and 138.)
    const bool huge = ACT != ACT_SIGN && tiles(64, 64) > 8192 && (a.K <= 32 || a.K == 64);
    if (a.K <= 64 && !wide && tiles(16, 64) > 256 && !huge) {
        if constexpr (WREAL) {
            if (vec) launch_chain_tile<2, 2, 2, 32, ACT, true, true, true>(a);
            else launch_chain_tile<2, 2, 2, 32, ACT, true, false, true>(a);
            return;
        } else if (vec) {
            if (tiles(16, 64) <= 512) return few(yes);   // (three of them per CU: 600 x 48 x 512 3.8 us, 4.7 in 64 x 64 tiles)
            const int64_t t = tiles(64, 128);            // (two of them per CU)
            if (t > 768 || (a.K <= 32 && t > 256 && t <= 512)) {
                if (a.K & 31) launch_chain_tile<2, 4, 2, 32, ACT, false, true, true>(a);
                else launch_chain_tile<2, 4, 2, 32, ACT, false, true>(a);
                return;
            }
            if (a.K <= 48) return launch_chain_tile<2, 2, 2, 64, ACT, false, true, true>(a);
        }
    }
    auto cost = [&](int tm, int tn, double rate) { return (double)((tiles(tm, tn) + 255) / 256) * tm * tn / rate; };
    const double c[5] = {cost(256, 128, 132), cost(128, 128, 129), cost(64, 64, 124), cost(32, 64, 112), cost(16, 64, few_rate)};
    if (!vec) {
        if (wide) launch_chain_tile<4, 4, 2, 32, ACT, WREAL, false>(a);
        else if (c[4] < c[2]) few(no);
        else launch_chain_tile<2, 2, 2, 64, ACT, WREAL, false>(a);
        return;
    }
    int best = 0;
    for (int i = 1; i < (wide ? 2 : 5); ++i)
        if (c[i] < c[best]) best = i;
    if (best == 0) launch_chain_tile<8, 4, 2, 32, ACT, WREAL, true>(a);
    else if (best == 1) launch_chain_tile<4, 4, 2, 32, ACT, WREAL, true>(a);
    else if (best == 2) launch_chain_tile<2, 2, 2, 64, ACT, WREAL, true>(a);
    else if (best == 3) launch_chain_tile<1, 2, 2, 64, ACT, WREAL, true>(a);
    else few(yes);
}
template <bool WREAL>
void launch_chain(const ChainArgs& a, int act) {
    if (act == ACT_SIGN) launch_chain_act<ACT_SIGN, WREAL>(a);
    else if (act == ACT_HARDTANH) launch_chain_act<ACT_HARDTANH, WREAL>(a);
    else if (act == ACT_SIGMOID) launch_chain_act<ACT_SIGMOID, WREAL>(a);
    else launch_chain_act<ACT_LINEAR, WREAL>(a);
}

}  // namespace
}  // namespace bnn
