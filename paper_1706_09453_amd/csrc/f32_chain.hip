// Launches of the ascending-k fp32 sums on the matrix cores.
#include "f32_chain_kernels.hpp"
#include "launch.hpp"

namespace bnn {
namespace {

template <int FM, int FN, int WR, int KC, int ACT, bool WREAL, bool VEC>
void launch_chain_tile(const ChainArgs& a) {
    constexpr int TM = 16 * FM * WR, TN = 64 * FN / WR;
    constexpr unsigned lds = f32_chain_lds(TM, TN, KC);
    static std::atomic<uint64_t> allowed{0};
    (void)allow_lds(&f32_chain_kernel<FM, FN, WR, KC, ACT, WREAL, VEC>, lds, allowed);   // (refused: the launch fails)
    const int cols = ACT == ACT_SIGN ? a.yw32 * 32 : a.N;   // Sign: every word of a row of Y is written
    const dim3 grid((unsigned)((a.M + TM - 1) / TM), (unsigned)((cols + TN - 1) / TN));
    f32_chain_kernel<FM, FN, WR, KC, ACT, WREAL, VEC><<<grid, 256, lds, a.st>>>(a.X, a.W, a.scale, a.bias, a.M, a.K, a.N, a.w32, a.Y, a.yw32);
}
// Workgroup tile: the one whose fullest CU has the least to multiply, counting what a tile of that size loses to its
// memory instructions (rates measured at 4096 x 2048 x 2048: 132 TFLOP/s with 256 x 128 tiles, 129 with 128 x 128, 124
// with 64 x 64, 86 with 32 x 64; at 256 x 2048 x 2048, where the large tiles leave most CUs idle, 8, 15, 58 and 80).
template <int ACT, bool WREAL>
void launch_chain_act(const ChainArgs& a) {
    // 32-bit byte offsets inside a workgroup's rows: 256 rows of at most 2^22 - 1 numbers
    const bool vec = (a.K & 3) == 0 && a.K < (1 << 22) && aligned(a.X, 16) && (!WREAL || aligned(a.W, 16));
    const bool wide = a.N > 65535 * 64 - 64;   // tiles of 64 outputs would not fit the second grid dimension
    // Up to 64 frames: tiles of 16 frames x 64 outputs, one fragment per wave.  The time is the chain itself (K / 4 dependent
    // MFMAs), the same for 1 frame and for 64 as long as the grid fits the chip.  Measured against the vector-ALU kernels
    // that took 1 or 2 frames per workgroup: real weights 16 x 440 x 2048 12.1 -> 5.8 us, 16 x 2048 x 2048 50 -> 14,
    // 16 x 2047 x 2048 547 -> 16; weight bits 64 x 2048 x 2048 23.6 -> 17.7, 64 x 4096 x 4096 69 -> 33.
    if (a.M <= 64 && !wide) {
        if (vec) launch_chain_tile<1, 1, 1, 128, ACT, WREAL, true>(a);
        else launch_chain_tile<1, 1, 1, 128, ACT, WREAL, false>(a);
        return;
    }
    if (!vec) {
        if (wide) launch_chain_tile<4, 4, 2, 32, ACT, WREAL, false>(a);
        else launch_chain_tile<2, 2, 2, 64, ACT, WREAL, false>(a);
        return;
    }
    auto cost = [&](int tm, int tn, double rate) {
        const int64_t wgs = (int64_t)((a.M + tm - 1) / tm) * ((a.N + tn - 1) / tn);
        return (double)((wgs + 255) / 256) * tm * tn / rate;
    };
    const double c[4] = {cost(256, 128, 132), cost(128, 128, 129), cost(64, 64, 124), cost(32, 64, 86)};
    int best = 0;
    for (int i = 1; i < (wide ? 2 : 4); ++i)
        if (c[i] < c[best]) best = i;
    if (best == 0) launch_chain_tile<8, 4, 2, 32, ACT, WREAL, true>(a);
    else if (best == 1) launch_chain_tile<4, 4, 2, 32, ACT, WREAL, true>(a);
    else if (best == 2) launch_chain_tile<2, 2, 2, 64, ACT, WREAL, true>(a);
    else launch_chain_tile<1, 2, 2, 128, ACT, WREAL, true>(a);
}
template <bool WREAL>
void launch_chain(const ChainArgs& a, int act) {
    if (act == ACT_SIGN) launch_chain_act<ACT_SIGN, WREAL>(a);
    else if (act == ACT_HARDTANH) launch_chain_act<ACT_HARDTANH, WREAL>(a);
    else if (act == ACT_SIGMOID) launch_chain_act<ACT_SIGMOID, WREAL>(a);
    else launch_chain_act<ACT_LINEAR, WREAL>(a);
}

}  // namespace

void launch_chain_bits(const ChainArgs& a, int act) { launch_chain<false>(a, act); }
void launch_chain_real(const ChainArgs& a, int act) { launch_chain<true>(a, act); }

}  // namespace bnn
