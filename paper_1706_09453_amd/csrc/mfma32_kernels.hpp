// Matrix-core arm of the binary x binary product (paper Sec. 2.3), large-batch version:
// V_MFMA_F32_32X32X64_F8F6F4 with both operands in the 4-bit float format, whose products and fp32 sums are the exact integers
// (see mfma_kernels.hpp).  On 16-byte rows with K % 512 == 0 the operands go through LDS and are multiplied as 0 and 1 (the
// pinned variants, below); other rows, and operands of 2 GiB and more, from memory to registers as +-1.
//
// Why this shape: every operand word a lane holds (32 elements of one row) has to be expanded from bits to nibbles by the
// vector ALU (five to seven instructions), and the SIMD issues either a VALU instruction or an MFMA per 4 clocks.  What counts is
// therefore expansions per multiply-accumulate: a wave that owns a 128 x 64 tile of [M][N] as 4 x 2 accumulator fragments of
// 32 x 32 expands 6 words for 8 MFMAs of 65536 MACs each, about half the expansion work per MAC of the 16 x 16 x 128 kernel with
// 64 x 64 wave tiles.
//
// K advances in super-steps of 512 bits; lane (r = lane%32, g = lane/32) takes eight words of row r of every fragment, one per
// MFMA step.  Inside a fragment the order of k is therefore permuted, identically for both operands.
// A workgroup is 2 x 2 waves: a (64 WM) x (64 WN) tile; at M = 4096, N = 2048 with WM = 4, WN = 2 that is
// 256 workgroups, one wave per SIMD of the chip.
#pragma once

#include "mfma_kernels.hpp"

namespace bnn {

typedef float v16f __attribute__((ext_vector_type(16)));

// 0/1 operands (pinned variants).  With h and w the bits of a frame and of a weight row read as 0 and 1,
//     sum_k (+-1)(+-1) = 4 sum_k h w - 2 popcount(h) - 2 popcount(w) + K,        sum_k h (+-1) = 2 sum_k h w - popcount(h),
// and a nibble of the 4-bit float format with a single bit set is a power of two (bit 0: 0.5, bit 1: 1, bit 2: 2), so most of
// an operand's dwords are one AND of the packed word with a mask, with the other operand's shifted to the reciprocal:
//     bit of the word's nibble      0            1            2            3
//     frames                   w & 1..: 0.5   w & 2..: 1   w & 4..: 2   (w >> 2) & 2..: 1
//     weights             (w << 2) & 4..: 2   w & 2..: 1   (w >> 2) & 1..: 0.5   (w >> 2) & 2..: 1
// Five and six instructions per word, and one for its popcount, where +-1 takes seven; and three quarters of the products are
// 0, which cost the matrix cores less energy: what bounds a large product here is the clock that the chip holds under them.
// 16384 x 4096 x 4096: 42.5 clocks per MFMA and SIMD at 1.86 GHz, matrix cores busy 75 % of them, 5.9 vector instructions per MFMA
// with the epilogue (profiles/forward_c3_c4_counters.txt).
struct ExpandMasks { uint32_t b0, b1, b2; };
__device__ __forceinline__ ExpandMasks expand_masks() {
    ExpandMasks m{0x11111111u, 0x22222222u, 0x44444444u};
    asm volatile("" : "+s"(m.b0), "+s"(m.b1), "+s"(m.b2));
    return m;
}

struct Raw8 {
    uint4 lo, hi;   // words 0..3 and 4..7 of a lane's share of a super-step
};

// Fetch words [16*S + 8*g, +8) of a packed row.  ALIGNED: rows are 16-byte aligned and whole super-steps
// long.  Otherwise each word is bounds-checked against the row length and reads as 0.
template <bool ALIGNED>
__device__ __forceinline__ Raw8 load_raw8(const uint32_t* __restrict__ row, int S, int g, int w32) {
    const int base = S * 16 + g * 8;
    Raw8 v;
    if constexpr (ALIGNED) {
        v.lo = *reinterpret_cast<const uint4*>(row + base);
        v.hi = *reinterpret_cast<const uint4*>(row + base + 4);
    } else {
        v.lo.x = (base + 0 < w32) ? row[base + 0] : 0u;
        v.lo.y = (base + 1 < w32) ? row[base + 1] : 0u;
        v.lo.z = (base + 2 < w32) ? row[base + 2] : 0u;
        v.lo.w = (base + 3 < w32) ? row[base + 3] : 0u;
        v.hi.x = (base + 4 < w32) ? row[base + 4] : 0u;
        v.hi.y = (base + 5 < w32) ? row[base + 5] : 0u;
        v.hi.z = (base + 6 < w32) ? row[base + 6] : 0u;
        v.hi.w = (base + 7 < w32) ? row[base + 7] : 0u;
    }
    return v;
}

// Sign(fma(scale, unit * a, bias)), with unit * a an integer below 2^24, as the sign bit of fma(neg_scale, a, neg_bias).  The two
// fused multiply-adds are each other's negative, up to a power of two that is taken from the side that stays in range, so the
// sign bit is set exactly where the first is above zero, if the second is never -0 and never a NaN.  neg_bias is never -0, and
// the exact result is a multiple of 2^-149 that does not underflow, so a zero comes out as +0.  NaNs are avoided by what the
// column is replaced with: a NaN anywhere gives bit 0 for every a; an infinite scale gives 1 where scale * a is +inf and bias is
// not -inf (at a = 0, or against a bias of -inf, the sum is a NaN or -inf).
struct SignColumn { float neg_scale, neg_bias; };
__device__ __forceinline__ SignColumn sign_column(float scale, float bias, float unit) {
    const float inf = __builtin_inff();
    const bool big = __builtin_fabsf(scale) == inf;
    const bool never = scale != scale || bias != bias || (big && bias == -inf);
    scale = never ? 0.0f : (big ? __builtin_copysignf(1.0f, scale) : scale);
    bias = never || big ? 0.0f : bias;
    // (a scale of 2^100 and more: beside any a but 0 a bias below 1 does not count, and at a = 0 only its sign does)
    const bool wide = __builtin_fabsf(scale) >= 0x1p100f;
    return {wide ? -scale : -scale * unit, 0.0f - (wide && __builtin_fabsf(bias) >= 1.0f ? bias / unit : bias)};
}

// 32 x 32 bits across the 32 lanes of a half wave: afterwards bit j of lane i is what bit i of lane j was.  Five exchanges with
// the lane whose number differs in one bit; a lane keeps the half of its bits that stays and takes the other one rotated.
struct TransposeBits {
    uint32_t keep[5], rot[5];
    __device__ __forceinline__ explicit TransposeBits(int lane) {
        constexpr uint32_t kLow[5] = {0x0000FFFFu, 0x00FF00FFu, 0x0F0F0F0Fu, 0x33333333u, 0x55555555u};
#pragma unroll
        for (int t = 0; t < 5; ++t) {
            const int s = 16 >> t;
            keep[t] = (lane & s) ? ~kLow[t] : kLow[t];
            rot[t] = (lane & s) ? (uint32_t)s : (uint32_t)(32 - s);   // to the right
        }
    }
    template <int S>
    static __device__ __forceinline__ uint32_t partner(uint32_t v) {
        return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, 0x1F | (S << 10));
    }
    template <int T, int N>
    __device__ __forceinline__ void step(uint32_t (&w)[N]) const {
        uint32_t p[N];
#pragma unroll
        for (int i = 0; i < N; ++i) p[i] = partner<(16 >> T)>(w[i]);
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const uint32_t o = __builtin_amdgcn_alignbit(p[i], p[i], rot[T]);
            w[i] = (w[i] & keep[T]) | (o & ~keep[T]);
        }
    }
    template <int N>
    __device__ __forceinline__ void run(uint32_t (&w)[N]) const {
        step<0>(w); step<1>(w); step<2>(w); step<3>(w); step<4>(w);
    }
};

// Called inside the product loop, after the first products: the loads that produced sc/bi then stay in front of
// the loop, where they were written, instead of moving next to their use in the epilogue, and by the time this
// point is reached they have long returned (the operand words used by those products were requested later).
template <int WN>
__device__ __forceinline__ void pin_loaded(float (&sc)[WN], float (&bi)[WN]) {
#pragma unroll
    for (int f = 0; f < WN; ++f) asm volatile("" : "+v"(sc[f]), "+v"(bi[f]));
}

__device__ __forceinline__ uint32_t word_of(const Raw8& v, int j) {
    return j < 4 ? word_of(v.lo, j) : word_of(v.hi, j - 4);
}

// Operand fetch of the pinned variants (PINGPONG): both operands of the workgroup's tile go to LDS as they are in memory, one
// bit per element, by loads that write LDS directly (no registers, no LDS store instructions), in stages of 512 bits of every
// row, three stages in rotation; a lane reads 16 bytes of its fragment rows per half-stage.  Fetched straight into registers, a
// fragment load touches 32 rows, 64 different pieces of 16 bytes, and the texture path takes those one after the other: at
// 16384 x 4096 x 4096 a wave then issued an MFMA every 29 ns, where the matrix core needs 13.6 and the expansion fits
// beside it (V independent vector instructions per MFMA, one or two waves per SIMD: V = 5 14.9 ns, V = 6 15.6 to 16.8).
// Measured against that, with the 0/1 operands above: Sign layers 16384 x 4096 x 4096 124 -> 95 us, 65536 x 4096 x 4096 465 -> 328,
// 4096 x 8192 x 2048 29.1 -> 23.8, 4096 x 2048 x 2048 10.5 -> 9.2.
// In LDS a row of a stage is 64 bytes, its four 16-byte slots at slot ^ (row / 4 % 4), so that the 16 lanes that are served
// together read 16 different slots of the 64 banks.
constexpr int kM32Stages = 3;
constexpr int kM32RowBytes = 64;
constexpr int kM32Ldw = 68;   // words per row of the transposing epilogue's slices: 64 columns and a pad
__host__ __device__ constexpr int m32_stage(int WM, int WN) { return (64 * WM + 64 * WN) * kM32RowBytes; }
__host__ __device__ constexpr unsigned m32_lds(int WM, int WN, int ACT, bool PINGPONG) {
    const unsigned loop = PINGPONG ? (unsigned)(kM32Stages * m32_stage(WM, WN) + 2 * 64 * WN * 4) : 0u;   // stages; scale and bias
    unsigned epi = ACT == ACT_SIGN ? 0u : 4u * 32u * kM32Ldw * 4u;
    if (ACT == ACT_LSM_COOP) epi += 4u * 32u * (unsigned)WM * 8u + 64u * (unsigned)WM * 4u;
    return loop > epi ? loop : epi;
}

// PINGPONG (aligned rows only): the fetch described above, with the issue order pinned by scheduling barriers and, for 128-row
// wave tiles (WM = 4), written out instruction slot by slot.  Without it the operands go from memory to registers in an order
// left to the compiler; kept for ragged rows and for operands of 2 GiB and more.
// X01: the activation bits are read as 0/1 instead of -1/+1 (paper Sec. 3.2).  With a the -1/+1 reading of the same
// bits, h = (a + 1) / 2 and h.w = (a.w + sum_k w_k) / 2: the product runs unchanged, every lane counts the 1 bits of
// the weight words it reads anyway (the two lanes that share a row add theirs up), and the epilogue forms
// 0.5 (a.w) + (popcount(w) - K/2), exact in fp32.
// Grid: x = ceil(M / (64*WM)), y = ceil(N / (64*WN)); block = 256 threads; dynamic LDS m32_lds(WM, WN, ACT, PINGPONG).
template <int WM, int WN, int ACT, bool ALIGNED, bool PINGPONG = false, bool X01 = false>
__global__ __launch_bounds__(256, 2) void binx_mfma32_kernel(const uint32_t* __restrict__ Xp, const uint32_t* __restrict__ Wp,
                                                          const float* __restrict__ scale, const float* __restrict__ bias,
                                                          int M, int K, int N, int w32, void* __restrict__ Y, int yw32,
                                                          unsigned int a_bytes, unsigned int b_bytes, int xcd_order,
                                                          const CoopLsm coop) {
    extern __shared__ __attribute__((aligned(16))) unsigned char m32_mem[];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = lane_id();
    const int r = lane & 31;   // row of the operand fragment / column of the accumulator fragment
    const int g = lane >> 5;   // k-group of the operand fragment / row-group of the accumulator fragment
    int tile_m = (int)blockIdx.x, tile_n = (int)blockIdx.y;
    if (xcd_order) {
        // Workgroups go to the 8 XCDs round-robin in dispatch order, and every XCD has its own L2.  Give XCD x a
        // contiguous run of tiles in (frames tile, outputs tile) order, outputs fastest: the workgroups that share
        // a frames tile then run on the same XCD, one after the other, and its rows are fetched into one L2 once.
        const int total = (int)(gridDim.x * gridDim.y);
        const int lin = (int)(blockIdx.y * gridDim.x + blockIdx.x);
        const int x = lin & 7, q = total >> 3, rem = total & 7;
        const int t = x * q + (x < rem ? x : rem) + (lin >> 3);
        tile_m = t / (int)gridDim.y;
        tile_n = t - tile_m * (int)gridDim.y;
    }
    const int m_base = (tile_m * 2 + (wave >> 1)) * (WM * 32);
    const int n_base = (tile_n * 2 + (wave & 1)) * (WN * 32);
    if constexpr (ACT != ACT_LSM_COOP && !PINGPONG) {   // (no barriers)
        if (m_base >= M || n_base >= N) return;   // wave-uniform
    }

    // Scale and bias of this lane's columns, requested before the product so that the epilogue does not wait for
    // them (the pinned variants take them through LDS, in front of the first stage).  Columns past N get scale = bias = 0:
    // their pre-activation is 0, their Sign bit 0 (pad bits stay 0).
    float sc[WN], bi[WN];
    if constexpr (!PINGPONG) {
#pragma unroll
        for (int f = 0; f < WN; ++f) {
            const int n = n_base + f * 32 + r;
            sc[f] = n < N ? (scale ? scale[n] : 1.0f) : 0.0f;
            bi[f] = n < N ? (bias ? bias[n] : 0.0f) : 0.0f;
        }
    }

    int ones[WN];   // X01: 1 bits of this lane's share of the weight rows
#pragma unroll
    for (int f = 0; f < WN; ++f) ones[f] = 0;
    auto count4 = [&](const uint4 (&b)[WN]) {
        if constexpr (X01 && !PINGPONG) {
#pragma unroll
            for (int f = 0; f < WN; ++f)
                ones[f] += __builtin_popcount(b[f].x) + __builtin_popcount(b[f].y) + __builtin_popcount(b[f].z) + __builtin_popcount(b[f].w);
        }
    };

    const float acc0 = PINGPONG && !X01 ? 0.25f * (float)K : 0.0f;
    v16f acc[WM][WN];
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = acc0;

    const int nS = (K + 511) >> 9;
    static_assert(ALIGNED || !PINGPONG, "the pinned pipelines fetch whole 16-byte pieces of whole super-steps");
    if constexpr (PINGPONG) {
        // ---- the wave's share of a stage's loads: 16 rows of the tile each (4 lanes a row), frames rows first.
        constexpr int kStage = m32_stage(WM, WN), AI = WM, BI = WN;   // load instructions per wave: 64 WM (WN) rows / 16 / 4 waves
        const i32x4m ars = raw_buffer(Xp, a_bytes), brs = raw_buffer(Wp, b_bytes);
        const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)m32_mem;
        const int lrow = lane >> 2, lslot = lane & 3;   // row of the instruction's 16, place in the row
        const int lsrc = (lslot ^ ((lrow >> 2) & 3)) * 16;
        int aofs[AI], bofs[BI];
#pragma unroll
        for (int i = 0; i < AI; ++i) {
            const int m = tile_m * (64 * WM) + (wave * AI + i) * 16 + lrow;
            aofs[i] = (m < M ? m : M - 1) * w32 * 4 + lsrc;
        }
#pragma unroll
        for (int i = 0; i < BI; ++i) {
            const int n = tile_n * (64 * WN) + (wave * BI + i) * 16 + lrow;
            bofs[i] = (n < N ? n : N - 1) * w32 * 4 + lsrc;
        }
        auto request = [&](int S, int slot) {   // stage S of K to LDS stage `slot`
            const uint32_t base = lds0 + (uint32_t)(slot * kStage);
#pragma unroll
            for (int i = 0; i < AI; ++i) load_lds16(ars, aofs[i], S * 64, base + (uint32_t)((wave * AI + i) * 16 * kM32RowBytes));
#pragma unroll
            for (int i = 0; i < BI; ++i) load_lds16(brs, bofs[i], S * 64, base + (uint32_t)((64 * WM + (wave * BI + i) * 16) * kM32RowBytes));
        };
        // ---- the lane's operand words of half-stage h: 16 bytes per fragment row, half 0 from slots 0 and 1, half 1 from 2 and 3
        const int arow = ((wave >> 1) * (WM * 32) + r) * kM32RowBytes, brow = (64 * WM + (wave & 1) * (WN * 32) + r) * kM32RowBytes;
        const int so0 = ((0 + g) ^ ((r >> 2) & 3)) * 16, so1 = ((2 + g) ^ ((r >> 2) & 3)) * 16;
        auto fetch = [&](uint4 (&a)[WM], uint4 (&b)[WN], int slot, int so) {
            const unsigned char* base = m32_mem + slot * kStage + so;
#pragma unroll
            for (int f = 0; f < WN; ++f) b[f] = *reinterpret_cast<const uint4*>(base + brow + f * (32 * kM32RowBytes));
#pragma unroll
            for (int f = 0; f < WM; ++f) a[f] = *reinterpret_cast<const uint4*>(base + arow + f * (32 * kM32RowBytes));
        };
        // One barrier per stage, in its middle: behind it stage S + 1 is complete in LDS and stage S has been read by every
        // wave, so its place takes stage S + 3.  (lgkmcnt: the wave's own reads of stage S, requested in front of the products of
        // its first half; the compiler places no wait for them, their first use comes behind the barrier.)
        auto turn = [&](int S) {
            if (S + 2 < nS) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(AI + BI) : "memory");   // stage S + 2 may be on its way
            else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
        };
        const uint32_t affine_lds = lds0 + (uint32_t)(kM32Stages * kStage);   // [2][64 WN]: scale, bias
        {
            static_assert(WN == 2, "two waves bring the tile's 128 scales, two its biases");
            const float* src = (wave >> 1) ? bias : scale;
            const int n = tile_n * (64 * WN) + (wave & 1) * 64 + lane;
            if (src) load_lds4(raw_buffer(src, (unsigned int)N * 4u), (n < N ? n : N - 1) * 4, 0, affine_lds + (uint32_t)wave * 256u);
        }
        auto next_slot = [](int s) { return s == kM32Stages - 1 ? 0 : s + 1; };
        request(0, 0);
        if (nS > 1) request(1, 1);
        if (nS > 2) request(2, 2);
#pragma unroll
        for (int i = 0; i < WM; ++i)
#pragma unroll
            for (int j = 0; j < WN; ++j) asm volatile("" : "+v"(acc[i][j]));   // the accumulators are set while the first stage is on its way
        const ExpandMasks em = expand_masks();
        int ones_a[WM], ones_b[WN];   // 1 bits of this lane's share of its fragment rows
#pragma unroll
        for (int f = 0; f < WM; ++f) ones_a[f] = 0;
#pragma unroll
        for (int f = 0; f < WN; ++f) ones_b[f] = 0;
        auto count = [](int& n, uint32_t w) { asm volatile("v_bcnt_u32_b32 %0, %1, %0" : "+v"(n) : "v"(w)); };   // (stays where it is written)
        auto clear_hi = [&](v8i& d) { d[4] = 0; d[5] = 0; d[6] = 0; d[7] = 0; };   // unused by the 4-bit format
        // the dwords of a frames word and of a weights word, by class
        auto frames_piece = [&](v8i& d, uint32_t w, int part) {
            if (part == 0) d[0] = (int)(w & em.b0);           // 0.5
            else if (part == 1) d[1] = (int)(w & em.b1);      // 1
            else if (part == 2) d[2] = (int)(w & em.b2);      // 2
            else d[3] = (int)((w >> 2) & em.b1);              // 1 (two instructions)
        };
        auto weights_piece = [&](v8i& d, uint32_t w, int part) {
            if (part == 0) d[0] = (int)((w << 2) & em.b2);    // 2 (two instructions)
            else if (part == 1) d[1] = (int)(w & em.b1);      // 1
            else if (part == 2) d[2] = (int)((w >> 2) & em.b0);   // 0.5 (the shift serves part 3 too)
            else d[3] = (int)((w >> 2) & em.b1);              // 1
        };
        if (nS > 2) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(2 * (AI + BI)) : "memory");
        else if (nS > 1) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(AI + BI) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        // A wave without rows or columns of its own brings its share of the stages and leaves (running along on clamped rows:
        // 10903 x 2048 x 1417 to fp32, 516 tiles of which 43 have 9 columns, 41.5 us, now 36.6; 14529 x 8192 x 32 14.0 and 13.1).  The
        // cooperative epilogue has workgroup barriers: there it does run along, and contributes nothing.
        if constexpr (ACT != ACT_LSM_COOP) {
            if (m_base >= M || n_base >= N) {   // wave-uniform
                for (int S = 0, slot = 0; S < nS; ++S, slot = next_slot(slot)) {
                    turn(S);
                    if (S + 3 < nS) request(S + 3, slot);
                }
                return;
            }
        }
        uint4 a0[WM], b0[WN], a1[WM], b1[WN];
        fetch(a0, b0, 0, so0);
        // (scale and bias here, not in front of the epilogue, where a wave has nothing else to do meanwhile)
        const float* affine_s = reinterpret_cast<const float*>(m32_mem + kM32Stages * kStage) + (wave & 1) * (32 * WN) + r;
#pragma unroll
        for (int f = 0; f < WN; ++f) {
            const bool in = n_base + f * 32 + r < N;
            sc[f] = in ? (scale ? affine_s[f * 32] : 1.0f) : 0.0f;
            bi[f] = in ? (bias ? affine_s[64 * WN + f * 32] : 0.0f) : 0.0f;
        }
        // Issue order inside a half-step, written out and pinned slot by slot.  A wave issues in order, and an MFMA that
        // finds the pipe busy (32 clocks per 32x32x64) blocks whatever follows it.  Here every MFMA is followed by four to
        // seven expansion instructions of operands needed two to eight MFMAs later, which issue in its shadow: the frames
        // fragment fm+1 of this step while fm is multiplied, and the two weights fragments and frames fragment 0 of the
        // NEXT step (taken from the next half-stage's words after the last step of a half-stage) spread over the slots.
        // (64-row tiles with the order left to the compiler, which starts every half-step with seventeen expansions in a row:
        // 315 x 7680 x 4096 15.4 -> 13.6 us, 600 x 2048 x 2048 6.2 -> 5.8.)
        static_assert((WM == 4 || WM == 2) && WN == 2, "the slot plans below are written for 4 x 2 and 2 x 2 fragments");
        v8i bx[2][WN];   // expanded weights: [parity of the step][fragment]
        v8i ax[2];       // expanded frames: fragment fm lives in ax[fm & 1]
        clear_hi(ax[0]); clear_hi(ax[1]);
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int f = 0; f < WN; ++f) clear_hi(bx[t][f]);
        auto half_step = [&](const uint4 (&a)[WM], const uint4 (&b)[WN], const uint4 (&an)[WM], const uint4 (&bn)[WN]) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int pc = j & 1, pn = pc ^ 1;
                // words of the next step: the next word of this set, or the first word of the next set
                const uint32_t wb0 = j < 3 ? word_of(b[0], j + 1) : word_of(bn[0], 0);
                const uint32_t wb1 = j < 3 ? word_of(b[1], j + 1) : word_of(bn[1], 0);
                const uint32_t wa0 = j < 3 ? word_of(a[0], j + 1) : word_of(an[0], 0);
                const uint32_t wa1 = word_of(a[1], j);
                auto count_a = [&](int f) { count(ones_a[f], word_of(a[f], j)); };
                auto count_b = [&](int f) { if constexpr (!X01) count(ones_b[f], word_of(b[f], j)); };
                auto fp = [&](int f, uint32_t w, int p) { frames_piece(ax[f & 1], w, p); };
                auto wp = [&](int f, uint32_t w, int p) { weights_piece(bx[pn][f], w, p); };
#define BNN_MFMA(fm, fn) acc[fm][fn] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(ax[(fm) & 1], bx[pc][fn], acc[fm][fn], 4, 4, 0, 0, 0, 0)
#define BNN_SLOT_END __builtin_amdgcn_sched_barrier(0)
                if constexpr (WM == 4) {
                    const uint32_t wa2 = word_of(a[2], j), wa3 = word_of(a[3], j);
                    BNN_MFMA(0, 0); fp(1, wa1, 0); fp(1, wa1, 1); fp(1, wa1, 2); count_a(0); BNN_SLOT_END;
                    BNN_MFMA(0, 1); fp(1, wa1, 3); wp(0, wb0, 0); wp(0, wb0, 1); BNN_SLOT_END;
                    BNN_MFMA(1, 0); fp(2, wa2, 0); fp(2, wa2, 1); fp(2, wa2, 2); count_a(1); BNN_SLOT_END;
                    BNN_MFMA(1, 1); fp(2, wa2, 3); wp(0, wb0, 2); wp(0, wb0, 3); BNN_SLOT_END;
                    BNN_MFMA(2, 0); fp(3, wa3, 0); fp(3, wa3, 1); fp(3, wa3, 2); count_a(2); count_b(0); BNN_SLOT_END;
                    BNN_MFMA(2, 1); fp(3, wa3, 3); wp(1, wb1, 0); wp(1, wb1, 1); BNN_SLOT_END;
                    // frames fragment 0 of the next step overwrites ax[0], which MFMA (2, *) has finished reading
                    BNN_MFMA(3, 0); fp(0, wa0, 0); fp(0, wa0, 1); fp(0, wa0, 2); count_a(3); count_b(1); BNN_SLOT_END;
                    BNN_MFMA(3, 1); fp(0, wa0, 3); wp(1, wb1, 2); wp(1, wb1, 3); BNN_SLOT_END;
                } else {
                    BNN_MFMA(0, 0); fp(1, wa1, 0); fp(1, wa1, 1); fp(1, wa1, 2); count_a(0); wp(0, wb0, 1); wp(1, wb1, 1); BNN_SLOT_END;
                    BNN_MFMA(0, 1); fp(1, wa1, 3); wp(0, wb0, 0); wp(0, wb0, 2); wp(0, wb0, 3); BNN_SLOT_END;
                    // as above: ax[0], which MFMA (0, *) has finished reading
                    BNN_MFMA(1, 0); fp(0, wa0, 0); fp(0, wa0, 1); fp(0, wa0, 2); count_a(1); count_b(0); wp(1, wb1, 0); BNN_SLOT_END;
                    BNN_MFMA(1, 1); fp(0, wa0, 3); wp(1, wb1, 2); wp(1, wb1, 3); count_b(1); BNN_SLOT_END;
                }
#undef BNN_MFMA
#undef BNN_SLOT_END
            }
        };
        auto pin_low = [](v8i& d) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                int v = d[i];
                asm volatile("" : "+v"(v));
                d[i] = v;
            }
        };
        {   // operands of the very first step
#pragma unroll
            for (int part = 0; part < 4; ++part) {
                weights_piece(bx[0][0], word_of(b0[0], 0), part);
                weights_piece(bx[0][1], word_of(b0[1], 0), part);
                frames_piece(ax[0], word_of(a0[0], 0), part);
            }
        }
        int slot = 0, S = 0;
        do {   // (K > 0: at least one stage)
            const int nslot = next_slot(slot);
            fetch(a1, b1, slot, so1);
            __builtin_amdgcn_sched_barrier(0);
            half_step(a0, b0, a1, b1);
            pin_low(ax[0]);   // expanded in front of the barrier, in the shadow of the last products, not behind it
#pragma unroll
            for (int f = 0; f < WN; ++f) pin_low(bx[0][f]);
            __builtin_amdgcn_sched_barrier(0);
            turn(S);
            fetch(a0, b0, S + 1 < nS ? nslot : slot, so0);   // (behind the last stage: read again, unused)
            if (S + 3 < nS) request(S + 3, slot);
            __builtin_amdgcn_sched_barrier(0);
            half_step(a1, b1, a0, b0);
            __builtin_amdgcn_sched_barrier(0);
            slot = nslot;
        } while (++S < nS);
        // The counts join the sum (see "0/1 operands" above) as one more product per fragment, in bfloat16, eight bits of a count
        // per element of k: acc - popcount(frame) / 2 [- popcount(weights) / 2].  Each of the two lanes of a row brings its own
        // share of the count, and the product adds them up.
        {
            typedef __bf16 bf16x8m __attribute__((ext_vector_type(8)));
            typedef uint32_t u32x4m __attribute__((ext_vector_type(4)));
            auto hi = [](float v) { return __float_as_uint(v) >> 16; };   // (eight significant bits: exact)
            const uint32_t h0 = hi(-0.5f), h1 = hi(-128.0f), h2 = hi(-32768.0f);
            auto share = [&](int ones, uint32_t (&q)[3]) {
                const uint32_t c = (uint32_t)ones;
                q[0] = hi((float)(c & 255u));
                q[1] = hi((float)((c >> 8) & 255u));
                q[2] = hi((float)(c >> 16));
            };
            bf16x8m cb[WN];
#pragma unroll
            for (int f = 0; f < WN; ++f) {
                uint32_t q[3] = {0u, 0u, 0u};
                if constexpr (!X01) share(ones_b[f], q);
                cb[f] = __builtin_bit_cast(bf16x8m, u32x4m{h0 | (h1 << 16), h2 | (q[0] << 16), q[1] | (q[2] << 16), 0u});
            }
#pragma unroll
            for (int f = 0; f < WM; ++f) {
                uint32_t q[3];
                share(ones_a[f], q);
                const bf16x8m ca = __builtin_bit_cast(bf16x8m, X01 ? u32x4m{q[0] | (q[1] << 16), q[2], 0u, 0u}
                                                                   : u32x4m{q[0] | (q[1] << 16), q[2] | (h0 << 16), h1 | (h2 << 16), 0u});
#pragma unroll
                for (int fn = 0; fn < WN; ++fn) acc[f][fn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ca, cb[fn], acc[f][fn], 0, 0, 0);
            }
        }
        // The epilogue takes the stages' place with no barrier of its own: behind the last stage's every wave has what it uses of
        // them in registers and no load is under way (what is read again behind it is not used).
    } else {
        const ExpandConsts ec = expand_consts();
        const uint32_t* arow[WM];
        const uint32_t* brow[WN];
#pragma unroll
        for (int f = 0; f < WM; ++f) {
            const int m = m_base + f * 32 + r;
            arow[f] = Xp + (size_t)(m < M ? m : M - 1) * w32;
        }
#pragma unroll
        for (int f = 0; f < WN; ++f) {
            const int n = n_base + f * 32 + r;
            brow[f] = Wp + (size_t)(n < N ? n : N - 1) * w32;
        }
        Raw8 araw[WM], braw[WN];
#pragma unroll
        for (int f = 0; f < WM; ++f) araw[f] = load_raw8<ALIGNED>(arow[f], 0, g, w32);
#pragma unroll
        for (int f = 0; f < WN; ++f) braw[f] = load_raw8<ALIGNED>(brow[f], 0, g, w32);

        for (int S = 0; S < nS; ++S) {
            Raw8 anext[WM], bnext[WN];
            const int Sn = (S + 1 < nS) ? S + 1 : S;   // the last prefetch re-reads the last step (in bounds, unused)
#pragma unroll
            for (int f = 0; f < WM; ++f) anext[f] = load_raw8<ALIGNED>(arow[f], Sn, g, w32);
#pragma unroll
            for (int f = 0; f < WN; ++f) bnext[f] = load_raw8<ALIGNED>(brow[f], Sn, g, w32);

            if constexpr (X01) {
                uint4 lo[WN], hi[WN];
#pragma unroll
                for (int f = 0; f < WN; ++f) { lo[f] = braw[f].lo; hi[f] = braw[f].hi; }
                count4(lo);
                count4(hi);
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                v8i bx[WN];
#pragma unroll
                for (int f = 0; f < WN; ++f) bx[f] = expand_pm1_fp4(word_of(braw[f], j), ec);
#pragma unroll
                for (int fm = 0; fm < WM; ++fm) {
                    const v8i ax = expand_pm1_fp4(word_of(araw[fm], j), ec);
#pragma unroll
                    for (int fn = 0; fn < WN; ++fn)
                        acc[fm][fn] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(ax, bx[fn], acc[fm][fn], 4, 4, 0, 0, 0, 0);
                }
            }
            pin_loaded(sc, bi);
#pragma unroll
            for (int f = 0; f < WM; ++f) araw[f] = anext[f];
#pragma unroll
            for (int f = 0; f < WN; ++f) braw[f] = bnext[f];
        }
    }

    // ---- epilogue.  Accumulator fragment (fm, fn), register v of lane (r, g) is
    //      dot[m_base + 32 fm + 8 (v/4) + 4 g + v%4][n_base + 32 fn + r] + pad.
    const float pad = (float)(nS * 512 - K);
    constexpr float kUnit = PINGPONG ? (X01 ? 2.0f : 4.0f) : 1.0f;   // what the accumulators are in units of
    float half_wsum[WN];   // X01: popcount(w) - K/2 = (sum_k w_k) / 2 of this lane's columns
#pragma unroll
    for (int f = 0; f < WN; ++f) {
        half_wsum[f] = 0.0f;
        if constexpr (X01 && !PINGPONG) half_wsum[f] = (float)(ones[f] + __shfl_xor(ones[f], 32, kWave)) - 0.5f * (float)K;
    }
    auto dot_of = [&](float a, int fn) -> float {
        const float d = ALIGNED ? a : a - pad;   // whole super-steps: no pad
        if constexpr (PINGPONG) return a * kUnit;
        else if constexpr (X01) return __builtin_fmaf(d, 0.5f, half_wsum[fn]);
        else return d;
    };
    if constexpr (ACT == ACT_SIGN) {
        // A lane gathers the bits of its column over the 32 frames of two fragments, two instructions a bit: the fused multiply-
        // add of the negated layer, whose sign bit is the output, and a funnel shift that takes it in.  The 32 x 32 bits of
        // a half wave are then transposed (TransposeBits) and leave as one word, two where the row allows it, per lane: a third
        // of the instructions of a compare, two v_writelane and their wait states per bit, and two stores instead of eight.
        float nsc[WN], nbi[WN];
#pragma unroll
        for (int f = 0; f < WN; ++f) {
            const SignColumn c = sign_column(sc[f], bi[f], kUnit);
            nsc[f] = c.neg_scale;
            nbi[f] = c.neg_bias;
        }
        const TransposeBits tr(lane);
        uint32_t* Yw = (uint32_t*)Y;
        const int wcol = n_base >> 5;
        const bool pairs = (yw32 & 1) == 0 && (reinterpret_cast<uintptr_t>(Y) & 7) == 0;
#pragma unroll
        for (int p = 0; p < WM / 2; ++p) {
            uint32_t w[WN];
#pragma unroll
            for (int fn = 0; fn < WN; ++fn) {
                w[fn] = 0u;
#pragma unroll
                for (int i = 31; i >= 0; --i) {   // bit i: frame row 8(v/4)+4g+v%4 of fragment 2p + i/16, v = i%16
                    const float a = acc[2 * p + (i >> 4)][fn][i & 15];
                    w[fn] = __builtin_amdgcn_alignbit(w[fn], __float_as_uint(affine(nsc[fn], PINGPONG ? a : dot_of(a, fn), nbi[fn])), 31);
                }
            }
            tr.run(w);
            const int v = r & 15, m = m_base + (2 * p + (r >> 4)) * 32 + 8 * (v >> 2) + 4 * g + (v & 3);
            if (m < M) {
                uint32_t* y = Yw + (size_t)m * yw32 + wcol;
                static_assert(WN == 2, "two words per lane");
                if (pairs && wcol + 1 < yw32) {
                    *reinterpret_cast<uint2*>(y) = make_uint2(w[0], w[1]);
                } else {
#pragma unroll
                    for (int fn = 0; fn < WN; ++fn)
                        if (wcol + fn < yw32) y[fn] = w[fn];
                }
            }
        }
    } else if constexpr (ACT == ACT_LSM_COOP) {
        // log-Softmax of whole rows without a second kernel.  The rows of this workgroup's tile continue in the other
        // tiles of the same frames (grid row tile_m): every workgroup reduces its 128 columns of each row to
        // (max, sum of exp(h - max)), publishes the pair, waits for the other tiles of its grid row, combines the pairs
        // to max + log sum exp and only then writes its share of the rows, normalised, straight from the accumulators.
        // Publishing: write-through stores (sc1), wait until they are acknowledged, then the flag.  Readers poll the
        // flags with loads that bypass the non-coherent caches (sc1) and then read the pairs with plain loads: no
        // cache of this launch can hold an older copy of a pair, because nothing reads a pair before its flag is up
        // and what earlier launches left in the caches is dropped at the kernel boundary.  The wait is bounded.
        static_assert(WN == 2, "the transposing epilogue is written for 64-column wave tiles");
        constexpr int LDW = kM32Ldw;
        constexpr int ROWS = 32 * WM;                          // rows of a wave; the workgroup has 2 ROWS
        uint32_t* st = reinterpret_cast<uint32_t*>(m32_mem) + wave * (32 * LDW);
        float2(*wave_part)[ROWS] = reinterpret_cast<float2(*)[ROWS]>(m32_mem + 4 * 32 * LDW * 4);   // [4][ROWS]
        float* lse_s = reinterpret_cast<float*>(m32_mem + 4 * 32 * LDW * 4 + 4 * ROWS * 8);          // [2 ROWS]
        const int c4 = (lane & 15) * 4;
        const int T = (int)gridDim.y;
        const float ninf = -__builtin_inff();
        // (a) pre-activations, in place; columns past N count as -inf (no share in any maximum or sum)
#pragma unroll
        for (int fm = 0; fm < WM; ++fm)
#pragma unroll
            for (int fn = 0; fn < WN; ++fn) {
                const bool col = n_base + fn * 32 + r < N;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const float h = affine(sc[fn], dot_of(acc[fm][fn][v], fn), bi[fn]);
                    acc[fm][fn][v] = col ? h : ninf;
                }
            }
        // (b) this wave's 64 columns of each of its rows: through its LDS slice, 32 rows at a time, so that lane
        //     (row = lane % 32, half = lane / 32) holds 32 consecutive columns of one row in registers: the maximum and
        //     the sum are then taken inside a lane, with a single exchange between the two halves of a row for each
        //     (8 consecutive lanes read 16 bytes each from rows 68 words apart: 32 different banks)
#pragma unroll
        for (int fm = 0; fm < WM; ++fm) {
#pragma unroll
            for (int fn = 0; fn < WN; ++fn)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    st[(8 * (v >> 2) + 4 * g + (v & 3)) * LDW + fn * 32 + r] = __float_as_uint(acc[fm][fn][v]);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
            float hv[32];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const uint4 q = *reinterpret_cast<const uint4*>(st + r * LDW + g * 32 + j * 4);
                hv[4 * j] = __uint_as_float(q.x); hv[4 * j + 1] = __uint_as_float(q.y);
                hv[4 * j + 2] = __uint_as_float(q.z); hv[4 * j + 3] = __uint_as_float(q.w);
            }
            float m4[4] = {hv[0], hv[1], hv[2], hv[3]};        // four chains: the maximum does not care about order
#pragma unroll
            for (int j = 4; j < 32; ++j) m4[j & 3] = __builtin_fmaxf(m4[j & 3], hv[j]);
            float mx = __builtin_fmaxf(__builtin_fmaxf(m4[0], m4[1]), __builtin_fmaxf(m4[2], m4[3]));
            mx = __builtin_fmaxf(mx, __shfl_xor(mx, 32, kWave));
            float s4[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            if (mx != ninf) {
#pragma unroll
                for (int j = 0; j < 32; ++j) s4[j & 3] += __expf(hv[j] - mx);
            }
            float s = (s4[0] + s4[1]) + (s4[2] + s4[3]);
            s += __shfl_xor(s, 32, kWave);
            if (g == 0) wave_part[wave][fm * 32 + r] = make_float2(mx, s);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        }
        __syncthreads();
        // (c) the two waves that share a row, then out to memory
        const int trow = (int)threadIdx.x;                     // row of the workgroup tile (threads below 2 ROWS)
        if (trow < 2 * ROWS) {
            const float2 pa = wave_part[2 * (trow / ROWS)][trow % ROWS], pb = wave_part[2 * (trow / ROWS) + 1][trow % ROWS];
            const float mx = __builtin_fmaxf(pa.x, pb.x);
            float s = 0.0f;
            if (pa.x != ninf) s += pa.y * __expf(pa.x - mx);
            if (pb.x != ninf) s += pb.y * __expf(pb.x - mx);
            const unsigned long long pair = (unsigned long long)__float_as_uint(mx) | ((unsigned long long)__float_as_uint(s) << 32);
            __hip_atomic_store(reinterpret_cast<unsigned long long*>(coop.partials + ((size_t)tile_m * T + tile_n) * (2 * ROWS) + trow), pair,
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // the pairs have arrived ...
        __syncthreads();
        if (threadIdx.x == 0)                                  // ... before the flag says so
            __hip_atomic_store(coop.flags + (size_t)tile_m * T + tile_n, coop.stamp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (wave == 0) {
            const unsigned long long* f = coop.flags + (size_t)tile_m * T;
            bool ok = false;
            for (int spin = 0; spin < coop.spin_limit; ++spin) {
                unsigned long long v = coop.stamp;
                if (lane < T) v = __hip_atomic_load(f + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (__builtin_amdgcn_ballot_w64(v == coop.stamp) == ~0ull) { ok = true; break; }
                __builtin_amdgcn_s_sleep(1);
            }
            if (!ok && lane == 0) atomicAdd(coop.timeouts, 1u);
        }
        __syncthreads();
        // (d) max + log sum exp of each row over all tiles of the grid row
        if (trow < 2 * ROWS) {
            // (consecutive lanes read consecutive rows of one tile's pairs: whole cache lines per request; 32 requests in
            // flight before the first pair is used)
            const unsigned long long* src = reinterpret_cast<const unsigned long long*>(coop.partials + (size_t)tile_m * T * (2 * ROWS) + trow);
            float mx = ninf, s = 0.0f;
            for (int t0 = 0; t0 < T; t0 += 32) {
                unsigned long long pr[32];
#pragma unroll
                for (int i = 0; i < 32; ++i)                    // (clamped: the same pair again, skipped below)
                    pr[i] = src[(size_t)(t0 + i < T ? t0 + i : T - 1) * (2 * ROWS)];
#pragma unroll
                for (int i = 0; i < 32; ++i) {
                    const float pm = __uint_as_float((uint32_t)pr[i]), ps = __uint_as_float((uint32_t)(pr[i] >> 32));
                    if (t0 + i < T && pm != ninf) {
                        if (pm > mx) { s = s * __expf(mx - pm) + ps; mx = pm; }   // (mx = -inf: s = 0, exp gives 0)
                        else s += ps * __expf(pm - mx);
                    }
                }
            }
            lse_s[trow] = mx + __logf(s);
        }
        __syncthreads();
        // (e) normalise and write: rows leave as contiguous 256-byte pieces, as in the plain fp32 epilogue
        const bool rows_vec = ((N & 3) == 0) && ((reinterpret_cast<uintptr_t>(Y) & 15) == 0);
#pragma unroll
        for (int fm = 0; fm < WM; ++fm) {
#pragma unroll
            for (int fn = 0; fn < WN; ++fn)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    st[(8 * (v >> 2) + 4 * g + (v & 3)) * LDW + fn * 32 + r] = __float_as_uint(acc[fm][fn][v]);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
#pragma unroll
            for (int it = 0; it < 8; ++it) {
                const int row = it * 4 + (lane >> 4);
                const int m = m_base + fm * 32 + row;
                const int n = n_base + c4;
                const uint4 q = *reinterpret_cast<const uint4*>(st + row * LDW + c4);
                const float l = lse_s[(wave >> 1) * ROWS + fm * 32 + row];
                float4 o;
                o.x = __uint_as_float(q.x) - l; o.y = __uint_as_float(q.y) - l; o.z = __uint_as_float(q.z) - l; o.w = __uint_as_float(q.w) - l;
                if (m < M) {
                    float* y = (float*)Y + (size_t)m * N + n;
                    if (rows_vec && n + 3 < N) {
                        *reinterpret_cast<float4*>(y) = o;
                    } else {
                        if (n + 0 < N) y[0] = o.x;
                        if (n + 1 < N) y[1] = o.y;
                        if (n + 2 < N) y[2] = o.z;
                        if (n + 3 < N) y[3] = o.w;
                    }
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        }
    } else {
        // 32-bit outputs: the accumulator layout gives a lane one column and 16 scattered rows, which would
        // store 128-byte pieces.  Each wave turns 32 rows x (32 WN) columns at a time through its own slice
        // of LDS so that 16 lanes write 256 contiguous bytes of a row (16 bytes per lane).
        static_assert(WN == 2, "the transposing epilogue is written for 64-column wave tiles");
        constexpr int LDW = kM32Ldw;
        uint32_t* st = reinterpret_cast<uint32_t*>(m32_mem) + wave * (32 * LDW);
        const bool rows_vec = ((N & 3) == 0) && ((reinterpret_cast<uintptr_t>(Y) & 15) == 0);
        const int c4 = (lane & 15) * 4;                        // this lane's 4 columns of the 64
#pragma unroll
        for (int fm = 0; fm < WM; ++fm) {
#pragma unroll
            for (int fn = 0; fn < WN; ++fn)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const float dot = dot_of(acc[fm][fn][v], fn);
                    uint32_t bits;
                    if constexpr (ACT == ACT_RAW_I32 || ACT == ACT_DOT_I16) {
                        bits = (uint32_t)(int)dot;
                    } else {
                        float h = affine(sc[fn], dot, bi[fn]);
                        if constexpr (ACT == ACT_HARDTANH) h = hardtanh(h);
                        if constexpr (ACT == ACT_SIGMOID) h = sigmoid(h);
                        bits = __float_as_uint(h);
                    }
                    st[(8 * (v >> 2) + 4 * g + (v & 3)) * LDW + fn * 32 + r] = bits;
                }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");   // this wave's LDS writes are done before it reads them back
            if constexpr (ACT == ACT_DOT_I16) {
                // int16 outputs: 8 lanes write the 128 bytes a row has in this wave tile (eight int16 = 16 bytes per lane),
                // so a store instruction covers 8 rows and the tile takes half as many of them as with 8 bytes per lane
                // (the stores, not their bytes, are what this epilogue costs).  The caller guarantees N % 4 == 0 and a
                // 16-byte aligned Y.
                const int c8 = (lane & 7) * 8;
#pragma unroll
                for (int it = 0; it < 4; ++it) {
                    const int row = it * 8 + (lane >> 3);
                    const int m = m_base + fm * 32 + row;
                    const int n = n_base + c8;
                    const uint4 q0 = *reinterpret_cast<const uint4*>(st + row * LDW + c8);
                    const uint4 q1 = *reinterpret_cast<const uint4*>(st + row * LDW + c8 + 4);
                    uint4 h;
                    h.x = (q0.x & 0xFFFFu) | (q0.y << 16);
                    h.y = (q0.z & 0xFFFFu) | (q0.w << 16);
                    h.z = (q1.x & 0xFFFFu) | (q1.y << 16);
                    h.w = (q1.z & 0xFFFFu) | (q1.w << 16);
                    if (m < M) {
                        uint16_t* y = reinterpret_cast<uint16_t*>(Y) + (size_t)m * 2 * N + n;
                        if (n + 7 < N) {
                            *reinterpret_cast<uint4*>(y) = h;
                        } else if (n < N) {   // N % 8 == 4: the last four outputs of the row
                            *reinterpret_cast<uint2*>(y) = make_uint2(h.x, h.y);
                        }
                    }
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");   // reads done before the next fragment row overwrites the slice
                continue;
            }
#pragma unroll
            for (int it = 0; it < 8; ++it) {
                const int row = it * 4 + (lane >> 4);
                const int m = m_base + fm * 32 + row;
                const int n = n_base + c4;
                const uint4 q = *reinterpret_cast<const uint4*>(st + row * LDW + c4);
                if (m < M) {
                    uint32_t* y = (uint32_t*)Y + (size_t)m * N + n;
                    if (rows_vec && n + 3 < N) {
                        *reinterpret_cast<uint4*>(y) = q;
                    } else {
                        if (n + 0 < N) y[0] = q.x;
                        if (n + 1 < N) y[1] = q.y;
                        if (n + 2 < N) y[2] = q.z;
                        if (n + 3 < N) y[3] = q.w;
                    }
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");   // reads done before the next fragment row overwrites the slice
        }
    }
}

}  // namespace bnn
