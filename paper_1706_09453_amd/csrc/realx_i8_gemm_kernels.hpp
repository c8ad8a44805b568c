// Real input x binary weights on the int8 matrix cores for batches of 128 frames or more (paper Alg. 1 forward; Alg. 2:
// Sign at a hidden layer, Softmax at l = L): the digit-plane product of realx_slab_kernels.hpp as a tiled matrix
// product with V_MFMA_I32_32X32X32_I8, workgroups of up to 128 frames x 256 outputs instead of 16 x 512, so that a weight
// byte fetched into LDS serves 128 frames.
//
// What is computed is the filter described in realx_fused_kernel.hpp and realx_slab_kernels.hpp: every frame is scaled by
// a power of two and rounded to integers xq, P = sum_k b_k xq_k is exact (b = the weight bit), a = 2 P - sum_k xq_k.
//   Sign layers (three 7-bit digits, |xq| <= 2^qb, qb = 29 - ceil(log2 K) at most 20): an output whose interval
//     [a - E, a + E] lies on one side of the threshold is decided; the others are listed in global memory, frame by
//     frame, and resolved by the fp32 sum in ascending k (realx_resolve_rows_kernel), so every bit is the bit of that sum.
//   Log-Softmax layers (four digits, |xq| <= 2^27): z = fma(scale, a 2^-s, bias), |a 2^-s - sum +-x| < K 2^-27 max|x|.
//
// Digits.  xq = d0 + 128 d1 + 16384 d2 (+ 2097152 d3) with d0, d1 (, d2) in 0..127 and the top digit signed.  Two
// digits share an accumulator: the odd digits are stored NEGATED and multiplied with -128 b (b << 7 as a byte), so
//     acc_lo = sum_k b (d0 + 128 d1),    acc_hi = sum_k b d2   or   sum_k b (d2 + 128 d3),    P = acc_lo + 16384 acc_hi,
// all exact in int32 (K <= 8192: below 2^27 each).  A fragment of b is read once from LDS and shifted in registers.
//
// Layout.  Planes [digit][frame][kpad] and weight bytes [output][kpad] (0 or 1), both in natural k order, kpad = K
// rounded up to 64, zeros past K.  The product kernel takes steps of 64 k = 64 bytes of a row: three LDS stages filled by loads that write LDS
// directly, two steps in flight, one barrier per step, one memory instruction between two MFMAs.  (Loads to registers and LDS
// stores, two stages: 4096 x 2048 x 2048 70 -> 62 us, 2048 outputs x 2048 x 4096 104 -> 91.)  2 x 2 waves of 64 frames x
// 128 outputs each, 2 x 4 accumulator fragments of 32 x 32, twice; smaller tiles where these leave part of the chip idle.
#pragma once

#include <type_traits>
#include <utility>

#include "realx_slab_kernels.hpp"

namespace bnn {

typedef int v16i32g __attribute__((ext_vector_type(16)));
typedef int v4i32g __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4g __attribute__((ext_vector_type(4)));

constexpr int kI8KStep = 64;                       // k per pipeline step
constexpr int kI8RowBytes = 64;
constexpr int kI8Threads = 256;
constexpr int kI8Stages = 3;
// A workgroup of 2 x 2 waves of 32 WM frames x 32 WN outputs each.
__host__ __device__ constexpr int i8_stage_a(int digits, int wm) { return digits * 64 * wm * kI8RowBytes; }
__host__ __device__ constexpr int i8_stage(int digits, int wm, int wn) { return i8_stage_a(digits, wm) + 64 * wn * kI8RowBytes; }
__host__ __device__ constexpr unsigned i8_gemm_lds(int digits, int wm, int wn) { return (unsigned)(kI8Stages * i8_stage(digits, wm, wn)); }
__host__ __device__ inline int i8_kpad(int K) { return (K + kI8KStep - 1) / kI8KStep * kI8KStep; }

// The outputs the filter could not decide, per frame and 128 outputs: a record of 16 bytes, one bit per output, so that it
// holds any number of them.  Records: [frame][ceil(N / 128)], written whole by the one workgroup that owns frame and outputs
// (no atomics in global memory, nothing to clear beforehand).  (As a list of at most 15 positions, the rest summed by the lane
// that found it, a single full record cost a chain of K dependent additions from global memory: 5464 x 7808 x 1024 1760 us, now 487.)
constexpr int kUndecidedOutputs = 128;
constexpr int kUndecidedRecord = kUndecidedOutputs / 8;

// B[n][k] = bit k of weight row n as a byte (0 past K).  One thread per 16 k; block `block` of byte_blocks() of 256 threads.
struct ByteRows {
    const uint32_t* Wp;
    int8_t* B;
    int64_t N;
    int w32;
};
__host__ __device__ inline int byte_blocks(int64_t N, int kpad) {
    const int64_t blocks = (N * (kpad / 16) + 255) / 256;
    return (int)(blocks < 16384 ? blocks : 16384);
}
__device__ __forceinline__ void expand_bytes(const ByteRows& b, int K, int kpad, int block) {
    const int blocks = byte_blocks(b.N, kpad);
    const int per_row = kpad >> 4;
    const int64_t total = b.N * per_row;
    for (int64_t i = (int64_t)block * 256 + threadIdx.x; i < total; i += (int64_t)blocks * 256) {
        const int64_t n = total < ((int64_t)1 << 31) ? (int64_t)((uint32_t)i / (uint32_t)per_row) : i / per_row;
        const int k0 = (int)(i - n * per_row) * 16;
        uint32_t bits = 0;
        if (k0 < K) bits = (b.Wp[(size_t)n * b.w32 + (k0 >> 5)] >> (k0 & 31)) & 0xFFFFu;
        if (K - k0 < 16 && K > k0) bits &= (1u << (K - k0)) - 1u;
        uint32_t w[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t nib = (bits >> (4 * j)) & 0xFu;
            w[j] = (nib & 1u) | ((nib & 2u) << 7) | ((nib & 4u) << 14) | ((nib & 8u) << 21);
        }
        *reinterpret_cast<uint4*>(b.B + (size_t)n * kpad + k0) = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

// Four bytes holding 0 .. 127 each, negated byte by byte: 0x80 - d needs no borrow, and the flipped top bit takes the 0x80 off.
__device__ __forceinline__ uint32_t negate_digits(uint32_t d) { return (0x80808080u - d) ^ 0x80808080u; }

// One wave per frame: scale, digits (odd digits negated), RowMeta (D = 3) or RowMeta4 (D = 4).  planes: [D][M][kpad].
// Four consecutive elements per lane and group of 256.  VEC: K % 4 == 0 and X 16-byte aligned.
// NG > 0 (with VEC): the frame has at most NG groups and is requested whole, NG loads of a lane in flight, and kept in
// registers; NG == 0 (without): it is read twice (largest element, then digits), one load after the other.
// Bound by memory: a number in, D bytes out.  Against one load after the other, twice:
// 4096 frames of 2048 15.5 -> 12.2 us, 2048 of 4096 26.2 -> 13.0 (5.2 TB/s).
// The weights' bytes are made in the same launch, by the workgroups behind those of the frames: neither waits for the other, and a launch
// of their own cost 2 to 3 us (600 frames through the mixed network, two such calls 141.7 -> 139.3 us; a training step, eleven, 1971 -> 1941).
// Grid: ceil(M / 4) workgroups of 256 threads, then byte_blocks().
template <int D, bool VEC, int NG>
__global__ __launch_bounds__(256) void realx_quantize_nat_kernel(const float* __restrict__ X, int M, int K, int kpad, int qbits,
                                                                 int8_t* __restrict__ planes, void* __restrict__ meta_out, ByteRows weights) {
    const int frame_blocks = (int)(((int64_t)M + 3) >> 2);
    if ((int)blockIdx.x >= frame_blocks) {
        expand_bytes(weights, K, kpad, (int)blockIdx.x - frame_blocks);
        return;
    }
    static_assert(D == 3 || D == 4, "three digits for Sign layers, four in front of the log-Softmax");
    static_assert((NG > 0) == VEC, "whole frames are requested in pieces of 16 bytes");
    const int m = (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6);
    if (m >= M) return;   // wave-uniform
    const int lane = lane_id();
    const float* x = X + (size_t)m * K;
    auto load4 = [&](int k) -> f32x4g {
        f32x4g v;
#pragma unroll
        for (int t = 0; t < 4; ++t) v[t] = (k + t < K) ? x[k + t] : 0.0f;
        return v;
    };
    unsigned int mx = 0;   // largest |x| of the row as a bit pattern (NaN/Inf have the largest patterns)
    auto largest = [&](const f32x4g& v) {
#pragma unroll
        for (int t = 0; t < 4; ++t) mx = max(mx, __float_as_uint(v[t]) & 0x7fffffffu);
    };
    f32x4g xs[NG > 0 ? NG : 1];
    if constexpr (NG > 0) {
#pragma unroll
        for (int i = 0; i < NG; ++i) {   // past the frame's end its first elements again, replaced below
            const int k = 256 * i + 4 * lane;
            xs[i] = *reinterpret_cast<const f32x4g*>(x + (k < K ? k : 0));
        }
#pragma unroll
        for (int i = 0; i < NG; ++i) {
            const bool in = 256 * i + 4 * lane < K;
#pragma unroll
            for (int t = 0; t < 4; ++t) xs[i][t] = in ? xs[i][t] : 0.0f;
            largest(xs[i]);
        }
    } else {
        for (int k0 = 0; k0 < K; k0 += 256) largest(load4(k0 + 4 * lane));
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mx = max(mx, (unsigned int)__shfl_xor((int)mx, off, kWave));
    const int e = (int)(mx >> 23) - 127;                 // floor(log2 max|x|) for normal numbers
    const int flags = (mx >= 0x7f800000u || e >= (D == 3 ? 100 : 90)) ? 1 : 0;
    int s = qbits - 1 - e;                                // max|x| < 2^(e+1)  =>  |x| 2^s < 2^qbits
    s = s > 100 ? 100 : s;
    const float qs = __uint_as_float((unsigned int)(s + 127) << 23);
    const size_t plane = (size_t)M * kpad;
    int8_t* row = planes + (size_t)m * kpad;
    long long R = 0, A = 0;
    auto digits = [&](int k, const f32x4g& v) {   // elements past K hold 0
        uint32_t w[D] = {};
        int sum = 0, abs = 0;   // of four |xq| <= 2^27
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int xq = flags ? 0 : (int)__builtin_rintf(v[t] * qs);
            sum += xq;
            if constexpr (D == 3) abs += xq < 0 ? -xq : xq;
            w[0] |= (uint32_t)(xq & 127) << (8 * t);
            w[1] |= (uint32_t)((xq >> 7) & 127) << (8 * t);
            if constexpr (D == 3) {
                w[2] |= ((uint32_t)(xq >> 14) & 0xFFu) << (8 * t);
            } else {
                w[2] |= (uint32_t)((xq >> 14) & 127) << (8 * t);
                w[3] |= ((uint32_t)(-(xq >> 21)) & 0xFFu) << (8 * t);
            }
        }
        w[1] = negate_digits(w[1]);
        R += sum;
        if constexpr (D == 3) A += abs;
#pragma unroll
        for (int d = 0; d < D; ++d) *reinterpret_cast<uint32_t*>(row + d * plane + k) = w[d];
    };
    // kpad is a multiple of 64: a lane's four elements are inside or outside together
    if constexpr (NG > 0) {
#pragma unroll
        for (int i = 0; i < NG; ++i)
            if (256 * i + 4 * lane < kpad) digits(256 * i + 4 * lane, xs[i]);
    } else {
        for (int k = 4 * lane; k < kpad; k += 256) digits(k, load4(k));
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        R += __shfl_xor(R, off, kWave);
        if constexpr (D == 3) A += __shfl_xor(A, off, kWave);
    }
    if (lane == 0) {
        const float inv = __uint_as_float((unsigned int)(127 - s) << 23);
        if constexpr (D == 3) {
            const float u = 5.9604644775390625e-08f;                            // 2^-24; all terms in units of 2^-s
            const float Kf = (float)K;
            const float sum_abs = (float)A * 1.0000002f + 0.5f * Kf;            // >= sum |x| 2^s ((float)A rounds: one ulp added)
            const float e_seq = (Kf - 1.0f) * u / (1.0f - Kf * u) * sum_abs;    // recursive fp32 summation
            const float e_quant = 0.5f * Kf;                                     // |x 2^s - xq| <= 1/2 each
            const float e_conv = u * (float)A * 1.0000002f;                      // (float)a
            RowMeta rm;
            rm.R = (int)R; rm.inv_scale = inv; rm.flags = flags;
            rm.E = flags ? __builtin_inff() : (e_seq + e_quant + e_conv) * 1.01f * inv;   // infinite bound: every output uncertain
            static_cast<RowMeta*>(meta_out)[m] = rm;
        } else {
            RowMeta4 rm;
            rm.R = R; rm.inv_scale = inv; rm.flags = flags;
            static_cast<RowMeta4*>(meta_out)[m] = rm;
        }
    }
}

// The product kernel.  D = 3: Sign bits into Yv (uint32 words [M][yw32]; bits of listed outputs are left 0) and the
// records of undecided outputs into `undecided` ([M][ceil(N / 128)] records); D = 4: z = fma(scale, a 2^-s, bias) into Yv
// (fp32 [M][N]), `undecided` unused.
// planes [D][M][kpad], Bb [N][kpad], both 16-byte aligned, kpad % 64 == 0; meta: RowMeta (D = 3) or RowMeta4 (D = 4) [M].
// X, Wp: the layer's own operands, for the fp32 sum in ascending k of frames that could not be quantised (D = 4).  Grid: x = ceil(M / (64 WM)), y = ceil(N / (64 WN)); block = 256 threads;
// dynamic LDS i8_gemm_lds(D, WM, WN).
template <int D, int WM, int WN>
__global__ __launch_bounds__(kI8Threads) __attribute__((amdgpu_waves_per_eu(1, WM * WN > 2 ? 1 : 2))) void realx_i8_gemm_kernel(
    const int8_t* __restrict__ planes, const int8_t* __restrict__ Bb, const void* __restrict__ meta_in, const float* __restrict__ X,
    const uint32_t* __restrict__ Wp, const float* __restrict__ scale, const float* __restrict__ bias, int M, int K, int kpad, int N,
    int w32, void* __restrict__ Yv, int yw32, unsigned char* __restrict__ undecided) {
    static_assert(D == 3 || D == 4, "three digits for Sign layers, four in front of the log-Softmax");
    extern __shared__ __attribute__((aligned(16))) unsigned char i8_lds[];
    static_assert((64 * WN) % kUndecidedOutputs == 0, "Sign layers: a record of undecided outputs belongs to one workgroup");
    constexpr int kTileM = 64 * WM, kTileN = 64 * WN;
    constexpr int NL = D * WM + WN;                           // loads per wave and step, of 16 rows each
    constexpr int NR = D * WM + WN;                           // fragment reads per wave and block
    constexpr int NM = D * WM * WN;                           // MFMAs per wave and block
    constexpr int kStageA = i8_stage_a(D, WM), kStage = i8_stage(D, WM, WN);
    const int tid = (int)threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = lane_id();
    const int r = lane & 31, g = lane >> 5;
    int tm = (int)blockIdx.x, tn = (int)blockIdx.y;
    // The XCDs' order from eight tile rows on (whole calls, launch's order -> XCDs': 4026 x 8124 x 1024 312 -> 218 us, 2048 x 4096 x 2048
    // 93 -> 80, 512 x 4096 x 4096 57.7 -> 52.7, 900 x 1024 x 1000 24.2 -> 21.5; with fewer 256 x 4096 x 4096 47.9 -> 49.5, 200 x 2048 x 2048
    // 28.0 -> 29.3).
    if ((int)gridDim.x >= 8) xcd_tile(tm, tn);
    const int m_tile = tm * kTileM, n_tile = tn * kTileN;
    const int m_base = m_tile + (wave >> 1) * (WM * 32);
    const int n_base = n_tile + (wave & 1) * (WN * 32);

    // ---- the wave's share of a step's loads, 16 rows each (four lanes a row): load i < D WM is digit i / WM, frames
    //      16 (WM wave + i % WM) .. of the tile; load D WM + j its weight rows 16 (WN wave + j) ...  One buffer per digit
    //      plane and one for the weights, over the rows of the tile (rows past the end: the last one again).
    const int lrow = lane >> 2, lsrc = ((lane & 3) ^ ((lrow >> 2) & 3)) * 16;
    const int rows_a = min(M - m_tile, kTileM), rows_b = min(N - n_tile, kTileN);
    i32x4m ars[D];
#pragma unroll
    for (int d = 0; d < D; ++d) ars[d] = raw_buffer(planes + ((size_t)d * M + m_tile) * kpad, (unsigned int)(rows_a * kpad));
    const i32x4m brs = raw_buffer(Bb + (size_t)n_tile * kpad, (unsigned int)(rows_b * kpad));
    int aofs[WM], bofs[WN];
#pragma unroll
    for (int i = 0; i < WM; ++i) aofs[i] = min(16 * (WM * wave + i) + lrow, rows_a - 1) * kpad + lsrc;
#pragma unroll
    for (int i = 0; i < WN; ++i) bofs[i] = min(16 * (WN * wave + i) + lrow, rows_b - 1) * kpad + lsrc;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)i8_lds;
    auto request_one = [&](int step, uint32_t stage, int i) {
        if (i < D * WM)
            load_lds16(ars[i < D * WM ? i / WM : 0], aofs[i % WM], step * kI8KStep,
                       stage + (uint32_t)(((i / WM) * kTileM + 16 * (WM * wave + i % WM)) * kI8RowBytes));
        else
            load_lds16(brs, bofs[i < D * WM ? 0 : i - D * WM], step * kI8KStep,
                       stage + (uint32_t)(kStageA + 16 * (WN * wave + i - D * WM) * kI8RowBytes));
    };

    // ---- the wave's operand fragments of block h (0 or 1) of a stage: digit fragments, then weight fragments
    struct Frags { v4i32g a[D][WM]; v4i32g b[WN]; };
    const int swz = (r >> 2) & 3;
    const int a_off = ((wave >> 1) * (WM * 32) + r) * kI8RowBytes;
    const int b_off = kStageA + ((wave & 1) * (WN * 32) + r) * kI8RowBytes;
    auto lread_one = [&](Frags& F, const unsigned char* stage, int h, int i) {
        const int so = ((2 * h + g) ^ swz) << 4;
        if (i < D * WM)
            F.a[i < D * WM ? i / WM : 0][i % WM] =
                *reinterpret_cast<const v4i32g*>(stage + (i / WM) * (kTileM * kI8RowBytes) + a_off + (i % WM) * (32 * kI8RowBytes) + so);
        else
            F.b[i < D * WM ? 0 : i - D * WM] = *reinterpret_cast<const v4i32g*>(stage + b_off + (i - D * WM) * (32 * kI8RowBytes) + so);
    };

    v16i32g acc[2][WM][WN];   // [0]: digits 0 and 1, [1]: digits 2 (and 3)
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int i = 0; i < WM; ++i)
#pragma unroll
            for (int j = 0; j < WN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[p][i][j][v] = 0;

    // One block of 32 k, written out MFMA by MFMA and pinned: behind each of the first ones a fragment read of the next
    // block, behind each of the last ones (REQ) a load of step `step` to `stage`.
    auto block = [&](const Frags& now, Frags& next, const unsigned char* rd, int rd_h, auto req, int step, uint32_t stage) {
        constexpr bool REQ = decltype(req)::value;
        v4i32g bneg[WN];   // -128 b: the byte 1 becomes 0x80
#pragma unroll
        for (int i = 0; i < NM; ++i) {
            const int d = i / (WM * WN), fm = (i / WN) % WM, fn = i % WN;
            acc[d >> 1][fm][fn] =
                __builtin_amdgcn_mfma_i32_32x32x32_i8(now.a[d][fm], (d & 1) ? bneg[fn] : now.b[fn], acc[d >> 1][fm][fn], 0, 0, 0);
            if (i < NR) lread_one(next, rd, rd_h, i);
            if (i < WN) bneg[i < WN ? i : 0] = now.b[i < WN ? i : 0] << 7;
            if (REQ && i >= NM - NL) request_one(step, stage, i - (NM - NL));
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    static_assert(NR <= NM && NL <= NM && WN <= WM * WN, "room for the reads, the loads and the shifted weights");

    // Three stages in rotation and one barrier per step, between its blocks: behind it step j + 1 is complete in LDS, and every
    // wave has read step j, so its place takes step j + 3.
    const int nS = kpad / kI8KStep;
    auto turn = [&](int j) {
        if (j + 2 < nS) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(NL) : "memory");   // step j + 2 may be on its way
        else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    Frags F0, F1;
#pragma unroll
    for (int st = 0; st < kI8Stages; ++st)
        if (st < nS)
#pragma unroll
            for (int i = 0; i < NL; ++i) request_one(st, lds0 + (uint32_t)(st * kStage), i);
    if (nS > 2) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(2 * NL) : "memory");
    else if (nS > 1) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(NL) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
    for (int i = 0; i < NR; ++i) lread_one(F0, i8_lds, 0, i);
    int slot = 0, j = 0;
    auto step = [&](auto req) {
        const int nslot = slot == kI8Stages - 1 ? 0 : slot + 1;
        block(F0, F1, i8_lds + slot * kStage, 1, std::false_type{}, 0, 0u);
        turn(j);
        // (behind the last step: its first block read again, unused)
        block(F1, F0, i8_lds + (j + 1 < nS ? nslot : slot) * kStage, 0, req, j + 3, lds0 + (uint32_t)(slot * kStage));
        slot = nslot;
    };
    for (; j + 3 < nS; ++j) step(std::true_type{});
    for (; j < nS; ++j) step(std::false_type{});
    __syncthreads();   // the buffers are free: the epilogue reuses them

    // ---- epilogue.  Accumulator fragment (fm, fn), register v of lane (r, g) belongs to frame
    //      m_base + 32 fm + 8 (v/4) + 4 g + v%4 and output n_base + 32 fn + r.
    if constexpr (D == 3) {
        const RowMeta* meta = static_cast<const RowMeta*>(meta_in);
        uint32_t* Y = static_cast<uint32_t*>(Yv);
        // A lane decides its 16 frames of a fragment on its own and keeps the answers as bit masks (bit v: frame v of
        // the fragment): no ballots, no scalar logic, no branch per sum.  The masks of all lanes go to LDS,
        // colmask[frame block of 32][g][output of the tile], and are turned into output words afterwards.
        // LDS: column masks 2 WM x 2 x 64 WN x 2 bytes | the frames' quantisation records | per frame and 128 outputs the record
        // of undecided ones (about one output in 250 is expected at K = 2048).
        uint16_t* colmask = reinterpret_cast<uint16_t*>(i8_lds);
        constexpr int kMaskBytes = 2 * WM * 2 * kTileN * 2, kRecs = kTileN / kUndecidedOutputs, kAllRecs = kTileM * kRecs;
        RowMeta* meta_s = reinterpret_cast<RowMeta*>(i8_lds + kMaskBytes);
        u32x4* und = reinterpret_cast<u32x4*>(i8_lds + kMaskBytes + kTileM * sizeof(RowMeta));   // [frame][kRecs]
        static_assert((kMaskBytes + kTileM * sizeof(RowMeta)) % 16 == 0 && sizeof(u32x4) == kUndecidedRecord &&
                          kMaskBytes + kTileM * sizeof(RowMeta) + kAllRecs * kUndecidedRecord <= i8_gemm_lds(3, WM, WN) &&
                          kAllRecs <= kI8Threads,
                      "epilogue LDS");
        if (tid < kTileM) {
            const int m = m_tile + tid;
            meta_s[tid] = meta[m < M ? m : M - 1];
        }
        if (tid < kAllRecs) und[tid] = u32x4{0u, 0u, 0u, 0u};
        __syncthreads();
        float sc[WN], bi[WN], asc[WN];
        bool nvalid[WN];
#pragma unroll
        for (int fn = 0; fn < WN; ++fn) {
            const int n = n_base + fn * 32 + r;
            nvalid[fn] = n < N;
            sc[fn] = nvalid[fn] ? (scale ? scale[n] : 1.0f) : 0.0f;
            bi[fn] = nvalid[fn] ? (bias ? bias[n] : 0.0f) : -1.0f;
            // |scale| (1 + 2^-16.6) covers the roundings of the margin; the floor covers a product that underflows
            asc[fn] = __builtin_fmaxf(__builtin_fabsf(sc[fn]) * 1.00001f, 1e-30f);
        }
#pragma unroll
        for (int fm = 0; fm < WM; ++fm) {
            const int fb = (wave >> 1) * WM + fm;   // block of 32 frames of the tile
            uint32_t bits[WN], ubits[WN];
#pragma unroll
            for (int fn = 0; fn < WN; ++fn) bits[fn] = ubits[fn] = 0u;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int ml = fb * 32 + 8 * (v >> 2) + 4 * g + (v & 3);   // frame in the tile
                const RowMeta rm = meta_s[ml];
                const bool mvalid = m_tile + ml < M;
#pragma unroll
                for (int fn = 0; fn < WN; ++fn) {
                    // With t = fma(scale, a, bias): if |t| > |scale| E (1 + 2^-16.6) + 1e-30, then scale x + bias has the
                    // sign of t, and at least 1e-30 in magnitude, for every real x within E of a, so its rounding has that
                    // sign too and the bit of the fp32 sum is (t > 0).  Anything else (NaN included) is uncertain.
                    const int P = acc[0][fm][fn][v] + (acc[1][fm][fn][v] << (2 * kDigitBits));
                    const float a = (float)(int)(((unsigned int)P << 1) - (unsigned int)rm.R) * rm.inv_scale;
                    const float t = affine(sc[fn], a, bi[fn]);
                    const float margin = __builtin_fmaf(asc[fn], rm.E, 1e-30f);
                    const bool certain = __builtin_fabsf(t) > margin;
                    bits[fn] |= (certain && t > 0.0f) ? (1u << v) : 0u;
                    ubits[fn] |= (!certain && mvalid) ? (1u << v) : 0u;
                }
            }
#pragma unroll
            for (int fn = 0; fn < WN; ++fn) {
                const int nl = (wave & 1) * (WN * 32) + fn * 32 + r;   // output in the tile
                uint32_t ub = nvalid[fn] ? ubits[fn] : 0u;
                uint32_t bt = nvalid[fn] ? bits[fn] : 0u;              // outputs past the layer's end: bit 0
                while (ub) {   // rare: about one lane in twenty has one
                    const int v = __builtin_ctz(ub);
                    ub &= ub - 1u;
                    const int ml = fb * 32 + 8 * (v >> 2) + 4 * g + (v & 3);
                    atomicOr(reinterpret_cast<uint32_t*>(und) + ml * (kTileN / 32) + (nl >> 5), 1u << (nl & 31));
                }
                colmask[(fb * 2 + g) * kTileN + nl] = (uint16_t)bt;
            }
        }
        __syncthreads();
        // Output words: a thread builds four words of a frame f (the 128 outputs of a record); bit j of word c is bit v(f) of the
        // mask of output 32 c + j, where f = 32 fb + 8 (v / 4) + 4 g + v % 4.
        if (tid < kAllRecs) {
            const int f = tid / kRecs, wq = (tid % kRecs) * 4;
            const int fb = f >> 5, fg = (f >> 2) & 1, fv = ((f >> 3) & 3) * 4 + (f & 3);
            const uint32_t* cm = reinterpret_cast<const uint32_t*>(colmask + (fb * 2 + fg) * kTileN);   // two masks per dword
            const int m = m_tile + f;
            const int w_first = (n_tile >> 5) + wq;
            uint32_t words[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                uint32_t w = 0u;
#pragma unroll
                for (int j2 = 0; j2 < 16; ++j2) {
                    const uint32_t two = cm[(wq + c) * 16 + j2] >> fv;   // outputs 32 (wq + c) + 2 j2 and + 1
                    w |= (two & 1u) << (2 * j2);
                    w |= ((two >> 16) & 1u) << (2 * j2 + 1);
                }
                words[c] = w;
            }
            if (m < M) {
                uint32_t* y = Y + (size_t)m * yw32 + w_first;
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (w_first + c < yw32) y[c] = words[c];
            }
        }
        // the frames' records, one per thread (the barrier above also ordered the entries written to them)
        if (tid < kAllRecs) {
            const int m = m_tile + tid / kRecs, q = n_tile / kUndecidedOutputs + tid % kRecs;
            const int recs = (N + kUndecidedOutputs - 1) / kUndecidedOutputs;
            if (m < M && q < recs) *reinterpret_cast<u32x4*>(undecided + ((size_t)m * recs + q) * kUndecidedRecord) = und[tid];
        }
    } else {
        const RowMeta4* meta = static_cast<const RowMeta4*>(meta_in);
        float* Z = static_cast<float*>(Yv);
        if (m_base >= M || n_base >= N) return;   // wave-uniform, after the last barrier
        // per wave 32 rows x 32 WN columns of outputs on their way to memory (a row is 128 WN contiguous bytes)
        constexpr int LDW = 32 * WN + 4;
        static_assert(4 * 32 * LDW * 4 <= (int)i8_gemm_lds(4, WM, WN), "epilogue LDS");
        float* stg = reinterpret_cast<float*>(i8_lds) + wave * (32 * LDW);
        float sc[WN], bi[WN];
#pragma unroll
        for (int fn = 0; fn < WN; ++fn) {
            const int n = n_base + fn * 32 + r;
            sc[fn] = (n < N && scale) ? scale[n] : 1.0f;
            bi[fn] = (n < N && bias) ? bias[n] : 0.0f;
        }
        const bool rows_vec = ((N & 3) == 0) && ((reinterpret_cast<uintptr_t>(Z) & 15) == 0);
        constexpr int kLanes = 8 * WN, kRows = kWave / kLanes;   // lanes that store a row, rows per pass
        const int c4 = (lane % kLanes) * 4;
#pragma unroll
        for (int fm = 0; fm < WM; ++fm) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int rowl = 8 * (v >> 2) + 4 * g + (v & 3);
                const int m = m_base + fm * 32 + rowl;
                const RowMeta4 rm = meta[m < M ? m : M - 1];
#pragma unroll
                for (int fn = 0; fn < WN; ++fn) {
                    // P = sum_k b_k xq_k from its two accumulators, a = 2 P - R as a 64-bit integer (below 2^40), rounded
                    // once: its upper part (below 2^24) and its lower 16 bits are exact floats, and one fma adds them
                    const long long P = (long long)acc[0][fm][fn][v] + ((long long)acc[1][fm][fn][v] << (2 * kDigitBits));
                    const long long a64 = 2 * P - rm.R;
                    const int hi = (int)(a64 >> 16);
                    const int lo = (int)(a64 & 0xFFFF);
                    float a = __builtin_fmaf((float)hi, 65536.0f, (float)lo) * rm.inv_scale;
                    const int n = n_base + fn * 32 + r;
                    if (rm.flags && m < M && n < N)   // rare: NaN, Inf, huge values
                        a = canonical_acc_global(X + (size_t)m * K, Wp + (size_t)n * w32, K);
                    stg[rowl * LDW + fn * 32 + r] = affine(sc[fn], a, bi[fn]);
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");   // this wave's LDS writes are done before it reads them back
#pragma unroll 4
            for (int it = 0; it < 32 / kRows; ++it) {
                const int rowl = it * kRows + lane / kLanes;
                const int m = m_base + fm * 32 + rowl;
                const int n = n_base + c4;
                const float4 qv = *reinterpret_cast<const float4*>(stg + rowl * LDW + c4);
                if (m < M) {
                    float* y = Z + (size_t)m * N + n;
                    if (rows_vec && n + 3 < N) {
                        *reinterpret_cast<float4*>(y) = qv;
                    } else {
                        if (n + 0 < N) y[0] = qv.x;
                        if (n + 1 < N) y[1] = qv.y;
                        if (n + 2 < N) y[2] = qv.z;
                        if (n + 3 < N) y[3] = qv.w;
                    }
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");   // reads done before the next fragment row overwrites the slice
        }
    }
}

// The undecided outputs, exactly: the fp32 sum in ascending k, acc + (+-x) at every step, written as fma(+-1, x, acc)
// (the product with +-1 is exact, so it rounds as the addition does), then bit = Sign(fma(scale, sum, bias)) ORed into Y
// (the product kernel left these bits 0).
// A sum is a chain of K dependent operations, and an output's terms are its frame's values with the signs of its weight
// row, so the frames are what is worth sharing: a workgroup of 256 threads takes 16 frames, collects their undecided
// outputs from the records (about 130 at K = 2048, N = 2048) and gives each to a lane.  The frames go through LDS in
// slabs of 256 k, twice buffered (the next slab is on its way from memory while this one is added up, one barrier per
// slab); a lane reads its frame's values from there (lanes of one frame read the same address, the 16 frames lie in
// different banks), forms the signs from its own weight words (eight per slab, read one slab ahead) and adds.
// More than 256 outputs: further passes over the frames; more than kResolveCap: further rounds, a thread keeping what its
// records still hold.  The last slab of a frame is padded with +0 and added up to the end of the block of 32 in which the
// frame ends.
// VEC: K % 4 == 0 and X 16-byte aligned.  Grid: ceil(M / 16) workgroups of 256 threads.
constexpr int kResolveFrames = 16;
constexpr int kResolveSlab = 256;
constexpr int kResolveLd = kResolveSlab + 4;   // floats per frame in a buffer: frame r starts at bank 4 r
constexpr int kResolveThreads = 256;
constexpr int kResolveCap = 1024;

// Term T of a slab and what stands around it (see the kernel); T = -16 .. -1 only start the stream.
// The factor +-1 of a term is a half-precision number: bits j and j + 16 of a weight word, moved to the sign bits of
// the two halves of a register over the bit pattern of (1.0, 1.0), serve terms j and j + 16 of the word's 32, and the
// mixed-precision fused multiply-add takes either half as its first factor (widened exactly; the operation itself is
// the fp32 one).  Two instructions per pair and one per term instead of three per term.
// Rings: a shifted word lives for four terms, a pair for twenty, an LDS read for twenty.
typedef _Float16 f16x2g __attribute__((ext_vector_type(2)));
// Returns false behind the last term of a block of 32 when the frame ends there or before (kn: terms of this slab).
template <int T>
__device__ __forceinline__ bool resolve_term(int kn, const float* xr, const uint32_t (&wc)[kResolveSlab / 32], uint32_t (&sh)[8], uint32_t (&pr)[16],
                                             f32x4g (&xv)[8], float& acc, uint32_t ones) {
    if constexpr (T + 16 < kResolveSlab && ((T + 16) & 3) == 0) xv[((T + 16) >> 2) & 7] = *reinterpret_cast<const f32x4g*>(xr + T + 16);
    if constexpr (T >= 0) {
        const f16x2g pm = __builtin_bit_cast(f16x2g, pr[T & 15]);
        acc = __builtin_fmaf((float)pm[(T >> 4) & 1], xv[(T >> 2) & 7][T & 3], acc);
    }
    if constexpr (T + 4 >= 0 && T + 4 < kResolveSlab && ((T + 4) & 31) < 16)   // one bit-field insert
        pr[(T + 4) & 15] = (sh[(T + 4) & 7] & 0x80008000u) | (ones & ~0x80008000u);
    if constexpr (T + 8 >= 0 && T + 8 < kResolveSlab && ((T + 8) & 31) < 16)
        sh[(T + 8) & 7] = ~wc[(T + 8) >> 5] << (15 - ((T + 8) & 31));   // weight bit 0: -x
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (T >= 0 && (T & 31) == 31 && T + 1 < kResolveSlab) return T + 1 < kn;   // wave-uniform
    return true;
}
template <int... I>
__device__ __forceinline__ void resolve_slab(int kn, const float* xr, const uint32_t (&wc)[kResolveSlab / 32], float& acc,
                                             std::integer_sequence<int, I...>) {
    uint32_t sh[8];
    uint32_t pr[16];
    f32x4g xv[8];
    uint32_t ones = 0x3C003C00u;   // (1.0, 1.0) in half precision, kept in a register as the insert's third operand
    asm volatile("" : "+v"(ones));
    (void)(resolve_term<I - 16>(kn, xr, wc, sh, pr, xv, acc, ones) && ...);
}

template <bool VEC>
__global__ __launch_bounds__(kResolveThreads) void realx_resolve_rows_kernel(const float* __restrict__ X, const uint32_t* __restrict__ Wp,
                                                                           const float* __restrict__ scale, const float* __restrict__ bias,
                                                                           int M, int K, int w32, const unsigned char* __restrict__ undecided,
                                                                           int recs, uint32_t* __restrict__ Y, int yw32, Clear clear) {
    clear_pieces<kResolveThreads>(clear);
    __shared__ __attribute__((aligned(16))) float xs[2][kResolveFrames][kResolveLd];
    __shared__ u32x4 ws[2][kResolveThreads][2];   // a lane's eight weight words of a slab
    __shared__ unsigned int ent[kResolveCap];   // (frame of the workgroup) << 28 | output
    __shared__ unsigned int total_s;
    const int tid = (int)threadIdx.x;
    const int m0 = (int)blockIdx.x * kResolveFrames;
    const int nsl = (K + kResolveSlab - 1) / kResolveSlab;
    // a slab is 16 frames x 64 pieces of four k: four pieces per thread
    constexpr int kPPR = kResolveSlab / 4, kPer = kResolveFrames * kPPR / kResolveThreads;
    struct Pieces { f32x4g x[kPer]; };   // native vectors: an array of them stays in registers
    auto request = [&](Pieces& P, int sl) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int p = tid + kResolveThreads * i;
            const int m = min(m0 + p / kPPR, M - 1);   // past the last frame: the last one again (unused)
            const int k = sl * kResolveSlab + 4 * (p % kPPR);
            const float* xr = X + (size_t)m * K;
            if (VEC) {   // past K: values of the frame's end (in bounds), replaced by deposit()
                P.x[i] = *reinterpret_cast<const f32x4g*>(xr + min(k, K - 4));
            } else {
                P.x[i] = f32x4g{xr[min(k, K - 1)], xr[min(k + 1, K - 1)], xr[min(k + 2, K - 1)], xr[min(k + 3, K - 1)]};
            }
        }
    };
    // past K: +0, which leaves a sum as it is with either sign in front (a sum that starts at +0 never becomes -0).
    // The first use of what was requested is here, after the slab in between has been added up.
    auto deposit = [&](const Pieces& P, int sl) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int p = tid + kResolveThreads * i;
            const int k = sl * kResolveSlab + 4 * (p % kPPR);
            f32x4g v = P.x[i];
            v.x = k < K ? v.x : 0.0f;
            v.y = k + 1 < K ? v.y : 0.0f;
            v.z = k + 2 < K ? v.z : 0.0f;
            v.w = k + 3 < K ? v.w : 0.0f;
            *reinterpret_cast<f32x4g*>(&xs[sl & 1][p / kPPR][4 * (p % kPPR)]) = v;
        }
    };
    Pieces P;
    request(P, 0);   // the frames' first slab is on its way while the records are read
    int t = tid;                          // the thread's record: frame t / recs of the workgroup
    u32x4 left{0u, 0u, 0u, 0u};           // its outputs that are still to be taken
    bool loaded = false, again = false;   // again: not the first pass over the frames
    for (;;) {
        if (tid == 0) total_s = 0u;
        __syncthreads();
        while (t < kResolveFrames * recs) {
            const int r = t / recs, q = t - r * recs;
            if (!loaded) {
                if (m0 + r < M) left = *reinterpret_cast<const u32x4*>(undecided + ((size_t)(m0 + r) * recs + q) * kUndecidedRecord);
                loaded = true;
            }
            const int cnt = __builtin_popcount(left.x) + __builtin_popcount(left.y) + __builtin_popcount(left.z) + __builtin_popcount(left.w);
            if (cnt) {
                // (places are given out without gaps, so a list that could not take everything is full)
                const unsigned int base = atomicAdd(&total_s, (unsigned int)cnt);
                const int room = base < (unsigned int)kResolveCap ? min(cnt, kResolveCap - (int)base) : 0;
                for (int i = 0; i < room; ++i) {
                    const int w = left.x ? 0 : left.y ? 1 : left.z ? 2 : 3;
                    const uint32_t v = left.x ? left.x : left.y ? left.y : left.z ? left.z : left.w;
                    const uint32_t rest = v & (v - 1u);
                    ent[base + i] = ((unsigned int)r << 28) | (unsigned int)(q * kUndecidedOutputs + 32 * w + __builtin_ctz(v));
                    if (w == 0) left.x = rest;
                    else if (w == 1) left.y = rest;
                    else if (w == 2) left.z = rest;
                    else left.w = rest;
                }
                if (room < cnt) break;
            }
            t += kResolveThreads;
            loaded = false;
        }
        __syncthreads();
        const unsigned int found = total_s;                          // workgroup-uniform
        const int total = (int)min(found, (unsigned int)kResolveCap);
        for (int first = 0; first < total; first += kResolveThreads) {   // workgroup-uniform
            const bool active = first + tid < total;
            const unsigned int e = ent[active ? first + tid : 0];
            const int r = (int)(e >> 28), n = (int)(e & 0x0FFFFFFFu);
            const uint32_t* wrow = Wp + (size_t)n * w32;
            const int wlast = (K - 1) >> 5;
            constexpr int kWords = kResolveSlab / 32;
            static_assert(kWords == 8, "eight weight words per slab and lane");
            float acc32 = 0.0f;
            struct Words { u32x4 lo, hi; };
            auto words = [&](Words& w, int sl) {
                uint32_t v[kWords];
    #pragma unroll
                for (int b = 0; b < kWords; ++b) v[b] = wrow[min(sl * kWords + b, wlast)];
                w.lo = u32x4{v[0], v[1], v[2], v[3]};
                w.hi = u32x4{v[4], v[5], v[6], v[7]};
            };
            // What comes from global memory (the frames' next slab, the lane's next eight weight words) is requested before
            // the slab is added up and goes to LDS after it: nothing in between waits for memory.
            Words W;
            __syncthreads();   // the previous pass no longer reads the buffers
            if (again) request(P, 0);
            again = true;
            words(W, 0);
            deposit(P, 0);
            ws[0][tid][0] = W.lo;
            ws[0][tid][1] = W.hi;
            __syncthreads();
            for (int sl = 0; sl < nsl; ++sl) {
                if (sl + 1 < nsl) {   // workgroup-uniform
                    request(P, sl + 1);
                    words(W, sl + 1);
                }
                if (active) {
                    // The slab's 256 terms as one stream (the last slab of a frame is padded with +0).  A result is ready some
                    // clocks after its instruction, and a wave has nothing else to issue meanwhile, so no instruction reads
                    // what one of the two before it wrote: around the addition of term t stand the mask of term t + 4, the
                    // shift of term t + 8 and, every fourth term, the LDS read of terms t + 16 .. t + 19.
                    const u32x4 lo = ws[sl & 1][tid][0], hi = ws[sl & 1][tid][1];
                    const uint32_t wc[kWords] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
                    resolve_slab(K - sl * kResolveSlab, &xs[sl & 1][r][0], wc, acc32, std::make_integer_sequence<int, kResolveSlab + 16>{});
                }
                if (sl + 1 < nsl) {
                    deposit(P, sl + 1);
                    ws[(sl + 1) & 1][tid][0] = W.lo;
                    ws[(sl + 1) & 1][tid][1] = W.hi;
                }
                __syncthreads();
            }
            if (active) {
                const int m = m0 + r;
                const float s1 = scale ? scale[n] : 1.0f, b1 = bias ? bias[n] : 0.0f;
                if (sign_bit(affine(s1, acc32, b1))) atomicOr(&Y[(size_t)m * yw32 + (n >> 5)], 1u << (n & 31));
            }
        }
        if (found <= (unsigned int)kResolveCap) return;   // every record is empty
        __syncthreads();                                  // (nobody clears total_s before all have read it)
    }
}

}  // namespace bnn
