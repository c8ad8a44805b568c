// A layer with real-valued weights and real-valued inputs in front of the log-Softmax (paper Sec. 3.1: the Softmax
// layer keeps real weights; Sec. 4.3: sigmoid networks hand it real inputs) on the bf16 matrix cores,
// V_MFMA_F32_32X32X16_BF16, at fp32 accuracy.
//
// Every fp32 operand v is written as v = p0 + p1 + p2 + rest with three bf16 pieces: p0 = bf16(v), p1 = bf16(v - p0),
// p2 = bf16(v - p0 - p1), each rounded to nearest, each difference exact in fp32; |rest| <= 2^-24 |v| (a bf16 keeps
// 8 significant bits).  A product x w is taken as the six piece products whose weights are 2^-16 or more,
//     x0 w2 + x1 w1 + x2 w0 + x0 w1 + x1 w0 + x0 w0,
// every one exact in the matrix core's fp32 (8 x 8 significant bits) and added to an fp32 accumulator.  What is left
// out (x1 w2, x2 w1, x2 w2 and the two rests) is below 2^-22 |x w| per term, so the sum differs from the exact one by
// at most 2^-22 sum_k |x_k w_k| plus ordinary fp32 rounding of the accumulation, the same kind of difference the fp32
// matrix-core kernel has (its own rounding bound is K 2^-24 sum_k |x_k w_k|).  One V_MFMA_F32_32X32X16_BF16 does 16 k
// in 8 passes where V_MFMA_F32_32X32X2_F32 needs 8 instructions of 16 passes: six of them are 2.7 times cheaper.
// Layers whose outputs are Sign bits never use this kernel: bits are defined from the fp32 sum in ascending k.
//
// Two kernels: the split (one pass over each operand, pieces to planes [piece][row][kpad] of bf16 in the caller's
// workspace, kpad = K rounded up to 32, zeros past K), then the product kernel below.
#pragma once

#include <type_traits>

#include "bnn_device.hpp"

namespace bnn {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float v16f32s __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kSplitPieces = 3;
constexpr int kSplitKStep = 32;                                  // k per pipeline step: 64 bytes of a plane row
constexpr int kSplitRowBytes = kSplitKStep * 2;
// A workgroup of 2 x 2 waves of 32 WM frames x 32 WN outputs each; two stages of 256 x 128 or three of 128 x 128 fit a CU's LDS.
__host__ __device__ constexpr int split_stage(int wm, int wn) { return kSplitPieces * 64 * (wm + wn) * kSplitRowBytes; }   // 73728 / 49152
__host__ __device__ constexpr int split_stages(int wm, int wn) { return 3 * split_stage(wm, wn) <= 163840 ? 3 : 2; }
__host__ __device__ constexpr unsigned split_dynamic_lds(int wm, int wn) { return (unsigned)(split_stages(wm, wn) * split_stage(wm, wn)); }

constexpr int kSplitLongRow = 1 << 22;   // kpad from which the offsets of 256 rows do not fit 31 bits

__host__ __device__ inline int split_kpad(int K) { return (K + kSplitKStep - 1) / kSplitKStep * kSplitKStep; }

// bf16 nearest to v (ties to even) as its 16 bits; a finite v that would round to infinity is truncated instead, so that
// the pieces of a finite value stay finite.
__device__ inline uint32_t bf16_bits(float v) {
    uint32_t h = (uint32_t)__builtin_bit_cast(unsigned short, (__bf16)v);
    const uint32_t u = __float_as_uint(v);
    if ((h & 0x7fffu) == 0x7f80u && (u & 0x7f800000u) != 0x7f800000u) h = u >> 16;
    return h;
}

// The three pieces of v.  A non-finite v gives p0 = v and NaN further down, so every sum it enters ends up NaN or
// infinite, as the exact sum does before the log-Softmax turns the row into NaN.
__device__ inline void split3(float v, uint32_t& p0, uint32_t& p1, uint32_t& p2) {
    p0 = bf16_bits(v);
    const float r1 = v - __uint_as_float(p0 << 16);
    p1 = bf16_bits(r1);
    const float r2 = r1 - __uint_as_float(p1 << 16);
    p2 = bf16_bits(r2);
}

// planes[p][row][kpad] <- piece p of A[row][k] (zero for K <= k < kpad).  One thread per 8 consecutive k.
// VEC: K % 4 == 0 and A 16-byte aligned.  Grid: any number of blocks of 256 threads (grid-stride).
template <bool VEC>
__global__ __launch_bounds__(256) void split_bf16x3_kernel(const float* __restrict__ A, int64_t rows, int K, int kpad,
                                                            uint16_t* __restrict__ planes) {
    const int per_row = kpad >> 3;
    const int64_t total = rows * per_row;
    const size_t plane = (size_t)rows * (size_t)kpad;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
        const int64_t row = i / per_row;
        const int k0 = (int)(i - row * per_row) * 8;
        const float* a = A + (size_t)row * K;
        float v[8];
        if (VEC && k0 + 7 < K) {
            const float4 lo = *reinterpret_cast<const float4*>(a + k0);
            const float4 hi = *reinterpret_cast<const float4*>(a + k0 + 4);
            v[0] = lo.x; v[1] = lo.y; v[2] = lo.z; v[3] = lo.w;
            v[4] = hi.x; v[5] = hi.y; v[6] = hi.z; v[7] = hi.w;
        } else {
#pragma unroll
            for (int t = 0; t < 8; ++t) v[t] = (k0 + t < K) ? a[k0 + t] : 0.0f;
        }
        uint32_t w[kSplitPieces][4];
#pragma unroll
        for (int t = 0; t < 8; t += 2) {
            uint32_t a0, a1, a2, b0, b1, b2;
            split3(v[t], a0, a1, a2);
            split3(v[t + 1], b0, b1, b2);
            w[0][t >> 1] = a0 | (b0 << 16);
            w[1][t >> 1] = a1 | (b1 << 16);
            w[2][t >> 1] = a2 | (b2 << 16);
        }
        const size_t at = (size_t)row * kpad + k0;
#pragma unroll
        for (int p = 0; p < kSplitPieces; ++p)
            *reinterpret_cast<uint4*>(planes + p * plane + at) = make_uint4(w[p][0], w[p][1], w[p][2], w[p][3]);
    }
}

// Y[m][n] = bias[n] + sum_k X[m][k] W[n][k] from the planes Xs [3][M][kpad] and Ws [3][N][kpad] (16-byte aligned,
// kpad % 32 == 0).  Grid: x = ceil(M / (64 WM)), y = ceil(N / (64 WN)); block = 256 threads; dynamic LDS split_dynamic_lds(WM, WN).
// One wave per SIMD.
//
// Pipeline, one step = 32 k = two MFMA blocks of 16: every tile row's 64 bytes of a piece go to LDS by loads that write it
// directly (16 bytes per lane, four lanes a row), two or three steps in rotation and one barrier per step, between its blocks:
// behind it step j + 1 is complete in LDS and every wave has read step j, whose place takes the next step.  A wave reads its
// operand fragments out of LDS one block ahead of the MFMAs that use them, one memory instruction between two MFMAs.  In LDS
// a row's four 16-byte slots are stored at slot ^ ((row / 4) % 4), which spreads the fragment reads of 16 lanes over all
// banks.  Lane (r = lane % 32, g = lane / 32) feeds row r, k = 8 g .. 8 g + 7 of a block to both operands.
// Against loads to registers and LDS stores (256 x 128 tiles only), whole layers: 4096 x 2048 x 3400 312 -> 298 us, 4221 x 4096 x 1024
// 283 -> 243, 600 x 2048 x 3400 128 -> 81.  What is slower: K above about 4800 with one round of large tiles and planes beyond the
// 256 MB of the last-level cache, 738 x 7200 x 7159 580 -> 640, 4812 x 5792 x 769 369 -> 401.
// LONG: kpad >= kSplitLongRow; addresses of 64 bits per lane instead of a buffer and an offset of 32.
template <int WM, int WN, bool LONG>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void realw_bf16x3_kernel(
    const uint16_t* __restrict__ Xs, const uint16_t* __restrict__ Ws, const float* __restrict__ bias, int M, int kpad, int N,
    float* __restrict__ Y) {
    extern __shared__ __attribute__((aligned(16))) unsigned char split_lds[];
    constexpr int kTileM = 64 * WM, kTileN = 64 * WN, kStages = split_stages(WM, WN), kStage = split_stage(WM, WN);
    constexpr int kStageA = kSplitPieces * kTileM * kSplitRowBytes;
    constexpr int NL = kSplitPieces * (WM + WN);     // loads per wave and step, of 16 rows each
    constexpr int NR = kSplitPieces * (WM + WN);     // fragment reads per wave and block
    constexpr int NM = 6 * WM * WN;                  // MFMAs per wave and block
    static_assert(NR <= NM && NL <= NM, "one read or load per MFMA");
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = lane_id();
    const int r = lane & 31, g = lane >> 5;
    // 4221 x 4096 x 1024, 17 x 8 tiles: 306 -> 248 us a layer with the tiles in the XCDs' order; 16 tile rows: nothing changes.  Short
    // sums are bound by the outputs, which the launch's own order stores faster (8206 x 16 x 898 47.6 and 51.4, 3828 x 50 x 2048
    // 34.6 and 37.3; from 200 terms on no difference).
    int tm = (int)blockIdx.x, tn = (int)blockIdx.y;
    if (kpad >= 256) xcd_tile(tm, tn);
    const int m_tile = tm * kTileM, n_tile = tn * kTileN;
    const int m_base = m_tile + (wave >> 1) * (WM * 32);
    const int n_base = n_tile + (wave & 1) * (WN * 32);

    // ---- the wave's share of a step's loads: piece i / (WM + WN); then frames 16 (WM wave + sub) .. of the tile for sub < WM,
    //      else weights rows 16 (WN wave + sub - WM) ..  One buffer per piece and operand, over the rows of the tile (rows past
    //      the end: the last one again).
    const int lrow = lane >> 2, lsrc = ((lane & 3) ^ ((lrow >> 2) & 3)) * 16;
    const int rows_a = min(M - m_tile, kTileM), rows_b = min(N - n_tile, kTileN), row_bytes = LONG ? 0 : 2 * kpad;
    i32x4m ars[kSplitPieces], brs[kSplitPieces];
    int aofs[WM], bofs[WN];
    const char *aptr[WM], *bptr[WN];
    if constexpr (LONG) {
#pragma unroll
        for (int i = 0; i < WM; ++i)
            aptr[i] = reinterpret_cast<const char*>(Xs + (size_t)(m_tile + min(16 * (WM * wave + i) + lrow, rows_a - 1)) * kpad) + lsrc;
#pragma unroll
        for (int i = 0; i < WN; ++i)
            bptr[i] = reinterpret_cast<const char*>(Ws + (size_t)(n_tile + min(16 * (WN * wave + i) + lrow, rows_b - 1)) * kpad) + lsrc;
    } else {
#pragma unroll
        for (int p = 0; p < kSplitPieces; ++p) {
            ars[p] = raw_buffer(Xs + ((size_t)p * M + m_tile) * kpad, (unsigned int)(rows_a * row_bytes));
            brs[p] = raw_buffer(Ws + ((size_t)p * N + n_tile) * kpad, (unsigned int)(rows_b * row_bytes));
        }
#pragma unroll
        for (int i = 0; i < WM; ++i) aofs[i] = min(16 * (WM * wave + i) + lrow, rows_a - 1) * row_bytes + lsrc;
#pragma unroll
        for (int i = 0; i < WN; ++i) bofs[i] = min(16 * (WN * wave + i) + lrow, rows_b - 1) * row_bytes + lsrc;
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)split_lds;
    auto request_one = [&](int step, uint32_t stage, int i) {
        const int p = i / (WM + WN), sub = i % (WM + WN), ia = sub < WM ? sub : 0, ib = sub < WM ? 0 : sub - WM;
        const uint32_t to = stage + (uint32_t)(sub < WM ? (p * kTileM + 16 * (WM * wave + ia)) * kSplitRowBytes
                                                        : kStageA + (p * kTileN + 16 * (WN * wave + ib)) * kSplitRowBytes);
        if constexpr (LONG) {
            const size_t at = (size_t)p * (sub < WM ? M : N) * kpad * 2 + (size_t)step * kSplitRowBytes;
            load_lds16_at((sub < WM ? aptr[ia] : bptr[ib]) + at, to);
        } else {
            load_lds16(sub < WM ? ars[p] : brs[p], sub < WM ? aofs[ia] : bofs[ib], step * kSplitRowBytes, to);
        }
    };

    // ---- the wave's operand fragments of block h (0 or 1) of a stage: NR reads, numbered like the loads
    struct Frags { bf16x8 a[kSplitPieces][WM]; bf16x8 b[kSplitPieces][WN]; };
    const int swz = (r >> 2) & 3;
    const int a_off = ((wave >> 1) * (WM * 32) + r) * kSplitRowBytes;
    const int b_off = kStageA + ((wave & 1) * (WN * 32) + r) * kSplitRowBytes;
    auto lread_one = [&](Frags& F, const unsigned char* stage, int h, int i) {
        const int so = ((2 * h + g) ^ swz) << 4;
        const int p = i / (WM + WN), sub = i % (WM + WN);
        if (sub < WM)
            F.a[p][sub < WM ? sub : 0] = *reinterpret_cast<const bf16x8*>(stage + p * (kTileM * kSplitRowBytes) + a_off +
                                                                         sub * (32 * kSplitRowBytes) + so);
        else
            F.b[p][sub < WM ? 0 : sub - WM] = *reinterpret_cast<const bf16x8*>(stage + p * (kTileN * kSplitRowBytes) + b_off +
                                                                              (sub - WM) * (32 * kSplitRowBytes) + so);
    };

    v16f32s acc[WM][WN];
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

    // One block of 16 k, written out MFMA by MFMA and pinned: the six piece products, smallest first; each accumulator is touched
    // once per WM WN MFMAs.  Behind each of the first ones a fragment read of the next block; REQ: the loads of step `step` to `stage`
    // spread evenly over the block.  (The four waves issue them together, 64 clocks in the one texture path: behind every one of the last
    // MFMAs they held these back, 4096 x 2048 x 3400 315 us a layer, spread 300.)
    auto block = [&](const Frags& now, Frags& next, const unsigned char* rd, int rd_h, auto req, int step, uint32_t stage) {
        constexpr bool REQ = decltype(req)::value;
        constexpr int px[6] = {0, 1, 2, 0, 1, 0};
        constexpr int pw[6] = {2, 1, 0, 1, 0, 0};
#pragma unroll
        for (int i = 0; i < NM; ++i) {
            const int q = i / (WM * WN), fm = (i / WN) % WM, fn = i % WN;
            acc[fm][fn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(now.a[px[q]][fm], now.b[pw[q]][fn], acc[fm][fn], 0, 0, 0);
            if (i < NR) lread_one(next, rd, rd_h, i);
            if (REQ && i * NL / NM != (i + 1) * NL / NM) request_one(step, stage, i * NL / NM);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    const int nS = kpad / kSplitKStep;
    auto turn = [&](int j) {   // step j + 2 may be on its way where there are three places
        if (kStages == 3 && j + 2 < nS) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(NL) : "memory");
        else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    Frags F0, F1;
#pragma unroll
    for (int st = 0; st < kStages; ++st)
        if (st < nS)
#pragma unroll
            for (int i = 0; i < NL; ++i) request_one(st, lds0 + (uint32_t)(st * kStage), i);
    if (kStages == 3 && nS > 2) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(2 * NL) : "memory");
    else if (nS > 1) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(NL) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
    for (int i = 0; i < NR; ++i) lread_one(F0, split_lds, 0, i);
    int slot = 0, j = 0;
    auto step = [&](auto req) {
        const int nslot = slot == kStages - 1 ? 0 : slot + 1;
        block(F0, F1, split_lds + slot * kStage, 1, std::false_type{}, 0, 0u);
        turn(j);
        // (behind the last step: its first block read again, unused)
        block(F1, F0, split_lds + (j + 1 < nS ? nslot : slot) * kStage, 0, req, j + kStages, lds0 + (uint32_t)(slot * kStage));
        slot = nslot;
    };
    for (; j + kStages < nS; ++j) step(std::true_type{});
    for (; j < nS; ++j) step(std::false_type{});
    __syncthreads();   // the buffers are free: the epilogue reuses them

    // ---- epilogue.  Accumulator fragment (fm, fn), register v of lane (r, g) is the sum for frame
    //      m_base + 32 fm + 8 (v/4) + 4 g + v%4 and output n_base + 32 fn + r.  Each wave turns 32 rows x 64 columns at
    //      a time through its own slice of LDS so that 16 lanes write 256 contiguous bytes of a row.
    if (m_base >= M || n_base >= N) return;   // wave-uniform, after the last barrier
    static_assert(WN == 2, "16 lanes store a row of 64 columns");
    constexpr int LDW = 32 * WN + 4;
    float* stg = reinterpret_cast<float*>(split_lds) + wave * (32 * LDW);
    float bi[WN];
#pragma unroll
    for (int f = 0; f < WN; ++f) {
        const int n = n_base + f * 32 + r;
        bi[f] = (n < N && bias) ? bias[n] : 0.0f;
    }
    const bool rows_vec = ((N & 3) == 0) && ((reinterpret_cast<uintptr_t>(Y) & 15) == 0);
    const int c4 = (lane & 15) * 4;
#pragma unroll
    for (int fm = 0; fm < WM; ++fm) {
#pragma unroll
        for (int fn = 0; fn < WN; ++fn)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                stg[(8 * (v >> 2) + 4 * g + (v & 3)) * LDW + fn * 32 + r] = acc[fm][fn][v] + bi[fn];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");   // this wave's LDS writes are done before it reads them back
#pragma unroll
        for (int it = 0; it < 8; ++it) {
            const int row = it * 4 + (lane >> 4);
            const int m = m_base + fm * 32 + row;
            const int n = n_base + c4;
            const float4 qv = *reinterpret_cast<const float4*>(stg + row * LDW + c4);
            if (m < M) {
                float* y = Y + (size_t)m * N + n;
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

}  // namespace bnn
