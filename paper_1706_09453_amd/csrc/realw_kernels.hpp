// Layers that keep real-valued weights (paper Sec. 2.2, last paragraph, and Sec. 3.1: the input layer and the Softmax
// layer are not binarised): acc[m][n] = sum_k W[n][k] x[m][k] in fp32, ascending k, one accumulator per output, one
// fused multiply-add per step -- the order of the binary-weight product of valu_kernels.hpp, to which this reduces
// bit for bit when every weight is +1 or -1.  Then h^ = acc + bias (one rounding) and the activation.
//
// The chains run in f32_chain_kernels.hpp.  Here:
//   realw_gemv_kernel         up to 4 frames, outputs that go into the log-Softmax: K split over the lanes
//   realw_frames16_kernel     up to 64 frames, the same outputs: K split over the waves, matrix cores
//   bits_to_real_kernel       packed bits of a binary layer -> the fp32 numbers they stand for (-1/+1 or 0/1), for a
//                             real-weight layer that follows a binary one
#pragma once

#include <type_traits>

#include "bnn_device.hpp"

namespace bnn {

// Real-weight layer in front of the log-Softmax for a handful of frames (streaming): z[m][n] = sum_k W[n][k] x[m][k]
// + bias[n] with K split over the lanes.  27.9 MB of fp32 weights (the paper's 2048 -> 3400 Softmax layer) have to
// pass through the chip once per 4 frames; with lanes <-> outputs only N / 64 waves would pull them, here
// N / 4 waves do, each reading whole rows with 16-byte loads (a wave reads 1 KiB of a row at a time).  Lane l
// sums k = 256 s + 4 l .. + 3 over s in fp32, then the 64 partial sums are added by a butterfly of lane exchanges:
// a fixed order, but not the ascending-k chain, so this serves only the layer whose outputs go straight into the
// log-Softmax (the same rule as the matrix-core kernel for large batches).
// K a multiple of 4, X and W 16-byte aligned.  Grid: x = ceil(N / 16), y = ceil(M / 4); 4 waves x 4 rows.
__global__ __launch_bounds__(256) void realw_gemv_kernel(const float* __restrict__ X, const float* __restrict__ W,
                                                         const float* __restrict__ bias, int M, int K, int N,
                                                         float* __restrict__ Z) {
    constexpr int R = 4, FR = 4;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = lane_id();
    const int n0 = ((int)blockIdx.x * 4 + wave) * R;
    if (n0 >= N) return;
    const int m0 = (int)blockIdx.y * FR;
    const float* wr[R];
    const float* xr[FR];
#pragma unroll
    for (int r = 0; r < R; ++r) wr[r] = W + (size_t)(n0 + r < N ? n0 + r : N - 1) * K;
#pragma unroll
    for (int i = 0; i < FR; ++i) xr[i] = X + (size_t)(m0 + i < M ? m0 + i : M - 1) * K;

    float acc[R][FR];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int i = 0; i < FR; ++i) acc[r][i] = 0.0f;

    const int nsteps = (K + 255) / 256;
#pragma unroll 2
    for (int s = 0; s < nsteps; ++s) {
        const int k = 256 * s + 4 * lane;
        const bool in = k < K;            // K % 4 == 0: all four or none; past K the row's first four are read and dropped
        const int kk = in ? k : 0;
        float4 w[R], x[FR];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            w[r] = *reinterpret_cast<const float4*>(wr[r] + kk);
            if (!in) w[r] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);   // fma(0, 0, acc) returns acc: no branch around the loads
        }
#pragma unroll
        for (int i = 0; i < FR; ++i) {
            x[i] = *reinterpret_cast<const float4*>(xr[i] + kk);
            if (!in) x[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        }
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int i = 0; i < FR; ++i) {
                acc[r][i] = __builtin_fmaf(w[r].x, x[i].x, acc[r][i]);
                acc[r][i] = __builtin_fmaf(w[r].y, x[i].y, acc[r][i]);
                acc[r][i] = __builtin_fmaf(w[r].z, x[i].z, acc[r][i]);
                acc[r][i] = __builtin_fmaf(w[r].w, x[i].w, acc[r][i]);
            }
    }
    // butterfly: after the step with distance d every lane holds the sum over its group of 2 d lanes
#pragma unroll
    for (int d = 1; d < 64; d <<= 1)
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int i = 0; i < FR; ++i) acc[r][i] += __shfl_xor(acc[r][i], d, 64);
    // lane r * FR + i stores output (frame m0 + i, row n0 + r)
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int i = 0; i < FR; ++i)
            if (lane == r * FR + i && n0 + r < N && m0 + i < M)
                Z[(size_t)(m0 + i) * N + n0 + r] = affine(1.0f, acc[r][i], bias ? bias[n0 + r] : 0.0f);
}

// The same for more frames, 16 of them at a time on the fp32 matrix cores: a workgroup takes 16 rows of W, its eight waves the
// groups of 16 k in turn, four and the next four requested ahead of the products.  Bound: the weights, once per
// 16 frames.  A group's four V_MFMA_F32_16X16X4_F32 go to one of eight accumulators, so that a sum is 64 chains of K / 64 terms (32
// at K = 2048, as many as a lane of the kernel above adds up), put together pairwise: within a wave, then over the waves.  Lane (r, g) holds
// k = 16 group + 4 g .. + 3 of row r of both operands, and step t multiplies the t-th of them.
// K a multiple of 4, X and W 16-byte aligned.  Grid: x = ceil(N / 16), y = ceil(M / 16).
// Whole layers with their log-Softmax, weights from memory (before: the kernel above with eight frames at a time): 16 frames of 2048 x
// 3400 20.0 -> 15.8 us, 64 of them 43.4 -> 37.4; 16 of 4096 x 4000 37.0 -> 25.9, 64 101 -> 69; 5 of 512 x 1000 8.8 -> 8.4; error
// against 64 bits the same.  124 registers leave room for two workgroups on a CU (with eight groups to a turn, 192, 64 frames took 45.0).
constexpr int kFrames16Waves = 8, kFrames16Threads = kFrames16Waves * kWave;
__global__ __launch_bounds__(kFrames16Threads, 4) void realw_frames16_kernel(const float* __restrict__ X, const float* __restrict__ W,
                                                                          const float* __restrict__ bias, int M, int K, int N,
                                                                          float* __restrict__ Z) {
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    constexpr int B = 4;   // groups of a turn: two turns in flight, accumulators of their own
    __shared__ f32x4 part[kFrames16Waves][kWave];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = lane_id(), r = lane & 15, g = lane >> 4;
    const int n0 = (int)blockIdx.x * 16, m0 = (int)blockIdx.y * 16;
    const float* wrow = W + (size_t)min(n0 + r, N - 1) * K;
    const float* xrow = X + (size_t)min(m0 + r, M - 1) * K;
    struct Groups { f32x4 w[B], x[B]; };
    auto request = [&](Groups& G, int turn) {
#pragma unroll
        for (int i = 0; i < B; ++i) {
            const int k = 16 * (kFrames16Waves * (B * turn + i) + wave) + 4 * g;
            const bool in = k < K;   // K % 4 == 0: all four or none; past K the row's first four are read and dropped
            G.w[i] = *reinterpret_cast<const f32x4*>(wrow + (in ? k : 0));
            G.x[i] = *reinterpret_cast<const f32x4*>(xrow + (in ? k : 0));
            if (!in) G.w[i] = G.x[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        }
    };
    f32x4 acc[2 * B];
#pragma unroll
    for (int i = 0; i < 2 * B; ++i) acc[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    auto multiply = [&](const Groups& G, auto to) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int i = 0; i < B; ++i) acc[decltype(to)::value + i] = __builtin_amdgcn_mfma_f32_16x16x4f32(G.w[i][t], G.x[i][t], acc[decltype(to)::value + i], 0, 0, 0);
    };
    const int turns = (K + 16 * kFrames16Waves * B - 1) / (16 * kFrames16Waves * B);
    Groups a, b;
    request(a, 0);
    request(b, 1);   // (past the end: zeros)
    for (int turn = 0; turn < turns; turn += 2) {
        multiply(a, std::integral_constant<int, 0>{});
        if (turn + 2 < turns) request(a, turn + 2);
        multiply(b, std::integral_constant<int, B>{});
        if (turn + 2 < turns) request(b, turn + 3);
    }
    part[wave][lane] = ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
    __syncthreads();
    if (wave != 0) return;
    f32x4 s[kFrames16Waves];
#pragma unroll
    for (int i = 0; i < kFrames16Waves; ++i) s[i] = part[i][lane];
    const f32x4 sum = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
    // register v of lane (r, g): frame m0 + r, output n0 + 4 g + v
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int n = n0 + 4 * g + v;
        if (n < N && m0 + r < M) Z[(size_t)(m0 + r) * N + n] = affine(1.0f, sum[v], bias ? bias[n] : 0.0f);
    }
}

// out[m][k] = bit k of row m ? 1.0f : (zero_one ? 0.0f : -1.0f).  One thread per element, grid-stride.
__global__ __launch_bounds__(256) void bits_to_real_kernel(const uint32_t* __restrict__ Xp, int64_t M, int K, int w32,
                                                           int zero_one, float* __restrict__ out) {
    const int64_t total = M * (int64_t)K;
    const float low = zero_one ? 0.0f : -1.0f;
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (int64_t)gridDim.x * 256) {
        const int64_t m = e / K;
        const int k = (int)(e - m * K);
        out[e] = ((Xp[m * w32 + (k >> 5)] >> (k & 31)) & 1u) ? 1.0f : low;
    }
}

}  // namespace bnn
