// Sign binarisation and bit packing (paper Eq. 3), and the per-layer scale mean|w|.
#pragma once

#include "bnn_device.hpp"

namespace bnn {

// One wavefront turns up to 64 B consecutive elements of a row into B ballots of 64: B coalesced 256-byte reads in
// flight, 2 B 32-bit words written by one store.  Bound by memory: long rows want eight (4096 x 2048 numbers took 18 us with
// one, now 10), rows of up to 64, 128 or 256 numbers no more than they fill (50000 x 64 17 us with eight, 7 with one).
// `w32` is the row length of the output in 32-bit words (for 64-bit packing it is twice the 64-bit word count, so the bytes
// are the same little-endian words).
template <int B>
__global__ __launch_bounds__(256) void pack_sign_kernel(const float* __restrict__ X, int64_t rows, int64_t K,
                                                        int64_t w32, uint32_t* __restrict__ out) {
    constexpr int kPackElems = 64 * B;
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t per_row = B < 8 ? 1 : (K + kPackElems - 1) / kPackElems;   // (fewer ballots: the row fits, see run_pack)
    const int64_t tasks = rows * per_row;
    const int64_t nwaves = (int64_t)gridDim.x * 4;
    for (int64_t task = (int64_t)blockIdx.x * 4 + wave; task < tasks; task += nwaves) {
        // (a wave-uniform 64-bit division is a long chain of scalar instructions: 32 bits where they suffice)
        const int64_t row = B < 8 ? task : tasks < ((int64_t)1 << 31) ? (int64_t)((uint32_t)task / (uint32_t)per_row) : task / per_row;
        const int64_t c = task - row * per_row;
        const float* x = X + row * K + c * kPackElems;
        const int n = (int)min(K - c * kPackElems, (int64_t)kPackElems);   // elements of this task
        float v[kPackElems / 64];
#pragma unroll
        for (int i = 0; i < kPackElems / 64; ++i) v[i] = x[min(64 * i + lane, n - 1)];
        uint32_t word = 0u;   // lane l: word l of the task
#pragma unroll
        for (int i = 0; i < kPackElems / 64; ++i) {
            const unsigned long long mask = __ballot(64 * i + lane < n && sign_bit(v[i]));
            word = lane == 2 * i ? (uint32_t)mask : (lane == 2 * i + 1 ? (uint32_t)(mask >> 32) : word);
        }
        const int64_t w = c * (kPackElems / 32) + lane;
        if (lane < kPackElems / 32 && w < w32) out[row * w32 + w] = word;
    }
}

// mean|w| over `count` elements: one workgroup, every thread keeps an fp64 partial over a fixed
// strided subset, then a fixed tree over LDS.  The order never depends on timing, so the result is
// reproducible bit for bit.  Off the per-frame path (runs once per layer when a model is prepared).
__global__ __launch_bounds__(1024) void mean_abs_kernel(const float* __restrict__ W, int64_t count,
                                                        float* __restrict__ out) {
    __shared__ double part[1024];
    double s = 0.0;
    for (int64_t i = threadIdx.x; i < count; i += 1024) s += (double)__builtin_fabsf(W[i]);
    part[threadIdx.x] = s;
    __syncthreads();
    for (int stride = 512; stride > 0; stride >>= 1) {
        if ((int)threadIdx.x < stride) part[threadIdx.x] += part[threadIdx.x + stride];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = (float)(part[0] / (double)count);
}

}  // namespace bnn
