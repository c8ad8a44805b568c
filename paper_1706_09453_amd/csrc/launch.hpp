// Launchers that live in translation units of their own (compiled side by side), and what they share.
#pragma once

#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>

#include "bnn_device.hpp"

namespace bnn {

inline bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

// Dynamic LDS above 64 KiB has to be allowed once per kernel and device.  `bytes` is the most the kernel ever asks for and
// the same in every call, so threads that get here together all set the same value.  false: refused.
template <class Kernel>
bool allow_lds(Kernel kernel, unsigned bytes, std::atomic<uint64_t>& allowed) {
    int dev = 0;
    (void)hipGetDevice(&dev);
    const uint64_t bit = dev >= 0 && dev < 64 ? 1ull << dev : 0;   // (devices past 64: asked for every time)
    if (allowed.load(std::memory_order_relaxed) & bit) return true;
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    allowed.fetch_or(bit);
    return true;
}

// A launch of this grid clears.
inline Clear cleared_by(Clear c, dim3 grid) {
    c.gx = (int)grid.x;
    c.blocks = (int)(grid.x * grid.y);
    return c;
}

// Ascending-k fp32 sums on the matrix cores (f32_chain_launch.hpp); arguments already checked.
struct ChainArgs {
    const float* X;
    const void* W;   // packed bits, or fp32 with real weights
    const float *scale, *bias;
    int M, K, N, w32;
    void* Y;
    int yw32;
    hipStream_t st;
    Clear clear{};   // Sign layers: memory that the launch sets to 0
};
void launch_chain_bits(const ChainArgs& a, int act);   // W packed bits
void launch_chain_real(const ChainArgs& a, int act);   // W fp32

}  // namespace bnn
