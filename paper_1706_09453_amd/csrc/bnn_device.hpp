// Device-side helpers shared by the gfx950 kernels of the binary-network forward pass.
// Written for CDNA4 only: 64-wide wavefronts, no portability layer.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace bnn {

constexpr int kWave = 64;

// Activation selectors; numerically identical to bnn_act in include/bnn.h.
enum : int { ACT_RAW_I32 = 0, ACT_LINEAR = 1, ACT_HARDTANH = 2, ACT_SIGN = 3, ACT_LOGSOFTMAX = 4, ACT_SIGMOID = 5 };
// Kernel-internal: the integer product as int16 in the first 2 N bytes of each fp32 output row (|dot| <= K < 2^15);
// the log-Softmax row kernel turns the row into fp32 log-posteriors in place.
enum : int { ACT_DOT_I16 = 100 };
// Kernel-internal: log-Softmax finished inside the product kernel.  The workgroups that share rows of frames hand each
// other their share of every row's maximum and sum of exponentials through memory (see CoopLsm); needs every workgroup
// of the launch resident at once.
enum : int { ACT_LSM_COOP = 101 };

// Hand-over area of ACT_LSM_COOP.  Tile (tm, tn) of the launch writes partials[(tm * n_tiles + tn) * rows_per_tile + row]
// = (max, sum of exp(h - max)) of `row` over its columns, then flags[tm * n_tiles + tn] = stamp.  Stamps are unique per
// launch, so what an earlier launch left in the area never reads as this launch's.
struct CoopLsm {
    float2* partials;
    unsigned long long* flags;
    unsigned long long stamp;
    unsigned int* timeouts;   // incremented by a workgroup whose bounded wait ran out (its rows are then wrong)
    int spin_limit;           // polls of the flags before a workgroup gives up
};

// The XCD that the wave runs on (bits 0..3 of hardware register 20, HW_REG_XCC_ID) and 1: what a workgroup marks data with that lies in
// its XCD's L2, so that whoever runs on another one does not take the mark for its own.  Never 0.
__device__ __forceinline__ uint32_t xcd_mark() { return (uint32_t)__builtin_amdgcn_s_getreg(20 | 3 << 11) + 1u; }

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & (kWave - 1)); }

typedef int i32x4m __attribute__((ext_vector_type(4)));
// 16 bytes per lane from byte `voff` (per lane) + `soff` (wave-uniform) of a buffer to LDS: lane i's go to lds + 16 i.  The
// request is counted by vmcnt only: whoever reads the LDS waits for it and then crosses a barrier.  (Written out because the
// compiler, not knowing which stage a later LDS read belongs to, makes every read wait for every such load.)
__device__ __forceinline__ void load_lds16(i32x4m rsrc, int voff, int soff, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
}
// the same with 4 bytes per lane: lane i's go to lds + 4 i
__device__ __forceinline__ void load_lds4(i32x4m rsrc, int voff, int soff, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, %3 offen lds" ::"s"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
}
// 16 bytes per lane from an address per lane: lane i's go to lds + 16 i
__device__ __forceinline__ void load_lds16_at(const void* p, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds), "v"(p) : "memory");
}
__device__ __forceinline__ i32x4m raw_buffer(const void* p, unsigned int bytes) {
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    return i32x4m{(int)(uint32_t)a, (int)((uint32_t)(a >> 32) & 0xFFFFu), (int)bytes, 0x00020000};
}

// The tile of a workgroup in a grid of gridDim.x tile rows by gridDim.y tile columns.  Workgroups go round the eight XCDs: here an
// XCD takes consecutive tiles in an order that runs down two tile rows at a time, so that its L2 serves few rows and many
// columns whatever the number of tile rows.  (In the launch's own order it does so only where that is a multiple of eight.)
__device__ __forceinline__ void xcd_tile(int& tm, int& tn) {
    const int gx = (int)gridDim.x, gy = (int)gridDim.y, total = gx * gy, id = (int)blockIdx.x + gx * (int)blockIdx.y;
    const int xcd = id & 7, t = xcd * (total >> 3) + min(xcd, total & 7) + (id >> 3);
    const int pair = t / (2 * gy), in = t - pair * (2 * gy);
    const bool two = 2 * pair + 1 < gx;   // (an odd number of tile rows: the last one alone)
    tm = 2 * pair + (two ? in & 1 : 0);
    tn = two ? in >> 1 : in;
}

// 16-byte pieces that a launch sets to 0 for the launch behind it (few_chain_kernel.hpp): by its first `blocks` workgroups, `gx` of them
// in x.  (Both are here and not read from the grid: with more than 112 bytes of arguments, what the runtime adds for the grid's size
// among them, a launch takes the host 3.5 us instead of 2.9.)
struct Clear {
    uint4* at;
    int pieces, gx, blocks;
};
template <int THREADS>
__device__ __forceinline__ void clear_pieces(const Clear& c) {
    const uint32_t block = blockIdx.y * (uint32_t)c.gx + blockIdx.x;
    for (uint32_t i = block * (uint32_t)THREADS + threadIdx.x; i < (uint32_t)c.pieces; i += (uint32_t)c.blocks * (uint32_t)THREADS) c.at[i] = make_uint4(0u, 0u, 0u, 0u);
}

// Memory that a launch's workgroups behind those of Clear pull into the L2s of the first `xcds` XCDs, for the launch behind it
// (few_chain_kernel.hpp): 32 of them on each XCD, workgroups going round the XCDs.  A first layer of few frames leaves most of the chip idle for
// 5 to 15 us.  Behind other work, which has used the L2s, one frame through six layers of 2048 units takes 23.4 -> 21.6 us; back to back
// it makes no difference.
constexpr int kPullLayers = 16, kPullGroups = 32;
struct Pull {
    const char* at[kPullLayers];
    uint32_t bytes[kPullLayers];
    int layers, xcds;
};
__device__ __forceinline__ void pull_memory(const Pull& p, int block, int from, int thread) {
    if ((block & 7) >= p.xcds) return;
    const uint32_t first = (uint32_t)((block - from) >> 3) * 256u + (uint32_t)thread;
    for (int j = 0; j < p.layers; ++j)
        for (uint32_t at = first * 128u; at < p.bytes[j]; at += kPullGroups * 256u * 128u) {
            const uint32_t t = *reinterpret_cast<const uint32_t*>(p.at[j] + at);
            asm volatile("" ::"v"(t));
        }
}

// Both, in front of a kernel of 256 threads.  false: this workgroup has pulled, there is nothing else for it to do.
__device__ __forceinline__ bool front_of_run(const Clear& c, const Pull& p) {
    const int block = (int)(blockIdx.y * (uint32_t)c.gx + blockIdx.x);
    if (block >= c.blocks) {
        pull_memory(p, block, c.blocks, (int)threadIdx.x);
        return false;
    }
    clear_pieces<256>(c);
    return true;
}

// Eq. 3 of the paper: +1 exactly when v > 0 (0, -0 and NaN give -1, i.e. bit 0).
__device__ __forceinline__ bool sign_bit(float v) { return v > 0.0f; }

// Eq. 1 with the per-layer scale: one fused multiply-add, a single rounding.
__device__ __forceinline__ float affine(float scale, float v, float bias) { return __builtin_fmaf(scale, v, bias); }

__device__ __forceinline__ float hardtanh(float v) {
    v = v > 1.0f ? 1.0f : v;
    v = v < -1.0f ? -1.0f : v;
    return v;
}

// exp(x) in fp64 for |x| <= 1000 (a NaN stays one): x = n ln 2 + r with |r| <= ln 2 / 2 (ln 2 in two parts, so that r is
// exact to fp64), the Taylor series of exp(r) up to r^13 / 13! (the rest is below 5e-18), times 2^n.  Within 1.5 units
// in the last place; about 20 instructions, half of what the library function takes with its range checks.
__device__ __forceinline__ double exp_f64(double x) {
    const double n = __builtin_rint(x * 1.4426950408889634074);
    double r = __builtin_fma(n, -0x1.62e42fefa3800p-1, x);    // ln 2, upper 42 bits: n times it is exact
    r = __builtin_fma(n, -0x1.ef35793c76730p-45, r);           // ln 2 - upper part
    double p = 1.0 / 6227020800.0;
    p = __builtin_fma(p, r, 1.0 / 479001600.0);
    p = __builtin_fma(p, r, 1.0 / 39916800.0);
    p = __builtin_fma(p, r, 1.0 / 3628800.0);
    p = __builtin_fma(p, r, 1.0 / 362880.0);
    p = __builtin_fma(p, r, 1.0 / 40320.0);
    p = __builtin_fma(p, r, 1.0 / 5040.0);
    p = __builtin_fma(p, r, 1.0 / 720.0);
    p = __builtin_fma(p, r, 1.0 / 120.0);
    p = __builtin_fma(p, r, 1.0 / 24.0);
    p = __builtin_fma(p, r, 1.0 / 6.0);
    p = __builtin_fma(p, r, 0.5);
    p = __builtin_fma(p, r, 1.0);
    p = __builtin_fma(p, r, 1.0);
    return __builtin_amdgcn_ldexp(p, (int)n);
}

// Sigmoid of the paper's real hidden layers (Sec. 3), evaluated in fp64 and rounded once to fp32, as the reference
// definition does: a layer of Sign units that reads these values must see the same fp32 numbers, bit for bit, or a
// unit whose pre-activation is nearly zero flips and every binary layer after it diverges.  (An fp32 exp is within
// 1e-6, which is fine for the values and fatal for the bits.)  Two fp64 evaluations can differ in the last
// places of the fp64 result; that survives the rounding to fp32 with probability about 2^-28 per value.
// The reciprocal of 1 + exp(-v) <= 1 + e^700 is the hardware's estimate and two Newton steps.
__device__ __forceinline__ float sigmoid(float v) {
    v = v < -700.0f ? -700.0f : v;   // 1 / (1 + e^700) is 0 in fp32 already; NaN passes
    v = v > 700.0f ? 700.0f : v;
    const double d = 1.0 + exp_f64(-(double)v);
    double y = __builtin_amdgcn_rcp(d);
    y = __builtin_fma(y, __builtin_fma(-d, y, 1.0), y);
    y = __builtin_fma(y, __builtin_fma(-d, y, 1.0), y);
    return (float)y;
}

// +1.0f or -1.0f from bit `pos` of `inv` where inv holds the COMPLEMENT of the weight bits
// (weight bit 1 <=> +1 <=> float sign bit clear).
__device__ __forceinline__ float pm1_from_inverted_bit(uint32_t inv, int pos) {
    const uint32_t s = (inv << (31 - pos)) & 0x80000000u;
    return __uint_as_float(s | 0x3f800000u);
}

}  // namespace bnn
