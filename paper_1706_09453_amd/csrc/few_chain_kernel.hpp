// A run of binary layers for a batch of a few frames, one launch for all of them (paper Alg. 2 forward, Sec. 2.3; the
// streaming batches of bnn_forward).
//
// Bound: latency.  One frame through a layer of 2048 units is 0.3 us of XOR and popcount on the chip; what a layer of its own costs is
// the launch (2.4 us from one dependent launch to the next).  Here the layers follow each other inside one launch, and the
// hand-over between them is made as short as the chip allows:
//   * frames are independent, so they are split over the eight XCDs: group g of workgroups (blockIdx mod 8, the order in which
//     workgroups go round the XCDs) takes frames g F .. g F + F - 1 through all layers, and what its waves hand each other
//     stays in that XCD's L2.  Between workgroups of one XCD a hand-over measured 0.55 us, across XCDs 2.7;
//   * a word of 32 output bits leaves as one 64-bit store with a mark in its upper half, and whoever needs it polls the word itself:
//     one way through the L2 and one back, no flag, no fence;
//   * a wave is on its own: it takes 32 outputs x the frames of its group, no barrier inside a layer; weights do not depend on the
//     layer before, so they are requested in front of the wait.
// No wave depends on another one being on the chip: a wave that has polled in vain `spins` times works out what is missing by itself, from
// the first layer on if need be, and every word has one possible value, so it makes no difference who publishes
// it.  That also covers workgroups of one group on different XCDs, which would not see each other's words, or later.  A word carries
// its mark, so it is complete wherever it is seen.  The last layer's pre-activations are stored apart from their marks, and of two lines
// in another XCD's L2 the mark's may be the first to reach memory: such a mark is the number of the writer's XCD (xcd_mark) and counts
// on that XCD only, whose L2 has the pre-activations since the store was acknowledged.  (On others: worked out again, the same numbers.)
// Only the speed rests on the order in which workgroups go round the XCDs.
// Workgroups of four waves with at most 128 registers and 16 KB of LDS, so that four launches fit on every CU, as many as the device's
// queues run at once.  Where fewer fit, runs on several streams each get a part of their workgroups, and all of them wait for the rest
// until they give up: with a fifth wave and 168 registers, two to a CU, 16 frames of 6 x 1536 units on four streams at once took 33 us a
// pass, 8.0 now (one launch per layer 10.0), 62 of 8 x 1088 73 and 15.3 (46).  (few_fresh keeps the
// registers down; the code for waits that run out had most of them.)  Alone, the two 18.9 -> 16.5 us and 36.5 -> 34.8.
// The marks have to be clear when the launch starts: the launch before it, which the first layer reads from, clears them.
//
// Measured: at few_chain_layers in bnn_api.hip.
#pragma once

#include <type_traits>

#include "bnn_device.hpp"
#include "softmax_kernels.hpp"

namespace bnn {

constexpr int kFewMaxLayers = 16, kFewMaxFrames = 64, kFewGroups = 8, kFewSlots = 32;   // (a group: 32 workgroups, one per CU of an XCD)
constexpr int kFewGroupFrames = kFewMaxFrames / kFewGroups;
constexpr int kFewWaves = 4, kFewThreads = kFewWaves * kWave;
constexpr int kFewMaxInputWords = 64;   // layers of up to 2048 inputs ...
constexpr int kFewMaxWords = 128, kFewMaxClasses = 32 * kFewMaxWords;   // ... and 4096 outputs

struct FewLayer {
    const uint32_t* W;          // [N][w32]
    const float *scale, *bias;  // nullptr: 1 and 0
    uint64_t* words;            // [M][LD], the last layer's [M][kFewMaxWords]: bits 31..0 a word of output bits
                                // (last layer: xcd_mark), bit 32 the mark
    int K, N, w32;
    int zero_one;               // input bits read as 0/1 instead of -1/+1
    // ceil(N / 32) blocks of 32 outputs; a wave takes one of them for f of the group's frames, so that every wave of the group has
    // at most one (parts of f frames * blocks <= 128); block and part of wave u: u - part * blocks and u * per_block >> 16
    int blocks, per_block, f;
};
struct FewArgs {
    FewLayer layer[kFewMaxLayers];
    const uint32_t* X;   // [M][layer[0].w32]
    void* Y;             // the last layer's output
    float* z;            // LOGSOFTMAX: its pre-activations, [M][z_ld]
    int layers, M, F, act, yw32, z_ld, spins;
};

typedef uint32_t u32x4g __attribute__((ext_vector_type(4)));
template <class T>
__device__ __forceinline__ __attribute__((address_space(1))) T* global_at(const void* base, uint32_t bytes) {
    typedef __attribute__((address_space(1))) char* bytes_t;
    return (__attribute__((address_space(1))) T*)((bytes_t) const_cast<void*>(base) + bytes);
}

// Log-Softmax of a row by the four waves of a workgroup, as log_softmax_rows_reg_kernel takes it (same order of additions, same
// results).  z is 8-byte aligned; what of it lies past N is not used.
__device__ __forceinline__ void few_log_softmax_row(const float* z, float* y, int N, float* red, int wave) {
    constexpr int PER = kFewMaxClasses / 256;
    const float neg_inf = -__builtin_inff();
    const int t = (int)threadIdx.x, lane = lane_id();
    float v[PER];
    asm volatile("" ::: "memory");
#pragma unroll
    for (int c = 0; c < PER; c += 2) {
        const int n = c / 4 * 1024 + 4 * t + c % 4;
        uint64_t q = 0;
        if (n < N) q = __hip_atomic_load(reinterpret_cast<const uint64_t*>(z + n), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // past the L1
        v[c] = n < N ? __uint_as_float((uint32_t)q) : neg_inf;
        v[c + 1] = n + 1 < N ? __uint_as_float((uint32_t)(q >> 32)) : neg_inf;
    }
    float mx = neg_inf;
#pragma unroll
    for (int e = 0; e < PER; ++e) mx = fmaxf(mx, v[e]);
    mx = wave_max(mx);
    if (lane == 0) red[wave] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    __syncthreads();
    float s = 0.0f;
#pragma unroll
    for (int e = 0; e < PER; ++e) s += __expf(v[e] - mx);
    s = wave_sum(s);
    if (lane == 0) red[wave] = s;
    __syncthreads();
    s = (red[0] + red[1]) + (red[2] + red[3]);
    __syncthreads();
    const float shift = mx + __logf(s);
#pragma unroll
    for (int c = 0; c < PER / 4; ++c) {
        const int n = c * 1024 + 4 * t;
        if ((N & 3) == 0 && n < N) {
            *reinterpret_cast<float4*>(y + n) = make_float4(v[4 * c] - shift, v[4 * c + 1] - shift, v[4 * c + 2] - shift, v[4 * c + 3] - shift);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (n + e < N) y[n + e] = v[4 * c + e] - shift;
        }
    }
}

// Rows of bits are kept with LD = 16 NR words, NR 16-byte pieces per lane: layers of up to 512 NR inputs.  VEC: rows are multiples of
// 16 bytes and aligned.  A wave's lanes are 16 quads; a quad takes two outputs, its lane g the pieces g, g + 4, ... of their rows.
constexpr uint64_t kFewMark = (uint64_t)1 << 32;
__device__ __forceinline__ uint64_t few_published(const uint64_t* words, uint32_t at) {   // past the L1
    return __hip_atomic_load(global_at<const uint64_t>(words, 8u * at), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void few_publish(uint64_t* words, uint32_t at, uint32_t word) {
    __hip_atomic_store(global_at<uint64_t>(words, 8u * at), kFewMark | word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
// Is this word published?  closing: of the last layer, on this XCD.
__device__ __forceinline__ bool few_there(uint64_t v, bool closing) { return closing ? v == (kFewMark | xcd_mark()) : (v & kFewMark) != 0; }
// A wave's lanes that parted meet again here, not at the next turn of a loop: there the compiler would take what a wave has one of
// (layer, pointers) for values per lane.
// The lane number, another one to the compiler each time: what follows from it is worked out where it is needed and not kept in registers.
__device__ __forceinline__ int few_fresh(int lane) {
    asm volatile("" : "+v"(lane));
    return lane;
}
__device__ __forceinline__ void few_join() { __builtin_amdgcn_wave_barrier(); }

// The weights of a block of 32 outputs: this lane's pieces of outputs n0 + 2 o and n0 + 2 o + 1 (past N: the last one again).
template <int NR, bool VEC>
struct FewWeights {
    uint4 w[2][NR];
    float scale[2], bias[2];
    __device__ __forceinline__ void request(const FewLayer& L, int n0, int lane) {
        const int w32 = L.w32, c0 = 4 * (lane & 3);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const uint32_t n = (uint32_t)min(n0 + 2 * (lane >> 2) + t, L.N - 1), r = n * (uint32_t)(4 * w32);   // (at most 4096 rows of 64 words)
#pragma unroll
            for (int p = 0; p < NR; ++p) {
                const int c = 16 * p + c0;
                auto word = [&](int i) { return *global_at<const uint32_t>(L.W, r + 4u * (uint32_t)min(i, w32 - 1)); };
                if constexpr (VEC) {
                    const u32x4g q = *global_at<const u32x4g>(L.W, r + 4u * (uint32_t)min(c, w32 - 4));
                    w[t][p] = make_uint4(q[0], q[1], q[2], q[3]);
                } else {
                    w[t][p] = make_uint4(word(c), word(c + 1), word(c + 2), word(c + 3));
                }
            }
            scale[t] = L.scale ? *global_at<const float>(L.scale, 4u * n) : 1.0f;
            bias[t] = L.bias ? *global_at<const float>(L.bias, 4u * n) : 0.0f;
        }
    }
};

// The block's outputs for nf frames from m0, whose bits are x[i LD ..].  words_out: returns the Sign bits of frame i as a word in lane
// i (outputs past N: bit 0); otherwise act of the pre-activations goes to Y[frame][Y_ld].
template <int NR, bool VEC>
__device__ __forceinline__ uint32_t few_products(FewWeights<NR, VEC>& r, const FewLayer& L, const uint32_t* x, int n0, int m0, int nf, int lane,
                                                 bool words_out, int act, float* Y, uint32_t Y_ld) {
    constexpr int LD = 16 * NR;
    const int g = lane & 3, n = n0 + 2 * (lane >> 2);
    if (L.w32 < LD) {   // pieces and words past the row count nothing
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int p = 0; p < NR; ++p) {
                const int c = 16 * p + 4 * g;
                uint4& q = r.w[t][p];
                q = make_uint4(c < L.w32 ? q.x : 0u, c + 1 < L.w32 ? q.y : 0u, c + 2 < L.w32 ? q.z : 0u, c + 3 < L.w32 ? q.w : 0u);
            }
    }
    auto quad_sum = [](int v) {
        v += __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, true);
        return v + __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, true);
    };
    int sum0[2] = {L.K, L.K}, factor = 2;   // -1/+1: K - 2 popcount(w XOR x)
    if (L.zero_one) {                       // 0/1: 2 popcount(w AND x) - popcount(x) = popcount(w) - popcount(w XOR x)
        factor = 1;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            int c = 0;
#pragma unroll
            for (int p = 0; p < NR; ++p) c += __builtin_popcount(r.w[t][p].x) + __builtin_popcount(r.w[t][p].y) + __builtin_popcount(r.w[t][p].z) + __builtin_popcount(r.w[t][p].w);
            sum0[t] = quad_sum(c);
        }
    }
    uint64_t even = 0, odd = 0;   // lane i: the Sign bits of frame i's outputs n and n + 1 of every quad
    uint4 v[NR];
    auto read = [&](int i) {
#pragma unroll
        for (int p = 0; p < NR; ++p) v[p] = *reinterpret_cast<const uint4*>(x + i * LD + 16 * p + 4 * g);
    };
    read(0);
#pragma unroll 1
    for (int i = 0;;) {
        int c[2] = {0, 0};
#pragma unroll
        for (int p = 0; p < NR; ++p)
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                c[t] += __builtin_popcount(r.w[t][p].x ^ v[p].x);
                c[t] += __builtin_popcount(r.w[t][p].y ^ v[p].y);
                c[t] += __builtin_popcount(r.w[t][p].z ^ v[p].z);
                c[t] += __builtin_popcount(r.w[t][p].w ^ v[p].w);
            }
        if (i + 1 < nf) read(i + 1);
        const float h0 = affine(r.scale[0], (float)(sum0[0] - factor * quad_sum(c[0])), r.bias[0]);
        const float h1 = affine(r.scale[1], (float)(sum0[1] - factor * quad_sum(c[1])), r.bias[1]);
        if (words_out) {
            const uint64_t b0 = __ballot(n < L.N && sign_bit(h0)), b1 = __ballot(n + 1 < L.N && sign_bit(h1));
            even = lane == i ? b0 : even;
            odd = lane == i ? b1 : odd;
        } else {   // lanes g = 0, 1 of a quad store its two
            float h = g & 1 ? h1 : h0;
            if (act == ACT_HARDTANH) h = hardtanh(h);
            if (act == ACT_SIGMOID) h = sigmoid(h);
            if (g < 2 && n + g < L.N) Y[(uint32_t)(m0 + i) * Y_ld + (uint32_t)(n + g)] = h;
        }
        if (++i >= nf) break;
    }
    uint64_t q = (even & 0x1111111111111111ull) | (odd & 0x2222222222222222ull);   // two bits of every quad's four
    q = (q | q >> 2) & 0x0F0F0F0F0F0F0F0Full;
    q = (q | q >> 4) & 0x00FF00FF00FF00FFull;
    q = (q | q >> 8) & 0x0000FFFF0000FFFFull;
    return (uint32_t)(q | q >> 16);
}

// The last layer's block b, with the weights in r.
template <int NR, bool VEC>
__device__ __forceinline__ void few_finish(FewWeights<NR, VEC>& r, const FewArgs& a, const FewLayer& L, const uint32_t* x, int b, int m0, int nf, int lane) {
    const bool lsm = a.act == ACT_LOGSOFTMAX;
    const uint32_t word = few_products(r, L, x, 32 * b, m0, nf, lane, a.act == ACT_SIGN, a.act, lsm ? a.z : static_cast<float*>(a.Y), (uint32_t)(lsm ? a.z_ld : L.N));
    if (a.act == ACT_SIGN) {
        uint32_t* out = static_cast<uint32_t*>(a.Y) + (uint32_t)(m0 + lane) * (uint32_t)a.yw32 + b;
        if (lane < nf) {
            out[0] = word;
            if (b == L.blocks - 1 && b + 1 < a.yw32) out[1] = 0u;
        }
    } else if (lsm) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // in the L2 before the mark is
        if (lane < nf) few_publish(L.words, (uint32_t)((m0 + lane) * kFewMaxWords + b), xcd_mark());
    }
    few_join();
}

// The first layer's input of nf frames.
template <int LD>
__device__ __forceinline__ void few_fill(const FewArgs& a, uint32_t* x, int m0, int nf, int lane) {
    const int w32 = a.layer[0].w32;
    for (int e = lane; e < nf * LD; e += kWave) {
        const int i = e / LD, c = e % LD;
        x[e] = c < w32 ? a.X[(uint32_t)((m0 + i) * w32 + c)] : 0u;
    }
    few_join();
}

// What a wave does that has waited long enough: the input of layer `target` (a.layers: every block of the last layer, of one frame)
// for these frames, from behind the last layer that is complete.  Blocks that are there by then are taken, the others worked out and
// published, every wave beginning at another one, so that the waves of a group share what workgroups that are not on the chip leave
// undone.  Result in x.
template <int NR, bool VEC>
__device__ __forceinline__ void few_catch_up(const FewArgs& a, int target, int m0, int nf, int wave_id, int lane_in, uint32_t* x, uint32_t* y) {
    constexpr int LD = 16 * NR;
    uint32_t *in = x, *out = y;
    uint64_t missing_lo = 0, missing_hi = 0;   // blocks of the layer that are not there
    auto look = [&](int layer, uint32_t* to) {
        const FewLayer& L = a.layer[layer];
        const int lane = few_fresh(lane_in);
        const bool closing = layer == a.layers - 1;
        const int ld = closing ? kFewMaxWords : LD, total = nf * ld;
        missing_lo = missing_hi = 0;
        for (int base = 0; base < total; base += kWave) {
            const int e = base + lane, c = e & (ld - 1);
            const bool wanted = e < total && c < L.blocks;
            uint64_t v = 0;
            if (wanted) v = few_published(L.words, (uint32_t)(m0 * ld + e));
            if (e < total) to[e] = (uint32_t)v;
            few_join();
            uint64_t not_there = __ballot(wanted && !few_there(v, closing));
            if (ld <= 32) not_there |= not_there >> 32;   // several frames in a ballot
            if (ld <= 16) not_there |= not_there >> 16;
            if (ld < 64) not_there &= ((uint64_t)1 << ld) - 1;
            if (base & (ld - 1) & 64) missing_hi |= not_there;
            else missing_lo |= not_there;
        }
        return (missing_lo | missing_hi) == 0;
    };
    int k = target - 1;
    while (k > 0 && !look(k - 1, in)) --k;
    if (k == 0) few_fill<LD>(a, in, m0, nf, few_fresh(lane_in));
    for (; k < target; ++k) {
        const FewLayer& L = a.layer[k];
        const bool closing = k == a.layers - 1;
        look(k, out);
        const int first = wave_id % L.blocks;
        for (int i = 0; i < L.blocks; ++i) {
            const int b = first + i < L.blocks ? first + i : first + i - L.blocks, lane = few_fresh(lane_in);
            if (!((b < 64 ? missing_lo >> b : missing_hi >> (b - 64)) & 1)) continue;
            uint64_t v = 0;
            if (lane < nf) v = few_published(L.words, (uint32_t)((m0 + lane) * (closing ? kFewMaxWords : LD) + b));
            if (!__all(lane >= nf || few_there(v, closing))) {
                FewWeights<NR, VEC> r;
                r.request(L, 32 * b, lane);
                if (closing) {
                    few_finish(r, a, L, in, b, m0, nf, lane);
                } else {
                    v = few_products(r, L, in, 32 * b, m0, nf, lane, true, 0, nullptr, 0u);
                    if (lane < nf) few_publish(L.words, (uint32_t)((m0 + lane) * LD + b), (uint32_t)v);
                }
            }
            if (!closing && lane < nf) out[lane * LD + b] = (uint32_t)v;
            few_join();
        }
        uint32_t* t = in;
        in = out, out = t;
    }
    if (in != x)
        for (int e = few_fresh(lane_in); e < nf * LD; e += kWave) x[e] = in[e];
    few_join();
}

// The later layers' weights into an XCD's L2, by kFewSlots workgroups, a load per 128 bytes.  Up to 1024 inputs: with 2048 the run takes
// longer with it (32 frames 22.2 -> 23.0 us a pass), and even the branch costs half a microsecond.
constexpr bool few_pulls(int NR) { return NR < 4; }
__device__ __forceinline__ void few_pull(const FewArgs& a, int slot) {
    constexpr uint32_t step = kFewSlots * kFewThreads * 128u;
    for (int j = 1; j < a.layers; ++j) {
        const uint32_t bytes = (uint32_t)a.layer[j].N * (uint32_t)a.layer[j].w32 * 4u;
        for (uint32_t at = ((uint32_t)slot * kFewThreads + threadIdx.x) * 128u; at < bytes; at += step) {
            const uint32_t t = *global_at<const uint32_t>(a.layer[j].W, at);
            asm volatile("" ::"v"(t));
        }
    }
}

// Grid: kFewGroups * kFewSlots, or twice that, where the second half pulls; kFewThreads threads, no dynamic LDS.
template <int NR, bool VEC>
__global__ __launch_bounds__(kFewThreads, 4) void few_chain_kernel(FewArgs a) {
    constexpr int LD = 16 * NR;
    __shared__ __attribute__((aligned(16))) uint32_t bits[kFewWaves][2][kFewGroupFrames * LD];   // (the second: for few_catch_up)
    __shared__ float red[kFewWaves];
    const int group = (int)blockIdx.x & (kFewGroups - 1), slot = (int)blockIdx.x / kFewGroups;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane0 = lane_id();
    const int first = group * a.F, frames = min(a.F, a.M - first);
    if (frames <= 0) return;

    if constexpr (few_pulls(NR)) {
        if (slot >= kFewSlots) return few_pull(a, slot - kFewSlots);
    }
    uint32_t *x = bits[wave][0], *y = bits[wave][1];
    const int u = wave * kFewSlots + slot;

    // The input bits of layer j (words: of the layer before, `blocks` to a row), as soon as they are there.  false: not within `spins` polls.
    auto input = [&](int j, const uint64_t* words, int blocks, int m0, int nf, int lane) -> bool {
        if (j == 0) {
            few_fill<LD>(a, x, m0, nf, lane);
            return true;
        }
        const int total = nf * LD;
        const uint64_t* from = words + (uint32_t)m0 * LD;
        int spin = 0;
        auto gather = [&](int base, auto loads) {   // `loads` of them in flight
            constexpr int B = decltype(loads)::value;
            uint64_t v[B];
            for (;; ++spin) {
                bool there = true;
#pragma unroll
                for (int i = 0; i < B; ++i) {
                    const int e = base + i * kWave + lane;
                    v[i] = kFewMark;
                    if (e < total && e % LD < blocks) v[i] = few_published(from, (uint32_t)e);
                }
#pragma unroll
                for (int i = 0; i < B; ++i) there = there && (v[i] & kFewMark);
                if (__all(there) || spin > a.spins) break;
            }
#pragma unroll
            for (int i = 0; i < B; ++i) {
                const int e = base + i * kWave + lane;
                if (e < total) x[e] = (uint32_t)v[i];
            }
            few_join();
        };
        if (total <= kWave) {
            gather(0, std::integral_constant<int, 1>{});
        } else {
            constexpr int B = NR < 4 ? 2 : 4;
            for (int base = 0; base < total && spin <= a.spins; base += B * kWave) gather(base, std::integral_constant<int, B>{});
        }
        return spin <= a.spins;   // (passed only where words were missing)
    };

    // A layer's arguments are read while the wave waits for the bits of the layer before it.
    FewLayer L = a.layer[0], next = L;
    const uint64_t* before = nullptr;   // of the layer before: its words and how many a row has
    int before_blocks = 0, j = 0;
    for (; j < a.layers - 1; ++j) {
        const int part = (u * L.per_block) >> 16, b = u - part * L.blocks, nf = min(L.f, frames - part * L.f), m0 = first + part * L.f, lane = few_fresh(lane0);
        FewWeights<NR, VEC> r;
        if (nf > 0) r.request(L, 32 * b, lane);
        next = a.layer[j + 1];
        asm volatile("" : "+s"(next.W), "+s"(next.scale), "+s"(next.bias), "+s"(next.words), "+s"(next.K), "+s"(next.N), "+s"(next.w32),
                          "+s"(next.zero_one), "+s"(next.blocks), "+s"(next.per_block), "+s"(next.f));
        if (nf > 0) {
            if (!input(j, before, before_blocks, m0, nf, lane)) break;
            const uint32_t word = few_products(r, L, x, 32 * b, m0, nf, lane, true, 0, nullptr, 0u);
            if (lane < nf) few_publish(L.words, (uint32_t)((m0 + lane) * LD + b), word);
            few_join();
        } else if (j > 0 && j < a.layers - 2) {   // no block here: on with the others (but in time for the last layer's weights)
            for (int spin = 0; spin < a.spins && !__all((few_published(before, (uint32_t)first * LD) & kFewMark) != 0); ++spin) __builtin_amdgcn_s_sleep(4);
        }
        before = L.words, before_blocks = L.blocks;
        L = next;
    }
    const int lane2 = few_fresh(lane0);
    if (j == a.layers - 1) {
        const int part = (u * L.per_block) >> 16, b = u - part * L.blocks, nf = min(L.f, frames - part * L.f), m0 = first + part * L.f;
        bool there = true;
        if (nf > 0) {
            FewWeights<NR, VEC> r;
            r.request(L, 32 * b, lane2);
            there = input(j, before, before_blocks, m0, nf, lane2);
            if (there) few_finish(r, a, L, x, b, m0, nf, lane2);
        }
        if (there) ++j;
    }
    // A wave that has waited in vain once waits no more.  (A loop of its own: its state would crowd the registers of the one above.)
    const bool in_time = j == a.layers;
    int lane3 = few_fresh(lane0);
    for (; j < a.layers; ++j) {
        const FewLayer& S = a.layer[j];
        const int part = (u * S.per_block) >> 16, b = u - part * S.blocks, nf = min(S.f, frames - part * S.f), m0 = first + part * S.f;
        if (nf <= 0) continue;
        few_catch_up<NR, VEC>(a, j, m0, nf, u, lane3, x, y);
        lane3 = few_fresh(lane3);
        FewWeights<NR, VEC> r;
        r.request(S, 32 * b, lane3);
        if (j < a.layers - 1) {
            const uint32_t word = few_products(r, S, x, 32 * b, m0, nf, lane3, true, 0, nullptr, 0u);
            if (lane3 < nf) few_publish(S.words, (uint32_t)((m0 + lane3) * LD + b), word);
            few_join();
        } else {
            few_finish(r, a, S, x, b, m0, nf, lane3);
        }
    }
    if (a.act != ACT_LOGSOFTMAX) return;
    const FewLayer& last = a.layer[a.layers - 1];
    for (int row = slot; row < frames; row += kFewSlots) {   // a workgroup per row
        const int m = first + row;
        bool there = false;
        for (int spin = 0; !there && spin <= (in_time ? a.spins : 8); ++spin) {
            const uint64_t mark = kFewMark | xcd_mark();
            uint64_t v0 = mark, v1 = mark;
            if (lane3 < last.blocks) v0 = few_published(last.words, (uint32_t)(m * kFewMaxWords + lane3));
            if (lane3 + kWave < last.blocks) v1 = few_published(last.words, (uint32_t)(m * kFewMaxWords + lane3 + kWave));
            there = __all(v0 == mark && v1 == mark);
        }
        if (!there) few_catch_up<NR, VEC>(a, a.layers, m, 1, u, lane3, x, y);
        few_log_softmax_row(a.z + (size_t)m * a.z_ld, static_cast<float*>(a.Y) + (size_t)m * last.N, last.N, red, wave);
    }
}

}  // namespace bnn
