// A run of equal Sign layers (as many units as inputs, a multiple of 512) for a mid-size batch, one launch for all of them (paper
// Alg. 2 forward, Sec. 2.3; inside bnn_forward).
//
// Bound: latency and launches.  333 frames through a layer of 1024 units are 1 us of work for the chip, the layer's launch is 4.4 us.  As
// in few_chain_kernel.hpp the frames are split over the eight XCDs (group = blockIdx mod 8) and stay there through all layers: what
// one layer hands the next is written to and read from that XCD's L2.  A group's 32 workgroups take the layer's outputs, 16 NF each
// (N = 512 NF), its frames go to the four waves of every workgroup in fragments of 16: wave w of each workgroup makes up crew w, which
// depends on nobody else.  So there is no barrier, and a hand-over is: words stored and acknowledged, a flag per workgroup and crew
// set, the crew's 32 flags polled by one load, the frames' words loaded.  Weights do not depend on the layer before and are requested
// in front of the wait: the whole block, 16 NF rows, packed, in registers.  Products on V_MFMA_F32_16X16X128_F8F6F4 as in
// mfma_kernels.hpp; 0/1 inputs are multiplied as -1/+1 and put right by the weights' popcounts, sum hw = (sum aw + sum w) / 2.
// Nobody depends on a workgroup that is not on the chip: a wave whose wait runs out works out the missing blocks of its crew's frames
// itself, from the last complete layer on; a word has one possible value, so it does not matter who writes it.  Every layer has
// memory of its own, so a late writer disturbs no one.  The flags are cleared by the launch before.  Words and flag lie on different
// lines: in the XCD of the workgroup that wrote them the words are in the L2 before the flag is, in another one a flag may come first.
// So a flag is the number of the writer's XCD (xcd_mark) and counts on that XCD only; on another the block is worked out again, to the
// same words.  Only the speed rests on the order in which workgroups go round the XCDs.
// What bounds it where there are many frames: one wave per SIMD, which expands 16 NF rows of weights once per layer and crew, 450
// vector instructions at 2048 units, beside 64 MFMAs per fragment of frames.
// Workgroups of four waves, four of them to a CU (three at 2048 units, whose 128 frames at most leave one wave of each), for the reason in
// few_chain_kernel.hpp: with a fifth wave 256 frames of 6 x 1536 units on four streams took 19.0 us a pass, now 14.6 (one launch per layer 16.2).
#pragma once

#include "few_chain_kernel.hpp"
#include "mfma_kernels.hpp"

namespace bnn {

constexpr int kRunMaxLayers = 16, kRunCrews = 4, kRunThreads = kRunCrews * kWave;
constexpr int kRunFlags = kFewGroups * kRunCrews * kFewSlots;   // of one layer

struct RunLayer {
    const uint32_t* W;          // [N][N / 32]
    const float *scale, *bias;  // nullptr: 1 and 0
    uint32_t* Y;                // [M][N / 32]
    int zero_one;               // input bits read as 0/1 instead of -1/+1
};
struct RunArgs {
    RunLayer layer[kRunMaxLayers];
    const uint32_t* X;   // [M][N / 32]
    uint32_t* flags;     // [layers][kFewGroups][kRunCrews][kFewSlots]: 0, or the xcd_mark of who has done it
    int layers, M, F, spins;   // F: frames of a group, a multiple of 16
};

// The packed weights of a workgroup's outputs, in a lane (r, g): pieces 4 S + g of row n0 + 16 f + r.
template <int NF>
struct RunWeights {
    u32x4g w[NF][NF];
    float scale[NF], bias[NF];
    __device__ __forceinline__ void request(const RunLayer& L, int n0, int lane) {
        const uint32_t n = (uint32_t)(n0 + (lane & 15)), at = n * (64u * NF) + 16u * (uint32_t)(lane >> 4);
#pragma unroll
        for (int f = 0; f < NF; ++f) {
#pragma unroll
            for (int S = 0; S < NF; ++S) w[f][S] = *global_at<const u32x4g>(L.W, at + 1024u * (uint32_t)(NF * f) + 64u * (uint32_t)S);
            scale[f] = L.scale ? *global_at<const float>(L.scale, 4u * n + 64u * (uint32_t)f) : 1.0f;
            bias[f] = L.bias ? *global_at<const float>(L.bias, 4u * n + 64u * (uint32_t)f) : 0.0f;
        }
    }
};

// Outputs n0 .. n0 + 16 NF - 1 of a crew's frames: fragments crew, crew + 4, ... of the `frames` frames from `first`, FM at a time.
// (More than one turn with 512 units only.  But without the loop it takes 114 registers with NF = FM = 2, not 92, and with four
// launches on the chip 1000 frames of 6 x 1024 units 22.6 us a pass, not 20.4.)
template <int NF, int FM>
__device__ __forceinline__ void run_block(RunWeights<NF>& w, const RunLayer& L, const uint32_t* X, int n0, int first, int frames, int crew, int lane) {
    const int r = lane & 15, g = lane >> 4;
    const ExpandConsts ec = expand_consts();
    float factor = 1.0f, more[NF];   // dot = factor * (sum of -1/+1 products) + more
#pragma unroll
    for (int f = 0; f < NF; ++f) more[f] = 0.0f;
    if (L.zero_one) {
        factor = 0.5f;
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            int ones = 0;
#pragma unroll
            for (int S = 0; S < NF; ++S)
#pragma unroll
                for (int i = 0; i < 4; ++i) ones += __builtin_popcount(w.w[f][S][i]);
            ones += __shfl_xor(ones, 16, kWave);
            ones += __shfl_xor(ones, 32, kWave);
            more[f] = (float)(ones - 256 * NF);   // (popcount(w) - K / 2)
        }
    }
    for (int frag = crew; 16 * frag < frames; frag += kRunCrews * FM) {
        // (the weights are expanded in every turn: kept expanded they would take four times the registers)
#pragma unroll
        for (int f = 0; f < NF; ++f)
#pragma unroll
            for (int S = 0; S < NF; ++S) asm volatile("" : "+v"(w.w[f][S]));
        u32x4g a[FM][NF];
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            // (a fragment past the last one: the first again.  Never a row of another crew's: it may not be there yet, and read now it
            // would stay in the L1 as it is)
            const int at = 16 * (frag + kRunCrews * i), m_at = at < frames ? at : 16 * frag;
            const uint32_t m = (uint32_t)(first + min(m_at + r, frames - 1));
#pragma unroll
            for (int S = 0; S < NF; ++S) a[i][S] = *global_at<const u32x4g>(X, m * (64u * NF) + 64u * (uint32_t)S + 16u * (uint32_t)g);
        }
        v4f acc[FM][NF];
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int f = 0; f < NF; ++f) acc[i][f] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int S = 0; S < NF; ++S)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                v8i bx[NF];
#pragma unroll
                for (int f = 0; f < NF; ++f) bx[f] = expand_pm1_fp4(w.w[f][S][j], ec);
#pragma unroll
                for (int i = 0; i < FM; ++i) {
                    const v8i ax = expand_pm1_fp4(a[i][S][j], ec);
#pragma unroll
                    for (int f = 0; f < NF; ++f) acc[i][f] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(ax, bx[f], acc[i][f], 4, 4, 0, 0, 0, 0);
                }
            }
        // register q of lane (r, g): frame 4 g + q of the fragment, output n0 + 16 f + r; a ballot's 16 bits from 16 g are frame 4 g + q
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            uint32_t half[NF];   // lane l < 16: frame l's 16 outputs of fragment f
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                half[f] = 0;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint64_t b = __ballot(sign_bit(affine(w.scale[f], __builtin_fmaf(factor, acc[i][f][q], more[f]), w.bias[f])));
                    half[f] = (lane & 3) == q ? (uint32_t)(b >> (16 * ((lane >> 2) & 3))) & 0xFFFFu : half[f];
                }
            }
            const int m = 16 * (frag + kRunCrews * i) + lane;
            if (lane < 16 && m < frames) {
                uint32_t* y = L.Y + (uint32_t)(first + m) * (uint32_t)(16 * NF);
                if constexpr (NF == 4) {
                    *reinterpret_cast<uint2*>(y + (n0 >> 5)) = make_uint2(half[0] | half[1] << 16, half[2] | half[3] << 16);
                } else if constexpr (NF == 2) {
                    y[n0 >> 5] = half[0] | half[1] << 16;
                } else {
#pragma unroll
                    for (int f = 0; f < NF; ++f) reinterpret_cast<uint16_t*>(y)[(n0 >> 4) + f] = (uint16_t)half[f];
                }
            }
        }
    }
}

// Grid: kFewGroups * kFewSlots, kRunThreads threads.
template <int NF, int FM>
__global__ __launch_bounds__(kRunThreads, NF == 4 ? 3 : 4) void hidden_run_kernel(RunArgs a) {
    const int group = (int)blockIdx.x & (kFewGroups - 1), slot = (int)blockIdx.x / kFewGroups;
    const int crew = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    int lane = lane_id();
    const int first = group * a.F, frames = min(a.F, a.M - first);
    if (frames <= 0) return;
    if (16 * crew >= frames) return;
    const int n0 = slot * 16 * NF;
    uint32_t* const flags = a.flags + (group * kRunCrews + crew) * kFewSlots;   // + layer * kRunFlags
    auto done = [&](int layer, int who) {   // (one lane) this crew's frames through block `who` of a layer; its words are in the L2 before
        __hip_atomic_store(global_at<uint32_t>(flags, 4u * (uint32_t)(layer * kRunFlags + who)), xcd_mark(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    auto blocks_done = [&](int layer, int lane) -> uint32_t {   // a bit per block that is done on this XCD; past the L1
        uint32_t f = 0;
        if (lane < kFewSlots) f = __hip_atomic_load(global_at<const uint32_t>(flags, 4u * (uint32_t)(layer * kRunFlags + lane)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return (uint32_t)__ballot(f == xcd_mark());
    };
    RunLayer L = a.layer[0], next = L;
    const uint32_t* X = a.X;
    int j = 0;
    for (; j < a.layers; ++j) {
        RunWeights<NF> w;
        w.request(L, n0, lane);
        next = a.layer[min(j + 1, a.layers - 1)];
        asm volatile("" : "+s"(next.W), "+s"(next.scale), "+s"(next.bias), "+s"(next.Y), "+s"(next.zero_one));
        if (j > 0) {
            int spin = 0;
            while (blocks_done(j - 1, lane) != 0xFFFFFFFFu && spin <= a.spins) ++spin;
            if (__builtin_expect(spin > a.spins, 0)) break;
            asm volatile("" ::: "memory");   // the frames' words are not read earlier
        }
        run_block<NF, FM>(w, L, X, n0, first, frames, crew, lane);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (lane == 0) done(j, slot);
        few_join();
        X = L.Y;
        L = next;
    }
    // A wave that has waited in vain once waits no more: what its crew's frames lack, from behind the last complete layer on, then its own
    // blocks, one after the other.  Waves begin at different blocks and look again before each, so they share what there is to do.
    asm volatile("" : "+v"(lane));   // (nothing of this is worked out ahead of the loop above)
    for (; j < a.layers; ++j) {
        int k = j;
        while (k > 0 && blocks_done(k - 1, lane) != 0xFFFFFFFFu) --k;
        for (; k <= j; ++k) {
            const RunLayer& S = a.layer[k];
            const uint32_t* in = k > 0 ? a.layer[k - 1].Y : a.X;
            for (int i = 0; i < kFewSlots; ++i) {
                const int who = (slot + i) % kFewSlots;
                if (blocks_done(k, lane) >> who & 1) continue;
                RunWeights<NF> w;
                w.request(S, who * 16 * NF, lane);
                run_block<NF, FM>(w, S, in, who * 16 * NF, first, frames, crew, lane);
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                if (lane == 0) done(k, who);
                few_join();
            }
        }
    }
}

}  // namespace bnn
