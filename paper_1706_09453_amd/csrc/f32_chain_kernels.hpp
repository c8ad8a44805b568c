// Real-input layers whose outputs are defined by the fp32 sum in ascending k (paper Alg. 1 forward: binary weights; Sec. 3.1:
// layers that keep real weights; Alg. 1 and Alg. 2 backward: the gradient products) on the fp32 matrix cores, bit for bit:
//     acc[m][n] = fma(w[n][K-1], x[m][K-1], ... fma(w[n][1], x[m][1], fma(w[n][0], x[m][0], 0)) ...)
//
// V_MFMA_F32_16X16X4_F32 computes exactly such a chain: its four products enter the accumulator one after the other, k = 0
// (lanes 0..15) to k = 3 (lanes 48..63), each as a fused multiply-add with one rounding, denormals kept (checked against
// chains of fmaf on normal, 40-binade wide, cancelling, denormal and non-finite operands: every result identical).  So a
// kernel that feeds k in its natural order gives the bits of the vector-ALU chain at the matrix cores' rate: 153 TFLOP/s
// register to register, where an fp32 fma with three register operands reaches 110 on the vector ALU, and
// without the sign-building, address and LDS instructions that the vector ALU has to issue between its fmas.
//
// Bound: fp32 matrix-core issue (32 clocks per MFMA of 16 x 16 x 4).  Tiling: a workgroup of four waves, WR of them along
// the frames; a wave owns FM x FN accumulator fragments of 16 frames x 16 outputs.  The weights are the A operand, so a
// lane ends up with four consecutive outputs of one frame: 16-byte stores without a detour through LDS.
// K advances in chunks of KC: both operands go through LDS (two buffers, one barrier per chunk, the chunk after the next
// one on its way from memory in registers), weight bits already as +-1.0f.  Lane (r, g) needs k = 4 t + g of row r at step
// t: one LDS instruction brings the operands of two steps, and with rows KC + 4 numbers apart its 64 lanes (16 rows, four
// neighbours each) read 64 different banks.
// Measured at 4096 x 2048 x 2048: binary weights 261 us = 132 TFLOP/s, real weights 272 us (vector-ALU kernels: 331 us,
// and 290 with real weights); at 256 x 2048 x 2048 21.6 us against 72; real weights at 16 x 2048 x 2048 13.9 us against 50.
// What is left to 153 TFLOP/s (register-only loop of the same MFMA): the sign-building and LDS instructions of the staging,
// and the first and last chunk of a workgroup.
// Columns past K are stored as +0 in the frames and as -0 in real weights: fma(-0, 0, acc) adds -0, which returns every acc,
// either zero included (a sum of real products that underflow below zero is -0).  Weight bits past K stand for +-1, and
// fma(+-1, 0, acc) returns acc too: sums of +-x start at +0, cannot underflow and so are never -0.
#pragma once

#include <type_traits>

#include "bnn_device.hpp"

namespace bnn {

typedef float f32x4c __attribute__((ext_vector_type(4)));

// VEC: K % 4 == 0, X (and real weights) 16-byte aligned; otherwise element loads.  WREAL: Wv is fp32 [N][K]; otherwise
// packed bits [N][w32].  ACT: ACT_LINEAR, ACT_HARDTANH, ACT_SIGMOID or ACT_SIGN.
// SKIP: the last chunk ends behind the last group of 16 columns that K reaches; otherwise it is multiplied to its end, without
// a branch between its groups (3 % faster at 2500 x 440 x 2048, where there is nothing to leave out).
// Grid: x = tiles of TM = 16 FM WR frames, y = tiles of TN = 64 FN / WR outputs (Sign: enough for yw32 words);
// block = 256 threads; dynamic LDS = f32_chain_lds(TM, TN, KC).
constexpr unsigned f32_chain_lds(int TM, int TN, int KC) { return 2u * (unsigned)(TM + TN) * (unsigned)(KC + 4) * 4u; }

template <int FM, int FN, int WR, int KC, int ACT, bool WREAL, bool VEC, bool SKIP>
__global__ __launch_bounds__(256) void f32_chain_kernel(const float* __restrict__ X, const void* __restrict__ Wv,
                                                        const float* __restrict__ scale, const float* __restrict__ bias, int M, int K,
                                                        int N, int w32, void* __restrict__ Y, int yw32, Clear clear) {
    if constexpr (ACT == ACT_SIGN) clear_pieces<256>(clear);
    constexpr int WC = 4 / WR, TM = 16 * FM * WR, TN = 16 * FN * WC, LD = KC + 4;
    constexpr int XPR = KC / 4, WPR = WREAL ? KC / 4 : KC / 16;   // pieces per row and chunk: 4 numbers, or 16 weight bits
    constexpr int NPX = TM * XPR / 256, NPW = TN * WPR / 256;      // pieces per thread
    constexpr int NS = KC / 16;                                   // groups of four MFMA steps per chunk
    // Real weights, one dependent chain per wave: the staging is spread over the whole chunk (16 x 2048 x 2048 16.4 -> 13.9 us;
    // with weight bits, an eighth of the loads, it gains nothing: 17.6 -> 17.9)
    constexpr bool kSpread = WREAL && FM * FN == 1;
    static_assert(TM * XPR % 256 == 0 && TN * WPR % 256 == 0 && NS % 2 == 0, "whole pieces per thread");
    extern __shared__ __attribute__((aligned(16))) float chain_lds[];   // [2][TM + TN][LD]
    const int tid = (int)threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = lane_id();
    const int r = lane & 15, g = lane >> 4;
    const int m_tile = (int)blockIdx.x * TM, n_tile = (int)blockIdx.y * TN;
    const int wm = (wave / WC) * (16 * FM), wn = (wave % WC) * (16 * FN);   // the wave's place in the tile

    // ---- this thread's pieces of a chunk: piece tid + 256 j is row (.. / pieces per row), columns from (.. % pieces per row).
    // Addresses are a wave-uniform pointer that moves along K plus an offset of the thread's own (32 bits suffice for VEC).
    typedef typename std::conditional<VEC, uint32_t, size_t>::type ofs_t;
    const int xcol = 4 * (tid % XPR), wcol = WREAL ? 4 * (tid % WPR) : 16 * (tid % WPR);
    ofs_t xofs[NPX], wofs[NPW];   // bytes
#pragma unroll
    for (int j = 0; j < NPX; ++j) xofs[j] = ((ofs_t)(min(m_tile + (tid + 256 * j) / XPR, M - 1) - m_tile) * (ofs_t)K + (ofs_t)xcol) * 4;
#pragma unroll
    for (int j = 0; j < NPW; ++j) {
        const ofs_t row = (ofs_t)(min(n_tile + (tid + 256 * j) / WPR, N - 1) - n_tile);
        wofs[j] = (WREAL ? row * (ofs_t)K + (ofs_t)wcol : row * (ofs_t)w32 + (ofs_t)(wcol >> 5)) * 4;
    }
    const char* xtile = reinterpret_cast<const char*>(X + (size_t)m_tile * K);
    const char* wtile = static_cast<const char*>(Wv) + (size_t)n_tile * (WREAL ? K : w32) * 4;
    struct Loads { f32x4c x[NPX]; f32x4c w[WREAL ? NPW : 1]; uint32_t b[WREAL ? 1 : NPW]; };
    // TAIL: chunk nC - 1, which may end past K: what lies there is read from inside the row and replaced
    auto load4 = [&](const char* base, ofs_t& ofs, int k, auto tail) -> f32x4c {
        asm volatile("" : "+v"(ofs));   // keeps the offset next to its load: scalar base + lane offset, no address arithmetic
        if constexpr (VEC) {
            const int back = decltype(tail)::value ? max(k - (K - 4), 0) : 0;
            return *reinterpret_cast<const f32x4c*>(base + (ofs - (ofs_t)(4 * back)));
        } else {
            f32x4c v;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                v[i] = *reinterpret_cast<const float*>(base + (ofs + (ofs_t)(4 * i) - (ofs_t)4 * (ofs_t)(decltype(tail)::value ? max(k + i - (K - 1), 0) : 0)));
            return v;
        }
    };
    auto gload_x = [&](Loads& L, int c, int j, auto tail) { L.x[j] = load4(xtile + (size_t)c * (KC * 4), xofs[j], c * KC + xcol, tail); };
    auto gload_w = [&](Loads& L, int c, int j, auto tail) {
        if constexpr (WREAL) {
            L.w[j] = load4(wtile + (size_t)c * (KC * 4), wofs[j], c * KC + wcol, tail);
        } else {
            asm volatile("" : "+v"(wofs[j]));
            const int back = decltype(tail)::value ? max(((c * KC + wcol) >> 5) - (w32 - 1), 0) : 0;
            L.b[j] = *reinterpret_cast<const uint32_t*>(wtile + (size_t)c * (KC / 8) + (wofs[j] - (ofs_t)(4 * back)));
        }
    };
    auto gload = [&](Loads& L, int c, auto tail) {
#pragma unroll
        for (int j = 0; j < NPX; ++j) gload_x(L, c, j, tail);
#pragma unroll
        for (int j = 0; j < NPW; ++j) gload_w(L, c, j, tail);
    };
    auto clean = [&](f32x4c v, int k, float pad, auto tail) {
        if constexpr (decltype(tail)::value) {
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = k + i < K ? v[i] : pad;
        }
        return v;
    };
    auto lstore_x = [&](float* buf, const Loads& L, int c, int j, auto tail) {
        *reinterpret_cast<f32x4c*>(buf + ((tid + 256 * j) / XPR) * LD + xcol) = clean(L.x[j], c * KC + xcol, 0.0f, tail);
    };
    constexpr int WST = WREAL ? 1 : 4;   // 16-byte stores of a weight piece
    auto lstore_w = [&](float* buf, const Loads& L, int c, int j, int q, auto tail) {
        float* row = buf + (TM + (tid + 256 * j) / WPR) * LD + wcol;
        if constexpr (WREAL) {
            *reinterpret_cast<f32x4c*>(row) = clean(L.w[j], c * KC + wcol, -0.0f, tail);
        } else {   // (bits past K: +-1 times a frame value stored as 0)
            const uint32_t inv = ~L.b[j] >> (wcol & 16);
            *reinterpret_cast<f32x4c*>(row + 4 * q) = f32x4c{pm1_from_inverted_bit(inv, 4 * q), pm1_from_inverted_bit(inv, 4 * q + 1),
                                                             pm1_from_inverted_bit(inv, 4 * q + 2), pm1_from_inverted_bit(inv, 4 * q + 3)};
        }
    };
    auto lstore = [&](float* buf, const Loads& L, int c, auto tail) {
#pragma unroll
        for (int j = 0; j < NPX; ++j) lstore_x(buf, L, c, j, tail);
#pragma unroll
        for (int j = 0; j < NPW; ++j)
#pragma unroll
            for (int q = 0; q < WST; ++q) lstore_w(buf, L, c, j, q, tail);
    };
    // operands of four MFMA steps: lane (r, g) takes k = 16 s + 4 t + g of its rows (two per LDS instruction)
    struct Frags { float x[FM][4]; float w[FN][4]; };
    const int xoff = (wm + r) * LD + g, woff = (TM + wn + r) * LD + g;
    auto lread = [&](Frags& F, const float* buf, int s) {
#pragma unroll
        for (int f = 0; f < FN; ++f)
#pragma unroll
            for (int t = 0; t < 4; ++t) F.w[f][t] = buf[woff + f * 16 * LD + 16 * s + 4 * t];
#pragma unroll
        for (int f = 0; f < FM; ++f)
#pragma unroll
            for (int t = 0; t < 4; ++t) F.x[f][t] = buf[xoff + f * 16 * LD + 16 * s + 4 * t];
    };
    f32x4c acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f32x4c{0.0f, 0.0f, 0.0f, 0.0f};
    auto products = [&](const Frags& F) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int fm = 0; fm < FM; ++fm)
#pragma unroll
                for (int fn = 0; fn < FN; ++fn)
                    acc[fm][fn] = __builtin_amdgcn_mfma_f32_16x16x4f32(F.w[fn][t], F.x[fm][t], acc[fm][fn], 0, 0, 0);
    };

    const int nC = (K + KC - 1) / KC;
    constexpr int kBuf = (TM + TN) * LD;
    float* buf0 = chain_lds;
    float* buf1 = chain_lds + kBuf;
    const std::true_type yes;
    const std::false_type no;
    Loads L;
    Frags F[2];
    // One chunk, odd or even (in buf1 or buf0).  store: chunk c + 1 goes from registers to LDS (st_tail: it is the last one);
    // load: chunk c + 2 is requested (ld_tail: it is the last one).
    // Memory instructions stand between MFMAs: a wave issues in order, and a run of them would leave the matrix core idle.
    auto chunk = [&](int c, auto odd, auto store, auto st_tail, auto load, auto ld_tail) {
        float* cur = decltype(odd)::value ? buf1 : buf0;
        float* nxt = decltype(odd)::value ? buf0 : buf1;
        constexpr bool kStore = decltype(store)::value, kLoad = decltype(load)::value;
        constexpr int kReads = 2 * (FM + FN);   // LDS reads of two values each
        constexpr int kMfma = 4 * FM * FN;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            if (SKIP && !kStore && s > 0 && c * KC + 16 * s >= K) break;
            const bool turn = s == NS - 1;      // the next operands come from the next chunk
            if (turn) {
                if (!kStore) {                  // last chunk: nothing follows
                    products(F[s & 1]);
                    break;
                }
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                __builtin_amdgcn_sched_barrier(0);
                lread(F[0], nxt, 0);
            } else {
                lread(F[(s + 1) & 1], cur, s + 1);
            }
            // (nxt was last read before the previous barrier)
            if constexpr (kSpread) {
                // a share of the stores with each group of products, every piece's next load behind its last store
                constexpr int U = NPX + WST * NPW;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (u * (NS - 1) / U != s) continue;
                    const int j = u < NPX ? u : (u - NPX) / WST, q = u < NPX ? 0 : (u - NPX) % WST;
                    if (u < NPX) {
                        if constexpr (kStore) lstore_x(nxt, L, c + 1, j, st_tail);
                        if constexpr (kLoad) gload_x(L, c + 2, j, ld_tail);
                    } else {
                        if constexpr (kStore) lstore_w(nxt, L, c + 1, j, q, st_tail);
                        if constexpr (kLoad) if (q == WST - 1) gload_w(L, c + 2, j, ld_tail);
                    }
                }
                products(F[s & 1]);
                __builtin_amdgcn_sched_barrier(0);
                continue;
            }
            if (s == 0) {
                if constexpr (kStore) lstore(nxt, L, c + 1, st_tail);
                if constexpr (kLoad) gload(L, c + 2, ld_tail);
            }
            products(F[s & 1]);
            constexpr int nW = kStore ? NPX + (WREAL ? NPW : 4 * NPW) : 0, nG = kLoad ? NPX + NPW : 0;
            constexpr int q0 = kMfma / (kReads + nW + nG), q = kMfma / kReads, per0 = q0 > 1 ? q0 : 1, per = q > 1 ? q : 1;   // MFMAs behind each
            if (s == 0) {
#pragma unroll
                for (int i = 0; i < kReads; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);     // LDS read
                    __builtin_amdgcn_sched_group_barrier(0x008, per0, 0);  // MFMA
                }
#pragma unroll
                for (int i = 0; i < nW; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);     // LDS write
                    __builtin_amdgcn_sched_group_barrier(0x008, per0, 0);
                }
#pragma unroll
                for (int i = 0; i < nG; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);     // load from memory
                    __builtin_amdgcn_sched_group_barrier(0x008, per0, 0);
                }
            } else {
#pragma unroll
                for (int i = 0; i < kReads; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x008, per, 0);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    if (nC == 1) gload(L, 0, yes);
    else gload(L, 0, no);
    if (nC == 1) lstore(buf0, L, 0, yes);
    else lstore(buf0, L, 0, no);
    if (nC == 2) gload(L, 1, yes);
    else if (nC > 2) gload(L, 1, no);
    __syncthreads();
    lread(F[0], buf0, 0);
    __builtin_amdgcn_sched_barrier(0);
    int c = 0;
    for (; c + 4 < nC; c += 2) {
        chunk(c, no, yes, no, yes, no);
        chunk(c + 1, yes, yes, no, yes, no);
    }
    // one to four chunks left, the first of them even
    if (c + 3 < nC) {
        chunk(c, no, yes, no, yes, no);
        chunk(c + 1, yes, yes, no, yes, yes);
        chunk(c + 2, no, yes, yes, no, no);
        chunk(c + 3, yes, no, no, no, no);
    } else if (c + 2 < nC) {
        chunk(c, no, yes, no, yes, yes);
        chunk(c + 1, yes, yes, yes, no, no);
        chunk(c + 2, no, no, no, no, no);
    } else if (c + 1 < nC) {
        chunk(c, no, yes, yes, no, no);
        chunk(c + 1, yes, no, no, no, no);
    } else {
        chunk(c, no, no, no, no, no);
    }

    // ---- epilogue: fragment (fm, fn), register v of lane (r, g): frame m_tile + wm + 16 fm + r, output n_tile + wn + 16 fn + 4 g + v
    const bool rows_vec = (N & 3) == 0 && (reinterpret_cast<uintptr_t>(Y) & 15) == 0;
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) {
        const int n = n_tile + wn + 16 * fn + 4 * g;
        float sc[4], bi[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            sc[v] = (scale && n + v < N) ? scale[n + v] : 1.0f;
            bi[v] = (bias && n + v < N) ? bias[n + v] : 0.0f;
        }
#pragma unroll
        for (int fm = 0; fm < FM; ++fm) {
            const int m = m_tile + wm + 16 * fm + r;
            if constexpr (ACT == ACT_SIGN) {
                // four bits of this lane, joined over the lanes of the frame's 16 outputs; outputs past N: bit 0
                uint32_t bits = 0;
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    bits |= (n + v < N && sign_bit(affine(sc[v], acc[fm][fn][v], bi[v]))) ? 1u << (4 * g + v) : 0u;
                bits |= (uint32_t)__shfl_xor((int)bits, 16, kWave);
                bits |= (uint32_t)__shfl_xor((int)bits, 32, kWave);
                const int half = (n_tile + wn + 16 * fn) >> 4;   // 16-bit half of a row of words
                if (g == 0 && m < M && half < 2 * yw32) reinterpret_cast<uint16_t*>(Y)[(size_t)m * 2 * yw32 + half] = (uint16_t)bits;
            } else {
                float h[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    h[v] = affine(sc[v], acc[fm][fn][v], bi[v]);
                    if constexpr (ACT == ACT_HARDTANH) h[v] = hardtanh(h[v]);
                    if constexpr (ACT == ACT_SIGMOID) h[v] = sigmoid(h[v]);
                }
                if (m < M) {
                    float* y = static_cast<float*>(Y) + (size_t)m * N + n;
                    if (rows_vec && n + 3 < N) {
                        *reinterpret_cast<f32x4c*>(y) = f32x4c{h[0], h[1], h[2], h[3]};
                    } else {
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            if (n + v < N) y[v] = h[v];
                    }
                }
            }
        }
    }
}

}  // namespace bnn
