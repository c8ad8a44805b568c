// C ABI of the gfx950 binary-network forward pass: argument checks, kernel selection, launches.
// See include/bnn.h for the contract of every entry point.
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>
#include <cstring>
#include <type_traits>

#include "../../include/bnn.h"
#include "mfma32_kernels.hpp"
#include "mfma_i8_kernels.hpp"
#include "few_chain_kernel.hpp"
#include "hidden_run_kernel.hpp"
#include "launch.hpp"
#include "realx_mfma_kernels.hpp"
#include "realw_kernels.hpp"
#include "realw_split_kernels.hpp"
#include "mfma_kernels.hpp"
#include "pack_kernels.hpp"
#include "realx_fused_kernel.hpp"
#include "realx_slab_kernels.hpp"
#include "realx_i8_gemm_kernels.hpp"
#include "softmax_kernels.hpp"
#include "train_kernels.hpp"
#include "valu_kernels.hpp"

#define BNN_EXPORT extern "C" __attribute__((visibility("default")))

// Hand-over area of the cooperative log-Softmax epilogue (BNN_OPT_COOPERATIVE): a fixed array in the library's device
// image, kCoopSlots launches' worth, handed out round-robin, so that the tail of one launch and the head of the next
// on another stream do not share a slot.  In host code the array's name is only a handle for hipGetSymbolAddress.
constexpr int kCoopSlots = 4;
constexpr int kCoopMaxTiles = 1024;                                         // workgroups of one cooperative launch, at most
constexpr size_t kCoopFlagBytes = (size_t)kCoopMaxTiles * 8;
constexpr size_t kCoopPairBytes = (size_t)kCoopMaxTiles * 256 * 8;         // 256 rows per tile, 8 bytes per (max, sum) pair
constexpr size_t kCoopSlotBytes = kCoopFlagBytes + kCoopPairBytes;
static __device__ __align__(256) unsigned char coop_area[256 + kCoopSlots * kCoopSlotBytes];   // [0, 4): timeouts

namespace {

using namespace bnn;

// Tuning knobs (bnn_set_option).  Plain atomics: set from the host thread that benchmarks.
std::atomic<int> g_default_arm{BNN_ARM_MFMA};
std::atomic<int> g_realx_tm{0};
std::atomic<int> g_binx_valu_tm{16};
std::atomic<int> g_mfma_wm{4};
std::atomic<int> g_realx_sign_mfma{1};
std::atomic<int> g_fused_softmax{0};
std::atomic<int> g_mfma_shape{0};
std::atomic<int> g_mfma32_wm{0};
std::atomic<int> g_mfma32_pipeline{0};
std::atomic<int> g_realx_f32_mfma{0};
std::atomic<int> g_mfma32_xcd_order{0};
std::atomic<int> g_stream_max_frames{64};
std::atomic<int> g_realx_i8_lsm{1};
std::atomic<int> g_realw_split_lsm{1};
std::atomic<int> g_cooperative{0};
std::atomic<int> g_coop_spin{1 << 20};

std::atomic<unsigned long long> g_coop_launches{0};
constexpr int kCoopMaxDevices = 64;
std::atomic<void*> g_coop_ptr[kCoopMaxDevices];
std::atomic<int> g_coop_capacity[kCoopMaxDevices][2];   // resident workgroups of the cooperative kernel, [0/1 input]

// Device address of coop_area on the current device (looked up once per device); *dev_out = that device.
unsigned char* coop_base(int* dev_out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kCoopMaxDevices) {
        (void)hipGetLastError();
        return nullptr;
    }
    *dev_out = dev;
    void* p = g_coop_ptr[dev].load(std::memory_order_acquire);
    if (p) return static_cast<unsigned char*>(p);
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(coop_area)) != hipSuccess || !p) {
        (void)hipGetLastError();
        return nullptr;
    }
    g_coop_ptr[dev].store(p, std::memory_order_release);
    return static_cast<unsigned char*>(p);
}

inline bool word_bits_ok(int wb) { return wb == 32 || wb == 64; }
inline int64_t words_per_row(int64_t K, int wb) { return (K + wb - 1) / wb; }
// Row length in 32-bit words (a 64-bit word is two little-endian 32-bit words).
inline int64_t row_w32(int64_t K, int wb) { return words_per_row(K, wb) * (wb / 32); }
inline bool overlap(const void* a, size_t na, const void* b, size_t nb) {
    const uintptr_t a0 = reinterpret_cast<uintptr_t>(a), b0 = reinterpret_cast<uintptr_t>(b);
    return na && nb && a0 < b0 + nb && b0 < a0 + na;
}
inline int launch_status() { return hipGetLastError() == hipSuccess ? BNN_OK : BNN_EDEVICE; }

constexpr int64_t kMaxDim = (int64_t)1 << 30;
constexpr int64_t kMaxN = (int64_t)1 << 22;   // outputs of a layer: the second grid dimension (65535) counts tiles of 128 or 256 of them

size_t out_bytes(int64_t M, int64_t N, int act, int wb) {
    if (act == BNN_ACT_SIGN) return (size_t)M * (size_t)row_w32(N, wb) * 4;
    return (size_t)M * (size_t)N * 4;
}

int check_layer_args(const void* X, const void* Wp, int64_t M, int64_t K, int64_t N, int act, int wb, const void* Y,
                     bool binx, bool realw = false) {
    if (!word_bits_ok(wb) || M < 0 || K <= 0 || N <= 0 || M > kMaxDim || K > kMaxDim || N > kMaxN) return BNN_ESHAPE;
    if (binx && K >= ((int64_t)1 << 24)) return BNN_ESHAPE;
    if (act < BNN_ACT_RAW_I32 || act > BNN_ACT_SIGMOID) return BNN_EINVAL;
    if (!binx && act == BNN_ACT_RAW_I32) return BNN_EINVAL;
    if (M == 0) return BNN_OK;
    if (!X || !Wp || !Y) return BNN_EINVAL;
    if (!aligned(Wp, realw ? 4 : wb / 8)) return BNN_EALIGN;
    if (!aligned(X, binx ? wb / 8 : 4)) return BNN_EALIGN;
    if (!aligned(Y, act == BNN_ACT_SIGN ? wb / 8 : 4)) return BNN_EALIGN;
    const size_t xb = binx ? (size_t)M * row_w32(K, wb) * 4 : (size_t)M * K * 4;
    const size_t wbytes = realw ? (size_t)N * K * 4 : (size_t)N * row_w32(K, wb) * 4;
    const size_t yb = out_bytes(M, N, act, wb);
    if (overlap(X, xb, Y, yb) || overlap(Wp, wbytes, Y, yb)) return BNN_EINVAL;
    return BNN_OK;
}

// ---------------------------------------------------------------- launches (arguments already checked)

// The comparison arm of the fp32 sums (BNN_OPT_REALX_F32_MFMA = 1), 128 frames or more, fp32 outputs.
template <int ACT, bool WREAL>
void launch_f32_mfma(const ChainArgs& a) {
    const dim3 grid((unsigned)((a.M + 255) / 256), (unsigned)((a.N + 127) / 128));
    float* Y = static_cast<float*>(a.Y);
    if (a.K % 16 == 0 && aligned(a.X, 16) && (!WREAL || aligned(a.W, 16)))
        realx_f32_mfma_kernel<ACT, true, WREAL><<<grid, 256, 0, a.st>>>(a.X, a.W, a.scale, a.bias, a.M, a.K, a.N, a.w32, Y);
    else
        realx_f32_mfma_kernel<ACT, false, WREAL><<<grid, 256, 0, a.st>>>(a.X, a.W, a.scale, a.bias, a.M, a.K, a.N, a.w32, Y);
}
// Sums of a real-input layer; arguments already checked.  few: a streaming batch, which has no comparison arm.
template <bool WREAL>
void launch_f32_sums(const ChainArgs& a, int act, bool few) {
    if (!few && act != BNN_ACT_SIGN && a.M >= 128 && g_realx_f32_mfma.load() == 1) {
        if (act == BNN_ACT_HARDTANH) launch_f32_mfma<ACT_HARDTANH, WREAL>(a);
        else if (act == BNN_ACT_SIGMOID) launch_f32_mfma<ACT_SIGMOID, WREAL>(a);
        else launch_f32_mfma<ACT_LINEAR, WREAL>(a);
    } else if (WREAL) {
        launch_chain_real(a, act);
    } else {
        launch_chain_bits(a, act);
    }
}

// What the launch in front of a run of binary layers does for it (few_chain_kernel.hpp, hidden_run_kernel.hpp): memory that it sets to
// 0, and memory that it pulls into the L2s if it can.  Whoever launches a kernel that clears sets `cleared`; without it there is no run,
// whichever kernel the options of the moment have chosen.
struct Front {
    Clear clear{};
    Pull pull{};
    bool cleared = false, pulled = false;
};
Clear clear_for(Front* front, int act) {
    if (!front || act != BNN_ACT_SIGN) return {};   // (only their Sign instances clear)
    front->cleared = true;
    return front->clear;
}

template <int TM, bool BCAST>
void launch_realx_tm_b(const float* X, const uint32_t* Wp, const float* scale, const float* bias, int M, int K, int N,
                       int w32, int act, void* Y, int yw32, hipStream_t st, Front* front) {
    dim3 grid((M + TM - 1) / TM, (N + 255) / 256), block(256);
    if constexpr (TM == 1) {   // (what batches of a few frames take)
        if (front && act == BNN_ACT_SIGN) {
            const Clear clear = cleared_by(clear_for(front, act), grid);
            if (front->pull.layers > 0) grid.y += (8 * kPullGroups + grid.x - 1) / grid.x;
            front->pulled = true;
            realx_valu_kernel<TM, ACT_SIGN, BCAST, Clear, Pull><<<grid, block, 0, st>>>(X, Wp, scale, bias, M, K, N, w32, Y, yw32, clear, front->pull);
            return;
        }
    }
    switch (act) {
        case BNN_ACT_SIGN:
            realx_valu_kernel<TM, ACT_SIGN, BCAST><<<grid, block, 0, st>>>(X, Wp, scale, bias, M, K, N, w32, Y, yw32);
            break;
        case BNN_ACT_HARDTANH:
            realx_valu_kernel<TM, ACT_HARDTANH, BCAST><<<grid, block, 0, st>>>(X, Wp, scale, bias, M, K, N, w32, Y, yw32);
            break;
        case BNN_ACT_SIGMOID:
            realx_valu_kernel<TM, ACT_SIGMOID, BCAST><<<grid, block, 0, st>>>(X, Wp, scale, bias, M, K, N, w32, Y, yw32);
            break;
        default:
            realx_valu_kernel<TM, ACT_LINEAR, BCAST><<<grid, block, 0, st>>>(X, Wp, scale, bias, M, K, N, w32, Y, yw32);
            break;
    }
}

// the row-broadcast variant reads 16 bytes of a frame per lane: rows 16-byte aligned
template <int TM>
void launch_realx_tm(const float* X, const uint32_t* Wp, const float* scale, const float* bias, int M, int K, int N,
                     int w32, int act, void* Y, int yw32, hipStream_t st, Front* front) {
    if ((K & 3) == 0 && aligned(X, 16)) launch_realx_tm_b<TM, true>(X, Wp, scale, bias, M, K, N, w32, act, Y, yw32, st, front);
    else launch_realx_tm_b<TM, false>(X, Wp, scale, bias, M, K, N, w32, act, Y, yw32, st, front);
}

void launch_log_softmax(float* Z, int M, int N, hipStream_t st) {
    const dim3 grid(M < 65536 ? M : 65536), block(256);
    const bool al = aligned(Z, 16);
    if (al && N <= 1024) log_softmax_rows_reg_kernel<4><<<grid, block, 0, st>>>(Z, M, N);
    else if (al && N <= 2048) log_softmax_rows_reg_kernel<8><<<grid, block, 0, st>>>(Z, M, N);
    else if (al && N <= 4096) log_softmax_rows_reg_kernel<16><<<grid, block, 0, st>>>(Z, M, N);
    else if (al && N <= 8192) log_softmax_rows_reg_kernel<32><<<grid, block, 0, st>>>(Z, M, N);
    else log_softmax_rows_kernel<<<grid, block, 0, st>>>(Z, M, N);
}

int run_realx(const float* X, const void* Wp, const float* scale, const float* bias, int64_t M, int64_t K, int64_t N,
              int act, int wb, void* Y, hipStream_t st, Front* front = nullptr) {
    if (M == 0) return BNN_OK;
    const int w32 = (int)row_w32(K, wb), yw32 = (int)row_w32(N, wb);
    const uint32_t* W = static_cast<const uint32_t*>(Wp);
    const bool few = M <= g_stream_max_frames.load();   // batches of a few frames (streaming): always the chains
    // Up to 16 of them on the vector ALU with one frame per workgroup: a lone wave takes 6.7 ns per k there, the chain of
    // matrix instructions 7.4 (16 x 2048 x 2048 14.5 against 15.1 us, 16 x 440 x 2048 4.8 against 5.2); rows that are no
    // multiple of 16 bytes cost the vector ALU a load per k, which only short rows hide (16 x 143 x 1000 3.7 against 3.9 us,
    // 16 x 429 x 1000 5.8 against 5.2, 16 x 2047 x 1000 20.7 against 15.0).  From 17 frames on the workgroups share the CUs and the matrix cores win (see
    // launch_chain_act).
    const bool rows_vec = (K & 3) == 0 && aligned(X, 16);
    const bool valu = M <= 16 && (K < 256 || rows_vec);
    int tm = few ? (valu ? 1 : 0) : g_realx_tm.load();
    // Rows of a few numbers that are no multiple of 16 bytes, in more tiles of 16 x 64 than the chip holds: the vector ALU with 4
    // frames per workgroup, 8 in large batches, while the bits of a row end in its first eight or little behind its first word
    // (4096 x 5 x 4096 26.7 us, 43 on the matrix cores; 4096 x 33 x 4096 30 and 45, x 39 40 and 47; but x 17 55 and 47, x 43 48
    // and 49; 1000 x 37 x 1000 5.2 us with 4 frames, 6.5 with 8, 5.8 on the matrix cores).
    if (!few && tm == 0 && !rows_vec && (K <= 8 || (K > 32 && K <= 40)) && N > 128 && ((M + 15) / 16) * ((N + 63) / 64) > 256 &&
        g_realx_f32_mfma.load() != 1)
        tm = ((M + 7) / 8) * ((N + 255) / 256) >= 2048 ? 8 : 4;
    if (tm == 0) {
        launch_f32_sums<false>({X, Wp, scale, bias, (int)M, (int)K, (int)N, w32, Y, yw32, st, clear_for(front, act)}, act, few);
        if (act == BNN_ACT_LOGSOFTMAX) launch_log_softmax(static_cast<float*>(Y), (int)M, (int)N, st);
        return launch_status();
    }
    switch (tm) {
        case 1: launch_realx_tm<1>(X, W, scale, bias, (int)M, (int)K, (int)N, w32, act, Y, yw32, st, front); break;
        case 2: launch_realx_tm<2>(X, W, scale, bias, (int)M, (int)K, (int)N, w32, act, Y, yw32, st, front); break;
        case 4: launch_realx_tm<4>(X, W, scale, bias, (int)M, (int)K, (int)N, w32, act, Y, yw32, st, front); break;
        case 8: launch_realx_tm<8>(X, W, scale, bias, (int)M, (int)K, (int)N, w32, act, Y, yw32, st, front); break;
        case 32: launch_realx_tm<32>(X, W, scale, bias, (int)M, (int)K, (int)N, w32, act, Y, yw32, st, front); break;
        default: launch_realx_tm<16>(X, W, scale, bias, (int)M, (int)K, (int)N, w32, act, Y, yw32, st, front); break;
    }
    if (act == BNN_ACT_LOGSOFTMAX) launch_log_softmax(static_cast<float*>(Y), (int)M, (int)N, st);
    return launch_status();
}

// A layer with real-valued weights.
int run_realw(const float* X, const float* W, const float* bias, int64_t M, int64_t K, int64_t N, int act, int wb,
              void* Y, hipStream_t st, Front* front = nullptr) {
    if (M == 0) return BNN_OK;
    const int yw32 = (int)row_w32(N, wb);
    const int f32_mfma = g_realx_f32_mfma.load();
    if (act == BNN_ACT_LOGSOFTMAX && f32_mfma != 2 && M <= 64 && M <= g_stream_max_frames.load() && (K & 3) == 0 &&
        aligned(X, 16) && aligned(W, 16)) {
        // a few frames in front of the log-Softmax: K split over the lanes, so that N / 4 waves pull the weights, or from 5 frames on
        // over the waves of a workgroup and the matrix cores (512 x 1000: 4 frames 6.9 and 7.7 us, 5 frames 8.8 and 8.4; 2048 x 3400: 4
        // frames 13.8 and 14.0, 5 frames 16.2 and 14.3)
        float* Yf = static_cast<float*>(Y);
        if (M <= 4) {
            realw_gemv_kernel<<<dim3((unsigned)((N + 15) / 16)), 256, 0, st>>>(X, W, bias, (int)M, (int)K, (int)N, Yf);
        } else {
            realw_frames16_kernel<<<dim3((unsigned)((N + 15) / 16), (unsigned)((M + 15) / 16)), kFrames16Threads, 0, st>>>(X, W, bias, (int)M, (int)K, (int)N, Yf);
        }
    } else {
        launch_f32_sums<true>({X, W, nullptr, bias, (int)M, (int)K, (int)N, 0, Y, yw32, st, clear_for(front, act)}, act, M <= g_stream_max_frames.load());
    }
    if (act == BNN_ACT_LOGSOFTMAX) launch_log_softmax(static_cast<float*>(Y), (int)M, (int)N, st);
    return launch_status();
}

int run_unpack(const void* Xp, int64_t M, int64_t K, int wb, int zero_one, float* X, hipStream_t st) {
    if (M == 0) return BNN_OK;
    const int64_t total = M * K;
    const int64_t blocks = (total + 255) / 256;
    bits_to_real_kernel<<<(unsigned)(blocks < 65536 ? blocks : 65536), 256, 0, st>>>(static_cast<const uint32_t*>(Xp), M, (int)K,
                                                                                     (int)row_w32(K, wb), zero_one, X);
    return launch_status();
}

template <int TM, bool VEC4, bool X01 = false>
void launch_binx_valu_tm(const uint32_t* Xp, const uint32_t* Wp, const float* scale, const float* bias, int M, int K,
                         int N, int w32, int act, void* Y, int yw32, hipStream_t st) {
    const dim3 grid((M + TM - 1) / TM, (N + 255) / 256), block(256);
    switch (act) {
        case BNN_ACT_RAW_I32:
            binx_valu_kernel<TM, ACT_RAW_I32, VEC4, X01><<<grid, block, 0, st>>>(Xp, Wp, scale, bias, M, K, N, w32, Y, yw32);
            break;
        case BNN_ACT_SIGN:
            binx_valu_kernel<TM, ACT_SIGN, VEC4, X01><<<grid, block, 0, st>>>(Xp, Wp, scale, bias, M, K, N, w32, Y, yw32);
            break;
        case BNN_ACT_HARDTANH:
            binx_valu_kernel<TM, ACT_HARDTANH, VEC4, X01><<<grid, block, 0, st>>>(Xp, Wp, scale, bias, M, K, N, w32, Y, yw32);
            break;
        case BNN_ACT_SIGMOID:
            binx_valu_kernel<TM, ACT_SIGMOID, VEC4, X01><<<grid, block, 0, st>>>(Xp, Wp, scale, bias, M, K, N, w32, Y, yw32);
            break;
        default:
            binx_valu_kernel<TM, ACT_LINEAR, VEC4, X01><<<grid, block, 0, st>>>(Xp, Wp, scale, bias, M, K, N, w32, Y, yw32);
            break;
    }
}

template <int TM, bool X01>
void launch_binx_split(const uint32_t* Xp, const uint32_t* Wp, const float* scale, const float* bias, int M, int K, int N,
                       int w32, int act, void* Y, int yw32, hipStream_t st) {
    const dim3 grid((M + TM - 1) / TM, (N + 63) / 64), block(256);
    switch (act) {
        case BNN_ACT_RAW_I32: binx_split_kernel<TM, ACT_RAW_I32, X01><<<grid, block, 0, st>>>(Xp, Wp, scale, bias, M, K, N, w32, Y, yw32); break;
        case BNN_ACT_SIGN: binx_split_kernel<TM, ACT_SIGN, X01><<<grid, block, 0, st>>>(Xp, Wp, scale, bias, M, K, N, w32, Y, yw32); break;
        case BNN_ACT_HARDTANH: binx_split_kernel<TM, ACT_HARDTANH, X01><<<grid, block, 0, st>>>(Xp, Wp, scale, bias, M, K, N, w32, Y, yw32); break;
        case BNN_ACT_SIGMOID: binx_split_kernel<TM, ACT_SIGMOID, X01><<<grid, block, 0, st>>>(Xp, Wp, scale, bias, M, K, N, w32, Y, yw32); break;
        default: binx_split_kernel<TM, ACT_LINEAR, X01><<<grid, block, 0, st>>>(Xp, Wp, scale, bias, M, K, N, w32, Y, yw32); break;
    }
}

template <int WM, bool AL, bool X01>
void launch_binx_mfma_wm(const uint32_t* Xp, const uint32_t* Wp, const float* scale, const float* bias, int M, int K,
                         int N, int w32, int act, void* Y, int yw32, hipStream_t st) {
    constexpr int WN = 4;
    const dim3 grid((M + 32 * WM - 1) / (32 * WM), (N + 32 * WN - 1) / (32 * WN)), block(256);
    switch (act) {
        case BNN_ACT_RAW_I32:
            binx_mfma_kernel<WM, WN, ACT_RAW_I32, AL, X01><<<grid, block, 0, st>>>(Xp, Wp, scale, bias, M, K, N, w32, Y, yw32);
            break;
        case BNN_ACT_SIGN:
            binx_mfma_kernel<WM, WN, ACT_SIGN, AL, X01><<<grid, block, 0, st>>>(Xp, Wp, scale, bias, M, K, N, w32, Y, yw32);
            break;
        case BNN_ACT_HARDTANH:
            binx_mfma_kernel<WM, WN, ACT_HARDTANH, AL, X01><<<grid, block, 0, st>>>(Xp, Wp, scale, bias, M, K, N, w32, Y, yw32);
            break;
        case BNN_ACT_SIGMOID:
            binx_mfma_kernel<WM, WN, ACT_SIGMOID, AL, X01><<<grid, block, 0, st>>>(Xp, Wp, scale, bias, M, K, N, w32, Y, yw32);
            break;
        default:
            binx_mfma_kernel<WM, WN, ACT_LINEAR, AL, X01><<<grid, block, 0, st>>>(Xp, Wp, scale, bias, M, K, N, w32, Y, yw32);
            break;
    }
}

template <int WM, bool AL, bool PP = false, bool X01 = false>
void launch_binx_mfma32(const uint32_t* Xp, const uint32_t* Wp, const float* scale, const float* bias, int M, int K, int N,
                        int w32, int act, void* Y, int yw32, hipStream_t st, const CoopLsm& coop = CoopLsm{}) {
    constexpr int WN = 2;
    // XCD-aware tile order pays when the default order thrashes the per-XCD L2s (a frames operand of more than
    // 8 x 4 MiB) or scatters a large packed output with long rows over many passes; it costs 5-15 % on mid-size
    // problems (measured on MI355X), so it is chosen by size unless forced.
    const int xsel = g_mfma32_xcd_order.load();
    const int xo = xsel == 1 || (xsel == 0 && ((size_t)M * w32 * 4 > ((size_t)32 << 20) ||
                                              (N >= 4096 && (size_t)M * N / 8 >= ((size_t)32 << 20))));
    const unsigned int ab = (unsigned int)((size_t)M * w32 * 4), bb = (unsigned int)((size_t)N * w32 * 4);   // used by the PP variants only
    const dim3 grid((M + 64 * WM - 1) / (64 * WM), (N + 64 * WN - 1) / (64 * WN)), block(256);
    auto go = [&](auto actc) {
        constexpr int ACT = decltype(actc)::value;
        constexpr unsigned lds = m32_lds(WM, WN, ACT, PP);
        if constexpr (lds > 65536) {
            static std::atomic<uint64_t> allowed{0};
            (void)allow_lds(&binx_mfma32_kernel<WM, WN, ACT, AL, PP, X01>, lds, allowed);   // (refused: the launch fails)
        }
        binx_mfma32_kernel<WM, WN, ACT, AL, PP, X01><<<grid, block, lds, st>>>(Xp, Wp, scale, bias, M, K, N, w32, Y, yw32, ab, bb, xo, coop);
    };
    switch (act) {
        case ACT_LSM_COOP:
            if constexpr (WM == 4 && AL && PP) go(std::integral_constant<int, ACT_LSM_COOP>{});
            break;
        case ACT_DOT_I16: go(std::integral_constant<int, ACT_DOT_I16>{}); break;
        case BNN_ACT_RAW_I32: go(std::integral_constant<int, ACT_RAW_I32>{}); break;
        case BNN_ACT_SIGN: go(std::integral_constant<int, ACT_SIGN>{}); break;
        case BNN_ACT_HARDTANH: go(std::integral_constant<int, ACT_HARDTANH>{}); break;
        case BNN_ACT_SIGMOID: go(std::integral_constant<int, ACT_SIGMOID>{}); break;
        default: go(std::integral_constant<int, ACT_LINEAR>{}); break;
    }
}

template <bool AL>
void launch_binx_mfma_i8(const uint32_t* Xp, const uint32_t* Wp, const float* scale, const float* bias, int M, int K, int N,
                         int w32, int act, void* Y, int yw32, hipStream_t st) {
    const dim3 grid((M + 127) / 128, (N + 127) / 128), block(256);
    switch (act) {
        case BNN_ACT_RAW_I32:
            binx_mfma_i8_kernel<ACT_RAW_I32, AL><<<grid, block, 0, st>>>(Xp, Wp, scale, bias, M, K, N, w32, Y, yw32);
            break;
        case BNN_ACT_SIGN:
            binx_mfma_i8_kernel<ACT_SIGN, AL><<<grid, block, 0, st>>>(Xp, Wp, scale, bias, M, K, N, w32, Y, yw32);
            break;
        case BNN_ACT_HARDTANH:
            binx_mfma_i8_kernel<ACT_HARDTANH, AL><<<grid, block, 0, st>>>(Xp, Wp, scale, bias, M, K, N, w32, Y, yw32);
            break;
        case BNN_ACT_SIGMOID:
            binx_mfma_i8_kernel<ACT_SIGMOID, AL><<<grid, block, 0, st>>>(Xp, Wp, scale, bias, M, K, N, w32, Y, yw32);
            break;
        default:
            binx_mfma_i8_kernel<ACT_LINEAR, AL><<<grid, block, 0, st>>>(Xp, Wp, scale, bias, M, K, N, w32, Y, yw32);
            break;
    }
}

int run_binx(const void* Xp, const void* Wp, const float* scale, const float* bias, int64_t M, int64_t K, int64_t N,
             int act, int wb, void* Y, int arm, hipStream_t st, bool x01 = false) {
    if (M == 0) return BNN_OK;
    // wide layers leave the vector-ALU kernel from where its workgroups no longer fit the chip at once: 64 frames of
    // 4096 x 4096 took 12.0 us there, 7.7 on the matrix cores (64 x 2048 x 2048, 256 workgroups: 5.1 against 5.4)
    const bool stream = arm == BNN_ARM_AUTO && M <= g_stream_max_frames.load() &&
                        (K < 2048 || ((M + 1) / 2) * ((N + 255) / 256) <= 256 || g_default_arm.load() != BNN_ARM_MFMA);
    if (arm == BNN_ARM_AUTO) arm = g_default_arm.load();
    if (x01) arm = BNN_ARM_MFMA;   // larger batches: the 0/1 reading of the input bits exists on the fp4 matrix-core kernels only
    const int w32 = (int)row_w32(K, wb), yw32 = (int)row_w32(N, wb);
    const uint32_t* A = static_cast<const uint32_t*>(Xp);
    const uint32_t* B = static_cast<const uint32_t*>(Wp);
    const bool rows16 = (w32 % 4 == 0) && aligned(Xp, 16) && aligned(Wp, 16);
    const int Mi = (int)M, Ki = (int)K, Ni = (int)N;
    // The 16x16x128 kernel with 16 x 64 wave tiles (32 x 128 per workgroup) while its grid fits the 256 CUs once: a layer
    // then lasts about one memory round trip plus a short epilogue, where larger tiles leave most CUs idle.  Measured
    // (Sign, K = N): 333 x 1024 4.4 us (64-row tiles of the same kernel 8.5, 64-row tiles of the 32x32x64 kernel 6.4),
    // 100 x 2048 5.5 (10.7, 6.8), 1000 x 512 3.6 (6.3, 4.0); with more than 256 tiles the 32x32x64 kernel is the faster
    // one: 600 x 2048 8.2 against 7.4, 1000 x 4096 23.2 against 12.2.
    const int64_t tiles1 = ((M + 31) / 32) * ((N + 127) / 128);
    const int mfma_shape = g_mfma_shape.load();
    // Output layer on the 32x32x64 kernel: the product goes to memory as int16 (half the bytes of fp32 pre-activations), and
    // the row kernel forms fma(scale, dot, bias) itself before the log-Softmax.
    const bool i16 = act == BNN_ACT_LOGSOFTMAX && K < 32768 && N % 4 == 0 && N <= 8192 && aligned(Y, 16) &&
                     (!scale || aligned(scale, 16)) && (!bias || aligned(bias, 16));
    // Exceptions to the line at 256 tiles.  An output layer whose product is short gains more from the int16 hand-over than from
    // the smaller tiles (K = 512: 1024 x 1000 outputs 8.8 us against 9.8, 1024 x 64 6.9 and 7.3; K = 1024: 1000 x 1000 9.9 and
    // 10.6, but 512 x 512 8.1 and 7.8, 200 x 4096 10.8 and 9.9; K = 2048: 1000 x 512 9.7 and 8.9).  Integer dot products of
    // fewer than 1024 frames whose rows are read word by word leave the 32x32x64 kernel more slowly than 64-row tiles of the
    // 16x16x128 kernel (1000 x 64 x 3400 8.5 us and 7.5, x 700 11.1 and 10.3).
    const bool al512 = rows16 && K % 512 == 0;
    const bool short_lsm = i16 && al512 && M >= 512 && (K <= 512 || (K <= 1024 && tiles1 > 128));
    const bool few_raw = act == BNN_ACT_RAW_I32 && !x01 && !al512 && M < 1024 && K < 1024 && tiles1 > 256;
    if (stream) {
        // Batches of a few frames (streaming): the matrix-core tiles would be nearly empty and a workgroup would
        // still walk all of K for its 64 or 128 rows.  The vector-ALU kernels with 1 or 2 frames per workgroup spread
        // the layer over the chip, and each workgroup is done after one pass over its weight rows.  K split over four lanes
        // while its workgroups fit the chip twice (one frame through six layers of 2048 units 33.8 -> 29.3 us a pass, 0.7 us a
        // layer; one layer of 1 x 4096 x 4096 launched back to back 5.9 -> 3.7 to 5.7 from run to run); with more of them
        // every lane's own row is as good or better (16 x 4096 x 4096 6.0 against 6.2, 32 x 4096 x 4096 6.1 against 7.3).
        const int tm = M <= 16 ? 1 : 2;
        const bool split = rows16 && ((M + tm - 1) / tm) * ((N + 63) / 64) <= 512;
        auto go = [&](auto tmc, auto z1) {
            constexpr int TM = decltype(tmc)::value;
            constexpr bool Z1 = decltype(z1)::value;
            if (split) launch_binx_split<TM, Z1>(A, B, scale, bias, Mi, Ki, Ni, w32, act, Y, yw32, st);
            else if (rows16) launch_binx_valu_tm<TM, true, Z1>(A, B, scale, bias, Mi, Ki, Ni, w32, act, Y, yw32, st);
            else launch_binx_valu_tm<TM, false, Z1>(A, B, scale, bias, Mi, Ki, Ni, w32, act, Y, yw32, st);
        };
        using I1 = std::integral_constant<int, 1>;
        using I2 = std::integral_constant<int, 2>;
        if (x01) { if (tm == 1) go(I1{}, std::true_type{}); else go(I2{}, std::true_type{}); }
        else { if (tm == 1) go(I1{}, std::false_type{}); else go(I2{}, std::false_type{}); }
    } else if (arm == BNN_ARM_VALU_XOR) {
        const int tm = g_binx_valu_tm.load();
        if (rows16) {
            if (tm == 1) launch_binx_valu_tm<1, true>(A, B, scale, bias, Mi, Ki, Ni, w32, act, Y, yw32, st);
            else if (tm == 2) launch_binx_valu_tm<2, true>(A, B, scale, bias, Mi, Ki, Ni, w32, act, Y, yw32, st);
            else if (tm == 4) launch_binx_valu_tm<4, true>(A, B, scale, bias, Mi, Ki, Ni, w32, act, Y, yw32, st);
            else if (tm == 8) launch_binx_valu_tm<8, true>(A, B, scale, bias, Mi, Ki, Ni, w32, act, Y, yw32, st);
            else if (tm == 32) launch_binx_valu_tm<32, true>(A, B, scale, bias, Mi, Ki, Ni, w32, act, Y, yw32, st);
            else launch_binx_valu_tm<16, true>(A, B, scale, bias, Mi, Ki, Ni, w32, act, Y, yw32, st);
        } else {
            if (tm == 8) launch_binx_valu_tm<8, false>(A, B, scale, bias, Mi, Ki, Ni, w32, act, Y, yw32, st);
            else if (tm == 32) launch_binx_valu_tm<32, false>(A, B, scale, bias, Mi, Ki, Ni, w32, act, Y, yw32, st);
            else launch_binx_valu_tm<16, false>(A, B, scale, bias, Mi, Ki, Ni, w32, act, Y, yw32, st);
        }
    } else if (arm == BNN_ARM_MFMA_I8) {
        if (rows16 && K % 512 == 0) launch_binx_mfma_i8<true>(A, B, scale, bias, Mi, Ki, Ni, w32, act, Y, yw32, st);
        else launch_binx_mfma_i8<false>(A, B, scale, bias, Mi, Ki, Ni, w32, act, Y, yw32, st);
    } else if (!x01 && act == BNN_ACT_LOGSOFTMAX && g_fused_softmax.load() && rows16 &&
               ((K % 512 == 0 && N <= 16 * 8 * 16) || (K % 256 == 0 && N <= 16 * 8 * 32)) &&
               (size_t)(M + 16) * w32 * 4 < 0x7fffffffu && (size_t)(N + 512) * w32 * 4 < 0x7fffffffu) {
        // output layer: product, affine step and log-Softmax fused, one workgroup per 16 frames
        const int nf = (int)((N + 127) / 128);
        const dim3 grid((Mi + 15) / 16), block(512);
        float* Yf = static_cast<float*>(Y);
        const unsigned int ab = (unsigned int)((size_t)M * w32 * 4), bb = (unsigned int)((size_t)N * w32 * 4);
        if (K % 512 == 0 && nf <= 8)
            binx_mfma_logsoftmax_kernel<8, 4><<<grid, block, 0, st>>>(A, B, scale, bias, Mi, Ki, Ni, w32, Yf, ab, bb);
        else if (K % 512 == 0 && nf <= 16)
            binx_mfma_logsoftmax_kernel<16, 4><<<grid, block, 0, st>>>(A, B, scale, bias, Mi, Ki, Ni, w32, Yf, ab, bb);
        else if (nf <= 28)
            binx_mfma_logsoftmax_kernel<28, 2><<<grid, block, 0, st>>>(A, B, scale, bias, Mi, Ki, Ni, w32, Yf, ab, bb);
        else
            binx_mfma_logsoftmax_kernel<32, 2><<<grid, block, 0, st>>>(A, B, scale, bias, Mi, Ki, Ni, w32, Yf, ab, bb);
        return launch_status();
    } else if (mfma_shape == 32 || (x01 && mfma_shape == 16) || (mfma_shape == 0 && (tiles1 > 256 || short_lsm) && !few_raw)) {
        // large batch: 32x32x64 MFMA, 128 x 64 (or 64 x 64) wave tiles
        const bool al = rows16 && (K % 512 == 0);
        if (i16) act = ACT_DOT_I16;
        const int64_t tiles_n4 = (N + 127) / 128, tiles4 = ((M + 255) / 256) * tiles_n4;
        // fetch through LDS, order pinned: 16384 x 4096 x 4096 95 us against 124 from memory to registers, 4096 x 2048 x 2048 9.3
        // and 10.5, 600 x 2048 x 2048 5.8 and 9.2.  Buffer addressing needs operands below 2 GiB, exact sums of 0/1 products and
        // counts in fp32 K < 2^22
        const bool pinned = g_mfma32_pipeline.load() != 2 && K < (1 << 22) && (size_t)M * w32 * 4 < 0x7fffffffu && (size_t)N * w32 * 4 < 0x7fffffffu;
        const bool lsm = act == BNN_ACT_LOGSOFTMAX || act == ACT_DOT_I16, coop_asked = lsm && g_cooperative.load();
        // 128-row wave tiles expand fewer operand words per MAC; 64-row ones give twice the workgroups, which
        // matters more while the 128-row grid leaves CUs without a workgroup (measured on MI355X: 64-row tiles win
        // up to 2048 frames x 2048 outputs, 128-row tiles from 4096 x 2048 on).  With a single stage of K a workgroup is mostly
        // its start and its end, and three 64-row ones on a CU cover each other better than two 128-row ones, unless the 128-row
        // ones are done in one round and the others are not (128 and 64 rows, K = 512: 9247 x 3808 16.9 and 15.1 us, 4998 x 4864 11.1
        // and 9.5, 5000 x 2048 6.5 and 5.5, 16384 x 3000 17.2 and 16.8; but 1798 x 6816 6.8 and 8.0, 6373 x 2554 8.1 and 8.4; K = 1024:
        // 11789 x 4410 25.7 and 26.1, 8192 x 2048 9.0 and 9.2).
        const int64_t blocks4 = ((M + 255) / 256) * ((N + 127) / 128), blocks2 = ((M + 127) / 128) * ((N + 127) / 128);
        const int wm32 = g_mfma32_wm.load();
        const bool one_stage = K == 512 && pinned && !coop_asked && (blocks4 > 512 || blocks2 <= 768);
        const bool wm2 = wm32 == 2 || (wm32 == 0 && (blocks4 < 200 || one_stage));
        // Cooperative log-Softmax (opt-in): the product kernel finishes the rows itself.  Its workgroups wait for each
        // other, so all of them have to be resident at once.
        CoopLsm coop{};
        if (coop_asked && al && pinned && !wm2 && tiles_n4 <= 64 &&
            tiles4 <= kCoopMaxTiles) {
            int dev = -1;
            unsigned char* base = coop_base(&dev);
            int cap = base ? g_coop_capacity[dev][x01 ? 1 : 0].load() : 0;
            if (base && cap == 0) {
                int per_cu = 0, cus = 0;
                const hipError_t e1 = x01 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, binx_mfma32_kernel<4, 2, ACT_LSM_COOP, true, true, true>, 256, m32_lds(4, 2, ACT_LSM_COOP, true))
                                          : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, binx_mfma32_kernel<4, 2, ACT_LSM_COOP, true, true, false>, 256, m32_lds(4, 2, ACT_LSM_COOP, true));
                const hipError_t e2 = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
                if (e1 != hipSuccess || e2 != hipSuccess) (void)hipGetLastError();
                cap = (e1 == hipSuccess && e2 == hipSuccess && per_cu > 0 && cus > 0) ? per_cu * cus : -1;
                g_coop_capacity[dev][x01 ? 1 : 0].store(cap);
            }
            if (base && tiles4 <= cap) {
                const unsigned long long launch = ++g_coop_launches;
                unsigned char* slot = base + 256 + (size_t)(launch % kCoopSlots) * kCoopSlotBytes;
                coop.flags = reinterpret_cast<unsigned long long*>(slot);
                coop.partials = reinterpret_cast<float2*>(slot + kCoopFlagBytes);
                coop.stamp = launch;
                coop.timeouts = reinterpret_cast<unsigned int*>(base);
                coop.spin_limit = g_coop_spin.load();
                act = ACT_LSM_COOP;
            }
        }
        if (x01) {
            if (!al) launch_binx_mfma32<2, false, false, true>(A, B, scale, bias, Mi, Ki, Ni, w32, act, Y, yw32, st);
            else if (!pinned) launch_binx_mfma32<2, true, false, true>(A, B, scale, bias, Mi, Ki, Ni, w32, act, Y, yw32, st);   // operands of 2 GiB or more
            else if (wm2) launch_binx_mfma32<2, true, true, true>(A, B, scale, bias, Mi, Ki, Ni, w32, act, Y, yw32, st);
            else launch_binx_mfma32<4, true, true, true>(A, B, scale, bias, Mi, Ki, Ni, w32, act, Y, yw32, st, coop);
        } else if (!al) {
            // ragged rows: bounds-checked word loads, 64-row wave tiles only
            launch_binx_mfma32<2, false>(A, B, scale, bias, Mi, Ki, Ni, w32, act, Y, yw32, st);
        } else if (wm2) {
            if (pinned) launch_binx_mfma32<2, true, true>(A, B, scale, bias, Mi, Ki, Ni, w32, act, Y, yw32, st);
            else launch_binx_mfma32<2, true>(A, B, scale, bias, Mi, Ki, Ni, w32, act, Y, yw32, st);
        } else {
            if (pinned) launch_binx_mfma32<4, true, true>(A, B, scale, bias, Mi, Ki, Ni, w32, act, Y, yw32, st, coop);
            else launch_binx_mfma32<4, true>(A, B, scale, bias, Mi, Ki, Ni, w32, act, Y, yw32, st);
        }
    } else {
        const bool al = rows16 && w32 % 16 == 0;   // whole super-steps of 512 bits, the pad bits among them
        const int wm = g_mfma_wm.load();
        auto go = [&](auto wmc, auto alc, auto z1) {
            launch_binx_mfma_wm<decltype(wmc)::value, decltype(alc)::value, decltype(z1)::value>(A, B, scale, bias, Mi, Ki, Ni, w32, act, Y, yw32, st);
        };
        using WM1 = std::integral_constant<int, 1>;
        using WM2 = std::integral_constant<int, 2>;
        using WM4 = std::integral_constant<int, 4>;
        const std::true_type yes;
        const std::false_type no;
        if (x01) { if (al) go(WM1{}, yes, yes); else go(WM1{}, no, yes); }
        else if (mfma_shape == 0 && !few_raw) { if (al) go(WM1{}, yes, no); else go(WM1{}, no, no); }
        else if (mfma_shape != 0 && wm == 2) { if (al) go(WM2{}, yes, no); else go(WM2{}, no, no); }
        else { if (al) go(WM4{}, yes, no); else go(WM4{}, no, no); }
    }
    if (act == BNN_ACT_LOGSOFTMAX) launch_log_softmax(static_cast<float*>(Y), Mi, Ni, st);
    if (act == ACT_DOT_I16) {
        constexpr int ROWS = 1;   // two rows per workgroup (shared scale/bias loads) measured slower
        const int nblk = (Mi + ROWS - 1) / ROWS;
        const dim3 grid(nblk < 65536 ? nblk : 65536), block(256);
        float* Z = static_cast<float*>(Y);
        if (Ni <= 1024) log_softmax_rows_i16_kernel<4, ROWS><<<grid, block, 0, st>>>(Z, scale, bias, Mi, Ni);
        else if (Ni <= 2048) log_softmax_rows_i16_kernel<8, ROWS><<<grid, block, 0, st>>>(Z, scale, bias, Mi, Ni);
        else if (Ni <= 4096) log_softmax_rows_i16_kernel<16, ROWS><<<grid, block, 0, st>>>(Z, scale, bias, Mi, Ni);
        else log_softmax_rows_i16_kernel<32, ROWS><<<grid, block, 0, st>>>(Z, scale, bias, Mi, Ni);
    }
    return launch_status();
}

int run_pack(const float* X, int64_t rows, int64_t K, int wb, void* out, hipStream_t st) {
    if (rows == 0) return BNN_OK;
    uint32_t* words = static_cast<uint32_t*>(out);
    auto go = [&](auto ballots) {
        constexpr int B = decltype(ballots)::value;
        const int64_t tasks = rows * ((K + 64 * B - 1) / (64 * B));
        int64_t blocks = (tasks + 3) / 4;
        if (blocks > 65536 * 4) blocks = 65536 * 4;
        pack_sign_kernel<B><<<dim3((unsigned)blocks), dim3(256), 0, st>>>(X, rows, K, row_w32(K, wb), words);
    };
    if (K <= 64) go(std::integral_constant<int, 1>{});
    else if (K <= 128) go(std::integral_constant<int, 2>{});
    else if (K <= 256) go(std::integral_constant<int, 4>{});
    else go(std::integral_constant<int, 8>{});
    return launch_status();
}

size_t round_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// The matrix-core path of a real-input Sign layer (first layer of a binary-activation network) applies when
// K is small enough for its integer arithmetic; it needs no scratch in global memory.
bool realx_sign_mfma_applies(const bnn_layer_desc& d) {
    return !d.x_is_binary && d.act == BNN_ACT_SIGN && d.K <= kRealxMfmaMaxK;
}

int run_realx_sign_mfma(const float* X, const void* Wp, const float* scale, const float* bias, int64_t M, int64_t K,
                        int64_t N, int wb, void* Y, hipStream_t st, Front* front) {
    const int Mi = (int)M, Ki = (int)K, Ni = (int)N;
    const int w32 = (int)row_w32(K, wb), yw32 = (int)row_w32(N, wb);
    const int kpad = (Ki + 63) / 64 * 64;
    // Outputs per workgroup.  A workgroup costs about 11 us (frames in, digits, the undecided outputs) and 4 us per 512
    // outputs, and a CU holds one at a time, so the outputs are split as far as that shortens the longest CU's work:
    // measured at 440 x 2048, 333 frames 27.7 us with all outputs in one workgroup, 15.5 with 512; 1500 frames 27.5 and
    // 19.4 (1024); 4096 frames 28.2 unsplit, 37.1 with 1024, 55.6 with 512.  (Rows of up to about 300 numbers leave LDS for
    // two or three workgroups per CU, which the rule does not count; of K = 16 to 520, 64 to 4096 outputs and 65 to 16384
    // frames no size measured slower than with all outputs in one workgroup.)
    const int chunks = min((Ni + kRealxChunk - 1) / kRealxChunk, kRealxMaxNB / kRealxChunk);
    const int64_t mt = (M + kRealxBM - 1) / kRealxBM;
    int nb = 0;
    double best = 0.0;
    for (int c = chunks; c >= 1; --c) {
        const int64_t wgs = mt * ((Ni + c * kRealxChunk - 1) / (c * kRealxChunk));
        const double cost = (double)((wgs + 255) / 256) * (11.0 + 4.1 * c);
        if (nb == 0 || cost < best) best = cost, nb = c * kRealxChunk;
    }
    const size_t lds = realx_dynamic_lds(Ki, kpad, w32, nb);
    const dim3 grid((Mi + kRealxBM - 1) / kRealxBM, (Ni + nb - 1) / nb), block(kRealxThreads);
    // (the LDS of a launch depends on nb, and so on the batch; what is allowed covers every K and nb)
    static std::atomic<uint64_t> allowed[2];
    constexpr unsigned most = (unsigned)realx_dynamic_lds(kRealxMfmaMaxK, (kRealxMfmaMaxK + 63) / 64 * 64, (kRealxMfmaMaxK + 63) / 64 * 2, kRealxMaxNB);
    const bool vec16 = aligned(Wp, 16);   // chunks start at multiples of 512 rows: 16-byte aligned whenever the matrix is
    if (!allow_lds(vec16 ? &realx_sign_fused_kernel<true> : &realx_sign_fused_kernel<false>, most, allowed[vec16])) return BNN_EDEVICE;
    const Clear clear = cleared_by(clear_for(front, BNN_ACT_SIGN), grid);
    if (vec16)
        realx_sign_fused_kernel<true><<<grid, block, lds, st>>>(X, static_cast<const uint32_t*>(Wp), scale, bias, Mi, Ki, kpad,
                                                               Ni, nb, w32, static_cast<uint32_t*>(Y), yw32, clear);
    else
        realx_sign_fused_kernel<false><<<grid, block, lds, st>>>(X, static_cast<const uint32_t*>(Wp), scale, bias, Mi, Ki, kpad,
                                                                Ni, nb, w32, static_cast<uint32_t*>(Y), yw32, clear);
    return launch_status();
}

// The same filter for any real-input Sign layer (any position in the network, K up to kSlabMaxK): the frames are
// quantised into digit planes in the caller's workspace first, then K streams through LDS in slabs.
bool realx_sign_slab_applies(const bnn_layer_desc& d) {
    return !d.x_is_binary && !d.w_is_real && d.act == BNN_ACT_SIGN && d.K <= kSlabMaxK;
}
size_t realx_sign_slab_bytes(int64_t M, int64_t K) {
    const size_t kpad = (size_t)(K + 63) / 64 * 64;
    return (kDigits * (size_t)M * kpad + 255) / 256 * 256 + ((size_t)M * sizeof(RowMeta) + 255) / 256 * 256;
}
int run_realx_sign_slab(const float* X, const void* Wp, const float* scale, const float* bias, int64_t M, int64_t K,
                        int64_t N, int wb, void* Y, void* scratch_mem, hipStream_t st) {
    const int Mi = (int)M, Ki = (int)K, Ni = (int)N;
    const int w32 = (int)row_w32(K, wb), yw32 = (int)row_w32(N, wb);
    const int kpad = (Ki + 63) / 64 * 64;
    int8_t* planes = static_cast<int8_t*>(scratch_mem);
    RowMeta* meta = reinterpret_cast<RowMeta*>(planes + (kDigits * (size_t)M * kpad + 255) / 256 * 256);
    if (Ki % 4 == 0 && Ki <= 2048 && aligned(X, 16))
        realx_quantize_kernel<true><<<dim3((Mi + 3) / 4), dim3(256), 0, st>>>(X, Mi, Ki, kpad, slab_quant_bits(Ki), planes, meta);
    else
        realx_quantize_kernel<false><<<dim3((Mi + 3) / 4), dim3(256), 0, st>>>(X, Mi, Ki, kpad, slab_quant_bits(Ki), planes, meta);
    const size_t lds = slab_dynamic_lds();
    const bool vec16 = aligned(Wp, 16) && (w32 % 4 == 0);
    static std::atomic<uint64_t> allowed[2];
    if (!allow_lds(vec16 ? &realx_sign_slab_kernel<true> : &realx_sign_slab_kernel<false>, (unsigned)lds, allowed[vec16])) return BNN_EDEVICE;
    const dim3 grid((Mi + kRealxBM - 1) / kRealxBM, (Ni + kSlabNB - 1) / kSlabNB), block(kSlabThreads);
    if (vec16)
        realx_sign_slab_kernel<true><<<grid, block, lds, st>>>(X, planes, meta, static_cast<const uint32_t*>(Wp), scale, bias, Mi, Ki,
                                                              kpad, Ni, w32, static_cast<uint32_t*>(Y), yw32);
    else
        realx_sign_slab_kernel<false><<<grid, block, lds, st>>>(X, planes, meta, static_cast<const uint32_t*>(Wp), scale, bias, Mi, Ki,
                                                               kpad, Ni, w32, static_cast<uint32_t*>(Y), yw32);
    return launch_status();
}

// Output layer with real inputs and binary weights on the int8 matrix cores (four digit planes), inside bnn_forward
// (the planes live in the workspace): product kernel, then the log-Softmax row kernel.
bool realx_i8_lsm_applies(const bnn_layer_desc& d, int64_t M) {
    return !d.x_is_binary && !d.w_is_real && d.act == BNN_ACT_LOGSOFTMAX && d.K <= kSlabMaxK && M >= 128;
}
size_t realx_i8_lsm_bytes(int64_t M, int64_t K) {
    const size_t kpad = (size_t)(K + 63) / 64 * 64;
    return (kDigits4 * (size_t)M * kpad + 255) / 256 * 256 + ((size_t)M * sizeof(RowMeta4) + 255) / 256 * 256;
}
int run_realx_i8_lsm(const float* X, const void* Wp, const float* scale, const float* bias, int64_t M, int64_t K, int64_t N,
                     int wb, float* Y, void* scratch_mem, hipStream_t st) {
    const int Mi = (int)M, Ki = (int)K, Ni = (int)N;
    const int w32 = (int)row_w32(K, wb);
    const int kpad = (Ki + 63) / 64 * 64;
    int8_t* planes = static_cast<int8_t*>(scratch_mem);
    RowMeta4* meta = reinterpret_cast<RowMeta4*>(planes + (kDigits4 * (size_t)M * kpad + 255) / 256 * 256);
    realx_quantize4_kernel<<<dim3((Mi + 3) / 4), dim3(256), 0, st>>>(X, Mi, Ki, kpad, planes, meta);
    const size_t lds = slab4_dynamic_lds();
    const bool vec16 = aligned(Wp, 16) && (w32 % 4 == 0);
    static std::atomic<uint64_t> allowed[2];
    if (!allow_lds(vec16 ? &realx_i8_linear_kernel<true> : &realx_i8_linear_kernel<false>, (unsigned)lds, allowed[vec16])) return BNN_EDEVICE;
    const dim3 grid((Mi + kRealxBM - 1) / kRealxBM, (Ni + kSlabNB - 1) / kSlabNB), block(kSlabThreads);
    if (vec16)
        realx_i8_linear_kernel<true><<<grid, block, lds, st>>>(X, planes, meta, static_cast<const uint32_t*>(Wp), scale, bias, Mi, Ki,
                                                              kpad, Ni, w32, Y);
    else
        realx_i8_linear_kernel<false><<<grid, block, lds, st>>>(X, planes, meta, static_cast<const uint32_t*>(Wp), scale, bias, Mi, Ki,
                                                               kpad, Ni, w32, Y);
    launch_log_softmax(Y, Mi, Ni, st);
    return launch_status();
}

// Softmax layer with real weights on the bf16 matrix cores (three bf16 pieces per operand, six piece products), inside
// bnn_forward (the planes of both operands live in the workspace): two split passes, the product kernel, then the
// log-Softmax row kernel.  `scratch_mem` is 256-byte aligned.
bool realw_split_lsm_applies(const bnn_layer_desc& d, int64_t M) {
    return d.w_is_real && d.act == BNN_ACT_LOGSOFTMAX && M >= 128;
}
size_t realw_split_planes_bytes(int64_t rows, int64_t K) {
    return (kSplitPieces * (size_t)rows * (size_t)split_kpad((int)K) * 2 + 255) / 256 * 256;
}
size_t realw_split_lsm_bytes(int64_t M, int64_t K, int64_t N) {
    return realw_split_planes_bytes(M, K) + realw_split_planes_bytes(N, K);
}
void launch_split(const float* A, int64_t rows, int K, int kpad, uint16_t* planes, hipStream_t st) {
    const int64_t blocks = (rows * (kpad / 8) + 255) / 256;
    const unsigned grid = (unsigned)(blocks < 16384 ? blocks : 16384);
    if ((K & 3) == 0 && aligned(A, 16)) split_bf16x3_kernel<true><<<grid, 256, 0, st>>>(A, rows, K, kpad, planes);
    else split_bf16x3_kernel<false><<<grid, 256, 0, st>>>(A, rows, K, kpad, planes);
}
template <int WM, int WN, bool LONG = false>
int launch_split_product(const uint16_t* xs, const uint16_t* ws, const float* bias, int M, int kpad, int N, float* Y, hipStream_t st) {
    constexpr unsigned lds = split_dynamic_lds(WM, WN);
    static std::atomic<uint64_t> allowed;
    if (!allow_lds(&realw_bf16x3_kernel<WM, WN, LONG>, lds, allowed)) return BNN_EDEVICE;
    const dim3 grid((unsigned)((M + 64 * WM - 1) / (64 * WM)), (unsigned)((N + 64 * WN - 1) / (64 * WN)));
    realw_bf16x3_kernel<WM, WN, LONG><<<grid, 256, lds, st>>>(xs, ws, bias, M, kpad, N, Y);
    return BNN_OK;
}
int run_realw_split_lsm(const float* X, const float* W, const float* bias, int64_t M, int64_t K, int64_t N, float* Y,
                        void* scratch_mem, hipStream_t st) {
    const int Mi = (int)M, Ki = (int)K, Ni = (int)N;
    const int kpad = split_kpad(Ki);
    uint16_t* xs = static_cast<uint16_t*>(scratch_mem);
    uint16_t* ws = reinterpret_cast<uint16_t*>(static_cast<char*>(scratch_mem) + realw_split_planes_bytes(M, K));
    launch_split(X, M, Ki, kpad, xs, st);
    launch_split(W, N, Ki, kpad, ws, st);
    // 256 x 128 outputs per workgroup or 128 x 128?  One workgroup per CU either way, and a round of the small ones takes 0.55 to
    // 0.65 of the time.  Whole layers, K = 2048, large -> small: 600 frames x 3400 outputs 127 -> 82 us, 4096 x 1000 138 -> 111, three
    // rounds against two 279 -> 246 (2600 x 3400); but two against one 162 -> 174 (2048 x 3400), five against three 456 -> 458 (6000 x 3400).
    const int64_t large = (int64_t)((Mi + 255) / 256) * ((Ni + 127) / 128), small = (int64_t)((Mi + 127) / 128) * ((Ni + 127) / 128);
    const bool small_tiles = 3 * ((small + 255) / 256) < 5 * ((large + 255) / 256);
    // (rows of 8 MiB and more: a device holds a few thousand of them, one tile is enough)
    const int rc = kpad >= kSplitLongRow ? launch_split_product<2, 2, true>(xs, ws, bias, Mi, kpad, Ni, Y, st)
                   : small_tiles         ? launch_split_product<2, 2>(xs, ws, bias, Mi, kpad, Ni, Y, st)
                                         : launch_split_product<4, 2>(xs, ws, bias, Mi, kpad, Ni, Y, st);
    if (rc != BNN_OK) return rc;
    launch_log_softmax(Y, Mi, Ni, st);
    return launch_status();
}

// kpad x N fp32 (256-byte aligned; K padded to 64) for a layer with real weights that is not in front of the log-Softmax, 512
// frames or more.  No kernel uses it: it is what bnn_forward asks of the caller's workspace beyond what it needs, as it always
// has, so that the sizes programs were built with stay what bnn_forward_workspace_bytes says.  The fixed array of
// bnn_forward_static is not charged for it.
bool realw_reserved_applies(const bnn_layer_desc& d, int64_t M) {
    return d.w_is_real && d.act != BNN_ACT_LOGSOFTMAX && M >= 512 && (d.K & 3) == 0 && d.K <= 65536 && d.N <= (1 << 22);
}
size_t realw_reserved_bytes(int64_t K, int64_t N) {
    return round_up((size_t)((K + 63) / 64 * 64) * (size_t)N * 4, 256);
}
// Real-input layers with binary weights on the int8 matrix cores as a tiled product (128 frames x 256 or 64 x 128 outputs
// per workgroup), inside bnn_forward for batches of 128 frames or more: Sign layers (three digit planes, exact bits: the
// outputs the filter cannot decide are listed and resolved by a second kernel) and the layer in front of the
// log-Softmax (four digit planes).  Scratch, all 256-byte aligned: digit planes, weight bytes, one quantisation record per
// frame, the undecided outputs as bits.
bool realx_i8_gemm_applies(const bnn_layer_desc& d, int64_t M) {
    return !d.x_is_binary && !d.w_is_real && d.K <= kSlabMaxK && M >= 128 &&
           (d.act == BNN_ACT_SIGN || d.act == BNN_ACT_LOGSOFTMAX);
}
struct I8GemmScratch {
    size_t planes, bytes, meta, undecided, total;
};
I8GemmScratch i8_gemm_scratch(int64_t M, int64_t K, int64_t N, int act) {
    const size_t kpad = (size_t)i8_kpad((int)K);
    const int digits = act == BNN_ACT_SIGN ? 3 : 4;
    I8GemmScratch s{};
    s.planes = 0;
    s.bytes = round_up((size_t)digits * (size_t)M * kpad, 256);
    s.meta = s.bytes + round_up((size_t)N * kpad, 256);
    s.undecided = s.meta + round_up((size_t)M * 16, 256);
    // Sign layers: a record per frame and 128 outputs, one bit each (the filter leaves about one output in 250 undecided at
    // K = 2048).  Charged as pairs of records, as it always was.
    const size_t pairs = (size_t)((N + 2 * kUndecidedOutputs - 1) / (2 * kUndecidedOutputs));
    s.total = s.undecided + (act == BNN_ACT_SIGN ? round_up((size_t)M * pairs * 2 * kUndecidedRecord, 256) : 0);
    return s;
}
// Frames in 16-byte pieces are held in registers, in as many groups of 256 as they need (a power of two: what a frame does not
// fill costs loads of its first elements again); 32 groups, the longest frames there are, take 214 to 216 registers, which leaves
// two waves per SIMD (4096 x 6144 43 -> 33 us against reading the frame twice).  Ragged frames need a load per element and are read twice.
template <int D>
void launch_quantize(const float* X, int M, int K, int kpad, int qbits, int8_t* planes, void* meta, const ByteRows& weights, hipStream_t st) {
    const dim3 grid((unsigned)(((int64_t)M + 3) / 4 + byte_blocks(weights.N, kpad)));
    const bool vec = (K & 3) == 0 && aligned(X, 16);
    if (!vec) realx_quantize_nat_kernel<D, false, 0><<<grid, 256, 0, st>>>(X, M, K, kpad, qbits, planes, meta, weights);
    else if (kpad <= 512) realx_quantize_nat_kernel<D, true, 2><<<grid, 256, 0, st>>>(X, M, K, kpad, qbits, planes, meta, weights);
    else if (kpad <= 1024) realx_quantize_nat_kernel<D, true, 4><<<grid, 256, 0, st>>>(X, M, K, kpad, qbits, planes, meta, weights);
    else if (kpad <= 2048) realx_quantize_nat_kernel<D, true, 8><<<grid, 256, 0, st>>>(X, M, K, kpad, qbits, planes, meta, weights);
    else if (kpad <= 4096) realx_quantize_nat_kernel<D, true, 16><<<grid, 256, 0, st>>>(X, M, K, kpad, qbits, planes, meta, weights);
    else realx_quantize_nat_kernel<D, true, 32><<<grid, 256, 0, st>>>(X, M, K, kpad, qbits, planes, meta, weights);
    static_assert(kSlabMaxK <= 32 * 256, "a frame fits the registers");
}
// Tiles of 128 frames x 256 outputs (one workgroup per CU) or of 64 x 128 (two per CU)?  A round of the small ones, 512
// workgroups, is half the outputs of a round of 256 large ones and takes 0.5 to 0.7 of its time (a weight byte in LDS serves
// half as many frames).  Whole calls, large -> small, K = 2048: 600 frames x 2048 outputs 65 -> 33 us, 2048 x 2048 68 -> 50, 600 x 3400
// 66 -> 45; two full rounds of small tiles against one of large ones 75 -> 79 (4096 x 2048), two against a nearly full one 72 -> 78
// (3400 x 2048).  Sign layers with what resolves their undecided outputs: 600 x 2048 71 -> 50, 2048 x 2048 72 -> 62, 4096 x 2048 77 -> 85.
// The rule counts whole rounds of both and is on the careful side: with the last round of small tiles less than half full they
// would win, too (2600 x 2048 70 -> 64, 6000 x 2048 128 -> 112), though not with the longest sums (5475 x 8000 x 1000 279 -> 293).
bool i8_small_tiles(int M, int N) {
    const int64_t large = (int64_t)((M + 127) / 128) * ((N + 255) / 256), small = (int64_t)((M + 63) / 64) * ((N + 127) / 128);
    return 2 * ((small + 511) / 512) < 3 * ((large + 255) / 256);
}
template <int D, int WM, int WN>
int launch_i8_product(const int8_t* planes, const int8_t* bytes, const void* meta, const float* X, const void* Wp, const float* scale,
                      const float* bias, int M, int K, int kpad, int N, int w32, void* Y, int yw32, unsigned char* undecided, hipStream_t st) {
    constexpr unsigned lds = i8_gemm_lds(D, WM, WN);
    static std::atomic<uint64_t> allowed;
    if (!allow_lds(&realx_i8_gemm_kernel<D, WM, WN>, lds, allowed)) return BNN_EDEVICE;
    const dim3 grid((unsigned)((M + 64 * WM - 1) / (64 * WM)), (unsigned)((N + 64 * WN - 1) / (64 * WN)));
    realx_i8_gemm_kernel<D, WM, WN><<<grid, kI8Threads, lds, st>>>(planes, bytes, meta, X, static_cast<const uint32_t*>(Wp), scale, bias, M, K,
                                                                   kpad, N, w32, Y, yw32, D == 3 ? undecided : nullptr);
    return BNN_OK;
}
template <int D>
int launch_realx_i8_gemm(const float* X, const void* Wp, const float* scale, const float* bias, int Mi, int Ki, int Ni, int w32,
                         void* Y, int yw32, char* mem, const I8GemmScratch& sc, hipStream_t st, Front* front = nullptr) {
    const int kpad = i8_kpad(Ki);
    int8_t* planes = reinterpret_cast<int8_t*>(mem + sc.planes);
    int8_t* bytes = reinterpret_cast<int8_t*>(mem + sc.bytes);
    void* meta = mem + sc.meta;
    unsigned char* undecided = reinterpret_cast<unsigned char*>(mem + sc.undecided);
    const int qbits = D == 3 ? slab_quant_bits(Ki) : kQuantBits4;
    launch_quantize<D>(X, Mi, Ki, kpad, qbits, planes, meta, {static_cast<const uint32_t*>(Wp), bytes, Ni, w32}, st);
    const int rc = i8_small_tiles(Mi, Ni)
        ? launch_i8_product<D, 1, 2>(planes, bytes, meta, X, Wp, scale, bias, Mi, Ki, kpad, Ni, w32, Y, yw32, undecided, st)
        : launch_i8_product<D, 2, 4>(planes, bytes, meta, X, Wp, scale, bias, Mi, Ki, kpad, Ni, w32, Y, yw32, undecided, st);
    if (rc != BNN_OK) return rc;
    const int recs = (Ni + kUndecidedOutputs - 1) / kUndecidedOutputs;
    if (D == 3) {
        const unsigned int rg = (unsigned int)((Mi + kResolveFrames - 1) / kResolveFrames);
        const Clear clear = cleared_by(clear_for(front, BNN_ACT_SIGN), dim3(rg));
        if ((Ki & 3) == 0 && aligned(X, 16))
            realx_resolve_rows_kernel<true><<<rg, kResolveThreads, 0, st>>>(X, static_cast<const uint32_t*>(Wp), scale, bias, Mi, Ki, w32,
                                                                          undecided, recs, static_cast<uint32_t*>(Y), yw32, clear);
        else
            realx_resolve_rows_kernel<false><<<rg, kResolveThreads, 0, st>>>(X, static_cast<const uint32_t*>(Wp), scale, bias, Mi, Ki, w32,
                                                                           undecided, recs, static_cast<uint32_t*>(Y), yw32, clear);
    }
    return BNN_OK;
}
int run_realx_i8_gemm(const float* X, const void* Wp, const float* scale, const float* bias, int64_t M, int64_t K, int64_t N, int wb,
                      int act, void* Y, void* scratch_mem, hipStream_t st, Front* front) {
    const I8GemmScratch sc = i8_gemm_scratch(M, K, N, act);
    const int w32 = (int)row_w32(K, wb), yw32 = (int)row_w32(N, wb);
    int rc;
    if (act == BNN_ACT_SIGN) {
        rc = launch_realx_i8_gemm<3>(X, Wp, scale, bias, (int)M, (int)K, (int)N, w32, Y, yw32, static_cast<char*>(scratch_mem), sc, st, front);
    } else {
        rc = launch_realx_i8_gemm<4>(X, Wp, scale, bias, (int)M, (int)K, (int)N, w32, Y, 0, static_cast<char*>(scratch_mem), sc, st);
        if (rc == BNN_OK) launch_log_softmax(static_cast<float*>(Y), (int)M, (int)N, st);
    }
    return rc != BNN_OK ? rc : launch_status();
}

int check_chain(const bnn_layer_desc* L, int n_layers, int64_t M) {
    if (!L || n_layers <= 0) return BNN_EINVAL;
    if (M < 0 || M > kMaxDim) return BNN_ESHAPE;
    for (int l = 0; l < n_layers; ++l) {
        const bnn_layer_desc& d = L[l];
        if (!word_bits_ok(d.word_bits) || d.K <= 0 || d.N <= 0 || d.K > kMaxDim || d.N > kMaxN) return BNN_ESHAPE;
        if (d.act < BNN_ACT_LINEAR || d.act > BNN_ACT_SIGMOID) return BNN_EINVAL;
        if (d.w_is_real < 0 || d.w_is_real > 1 || (d.w_is_real && d.scale)) return BNN_EINVAL;
        if (d.x_is_binary < 0 || d.x_is_binary > 2) return BNN_EINVAL;
        if (!d.Wp) return BNN_EINVAL;
        if (l > 0) {
            const bnn_layer_desc& p = L[l - 1];
            if (d.K != p.N) return BNN_ESHAPE;
            if ((d.x_is_binary != 0) != (p.act == BNN_ACT_SIGN)) return BNN_ESHAPE;
            if (d.x_is_binary && d.word_bits != p.word_bits) return BNN_ESHAPE;
            if (p.act == BNN_ACT_LOGSOFTMAX) return BNN_ESHAPE;   // Softmax only closes a network (Alg. 2)
        }
    }
    return BNN_OK;
}

}  // namespace

// ------------------------------------------------------------------------------------------------ C ABI

BNN_EXPORT size_t bnn_packed_words(int64_t K, int word_bits) {
    if (K <= 0 || !word_bits_ok(word_bits)) return 0;
    return (size_t)words_per_row(K, word_bits);
}

BNN_EXPORT const char* bnn_status_string(int status) {
    switch (status) {
        case BNN_OK: return "ok";
        case BNN_EINVAL: return "invalid argument (null pointer, unknown activation or arm, overlapping buffers)";
        case BNN_ESHAPE: return "invalid shape (M < 0, K or N <= 0, word_bits not 32/64, or inconsistent layer chain)";
        case BNN_EALIGN: return "misaligned pointer";
        case BNN_EWORKSPACE: return "workspace missing or too small";
        case BNN_EDEVICE: return "HIP launch failed";
        default: return "unknown status";
    }
}

BNN_EXPORT int bnn_set_option(int option, int value) {
    switch (option) {
        case BNN_OPT_BINX_ARM:
            if (value != BNN_ARM_VALU_XOR && value != BNN_ARM_MFMA && value != BNN_ARM_MFMA_I8) return BNN_EINVAL;
            g_default_arm.store(value);
            return BNN_OK;
        case BNN_OPT_REALX_TM:
            if (value != 0 && value != 1 && value != 2 && value != 4 && value != 8 && value != 16 && value != 32) return BNN_EINVAL;
            g_realx_tm.store(value);
            return BNN_OK;
        case BNN_OPT_STREAM_MAX_FRAMES:
            if (value < 0 || value > 4096) return BNN_EINVAL;
            g_stream_max_frames.store(value);
            return BNN_OK;
        case BNN_OPT_BINX_VALU_TM:
            if (value != 1 && value != 2 && value != 4 && value != 8 && value != 16 && value != 32) return BNN_EINVAL;
            g_binx_valu_tm.store(value);
            return BNN_OK;
        case BNN_OPT_MFMA_WM:
            if (value != 2 && value != 4) return BNN_EINVAL;
            g_mfma_wm.store(value);
            return BNN_OK;
        case BNN_OPT_MFMA_SHAPE:
            if (value != 0 && value != 16 && value != 32) return BNN_EINVAL;
            g_mfma_shape.store(value);
            return BNN_OK;
        case BNN_OPT_MFMA32_WM:
            if (value != 0 && value != 2 && value != 4) return BNN_EINVAL;
            g_mfma32_wm.store(value);
            return BNN_OK;
        case BNN_OPT_MFMA32_XCD_ORDER:
            if (value < 0 || value > 2) return BNN_EINVAL;
            g_mfma32_xcd_order.store(value);
            return BNN_OK;
        case BNN_OPT_REALX_F32_MFMA:
            if (value < 0 || value > 2) return BNN_EINVAL;
            g_realx_f32_mfma.store(value);
            return BNN_OK;
        case BNN_OPT_MFMA32_PIPELINE:
            if (value < 0 || value > 2) return BNN_EINVAL;
            g_mfma32_pipeline.store(value);
            return BNN_OK;
        case BNN_OPT_FUSED_LOGSOFTMAX:
            if (value != 0 && value != 1) return BNN_EINVAL;
            g_fused_softmax.store(value);
            return BNN_OK;
        case BNN_OPT_REALX_SIGN_MFMA:
            if (value < 0 || value > 2) return BNN_EINVAL;
            g_realx_sign_mfma.store(value);
            return BNN_OK;
        case BNN_OPT_COOPERATIVE:
            if (value != 0 && value != 1) return BNN_EINVAL;
            g_cooperative.store(value);
            return BNN_OK;
        case BNN_OPT_REALX_I8_LOGSOFTMAX:
            if (value < 0 || value > 2) return BNN_EINVAL;
            g_realx_i8_lsm.store(value);
            return BNN_OK;
        case BNN_OPT_REALW_SPLIT_LOGSOFTMAX:
            if (value < 0 || value > 2) return BNN_EINVAL;
            g_realw_split_lsm.store(value);
            return BNN_OK;
        case BNN_OPT_REALW_VALU_LDS:
            if (value != 0 && value != 1) return BNN_EINVAL;
            return BNN_OK;   // one kernel, the same bits
        case BNN_OPT_COOPERATIVE_SPIN:
            if (value < 1) return BNN_EINVAL;
            g_coop_spin.store(value);
            return BNN_OK;
        case BNN_OPT_MFMA32_SPLITK:
            if (value != 0 && value != 1) return BNN_EINVAL;
            return BNN_OK;   // one kernel, the same bits
        default: return BNN_EINVAL;
    }
}

BNN_EXPORT int bnn_cooperative_timeouts(uint64_t* count) {
    if (!count) return BNN_EINVAL;
    int dev = -1;
    unsigned char* base = coop_base(&dev);
    if (!base) return BNN_EDEVICE;
    unsigned int v = 0;
    if (hipDeviceSynchronize() != hipSuccess || hipMemcpy(&v, base, sizeof(v), hipMemcpyDeviceToHost) != hipSuccess) {
        (void)hipGetLastError();
        return BNN_EDEVICE;
    }
    *count = v;
    return BNN_OK;
}

BNN_EXPORT int bnn_pack_weights(const float* W, int64_t N, int64_t K, int word_bits, void* Wp, float* scale_out,
                                void* stream) {
    if (!word_bits_ok(word_bits) || N <= 0 || K <= 0 || N > kMaxDim || K > kMaxDim) return BNN_ESHAPE;
    if (!W || !Wp) return BNN_EINVAL;
    if (!aligned(W, 4) || !aligned(Wp, word_bits / 8) || (scale_out && !aligned(scale_out, 4))) return BNN_EALIGN;
    const size_t wb = (size_t)N * K * 4, pb = (size_t)N * row_w32(K, word_bits) * 4;
    if (overlap(W, wb, Wp, pb) || (scale_out && (overlap(W, wb, scale_out, 4) || overlap(Wp, pb, scale_out, 4))))
        return BNN_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int rc = run_pack(W, N, K, word_bits, Wp, st);
    if (rc != BNN_OK) return rc;
    if (scale_out) {
        mean_abs_kernel<<<dim3(1), dim3(1024), 0, st>>>(W, N * K, scale_out);
        return launch_status();
    }
    return BNN_OK;
}

BNN_EXPORT int bnn_pack_activations(const float* X, int64_t M, int64_t K, int word_bits, void* Xp, void* stream) {
    if (!word_bits_ok(word_bits) || M < 0 || K <= 0 || M > kMaxDim || K > kMaxDim) return BNN_ESHAPE;
    if (M == 0) return BNN_OK;
    if (!X || !Xp) return BNN_EINVAL;
    if (!aligned(X, 4) || !aligned(Xp, word_bits / 8)) return BNN_EALIGN;
    if (overlap(X, (size_t)M * K * 4, Xp, (size_t)M * row_w32(K, word_bits) * 4)) return BNN_EINVAL;
    return run_pack(X, M, K, word_bits, Xp, static_cast<hipStream_t>(stream));
}

BNN_EXPORT int bnn_layer_binw_realx(const float* X, const void* Wp, const float* scale, const float* bias, int64_t M,
                                    int64_t K, int64_t N, int act, int word_bits, void* Y, void* stream) {
    const int rc = check_layer_args(X, Wp, M, K, N, act, word_bits, Y, false);
    if (rc != BNN_OK) return rc;
    return run_realx(X, Wp, scale, bias, M, K, N, act, word_bits, Y, static_cast<hipStream_t>(stream));
}

BNN_EXPORT int bnn_layer_binw_binx_arm(const void* Xp, const void* Wp, const float* scale, const float* bias, int64_t M,
                                       int64_t K, int64_t N, int act, int word_bits, void* Y, int arm, void* stream) {
    if (arm != BNN_ARM_AUTO && arm != BNN_ARM_VALU_XOR && arm != BNN_ARM_MFMA && arm != BNN_ARM_MFMA_I8) return BNN_EINVAL;
    const int rc = check_layer_args(Xp, Wp, M, K, N, act, word_bits, Y, true);
    if (rc != BNN_OK) return rc;
    return run_binx(Xp, Wp, scale, bias, M, K, N, act, word_bits, Y, arm, static_cast<hipStream_t>(stream));
}

BNN_EXPORT int bnn_layer_binw_binx01(const void* Xp, const void* Wp, const float* scale, const float* bias, int64_t M,
                                     int64_t K, int64_t N, int act, int word_bits, void* Y, void* stream) {
    const int rc = check_layer_args(Xp, Wp, M, K, N, act, word_bits, Y, true);
    if (rc != BNN_OK) return rc;
    return run_binx(Xp, Wp, scale, bias, M, K, N, act, word_bits, Y, BNN_ARM_MFMA, static_cast<hipStream_t>(stream), true);
}

BNN_EXPORT int bnn_layer_binw_binx(const void* Xp, const void* Wp, const float* scale, const float* bias, int64_t M,
                                   int64_t K, int64_t N, int act, int word_bits, void* Y, void* stream) {
    return bnn_layer_binw_binx_arm(Xp, Wp, scale, bias, M, K, N, act, word_bits, Y, BNN_ARM_AUTO, stream);
}

BNN_EXPORT int bnn_layer_realw(const float* X, const float* W, const float* bias, int64_t M, int64_t K, int64_t N, int act,
                               int word_bits, void* Y, void* stream) {
    const int rc = check_layer_args(X, W, M, K, N, act, word_bits, Y, false, true);
    if (rc != BNN_OK) return rc;
    return run_realw(X, W, bias, M, K, N, act, word_bits, Y, static_cast<hipStream_t>(stream));
}

BNN_EXPORT int bnn_unpack_activations(const void* Xp, int64_t M, int64_t K, int word_bits, int zero_one, float* X,
                                      void* stream) {
    if (!word_bits_ok(word_bits) || M < 0 || K <= 0 || M > kMaxDim || K > kMaxDim) return BNN_ESHAPE;
    if (zero_one < 0 || zero_one > 1) return BNN_EINVAL;
    if (M == 0) return BNN_OK;
    if (!Xp || !X) return BNN_EINVAL;
    if (!aligned(Xp, word_bits / 8) || !aligned(X, 4)) return BNN_EALIGN;
    if (overlap(Xp, (size_t)M * row_w32(K, word_bits) * 4, X, (size_t)M * K * 4)) return BNN_EINVAL;
    return run_unpack(Xp, M, K, word_bits, zero_one, X, static_cast<hipStream_t>(stream));
}

// ------------------------------------------------------------------------------------------------ training side

namespace {
unsigned elementwise_blocks(int64_t count) {
    const int64_t b = (count + 255) / 256;
    return (unsigned)(b < 65536 ? (b > 0 ? b : 1) : 65536);
}
// blocks for `count` elements, four consecutive ones per thread where the arrays are 16-byte aligned
unsigned quad_blocks(int64_t count) { return elementwise_blocks((count + 3) / 4); }
bool dims_ok(int64_t a, int64_t b) { return a > 0 && b > 0 && a <= kMaxDim && b <= kMaxDim; }
}  // namespace

BNN_EXPORT int bnn_pack_weights_transposed(const float* W, int64_t N, int64_t K, int word_bits, void* WpT, void* stream) {
    if (!word_bits_ok(word_bits) || !dims_ok(N, K)) return BNN_ESHAPE;
    if (!W || !WpT) return BNN_EINVAL;
    if (!aligned(W, 4) || !aligned(WpT, word_bits / 8)) return BNN_EALIGN;
    const int w32t = (int)row_w32(N, word_bits);
    if (overlap(W, (size_t)N * K * 4, WpT, (size_t)K * w32t * 4)) return BNN_EINVAL;
    const dim3 grid((unsigned)((K + 255) / 256), (unsigned)((N + 63) / 64));
    pack_sign_transposed_kernel<<<grid, 256, 0, static_cast<hipStream_t>(stream)>>>(W, (int)N, (int)K, w32t,
                                                                                     static_cast<uint32_t*>(WpT));
    return launch_status();
}

BNN_EXPORT int bnn_transpose_f32(const float* A, int64_t R, int64_t C, float* out, void* stream) {
    if (!dims_ok(R, C)) return BNN_ESHAPE;
    if (!A || !out) return BNN_EINVAL;
    if (!aligned(A, 4) || !aligned(out, 4)) return BNN_EALIGN;
    if (overlap(A, (size_t)R * C * 4, out, (size_t)R * C * 4)) return BNN_EINVAL;
    const dim3 grid((unsigned)((C + 63) / 64), (unsigned)((R + 63) / 64));
    transpose_f32_kernel<<<grid, 256, 0, static_cast<hipStream_t>(stream)>>>(A, (int)R, (int)C, out);
    return launch_status();
}

BNN_EXPORT int bnn_softmax_xent_grad(const float* logp, const int32_t* labels, int64_t M, int64_t N, float* g, void* stream) {
    if (M < 0 || N <= 0 || M > kMaxDim || N > kMaxDim) return BNN_ESHAPE;
    if (M == 0) return BNN_OK;
    if (!logp || !labels || !g) return BNN_EINVAL;
    if (!aligned(logp, 4) || !aligned(labels, 4) || !aligned(g, 4)) return BNN_EALIGN;
    hipStream_t st = static_cast<hipStream_t>(stream);
    // A workgroup per frame from 1024 frames of 512 classes on (4096 x 3307 22 us, 31 by elements), by elements otherwise
    // (by frames and by elements: 256 x 3400 5.6 and 3.7 us, 16 x 3400 5.3 and 3.5, 1 x 100000 49 and 3.6, 4096 x 128 4.3 and
    // 3.6, 50000 x 4 28 and 3.6).
    auto go = [&](auto vec, unsigned blocks) {
        constexpr bool V = decltype(vec)::value;
        if (M >= 1024 && N >= 512) softmax_xent_grad_rows_kernel<V><<<(unsigned)(M < 65536 ? M : 65536), 256, 0, st>>>(logp, labels, M, (int)N, g);
        else if (M * N < ((int64_t)1 << 32)) softmax_xent_grad_kernel<V, uint32_t><<<blocks, 256, 0, st>>>(logp, labels, M, (int)N, g);
        else softmax_xent_grad_kernel<V, uint64_t><<<blocks, 256, 0, st>>>(logp, labels, M, (int)N, g);
    };
    if (N % 4 == 0 && aligned(logp, 16) && aligned(g, 16)) go(std::true_type{}, quad_blocks(M * N));
    else go(std::false_type{}, elementwise_blocks(M * N));
    return launch_status();
}

BNN_EXPORT int bnn_mask_grad(const float* g_h, const float* hhat, int64_t count, float k, float* g_hhat, void* stream) {
    if (count < 0) return BNN_ESHAPE;
    if (!(k > 0.0f)) return BNN_EINVAL;
    if (count == 0) return BNN_OK;
    if (!g_h || !hhat || !g_hhat) return BNN_EINVAL;
    if (!aligned(g_h, 4) || !aligned(hhat, 4) || !aligned(g_hhat, 4)) return BNN_EALIGN;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (aligned(g_h, 16) && aligned(hhat, 16) && aligned(g_hhat, 16)) mask_grad_kernel<true><<<quad_blocks(count), 256, 0, st>>>(g_h, hhat, count, k, g_hhat);
    else mask_grad_kernel<false><<<elementwise_blocks(count), 256, 0, st>>>(g_h, hhat, count, k, g_hhat);
    return launch_status();
}

BNN_EXPORT int bnn_sigmoid_grad(const float* g_h, const float* h, int64_t count, float* g_hhat, void* stream) {
    if (count < 0) return BNN_ESHAPE;
    if (count == 0) return BNN_OK;
    if (!g_h || !h || !g_hhat) return BNN_EINVAL;
    if (!aligned(g_h, 4) || !aligned(h, 4) || !aligned(g_hhat, 4)) return BNN_EALIGN;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (aligned(g_h, 16) && aligned(h, 16) && aligned(g_hhat, 16)) sigmoid_grad_kernel<true><<<quad_blocks(count), 256, 0, st>>>(g_h, h, count, g_hhat);
    else sigmoid_grad_kernel<false><<<elementwise_blocks(count), 256, 0, st>>>(g_h, h, count, g_hhat);
    return launch_status();
}

BNN_EXPORT size_t bnn_layer_binw_realx_i8_workspace_bytes(int64_t M, int64_t K, int64_t N) {
    if (M <= 0 || K <= 0 || N <= 0 || M > kMaxDim || K > kSlabMaxK || N > kMaxN) return 0;
    return i8_gemm_scratch(M, K, N, BNN_ACT_LINEAR).total;
}

BNN_EXPORT int bnn_layer_binw_realx_i8(const float* X, const void* Wp, const float* scale, const float* bias, int64_t M,
                                       int64_t K, int64_t N, int word_bits, float* Y, void* workspace, size_t workspace_bytes,
                                       void* stream) {
    const int rc = check_layer_args(X, Wp, M, K, N, BNN_ACT_LINEAR, word_bits, Y, false);
    if (rc != BNN_OK) return rc;
    if (K > kSlabMaxK) return BNN_ESHAPE;
    if (M == 0) return BNN_OK;
    const I8GemmScratch sc = i8_gemm_scratch(M, K, N, BNN_ACT_LINEAR);
    if (!workspace || workspace_bytes < sc.total) return BNN_EWORKSPACE;
    if (!aligned(workspace, 256)) return BNN_EALIGN;
    const size_t yb = (size_t)M * N * 4;
    if (overlap(workspace, sc.total, Y, yb) || overlap(workspace, sc.total, X, (size_t)M * K * 4) ||
        overlap(workspace, sc.total, Wp, (size_t)N * row_w32(K, word_bits) * 4))
        return BNN_EINVAL;
    const int lrc = launch_realx_i8_gemm<4>(X, Wp, scale, bias, (int)M, (int)K, (int)N, (int)row_w32(K, word_bits), Y, 0,
                                            static_cast<char*>(workspace), sc, static_cast<hipStream_t>(stream));
    return lrc != BNN_OK ? lrc : launch_status();
}

BNN_EXPORT int bnn_backward_input_binw(const float* g_hhat, const void* WpT, int64_t M, int64_t N, int64_t K, int word_bits,
                                       float* g_h, void* stream) {
    // the forward layer with the roles exchanged: "inputs" are the N gradients of a frame, "outputs" the K inputs
    const int rc = check_layer_args(g_hhat, WpT, M, N, K, BNN_ACT_LINEAR, word_bits, g_h, false);
    if (rc != BNN_OK) return rc;
    return run_realx(g_hhat, WpT, nullptr, nullptr, M, N, K, BNN_ACT_LINEAR, word_bits, g_h, static_cast<hipStream_t>(stream));
}

BNN_EXPORT int bnn_backward_input_realw(const float* g_hhat, const float* Wt, int64_t M, int64_t N, int64_t K, float* g_h,
                                        void* stream) {
    const int rc = check_layer_args(g_hhat, Wt, M, N, K, BNN_ACT_LINEAR, 32, g_h, false, true);
    if (rc != BNN_OK) return rc;
    return run_realw(g_hhat, Wt, nullptr, M, N, K, BNN_ACT_LINEAR, 32, g_h, static_cast<hipStream_t>(stream));
}

BNN_EXPORT int bnn_backward_weight(const float* g_hhat_t, const float* h_t, int64_t N, int64_t K, int64_t M, float* g_w,
                                   void* stream) {
    // rows of the "frame" operand are the N outputs, the sum runs over the M frames, "outputs" are the K inputs
    if (M <= 0) return BNN_ESHAPE;
    const int rc = check_layer_args(g_hhat_t, h_t, N, M, K, BNN_ACT_LINEAR, 32, g_w, false, true);
    if (rc != BNN_OK) return rc;
    return run_realw(g_hhat_t, h_t, nullptr, N, M, K, BNN_ACT_LINEAR, 32, g_w, static_cast<hipStream_t>(stream));
}

BNN_EXPORT int bnn_backward_weight_binh(const float* g_hhat_t, const void* HpT, int64_t N, int64_t K, int64_t M, int word_bits,
                                        float* g_w, void* stream) {
    if (M <= 0) return BNN_ESHAPE;
    const int rc = check_layer_args(g_hhat_t, HpT, N, M, K, BNN_ACT_LINEAR, word_bits, g_w, false);
    if (rc != BNN_OK) return rc;
    return run_realx(g_hhat_t, HpT, nullptr, nullptr, N, M, K, BNN_ACT_LINEAR, word_bits, g_w, static_cast<hipStream_t>(stream));
}

BNN_EXPORT int bnn_bias_grad(const float* g_hhat, int64_t M, int64_t N, float* g_r, void* stream) {
    if (M < 0 || N <= 0 || M > kMaxDim || N > kMaxDim) return BNN_ESHAPE;
    if (!g_hhat || !g_r) return BNN_EINVAL;
    if (!aligned(g_hhat, 4) || !aligned(g_r, 4)) return BNN_EALIGN;
    if (overlap(g_hhat, (size_t)M * N * 4, g_r, (size_t)N * 4)) return BNN_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    // Slabs through LDS up to three workgroups of 16 columns per CU; beyond that one wave per 64 columns, which also keeps the
    // grid of 2^30 columns in range.  Measured, slabs against waves: 4096 x 8192 40 and 56 us, 1000 x 12000 16.4 and 18.9,
    // 300 x 12000 6.0 and 5.7, 300 x 16384 8.9 and 5.5, 4096 x 16384 81 and 61, 16 x 20000 4.6 and 3.5.
    if (N > kColsumMaxCols) {
        colsum_wave_kernel<<<(unsigned)((N + kWave - 1) / kWave), kWave, 0, st>>>(g_hhat, (int)M, (int)N, g_r);
        return launch_status();
    }
    const unsigned blocks = (unsigned)((N + kColsumCols - 1) / kColsumCols);
    if (N % 4 == 0 && aligned(g_hhat, 16)) colsum_kernel<true><<<blocks, 256, 0, st>>>(g_hhat, (int)M, (int)N, g_r);
    else colsum_kernel<false><<<blocks, 256, 0, st>>>(g_hhat, (int)M, (int)N, g_r);
    return launch_status();
}

BNN_EXPORT int bnn_update_clip(float* w, const float* g, int64_t count, float eta, int clip, void* stream) {
    if (count < 0) return BNN_ESHAPE;
    if (clip < 0 || clip > 1) return BNN_EINVAL;
    if (count == 0) return BNN_OK;
    if (!w || !g) return BNN_EINVAL;
    if (!aligned(w, 4) || !aligned(g, 4)) return BNN_EALIGN;
    if (overlap(w, (size_t)count * 4, g, (size_t)count * 4)) return BNN_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (aligned(w, 16) && aligned(g, 16)) update_clip_kernel<true><<<quad_blocks(count), 256, 0, st>>>(w, g, count, eta, clip);
    else update_clip_kernel<false><<<elementwise_blocks(count), 256, 0, st>>>(w, g, count, eta, clip);
    return launch_status();
}

BNN_EXPORT int bnn_grad_norm_clip(float* g, int64_t count, float alpha, void* workspace, float* norm_out, void* stream) {
    if (count < 0) return BNN_ESHAPE;
    if (!(alpha > 0.0f)) return BNN_EINVAL;
    if (!g || !workspace || !norm_out) return BNN_EINVAL;
    if (!aligned(g, 4) || !aligned(workspace, 8) || !aligned(norm_out, 4)) return BNN_EALIGN;
    hipStream_t st = static_cast<hipStream_t>(stream);
    double* partial = static_cast<double*>(workspace);
    const bool inside = overlap(workspace, kSumsqBlocks * sizeof(double), norm_out, sizeof(float));
    auto go = [&](auto vec, unsigned blocks) {
        constexpr bool V = decltype(vec)::value;
        sumsq_partial_kernel<V><<<kSumsqBlocks, kSumsqThreads, 0, st>>>(g, count, partial);
        if (inside) sumsq_final_kernel<<<1, kWave, 0, st>>>(partial, norm_out);
        scale_if_above_kernel<V><<<min(blocks, 1024u), 256, 0, st>>>(g, count, alpha, inside ? nullptr : partial, norm_out);
    };
    if (aligned(g, 16)) go(std::true_type{}, quad_blocks(count));
    else go(std::false_type{}, elementwise_blocks(count));
    return launch_status();
}

BNN_EXPORT int bnn_subtract_log_prior(float* logp, const float* log_prior, int64_t M, int64_t N, void* stream) {
    if (M < 0 || N <= 0 || M > kMaxDim || N > kMaxN) return BNN_ESHAPE;
    if (M == 0) return BNN_OK;
    if (!logp || !log_prior) return BNN_EINVAL;
    if (!aligned(logp, 4) || !aligned(log_prior, 4)) return BNN_EALIGN;
    if (overlap(logp, (size_t)M * (size_t)N * 4, log_prior, (size_t)N * 4)) return BNN_EINVAL;
    subtract_log_prior_kernel<<<elementwise_blocks(M * N), 256, 0, static_cast<hipStream_t>(stream)>>>(logp, log_prior, M, (int)N);
    return launch_status();
}

BNN_EXPORT int bnn_semi_stochastic_binarize(float* w, const float* u, int64_t count, void* stream) {
    if (count < 0) return BNN_ESHAPE;
    if (count == 0) return BNN_OK;
    if (!w || !u) return BNN_EINVAL;
    if (!aligned(w, 4) || !aligned(u, 4)) return BNN_EALIGN;
    if (overlap(w, (size_t)count * 4, u, (size_t)count * 4)) return BNN_EINVAL;
    semi_stochastic_kernel<<<elementwise_blocks(count), 256, 0, static_cast<hipStream_t>(stream)>>>(w, u, count);
    return launch_status();
}

// Runs of binary layers of a streaming batch in one launch (few_chain_kernel.hpp), inside bnn_forward: the layers from l on, as many
// as bits pass between, behind a layer with real inputs or weights (whose launch clears the marks).  0: none.
// Whole passes back to back, 440 inputs, six hidden layers, 3400 outputs, one launch per layer -> this: 1 frame 25.5 -> 12.9 us (512
// units), 25.4 -> 13.4 (1024), 27.1 -> 15.3 (2048); 16 frames 27.8 -> 15.5 and 27.3 -> 17.8 (1024, 2048); 64 frames 28.9 -> 18.3
// and 37.3 -> 27.3.  Rows that are no multiple of 16 bytes gain more, having no split of K over lanes otherwise (51 frames of 1344 units
// 64.5 -> 31.0).  Four streams at once: 16 frames 9.3 -> 5.8 and 13.0 -> 9.7, 64 frames 12.8 -> 7.5 and 20.4 -> 12.3.  Wider layers stay apart: every XCD reads all weights here, and 4096 units are 2 MB a layer (6 layers, 32 frames
// 48.9 -> 45.5 us, but 1 frame 27.0 -> 28.0, 64 frames 56.7 -> 68.6), in registers that leave no room for a second launch beside
// this one.  Two hidden layers alone gain nothing where their rows are whole pieces (1 frame, 3584 units 52.2 -> 54.2).
static int few_chain_layers(const bnn_layer_desc* layers, int n_layers, int l, int64_t M) {
    if (l < 1 || l >= n_layers || M > kFewMaxFrames) return 0;
    auto binary = [](const bnn_layer_desc& d) { return d.x_is_binary && !d.w_is_real; };
    if (binary(layers[l - 1])) return 0;
    int n = 0;
    bool whole = true;   // rows of whole 16-byte pieces
    for (; l + n < n_layers && n < kFewMaxLayers && binary(layers[l + n]); ++n) {
        const bnn_layer_desc& d = layers[l + n];
        const int64_t w32 = row_w32(d.K, d.word_bits);
        if (w32 > kFewMaxInputWords || d.N > kFewMaxClasses) break;
        whole = whole && w32 % 4 == 0 && aligned(d.Wp, 16);
    }
    const bool lsm = n > 0 && layers[l + n - 1].act == BNN_ACT_LOGSOFTMAX;
    return n >= (whole && !lsm ? 3 : 2) ? n : 0;
}
static int few_chain_pieces(const bnn_layer_desc* layers, int l, int n) {   // 16-byte pieces of a row of bits per lane
    int nr = 1;
    for (int j = l; j < l + n; ++j)
        while (row_w32(layers[j].K, layers[j].word_bits) > 16 * nr) nr *= 2;
    return nr;
}
static_assert(kFewMaxLayers <= kPullLayers && kFewSlots == kPullGroups, "as many layers and workgroups");
struct FewScratch {
    size_t words, z, total;   // the layers' marked words, one behind the other; the last layer's pre-activations; both
};
static FewScratch few_chain_scratch(const bnn_layer_desc* layers, int l, int n, int64_t M) {
    FewScratch s{};
    const bnn_layer_desc& last = layers[l + n - 1];
    const bool lsm = last.act == BNN_ACT_LOGSOFTMAX;
    s.words = round_up((size_t)M * 8 * ((size_t)(n - 1) * 16 * few_chain_pieces(layers, l, n) + (lsm ? kFewMaxWords : 0)), 256);
    s.z = lsm ? round_up((size_t)M * round_up((size_t)last.N, 2) * 4, 256) : 0;
    s.total = s.words + s.z;
    return s;
}
// The output of a run is written while its earlier layers are still read, which one launch per layer never does: it must not lie over
// their weights.
static bool apart(const bnn_layer_desc* layers, int l, int n, int64_t M, const void* Y) {
    const bnn_layer_desc& last = layers[l + n - 1];
    const size_t yb = out_bytes(M, last.N, last.act, last.word_bits);
    for (int j = l; j < l + n; ++j) {
        const bnn_layer_desc& d = layers[j];
        if (overlap(Y, yb, d.Wp, (size_t)d.N * row_w32(d.K, d.word_bits) * 4) || overlap(Y, yb, d.scale, d.scale ? (size_t)d.N * 4 : 0) ||
            overlap(Y, yb, d.bias, d.bias ? (size_t)d.N * 4 : 0))
            return false;
    }
    return true;
}
// In this call?  Y: where the last of the n layers writes.
static bool few_chain_runs(const bnn_layer_desc* layers, int l, int n, int64_t M, const void* Y) {
    if (n == 0 || M > g_stream_max_frames.load() || g_default_arm.load() != BNN_ARM_MFMA) return false;
    const bnn_layer_desc& last = layers[l + n - 1];
    if (last.act == BNN_ACT_LOGSOFTMAX && !aligned(Y, 16)) return false;
    return apart(layers, l, n, M, Y);
}
// pulled: the launch in front has pulled the weights into the L2s.  Otherwise the run does, by workgroups of its own behind the others (64 frames
// of 6 x 512 and 6 x 1024 units 17.5 -> 16.7 us and 20.4 -> 18.3 a pass), where few_pulls says so.
static int run_few_chain(const bnn_layer_desc* layers, int l, int n, const void* X, int64_t M, void* Y, char* scratch_mem, hipStream_t st, bool pulled) {
    const FewScratch s = few_chain_scratch(layers, l, n, M);
    const int nr = few_chain_pieces(layers, l, n);
    FewArgs a{};
    a.F = ((int)M + kFewGroups - 1) / kFewGroups;
    bool vec = true;
    uint64_t* words = reinterpret_cast<uint64_t*>(scratch_mem);
    for (int j = 0; j < n; ++j) {
        const bnn_layer_desc& d = layers[l + j];
        FewLayer& f = a.layer[j];
        f = {static_cast<const uint32_t*>(d.Wp), d.scale, d.bias, words, (int)d.K, (int)d.N, (int)row_w32(d.K, d.word_bits), d.x_is_binary == 2, 0, 0, 0};
        f.blocks = (f.N + 31) / 32;
        f.per_block = (65536 + f.blocks - 1) / f.blocks;   // (exact for the 128 waves of a group)
        const int parts = max(1, min(a.F, kFewWaves * kFewSlots / f.blocks));
        f.f = (a.F + parts - 1) / parts;
        words += (size_t)M * (j < n - 1 ? 16 * nr : kFewMaxWords);
        vec = vec && f.w32 % 4 == 0 && aligned(d.Wp, 16);
    }
    const bnn_layer_desc& last = layers[l + n - 1];
    a.X = static_cast<const uint32_t*>(X);
    a.Y = Y;
    a.z = reinterpret_cast<float*>(scratch_mem + s.words);
    a.layers = n;
    a.M = (int)M;
    a.act = last.act;
    a.yw32 = (int)row_w32(last.N, last.word_bits);
    a.z_ld = (int)round_up((size_t)last.N, 2);
    a.spins = min(g_coop_spin.load(), 48);   // 15 to 20 us
    auto go = [&](auto nrc) {
        constexpr int NR = decltype(nrc)::value;
        const int grid = (few_pulls(NR) && !pulled ? 2 : 1) * kFewGroups * kFewSlots;
        if (vec) few_chain_kernel<NR, true><<<grid, kFewThreads, 0, st>>>(a);
        else few_chain_kernel<NR, false><<<grid, kFewThreads, 0, st>>>(a);
    };
    if (nr == 1) go(std::integral_constant<int, 1>{});
    else if (nr == 2) go(std::integral_constant<int, 2>{});
    else go(std::integral_constant<int, 4>{});
    return launch_status();
}

// The weights of a run, for the launch in front of it to pull into the L2s.
static Pull few_chain_pull(const bnn_layer_desc* layers, int l, int n, int64_t M) {
    Pull p{};
    for (int j = l; j < l + n; ++j) {
        p.at[p.layers] = static_cast<const char*>(layers[j].Wp);
        p.bytes[p.layers++] = (uint32_t)(layers[j].N * row_w32(layers[j].K, layers[j].word_bits) * 4);
    }
    p.xcds = (int)(M < kFewGroups ? M : kFewGroups);
    return p;
}

// Runs of equal Sign layers of a mid-size batch in one launch (hidden_run_kernel.hpp), inside bnn_forward: the layers from l on,
// behind a real-input Sign layer whose last launch clears the flags.  0: none.
// Passes back to back, 440 inputs, six hidden layers, 3400 outputs, one launch per layer -> this: 320 frames 42.0 -> 32.2 us (512
// units), 47.1 -> 34.4 (1024), 49.8 -> 38.4 (1536); 128 of 2048 51.4 -> 39.3; 1000 frames 45.1 -> 36.9 and 50.2 -> 41.1 (512, 1024).
// How many frames: alone, a run is faster far beyond these lines, and with four batches in flight that one thread launches one by one,
// too.  But where graphs or threads keep as many batches on the chip as the device has queues, the tiles of one launch per layer win with every
// fragment that a wave takes.  The lines are where that costs up to 8 %.  Alone, and a pass of four graphs at once: 512 units, 2048 frames
// 53.0 -> 46.5 and 22.7 -> 21.7, 3200 62.2 -> 56.0 and 32.6 -> 33.0 (at worst, eight layers and 100 outputs, 53.0 -> 41.9 and 22.5 -> 27.6); 1024 units,
// 1024 frames 49.6 -> 41.2 and 21.6 -> 20.0, but 1152 55.2 -> 45.3 and 21.6 -> 26.2; 1536 units, 320 frames 48.8 -> 37.7 and 17.2 -> 16.0, 512 47.2 ->
// 39.6 and 18.4 -> 19.6; 2048 units, 128 frames 50.6 -> 39.4 and 19.4 -> 16.4, but 200 53.3 -> 43.5 and 21.3 -> 23.3, 333 54.9 -> 47.0 and 21.5 -> 30.5.
static int hidden_run_layers(const bnn_layer_desc* layers, int n_layers, int l, int64_t M) {
    if (l < 1 || l >= n_layers || M <= kFewMaxFrames) return 0;
    const bnn_layer_desc& before = layers[l - 1];
    if (before.x_is_binary || before.w_is_real || !(l == 1 && realx_sign_mfma_applies(before) ? true : realx_i8_gemm_applies(before, M))) return 0;
    const int64_t N = layers[l].N;
    if (N % 512 != 0 || N > 2048 || M > (N == 512 ? 4096 : N == 1024 ? 1024 : N == 1536 ? 512 : 128)) return 0;
    int n = 0;
    while (l + n < n_layers && n < kRunMaxLayers && layers[l + n].x_is_binary && !layers[l + n].w_is_real && layers[l + n].act == BNN_ACT_SIGN &&
           layers[l + n].K == N && layers[l + n].N == N && aligned(layers[l + n].Wp, 16))
        ++n;
    return n >= 2 ? n : 0;
}
struct RunScratch {
    size_t flags, rows, total;   // all layers' flags; one layer's words (each but the last has its own); everything
};
static RunScratch hidden_run_scratch(int64_t N, int n, int64_t M) {
    RunScratch s{};
    s.flags = (size_t)n * kRunFlags * 4;
    s.rows = round_up((size_t)M * (size_t)(N / 8), 256);
    s.total = s.flags + (size_t)(n - 1) * s.rows;
    return s;
}
static bool hidden_run_runs(const bnn_layer_desc* layers, int l, int n, int64_t M, const void* Y) {
    if (n == 0 || M <= g_stream_max_frames.load() || g_default_arm.load() != BNN_ARM_MFMA || g_realx_sign_mfma.load() != 1 ||
        g_mfma_shape.load() != 0 || g_mfma32_wm.load() != 0 || g_mfma32_pipeline.load() == 2 || !aligned(Y, 16))
        return false;
    return apart(layers, l, n, M, Y);
}
static int run_hidden_run(const bnn_layer_desc* layers, int l, int n, const void* X, int64_t M, void* Y, char* scratch_mem, hipStream_t st) {
    const int64_t N = layers[l].N;
    const RunScratch s = hidden_run_scratch(N, n, M);
    RunArgs a{};
    for (int j = 0; j < n; ++j) {
        const bnn_layer_desc& d = layers[l + j];
        a.layer[j] = {static_cast<const uint32_t*>(d.Wp), d.scale, d.bias,
                      static_cast<uint32_t*>(j == n - 1 ? Y : static_cast<void*>(scratch_mem + s.flags + (size_t)j * s.rows)), d.x_is_binary == 2};
    }
    a.X = static_cast<const uint32_t*>(X);
    a.flags = reinterpret_cast<uint32_t*>(scratch_mem);
    a.layers = n;
    a.M = (int)M;
    a.F = 16 * (((int)M + 16 * kFewGroups - 1) / (16 * kFewGroups));
    a.spins = min(g_coop_spin.load(), 48);   // 15 to 20 us
    // fragments of a wave: up to 8 with 512 units, up to 2 with 1024, else 1; FM of them at a time
    const int per_wave = (a.F / 16 + kRunCrews - 1) / kRunCrews, passes = (per_wave + 3) / 4, fm = (per_wave + passes - 1) / passes;
    auto go = [&](auto nfc, auto fmc) {
        hidden_run_kernel<decltype(nfc)::value, decltype(fmc)::value><<<kFewGroups * kFewSlots, kRunThreads, 0, st>>>(a);
    };
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using I3 = std::integral_constant<int, 3>;
    using I4 = std::integral_constant<int, 4>;
    if (N == 512 && fm == 1) go(I1{}, I1{});
    else if (N == 512 && fm == 2) go(I1{}, I2{});
    else if (N == 512 && fm == 3) go(I1{}, I3{});
    else if (N == 512) go(I1{}, I4{});
    else if (N == 1024 && fm == 1) go(I2{}, I1{});
    else if (N == 1024) go(I2{}, I2{});
    else if (N == 1536) go(I3{}, I1{});
    else go(I4{}, I1{});
    return launch_status();
}

// Workspace layout of bnn_forward: two ping-pong buffers of `half` bytes, then `unpacked` bytes for the fp32 copy of
// the bits that a real-weight layer reads, or for the digit planes of a real-input Sign layer (whichever is larger).
// and, beyond what a call has to have, `few` bytes for runs of binary layers (used if they are there).
struct ForwardWorkspace {
    size_t half, unpacked, few;
    size_t needed() const { return 2 * half + unpacked; }
    size_t total() const { return needed() + few; }
};
// `roomy`: with the scratch of the tiled matrix-core products (the weight bytes and the list of realx_i8_gemm, the bf16
// planes of a Softmax layer with real weights); without it those layers run on the kernels that need less or none
// `callers`: a workspace of the caller's, with what is only reserved (realw_reserved_bytes)
static ForwardWorkspace forward_workspace(const bnn_layer_desc* layers, int n_layers, int64_t M, bool callers, bool roomy = true) {
    size_t biggest = 0, unpacked = 0, few = 0;
    for (int l = 0; l < n_layers; ++l) {
        if (const int n = few_chain_layers(layers, n_layers, l, M)) {
            const size_t b = few_chain_scratch(layers, l, n, M).total;
            if (b > few) few = b;
        }
        if (const int n = hidden_run_layers(layers, n_layers, l, M)) {
            const size_t b = hidden_run_scratch(layers[l].N, n, M).total;
            if (b > few) few = b;
        }
        if (l + 1 < n_layers) {
            const size_t b = out_bytes(M, layers[l].N, layers[l].act, layers[l].word_bits);
            if (b > biggest) biggest = b;
        }
        if (layers[l].w_is_real) {
            // unpacked binary input first, then the bf16 planes of both operands of a Softmax layer with real weights
            size_t b = layers[l].x_is_binary ? round_up((size_t)M * (size_t)layers[l].K * 4, 256) : 0;
            if (roomy && realw_split_lsm_applies(layers[l], M)) b += realw_split_lsm_bytes(M, layers[l].K, layers[l].N);
            if (callers && realw_reserved_applies(layers[l], M)) b += realw_reserved_bytes(layers[l].K, layers[l].N);
            if (b > unpacked) unpacked = b;
        }
        if (realx_i8_lsm_applies(layers[l], M)) {
            const size_t b = realx_i8_lsm_bytes(M, layers[l].K);
            if (b > unpacked) unpacked = b;
        }
        if (roomy && realx_i8_gemm_applies(layers[l], M) && !(l == 0 && realx_sign_mfma_applies(layers[l]))) {
            const size_t b = i8_gemm_scratch(M, layers[l].K, layers[l].N, layers[l].act).total;
            if (b > unpacked) unpacked = b;
        }
        // digit planes of a real-input Sign layer that the first-layer kernel does not take (same region: one layer at a time)
        if (realx_sign_slab_applies(layers[l]) && !(l == 0 && realx_sign_mfma_applies(layers[l]))) {
            const size_t b = realx_sign_slab_bytes(M, layers[l].K);
            if (b > unpacked) unpacked = b;
        }
    }
    return {round_up(biggest, 256), round_up(unpacked, 256), few};
}

BNN_EXPORT size_t bnn_forward_workspace_bytes(const bnn_layer_desc* layers, int n_layers, int64_t M) {
    if (check_chain(layers, n_layers, M) != BNN_OK) return 0;
    return forward_workspace(layers, n_layers, M, true).total();
}

// Scratch of bnn_forward_static: a fixed array in the library's device image (every GPU the library runs on holds its
// own copy at its own address until the process ends).  In host code the array's name is only a handle for
// hipGetSymbolAddress; kernels and copies get the device address that call returns.
constexpr size_t kStaticScratchBytes = (size_t)BNN_FORWARD_STATIC_MAX_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::atomic<void*> g_scratch_ptr[kMaxDevices];

// Device address of `scratch` on the current device, looked up once per device.
void* static_scratch() {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
        (void)hipGetLastError();
        return nullptr;
    }
    void* p = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (p) return p;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
        (void)hipGetLastError();
        return nullptr;
    }
    g_scratch_ptr[dev].store(p, std::memory_order_release);
    return p;
}
}  // namespace

static int forward_run(const bnn_layer_desc* layers, int n_layers, const void* X, int64_t M, void* out, void* workspace,
                       size_t workspace_bytes, void* stream, bool callers, bool roomy);

BNN_EXPORT int bnn_forward_static(const bnn_layer_desc* layers, int n_layers, const void* X, int64_t M, void* out,
                                  void* stream) {
    const int rc = check_chain(layers, n_layers, M);
    if (rc != BNN_OK) return rc;
    if (M == 0) return BNN_OK;
    // The scratch of the tiled matrix-core products (a byte per weight of a real-input layer, six bytes per weight of a
    // Softmax layer with real weights) is left out when it does not fit the array: those layers then run on the kernels
    // bnn_forward uses with these products switched off.
    bool roomy = true;
    ForwardWorkspace ws = forward_workspace(layers, n_layers, M, false);
    if (ws.needed() > kStaticScratchBytes) {
        roomy = false;
        ws = forward_workspace(layers, n_layers, M, false, false);
    }
    if (ws.needed() > kStaticScratchBytes) return BNN_EWORKSPACE;
    const size_t need = ws.total() > kStaticScratchBytes ? ws.needed() : ws.total();
    void* mem = nullptr;
    if (need) {
        mem = static_scratch();
        if (!mem) return BNN_EDEVICE;
    }
    return forward_run(layers, n_layers, X, M, out, mem, need, stream, false, roomy);
}

BNN_EXPORT int bnn_forward(const bnn_layer_desc* layers, int n_layers, const void* X, int64_t M, void* out,
                           void* workspace, size_t workspace_bytes, void* stream) {
    return forward_run(layers, n_layers, X, M, out, workspace, workspace_bytes, stream, true, true);
}

static int forward_run(const bnn_layer_desc* layers, int n_layers, const void* X, int64_t M, void* out, void* workspace,
                       size_t workspace_bytes, void* stream, bool callers, bool roomy) {
    int rc = check_chain(layers, n_layers, M);
    if (rc != BNN_OK) return rc;
    if (M == 0) return BNN_OK;
    if (!X || !out) return BNN_EINVAL;
    const ForwardWorkspace ws = forward_workspace(layers, n_layers, M, callers, roomy);
    const size_t need = ws.needed();
    if (need && (!workspace || workspace_bytes < need)) return BNN_EWORKSPACE;
    if (need && !aligned(workspace, 256)) return BNN_EALIGN;
    // Check every layer's arguments before anything is enqueued.
    char* buf[2] = {static_cast<char*>(workspace), static_cast<char*>(workspace) + ws.half};
    float* unpacked = reinterpret_cast<float*>(static_cast<char*>(workspace) + 2 * ws.half);
    char* few = ws.few && workspace_bytes >= ws.total() ? static_cast<char*>(workspace) + need : nullptr;
    hipStream_t st = static_cast<hipStream_t>(stream);
    for (int pass = 0; pass < 2; ++pass) {
        const void* in = X;
        for (int l = 0; l < n_layers; ++l) {
            const bnn_layer_desc& d = layers[l];
            auto output = [&](const void* input, int layer) -> void* { return layer == n_layers - 1 ? out : input == buf[0] ? buf[1] : buf[0]; };
            void* o = output(in, l);
            // a run of binary layers behind this one that takes a single launch: its marks are cleared by this layer's
            int run = 0;
            Front front;
            void* run_out = nullptr;
            if (pass == 1 && few) {
                const bool streaming = M <= kFewMaxFrames;
                run = streaming ? few_chain_layers(layers, n_layers, l + 1, M) : hidden_run_layers(layers, n_layers, l + 1, M);
                if (!streaming && !roomy && !(l == 0 && realx_sign_mfma_applies(d))) run = 0;   // (the layer in front runs on other kernels)
                run_out = output(o, l + run);
                if (run && (streaming ? few_chain_runs : hidden_run_runs)(layers, l + 1, run, M, run_out))
                    front.clear = {reinterpret_cast<uint4*>(few), (int)((streaming ? few_chain_scratch(layers, l + 1, run, M).words : hidden_run_scratch(d.N, run, M).flags) / 16), 0, 0};
                else
                    run = 0;
                if (run && streaming) front.pull = few_chain_pull(layers, l + 1, run, M);
            }
            Front* const f = run ? &front : nullptr;
            if (pass == 0) {
                if (d.w_is_real && d.x_is_binary) {
                    if (!aligned(in, d.word_bits / 8)) return BNN_EALIGN;
                    rc = check_layer_args(unpacked, d.Wp, M, d.K, d.N, d.act, d.word_bits, o, false, true);
                } else {
                    rc = check_layer_args(in, d.Wp, M, d.K, d.N, d.act, d.word_bits, o, d.x_is_binary != 0, d.w_is_real != 0);
                }
            } else if (d.w_is_real) {
                const float* xin = static_cast<const float*>(in);
                char* planes = reinterpret_cast<char*>(unpacked);
                if (d.x_is_binary) {
                    rc = run_unpack(in, M, d.K, d.word_bits, d.x_is_binary == 2, unpacked, st);
                    if (rc != BNN_OK) return rc;
                    xin = unpacked;
                    planes += round_up((size_t)M * (size_t)d.K * 4, 256);
                }
                if (roomy && realw_split_lsm_applies(d, M) && g_realw_split_lsm.load() && g_realx_f32_mfma.load() != 2 &&
                    M > g_stream_max_frames.load())
                    rc = run_realw_split_lsm(xin, static_cast<const float*>(d.Wp), d.bias, M, d.K, d.N,
                                             static_cast<float*>(o), planes, st);
                else
                    rc = run_realw(xin, static_cast<const float*>(d.Wp), d.bias, M, d.K, d.N, d.act, d.word_bits, o, st, f);
            } else if (d.x_is_binary) {
                rc = run_binx(in, d.Wp, d.scale, d.bias, M, d.K, d.N, d.act, d.word_bits, o, BNN_ARM_AUTO, st,
                              d.x_is_binary == 2);
            } else if (l == 0 && realx_sign_mfma_applies(d) && g_realx_sign_mfma.load() && M > g_stream_max_frames.load()) {
                rc = run_realx_sign_mfma(static_cast<const float*>(in), d.Wp, d.scale, d.bias, M, d.K, d.N, d.word_bits,
                                         o, st, f);
            } else if (roomy && realx_i8_gemm_applies(d, M) && M > g_stream_max_frames.load() &&
                       (d.act == BNN_ACT_SIGN ? g_realx_sign_mfma.load() == 1
                                              : (g_realx_i8_lsm.load() == 1 && g_realx_f32_mfma.load() != 2))) {
                rc = run_realx_i8_gemm(static_cast<const float*>(in), d.Wp, d.scale, d.bias, M, d.K, d.N, d.word_bits, d.act, o,
                                       unpacked, st, f);
            } else if (realx_i8_lsm_applies(d, M) && g_realx_i8_lsm.load() && g_realx_f32_mfma.load() != 2 &&
                       M > g_stream_max_frames.load()) {
                rc = run_realx_i8_lsm(static_cast<const float*>(in), d.Wp, d.scale, d.bias, M, d.K, d.N, d.word_bits,
                                      static_cast<float*>(o), unpacked, st);
            } else if (realx_sign_slab_applies(d) && g_realx_sign_mfma.load() && M > g_stream_max_frames.load()) {
                rc = run_realx_sign_slab(static_cast<const float*>(in), d.Wp, d.scale, d.bias, M, d.K, d.N, d.word_bits, o,
                                         unpacked, st);
            } else {
                rc = run_realx(static_cast<const float*>(in), d.Wp, d.scale, d.bias, M, d.K, d.N, d.act, d.word_bits, o,
                               st, f);
            }
            if (rc != BNN_OK) return rc;
            in = o;
            if (front.cleared) {
                rc = M <= kFewMaxFrames ? run_few_chain(layers, l + 1, run, in, M, run_out, few, st, front.pulled)
                                        : run_hidden_run(layers, l + 1, run, in, M, run_out, few, st);
                if (rc != BNN_OK) return rc;
                in = run_out;
                l += run;
            }
        }
    }
    return BNN_OK;
}
