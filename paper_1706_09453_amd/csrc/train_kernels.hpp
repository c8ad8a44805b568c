// Training-side kernels (paper Alg. 1 and Alg. 2, backward propagation and update; Sec. 2.1-2.3).
//
// The two matrix products of the backward pass are the forward products with the operands' roles exchanged and run
// on the forward kernels:
//   g_{h_{l-1}} = g_{h^_l} w^b_l      realx kernels on the TRANSPOSED packed signs (pack_sign_transposed_kernel below)
//   g_{w_l}     = g_{h^_l}^T h_{l-1}  realw kernels on the two transposed operands (transpose_f32_kernel below)
// so their sums run in ascending n and ascending frame m, one accumulator per result.  What is here are the remaining
// steps: the transposes, the gradient through the Softmax/cross-entropy and through the binarisation layer (Mask),
// the bias gradient, the clipped update, gradient-norm clipping and the semi-stochastic binarisation.
#pragma once

#include <type_traits>

#include "bnn_device.hpp"

namespace bnn {

// WpT[k][n / 32] bit (n % 32) = (W[n][k] > 0): the signs of W^T, packed along n.  A lane owns one column k and walks 64
// rows n: every row is read coalesced along k, 32 requests in flight, and the lane's two words need no exchange with other
// lanes.  (Bound by memory: 4096 x 2048 numbers in 10.6 us; through a 64 x 64 tile in LDS with one ballot per output word it
// took 15.)  Pad bits (n >= N) are 0.  Grid: x = ceil(K / 256), y = ceil(N / 64).
__global__ __launch_bounds__(256) void pack_sign_transposed_kernel(const float* __restrict__ W, int N, int K, int w32t,
                                                                   uint32_t* __restrict__ WpT) {
    const int k = (int)blockIdx.x * 256 + (int)threadIdx.x, n0 = (int)blockIdx.y * 64;
    if (k >= K) return;
    uint32_t words[2] = {0u, 0u};
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        float v[32];
#pragma unroll
        for (int i = 0; i < 32; ++i) v[i] = W[(size_t)min(n0 + 32 * h + i, N - 1) * K + k];
#pragma unroll
        for (int i = 0; i < 32; ++i) words[h] |= (n0 + 32 * h + i < N && sign_bit(v[i])) ? 1u << i : 0u;
    }
    uint32_t* row = WpT + (size_t)k * w32t + (n0 >> 5);
    if ((w32t & 1) == 0 && (reinterpret_cast<uintptr_t>(WpT) & 7) == 0) {   // (n0 / 32 is even)
        *reinterpret_cast<uint2*>(row) = make_uint2(words[0], words[1]);
    } else {
        row[0] = words[0];
        if ((n0 >> 5) + 1 < w32t) row[1] = words[1];
    }
}

// out[c][r] = A[r][c], 64 x 64 tiles through LDS, both sides coalesced.  Bound by memory, small matrices by its latency: all
// sixteen rows of a wave are requested before the first is used (4096 x 2048 13.0 -> 10.8 us, 256 x 2048 8.1 -> 4.1).
// Grid: x = ceil(C / 64), y = ceil(R / 64).
__global__ __launch_bounds__(256) void transpose_f32_kernel(const float* __restrict__ A, int R, int C, float* __restrict__ out) {
    __shared__ float tile[64][65];
    const int c0 = (int)blockIdx.x * 64, r0 = (int)blockIdx.y * 64;
    const int wave = (int)threadIdx.x >> 6, lane = lane_id();
    float v[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) v[j] = A[(size_t)min(r0 + wave + 4 * j, R - 1) * C + min(c0 + lane, C - 1)];   // (past the edge: unused)
#pragma unroll
    for (int j = 0; j < 16; ++j) tile[wave + 4 * j][lane] = v[j];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const int c = wave + 4 * j;
        if (c0 + c < C && r0 + lane < R) out[(size_t)(c0 + c) * R + r0 + lane] = tile[lane][c];
    }
}

// f(e, n) for every element: n = 4 consecutive ones at a time (VEC: 16-byte accesses; the arrays are 16-byte aligned),
// the last count % 4 one by one.  These kernels are bound by memory: 16 bytes per lane and access, four accesses of a
// thread in flight.
template <bool VEC, class F>
__device__ __forceinline__ void for_each_element(int64_t count, F&& f) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x, stride = (int64_t)gridDim.x * 256;
    if constexpr (VEC) {
        const int64_t quads = count >> 2;
        for (int64_t i = t; i < quads; i += stride) f(4 * i, std::integral_constant<int, 4>{});
        if (t < (count & 3)) f(4 * quads + t, std::integral_constant<int, 1>{});
    } else {
        for (int64_t e = t; e < count; e += stride) f(e, std::integral_constant<int, 1>{});
    }
}
template <int N>
struct Few { float v[N]; };
template <int N>
__device__ __forceinline__ Few<N> load_few(const float* p, std::integral_constant<int, N>) {
    Few<N> r;
    if constexpr (N == 4) {
        const float4 q = *reinterpret_cast<const float4*>(p);
        r.v[0] = q.x; r.v[1] = q.y; r.v[2] = q.z; r.v[3] = q.w;
    } else {
        r.v[0] = *p;
    }
    return r;
}
template <int N>
__device__ __forceinline__ void store_few(float* p, const Few<N>& r) {
    if constexpr (N == 4) *reinterpret_cast<float4*>(p) = make_float4(r.v[0], r.v[1], r.v[2], r.v[3]);
    else *p = r.v[0];
}

// Alg. 1/2: gradient of the summed cross entropy through the Softmax layer, g[m][n] = exp(logp[m][n]) - (n == label[m]),
// evaluated in fp64 from the fp32 log-posteriors and rounded once.  g may be logp itself.  VEC: N % 4 == 0, arrays 16-byte
// aligned.
__device__ __forceinline__ float softmax_xent_grad_of(float logp, bool is_label) {
    const float z = logp < -1000.0f ? -1000.0f : (logp > 1000.0f ? 1000.0f : logp);   // exp is 0 / inf beyond
    const double p = exp_f64((double)z);
    return (float)(is_label ? p - 1.0 : p);
}

// Many frames of many classes: a workgroup takes whole frames.
template <bool VEC>
__global__ __launch_bounds__(256) void softmax_xent_grad_rows_kernel(const float* logp, const int32_t* __restrict__ labels,
                                                                     int64_t M, int N, float* g) {
    const std::integral_constant<int, VEC ? 4 : 1> few;
    for (int64_t m = blockIdx.x; m < M; m += gridDim.x) {
        const int label = labels[m];
#pragma unroll 4
        for (int n = (int)threadIdx.x * few.value; n < N; n += 256 * few.value) {
            Few<few.value> r = load_few(logp + m * N + n, few);
#pragma unroll
            for (int i = 0; i < few.value; ++i) r.v[i] = softmax_xent_grad_of(r.v[i], n + i == label);
            store_few(g + m * N + n, r);
        }
    }
}

// Any other shape: threads take elements (VEC: four consecutive ones, all of one frame) of the whole matrix and find the
// frame by a division.  With a workgroup per frame, few classes leave its threads and few frames the chip idle.
// I: type that holds M N.
template <bool VEC, class I>
__global__ __launch_bounds__(256) void softmax_xent_grad_kernel(const float* logp, const int32_t* __restrict__ labels,
                                                                int64_t M, int N, float* g) {
    for_each_element<VEC>(M * N, [&](int64_t e, auto few) {
        const I m = (I)e / (I)N;
        const int n = (int)((I)e - m * (I)N), label = labels[m];
        auto r = load_few(logp + e, few);
#pragma unroll
        for (int i = 0; i < few.value; ++i) r.v[i] = softmax_xent_grad_of(r.v[i], n + i == label);
        store_few(g + e, r);
    });
}

// Sec. 2.2: g_{h^} = g_h (.) Mask(h^, k); Mask = 0 where |h^| > k, 1 otherwise.  out may be g_h itself.
template <bool VEC>
__global__ __launch_bounds__(256) void mask_grad_kernel(const float* g_h, const float* __restrict__ hhat, int64_t count, float k, float* out) {
    for_each_element<VEC>(count, [&](int64_t e, auto n) {
        auto g = load_few(g_h + e, n);
        const auto h = load_few(hhat + e, n);
#pragma unroll
        for (int i = 0; i < n.value; ++i) g.v[i] = __builtin_fabsf(h.v[i]) > k ? 0.0f : g.v[i];
        store_few(out + e, g);
    });
}

// Alg. 1 backward through a Sigmoid layer: g_{h^} = g_h * (h * (1 - h)) with h the layer's output, every operation
// rounded in fp32 (no contraction: the library is built with -ffp-contract=off).  out may be g_h itself.
template <bool VEC>
__global__ __launch_bounds__(256) void sigmoid_grad_kernel(const float* g_h, const float* __restrict__ h, int64_t count, float* out) {
    for_each_element<VEC>(count, [&](int64_t e, auto n) {
        auto g = load_few(g_h + e, n);
        const auto v = load_few(h + e, n);
#pragma unroll
        for (int i = 0; i < n.value; ++i) {
            const float d = v.v[i] * (1.0f - v.v[i]);
            g.v[i] = g.v[i] * d;
        }
        store_few(out + e, g);
    });
}

// g_r[n] = sum_m g[m][n] in fp32, ascending m, one accumulator per n.  The sum of a column is a chain of M dependent
// additions; what there is to gain is that the chain never waits for memory and that the chip reads the matrix with enough
// requests in flight: a workgroup of four waves takes 16 columns, all of it brings slabs of 256 rows into LDS (two
// buffers, the next slab in registers meanwhile), 16 lanes of its first wave add.  4096 x 2048: 63 -> 18 us against one
// wave per 64 columns that loads and adds by itself.  VEC: N % 4 == 0, g 16-byte aligned.  Grid: ceil(N / 16).
// In LDS a column's rows lie side by side, so the adding lanes read four rows at a time, 32 rows ahead of the additions
// (a lone wave issues one vector instruction per 2.6 ns, and the chain should be all it issues).
constexpr int kColsumRows = 256, kColsumCols = 16, kColsumLd = kColsumRows + 4;
constexpr int64_t kColsumMaxCols = 3 * 256 * kColsumCols;   // wider matrices: colsum_wave_kernel
template <bool VEC>
__global__ __launch_bounds__(256) void colsum_kernel(const float* __restrict__ g, int M, int N, float* __restrict__ out) {
    __shared__ __attribute__((aligned(16))) float slab[2][kColsumCols][kColsumLd];
    const int tid = (int)threadIdx.x, row = tid >> 2, col = 4 * (tid & 3);
    const int n0 = (int)blockIdx.x * kColsumCols;
    float4 next[4];
    auto request = [&](int s) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float* p = g + (size_t)min(s * kColsumRows + row + 64 * j, M - 1) * N + n0 + col;
            if constexpr (VEC) {
                next[j] = *reinterpret_cast<const float4*>(n0 + col < N ? p : p - col);   // (columns past N: any value)
            } else {
                const int last = N - 1 - n0 - col;
                next[j] = make_float4(p[min(0, last)], p[min(1, last)], p[min(2, last)], p[min(3, last)]);
            }
        }
    };
    auto deposit = [&](int s) {   // rows past M: +0, which leaves a sum that started at +0 as it is
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool in = s * kColsumRows + row + 64 * j < M;
            float (*t)[kColsumLd] = &slab[s & 1][col];
            t[0][row + 64 * j] = in ? next[j].x : 0.0f;
            t[1][row + 64 * j] = in ? next[j].y : 0.0f;
            t[2][row + 64 * j] = in ? next[j].z : 0.0f;
            t[3][row + 64 * j] = in ? next[j].w : 0.0f;
        }
    };
    const int slabs = (M + kColsumRows - 1) / kColsumRows;
    float sum = 0.0f;
    if (slabs > 0) {   // (no frames: the sums are 0)
        request(0);
        deposit(0);
    }
    __syncthreads();
    for (int s = 0; s < slabs; ++s) {
        if (s + 1 < slabs) request(s + 1);   // workgroup-uniform
        if (tid < kColsumCols) {
            const float* t = slab[s & 1][tid];
            float4 a[8], b[8];
            auto read = [&](float4 (&v)[8], int m) {
#pragma unroll
                for (int i = 0; i < 8; ++i) v[i] = *reinterpret_cast<const float4*>(t + m + 4 * i);
            };
            auto add = [&](const float4 (&v)[8]) {
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    sum = sum + v[i].x;
                    sum = sum + v[i].y;
                    sum = sum + v[i].z;
                    sum = sum + v[i].w;
                }
            };
            read(a, 0);
#pragma unroll
            for (int m = 0; m < kColsumRows; m += 64) {
                read(b, m + 32);
                __builtin_amdgcn_sched_barrier(0);
                add(a);
                if (m + 64 < kColsumRows) read(a, m + 64);
                __builtin_amdgcn_sched_barrier(0);
                add(b);
            }
        }
        if (s + 1 < slabs) deposit(s + 1);   // that buffer was last read before the previous barrier
        __syncthreads();
    }
    if (tid < kColsumCols && n0 + tid < N) out[n0 + tid] = sum;
}

// The same sums, one wave per 64 columns (lanes <-> n: every row is read coalesced, 32 rows requested at a time, the
// additions in order).  Where the columns alone fill the chip the slabs' way through LDS only costs: the
// rule is in bnn_bias_grad.  Grid: ceil(N / 64), one wave per workgroup.
__global__ __launch_bounds__(kWave) void colsum_wave_kernel(const float* __restrict__ g, int M, int N, float* __restrict__ out) {
    const int n = (int)blockIdx.x * kWave + (int)threadIdx.x;
    if (n >= N) return;
    float s = 0.0f;
    int m = 0;
    for (; m + 32 <= M; m += 32) {
        float v[32];
#pragma unroll
        for (int i = 0; i < 32; ++i) v[i] = g[(size_t)(m + i) * N + n];
#pragma unroll
        for (int i = 0; i < 32; ++i) s = s + v[i];
    }
    for (; m < M; ++m) s = s + g[(size_t)m * N + n];
    out[n] = s;
}

// Alg. 1 Update: w <- Clip(w - eta g) with Clip to [-1, +1] (Sec. 2.1); clip == 0: the plain update.  One fma.
template <bool VEC>
__global__ __launch_bounds__(256) void update_clip_kernel(float* __restrict__ w, const float* __restrict__ g, int64_t count,
                                                          float eta, int clip) {
    for_each_element<VEC>(count, [&](int64_t e, auto n) {
        auto v = load_few(w + e, n);
        const auto d = load_few(g + e, n);
#pragma unroll
        for (int i = 0; i < n.value; ++i) {
            v.v[i] = __builtin_fmaf(-eta, d.v[i], v.v[i]);
            if (clip) {
                v.v[i] = v.v[i] > 1.0f ? 1.0f : v.v[i];
                v.v[i] = v.v[i] < -1.0f ? -1.0f : v.v[i];
            }
        }
        store_few(w + e, v);
    });
}

// Sec. 2.3, gradient-norm clipping, in launches whose order of additions is fixed (reproducible bit for bit):
// 256 workgroups each sum the squares of a fixed strided subset in fp64 (four sums per thread, one per element of a
// 16-byte piece, then a tree over LDS) ...
constexpr int kSumsqBlocks = 256, kSumsqThreads = 1024;
template <bool VEC>
__global__ __launch_bounds__(kSumsqThreads) void sumsq_partial_kernel(const float* __restrict__ g, int64_t count, double* __restrict__ partial) {
    __shared__ double part[kSumsqThreads];
    const int64_t t = (int64_t)blockIdx.x * kSumsqThreads + threadIdx.x, stride = (int64_t)kSumsqBlocks * kSumsqThreads;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    const int64_t quads = count >> 2;
#pragma unroll 4
    for (int64_t i = t; i < quads; i += stride) {
        float v[4];
        if constexpr (VEC) {
            const float4 q = *reinterpret_cast<const float4*>(g + 4 * i);
            v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = g[4 * i + j];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) s[j] = __builtin_fma((double)v[j], (double)v[j], s[j]);   // (the product is exact in fp64)
    }
    if (t < (count & 3)) {
        const double v = (double)g[4 * quads + t];
        s[0] = __builtin_fma(v, v, s[0]);
    }
    part[threadIdx.x] = (s[0] + s[1]) + (s[2] + s[3]);
    __syncthreads();
    for (int width = kSumsqThreads / 2; width > 0; width >>= 1) {
        if ((int)threadIdx.x < width) part[threadIdx.x] += part[threadIdx.x + width];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = part[0];
}
// ... then the 256 partial sums are added, in one and the same order wherever that is done ...
__device__ __forceinline__ float norm_of_partials(const double* partial) {
    const int lane = lane_id();
    static_assert(kSumsqBlocks == 4 * kWave, "four partial sums per lane");
    double sum = (partial[lane] + partial[lane + 64]) + (partial[lane + 128] + partial[lane + 192]);
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) sum += __shfl_xor(sum, d, kWave);
    return (float)sqrt(sum);
}
// ... by one wave in a launch of its own where norm_out lies among the partial sums (nothing may read them once it is stored) ...
__global__ __launch_bounds__(kWave) void sumsq_final_kernel(const double* partial, float* norm_out) {
    const float nrm = norm_of_partials(partial);
    if (threadIdx.x == 0) norm_out[0] = nrm;
}
// ... otherwise by every wave of the second launch (a third of a microsecond instead of a launch), the first one storing
// ||g||_2 as fp32; and every element is multiplied by alpha / ||g||_2 if the norm is above alpha.  partial: nullptr if
// norm_out holds the norm already.
template <bool VEC>
__global__ __launch_bounds__(256) void scale_if_above_kernel(float* __restrict__ g, int64_t count, float alpha,
                                                             const double* __restrict__ partial, float* __restrict__ norm_out) {
    const float nrm = partial ? norm_of_partials(partial) : norm_out[0];
    if (partial && blockIdx.x == 0 && threadIdx.x == 0) norm_out[0] = nrm;
    if (!(nrm > alpha)) return;
    const float factor = alpha / nrm;
    for_each_element<VEC>(count, [&](int64_t e, auto n) {
        auto v = load_few(g + e, n);
#pragma unroll
        for (int i = 0; i < n.value; ++i) v.v[i] = v.v[i] * factor;
        store_few(g + e, v);
    });
}

// Sec. 2.1 (Alg. 1 Update, optional step): w <- Sign(w) where the given draw u in [0, 1) is below p(|w|) = |w|.
__global__ __launch_bounds__(256) void semi_stochastic_kernel(float* __restrict__ w, const float* __restrict__ u, int64_t count) {
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < count; e += (int64_t)gridDim.x * 256) {
        const float v = w[e];
        if (u[e] < __builtin_fabsf(v)) w[e] = v > 0.0f ? 1.0f : -1.0f;
    }
}

}  // namespace bnn
