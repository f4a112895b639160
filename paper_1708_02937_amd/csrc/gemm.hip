// Dense-W comparison arms: Z^T = W^T Y^T on the matrix cores with the bias and activation fused.
//
// This is the layer product with every zero of W_k stored explicitly, the dense-linear-algebra version
// the paper measures its sparse library against (Sec. V.A, V.B).  C (M x N) = A (M x K) B (K x N) with
// A = W_k^T (n_out x n_in), B = Y^T (n_in x batch, fp32), C = Y_{k+1}^T.
//
// Arithmetic.  fp64 arm: the fp32 operands are widened to fp64 (exactly) and multiplied on the fp64 matrix cores
// (v_mfma_f64_16x16x4_f64), so every product is exact and partial sums carry fp64 rounding only, the same
// arithmetic as the sparse paths; the epilogue adds b_j in fp64, applies h and rounds once to fp32.  fp32 arm: fp32
// operands and sums (v_mfma_f32_16x16x4_f32), the arithmetic of a single-precision BLAS.
//
// Layout.  A 16 x 16 x 4 matrix instruction takes element (row l % 16, k l / 16) from lane l, and which four k make
// up an instruction is free as long as both operands agree.  So K goes in blocks of 16, and lane group q = l / 16
// holds four of them: the four rows of C that the same lane group holds after a product (4 q + v in fp32, q + 4 v in
// fp64).  Activations are stored as [k block][q][sample][4 values] and W as [k block][q][output][4 values] (fp64: two
// halves of two): every global and LDS access is 16 bytes per lane and contiguous over lanes, one LDS read feeds four
// matrix instructions, and a product's output is one 16-byte store per 16 x 16 block in the layout the next layer
// reads.  K is padded with zeros to a multiple of 32 (W and activations), outputs to one of 128 (W); samples past the
// batch read the last one and are not stored.
//
// Tiling for CDNA4: a workgroup of eight wave64s computes a 128 x 64 tile of C, each wave a 32 x 32 part as 2 x 2
// blocks of 16 x 16 MFMAs.  Two workgroups share a CU (80 KiB of LDS each in fp64), so one's barrier and LDS waits are
// covered by the other's MFMAs.  K advances 32 at a time through double-buffered LDS (one barrier per step): the next
// slab is loaded into registers ahead of the current one's products and stored into the other buffer after them.
// MFMA-bound: the matrix cores are busy 78% (fp32) and 82% (fp64) of a launch at n 4096, batch 1024.  Measured on MI355X against
// k-major operands read 4 or 8 bytes per lane, 4 waves of 64 x 32, guarded element loads at ragged sizes (us per
// forward, before -> after): n 4096 batch 1024 L 2 fp32 603 -> 567, fp64 1069 -> 1069; n 1236 batch 906 L 2 fp32 198 ->
// 95; n 3001 batch 1001 fp64 526 -> 316; n 4096 batch 64 fp32 38.8 -> 34.9, fp64 53.5 -> 54.6 (with K split, n 1024 batch 512 to n 4096 batch
// 128 it is 2 to 4% above at a few sizes, in the product itself).  Not kept: four waves of
// 64 x 32 (fp64 1093), fragments read a part ahead with the barrier between the parts (fp32 571-582, fp64 1129-1157),
// 32 x 32 x 2 fp32 MFMAs (590), raised wave priority around the MFMAs (570), K steps of 16 in fp64 (1075).
//
// Small batches give few tiles (n = 4096, batch 64: 32 workgroups for 256 CUs), so K is then split over
// blockIdx.z: each split writes its partial tile, and a second kernel adds the splits in a fixed
// order, then the bias, h and the rounding.
#include <algorithm>

#include "common.h"

namespace sdnn {

namespace {

typedef double doublex4 __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef double doublex2 __attribute__((ext_vector_type(2)));

constexpr int BM = kGemmM, BN = kGemmN, BK = kGemmK, kKPad = kGemmKPad;
constexpr int kThreads = 512;  // 8 waves of 32 x 32 outputs

// Neuron of value v of lane group q in a block of 16.
template <typename T>
__host__ __device__ __forceinline__ int quad_neuron(int q, int v);
template <>
__host__ __device__ __forceinline__ int quad_neuron<float>(int q, int v) {
    return 4 * q + v;
}
template <>
__host__ __device__ __forceinline__ int quad_neuron<double>(int q, int v) {
    return q + 4 * v;
}

// ------------------------------------------------------------------------------------------ layout changes

// batch-major <-> [k block][q][sample][4], R samples x R neurons per workgroup through LDS (padded pitch): R = 64 moves
// whole 256-byte segments, 32 gives small batches enough workgroups (4096 neurons, 64 samples: 7.2 us at 64, 4.8 at 32)
// and more loads in flight on the way in (2048 neurons, 1024 samples: 8.5 us at 64, 5.6 at 32; the way out 5.5 at
// either).
template <typename T, int R>
__global__ __launch_bounds__(256) void to_quads_kernel(int64_t n, int64_t batch, const float *__restrict__ y,
                                                       float4 *__restrict__ yq) {
    __shared__ float tile[R][R + 1];
    const int64_t r0 = (int64_t)blockIdx.x * R, j0 = (int64_t)blockIdx.y * R;
    constexpr int kRows = 256 / R;
    const int lane = threadIdx.x % R, row = threadIdx.x / R;
#pragma unroll
    for (int rr = row; rr < R; rr += kRows) {
        const int64_t r = r0 + rr, j = j0 + lane;
        tile[rr][lane] = (r < batch && j < n) ? y[r * n + j] : 0.0f;
    }
    __syncthreads();
    const int64_t blocks = (n + kKPad - 1) / kKPad * (kKPad / BK);
#pragma unroll
    for (int u = row; u < R / 4; u += kRows) {
        const int64_t kb = j0 / BK + u / 4, r = r0 + lane;
        const int q = u % 4;
        if (r < batch && kb < blocks) {
            const float *t = &tile[lane][(u / 4) * BK];
            yq[(kb * 4 + q) * batch + r] = make_float4(t[quad_neuron<T>(q, 0)], t[quad_neuron<T>(q, 1)],
                                                       t[quad_neuron<T>(q, 2)], t[quad_neuron<T>(q, 3)]);
        }
    }
}

template <typename T, int R>
__global__ __launch_bounds__(256) void from_quads_kernel(int64_t n, int64_t batch, const float4 *__restrict__ yq,
                                                         float *__restrict__ y) {
    __shared__ float tile[R][R + 1];
    const int64_t r0 = (int64_t)blockIdx.x * R, j0 = (int64_t)blockIdx.y * R;
    constexpr int kRows = 256 / R;
    const int lane = threadIdx.x % R, row = threadIdx.x / R;
    const int64_t blocks = (n + kKPad - 1) / kKPad * (kKPad / BK);
#pragma unroll
    for (int u = row; u < R / 4; u += kRows) {
        const int64_t kb = j0 / BK + u / 4, r = r0 + lane;
        const int q = u % 4;
        if (r < batch && kb < blocks) {
            const float4 f = yq[(kb * 4 + q) * batch + r];
            float *t = &tile[lane][(u / 4) * BK];
            t[quad_neuron<T>(q, 0)] = f.x;
            t[quad_neuron<T>(q, 1)] = f.y;
            t[quad_neuron<T>(q, 2)] = f.z;
            t[quad_neuron<T>(q, 3)] = f.w;
        }
    }
    __syncthreads();
#pragma unroll
    for (int rr = row; rr < R; rr += kRows) {
        const int64_t r = r0 + rr, j = j0 + lane;
        if (r < batch && j < n) y[r * n + j] = tile[rr][lane];
    }
}

// W (i, j) in the operand layout: fp32 [k block][q][m][4]; fp64 [k block][half][q][m][2]
template <typename T>
__device__ __forceinline__ int64_t weight_index(int64_t i, int64_t j, int64_t mp);
template <>
__device__ __forceinline__ int64_t weight_index<float>(int64_t i, int64_t j, int64_t mp) {
    const int64_t kb = i / BK, k = i % BK;
    return ((kb * 4 + k / 4) * mp + j) * 4 + k % 4;
}
template <>
__device__ __forceinline__ int64_t weight_index<double>(int64_t i, int64_t j, int64_t mp) {
    const int64_t kb = i / BK, k = i % BK, v = k / 4;
    return (((kb * 2 + v / 2) * 4 + k % 4) * mp + j) * 2 + v % 2;
}

template <typename T>
__global__ void dense_weights_kernel(int64_t n, int64_t mp, const int64_t *__restrict__ fan_ptr,
                                     const Edge *__restrict__ fan, T *__restrict__ wk) {
    const int64_t j = blockIdx.x;
    for (int64_t e = fan_ptr[j] + threadIdx.x; e < fan_ptr[j + 1]; e += blockDim.x) {
        const Edge ed = fan[e];
        wk[weight_index<T>(ed.idx, j, mp)] = (T)ed.w;
    }
}

// ------------------------------------------------------------------------------------------ product

template <typename T>
struct Arm;
template <>
struct Arm<float> {
    using Acc = floatx4;
    using Unit = floatx4;                  // 16 bytes of W
    static constexpr int kHalves = 1;      // units per (q, m) and k block
    static __device__ __forceinline__ Acc mfma(float a, float b, Acc c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ float finish(float z, float bias, double ymax) {
        return activate((double)(z + bias), ymax);
    }
};
template <>
struct Arm<double> {
    using Acc = doublex4;
    using Unit = doublex2;
    static constexpr int kHalves = 2;
    static __device__ __forceinline__ Acc mfma(double a, double b, Acc c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ float finish(double z, float bias, double ymax) {
        return activate(z + (double)bias, ymax);
    }
};

// kc: k blocks per split.  C in the activation layout (blocks = k blocks of the layer), or this split's sums in the same
// order (fp64: two planes of two values) when partial is not null.
template <typename T>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4, 4))) void gemm_dense_layer_kernel(
    int64_t n, int64_t batch, int64_t mp, int64_t blocks, int64_t kc, const typename Arm<T>::Unit *__restrict__ W,
    const floatx4 *__restrict__ B, const float *__restrict__ bias, double ymax, float4 *__restrict__ C,
    T *__restrict__ partial) {
    using A = Arm<T>;
    using Unit = typename A::Unit;
    constexpr int kH = A::kHalves, kS = kKPad / BK;
    __shared__ __align__(16) Unit As[2][kS][kH][4][BM];
    __shared__ __align__(16) floatx4 Bs[2][kS][4][BN];
    constexpr int kUA = kS * kH * 4 * BM / kThreads;  // units of A per thread and step, and one of B
    static_assert(kS * 4 * BN == kThreads, "one unit of B per thread");

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    // blockIdx.x walks M: consecutive workgroups (dealt round-robin to the XCDs) take different column
    // blocks of W, and the batch blocks of one of them land on one XCD and share it in its L2.
    const int64_t m0 = (int64_t)blockIdx.x * BM, n0 = (int64_t)blockIdx.y * BN;
    const int64_t kb = (int64_t)blockIdx.z * kc, ke = min(blocks, kb + kc);  // multiples of kS

    Unit ra[kUA];
    floatx4 rb;
    const int bm = tid % BM, bt = tid / BM;  // unit u of A: (step, half, q) 4 u + bt, output bm
    const int64_t br = min(batch - 1, n0 + tid % BN);
    const int bq = tid / BN;  // B: (step, q) bq
    auto load = [&](int64_t k) {
#pragma unroll
        for (int u = 0; u < kUA; ++u) ra[u] = W[(k * kH * 4 + (kThreads / BM) * u + bt) * mp + m0 + bm];
        rb = B[(k * 4 + bq) * batch + br];
    };
    auto store = [&](int buf) {
        Unit *a = &As[buf][0][0][0][0];
        floatx4 *b = &Bs[buf][0][0][0];
#pragma unroll
        for (int u = 0; u < kUA; ++u) a[u * kThreads + tid] = ra[u];
        b[tid] = rb;
    };

    typename A::Acc acc[2][2];
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int ni = 0; ni < 2; ++ni) acc[mi][ni] = typename A::Acc{0, 0, 0, 0};

    const int rc = lane & 15, q = lane >> 4;
    auto compute = [&](int cur) {
#pragma unroll
        for (int st = 0; st < kS; ++st) {
            // the first half of every fragment first: the products over it start while the rest is on its way
            Unit ua[kH][2];
            floatx4 ub[2];
#pragma unroll
            for (int ni = 0; ni < 2; ++ni) ub[ni] = Bs[cur][st][q][wn * 32 + ni * 16 + rc];
#pragma unroll
            for (int h = 0; h < kH; ++h)
#pragma unroll
                for (int mi = 0; mi < 2; ++mi) ua[h][mi] = As[cur][st][h][q][wm * 32 + mi * 16 + rc];
            T a[2][4], b[2][4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
#pragma unroll
                for (int mi = 0; mi < 2; ++mi) a[mi][v] = ua[v * kH / 4][mi][v % (4 / kH)];
#pragma unroll
                for (int ni = 0; ni < 2; ++ni) b[ni][v] = (T)ub[ni][v];
            }
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int mi = 0; mi < 2; ++mi)
#pragma unroll
                    for (int ni = 0; ni < 2; ++ni) acc[mi][ni] = A::mfma(a[mi][v], b[ni][v], acc[mi][ni]);
        }
    };

    load(kb);
    store(0);
    __syncthreads();
    int cur = 0;
    for (int64_t k = kb + kS; k < ke; k += kS) {
        load(k);
        __builtin_amdgcn_sched_barrier(0);  // the loads stay ahead of the products
        compute(cur);
        store(cur ^ 1);  // last read one step earlier, before the barrier
        cur ^= 1;
        __syncthreads();
    }
    compute(cur);

#pragma unroll
    for (int mi = 0; mi < 2; ++mi) {
        const int64_t mb = (m0 + wm * 32) / BK + mi;  // the block of 16 outputs is the next layer's k block
        if (mb >= blocks) continue;
        float bv[4];
        bool real[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int64_t m = mb * BK + quad_neuron<T>(q, v);
            real[v] = m < n;
            bv[v] = real[v] && !partial ? bias[m] : 0.0f;
        }
#pragma unroll
        for (int ni = 0; ni < 2; ++ni) {
            const int64_t r = n0 + wn * 32 + ni * 16 + rc;
            if (r >= batch) continue;
            const int64_t at = (mb * 4 + q) * batch + r;
            if (partial) {
                Unit *p = reinterpret_cast<Unit *>(partial) + (int64_t)blockIdx.z * kH * blocks * 4 * batch + at;
#pragma unroll
                for (int h = 0; h < kH; ++h) {
                    Unit u;
#pragma unroll
                    for (int v = 0; v < 4 / kH; ++v) u[v] = acc[mi][ni][h * (4 / kH) + v];
                    p[h * blocks * 4 * batch] = u;
                }
            } else {
                float f[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) f[v] = real[v] ? A::finish(acc[mi][ni][v], bv[v], ymax) : 0.0f;
                C[at] = make_float4(f[0], f[1], f[2], f[3]);
            }
        }
    }
}

// Sum of the K splits in split order, then the bias, h and one rounding.
template <typename T>
__global__ __launch_bounds__(256) void gemm_reduce_kernel(int64_t n, int64_t batch, int64_t blocks, int splits,
                                                          const T *__restrict__ partial, const float *__restrict__ bias,
                                                          double ymax, float4 *__restrict__ C) {
    const int64_t at = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, count = blocks * 4 * batch;
    if (at >= count) return;
    constexpr int kH = Arm<T>::kHalves;
    T z[4] = {0, 0, 0, 0};
#pragma unroll 4
    for (int sp = 0; sp < splits; ++sp) {
#pragma unroll
        for (int h = 0; h < kH; ++h) {
            const auto u = reinterpret_cast<const typename Arm<T>::Unit *>(partial)[(sp * kH + h) * count + at];
#pragma unroll
            for (int v = 0; v < 4 / kH; ++v) z[h * (4 / kH) + v] += u[v];
        }
    }
    const int64_t mb = at / (4 * batch);
    const int q = (int)(at / batch % 4);
    float f[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int64_t m = mb * BK + quad_neuron<T>(q, v);
        f[v] = m < n ? Arm<T>::finish(z[v], bias[m], ymax) : 0.0f;
    }
    C[at] = make_float4(f[0], f[1], f[2], f[3]);
}

template <typename T>
hipError_t launch_weights(int64_t n, const int64_t *fan_ptr, const Edge *fan, T *wt, hipStream_t s) {
    hipError_t e = hipMemsetAsync(wt, 0, gemm_weight_elems(n) * sizeof(T), s);
    if (e != hipSuccess) return e;
    dense_weights_kernel<T><<<(unsigned)n, 256, 0, s>>>(n, gemm_m_pitch(n), fan_ptr, fan, wt);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_gemm(int64_t n, int64_t batch, const T *wt, const float *bias, double ymax, const float *yq, float *zq,
                       T *partial, int splits, hipStream_t s) {
    if (n == 0 || batch == 0) return hipSuccess;
    const int64_t gx = (n + BM - 1) / BM, gy = (batch + BN - 1) / BN, blocks = gemm_k_blocks(n);
    if (gx > 0x7fffffffLL || gy > 65535) return hipErrorInvalidValue;
    // split length in whole K steps; the last split may be shorter, none is empty
    const int64_t steps = blocks / (kKPad / BK);
    const int64_t kc = (steps + splits - 1) / splits * (kKPad / BK);
    const int sp = (int)((blocks + kc - 1) / kc);
    T *part = sp > 1 ? partial : nullptr;
    const dim3 grid((unsigned)gx, (unsigned)gy, (unsigned)sp);
    gemm_dense_layer_kernel<T><<<grid, kThreads, 0, s>>>(n, batch, gemm_m_pitch(n), blocks, kc,
                                        reinterpret_cast<const typename Arm<T>::Unit *>(wt),
                                        reinterpret_cast<const floatx4 *>(yq), bias, ymax, reinterpret_cast<float4 *>(zq),
                                        part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || sp == 1) return e;
    gemm_reduce_kernel<T><<<(unsigned)((blocks * 4 * batch + 255) / 256), 256, 0, s>>>(
        n, batch, blocks, sp, partial, bias, ymax, reinterpret_cast<float4 *>(zq));
    return hipGetLastError();
}

}  // namespace

hipError_t launch_dense_from_fanin(int64_t n, const int64_t *fan_ptr, const Edge *fan, double *wt, hipStream_t s) {
    return launch_weights<double>(n, fan_ptr, fan, wt, s);
}
hipError_t launch_dense32_from_fanin(int64_t n, const int64_t *fan_ptr, const Edge *fan, float *wt, hipStream_t s) {
    return launch_weights<float>(n, fan_ptr, fan, wt, s);
}

hipError_t launch_gemm_dense_layer(int64_t n, int64_t batch, const double *wt, const float *bias, double ymax,
                                   const float *yq, float *zq, double *partial, int splits, hipStream_t s) {
    return launch_gemm<double>(n, batch, wt, bias, ymax, yq, zq, partial, splits, s);
}
hipError_t launch_gemm32_dense_layer(int64_t n, int64_t batch, const float *wt, const float *bias, double ymax,
                                     const float *yq, float *zq, float *partial, int splits, hipStream_t s) {
    return launch_gemm<float>(n, batch, wt, bias, ymax, yq, zq, partial, splits, s);
}

namespace {

template <typename T>
hipError_t launch_quads(int64_t n, int64_t batch, bool to, const float *in, float *out, hipStream_t s) {
    const int64_t R = n * batch <= (int64_t(1) << (to ? 24 : 20)) ? 32 : 64, cols = to ? gemm_k_blocks(n) * BK : n;
    const dim3 grid((unsigned)((batch + R - 1) / R), (unsigned)((cols + R - 1) / R));
    if ((cols + R - 1) / R > 65535) return hipErrorInvalidValue;
    if (to && R == 32)
        to_quads_kernel<T, 32><<<grid, 256, 0, s>>>(n, batch, in, reinterpret_cast<float4 *>(out));
    else if (to)
        to_quads_kernel<T, 64><<<grid, 256, 0, s>>>(n, batch, in, reinterpret_cast<float4 *>(out));
    else if (R == 32)
        from_quads_kernel<T, 32><<<grid, 256, 0, s>>>(n, batch, reinterpret_cast<const float4 *>(in), out);
    else
        from_quads_kernel<T, 64><<<grid, 256, 0, s>>>(n, batch, reinterpret_cast<const float4 *>(in), out);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_to_quads(int64_t n, int64_t batch, bool f64, const float *y, float *yq, hipStream_t s) {
    return f64 ? launch_quads<double>(n, batch, true, y, yq, s) : launch_quads<float>(n, batch, true, y, yq, s);
}
hipError_t launch_from_quads(int64_t n, int64_t batch, bool f64, const float *yq, float *y, hipStream_t s) {
    return f64 ? launch_quads<double>(n, batch, false, yq, y, s) : launch_quads<float>(n, batch, false, yq, y, s);
}

}  // namespace sdnn
