// Dense-Y forward with the activations of a few samples resident in LDS (Sec. III batched inference equation;
// Sec. IV loop body), for layers of at most 5119 neurons.  (Layers of 4097 neurons on with short lists at batch 256 and
// more run on the sample-blocked layout, whose choice is made first.)
//
// A workgroup (16 wave64s, one per CU) owns V samples (4, 2 or 1) and keeps all n activations of them in LDS as
// rows of V floats, one row per neuron; a lane owns one output neuron, walks its fan-in list in ascending input
// order, reads the input's row (one LDS read of V floats) and adds the V exact products to its fp64 sums (or folds
// them over another semiring of Sec. II, one layer without bias and activation).  The bias, h and the rounding follow,
// and the outputs form the next layer's rows in a second LDS buffer, so a whole range of layers is one launch: the
// batch is read once, batch-major, and written once, and nothing else of it touches memory.
//
// What bounds it: at V = 4 LDS (64 lanes reading random 16-byte rows; the LDS pipe is busy 75% of the time, two
// thirds of that bank conflicts) and VALU issue (44 instructions per block of 4 x 64 entries, 36 of them the
// conversions and fp64 multiply-adds, issuing 75-80% of the time) together; below that the list stream from L2.  The
// neuron-major gather it replaces at these widths moves 4 bytes per product through the L1 from L2, and pays two
// transposes and a launch per layer.  Measured on MI355X (before -> after): n 4096, two layers of 10%, batch 1024 490 -> 343 us; four
// layers of 1%, batch 1021 262 -> 88 us; n 2999, six layers of 32 entries, batch 777 282 -> 82 us; n 1024, four
// layers of 16 entries, batch 64 25.3 -> 11.5 us (on lists used before: the first call on a net is 36.5 against 49.5
// us for the last, and one layer of 4096 neurons, 64 entries, batch 64 37.5 against 39.7, 9.6 against 17.2 later).  Lists two, three or four blocks ahead: 363, 352, 351 us on the
// first of these, 80.8, 81.9, 83.2 on the third.
//
// Lists.  Set-up sorts each run of 1024 neurons by list length and cuts it into 16 slices of 64 (one lane per
// neuron).  A slice holds its lists interleaved, in blocks of four entries per lane: 64 x 4 input indices of 16
// bits, then 64 x 4 fp32 weights (1536 bytes, read with one 8-byte and one 16-byte load per lane, 6 bytes per
// entry).  Lists are padded to their slice's longest with entries of weight 0 at input n, a row that holds
// zeros, which leave a sum as it is.
#include <algorithm>

#include "common.h"

namespace sdnn {

namespace {

constexpr int kRThreads = 1024;
constexpr int kRWaves = kRThreads / 64;
constexpr int kRunLen = 1024;             // neurons sorted together: one slice per wave
constexpr int kRunSlices = kRunLen / 64;
static_assert(kRunSlices == kRWaves, "a run is one slice per wave");
constexpr int kBlockBytes = 64 * 4 * (2 + 4);

// Slices of a run are ordered by length: a wave alternates between their ends.
__device__ __forceinline__ int slice_of(int run, int wave) {
    return run * kRunSlices + ((run & 1) ? kRunSlices - 1 - wave : wave);
}

// ------------------------------------------------------------------------------------------ set-up

// One workgroup per run: its neurons by list length (longest first, ties by index) into order[], and the block
// counts of every slice (low half: of its longest list; high half: whole blocks of its shortest).
__global__ __launch_bounds__(kRunLen) void resident_order_kernel(int64_t n, const int64_t *__restrict__ fan_ptr,
                                                                 uint16_t *__restrict__ order,
                                                                 uint2 *__restrict__ slices) {
    __shared__ uint32_t key[kRunLen];  // (complemented length, place in the run)
    const int t = threadIdx.x;
    const int64_t j = (int64_t)blockIdx.x * kRunLen + t;
    const uint32_t len = j < n ? (uint32_t)(fan_ptr[j + 1] - fan_ptr[j]) : 0u;
    key[t] = j < n ? ((kResidentMaxN - len) << 10 | (uint32_t)t) : 0xffffffffu;
    __syncthreads();
    for (int k = 2; k <= kRunLen; k <<= 1)
        for (int d = k >> 1; d > 0; d >>= 1) {
            const int u = t ^ d;
            if (u > t) {
                const uint32_t a = key[t], b = key[u];
                if ((a > b) == ((t & k) == 0)) {
                    key[t] = b;
                    key[u] = a;
                }
            }
            __syncthreads();
        }
    const uint32_t mine = key[t];
    order[j] = mine == 0xffffffffu ? (uint16_t)0xffffu : (uint16_t)((int64_t)blockIdx.x * kRunLen + (mine & 1023u));
    // the slice's first list is its longest, its last the shortest: blocks, and those no list is padded in
    const uint32_t l = mine == 0xffffffffu ? 0u : kResidentMaxN - (mine >> 10);
    const uint32_t shortest = __shfl(l, 63);
    if ((t & 63) == 0) slices[j / 64].y = (l + 3u) / 4u | shortest / 4u << 16;
}

// Blocks of every slice: a wave takes blocks blockIdx.y, + gridDim.y, ... of its slice.  The slice's first block is
// the sum of the counts before it, which every wave adds up for itself (at most 80 slices); the first wave of a slice
// writes it down, the last slice's the total, and the first slice's the blocks of the product's busiest wave.
__global__ __launch_bounds__(64) void resident_fill_kernel(int64_t n, const int64_t *__restrict__ fan_ptr,
                                                           const Edge *__restrict__ fan,
                                                           const uint16_t *__restrict__ order, uint2 *slices,
                                                           char *__restrict__ blocks, int32_t *__restrict__ report) {
    const int lane = threadIdx.x;
    uint32_t before = 0;
    for (uint32_t q = lane; q < blockIdx.x; q += 64) before += slices[q].y & 0xffffu;
    for (int d = 32; d > 0; d >>= 1) before += __shfl_xor(before, d);
    const uint2 sl = make_uint2(before, slices[blockIdx.x].y);
    if (lane == 0 && blockIdx.y == 0) {
        slices[blockIdx.x].x = before;
        if (blockIdx.x + 1 == gridDim.x) report[0] = (int32_t)(before + (sl.y & 0xffffu));
    }
    if (blockIdx.x == 0 && blockIdx.y == 0) {
        uint32_t wave = 0;
        for (int run = 0; lane < kRWaves && run * kRunSlices < (int)gridDim.x; ++run)
            wave += slices[slice_of(run, lane)].y & 0xffffu;
        for (int d = 32; d > 0; d >>= 1) wave = max(wave, (uint32_t)__shfl_xor(wave, d));
        if (lane == 0) report[1] = (int32_t)wave;
    }
    const uint32_t j = order[(int64_t)blockIdx.x * 64 + lane];
    int64_t e0 = 0;
    uint32_t len = 0;
    if (j != 0xffffu) {
        e0 = fan_ptr[j];
        len = (uint32_t)(fan_ptr[j + 1] - e0);
    }
    for (uint32_t b = blockIdx.y; b < (sl.y & 0xffffu); b += gridDim.y) {
        uint32_t idx[4];
        float w[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            idx[u] = (uint32_t)n;
            w[u] = 0.0f;
            if (4 * b + u < len) {
                const Edge e = fan[e0 + 4 * b + u];
                idx[u] = (uint32_t)e.idx;
                w[u] = e.w;
            }
        }
        char *p = blocks + (size_t)(sl.x + b) * kBlockBytes;
        reinterpret_cast<uint2 *>(p)[lane] = make_uint2(idx[0] | idx[1] << 16, idx[2] | idx[3] << 16);
        reinterpret_cast<float4 *>(p + 512)[lane] = make_float4(w[0], w[1], w[2], w[3]);
    }
}

// ------------------------------------------------------------------------------------------ product

struct ResidentArgs {
    ResidentLayer layer[kResidentLayers];
};

template <int V>
struct RowOf;
template <>
struct RowOf<1> {
    using T = float;
};
template <>
struct RowOf<2> {
    using T = float2;
};
template <>
struct RowOf<4> {
    using T = float4;
};

template <int V>
__device__ __forceinline__ void unpack(const typename RowOf<V>::T &r, float (&y)[V]) {
    if constexpr (V == 1) {
        y[0] = r;
    } else {
        y[0] = r.x;
        y[1] = r.y;
        if constexpr (V == 4) {
            y[2] = r.z;
            y[3] = r.w;
        }
    }
}

template <int V>
__device__ __forceinline__ typename RowOf<V>::T pack(const float (&y)[V]) {
    if constexpr (V == 1)
        return y[0];
    else if constexpr (V == 2)
        return make_float2(y[0], y[1]);
    else
        return make_float4(y[0], y[1], y[2], y[3]);
}

// What a lane does with an entry: acc (+)= y (x) w, starting from the 0-element, which is also what the padding's
// input row holds.  The forward's products are exact and summed in fp64.  The semirings that only select or add
// once work in fp32: rounding is monotonic, so the largest rounded sum is the rounded largest sum, and a sum of two
// fp32 values rounded through fp64 is the fp32 sum.  A selection keeps a NaN only until the next entry, so there
// padded entries are skipped (kGuard) rather than folded in.
template <bool kPattern_>
struct Forward {
    using Acc = double;
    static constexpr bool kLayer = true, kPattern = kPattern_, kGuard = false;
    static __device__ float zero() { return 0.0f; }
    static __device__ void fold(double &a, float y, float w) { a = __builtin_fma((double)y, (double)w, a); }
};
struct PlusTimes {
    using Acc = double;
    static constexpr bool kLayer = false, kPattern = false, kGuard = false;
    static __device__ float zero() { return 0.0f; }
    static __device__ void fold(double &a, float y, float w) { a = __builtin_fma((double)y, (double)w, a); }
};
struct MaxPlus {
    using Acc = float;
    static constexpr bool kLayer = false, kPattern = false, kGuard = true;
    static __device__ float zero() { return -__builtin_huge_valf(); }
    static __device__ void fold(float &a, float y, float w) {
        const float p = y + w;
        a = a > p ? a : p;
    }
};
struct MaxMin {
    using Acc = float;
    static constexpr bool kLayer = false, kPattern = false, kGuard = true;
    static __device__ float zero() { return -__builtin_huge_valf(); }
    static __device__ void fold(float &a, float y, float w) {
        const float p = y < w ? y : w;
        a = a > p ? a : p;
    }
};
struct MinMax {
    using Acc = float;
    static constexpr bool kLayer = false, kPattern = false, kGuard = true;
    static __device__ float zero() { return __builtin_huge_valf(); }
    static __device__ void fold(float &a, float y, float w) {
        const float p = y > w ? y : w;
        a = a < p ? a : p;
    }
};
struct XorAnd {  // GF(2): a value counts as 1 when it is nonzero
    using Acc = uint32_t;
    static constexpr bool kLayer = false, kPattern = false, kGuard = false;
    static __device__ float zero() { return 0.0f; }
    static __device__ void fold(uint32_t &a, float y, float w) { a ^= (uint32_t)(y != 0.0f) & (uint32_t)(w != 0.0f); }
};

constexpr int kAhead = 3;  // blocks in flight per wave

// A slice a wave is about to walk: its first blocks are already on their way.
struct Slice {
    uint32_t first, count, whole;
    uint32_t j;
    uint2 i[kAhead];
    float4 w[kAhead];
};

// grid: (sample groups, neuron parts).  A part is `runs` consecutive runs of kRunLen neurons; with more than one
// part (a single layer then) every part's workgroup reads all input rows and writes its own neurons.
template <int V, class Op>
__global__ __launch_bounds__(kRThreads) void spmm_resident_kernel(ResidentArgs args, int layers, int n, int64_t batch,
                                                                  int nslices, int runs, double ymax,
                                                                  ResidentIo io) {
    using Row = typename RowOf<V>::T;
    extern __shared__ __align__(16) char resident_lds[];
    Row *src = reinterpret_cast<Row *>(resident_lds);
    Row *dst = src + (n + 1);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t r0 = (int64_t)blockIdx.x * V;
    const int rows = (int)(batch - r0 < V ? batch - r0 : V);
    const int run0 = blockIdx.y * runs;
    const int run1 = min(run0 + runs, (nslices + kRunSlices - 1) / kRunSlices);
    const int j0 = run0 * kRunLen;  // first neuron of the part: its outputs sit at dst[j - j0]

    auto load = [&](const char *blocks, uint32_t b, uint2 &i, float4 &w) {
        const char *p = blocks + (size_t)b * kBlockBytes;  // wave-uniform: a scalar base and 32-bit lane offsets
        i = *reinterpret_cast<const uint2 *>(p + (uint32_t)lane * 8u);
        w = *reinterpret_cast<const float4 *>(p + (512u + (uint32_t)lane * 16u));
    };
    auto fetch = [&](const ResidentLayer &l, int run, Slice &s) {
        const int q = slice_of(run, wave);
        s.count = s.whole = 0;
        s.first = 0;
        s.j = 0xffffu;
        if (q < nslices) {
            const uint2 d = l.slices[q];
            s.first = __builtin_amdgcn_readfirstlane(d.x);
            s.count = __builtin_amdgcn_readfirstlane(d.y & 0xffffu);
            s.whole = __builtin_amdgcn_readfirstlane(d.y >> 16);
            s.j = l.order[q * 64 + lane];
            if (s.count > 0) {
#pragma unroll
                for (int q = 0; q < kAhead; ++q)
                    load(l.blocks, s.first + min((uint32_t)q, s.count - 1), s.i[q], s.w[q]);
            }
        }
    };

    Slice next;
    fetch(args.layer[0], run0, next);
    const bool csr = io.col != nullptr || io.row_ptr != nullptr;
    for (int i = tid; i <= n; i += kRThreads) {
        float y[V];
#pragma unroll
        for (int v = 0; v < V; ++v) y[v] = (!csr && v < rows && i < n) ? io.y_in[(r0 + v) * n + i] : Op::zero();
        src[i] = pack<V>(y);
        // both buffers end in the zero row (with several parts, dst holds one part's outputs and is never read as
        // an input)
        if (i == n && gridDim.y == 1) dst[i] = pack<V>(y);
    }
    if (csr) {
        // sparse rows, placed into the cleared rows: each sample by 16 / V waves, extents and columns checked
        __syncthreads();
        const int v = wave % V;
        const int64_t r = r0 + v;
        int64_t b = 0, len = 0;
        if (v < rows) {
            if (io.row_ptr) {
                const int64_t nnz = (io.col && io.val) ? io.row_ptr[batch] : 0;
                b = io.row_ptr[r];
                len = io.row_ptr[r + 1] - b;
                if (b < 0 || len < 0 || len > n || b + len > nnz) {
                    if (lane == 0 && blockIdx.y == 0) atomicOr(io.err, 1u);
                    len = 0;
                }
            } else {
                b = r * n;
                len = io.cnt_in[r];
            }
        }
        float *y = reinterpret_cast<float *>(src);
        for (int64_t t = (int64_t)(wave / V) * 64 + lane; t < len; t += kRThreads / V) {
            const int32_t i = io.col[b + t];
            const float f = io.val[b + t];
            if (i < 0 || i >= n)
                atomicOr(io.err, 1u);
            else
                y[i * V + v] = f;
        }
    }
    __syncthreads();

    for (int k = 0; k < layers; ++k) {
        const ResidentLayer &l = args.layer[k];
        for (int run = run0; run < run1; ++run) {
            Slice cur = next;
            // the wave's next slice, in this layer or the next, starts loading now
            if (run + 1 < run1)
                fetch(l, run + 1, next);
            else if (k + 1 < layers)
                fetch(args.layer[k + 1], run0, next);
            const char *blocks = l.blocks;
            const bool real = cur.j != 0xffffu;
            float bj = 0.0f;
            if constexpr (Op::kLayer) bj = l.bias[real ? cur.j : 0];
            typename Op::Acc acc[V];
            uint32_t hit[V];
#pragma unroll
            for (int v = 0; v < V; ++v) {
                acc[v] = (typename Op::Acc)Op::zero();
                hit[v] = 0u;
            }
            auto block = [&](const uint2 &i, const float4 &w, bool whole) {
                const uint32_t at[4] = {i.x & 0xffffu, i.x >> 16, i.y & 0xffffu, i.y >> 16};
                const float wv[4] = {w.x, w.y, w.z, w.w};
                Row r[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) r[u] = src[at[u]];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    float y[V];
                    unpack<V>(r[u], y);
#pragma unroll
                    for (int v = 0; v < V; ++v) {
                        typename Op::Acc a = acc[v];
                        Op::fold(a, y[v], wv[u]);
                        acc[v] = (!Op::kGuard || whole || at[u] != (uint32_t)n) ? a : acc[v];
                        if constexpr (Op::kPattern) hit[v] |= __float_as_uint(y[v]);
                    }
                }
            };
            // kAhead blocks are in flight; a register set is loaded again as soon as its block is used, with the
            // last block again past the end (loaded and not used)
            const uint32_t count = __builtin_amdgcn_readfirstlane(cur.count);
            const uint32_t first = __builtin_amdgcn_readfirstlane(cur.first);
            const uint32_t last = first + count - 1;
            const uint32_t whole = Op::kGuard ? __builtin_amdgcn_readfirstlane(cur.whole) : count;
            uint32_t b = 0;
            // whole blocks, kAhead at a time
            for (; b + kAhead <= whole; b += kAhead) {
#pragma unroll
                for (int q = 0; q < kAhead; ++q) {
                    block(cur.i[q], cur.w[q], true);
                    load(blocks, min(first + b + kAhead + q, last), cur.i[q], cur.w[q]);
                    __builtin_amdgcn_sched_barrier(0);  // the load stays here, a block ahead of the next set's
                }
            }
            if constexpr (Op::kGuard) {
                for (; b + kAhead <= count; b += kAhead) {
#pragma unroll
                    for (int q = 0; q < kAhead; ++q) {
                        block(cur.i[q], cur.w[q], false);
                        load(blocks, min(first + b + kAhead + q, last), cur.i[q], cur.w[q]);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
#pragma unroll
            for (int q = 0; q + 1 < kAhead; ++q)
                if (b + q < count) block(cur.i[q], cur.w[q], false);
            if (real) {
                float out[V];
#pragma unroll
                for (int v = 0; v < V; ++v)
                    if constexpr (Op::kLayer)
                        out[v] = (Op::kPattern && (hit[v] & 0x7fffffffu) == 0u) ? 0.0f : activate(acc[v] + (double)bj, ymax);
                    else
                        out[v] = (float)acc[v];
                dst[(int)cur.j - j0] = pack<V>(out);
            }
        }
        __syncthreads();
        Row *t = src;
        src = dst;
        dst = t;
    }
    // the part's outputs, batch-major, and the nonzeros of each sample (counted in the buffer no one reads any more;
    // a whole sample's only: one part)
    int *total = reinterpret_cast<int *>(dst);
    if (io.cnt_out) {
        if (tid < V) total[tid] = 0;
        __syncthreads();
    }
    int nonzero[V];
#pragma unroll
    for (int v = 0; v < V; ++v) nonzero[v] = 0;
    const int count = min(n, run1 * kRunLen) - j0;
    for (int i = tid; i < count; i += kRThreads) {
        float y[V];
        unpack<V>(src[i], y);
#pragma unroll
        for (int v = 0; v < V; ++v) {
            if (v < rows) io.y_out[(r0 + v) * n + j0 + i] = y[v];
            nonzero[v] += y[v] != 0.0f ? 1 : 0;
        }
    }
    if (io.cnt_out) {
#pragma unroll
        for (int v = 0; v < V; ++v) {
            for (int d = 32; d > 0; d >>= 1) nonzero[v] += __shfl_xor(nonzero[v], d);
            if (lane == 0) atomicAdd(&total[v], nonzero[v]);
        }
        __syncthreads();
        if (tid < rows) io.cnt_out[r0 + tid] = total[tid];
    }
}

int64_t resident_slices(int64_t n) { return (n + kRunLen - 1) / kRunLen * kRunSlices; }

}  // namespace

// Bytes of a layer's interleaved lists: the order and slice table, then the blocks.  Lists of a run are sorted by
// length, so a slice's longest list is at most the shortest of the slice before it: the padding of a run is at
// most one longest list (n entries) per lane, and the rounding to blocks of four at most a block per slice.
size_t resident_bytes(int64_t n, int64_t nnz) {
    const int64_t runs = (n + kRunLen - 1) / kRunLen;
    const int64_t blocks = runs * (std::min(n, nnz) / 4 + 1 + kRunSlices) + nnz / 256 + 1;
    return (size_t)(resident_slices(n) * (64 * 2 + 8) + 256 + blocks * kBlockBytes);
}

bool resident_planned(int64_t n) { return n <= kResidentMaxN; }

ResidentLayer resident_layer(void *mem, int64_t n, const float *bias) {
    ResidentLayer l;
    char *p = static_cast<char *>(mem);
    l.order = reinterpret_cast<uint16_t *>(p);
    p += (resident_slices(n) * 64 * 2 + 255) / 256 * 256;
    l.slices = reinterpret_cast<uint2 *>(p);
    p += (resident_slices(n) * 8 + 255) / 256 * 256;
    l.blocks = p;
    l.bias = bias;
    return l;
}

hipError_t launch_resident_lists(int64_t n, const int64_t *fan_ptr, const Edge *fan, void *mem, int32_t *report,
                                 hipStream_t s) {
    const ResidentLayer l = resident_layer(mem, n, nullptr);
    const int64_t slices = resident_slices(n);
    resident_order_kernel<<<(unsigned)(slices / kRunSlices), kRunLen, 0, s>>>(
        n, fan_ptr, const_cast<uint16_t *>(l.order), const_cast<uint2 *>(l.slices));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    resident_fill_kernel<<<dim3((unsigned)slices, 16), 64, 0, s>>>(
        n, fan_ptr, fan, l.order, const_cast<uint2 *>(l.slices), const_cast<char *>(l.blocks), report);
    return hipGetLastError();
}

namespace {

template <int V, class Op>
hipError_t launch_v(const ResidentArgs &args, int layers, int64_t n, int64_t batch, int parts, double ymax,
                    const ResidentIo &io, hipStream_t s) {
    const int64_t runs = (n + kRunLen - 1) / kRunLen;
    const int per = (int)((runs + parts - 1) / parts);
    parts = (int)((runs + per - 1) / per);
    const size_t lds = resident_lds(n, V, parts > 1 ? (int64_t)per * kRunLen : n + 1);
    if (lds > kResidentLds) return hipErrorInvalidValue;
    static std::atomic<unsigned long long> attr_devices{0};
    const hipError_t e = raise_lds_limit((const void *)spmm_resident_kernel<V, Op>, kResidentLds, attr_devices);
    if (e != hipSuccess) return e;
    const int64_t groups = (batch + V - 1) / V;
    const int64_t seg = (int64_t(1) << 21) / parts;  // groups per launch: fewer than 2^32 work-items
    for (int64_t g0 = 0; g0 < groups; g0 += seg) {
        const int64_t r0 = g0 * V;  // the launch's first sample: everything indexed by sample starts there
        ResidentIo part = io;
        if (io.y_in) part.y_in += r0 * n;
        if (io.row_ptr) part.row_ptr += r0;
        if (io.cnt_in) {
            part.cnt_in += r0;
            part.col += r0 * n;
            part.val += r0 * n;
        }
        part.y_out += r0 * n;
        if (io.cnt_out) part.cnt_out += r0;
        spmm_resident_kernel<V, Op><<<dim3((unsigned)std::min(seg, groups - g0), (unsigned)parts), kRThreads, lds, s>>>(
            args, layers, (int)n, batch - r0, (int)((n + 63) / 64), per, ymax, part);
        const hipError_t el = hipGetLastError();
        if (el != hipSuccess) return el;
    }
    return hipSuccess;
}

template <class Op>
hipError_t launch_op(const ResidentArgs &args, int layers, int64_t n, int64_t batch, int v, int parts, double ymax,
                     const ResidentIo &io, hipStream_t s) {
    switch (v) {
        case 1: return launch_v<1, Op>(args, layers, n, batch, parts, ymax, io, s);
        case 2: return launch_v<2, Op>(args, layers, n, batch, parts, ymax, io, s);
        case 4: return launch_v<4, Op>(args, layers, n, batch, parts, ymax, io, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_spmm_resident(const ResidentLayer *layer, int layers, int64_t n, int64_t batch, int v, int parts,
                                double ymax, int pattern, const ResidentIo &io, hipStream_t s) {
    if (layers < 1 || layers > kResidentLayers || n > kResidentMaxN || (parts > 1 && (layers > 1 || io.cnt_out)))
        return hipErrorInvalidValue;
    ResidentArgs args;
    for (int k = 0; k < layers; ++k) args.layer[k] = layer[k];
    return pattern ? launch_op<Forward<true>>(args, layers, n, batch, v, parts, ymax, io, s)
                   : launch_op<Forward<false>>(args, layers, n, batch, v, parts, ymax, io, s);
}

hipError_t launch_semiring_resident(int semiring, const ResidentLayer &layer, int64_t n, int64_t batch, int v, int parts,
                                    const float *y, float *z, hipStream_t s) {
    if (n > kResidentMaxN) return hipErrorInvalidValue;
    ResidentArgs args;
    args.layer[0] = layer;
    ResidentIo io;
    io.y_in = y;
    io.y_out = z;
    switch (semiring) {
        case kSemiringPlusTimes: return launch_op<PlusTimes>(args, 1, n, batch, v, parts, 0.0, io, s);
        case kSemiringMaxPlus: return launch_op<MaxPlus>(args, 1, n, batch, v, parts, 0.0, io, s);
        case kSemiringMaxMin: return launch_op<MaxMin>(args, 1, n, batch, v, parts, 0.0, io, s);
        case kSemiringMinMax: return launch_op<MinMax>(args, 1, n, batch, v, parts, 0.0, io, s);
        case kSemiringXorAnd: return launch_op<XorAnd>(args, 1, n, batch, v, parts, 0.0, io, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace sdnn
