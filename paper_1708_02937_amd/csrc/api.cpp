// Host runtime behind the C ABI of include/sdnn.h: argument checks, layer set-up, workspace carving and
// the layer loop of the forward pass (the loop of the paper's dnn() function, Fig. 4, Sec. IV), with every
// layer's work enqueued on the net's HIP stream.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "common.h"
#include "sdnn.h"

using sdnn::Edge;

namespace {

thread_local std::string g_last_error;

sdnn_status fail(sdnn_status s, const std::string &msg) {
    g_last_error = msg;
    return s;
}

sdnn_status fail_hip(hipError_t e, const char *what) {
    return fail(SDNN_ERR_DEVICE, std::string(what) + ": " + hipGetErrorString(e));
}

// Makes the net's device current for one call and gives the caller's device back on return.
struct DeviceScope {
    int prev = -1;  // the caller's device when it has to be restored
    hipError_t err = hipSuccess;
    explicit DeviceScope(int dev) {
        int cur = 0;
        err = hipGetDevice(&cur);
        if (err == hipSuccess && cur != dev) {
            err = hipSetDevice(dev);
            if (err == hipSuccess) prev = cur;
        }
    }
    ~DeviceScope() {
        if (prev >= 0) (void)hipSetDevice(prev);
    }
    DeviceScope(const DeviceScope &) = delete;
    DeviceScope &operator=(const DeviceScope &) = delete;
};

// Allows the calling thread's allocation calls while another thread records a graph (a capture in global mode would
// otherwise be broken by them).
struct CaptureScope {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    CaptureScope() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    ~CaptureScope() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    CaptureScope(const CaptureScope &) = delete;
    CaptureScope &operator=(const CaptureScope &) = delete;
};

#define SDNN_ON_DEVICE(net)                                                     \
    DeviceScope device_scope_((net)->device);                                   \
    if (device_scope_.err != hipSuccess) return fail_hip(device_scope_.err, "hipSetDevice")

#define SDNN_HIP(call)                                      \
    do {                                                    \
        hipError_t e_ = (call);                             \
        if (e_ != hipSuccess) return fail_hip(e_, #call);   \
    } while (0)

struct Layer {
    bool set = false;
    int64_t nnz = 0;
    const int64_t *row_ptr = nullptr;  // caller-owned fan-out CSR and bias
    const int32_t *col = nullptr;
    const float *val = nullptr;
    const float *bias = nullptr;
    bool bias_nonpos = true;
    bool bias_uniform = false;  // every b_j has the same bits
    int64_t pos_bias = 0;      // neurons with b_j > 0
    double zero_below = -INFINITY;  // every b_j <= 0: -max_j b_j (a sum at most this is zero after h), else -inf
    int32_t max_fanout = 0;    // longest fan-out row of W_k
    int32_t max_fanin = 0;     // longest fan-in list
    Edge *w_pack = nullptr;    // fan-out entries packed as (column, weight)
    int64_t *fan_ptr = nullptr;  // fan-in CSR (W_k^T)
    Edge *fan = nullptr;
    uint16_t *tile_mask = nullptr;  // which rows of each 16-row input tile each fan-in list holds (high fan-in only)
    double *slots = nullptr;        // fp64 weight of every (input, output) pair, tile-major (high fan-in, n^2 fits)
    int32_t *w_seg = nullptr;     // where each fan-out row crosses each accumulator window (wide layers only)
    sdnn::BlockedSched *sched = nullptr;  // schedule of the blocked product (wide layers, short lists)
    Edge *stage = nullptr;                 // its lists in schedule order, one region per workgroup
    sdnn::BlockedRegion *regions = nullptr;  // the regions (null when one exceeds the product's LDS capacity)
    void *resident = nullptr;    // lists interleaved for the LDS-resident product (n <= kResidentMaxN)
    int32_t resident_blocks = 0; // its blocks of four entries per lane
    int32_t resident_wave = 0;   // blocks of a workgroup's busiest wave
    double *dense_wt = nullptr;  // n x n, W_k k-major in fp64 (zeros explicit), for the fp64 dense arm
    float *dense_wt32 = nullptr; // the same in fp32, for the fp32 dense arm
    bool dense_ready = false, dense32_ready = false;  // the dense copies hold the current W_k
};

using sdnn::align_up;
constexpr size_t kAlign = 256;

// ---------------------------------------------------------------------------------------- net arena
// All device memory a net keeps lives in one caller-owned arena, laid out once at creation from n, L, the
// entry capacity of every layer and which dense copies are wanted.  Per layer, at fixed offsets: the packed
// fan-out rows, the fan-in (W_k^T) pointers and lists (plus a zero guard entry), and the optional structures
// whose need follows from n and the capacity (tile masks and fp64 weight slots for dense-ish layers, window
// offsets for the SpGEMM of wide layers, the blocked product's schedule and staged lists, the dense
// copies).  Shared: the set-up scratch (counts, scan, radix-sort buffers, sized for the largest layer) and
// the small per-forward flags and counters.
constexpr size_t kAbsent = ~size_t(0);

struct LayerPlan {
    size_t w_pack = kAbsent, fan_ptr = kAbsent, fan = kAbsent, tile_mask = kAbsent, slots = kAbsent,
           w_seg = kAbsent, sched = kAbsent, stage = kAbsent, regions = kAbsent, starts = kAbsent,
           resident = kAbsent, dense64 = kAbsent, dense32 = kAbsent;
    size_t bytes = 0;
};

constexpr int kSetupInts = 8;  // what a layer's set-up reports to the host (the first four also its validation's flags)

struct NetPlan {
    size_t flags = 0, d_int = 0, stats = 0, counts = 0, tmp = 0, sort = 0;
    std::vector<size_t> layer_off;
    std::vector<LayerPlan> layer;
    size_t bytes = 0;
};

size_t take(size_t &off, size_t bytes) {
    const size_t at = off;
    off = align_up(off + bytes);
    return at;
}

LayerPlan plan_layer(int64_t n, int64_t cap, int32_t dense_flags) {
    LayerPlan lp;
    size_t off = 0;
    // one entry more than the layer's: 16-byte loads of entry pairs may read one entry past a row's end
    lp.w_pack = take(off, (size_t)(std::max<int64_t>(cap, 1) + 1) * sizeof(Edge));
    lp.fan_ptr = take(off, (size_t)(n + 1) * sizeof(int64_t));
    lp.fan = take(off, (size_t)(cap + 1) * sizeof(Edge));
    if (sdnn::spmm_wants_tiles(n, cap)) lp.tile_mask = take(off, sdnn::spmm_tile_mask_elems(n) * sizeof(uint16_t));
    if (sdnn::spmm_wants_slots(n, cap)) lp.slots = take(off, sdnn::spmm_slot_elems(n) * sizeof(double));
    if (sdnn::spgemm_wants_window_index(n))
        lp.w_seg = take(off, (size_t)n * (size_t)(sdnn::spgemm_windows(n) + 1) * sizeof(int32_t));
    if (sdnn::blocked_planned(n, cap)) {
        lp.sched = take(off, (size_t)sdnn::blocked_sched_elems(n) * sizeof(sdnn::BlockedSched));
        lp.stage = take(off, sdnn::blocked_stage_elems(n, cap) * sizeof(Edge));
        lp.regions = take(off, (size_t)sdnn::blocked_regions(n) * sizeof(sdnn::BlockedRegion));
        lp.starts = take(off, (size_t)(sdnn::blocked_regions(n) + 1) * sizeof(int64_t));
    }
    if (sdnn::resident_planned(n)) lp.resident = take(off, sdnn::resident_bytes(n, cap));
    if (dense_flags & SDNN_ARENA_DENSE_F64) lp.dense64 = take(off, sdnn::gemm_weight_elems(n) * sizeof(double));
    if (dense_flags & SDNN_ARENA_DENSE_F32) lp.dense32 = take(off, sdnn::gemm_weight_elems(n) * sizeof(float));
    lp.bytes = off;
    return lp;
}

NetPlan plan_net(int64_t n, int32_t L, const int64_t *caps, int32_t dense_flags) {
    NetPlan np;
    size_t off = 0;
    int64_t max_cap = 0;
    for (int32_t k = 0; k < L; ++k) max_cap = std::max(max_cap, caps[k]);
    np.flags = take(off, 4 * sizeof(uint32_t));
    np.d_int = take(off, kSetupInts * sizeof(int32_t));
    np.stats = take(off, (size_t)std::max<int32_t>(L, 1) * sdnn::kSpgemmStats * sizeof(unsigned long long));
    np.counts = take(off, (size_t)n * sizeof(int32_t));
    np.tmp = take(off, (size_t)sdnn::scan_tmp_elems(n) * sizeof(int64_t));
    np.sort = take(off, sdnn::fanin_sort_bytes(max_cap));
    for (int32_t k = 0; k < L; ++k) {
        np.layer.push_back(plan_layer(n, caps[k], dense_flags));
        np.layer_off.push_back(take(off, np.layer.back().bytes));
    }
    np.bytes = off;
    return np;
}

template <typename T>
T *at(char *base, size_t off) {
    return off == kAbsent ? nullptr : reinterpret_cast<T *>(base + off);
}

sdnn_status check_plan_args(int64_t n, int32_t L, const int64_t *caps, int32_t dense_flags) {
    if (n < 1 || n > 0x7fffffffLL) return fail(SDNN_ERR_INVALID_VALUE, "n must be in [1, 2^31-1]");
    if (L < 0) return fail(SDNN_ERR_INVALID_VALUE, "L must be >= 0");
    if (L > 0 && !caps) return fail(SDNN_ERR_NULL_POINTER, "nnz_per_layer is required when L > 0");
    if (dense_flags & ~(SDNN_ARENA_DENSE_F64 | SDNN_ARENA_DENSE_F32))
        return fail(SDNN_ERR_INVALID_VALUE, "unknown dense-copy flags");
    for (int32_t k = 0; k < L; ++k)
        if (caps[k] < 0 || caps[k] > 0x7fffffffLL) return fail(SDNN_ERR_INVALID_VALUE, "layer capacities must be in [0, 2^31-1]");
    return SDNN_OK;
}

// Workspace of a CSR forward: two slot buffers (count[batch], col[n*ld], val[n*ld] with ld = act_ld(n, batch)
// >= batch, so that a pair of them also holds two n x batch activation buffers at row pitch ld) and a scan area.
struct CsrWs {
    int32_t *cnt[2];
    int32_t *col[2];
    float *val[2];
    int32_t *lists;  // 3 * batch: the sample lists of the layer being computed
    int64_t *scan_tmp;
    int32_t *pcnt;   // per (part, sample) counts of the blocked -> CSR packing
    uint32_t *nzrows;  // nonzero-row maps of a sparse input in the blocked layout
    size_t bytes;
};

CsrWs carve_csr(void *base, int64_t n, int64_t batch) {
    CsrWs w{};
    char *p = (char *)base;
    size_t off = 0;
    const size_t slots = (size_t)sdnn::act_ld(n, batch) * (size_t)n;
    for (int b = 0; b < 2; ++b) {
        w.cnt[b] = (int32_t *)(p + off);
        off = align_up(off + (size_t)batch * sizeof(int32_t));
        w.col[b] = (int32_t *)(p + off);
        off = align_up(off + slots * sizeof(int32_t));
        w.val[b] = (float *)(p + off);
        off = align_up(off + slots * sizeof(float));
    }
    w.lists = (int32_t *)(p + off);
    off = align_up(off + 3 * (size_t)batch * sizeof(int32_t));
    w.scan_tmp = (int64_t *)(p + off);
    off = align_up(off + (size_t)sdnn::scan_tmp_elems(batch) * sizeof(int64_t));
    w.pcnt = (int32_t *)(p + off);
    w.nzrows = nullptr;
    if (sdnn::blocked_wanted(n, batch)) {
        off = align_up(off + sdnn::blocked_pack_elems(n, batch) * sizeof(int32_t));
        w.nzrows = (uint32_t *)(p + off);
        off = align_up(off + (size_t)sdnn::blocked_chunks(batch) * (size_t)sdnn::blocked_nz_words(n) * sizeof(uint32_t));
    }
    w.bytes = off;
    return w;
}

constexpr int64_t kMaxScan = 16777216;  // longest array the device prefix sum handles (fan-in pointers, row pointers)

// a dense-Y call's workspace: two neuron-major activation buffers, or, for a net with dense copies, what the arms need
size_t dense_ws_bytes(int64_t n, int64_t batch, int32_t dense_flags, int num_cu) {
    const size_t sparse = 2 * sdnn::act_bytes(n, sdnn::act_ld(n, batch));
    return dense_flags ? std::max(sparse, sdnn::arm_ws_bytes(n, batch, sdnn::gemm_splits(n, batch, num_cu))) : sparse;
}

// Workspace of sdnn_forward_dense_noalloc: a fixed device array, one copy per GPU, held until the process
// ends.  In host code the symbol is only a host-side stand-in; kernels get the device address that
// hipGetSymbolAddress returns for the current device (kept per device in g_scratch).
constexpr size_t kScratchBytes = size_t(64) << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
struct ScratchSlot {
    std::once_flag once;
    void *ptr = nullptr;
    hipError_t err = hipErrorNotInitialized;
};
ScratchSlot g_scratch[kMaxDevices];

// Looks up this device's copy of the scratch array once; the device must be current.
void scratch_init(int dev) {
    if (dev < 0 || dev >= kMaxDevices) return;
    ScratchSlot &slot = g_scratch[dev];
    std::call_once(slot.once, [&slot]() {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        slot.err = e;
        slot.ptr = e == hipSuccess ? p : nullptr;
        if (e != hipSuccess) (void)hipGetLastError();
    });
}

}  // namespace

struct sdnn_net_s {
    int64_t n = 0;
    int32_t L = 0;
    double ymax = INFINITY;
    int bias_pattern = 0;  // SDNN_BIAS_PATTERN: bias only on the structural pattern of Y_k W_k
    hipStream_t stream = nullptr;
    int device = 0;
    std::vector<Layer> layers;
    uint32_t *d_flags = nullptr;
    int32_t *d_int = nullptr;
    unsigned long long *d_stats = nullptr;  // kSpgemmStats counters per layer of a forward call
    int num_cu = 256;
    // pinned host memory: what the kernels of a CSR call report, and the words the set-up copies back
    sdnn::HostSlot *host = nullptr;
    uint32_t *host_words = nullptr;
    char *arena = nullptr;  // caller-owned device memory holding everything above and every layer's copies
    NetPlan plan;
    std::vector<int64_t> caps;  // entry capacity of each layer
    int32_t dense_flags = 0;
    // profiling log (sdnn_net_set_profiling): one pair of events around each timed launch sequence
    struct ProfRec {
        int32_t layer, kernel;
        hipEvent_t a, b;
    };
    bool profiling = false;
    std::vector<ProfRec> prof;
    std::vector<hipEvent_t> ev_free;
};

namespace {

// Whether dense-Y layers [k0, k1) run on the sample-blocked layout: always beyond 16384 neurons; from 4097 to
// 16384 only when every layer of the range stages its lists (short lists), since the other dense-Y products
// share the neuron-major layout and the forward keeps one layout throughout.
bool use_blocked(const sdnn_net_s *net, int32_t k0, int32_t k1, int64_t batch) {
    if (!sdnn::blocked_wanted(net->n, batch)) return false;
    if (sdnn::blocked_only(net->n)) return true;
    for (int32_t k = k0; k < k1; ++k)
        if (!net->layers[(size_t)k].regions) return false;
    return true;
}

// Samples a layer's neuron-major product computes (at least the batch, at most the pitch).
int64_t layer_batch(const sdnn_net_s *net, const Layer &l, int64_t batch, int64_t ld) {
    return sdnn::spmm_batch(net->n, l.nnz, l.max_fanin, l.tile_mask != nullptr, batch, ld, net->num_cu);
}

// How a dense-Y range runs on the LDS-resident product: samples per workgroup, workgroups per sample group (the
// neurons split over them), and whether the whole range is one launch.
struct ResidentPlan {
    int v = 0, parts = 1;
    bool fused = true;
};

// The rule, in microseconds measured on MI355X (n 150 to 5000, 4 to 1200 entries per neuron, batch 1 to 3045; within 10%
// at 13 sizes with every number of samples and parts).
// A workgroup takes 0.015, 0.0163 or 0.0238 us per block of 4 x 64 entries at 1, 2 or 4 samples, a CU gets through
// one workgroup's blocks at a time, a layer costs 0.85 us per run of 1024 neurons beyond that (n 4097, 12 entries,
// batch 1, four layers: 33.8 us), a launch 2 to 3 us, and its rows in and out 0.12 per 1024 neurons and sample, in every
// round of workgroups where the neurons are split.
// So few samples per workgroup where that still fills the CUs once, four where the batch does so several times
// over, and the neurons split over workgroups (then a launch per layer) where a small batch leaves CUs idle: one
// layer of 4096 neurons and 64 entries each at batch 64 takes 23.7 us whole and 9.2 in four parts, four layers of
// 1024 neurons and 16 entries 11.5 us fused and 18 launch by launch.  The neuron-major products move 4 bytes
// per product from L2 (about 27 TB/s with four samples per lane, from batch 256 on, and 12 to 16 below) and cost 6 us
// per layer and two transposes; they win only where the last round of workgroups is nearly empty.  The LDS-tiled
// product of high fan-in layers takes 1.76 + 1.21 density us per tile of 16 inputs and round of workgroups (64 neurons
// x 256 samples): 157 us per layer at n 1000, batch 129, where the resident product takes 40.
// A few long lists bound both: the wave that walks them in the resident product takes 0.095, 0.113 or 0.142 us per block
// by itself and 0.15 of the even share beside it, or 0.65 where two workgroups share a CU (at 1 and 2 samples, where
// their LDS fits), and the gather 0.055 to 0.11 us per entry beyond the mean, once per layer whatever the batch.  One
// list of 1459 entries in 2918 neurons, batch 3045, four layers: 617 us at two samples per workgroup, 670 at four, 605 by
// the gather; one of 2048 in 4096, batch 1024: 292, 308 and 603.
// With profiling on every layer is a launch of its own, and ranges with a layer of under 2^24 products stay on the
// neuron-major products: the one launch is what they gain from.
bool plan_resident(const sdnn_net_s *net, int32_t k0, int32_t k1, int64_t batch, bool may_split, bool semiring,
                   ResidentPlan *plan) {
    const int64_t n = net->n;
    if (n > sdnn::kResidentMaxN) return false;
    const double cus = (double)net->num_cu, size = (double)n, samples = (double)batch;
    const int64_t ld = sdnn::act_ld(n, batch);
    double gather = 6.0 + 4e-6 * size * samples;
    // the gather's us per list entry: whole chunks of 256 samples, each on its own XCDs when there are 1, 2, 4 or 8
    const int64_t chunks = (batch + 255) / 256;
    const bool apart = chunks <= 8 && (chunks & (chunks - 1)) == 0;
    const double per_entry = batch <= 252        ? samples * (n >= 4096 ? 1 / 4.1e6 : 1 / 3.0e6)
                             : apart || n <= 1024 ? (double)chunks * (256.0 / 6.75e6)
                                                  : (double)chunks * (256.0 / 4.5e6);
    for (int32_t k = k0; k < k1; ++k) {
        const Layer &l = net->layers[(size_t)k];
        const double nnz = (double)l.nnz;
        if (!l.resident) return false;
        if (!semiring && net->profiling && nnz * samples < (double)(1 << 24)) return false;  // (semirings are not logged)
        const int64_t lb = layer_batch(net, l, batch, ld);
        if (!semiring && l.slots && lb % 4 == 0 && lb >= 128) {
            gather += 6.0 + (double)(((n + 63) / 64 * ((batch + 255) / 256) + net->num_cu - 1) / net->num_cu) *
                                (double)((n + 15) / 16) * (1.76 + 1.21 * nnz / (size * size));
        } else if (lb % 4 != 0) {
            gather += 6.0 + 1.5 * sdnn::spmm_gather_us(l.nnz, l.max_fanin, batch);
        } else {
            const double longest = (double)l.max_fanin;
            const double entry = batch <= 252 ? (n >= 4096 ? 0.085 : 0.055)
                                 : n > 4096   ? 0.11
                                 : batch <= 1100 ? 0.068 : 0.1 - 0.045 * longest / size;
            gather += 6.0 + nnz * per_entry + entry * std::max(0.0, longest - nnz / size);
        }
    }
    const int64_t runs = (n + 1023) / 1024;
    const double layers = (double)(k1 - k0);
    const double per_block[] = {0.015, 0.0163, 0.0238}, alone[] = {0.095, 0.113, 0.142};
    const double cu_share = 1.0 / cus, run_share = 1.0 / (double)runs;
    auto up = [](double x) {  // the next whole number
        const double whole = (double)(int64_t)x;
        return whole + 1e-9 < x ? whole + 1.0 : whole;
    };
    const int32_t most_parts = may_split ? (int32_t)runs : 1;
    double best = 0.0;
    for (int i = 0; i < 3; ++i) {
        const int v = 1 << i;
        const int64_t groups = (batch + v - 1) >> i;
        for (int32_t parts = 1; parts <= most_parts; ++parts) {
            const int32_t per = parts == 1 ? (int32_t)runs : ((int32_t)runs + parts - 1) / parts;  // runs of a part
            const double workgroups = (double)(groups * (parts == 1 ? 1 : ((int32_t)runs + per - 1) / per));
            const bool two = v < 4 && sdnn::resident_lds(n, v, parts == 1 ? n + 1 : per * 1024) <= sdnn::kResidentLds / 2;
            const double load = std::max(1.0, workgroups * cu_share);
            const double rounds = up(load), turns = two ? up(0.5 * load) : rounds;
            const double block = per_block[i] * (double)per * run_share;
            const double beside = (two && load > 1.0 ? 0.65 : 0.15) * rounds;
            double t = 0.0;
            for (int32_t k = k0; k < k1; ++k) {
                const Layer &l = net->layers[(size_t)k];
                const double blocks = (double)l.resident_blocks * block;
                const double wave = (double)std::min(l.resident_wave, (l.max_fanin + 3) / 4 * per);
                t += std::max(rounds * blocks + 0.5 * (rounds - 1.0),
                              turns * alone[i] * wave + beside * blocks + 0.5 * (turns - 1.0));
            }
            const bool fused = parts == 1 && (semiring || !net->profiling);
            const double rows = 0.12 * (double)(runs << i);
            if (parts == 1)
                t += (fused ? 1.0 : layers) * (2.0 + rows) + 0.85 * (double)runs * layers;
            else
                t += (3.0 + rounds * (rows + 0.85 * (double)per)) * layers;
            if (plan->v == 0 || t < 0.98 * best) {  // near ties: fewer samples and parts
                best = t;
                plan->v = v;
                plan->parts = (int)parts;
                plan->fused = fused;
            }
        }
    }
    return best <= gather;
}

// Row pitch of the neuron-major buffers for layers [k0, k1).
int64_t range_ld(const sdnn_net_s *net, int32_t k0, int32_t k1, int64_t batch) {
    for (int32_t k = k0; k < k1; ++k) {
        const Layer &l = net->layers[(size_t)k];
        if (l.tile_mask || !sdnn::spmm_long_list(net->n, l.nnz, l.max_fanin, batch)) return sdnn::act_ld(net->n, batch);
    }
    return sdnn::act_ld_tight(net->n, batch);
}

bool overlap(const float *a, const float *b, size_t count) {
    const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b, bytes = count * sizeof(float);
    return x < y + bytes && y < x + bytes;
}

hipError_t prof_event(sdnn_net net, hipEvent_t *e) {
    if (!net->ev_free.empty()) {
        *e = net->ev_free.back();
        net->ev_free.pop_back();
        return hipSuccess;
    }
    return hipEventCreate(e);
}

// Opens a profiling record for the launches that follow (layer -1: not a layer's product); *idx = -1 when
// profiling is off.
hipError_t prof_begin(sdnn_net net, int32_t layer, int kind, int *idx) {
    *idx = -1;
    if (!net->profiling) return hipSuccess;
    sdnn_net_s::ProfRec r{layer, kind, nullptr, nullptr};
    hipError_t e = prof_event(net, &r.a);
    if (e != hipSuccess) return e;
    e = prof_event(net, &r.b);
    if (e == hipSuccess) e = hipEventRecord(r.a, net->stream);
    if (e != hipSuccess) {
        net->ev_free.push_back(r.a);
        if (r.b) net->ev_free.push_back(r.b);
        return e;
    }
    net->prof.push_back(r);
    *idx = (int)net->prof.size() - 1;
    return hipSuccess;
}

// Closes record idx (kind >= 0 replaces the kernel kind given at the start).
hipError_t prof_end(sdnn_net net, int idx, int kind = -1) {
    if (idx < 0) return hipSuccess;
    if (kind >= 0) net->prof[(size_t)idx].kernel = kind;
    return hipEventRecord(net->prof[(size_t)idx].b, net->stream);
}

void prof_clear(sdnn_net net) {
    for (auto &r : net->prof) {
        net->ev_free.push_back(r.a);
        net->ev_free.push_back(r.b);
    }
    net->prof.clear();
}

}  // namespace

static_assert(SDNN_KERNEL_TRANSPOSE == sdnn::kKernTranspose && SDNN_KERNEL_GATHER == sdnn::kKernGather &&
                  SDNN_KERNEL_NARROW == sdnn::kKernNarrow && SDNN_KERNEL_SLOTS == sdnn::kKernSlots &&
                  SDNN_KERNEL_TILED == sdnn::kKernTiled && SDNN_KERNEL_DENSE_GEMM == sdnn::kKernDenseGemm &&
                  SDNN_KERNEL_SPGEMM == sdnn::kKernSpgemm && SDNN_KERNEL_DENSIFY == sdnn::kKernDensify &&
                  SDNN_KERNEL_PACK == sdnn::kKernPack && SDNN_KERNEL_COMPACT == sdnn::kKernCompact &&
                  SDNN_KERNEL_BLOCKED == sdnn::kKernBlocked && SDNN_KERNEL_DENSE_GEMM32 == sdnn::kKernDenseGemm32 &&
                  SDNN_KERNEL_RESIDENT == sdnn::kKernResident,
              "profiling kernel ids of the header and the library agree");

extern "C" {

const char *sdnn_status_string(sdnn_status s) {
    switch (s) {
        case SDNN_OK: return "SDNN_OK";
        case SDNN_ERR_NULL_POINTER: return "SDNN_ERR_NULL_POINTER";
        case SDNN_ERR_INVALID_VALUE: return "SDNN_ERR_INVALID_VALUE";
        case SDNN_ERR_INVALID_INDEX: return "SDNN_ERR_INVALID_INDEX";
        case SDNN_ERR_DIMENSION_MISMATCH: return "SDNN_ERR_DIMENSION_MISMATCH";
        case SDNN_ERR_INVALID_OBJECT: return "SDNN_ERR_INVALID_OBJECT";
        case SDNN_ERR_WORKSPACE_TOO_SMALL: return "SDNN_ERR_WORKSPACE_TOO_SMALL";
        case SDNN_ERR_OUT_OF_MEMORY: return "SDNN_ERR_OUT_OF_MEMORY";
        case SDNN_ERR_DEVICE: return "SDNN_ERR_DEVICE";
        case SDNN_ERR_UNSUPPORTED: return "SDNN_ERR_UNSUPPORTED";
    }
    return "SDNN_ERR_UNKNOWN";
}

const char *sdnn_last_error(void) { return g_last_error.c_str(); }

sdnn_status sdnn_net_arena_size(int64_t n, int32_t L, const int64_t *nnz_per_layer, int32_t dense_flags,
                                int64_t *bytes) {
    g_last_error.clear();
    if (!bytes) return fail(SDNN_ERR_NULL_POINTER, "bytes is NULL");
    sdnn_status st = check_plan_args(n, L, nnz_per_layer, dense_flags);
    if (st != SDNN_OK) return st;
    *bytes = (int64_t)plan_net(n, L, nnz_per_layer, dense_flags).bytes;
    return SDNN_OK;
}

sdnn_status sdnn_net_create(sdnn_net *out, int64_t n, int32_t L, float ymax, const int64_t *nnz_per_layer,
                            int32_t dense_flags, void *arena, int64_t arena_bytes, void *stream) {
    g_last_error.clear();
    if (!out) return fail(SDNN_ERR_NULL_POINTER, "net is NULL");
    *out = nullptr;
    sdnn_status st = check_plan_args(n, L, nnz_per_layer, dense_flags);
    if (st != SDNN_OK) return st;
    if (!(ymax > 0.0f)) return fail(SDNN_ERR_INVALID_VALUE, "ymax must be > 0 (INFINITY for plain ReLU)");
    if (!arena) return fail(SDNN_ERR_NULL_POINTER, "arena is NULL");
    if (((uintptr_t)arena) % kAlign != 0) return fail(SDNN_ERR_INVALID_VALUE, "arena must be 256-byte aligned");
    NetPlan plan = plan_net(n, L, nnz_per_layer, dense_flags);
    if (arena_bytes < (int64_t)plan.bytes)
        return fail(SDNN_ERR_WORKSPACE_TOO_SMALL, "arena smaller than sdnn_net_arena_size(): need " +
                                                      std::to_string(plan.bytes) + " bytes");
    int dev = 0;
    SDNN_HIP(hipGetDevice(&dev));
    hipDeviceProp_t prop;
    SDNN_HIP(hipGetDeviceProperties(&prop, dev));
    if (std::strncmp(prop.gcnArchName, "gfx950", 6) != 0)
        return fail(SDNN_ERR_UNSUPPORTED, std::string("built for gfx950, device is ") + prop.gcnArchName);
    sdnn_net net = new (std::nothrow) sdnn_net_s();
    if (!net) return fail(SDNN_ERR_OUT_OF_MEMORY, "host allocation failed");
    const CaptureScope capture_scope;
    if (const hipError_t e = hipHostMalloc((void **)&net->host, sizeof(sdnn::HostSlot) + kSetupInts * sizeof(uint32_t), hipHostMallocDefault);
        e != hipSuccess) {
        delete net;
        (void)hipGetLastError();
        return fail(SDNN_ERR_OUT_OF_MEMORY, std::string("pinned host allocation failed: ") + hipGetErrorString(e));
    }
    net->host_words = reinterpret_cast<uint32_t *>(net->host + 1);
    net->n = n;
    net->L = L;
    net->ymax = (double)ymax;
    net->stream = (hipStream_t)stream;
    net->device = dev;
    net->num_cu = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 256;
    net->layers.resize((size_t)L);
    net->arena = (char *)arena;
    net->plan = std::move(plan);
    net->caps.assign(nnz_per_layer, nnz_per_layer + L);
    net->dense_flags = dense_flags;
    net->d_flags = at<uint32_t>(net->arena, net->plan.flags);
    net->d_int = at<int32_t>(net->arena, net->plan.d_int);
    net->d_stats = at<unsigned long long>(net->arena, net->plan.stats);
    scratch_init(dev);  // this device's copy of the allocation-free entry point's scratch array
    *out = net;
    return SDNN_OK;
}

sdnn_status sdnn_net_set_stream(sdnn_net net, void *stream) {
    g_last_error.clear();
    if (!net) return fail(SDNN_ERR_INVALID_OBJECT, "net is NULL");
    net->stream = (hipStream_t)stream;
    return SDNN_OK;
}

sdnn_status sdnn_net_set_bias_mode(sdnn_net net, int32_t mode) {
    g_last_error.clear();
    if (!net) return fail(SDNN_ERR_INVALID_OBJECT, "net is NULL");
    if (mode != SDNN_BIAS_EVERYWHERE && mode != SDNN_BIAS_PATTERN) return fail(SDNN_ERR_INVALID_VALUE, "unknown bias mode");
    net->bias_pattern = mode == SDNN_BIAS_PATTERN ? 1 : 0;
    return SDNN_OK;
}

sdnn_status sdnn_net_set_layer(sdnn_net net, int32_t k, int64_t nnz, const int64_t *row_ptr, const int32_t *col_idx,
                               const float *val, const float *bias) {
    g_last_error.clear();
    if (!net) return fail(SDNN_ERR_INVALID_OBJECT, "net is NULL");
    if (k < 0 || k >= net->L) return fail(SDNN_ERR_DIMENSION_MISMATCH, "layer index outside [0, L)");
    if (!row_ptr || !bias) return fail(SDNN_ERR_NULL_POINTER, "row_ptr and bias are required");
    if (nnz < 0 || nnz > 0x7fffffffLL) return fail(SDNN_ERR_INVALID_VALUE, "nnz must be in [0, 2^31-1]");
    if (nnz > 0 && (!col_idx || !val)) return fail(SDNN_ERR_NULL_POINTER, "col_idx and val are required when nnz > 0");
    if (nnz > net->caps[(size_t)k])
        return fail(SDNN_ERR_WORKSPACE_TOO_SMALL, "the arena holds " + std::to_string(net->caps[(size_t)k]) +
                                                      " entries for this layer (sdnn_net_create's nnz_per_layer)");
    const int64_t n = net->n;
    hipStream_t s = net->stream;
    if (n > kMaxScan) return fail(SDNN_ERR_UNSUPPORTED, "layers wider than 2^24 neurons are not supported");
    SDNN_ON_DEVICE(net);

    // 1. validate on the device
    // (the flags and the set-up's integers are cleared together: d_int follows the flags in the arena)
    SDNN_HIP(hipMemsetAsync(net->d_flags, 0, (size_t)((char *)(net->d_int + kSetupInts) - (char *)net->d_flags), s));
    SDNN_HIP(sdnn::launch_validate_layer(n, nnz, row_ptr, col_idx, val, bias, net->d_flags, s));
    const uint32_t *fl = net->host_words;
    SDNN_HIP(hipMemcpyAsync(net->host_words, net->d_flags, 4 * sizeof(uint32_t), hipMemcpyDeviceToHost, s));
    SDNN_HIP(hipStreamSynchronize(s));
    const uint32_t flags = fl[0];
    if (flags & 1u)
        return fail(SDNN_ERR_INVALID_INDEX,
                    "W_k is not valid CSR (row_ptr monotone from 0 to nnz, columns in [0,n) strictly increasing)");
    if (flags & 2u) return fail(SDNN_ERR_INVALID_VALUE, "W_k or b_k holds a non-finite value");

    // 2. derived copies, built in the layer's region of the arena (its previous copies are overwritten; any
    //    forward that still reads them was enqueued earlier on the same stream)
    Layer &l = net->layers[(size_t)k];
    l = Layer();  // not set until the build below completes
    char *base = net->arena + net->plan.layer_off[(size_t)k];
    const LayerPlan &lp = net->plan.layer[(size_t)k];
    Layer nl;
    nl.set = true;
    nl.nnz = nnz;
    nl.row_ptr = row_ptr;
    nl.col = col_idx;
    nl.val = val;
    nl.bias = bias;
    nl.bias_nonpos = (flags & 4u) == 0;
    nl.pos_bias = (int64_t)fl[1];
    {
        // with every b_j <= 0, an accumulated sum at most -max_j b_j gives h(sum + b_j) = 0 for every j
        const uint32_t key = fl[2];
        const uint32_t u = (key & 0x80000000u) ? (key & 0x7fffffffu) : ~key;
        float bmax;
        std::memcpy(&bmax, &u, sizeof(bmax));
        nl.zero_below = nl.bias_nonpos ? -(double)bmax : -INFINITY;
        // fl[3] holds the complement of the smallest key: equal keys mean every b_j has the same bits
        nl.bias_uniform = ~fl[3] == key;
    }
    nl.w_pack = at<Edge>(base, lp.w_pack);
    nl.fan_ptr = at<int64_t>(base, lp.fan_ptr);
    nl.fan = at<Edge>(base, lp.fan);
    // optional structures: present when this layer's density (not only the capacity) wants them
    nl.w_seg = at<int32_t>(base, lp.w_seg);
    nl.sched = at<sdnn::BlockedSched>(base, lp.sched);
    nl.stage = at<Edge>(base, lp.stage);
    sdnn::BlockedRegion *regions = at<sdnn::BlockedRegion>(base, lp.regions);
    int64_t *starts = at<int64_t>(base, lp.starts);
    nl.tile_mask = sdnn::spmm_wants_tiles(n, nnz) ? at<uint16_t>(base, lp.tile_mask) : nullptr;
    nl.slots = sdnn::spmm_wants_slots(n, nnz) ? at<double>(base, lp.slots) : nullptr;
    nl.resident = sdnn::resident_planned(n) ? at<void>(base, lp.resident) : nullptr;
    nl.dense_wt = at<double>(base, lp.dense64);
    nl.dense_wt32 = at<float>(base, lp.dense32);
    int32_t *counts = at<int32_t>(net->arena, net->plan.counts);
    int64_t *tmp = at<int64_t>(net->arena, net->plan.tmp);
    char *sort_scratch = net->arena + net->plan.sort;

    hipError_t e;
#define SETUP_HIP(call)                                  \
    do {                                                 \
        e = (call);                                      \
        if (e != hipSuccess) return fail_hip(e, #call);  \
    } while (0)
    SETUP_HIP(sdnn::launch_pack_edges(nnz, col_idx, val, nl.w_pack, s));
    SETUP_HIP(hipMemsetAsync(counts, 0, (size_t)n * sizeof(int32_t), s));
    SETUP_HIP(sdnn::launch_fanin_counts(nnz, col_idx, counts, s));
    SETUP_HIP(sdnn::launch_exclusive_scan_i32_to_i64(n, counts, nl.fan_ptr, tmp, s));
    SETUP_HIP(sdnn::launch_fanin_lists(n, nnz, row_ptr, col_idx, val, nl.fan, sort_scratch, s));
    SETUP_HIP(hipMemsetAsync(nl.fan + nnz, 0, sizeof(Edge), s));
    SETUP_HIP(sdnn::launch_max_segment(n, row_ptr, net->d_int, s));
    SETUP_HIP(sdnn::launch_max_segment(n, nl.fan_ptr, net->d_int + 2, s));
    if (nl.w_seg) SETUP_HIP(sdnn::launch_window_seg(n, row_ptr, col_idx, nl.w_seg, s));
    if (nl.sched) {
        SETUP_HIP(sdnn::launch_blocked_order(n, nl.fan_ptr, nl.sched, s));
        SETUP_HIP(sdnn::launch_blocked_stage(n, nnz, nl.fan, nl.sched, nl.stage, regions, counts, starts, tmp,
                                             net->d_int + 1, s));
    }
    if (nl.tile_mask) SETUP_HIP(sdnn::launch_spmm_tile_mask(n, nl.fan_ptr, nl.fan, nl.tile_mask, s));
    if (nl.slots) SETUP_HIP(sdnn::launch_spmm_slots(n, nl.fan_ptr, nl.fan, nl.slots, s));
    if (nl.resident) SETUP_HIP(sdnn::launch_resident_lists(n, nl.fan_ptr, nl.fan, nl.resident, net->d_int + 4, s));
    SETUP_HIP(hipMemcpyAsync(net->host_words, net->d_int, kSetupInts * sizeof(int32_t), hipMemcpyDeviceToHost, s));
    SETUP_HIP(hipStreamSynchronize(s));
    nl.max_fanout = (int32_t)net->host_words[0];
    const int32_t region_max = (int32_t)net->host_words[1];
    nl.max_fanin = (int32_t)net->host_words[2];
    nl.resident_blocks = (int32_t)net->host_words[4];
    nl.resident_wave = (int32_t)net->host_words[5];
#undef SETUP_HIP
    // the product stages each workgroup's lists in LDS when the longest region fits; otherwise it reads the
    // same staged copy entry by entry
    if (nl.sched && region_max <= sdnn::blocked_stage_cap()) nl.regions = regions;
    l = nl;
    return SDNN_OK;
}

sdnn_status sdnn_net_build_dense(sdnn_net net) {
    g_last_error.clear();
    if (!net) return fail(SDNN_ERR_INVALID_OBJECT, "net is NULL");
    if (!net->dense_flags) return fail(SDNN_ERR_INVALID_OBJECT, "the arena holds no dense copies (dense_flags 0)");
    SDNN_ON_DEVICE(net);
    const int64_t n = net->n;
    for (int32_t k = 0; k < net->L; ++k) {
        Layer &l = net->layers[(size_t)k];
        if (!l.set) return fail(SDNN_ERR_INVALID_OBJECT, "every layer must be set before build_dense");
        if (l.dense_wt && !l.dense_ready) {
            SDNN_HIP(sdnn::launch_dense_from_fanin(n, l.fan_ptr, l.fan, l.dense_wt, net->stream));
            l.dense_ready = true;
        }
        if (l.dense_wt32 && !l.dense32_ready) {
            SDNN_HIP(sdnn::launch_dense32_from_fanin(n, l.fan_ptr, l.fan, l.dense_wt32, net->stream));
            l.dense32_ready = true;
        }
    }
    SDNN_HIP(hipStreamSynchronize(net->stream));
    return SDNN_OK;
}

sdnn_status sdnn_workspace_size(sdnn_net net, int64_t batch, int32_t y_is_csr, int64_t *bytes) {
    g_last_error.clear();
    if (!net) return fail(SDNN_ERR_INVALID_OBJECT, "net is NULL");
    if (!bytes) return fail(SDNN_ERR_NULL_POINTER, "bytes is NULL");
    if (batch < 0) return fail(SDNN_ERR_INVALID_VALUE, "batch must be >= 0");
    *bytes = y_is_csr ? (int64_t)carve_csr(nullptr, net->n, batch).bytes : (int64_t)dense_ws_bytes(net->n, batch, net->dense_flags, net->num_cu);
    return SDNN_OK;
}

static sdnn_status check_range(sdnn_net net, int32_t k0, int32_t k1) {
    if (k0 < 0 || k1 < k0 || k1 > net->L) return fail(SDNN_ERR_DIMENSION_MISMATCH, "need 0 <= k0 <= k1 <= L");
    for (int32_t k = k0; k < k1; ++k)
        if (!net->layers[(size_t)k].set) return fail(SDNN_ERR_INVALID_OBJECT, "a layer in [k0, k1) is not set");
    return SDNN_OK;
}

static sdnn_status forward_dense_impl(sdnn_net net, int32_t k0, int32_t k1, int64_t batch, const float *Y_in,
                                      float *Y_out, void *ws, int64_t ws_bytes, int32_t arm, bool static_ws);

sdnn_status sdnn_forward_dense(sdnn_net net, int32_t k0, int32_t k1, int64_t batch, const float *Y_in, float *Y_out,
                               void *ws, int64_t ws_bytes, int32_t arm) {
    g_last_error.clear();
    return forward_dense_impl(net, k0, k1, batch, Y_in, Y_out, ws, ws_bytes, arm, false);
}

sdnn_status sdnn_forward_dense_noalloc(sdnn_net net, int32_t k0, int32_t k1, int64_t batch, const float *Y_in,
                                       float *Y_out, int32_t arm) {
    g_last_error.clear();
    return forward_dense_impl(net, k0, k1, batch, Y_in, Y_out, nullptr, 0, arm, true);
}

int64_t sdnn_noalloc_scratch_bytes(void) { return (int64_t)kScratchBytes; }

// Layers [k0, k1) on the LDS-resident product (io.y_in may equal io.y_out unless the plan splits the neurons); buf:
// two buffers of batch x n floats for the layers between separate launches.
static sdnn_status run_resident(sdnn_net net, int32_t k0, int32_t k1, int64_t batch, const ResidentPlan &plan,
                                const sdnn::ResidentIo &io, float *const buf[2]) {
    sdnn::ResidentIo cur = io;
    const int32_t step = plan.fused ? sdnn::kResidentLayers : 1;
    for (int32_t k = k0; k < k1; k += step) {
        sdnn::ResidentLayer rl[sdnn::kResidentLayers];
        const int32_t count = std::min(step, k1 - k);
        for (int32_t i = 0; i < count; ++i) {
            const Layer &l = net->layers[(size_t)(k + i)];
            rl[i] = sdnn::resident_layer(l.resident, net->n, l.bias);
        }
        const bool last = k + count >= k1;
        cur.y_out = last ? io.y_out : buf[((k - k0) / step) & 1];
        cur.cnt_out = last ? io.cnt_out : nullptr;
        int pr = -1;
        SDNN_HIP(prof_begin(net, k, sdnn::kKernResident, &pr));
        SDNN_HIP(sdnn::launch_spmm_resident(rl, count, net->n, batch, plan.v, plan.parts, net->ymax,
                                            net->bias_pattern, cur, net->stream));
        SDNN_HIP(prof_end(net, pr));
        cur = sdnn::ResidentIo();
        cur.y_in = last ? io.y_out : buf[((k - k0) / step) & 1];
    }
    return SDNN_OK;
}

// Layers [k0, k1) on a dense arm, activations in the matrix cores' operand layout throughout; ws holds
// arm_ws_bytes(n, batch, splits) bytes.
static sdnn_status run_arm(sdnn_net net, int32_t k0, int32_t k1, int64_t batch, const float *Y_in, float *Y_out, void *ws,
                           int32_t arm, int splits) {
    const int64_t n = net->n;
    hipStream_t s = net->stream;
    const bool f64 = arm == SDNN_ARM_DENSE;
    const size_t bytes = sdnn::arm_act_bytes(n, batch);
    float *act[2] = {(float *)ws, (float *)((char *)ws + bytes)};
    void *partial = (char *)ws + 2 * bytes;
    int pr = -1;
    SDNN_HIP(prof_begin(net, -1, sdnn::kKernTranspose, &pr));
    SDNN_HIP(sdnn::launch_to_quads(n, batch, f64, Y_in, act[0], s));
    SDNN_HIP(prof_end(net, pr));
    int cur = 0;
    for (int32_t k = k0; k < k1; ++k) {
        const Layer &l = net->layers[(size_t)k];
        SDNN_HIP(prof_begin(net, k, f64 ? sdnn::kKernDenseGemm : sdnn::kKernDenseGemm32, &pr));
        if (f64)
            SDNN_HIP(sdnn::launch_gemm_dense_layer(n, batch, l.dense_wt, l.bias, net->ymax, act[cur], act[cur ^ 1],
                                                   (double *)partial, splits, s));
        else
            SDNN_HIP(sdnn::launch_gemm32_dense_layer(n, batch, l.dense_wt32, l.bias, net->ymax, act[cur], act[cur ^ 1],
                                                     (float *)partial, splits, s));
        SDNN_HIP(prof_end(net, pr));
        cur ^= 1;
    }
    SDNN_HIP(prof_begin(net, -1, sdnn::kKernTranspose, &pr));
    SDNN_HIP(sdnn::launch_from_quads(n, batch, f64, act[cur], Y_out, s));
    SDNN_HIP(prof_end(net, pr));
    return SDNN_OK;
}

static sdnn_status forward_dense_impl(sdnn_net net, int32_t k0, int32_t k1, int64_t batch, const float *Y_in,
                                      float *Y_out, void *ws, int64_t ws_bytes, int32_t arm, bool static_ws) {
    if (!net) return fail(SDNN_ERR_INVALID_OBJECT, "net is NULL");
    sdnn_status st = check_range(net, k0, k1);
    if (st != SDNN_OK) return st;
    if (batch < 0) return fail(SDNN_ERR_DIMENSION_MISMATCH, "batch must be >= 0");
    if (arm != SDNN_ARM_SPARSE && arm != SDNN_ARM_DENSE && arm != SDNN_ARM_DENSE_F32)
        return fail(SDNN_ERR_INVALID_VALUE, "unknown arm");
    if (arm != SDNN_ARM_SPARSE && net->bias_pattern)
        return fail(SDNN_ERR_UNSUPPORTED, "the dense arms store every zero of W_k, so they have no bias pattern");
    if (batch == 0) return SDNN_OK;
    if (!Y_in || !Y_out) return fail(SDNN_ERR_NULL_POINTER, "Y_in and Y_out are required");
    SDNN_ON_DEVICE(net);
    const int64_t n = net->n;
    hipStream_t s = net->stream;
    if (k0 == k1) {
        if (Y_out != Y_in)
            SDNN_HIP(hipMemcpyAsync(Y_out, Y_in, (size_t)batch * (size_t)n * sizeof(float), hipMemcpyDeviceToDevice, s));
        return SDNN_OK;
    }
    int64_t ld = sdnn::act_ld(n, batch);
    if (static_ws) {
        // the library's fixed scratch array of this device replaces the caller's workspace
        const ScratchSlot *slot = net->device < kMaxDevices ? &g_scratch[net->device] : nullptr;
        if (!slot || !slot->ptr)
            return fail(SDNN_ERR_DEVICE, std::string("scratch array of the allocation-free entry point unavailable: ") +
                                             hipGetErrorString(slot ? slot->err : hipErrorInvalidDevice));
        if (sdnn::noalloc_bytes(n, batch, net->num_cu) > kScratchBytes)
            return fail(SDNN_ERR_UNSUPPORTED,
                        "batch x n needs " + std::to_string(sdnn::noalloc_bytes(n, batch, net->num_cu)) +
                            " bytes of scratch; the allocation-free entry point holds " + std::to_string(kScratchBytes));
        if (2 * sdnn::act_bytes(n, ld) > kScratchBytes) ld = sdnn::act_ld_tight(n, batch);
        ws = slot->ptr;
        ws_bytes = (int64_t)kScratchBytes;
    }
    if (!ws) return fail(SDNN_ERR_NULL_POINTER, "ws is required");
    if (!static_ws && ws_bytes < (int64_t)dense_ws_bytes(n, batch, net->dense_flags, net->num_cu))
        return fail(SDNN_ERR_WORKSPACE_TOO_SMALL, "workspace smaller than sdnn_workspace_size(net, batch, 0)");
    for (int32_t k = k0; k < k1; ++k) {
        const Layer &l = net->layers[(size_t)k];
        if ((arm == SDNN_ARM_DENSE && !l.dense_ready) || (arm == SDNN_ARM_DENSE_F32 && !l.dense32_ready))
            return fail(SDNN_ERR_INVALID_OBJECT, "dense arm requested before sdnn_net_build_dense (or without its copy "
                                                 "in the arena)");
    }
    if (arm != SDNN_ARM_SPARSE) {
        const sdnn::ArmPlan plan = sdnn::plan_arm(n, batch, net->num_cu, (size_t)ws_bytes);
        if (plan.rows == 0) return fail(SDNN_ERR_UNSUPPORTED, "one sample does not fit the scratch array");
        // parts in the order in which none overwrites rows of Y_in that a later one reads
        const int64_t parts = (batch + plan.rows - 1) / plan.rows;
        for (int64_t i = 0; i < parts; ++i) {
            const int64_t r0 = ((uintptr_t)Y_out > (uintptr_t)Y_in ? parts - 1 - i : i) * plan.rows;
            st = run_arm(net, k0, k1, std::min(plan.rows, batch - r0), Y_in + r0 * n, Y_out + r0 * n, ws, arm, plan.splits);
            if (st != SDNN_OK) return st;
        }
        return SDNN_OK;
    }
    int pr = -1;
    float *buf[2] = {(float *)ws, (float *)((char *)ws + sdnn::act_bytes(n, ld))};
    if (use_blocked(net, k0, k1, batch)) {
        // the sample-blocked layout (each buffer holds n x ld >= n x round32(batch) floats)
        SDNN_HIP(prof_begin(net, -1, sdnn::kKernTranspose, &pr));
        SDNN_HIP(sdnn::launch_to_blocked(n, batch, n, Y_in, buf[0], s));
        SDNN_HIP(prof_end(net, pr));
        int cb = 0;
        for (int32_t k = k0; k < k1; ++k) {
            const Layer &l = net->layers[(size_t)k];
            SDNN_HIP(prof_begin(net, k, sdnn::kKernBlocked, &pr));
            SDNN_HIP(sdnn::launch_spmm_blocked(n, batch, l.sched, l.stage, l.regions, nullptr, l.bias, net->ymax, net->bias_pattern, buf[cb],
                                               buf[cb ^ 1], nullptr, s));
            SDNN_HIP(prof_end(net, pr));
            cb ^= 1;
        }
        SDNN_HIP(prof_begin(net, -1, sdnn::kKernTranspose, &pr));
        SDNN_HIP(sdnn::launch_from_blocked(n, batch, n, buf[cb], Y_out, s));
        SDNN_HIP(prof_end(net, pr));
        return SDNN_OK;
    }
    if ((Y_in == Y_out || !overlap(Y_in, Y_out, (size_t)batch * (size_t)n))) {
        ResidentPlan plan;
        if (plan_resident(net, k0, k1, batch, Y_in != Y_out, false, &plan)) {
            sdnn::ResidentIo io;
            io.y_in = Y_in;
            io.y_out = Y_out;
            return run_resident(net, k0, k1, batch, plan, io, buf);
        }
    }
    ld = std::min(ld, range_ld(net, k0, k1, batch));
    SDNN_HIP(prof_begin(net, -1, sdnn::kKernTranspose, &pr));
    SDNN_HIP(sdnn::launch_transpose(Y_in, n, buf[0], ld, batch, n, s));  // batch x n -> n x batch
    SDNN_HIP(prof_end(net, pr));
    int cur = 0;
    for (int32_t k = k0; k < k1; ++k) {
        const Layer &l = net->layers[(size_t)k];
        int kind = sdnn::kKernGather;
        SDNN_HIP(prof_begin(net, k, kind, &pr));
        SDNN_HIP(sdnn::launch_spmm_fanin(n, layer_batch(net, l, batch, ld), ld, l.fan_ptr, l.fan, l.tile_mask, l.slots,
                                         l.bias, net->ymax, net->bias_pattern, buf[cur], buf[cur ^ 1], s, &kind));
        SDNN_HIP(prof_end(net, pr, kind));
        cur ^= 1;
    }
    SDNN_HIP(prof_begin(net, -1, sdnn::kKernTranspose, &pr));
    SDNN_HIP(sdnn::launch_transpose(buf[cur], ld, Y_out, n, n, batch, s));  // n x batch -> batch x n
    SDNN_HIP(prof_end(net, pr));
    return SDNN_OK;
}

sdnn_status sdnn_forward_csr(sdnn_net net, int32_t k0, int32_t k1, int64_t batch, const int64_t *y_row_ptr,
                             const int32_t *y_col, const float *y_val, void *ws, int64_t ws_bytes,
                             int64_t *out_row_ptr, int32_t **out_col, float **out_val, int64_t *out_nnz) {
    g_last_error.clear();
    if (!net) return fail(SDNN_ERR_INVALID_OBJECT, "net is NULL");
    sdnn_status st = check_range(net, k0, k1);
    if (st != SDNN_OK) return st;
    if (batch < 0 || batch > 0x7fffffffLL) return fail(SDNN_ERR_DIMENSION_MISMATCH, "batch must be in [0, 2^31-1]");
    if (batch > kMaxScan) return fail(SDNN_ERR_UNSUPPORTED, "CSR batches above 2^24 samples are not supported");
    if (!y_row_ptr || !out_row_ptr || !out_col || !out_val || !out_nnz)
        return fail(SDNN_ERR_NULL_POINTER, "y_row_ptr and the four outputs are required");
    if (!ws) return fail(SDNN_ERR_NULL_POINTER, "ws is required");
    SDNN_ON_DEVICE(net);
    const int64_t n = net->n;
    hipStream_t s = net->stream;
    CsrWs w = carve_csr(ws, n, batch);
    if (ws_bytes < (int64_t)w.bytes)
        return fail(SDNN_ERR_WORKSPACE_TOO_SMALL, "workspace smaller than sdnn_workspace_size(net, batch, 1)");
    if (k0 == k1) {  // identity: copy the input CSR into the workspace
        int64_t in_nnz = 0;
        SDNN_HIP(hipMemcpyAsync(&in_nnz, y_row_ptr + batch, sizeof(int64_t), hipMemcpyDeviceToHost, s));
        SDNN_HIP(hipStreamSynchronize(s));
        if (in_nnz < 0 || in_nnz > batch * n)
            return fail(SDNN_ERR_DIMENSION_MISMATCH, "y_row_ptr[batch] outside [0, batch*n]");
        if (in_nnz > 0 && (!y_col || !y_val)) return fail(SDNN_ERR_NULL_POINTER, "y_col and y_val are required");
        SDNN_HIP(hipMemcpyAsync(out_row_ptr, y_row_ptr, (size_t)(batch + 1) * sizeof(int64_t), hipMemcpyDeviceToDevice, s));
        if (in_nnz > 0) {
            SDNN_HIP(hipMemcpyAsync(w.col[0], y_col, (size_t)in_nnz * sizeof(int32_t), hipMemcpyDeviceToDevice, s));
            SDNN_HIP(hipMemcpyAsync(w.val[0], y_val, (size_t)in_nnz * sizeof(float), hipMemcpyDeviceToDevice, s));
        }
        SDNN_HIP(hipStreamSynchronize(s));
        *out_col = w.col[0];
        *out_val = w.val[0];
        *out_nnz = in_nnz;
        return SDNN_OK;
    }
    if (batch == 0) {  // no samples: an empty result (row_ptr = {0})
        SDNN_HIP(hipMemsetAsync(out_row_ptr, 0, sizeof(int64_t), s));
        SDNN_HIP(hipStreamSynchronize(s));
        *out_col = w.col[0];
        *out_val = w.val[0];
        *out_nnz = 0;
        return SDNN_OK;
    }
    // what the host waits for comes through pinned memory the kernels write to (a copy to pageable memory costs 10 us
    // more than a kernel's store and the same synchronisation); the first report also clears the flags and counters
    SDNN_HIP(sdnn::launch_csr_begin(net->d_flags, net->d_stats, (int64_t)(k1 - k0) * sdnn::kSpgemmStats,
                                    y_row_ptr + batch, net->host, s));
    const sdnn::HostReport report{net->host, net->d_flags};
    auto read_count = [&](int32_t k) -> hipError_t {  // the output entries of sparse layer k, into net->host->nnz
        const unsigned long long *at = net->d_stats + sdnn::kSpgemmStats * (k - k0) + sdnn::kSpgemmStatNnz;
        const hipError_t e = sdnn::launch_report(reinterpret_cast<const int64_t *>(at), report, s);
        return e != hipSuccess ? e : hipStreamSynchronize(s);
    };

    // Activation format per layer.  While outputs are sparse they stay as slot rows (row-wise SpGEMM).
    // From the first layer whose input is dense enough, activations are kept dense and neuron-major and
    // each layer gathers over fan-in lists (the dense-Y product); the result is packed back into rows at
    // the end.  A layer's input counts as dense when it holds at least 1/8 of batch * n entries, or when
    // the layer's bias is positive on at least a quarter of its neurons and applies everywhere (every such
    // neuron is then h(b_j) > 0 in every sample that does not push it below zero, so the output is dense
    // whatever the input).  On the sample-blocked layout the switch comes at 1/16 (measured on n 16384, 32
    // entries per neuron, batch 4096, a 10%-dense input: the SpGEMM takes 0.69 ms and densifying its 5x
    // larger output 0.42 ms; densifying the input 0.15 ms and the blocked product 0.42 ms).  The input size
    // is known on the host only through a synchronisation, so the host keeps an upper bound (a layer whose
    // untouched columns stay zero, every b_j <= 0 or bias on the pattern only, writes at most (longest
    // fan-out row) entries per input entry) and reads the exact count from the device only when the bound
    // reaches the threshold.
    // Where the LDS-resident product takes over it comes at 1/32, for ranges too short to be stopped early at an empty
    // activation (n 3001, 32 entries per neuron, batch 1000, a 10%-dense input: the SpGEMM takes 118 us, the resident
    // product about 12 us per layer and reads the sparse rows itself).
    constexpr int32_t kEmptyCheckLayers = 8;
    ResidentPlan probe;
    const double dense_at =
        (double)batch * (double)n /
        (use_blocked(net, k0, k1, batch) ? 16.0
         : k1 - k0 <= kEmptyCheckLayers && plan_resident(net, k0, k1, batch, false, false, &probe) ? 32.0 : 8.0);
    double nnz_hi = (double)batch * (double)n;  // upper bound of the current layer's input entries
    bool exact = false;
    if (nnz_hi >= dense_at) {
        SDNN_HIP(hipStreamSynchronize(s));
        nnz_hi = (double)net->host->nnz;
        exact = true;
    }
    int32_t kd = k1;
    int cur = 0;  // slot buffer that receives the next sparse layer's output
    // An empty activation stays empty through every layer whose untouched columns stay zero (every b_j <= 0,
    // or the bias on the pattern only).  After the 1st, 2nd, 4th, 8th ... sparse layer, when at least
    // kEmptyCheckLayers such layers follow, the host reads the layer's output count (one synchronisation) and
    // stops at an empty output, which is then Y_{k1} (the deep sparse network dies out this way after its
    // second layer; the rest would cost launches only).
    int64_t next_check = 1;
    for (int32_t k = k0; k < k1; ++k) {
        const Layer &l = net->layers[(size_t)k];
        if (!net->bias_pattern && 4 * l.pos_bias >= n) {
            kd = k;
            break;
        }
        if (nnz_hi >= dense_at && !exact) {
            SDNN_HIP(read_count(k - 1));
            nnz_hi = (double)net->host->nnz;
            exact = true;
        }
        if (nnz_hi >= dense_at) {
            kd = k;
            break;
        }
        const bool first = k == k0;
        int pr = -1;
        SDNN_HIP(prof_begin(net, k, sdnn::kKernSpgemm, &pr));
        SDNN_HIP(sdnn::launch_spgemm_layer(n, batch, first ? y_row_ptr : nullptr, first ? nullptr : w.cnt[cur ^ 1],
                                           first ? y_col : w.col[cur ^ 1], first ? y_val : w.val[cur ^ 1], l.row_ptr,
                                           l.w_seg, l.w_pack, l.nnz, l.max_fanout, l.bias, l.bias_nonpos ? 1 : 0,
                                           l.bias_uniform ? 1 : 0, l.zero_below,
                                           net->bias_pattern, net->ymax, w.cnt[cur], w.col[cur], w.val[cur], w.lists,
                                           net->d_stats + sdnn::kSpgemmStats * (k - k0), net->d_flags, net->num_cu, s));
        SDNN_HIP(prof_end(net, pr));
        cur ^= 1;
        const double full = (double)batch * (double)n;
        nnz_hi = (l.bias_nonpos || net->bias_pattern) ? std::min(full, nnz_hi * (double)l.max_fanout) : full;
        exact = false;
        if (k - k0 + 1 == next_check) {
            next_check *= 2;
            bool stays_empty = k1 - k - 1 >= kEmptyCheckLayers;
            for (int32_t j = k + 1; stays_empty && j < k1; ++j)
                stays_empty = net->layers[(size_t)j].bias_nonpos || net->bias_pattern;
            if (stays_empty) {
                SDNN_HIP(read_count(k));
                nnz_hi = (double)net->host->nnz;
                exact = true;
                if (net->host->nnz == 0) break;  // Y_{k+1} is empty, and so is every later activation
            }
        }
    }
    int outb;  // the buffer the packed CSR goes to
    if (kd < k1 && use_blocked(net, kd, k1, batch)) {
        // dense activations in the sample-blocked layout, packed straight into CSR at the end
        const bool from_user = kd == k0;
        const int db = from_user ? 0 : cur;  // the input rows (if any) sit in buffer cur ^ 1
        float *dense[2] = {reinterpret_cast<float *>(w.col[db]), w.val[db]};
        // a sparse input (at most 1/16 of batch * n entries: a 32-sample row is then entirely zero with
        // probability >= (15/16)^32, about 13%, at uniform density): the first product skips the zero rows
        // (only when the first layer stages its lists: the product reads the map only then, and densify does
        // not store the zero rows when it writes one)
        uint32_t *nz = (nnz_hi <= (double)batch * (double)n / 16.0 && net->layers[(size_t)kd].regions) ? w.nzrows : nullptr;
        int pr = -1;
        SDNN_HIP(prof_begin(net, -1, sdnn::kKernDensify, &pr));
        SDNN_HIP(sdnn::launch_densify_blocked(n, batch, from_user ? y_row_ptr : nullptr, from_user ? nullptr : w.cnt[cur ^ 1],
                                              from_user ? y_col : w.col[cur ^ 1], from_user ? y_val : w.val[cur ^ 1],
                                              dense[0], nz, net->d_flags, s));
        SDNN_HIP(prof_end(net, pr));
        int dc = 0;
        // the last product counts its nonzeros for the packing, into the value buffer the packed rows go to (at least
        // n * batch floats, a thirty-second of it used: n * batch / 8 bytes; free until then)
        uint8_t *counts = net->layers[(size_t)(k1 - 1)].regions ? reinterpret_cast<uint8_t *>(w.val[db ^ 1]) : nullptr;
        for (int32_t k = kd; k < k1; ++k) {
            const Layer &l = net->layers[(size_t)k];
            SDNN_HIP(prof_begin(net, k, sdnn::kKernBlocked, &pr));
            SDNN_HIP(sdnn::launch_spmm_blocked(n, batch, l.sched, l.stage, l.regions, k == kd ? nz : nullptr, l.bias,
                                               net->ymax, net->bias_pattern, dense[dc], dense[dc ^ 1],
                                               k + 1 == k1 ? counts : nullptr, s));
            SDNN_HIP(prof_end(net, pr));
            dc ^= 1;
        }
        SDNN_HIP(prof_begin(net, -1, sdnn::kKernPack, &pr));
        SDNN_HIP(sdnn::launch_blocked_to_csr(n, batch, dense[dc], counts, w.pcnt, w.cnt[db ^ 1], out_row_ptr, w.scan_tmp, report,
                                             w.col[db ^ 1], w.val[db ^ 1], s));
        SDNN_HIP(prof_end(net, pr));
        outb = db ^ 1;
    } else if (kd < k1) {
        const bool from_user = kd == k0;
        const int db = from_user ? 0 : cur;  // the input rows (if any) sit in buffer cur ^ 1
        // two buffers of n x batch floats at row pitch ld
        float *dense[2] = {reinterpret_cast<float *>(w.col[db]), w.val[db]};
        const int64_t ld = range_ld(net, kd, k1, batch);
        ResidentPlan plan;
        int pr = -1;
        int dc = 0;
        const float *rows;  // Y_{k1}, batch-major
        bool counted = false;
        if (plan_resident(net, kd, k1, batch, false, false, &plan)) {
            // the sparse rows go straight into the product's LDS, and its last launch counts the nonzeros of every row
            sdnn::ResidentIo io;
            io.row_ptr = from_user ? y_row_ptr : nullptr;
            io.cnt_in = from_user ? nullptr : w.cnt[cur ^ 1];
            io.col = from_user ? y_col : w.col[cur ^ 1];
            io.val = from_user ? y_val : w.val[cur ^ 1];
            io.err = net->d_flags;
            io.y_out = dense[0];
            io.cnt_out = w.cnt[db];
            sdnn_status rs = run_resident(net, kd, k1, batch, plan, io, dense);
            if (rs != SDNN_OK) return rs;
            rows = dense[0];
            counted = true;
        } else {
            // dense[1] is free until the first layer: it stages the rows batch-major when they hold at least a
            // quarter of batch * n entries (measured on MI355X: 0.34 instead of 0.69 ms for 32M entries into
            // 16384 x 4096; at 2% density the extra transpose costs more than the scattered stores it saves)
            float *stage = nnz_hi >= (double)batch * (double)n / 4.0 ? dense[1] : nullptr;
            SDNN_HIP(prof_begin(net, -1, sdnn::kKernDensify, &pr));
            SDNN_HIP(sdnn::launch_densify(n, batch, ld, from_user ? y_row_ptr : nullptr,
                                          from_user ? nullptr : w.cnt[cur ^ 1], from_user ? y_col : w.col[cur ^ 1],
                                          from_user ? y_val : w.val[cur ^ 1], dense[0], stage, net->d_flags, s));
            SDNN_HIP(prof_end(net, pr));
            for (int32_t k = kd; k < k1; ++k) {
                const Layer &l = net->layers[(size_t)k];
                int kind = sdnn::kKernGather;
                SDNN_HIP(prof_begin(net, k, kind, &pr));
                SDNN_HIP(sdnn::launch_spmm_fanin(n, layer_batch(net, l, batch, ld), ld, l.fan_ptr, l.fan, l.tile_mask,
                                                 l.slots, l.bias, net->ymax, net->bias_pattern, dense[dc],
                                                 dense[dc ^ 1], s, &kind));
                SDNN_HIP(prof_end(net, pr, kind));
                dc ^= 1;
            }
            rows = dense[dc ^ 1];
        }
        SDNN_HIP(prof_begin(net, -1, sdnn::kKernPack, &pr));
        if (!counted) SDNN_HIP(sdnn::launch_transpose(dense[dc], ld, dense[dc ^ 1], n, n, batch, s));  // -> batch x n
        SDNN_HIP(sdnn::launch_dense_to_csr(n, batch, rows, counted ? w.cnt[db] : w.cnt[db ^ 1], counted, out_row_ptr,
                                           w.scan_tmp, report, w.col[db ^ 1], w.val[db ^ 1], s));
        outb = db ^ 1;
        SDNN_HIP(prof_end(net, pr));
    } else {
        const int last = cur ^ 1;  // slot buffer holding Y_{k1}
        outb = cur;
        int pr = -1;
        SDNN_HIP(prof_begin(net, -1, sdnn::kKernCompact, &pr));
        SDNN_HIP(sdnn::launch_row_ptr(batch, w.cnt[last], out_row_ptr, w.scan_tmp, report, s));
        SDNN_HIP(sdnn::launch_compact_rows(n, batch, w.cnt[last], out_row_ptr, w.col[last], w.val[last],
                                           w.col[outb], w.val[outb], s));
        SDNN_HIP(prof_end(net, pr));
    }
    SDNN_HIP(hipStreamSynchronize(s));
    const int64_t nnz = net->host->nnz;
    const uint32_t flags = net->host->flags;
    if (flags & 1u)
        return fail(SDNN_ERR_INVALID_INDEX, "Y_in is not valid CSR (row extents or column indices out of range)");
    *out_col = w.col[outb];
    *out_val = w.val[outb];
    *out_nnz = nnz;
    return SDNN_OK;
}

static sdnn_status mxm_common(sdnn_net net, int32_t k, int32_t semiring, int64_t batch, void *ws, int64_t ws_bytes,
                              bool needs_ws) {
    if (!net) return fail(SDNN_ERR_INVALID_OBJECT, "net is NULL");
    if (k < 0 || k >= net->L) return fail(SDNN_ERR_DIMENSION_MISMATCH, "layer index outside [0, L)");
    if (!net->layers[(size_t)k].set) return fail(SDNN_ERR_INVALID_OBJECT, "layer k is not set");
    if (semiring < SDNN_SEMIRING_PLUS_TIMES || semiring > SDNN_SEMIRING_XOR_AND)
        return fail(SDNN_ERR_INVALID_VALUE, "unknown semiring");
    if (batch < 0) return fail(SDNN_ERR_DIMENSION_MISMATCH, "batch must be >= 0");
    if (!needs_ws) return SDNN_OK;
    if (batch > 0 && !ws) return fail(SDNN_ERR_NULL_POINTER, "ws is required");
    if (batch > 0 && ws_bytes < (int64_t)dense_ws_bytes(net->n, batch, net->dense_flags, net->num_cu))
        return fail(SDNN_ERR_WORKSPACE_TOO_SMALL, "workspace smaller than sdnn_workspace_size(net, batch, 0)");
    return SDNN_OK;
}

sdnn_status sdnn_mxm_dense(sdnn_net net, int32_t k, int32_t semiring, int64_t batch, const float *Y, float *Z,
                           void *ws, int64_t ws_bytes) {
    g_last_error.clear();
    sdnn_status st = mxm_common(net, k, semiring, batch, ws, ws_bytes, true);
    if (st != SDNN_OK || batch == 0) return st;
    if (!Y || !Z) return fail(SDNN_ERR_NULL_POINTER, "Y and Z are required");
    SDNN_ON_DEVICE(net);
    const int64_t n = net->n;
    hipStream_t s = net->stream;
    const Layer &l = net->layers[(size_t)k];
    ResidentPlan plan;
    if ((Y == Z || !overlap(Y, Z, (size_t)batch * (size_t)n)) && plan_resident(net, k, k + 1, batch, Y != Z, true, &plan)) {
        SDNN_HIP(sdnn::launch_semiring_resident(semiring, sdnn::resident_layer(l.resident, n, nullptr), n, batch, plan.v,
                                                plan.parts, Y, Z, s));
        return SDNN_OK;
    }
    const int64_t ld = sdnn::act_ld(n, batch);
    float *yt = (float *)ws;
    float *zt = (float *)((char *)ws + sdnn::act_bytes(n, ld));
    SDNN_HIP(sdnn::launch_transpose(Y, n, yt, ld, batch, n, s));  // batch x n -> n x batch
    // rounded up to a multiple of four where that gives the gather two or four columns per lane, unless one long list
    // sets its time
    const int64_t up = (batch + 3) / 4 * 4;
    const bool round = up >= 128 && up <= ld && !sdnn::spmm_long_list(n, l.nnz, l.max_fanin, batch);
    SDNN_HIP(sdnn::launch_semiring_mxm(semiring, n, round ? up : batch, ld, l.fan_ptr, l.fan, yt, zt, s));
    SDNN_HIP(sdnn::launch_transpose(zt, ld, Z, n, n, batch, s));  // n x batch -> batch x n
    return SDNN_OK;
}

sdnn_status sdnn_mxm_csr(sdnn_net net, int32_t k, int32_t semiring, int64_t batch, const int64_t *y_row_ptr,
                         const int32_t *y_col, const float *y_val, float *Z, void *ws, int64_t ws_bytes) {
    g_last_error.clear();
    (void)ws;
    (void)ws_bytes;
    sdnn_status st = mxm_common(net, k, semiring, batch, ws, ws_bytes, false);
    if (st != SDNN_OK || batch == 0) return st;
    if (!y_row_ptr || !Z) return fail(SDNN_ERR_NULL_POINTER, "y_row_ptr and Z are required");
    SDNN_ON_DEVICE(net);
    const int64_t n = net->n;
    hipStream_t s = net->stream;
    const Layer &l = net->layers[(size_t)k];
    SDNN_HIP(sdnn::launch_csr_begin(net->d_flags, net->d_stats, 0, y_row_ptr + batch, net->host, s));
    // row by row over the stored entries (the SpGEMM skeleton): Y is never densified
    SDNN_HIP(sdnn::launch_semiring_rows(semiring, n, batch, l.nnz, y_row_ptr, y_col, y_val, l.row_ptr, l.w_pack, Z,
                                        net->d_flags, s));
    SDNN_HIP(sdnn::launch_report(y_row_ptr + batch, sdnn::HostReport{net->host, net->d_flags}, s));
    SDNN_HIP(hipStreamSynchronize(s));
    const uint32_t flags = net->host->flags;
    if (flags & 1u) return fail(SDNN_ERR_INVALID_INDEX, "Y is not valid CSR (row extents or column indices out of range)");
    return SDNN_OK;
}

sdnn_status sdnn_net_set_profiling(sdnn_net net, int32_t enable) {
    g_last_error.clear();
    if (!net) return fail(SDNN_ERR_INVALID_OBJECT, "net is NULL");
    if (enable) prof_clear(net);
    net->profiling = enable != 0;
    return SDNN_OK;
}

sdnn_status sdnn_net_read_profile(sdnn_net net, sdnn_kernel_time *out, int32_t max_records, int32_t *count) {
    g_last_error.clear();
    if (!net) return fail(SDNN_ERR_INVALID_OBJECT, "net is NULL");
    if (!count || (max_records > 0 && !out)) return fail(SDNN_ERR_NULL_POINTER, "count (and out) are required");
    SDNN_ON_DEVICE(net);
    SDNN_HIP(hipStreamSynchronize(net->stream));
    *count = (int32_t)std::min<size_t>(net->prof.size(), 0x7fffffff);
    for (size_t i = 0; i < net->prof.size() && (int64_t)i < (int64_t)max_records; ++i) {
        float ms = 0.0f;
        SDNN_HIP(hipEventElapsedTime(&ms, net->prof[i].a, net->prof[i].b));
        out[i].layer = net->prof[i].layer;
        out[i].kernel = net->prof[i].kernel;
        out[i].ms = ms;
    }
    prof_clear(net);
    return SDNN_OK;
}

sdnn_status sdnn_net_free(sdnn_net net) {
    g_last_error.clear();
    if (!net) return SDNN_OK;
    DeviceScope device_scope(net->device);  // frees on the net's device even if it cannot be made current
    (void)hipStreamSynchronize(net->stream);
    prof_clear(net);
    for (hipEvent_t e : net->ev_free) (void)hipEventDestroy(e);
    (void)hipHostFree(net->host);
    delete net;  // the arena belongs to the caller
    return SDNN_OK;
}

}  // extern "C"
