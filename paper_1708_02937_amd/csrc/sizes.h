// Sizes of the dense-Y paths' buffers: plain host arithmetic, without HIP.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>

namespace sdnn {

inline size_t align_up(size_t x) { return (x + 255) / 256 * 256; }

// Row pitch (floats) of the neuron-major activation buffers Y^T (n rows of `batch` samples).  Lines taken one
// per row at a power-of-two byte pitch fall into a fraction of an XCD's L2 sets (measured on MI355X: at a
// 16 KiB pitch a 1 MiB working set already misses about half the time, at 16 KiB + 256 B a 3 MiB one stays
// resident), so for wide layers (n > 4096) of 256 samples or more the pitch is an odd multiple of 64 floats
// (256 bytes).  At n = 4096, batch 1024 the padding measured 1-3% slower per layer, so narrower layers and
// smaller batches keep the dense pitch, rounded up to whole 16-byte loads.
inline int64_t act_ld(int64_t n, int64_t batch) {
    return (n <= 4096 || batch < 256) ? (batch + 3) / 4 * 4 : (((batch + 63) / 64) | 1) * 64;
}
// The same without the rounding, for a workspace that has no room for it.
inline int64_t act_ld_tight(int64_t n, int64_t batch) {
    return (n <= 4096 || batch < 256) ? batch : act_ld(n, batch);
}
// Bytes of one neuron-major activation buffer at row pitch ld.
inline size_t act_bytes(int64_t n, int64_t ld) { return align_up((size_t)n * (size_t)ld * sizeof(float)); }

// The dense-W arms: a workgroup computes kGemmM outputs of kGemmN samples over K blocks of kGemmK, and the operand
// layout pads K to kGemmKPad.
constexpr int kGemmM = 128, kGemmN = 64, kGemmK = 16, kGemmKPad = 32;
inline int64_t gemm_k_blocks(int64_t n) { return (n + kGemmKPad - 1) / kGemmKPad * (kGemmKPad / kGemmK); }
inline int64_t gemm_m_pitch(int64_t n) { return (n + kGemmM - 1) / kGemmM * kGemmM; }
// values of one dense copy of a layer
inline size_t gemm_weight_elems(int64_t n) { return (size_t)(gemm_k_blocks(n) * kGemmK) * (size_t)gemm_m_pitch(n); }
// floats of one activation buffer
inline size_t gemm_act_elems(int64_t n, int64_t batch) { return (size_t)(gemm_k_blocks(n) * kGemmK) * (size_t)batch; }

// K splits for an n x n layer on `batch` samples: enough workgroups for two per CU, at least 128 inputs (four K steps)
// each.
inline int gemm_splits(int64_t n, int64_t batch, int num_cu) {
    const int64_t tiles = ((n + kGemmM - 1) / kGemmM) * ((batch + kGemmN - 1) / kGemmN);
    if (tiles == 0 || tiles >= 2 * (int64_t)num_cu) return 1;
    const int64_t sp = std::min<int64_t>({(2 * (int64_t)num_cu + tiles - 1) / tiles, n / 128, 64});
    return sp < 1 ? 1 : (int)sp;
}

// Workspace of a dense arm: two activation buffers in its operand layout, and the sums of `splits` K splits in fp64.
inline size_t arm_act_bytes(int64_t n, int64_t batch) { return align_up(gemm_act_elems(n, batch) * sizeof(float)); }
inline size_t arm_ws_bytes(int64_t n, int64_t batch, int splits) {
    const size_t sums = splits > 1 ? (size_t)splits * gemm_act_elems(n, batch) * sizeof(double) : 0;
    return 2 * arm_act_bytes(n, batch) + align_up(sums);
}

// What decides whether the fixed scratch array takes a batch: two buffers of n x batch and fp64 sums of every K split.
inline size_t noalloc_bytes(int64_t n, int64_t batch, int num_cu) {
    const int sp = gemm_splits(n, batch, num_cu);
    const size_t sums = sp > 1 ? (size_t)sp * (size_t)n * (size_t)batch * sizeof(double) : 0;
    return 2 * act_bytes(n, act_ld_tight(n, batch)) + align_up(sums);
}

// How a dense arm runs a batch in a workspace of `bytes`: the K splits of the whole batch (which fix the order of the
// sums) and the samples per part, all of them where the workspace has room for the padding of the operand layout, else
// as many whole 64-sample tiles as it takes (single samples below one tile); 0 where not even one sample fits.
struct ArmPlan {
    int64_t rows;
    int splits;
};
inline ArmPlan plan_arm(int64_t n, int64_t batch, int num_cu, size_t bytes) {
    ArmPlan p{batch, gemm_splits(n, batch, num_cu)};
    if (arm_ws_bytes(n, batch, p.splits) <= bytes) return p;
    p.rows = std::min<int64_t>(batch, (int64_t)(bytes / arm_ws_bytes(n, 64, p.splits) * 64));
    if (p.rows == 0)
        for (p.rows = std::min<int64_t>(batch, 63); p.rows > 0 && arm_ws_bytes(n, p.rows, p.splits) > bytes;) --p.rows;
    return p;
}

}  // namespace sdnn
