"""Host arithmetic of the dense-Y paths' buffers (csrc/sizes.h), compiled by g++ and looped over sizes without a GPU."""

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SCRATCH = r"""
#include <cstdio>
#include "sizes.h"
using namespace sdnn;

// Every batch the 64 MiB array accepts by its n x batch buffers must run on a dense arm: in parts that fit, at the whole
// batch's K splits.
int main() {
    const size_t cap = size_t(64) << 20;
    const int cu = 256;
    long checked = 0, in_parts = 0, bad = 0;
    auto check = [&](int64_t n, int64_t batch) {
        if (batch < 1 || noalloc_bytes(n, batch, cu) > cap) return;
        const ArmPlan p = plan_arm(n, batch, cu, cap);
        ++checked;
        in_parts += p.rows < batch;
        const bool ok = p.rows >= 1 && p.rows <= batch && p.splits == gemm_splits(n, batch, cu) &&
                        arm_ws_bytes(n, p.rows, p.splits) <= cap && (p.rows == batch || p.rows % 64 == 0 || p.rows < 64);
        if (!ok && ++bad <= 5) std::printf("n %ld batch %ld rows %ld splits %d\n", (long)n, (long)batch, (long)p.rows, p.splits);
    };
    for (int64_t n = 1; n < 20000; ++n) {
        const int64_t most = (int64_t)(cap / (8 * (size_t)n));  // two buffers fill the array
        for (int64_t d = 0; d < 40; ++d) check(n, most - d);
        for (int64_t b : {most / 2, most / 3, most / 5, most / 9, most / 17}) {  // with sums of 2, 4, 8 ... splits
            for (int64_t d = -70; d <= 70; d += 7) check(n, b + d);
        }
        check(n, 1);
    }
    for (int64_t n = 20000; n < 140000; n += 37)
        for (int64_t d = 0; d < 4; ++d) check(n, (int64_t)(cap / (8 * (size_t)n)) - d);
    // the named sizes: accepted, in parts, and half of the batch alone would ask for more sums than fit
    const int64_t named[][2] = {{3835, 2185}, {609, 13108}, {639, 13108}, {1914, 4378}};
    for (const auto &c : named) {
        check(c[0], c[1]);
        if (noalloc_bytes(c[0], c[1], cu) > cap || plan_arm(c[0], c[1], cu, cap).rows == c[1]) ++bad;
    }
    std::printf("%ld checked, %ld in parts, %ld bad\n", checked, in_parts, bad);
    return bad || !in_parts ? 1 : 0;
}
"""


def _run(tmp_path, source):
    src, exe = tmp_path / "sizes.cpp", tmp_path / "sizes"
    src.write_text(source)
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_1708_02937_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
    return r.stdout


def test_scratch_array_parts_fit_every_accepted_batch(tmp_path):
    print(_run(tmp_path, SCRATCH))
