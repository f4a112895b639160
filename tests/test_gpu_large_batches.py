"""Batches whose launches would exceed 2^32 work-items in one piece: the result must be that of the same rows in smaller
calls, bit for bit."""

import numpy as np
import pytest

from tests.test_gpu_parity import _mixed_length_layer
from workloads import Problem

pytestmark = pytest.mark.gpu

N, CHUNK = 256, 1 << 21


def _net(sd):
    layer = _mixed_length_layer(np.random.default_rng(3), N, [16, 12, 20])
    layer.bias[:] = -0.2
    return sd.net_from_problem(Problem("large-batch", N, 1, 1, float("inf"), [layer]))


def test_dense_batch_past_one_launch_of_the_resident_product():
    """16,777,213 samples, four per workgroup of 1024 threads, reach 2^32 work-items: forward and semiring multiply."""
    import torch

    import paper_1708_02937_amd as sd

    net = _net(sd)
    batch = (1 << 24) + 1001
    g = torch.Generator(device="cuda").manual_seed(1)
    y = torch.rand((batch, N), generator=g, device="cuda")
    out = torch.empty_like(y)
    print("[case] large dense batch", batch, flush=True)
    net.set_profiling(True)
    net.forward_dense(y, out=out)
    assert [name for _, name, _ in net.read_profile()] == ["spmm_resident_kernel"]
    net.set_profiling(False)
    want = torch.empty((CHUNK, N), device="cuda")
    for r in range(0, batch, CHUNK):
        part = y[r:r + CHUNK]
        assert torch.equal(out[r:r + CHUNK], net.forward_dense(part, out=want[:part.shape[0]]))
    print("[case] large dense batch, max.+", flush=True)
    net.mxm(0, sd.SDNN_SEMIRING_MAX_PLUS, y, out=out)
    for r in range(0, batch, CHUNK):
        part = y[r:r + CHUNK]
        assert torch.equal(out[r:r + CHUNK], net.mxm(0, sd.SDNN_SEMIRING_MAX_PLUS, part, out=want[:part.shape[0]]))
    net.free()


def test_csr_batch_past_one_launch_of_the_packing():
    """4,194,304 rows of a 1024-thread workgroup each reach 2^32 work-items in the packing of a dense result."""
    import torch

    import paper_1708_02937_amd as sd

    net = _net(sd)
    batch = (1 << 22) + 1001
    g = torch.Generator(device="cuda").manual_seed(2)
    mask = torch.rand((batch, N), generator=g, device="cuda") < 1 / 16
    rp = torch.zeros(batch + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(mask.sum(1), 0, out=rp[1:])
    col = mask.nonzero()[:, 1].to(torch.int32)
    val = torch.rand(col.numel(), generator=g, device="cuda") + 0.1
    del mask
    print("[case] large csr batch", batch, flush=True)
    got_rp, got_col, got_val = (x.clone() for x in net.forward_csr(rp, col, val))
    assert 0 < got_col.numel() == int(got_rp[-1])
    for r in range(0, batch, CHUNK):
        e = min(batch, r + CHUNK)
        a, b = int(rp[r]), int(rp[e])
        want = net.forward_csr(rp[r:e + 1] - a, col[a:b], val[a:b])
        ga, gb = int(got_rp[r]), int(got_rp[e])
        assert torch.equal(got_rp[r:e + 1] - ga, want[0])
        assert torch.equal(got_col[ga:gb], want[1]) and torch.equal(got_val[ga:gb], want[2])
    net.free()
