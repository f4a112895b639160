"""Nets beside a graph capture, and calls whose output overlaps their input."""

import threading

import numpy as np
import pytest

from workloads import tiny_random

pytestmark = pytest.mark.gpu


def test_net_created_while_another_thread_captures():
    """The pinned slot a net allocates must not break a capture that another thread records in global mode; the graph is
    replayed three times, with eager work between."""
    import torch

    import paper_1708_02937_amd as sd

    p = tiny_random(11, 600, 2, 70, w_density=0.03, dense_input=True, y_density=0.5)
    net = sd.net_from_problem(p)
    y = torch.from_numpy(p.y0_dense).cuda()
    want = net.forward_dense(y)
    out, ws = torch.empty_like(y), net.workspace(70, 0)
    arena = torch.empty(sd.sdnn_net_arena_size(300, 1, [900], 0), dtype=torch.uint8, device="cuda")
    side = torch.cuda.Stream()
    made, failed = [], []

    def other():
        try:
            made.append(sd.sdnn_net_create(300, 1, 1.0, [900], 0, arena, arena.numel(), side.cuda_stream))
        except Exception as e:  # reported by the capturing thread
            failed.append(e)

    g = torch.cuda.CUDAGraph()
    print("[case] net beside a capture", flush=True)
    prev = torch.cuda.current_stream().cuda_stream
    try:
        with torch.cuda.graph(g, stream=torch.cuda.Stream()):
            sd.sdnn_net_set_stream(net.handle, torch.cuda.current_stream().cuda_stream)
            t = threading.Thread(target=other)
            t.start()
            t.join(60)
            sd.sdnn_forward_dense(net.handle, 0, 2, 70, y, out, ws, ws.numel(), sd.SDNN_ARM_SPARSE)
    finally:
        sd.sdnn_net_set_stream(net.handle, prev)
    assert made and not failed
    sd.sdnn_net_free(made[0])
    for _ in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        assert torch.equal(net.forward_dense(y), want)
    net.free()


@pytest.mark.parametrize("n,batch,arm", [(300, 50, 0), (3000, 520, 0), (5200, 131, 0), (4500, 300, 0), (300, 50, 1), (300, 50, 2),
                                         (700, 40, "mxm"), (6000, 40, "mxm")])
def test_output_overlapping_the_input(n, batch, arm):
    """Y_out a few rows or elements before or after Y_in, on every product: as with an output of its own."""
    import torch

    import paper_1708_02937_amd as sd

    p = tiny_random(13, n, 2, 4, w_density=20 / n, dense_input=True, bias_lo=-0.1, bias_hi=0.1)
    net = sd.net_from_problem(p, dense=arm if arm in (1, 2) else 0)
    y = torch.from_numpy(np.random.default_rng(n).random((batch, n), dtype=np.float32)).cuda()

    def call(src, dst):
        if arm == "mxm":
            return net.mxm(0, sd.SDNN_SEMIRING_MAX_PLUS, src, out=dst)
        return net.forward_dense(src, arm=arm, out=dst)

    want = call(y, torch.empty_like(y))
    for shift in (3 * n, -3 * n, 7, -7):
        print("[case] overlap", n, batch, arm, shift, flush=True)
        room = torch.empty(batch * n + 3 * n, device="cuda")
        lo = max(0, -shift)
        src = room[lo:lo + batch * n].view(batch, n)
        src.copy_(y)
        dst = room[lo + shift:lo + shift + batch * n].view(batch, n)
        assert torch.equal(call(src, dst), want)
    net.free()
