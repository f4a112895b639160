"""The dense-W arms at the edges of their tiles (16-row blocks, K steps of 32, tiles of 128 outputs x 64 samples), with and
without split K, and on the fixed scratch array where their padded layout does not fit whole."""

import numpy as np
import pytest

from tests import parity
from workloads import dense_to_csr, integer_shadow, tiny_random

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("arm", ["f64", "f32"])
@pytest.mark.parametrize("n,batch,L", [(1, 1, 2), (15, 63, 2), (17, 64, 1), (31, 65, 2), (33, 1, 2), (127, 130, 2), (129, 5, 2),
                                       (256, 64, 1), (1000, 257, 2), (2049, 33, 1), (4127, 64, 1)])
def test_tile_edges(arm, n, batch, L):
    """Integer values: sums stay exact in fp32 too, so both arms match the oracle bit for bit."""
    import torch

    import paper_1708_02937_amd as sd

    p = integer_shadow(tiny_random(n, n, L, batch, w_density=min(1.0, 20 / n), y_density=0.6, dense_input=True))
    print("[case] dense arm", arm, n, batch, L, flush=True)
    code, flag = {"f64": (sd.SDNN_ARM_DENSE, 1), "f32": (sd.SDNN_ARM_DENSE_F32, 2)}[arm]
    net = sd.net_from_problem(p, dense=flag)
    y = torch.from_numpy(p.y0_dense).cuda()
    got = net.forward_dense(y, arm=code).cpu().numpy()
    net.forward_dense(y, arm=code, out=y)  # in place
    net.free()
    assert y.cpu().numpy().tobytes() == got.tobytes()
    parity.compare(p, dense_to_csr(got), exact=True)


@pytest.mark.parametrize("arm", ["f64", "f32"])
def test_scratch_array_in_halves(arm):
    """A batch the scratch array takes by its n x batch buffers, but not with K padded to 32, runs as two halves; in
    place as well."""
    import torch

    import paper_1708_02937_amd as sd

    n = 1001
    batch = sd.sdnn_noalloc_scratch_bytes() // (8 * n)
    assert 8 * 1024 * batch > sd.sdnn_noalloc_scratch_bytes()
    p = tiny_random(3, n, 1, 4, w_density=0.02, dense_input=True)
    code, flag = {"f64": (sd.SDNN_ARM_DENSE, 1), "f32": (sd.SDNN_ARM_DENSE_F32, 2)}[arm]
    net = sd.net_from_problem(p, dense=flag)
    y = torch.from_numpy(np.random.default_rng(2).random((batch, n), dtype=np.float32)).cuda()
    want = net.forward_dense(y, arm=code)
    out = torch.empty_like(y)
    print("[case] scratch halves", arm, batch, flush=True)
    sd.sdnn_forward_dense_noalloc(net.handle, 0, 1, batch, y, out, code)
    assert torch.equal(out, want)
    sd.sdnn_forward_dense_noalloc(net.handle, 0, 1, batch, y, y, code)
    assert torch.equal(y, want)
    net.free()


@pytest.mark.parametrize("arm", ["f64", "f32"])
@pytest.mark.parametrize("n,batch", [(639, 13108), (3835, 2185)])
def test_scratch_array_parts_keep_the_splits(arm, n, batch):
    """Batches of which a half alone has few enough tiles to ask for K splits the whole batch has none of: the parts run
    at the whole batch's splits, so the result is that of the workspace entry point bit for bit; out of place, in place,
    and with the output shifted by a few rows over the input in either direction."""
    import torch

    import paper_1708_02937_amd as sd

    p = tiny_random(3, n, 1, 4, w_density=0.01, dense_input=True)
    code, flag = {"f64": (sd.SDNN_ARM_DENSE, 1), "f32": (sd.SDNN_ARM_DENSE_F32, 2)}[arm]
    net = sd.net_from_problem(p, dense=flag)
    y = torch.from_numpy(np.random.default_rng(2).random((batch, n), dtype=np.float32)).cuda()
    want = net.forward_dense(y, arm=code)
    for shift in (None, 0, 5, -5):
        print("[case] scratch parts", arm, n, batch, shift, flush=True)
        room = torch.empty((batch + 5, n), device="cuda")
        lo = 5 if shift is not None and shift < 0 else 0  # where the input starts
        src = room[lo:lo + batch]
        src.copy_(y)
        out = torch.empty_like(y) if shift is None else room[lo + shift:lo + shift + batch]
        sd.sdnn_forward_dense_noalloc(net.handle, 0, 1, batch, src, out, code)
        assert torch.equal(out, want)
    net.free()


@pytest.mark.parametrize("arm", ["f64", "f32"])
def test_layout_changes_of_large_batches(arm):
    """Beyond 2^24 values the batch goes into the operand layout in 64 x 64 tiles, below in 32 x 32: the rows of a large
    batch in two calls, bit for bit (no K splits at either size)."""
    import torch

    import paper_1708_02937_amd as sd

    n, batch = 1001, 16799
    p = tiny_random(4, n, 1, 4, w_density=0.02, dense_input=True)
    code, flag = {"f64": (sd.SDNN_ARM_DENSE, 1), "f32": (sd.SDNN_ARM_DENSE_F32, 2)}[arm]
    net = sd.net_from_problem(p, dense=flag)
    y = torch.from_numpy(np.random.default_rng(5).random((batch, n), dtype=np.float32)).cuda()
    print("[case] layout changes", arm, flush=True)
    whole = net.forward_dense(y, arm=code)
    assert torch.equal(whole[:8001], net.forward_dense(y[:8001], arm=code))
    assert torch.equal(whole[8001:], net.forward_dense(y[8001:], arm=code))
    net.free()
