"""The dense backward contraction at the edges of its shapes and rules: ragged
input chunks and neuron tiles, one neuron per lane, the longest grid, batch
splits, more neuron tiles than dt_in buffers, unaligned weight rows, no gradient
at all, each gradient alone, and unaligned gradient buffers. Against the oracle
with the error models of the dense and multi-spike tests."""
import numpy as np
import pytest

from tests.test_gpu_dense import (_fwd_bwd_parity, _gpu_backward, _gpu_forward, _layer_case,
                                  _special_inputs, dev)  # noqa: F401
from tests.test_gpu_multispike import _case as _ms_case
from tests.test_gpu_multispike import _parity as _ms_parity

pytestmark = pytest.mark.gpu

DENSE = [
    # B, N_in, N_out, M, bf16
    (5, 1, 1, 1, False),
    (3, 17, 64, 12, False),
    (9, 33, 65, 16, False),
    (40, 300, 129, 16, False),   # batch split
    (700, 20, 600, 8, False),    # tiles in two launches
    (3, 20, 70, 256, False),     # one neuron per lane
    (5, 30, 130, 20, True),      # 60-byte weight rows
    (6, 272, 140, 20, True),     # two blocks over the inputs
]


@pytest.mark.parametrize("B,N_in,N_out,M,bf16", DENSE)
def test_dense_backward_shapes(dev, B, N_in, N_out, M, bf16):  # noqa: F811
    p, t, W = _layer_case(11, B, N_in, N_out, M, 1.0, 0.3)
    if N_in > 12:
        t = _special_inputs(t, p, np.random.default_rng(12))
    _fwd_bwd_parity(dev, p, t, W, f"back {B}x{N_in}->{N_out} M={M}", bf16=bf16)


def test_dense_backward_alone_and_without_gradient(dev):  # noqa: F811
    p, t, W = _layer_case(13, 50, 100, 150, 16, 1.0, 0.3)
    gpu, h = _gpu_forward(dev, p, t, W)
    g = np.random.default_rng(14).standard_normal(gpu["t_out"].shape)
    g = np.where(gpu["q"] >= 0, g, 0.0).astype(np.float32)
    gW, gx = _gpu_backward(dev, h, g)
    only_W, none = _gpu_backward(dev, h, g, need_t=False)
    assert none is None and np.array_equal(only_W, gW)
    none, only_x = _gpu_backward(dev, h, g, need_W=False)
    assert none is None and np.array_equal(only_x, gx)
    zW, zx = _gpu_backward(dev, h, np.zeros_like(g))
    assert not zW.any() and not zx.any() and gW.any() and gx.any()


def test_dense_backward_unaligned_buffers(dev):  # noqa: F811
    """Gradient buffers and weights four bytes past a 16-byte boundary."""
    import ctypes
    import torch
    from paper_2607_14672_amd import dstd
    p, t, W = _layer_case(15, 64, 96, 132, 16, 1.0, 0.3)
    gpu, h = _gpu_forward(dev, p, t, W)
    g = np.where(gpu["q"] >= 0, 1.0, 0.0).astype(np.float32)
    gW, gx = _gpu_backward(dev, h, g)
    prm, tt, Wt, to, sl, q = h

    def off(x):
        buf = torch.zeros(x.numel() + 1, dtype=torch.float32, device=dev)
        v = buf[1:].view(x.shape)
        v.copy_(x)
        return v
    Wo, oW, ox = off(Wt), off(torch.zeros_like(Wt)), off(torch.zeros_like(tt))
    gt = torch.from_numpy(g).to(dev)
    lib = dstd._load()
    B, N_in, N_out = 64, 96, 132
    n = lib.dstd_lif_backward_workspace_size(ctypes.addressof(prm), B, N_in, N_out)
    ws = torch.empty(n, dtype=torch.uint8, device=dev)
    st = lib.dstd_lif_backward(ctypes.addressof(prm), B, N_in, N_out, tt.data_ptr(), Wo.data_ptr(), 0,
                               to.data_ptr(), sl.data_ptr(), q.data_ptr(), gt.data_ptr(), oW.data_ptr(),
                               ox.data_ptr(), ws.data_ptr(), n, torch.cuda.current_stream().cuda_stream)
    assert st == 0
    torch.cuda.synchronize()
    assert np.array_equal(oW.cpu().numpy(), gW) and np.array_equal(ox.cpu().numpy(), gx)


@pytest.mark.parametrize("B,N_in,F_in,N_out,M,bf16", [
    (2, 17, 5, 65, 12, False), (40, 33, 2, 140, 16, False), (3, 9, 3, 70, 250, False),
    (30, 20, 8, 300, 8, True)])  # the last: tiles in several launches
def test_multispike_backward_shapes(dev, B, N_in, F_in, N_out, M, bf16):  # noqa: F811
    p, t, W = _ms_case(21, B, N_in, F_in, N_out, M, 1.0, 0.3, k=3.0)
    _ms_parity(dev, p, t, W, 3, f"multispike back {B}x{N_in}x{F_in}->{N_out} M={M}", bf16=bf16)


@pytest.mark.parametrize("B,N_in,N_out,M", [
    (1, 5, 3, 4), (24, 400, 120, 64), (9, 100, 129, 20), (64, 33, 200, 100), (5, 700, 65, 200)])
def test_dense_backward_alone_is_the_same(dev, B, N_in, N_out, M):  # noqa: F811
    """Each gradient alone has the bits that both together give it, whatever the
    launch shapes; both are checked against the oracle."""
    p, t, W = _layer_case(23, B, N_in, N_out, M, 1.0, 0.3)
    _fwd_bwd_parity(dev, p, t, W, f"back alone {B}x{N_in}->{N_out} M={M}")
    gpu, h = _gpu_forward(dev, p, t, W)
    g = np.random.default_rng(24).standard_normal(gpu["t_out"].shape).astype(np.float32)
    gW, gx = _gpu_backward(dev, h, g)
    assert np.array_equal(_gpu_backward(dev, h, g, need_t=False)[0], gW)
    assert np.array_equal(_gpu_backward(dev, h, g, need_W=False)[1], gx)


@pytest.mark.parametrize("B,N_in,F_in,N_out,M", [
    (2, 5, 1, 3, 4), (24, 60, 4, 40, 65), (9, 30, 2, 129, 20), (16, 100, 3, 70, 128)])
def test_multispike_backward_alone_is_the_same(dev, B, N_in, F_in, N_out, M):  # noqa: F811
    import torch
    from paper_2607_14672_amd import dstd
    p, t, W = _ms_case(25, B, N_in, F_in, N_out, M, 1.0, 0.3, k=3.0)
    _ms_parity(dev, p, t, W, 3, f"multispike back {B}x{N_in}x{F_in}->{N_out} M={M}")
    prm = dstd.make_params(1.0, 0.3, 1.0, M, 0.0, 1.0 / M)
    tt, Wt = (torch.from_numpy(np.ascontiguousarray(x, np.float32)).to(dev) for x in (t, W))
    r = dstd.multispike_forward(prm, tt, Wt, 3)
    g = torch.randn(r[0].shape, device=dev, generator=torch.Generator(device=dev).manual_seed(26))
    gW, gx = dstd.multispike_backward(prm, tt, Wt, *r, g)
    assert torch.equal(dstd.multispike_backward(prm, tt, Wt, *r, g, need_t_in=False)[0], gW)
    assert torch.equal(dstd.multispike_backward(prm, tt, Wt, *r, g, need_W=False)[1], gx)


def _layer(dev, B, N_in, N_out, M, seed=0):  # noqa: F811
    """A layer's forward with inputs and weights made on the GPU."""
    import torch
    from paper_2607_14672_amd import dstd
    gen = torch.Generator(device=dev).manual_seed(seed)
    prm = dstd.make_params(1.0, 0.3, 1.0, M, 0.0, 1.0 / M)
    t = torch.rand((B, N_in), device=dev, generator=gen)
    t[torch.rand((B, N_in), device=dev, generator=gen) < 0.1] = float("inf")
    W = (6.0 / N_in) * (1 + 0.3 * N_in ** 0.5 * torch.randn((N_out, N_in), device=dev, generator=gen))
    r = dstd.forward(prm, t, W)
    return prm, t, W, r, torch.randn(r[0].shape, device=dev, generator=gen)


# (B, N_in, N_out, M): inputs along the lanes from 2.5 million pairs, 96 inputs, M <= 128:
# ragged inputs and neurons, a split, the longest grid, one and two inputs per thread
BY_INPUT = [(64, 257, 200, 16), (300, 96, 100, 128), (40, 1100, 65, 33), (128, 700, 90, 1),
            (3, 3100, 5000, 16), (4, 3073, 4990, 40)]


@pytest.mark.parametrize("synfire", [False, True])
@pytest.mark.parametrize("B,N_in,N_out,M", BY_INPUT)
def test_dense_dw_by_input_is_the_same(dev, B, N_in, N_out, M, synfire):  # noqa: F811
    import torch
    from paper_2607_14672_amd import dstd
    prm, t, W, r, g = _layer(dev, B, N_in, N_out, M)
    sp = dstd.make_synfire(0.2, 0.3, 0.1, 0.8, 0.05, 1.0 / B) if synfire else None
    gW, gx = dstd.backward(prm, t, W, *r, g, synfire=sp)
    assert bool(gW.any())
    only, none = dstd.backward(prm, t, W, *r, g, need_t_in=False, synfire=sp)
    assert none is None and torch.equal(only, gW)
    g[B // 2:] = 0.0  # samples without gradient
    gW, _ = dstd.backward(prm, t, W, *r, g, synfire=sp)
    assert torch.equal(dstd.backward(prm, t, W, *r, g, need_t_in=False, synfire=sp)[0], gW)


def test_dense_dw_by_input_parity(dev):  # noqa: F811
    p, t, W = _layer_case(27, 64, 257, 200, 16, 1.0, 0.3)
    t = _special_inputs(t, p, np.random.default_rng(28))
    _fwd_bwd_parity(dev, p, t, W, "dW by input 64x257->200", need_t=False)


@pytest.mark.parametrize("M", [8, 32])
def test_dw_alone_costs_less_than_half_of_both(dev, M):  # noqa: F811
    """4096 -> 4096, batch 256: dW alone 0.32 and 0.41 of both gradients' time
    (0.67 and 0.71 with the inputs in the rows of the contraction)."""
    import torch
    from paper_2607_14672_amd import dstd
    prm, t, W, r, g = _layer(dev, 256, 4096, 4096, M)
    ws = dstd.workspace(dstd.dstd_lif_backward_workspace_size(prm, 256, 4096, 4096), dev)

    def best(need_t):
        out = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(3):
                dstd.backward(prm, t, W, *r, g, need_t_in=need_t, ws=ws)
            b.record()
            b.synchronize()
            out.append(a.elapsed_time(b))
        return min(out)
    assert best(False) < 0.55 * best(True)
