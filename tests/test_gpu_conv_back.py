"""The conv backward contraction at the edges of its shapes and rules: tap
groups (kernel widths 1, 3, 5, 7; strides), grids whose tables leave one tap or
one channel per lane, channel tiles in several launches, ragged input chunks,
upstream gradients with gaps, and each gradient alone. Against the oracle with
the error model of the conv tests."""
import numpy as np
import pytest

import oracle
from tests.parity import check_forward
from tests.test_gpu_conv import (_conv_case, _conv_grad_check, _cs, _gpu_backward, _gpu_forward,
                                 _special_inputs, _taus, _window, dev)  # noqa: F401

pytestmark = pytest.mark.gpu

CASES = [
    # label, B, conv shape, M, tau_m, tau_s, k, share of positions with gradient
    ("7 wide, three tap groups", 2, _cs(9, 8, 11, 20, K=7), 12, 1.0, 0.3, 7.0, 1.0),
    ("5x5 stride 2, 17 channels in", 2, _cs(17, 9, 11, 70, K=5, stride=2), 16, 1.0, 0.5, 7.0, 1.0),
    ("M 256: one tap per wave", 1, _cs(8, 5, 6, 40), 256, 1.0, 0.3, 7.0, 1.0),
    ("M 100: one channel per lane, two tiles", 1, _cs(16, 5, 6, 100), 100, 1.0, 0.3, 7.0, 1.0),
    ("400 channels out, 1x1: two dt_in launches", 2, _cs(33, 4, 5, 400, K=1, pad=0), 16, 1.0, 0.3,
     7.0, 1.0),
    ("rows of 70 positions, gradient in gaps", 2, _cs(5, 3, 70, 24), 10, 1.5, 0.5, 7.0, 0.04),
    ("pooled, gradient in gaps", 3, _cs(10, 8, 12, 66, pool_in=2), 16, 1.0, 0.3, 7.0, 0.1),
    ("stride 2, gradient in gaps", 3, _cs(6, 9, 15, 30, stride=2), 12, 0.5, 0.5, 7.0, 0.1),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_conv_backward_shapes(dev, case):  # noqa: F811
    label, B, cs, M, tm, ts, k, share = case
    p, t, W = _conv_case(77, B, cs, M, tm, ts, k=k)
    rng = np.random.default_rng(78)
    t = _special_inputs(t, p, rng)
    gpu, h = _gpu_forward(dev, p, cs, t, W)
    orc = oracle.conv_forward(p, cs, t, W)
    mask, stats = check_forward(gpu, orc, None, _window(p), label=label, taus=_taus(p))
    g = rng.standard_normal(orc["t_out"].shape)
    on = rng.random((B, 1) + g.shape[2:]) < share  # whole positions, all their channels
    g = np.where(mask | ~on, 0.0, g).astype(np.float32)
    gW, gx = _gpu_backward(dev, h, g)
    _conv_grad_check(p, cs, t, W, orc, mask, stats, g, gW, gx, label)
    only_W, none = _gpu_backward(dev, h, g, need_t=False)
    assert none is None and np.array_equal(only_W, gW)
    none, only_x = _gpu_backward(dev, h, g, need_W=False)
    assert none is None and np.array_equal(only_x, gx)


@pytest.mark.parametrize("c_out", [20, 70])
def test_conv_backward_interval_index_past_the_grid(dev, c_out):  # noqa: F811
    """Interval indices past M are taken as M: same gradients, no entry past the table."""
    import torch
    cs = _cs(6, 5, 7, c_out)
    p, t, W = _conv_case(79, 2, cs, 10, 1.0, 0.3, k=7.0)
    gpu, (prm, c, tt, Wt, to, sl, q) = _gpu_forward(dev, p, cs, t, W)
    g = np.random.default_rng(80).standard_normal(gpu["t_out"].shape).astype(np.float32)
    last = torch.where(q >= 0, torch.full_like(q, p["M"]), q)
    past = torch.where((q >= 0) & (q % 2 == 0), q + p["M"] + 1000, last)
    a = _gpu_backward(dev, (prm, c, tt, Wt, to, sl, last), g)
    b = _gpu_backward(dev, (prm, c, tt, Wt, to, sl, past), g)
    assert all(np.isfinite(x).all() and x.any() for x in a)
    assert all(np.array_equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("B,cs,M,share", [
    (3, _cs(1, 9, 11, 17, K=5), 12, 1.0),           # few pairs, one block of them
    (2, _cs(30, 6, 7, 65), 16, 0.3),                # 270 pairs, two channel tiles, gaps
    (2, _cs(7, 10, 12, 33, pool_in=2), 90, 0.05),   # four raw pixels, 32 channels per block
    (3, _cs(20, 3, 4, 10, K=1, pad=0, pool_in=0), 16, 1.0),  # twelve raw pixels
    (2, _cs(9, 9, 13, 70, stride=2), 256, 0.5),     # the longest grid
    (4, _cs(70, 5, 5, 40, K=1, pad=0), 8, 0.5),
    (2, _cs(3, 8, 66, 20), 20, 0.02),               # rows longer than 64 positions, most without
    # batches that choose each of the contraction's other tiles (taps, channels and
    # inputs per lane or wave), both together and each alone
    (64, _cs(9, 2, 2, 3, K=5), 8, 0.6),
    (128, _cs(9, 28, 28, 3, K=1, pad=0), 8, 0.3),
    (64, _cs(1, 4, 4, 65), 8, 1.0),
    (64, _cs(1, 12, 12, 65, K=1, pad=0), 16, 0.3),
    (64, _cs(17, 4, 4, 65), 90, 0.6),
    (64, _cs(1, 12, 12, 3), 8, 0.6),
    (64, _cs(1, 4, 4, 3, K=5), 90, 1.0),
    (128, _cs(9, 4, 4, 3, K=5), 90, 0.6),
    (64, _cs(1, 12, 12, 65), 16, 0.3),
    (128, _cs(1, 4, 4, 65, K=5), 16, 1.0),
])
def test_conv_backward_alone_is_the_same(dev, B, cs, M, share):  # noqa: F811
    """Each gradient alone has the bits that both together give it (dW alone runs
    with the (tap, input) pairs along the lanes), and dW agrees with the oracle."""
    p, t, W = _conv_case(81, B, cs, M, 1.0, 0.3, k=7.0)
    rng = np.random.default_rng(82)
    t = _special_inputs(t, p, rng)
    gpu, h = _gpu_forward(dev, p, cs, t, W)
    orc = oracle.conv_forward(p, cs, t, W)
    mask, stats = check_forward(gpu, orc, None, _window(p), label="alone", taus=_taus(p))
    g = rng.standard_normal(orc["t_out"].shape)
    on = rng.random((B, 1) + g.shape[2:]) < share
    g = np.where(mask | ~on, 0.0, g).astype(np.float32)
    only_W, none = _gpu_backward(dev, h, g, need_t=False)
    assert none is None
    _conv_grad_check(p, cs, t, W, orc, mask, stats, g, only_W, None, "dW alone")
    gW, gx = _gpu_backward(dev, h, g)
    assert np.array_equal(only_W, gW)
    assert np.array_equal(_gpu_backward(dev, h, g, need_W=False)[1], gx)
    zW, _ = _gpu_backward(dev, h, np.zeros_like(g), need_t=False)
    assert not zW.any()


@pytest.mark.parametrize("C_in,K", [(1, 5), (12, 3)])
def test_conv_dw_alone_costs_less_than_both(dev, C_in, K):  # noqa: F811
    """A small layer's dW alone against both gradients: 0.34 and 0.62 of their time
    (0.78 and 0.85 with a wave per input)."""
    import torch
    from paper_2607_14672_amd import dstd
    gen = torch.Generator(device=dev).manual_seed(83)
    cs = dstd.make_conv_shape(C_in, 28, 28, 32, K, K, 1, K // 2, 1)
    prm = dstd.make_params(1.0, 0.3, 1.0, 32, 0.0, 1.0 / 32)
    t = torch.rand((64, C_in, 28, 28), device=dev, generator=gen)
    n = C_in * K * K
    W = (6.0 / n) * (1 + 0.3 * n ** 0.5 * torch.randn((32, C_in, K, K), device=dev, generator=gen))
    ws = dstd.workspace(dstd.dstd_lif_conv_backward_workspace_size(prm, cs, 64), dev)
    r = dstd.conv_forward(prm, cs, t, W, ws=ws)
    g = torch.randn(r[0].shape, device=dev, generator=gen)

    def best(need_t):
        out = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(5):
                dstd.conv_backward(prm, cs, t, W, *r, g, need_t_in=need_t, ws=ws)
            b.record()
            b.synchronize()
            out.append(a.elapsed_time(b))
        return min(out)
    x, y = best(False), best(True)
    print(f"dW alone / both {x / y:.2f}", flush=True)
    assert x < 0.75 * y


@pytest.mark.parametrize("B,cs,share", [
    (48, _cs(5, 12, 12, 12), 0.05), (96, _cs(17, 8, 8, 70), 0.3), (96, _cs(9, 8, 8, 12), 0.1),
    (64, _cs(9, 8, 8, 12, pool_in=2), 0.2), (128, _cs(5, 6, 6, 24, K=7), 0.05),
    (3, _cs(6, 9, 15, 30, stride=2), 0.1)])
def test_conv_backward_odd_weights_reach_only_their_inputs(dev, B, cs, share):  # noqa: F811
    """Infinite and NaN weights: dt_in is not finite exactly where a position with
    gradient up to the input's event row joins it through such a weight; elsewhere it
    has the bits of the same weights at 0. (Three taps per wave, but for the last.)"""
    import torch
    from paper_2607_14672_amd import dstd
    M, K, st, pad = 10, cs["KH"], cs["stride"], cs["pad"]
    pool = cs["pool_in"]
    p, t, W = _conv_case(85, B, cs, M, 1.0, 0.3, k=7.0)
    gpu, h = _gpu_forward(dev, p, cs, t, W)
    rng = np.random.default_rng(86)
    g = rng.standard_normal(gpu["t_out"].shape).astype(np.float32)
    g *= rng.random((B, 1) + g.shape[2:]) < share
    odd = rng.random((1,) + W.shape[1:]) < 0.02  # (input channel, tap)s with one odd weight each
    odd[0, 0, 0, 0] = True
    at = rng.integers(0, W.shape[0], W.shape[1:])[None] == np.arange(W.shape[0])[:, None, None, None]
    at = at & odd
    Wo = np.where(at, rng.choice([np.inf, -np.inf, np.nan], W.shape), W).astype(np.float32)
    prm, c, tt, _, to, sl, q = h
    dev_w = [torch.from_numpy(np.ascontiguousarray(x, np.float32)).to(dev) for x in (Wo, np.where(at, 0.0, W))]
    gW, gx = _gpu_backward(dev, (prm, c, tt, dev_w[0], to, sl, q), g)
    zW, zx = _gpu_backward(dev, (prm, c, tt, dev_w[1], to, sl, q), g)
    assert np.array_equal(gW, zW) and np.isfinite(zx).all()
    # the last event row that meets gradient at each position (-1: none), and the inputs' rows
    live = (gpu["q"] >= 0) & (g != 0)
    last = np.where(live, gpu["q"] + 1, -1).max(axis=1)
    row = np.floor(t.astype(np.float64) * M).astype(int) + 1
    bad = np.zeros(t.shape, bool)
    Hp, Wp = cs["H"] // pool, cs["W"] // pool
    for ky in range(K):
        for kx in range(K):
            for oy in range(last.shape[1]):
                for ox in range(last.shape[2]):
                    y, x = oy * st - pad + ky, ox * st - pad + kx
                    if 0 <= y < Hp and 0 <= x < Wp:
                        s = np.s_[:, :, y * pool:(y + 1) * pool, x * pool:(x + 1) * pool]
                        bad[s] |= (row[s] <= last[:, oy, ox][:, None, None, None]) & odd[0, :, ky, kx][None, :, None, None]
    assert bad.any() and not bad.all()
    assert np.array_equal(~np.isfinite(gx), bad)
    assert np.array_equal(gx[~bad], zx[~bad])
