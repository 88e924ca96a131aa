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
