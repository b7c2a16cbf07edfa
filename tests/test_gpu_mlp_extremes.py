"""GPU: the network at pre-activations whose exponential overflows, underflows or
is infinite: SiLU and its derivative are those of the general division z / (1 +
exp(-z)), through every variant of the forward pass (cached, small batches, large
batches) and the backward pass; gradients of infinite loss gradients and of ones
past the largest BF16 value."""
import numpy as np
import pytest

from oracle import mlp as omlp
from paper_1710_09995_amd import cases
from test_gpu_mlp import _rel, round_bf16

pytestmark = pytest.mark.gpu

FAR = [-1e38, -1e33, -1e30, -1e20, -200.0, -100.0, -90.0]     # exp(-z) beyond FP32: SiLU is -0
MID = [-88.5, -87.5, -85.0, -75.0, -70.0, -69.0, -50.0, -3.0, -1.0, 0.0, 1.0, 50.0, 69.0, 100.0, 1e30, 1e38]


def _net():
    """Every hidden pre-activation is the input, the output the hidden activations' mean."""
    from paper_1710_09995_amd.binding import Mlp
    return Mlp([(np.ones((16, 1)), np.zeros(16)), (np.full((1, 16), 1.0 / 16.0), np.zeros(1))], d_in=1, d_hidden=16,
               n_hidden=1, d_out=1)


def _points():
    z = round_bf16(np.array(FAR + MID))
    want = np.zeros(len(z))
    want[len(FAR):] = [v / (1.0 + np.exp(-v)) for v in z[len(FAR):]]
    return z, want


@pytest.mark.parametrize("n,cache", [(26, False), (26, True), (1000, False), (131072 + 77, False)])
def test_silu_is_the_general_quotient(n, cache):
    """Within the BF16 rounding of the activation (2^-8) where the quotient is in
    range, zero where the exponential overflows, infinite and NaN as the division."""
    import torch
    z, want = _points()
    z, want = np.r_[z, np.inf, -np.inf, np.nan], np.r_[want, np.inf, np.nan, np.nan]
    pick = np.random.default_rng(n).integers(0, len(z), n)
    pick[:min(n, len(z))] = np.arange(min(n, len(z)))
    y = _net().forward(torch.from_numpy(z[pick, None].astype(np.float32)).cuda(), cache=cache)
    y = (y[0] if cache else y).cpu().numpy()[:, 0].astype(np.float64)
    w = want[pick]
    assert np.array_equal(np.isnan(y), np.isnan(w))
    assert np.array_equal(y[np.isinf(w)], w[np.isinf(w)])
    ok = np.isfinite(w)
    assert np.all(np.abs(y[ok] - w[ok]) <= 2.0 ** -8 * np.abs(w[ok]))


def test_silu_derivative_is_the_general_quotients():
    """To the rounding of exp's argument (|z| 2^-24 relative, 1e-5 with a margin
    of 2 at |z| = 88) where the logistic is normal, zero where the exponential
    overflows."""
    import torch
    from paper_1710_09995_amd.binding import unpack_params
    m = _net()
    for v in round_bf16(np.array(FAR + [x for x in MID if x not in (-88.5, -87.5, -1.0)])):
        y, c = m.forward(torch.full((1, 1), float(v), device="cuda"), cache=True)
        (_, db), _ = unpack_params(m.backward(c, torch.ones_like(y)).cpu().numpy(), 1, 16, 1, 1)
        s = 0.0 if v < -89.0 else 1.0 / (1.0 + np.exp(-v))
        want = s * (1.0 + v * (1.0 - s)) / 16.0
        assert np.all(np.abs(db - want) <= 1e-5 * abs(want)), v


def _positive(scale):
    """A net of positive weights over positive inputs (every activation and
    derivative is positive), its cached activations and the size of its outputs."""
    import torch
    from paper_1710_09995_amd.binding import Mlp
    params = [(scale * np.abs(W), b) for W, b in cases.mlp_init(5, 32, 2, 5, seed=1, out_scale=1.0)]
    m = Mlp(params, d_hidden=32, n_hidden=2)
    x = np.random.default_rng(2).uniform(0.1, 1.0, (40, 5)).astype(np.float32)
    y, cache = m.forward(torch.from_numpy(x).cuda(), cache=True)
    return m, y, cache


@pytest.mark.parametrize("v", [np.inf, -np.inf])
def test_infinite_loss_gradients_give_infinite_gradients(v):
    import torch
    from paper_1710_09995_amd.binding import unpack_params
    m, y, cache = _positive(1.0)
    dy = torch.zeros_like(y)
    dy[3, 1] = float(v)
    g = unpack_params(m.backward(cache, dy).cpu().numpy(), 5, 32, 2, 5)
    for gw, gb in g[:2]:
        assert np.all(gw == v) and np.all(gb == v)
    rest = [0, 2, 3, 4]
    assert np.all(g[2][0][1] == v) and g[2][1][1] == v
    assert np.all(g[2][0][rest] == 0.0) and np.all(g[2][1][rest] == 0.0)


@pytest.mark.parametrize("v", [3.3895314e38, 3.39e38, -3.4e38])
def test_loss_gradients_past_the_largest_bf16_value(v):
    """The gates of the gradients at ordinary sizes (FP32 rounding: 2e-6)."""
    import torch
    from paper_1710_09995_amd.binding import unpack_params
    m, y, cache = _positive(0.1)
    dy = np.zeros((40, 5), np.float32)
    dy[3, 1] = v
    got = unpack_params(m.backward(cache, torch.from_numpy(dy).cuda()).cpu().numpy(), 5, 32, 2, 5)
    c = cache.cpu().numpy().astype(np.float64)
    kept = [(c[:, :5], c[:, 16:48]), (c[:, 48:80], c[:, 80:112]), (c[:, 112:144], c[:, 144:149])]
    want = omlp.backward(m.bf16_params(), kept, dy.astype(np.float64))
    for (gw, gb), (ww, wb) in zip(got, want):
        gw, gb = gw.astype(np.float64), gb.astype(np.float64)
        assert _rel(gw, ww) <= 2e-6 and _rel(gb, wb) <= 2e-6
