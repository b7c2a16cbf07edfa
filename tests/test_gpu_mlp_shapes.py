"""GPU: the network kernels at the widths, depths and batch sizes where their
tiles end: one point, partial 16-point tiles and 64-point groups, the persistent
grid's second round, every hidden width's tile count, and nets that do and do
not fit in a workgroup's LDS.

Outputs agree with the FP64 oracle on BF16-rounded weights to the BF16 rounding
of the activations (2e-2, as for the reference shape).  Gradients are compared
with FP64 sums over the same stored activations, so only FP32 rounding remains:
up to 9 layers of about 2 roundings of 6e-8 each, 2e-6 with a margin of 2."""
import numpy as np
import pytest

from oracle import mlp as omlp
from paper_1710_09995_amd import cases
from test_gpu_mlp import _rel, round_bf16

pytestmark = pytest.mark.gpu

NETS = [(128, 4, 1), (128, 4, 16), (128, 4, 65), (128, 4, 1000), (128, 4, 131072 + 37), (128, 8, 300), (128, 8, 131101),
        (112, 3, 17), (96, 2, 63), (80, 5, 48), (64, 1, 129), (48, 8, 15), (32, 2, 64), (16, 1, 33)]


def _inputs(hidden, layers, n):
    import torch
    rng = np.random.default_rng(hidden + layers + n)
    params = [(W, 0.05 * rng.standard_normal(b.shape)) for W, b in cases.mlp_init(5, hidden, layers, 5, seed=1,
                                                                                 out_scale=1.0)]
    X = rng.uniform(-1, 1, (n, 5)).astype(np.float32)
    T = rng.normal(0, 0.3, (n, 5)).astype(np.float32)
    return params, torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda()


@pytest.mark.parametrize("hidden,layers,n", NETS)
def test_forward_at_tile_edges(hidden, layers, n):
    from paper_1710_09995_amd.binding import Mlp
    params, x, _ = _inputs(hidden, layers, n)
    m = Mlp(params, d_hidden=hidden, n_hidden=layers)
    y = m.forward(x).cpu().numpy()
    pb = [(round_bf16(W), round_bf16(b)) for W, b in params]
    pick = np.unique(np.r_[0:min(n, 40), max(0, n - 70):n, np.linspace(0, n - 1, 200).astype(int)])
    want, _ = omlp.forward(pb, round_bf16(x.cpu().numpy()[pick]))
    assert _rel(y[pick], want) <= 2e-2


@pytest.mark.parametrize("hidden,layers,n", [c for c in NETS if c[2] <= 1000])
def test_gradients_at_tile_edges(hidden, layers, n):
    from paper_1710_09995_amd.binding import Mlp, unpack_params
    params, x, t = _inputs(hidden, layers, n)
    m = Mlp(params, d_hidden=hidden, n_hidden=layers)
    y, cache = m.forward(x, cache=True)
    assert np.array_equal(y.cpu().numpy(), m.forward(x).cpu().numpy())
    loss, dy = m.mse(y, t)
    d0 = y.cpu().numpy().astype(np.float64) - t.cpu().numpy()
    assert abs(float(loss.item()) - np.mean(d0 * d0)) <= 1e-6 * np.mean(d0 * d0)
    got = unpack_params(m.backward(cache, dy).cpu().numpy(), 5, hidden, layers, 5)
    c, kept, off = cache.cpu().numpy().astype(np.float64), [], 0
    for l in range(layers + 1):
        K, N = (16 if l == 0 else hidden), (16 if l == layers else hidden)
        kept.append((c[:, off:off + (5 if l == 0 else K)], c[:, off + K:off + K + (5 if l == layers else N)]))
        off += K + N
    want = omlp.backward(m.bf16_params(), kept, dy.cpu().numpy().astype(np.float64))
    for l, ((gw, gb), (ww, wb)) in enumerate(zip(got, want)):
        assert _rel(gw, ww) <= 2e-6 and _rel(gb, wb) <= 2e-6, l
