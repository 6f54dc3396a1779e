"""Scores where layer 2's activations are far from one: near the half range's
lower end, below it, spread over many powers of two, and where a weight of the
layer rounds to infinity.

Bound, as in test_gpu_policy_tiles: 160 2^-24 times the same network of
magnitudes (sums of 17, 65 and 65 terms inside one another; a sum over the
pieces of the activations adds two roundings).  With b1 = b2 = 0 it scales
with the activations, so that nothing may be rounded at a fixed place.  (What
float32 itself rounds at a fixed place, below 2^-126, is far under it.)"""
import numpy as np
import pytest
from test_gpu_policy_tiles import E, _layers

pytestmark = pytest.mark.gpu


def _network(seed, scale):
    from paper_1908_06418_amd.policy import init_params
    w = init_params(seed).astype(np.float64)
    w[:1024] *= scale
    w = w.astype(np.float32)
    with np.errstate(over="ignore"):
        h = w.astype(np.float16).astype(np.float64)
    return w, (h[:1024].reshape(64, 16), h[1024:1088], h[1088:5184].reshape(64, 64),
               h[5184:5248], h[5248:5312], h[5312])


def _scores(w, x):
    import torch
    from paper_1908_06418_amd.policy import Policy
    return Policy(w).forward(torch.from_numpy(x).cuda()).cpu().numpy()


@pytest.mark.parametrize("scale,size", [(1.0, 1e-2), (1.0, 1e-4), (1e-3, 1.0), (1e-3, 1e-2), (1e-3, 1e-3),
                                        (1e-3, 1e-4), (1e-4, 1e-4), (1e-6, 1.0)])
@pytest.mark.parametrize("rows", [31, 4096])
def test_scores_of_small_activations(gpu, rows, scale, size):
    w, net = _network(3, scale)
    x = (np.random.default_rng(rows).random((rows, 16)) * size).astype(np.float16)
    x64 = x.astype(np.float64)
    z = _layers(net, x64)[2]
    bound = 160 * E * _layers(tuple(np.abs(v) for v in net), x64)[2]
    assert (np.abs(_scores(w, x) - z) <= bound).all()


def test_scores_over_many_powers_of_two(gpu):
    """Rows of very different sizes in one tile, down to a few 2^-24."""
    w, net = _network(4, 1e-2)
    rng = np.random.default_rng(8)
    x = (rng.random((3000, 16)) * 2.0 ** rng.integers(-22, 16, (3000, 1))).astype(np.float16)
    x64 = x.astype(np.float64)
    z = _layers(net, x64)[2]
    bound = 160 * E * _layers(tuple(np.abs(v) for v in net), x64)[2]
    assert (np.abs(_scores(w, x) - z) <= bound).all()


def test_weights_that_round_to_infinity(gpu):
    """As in float32: infinity times a positive activation is infinite, times
    zero no number, which the ReLU turns into zero."""
    w, net = _network(5, 1.0)
    w[1088 + 64 * 3 + 7] = 1e6     # W2[3][7]
    w[1088 + 64 * 9 + 20] = -1e6   # W2[9][20]
    with np.errstate(over="ignore", invalid="ignore"):
        W2 = w[1088:5184].astype(np.float16).astype(np.float64).reshape(64, 64)
        assert np.isinf(W2[3, 7]) and np.isinf(W2[9, 20])
        x = np.random.default_rng(9).random((200, 16)).astype(np.float16)
        net = net[:2] + (W2,) + net[3:]
        h1 = np.maximum(_layers(net, x.astype(np.float64))[0], 0)
        z = np.fmax(h1 @ W2.T + net[3], 0) @ net[4] + net[5]
    assert np.isinf(z).any() and np.isfinite(z).any()
    got = _scores(w, x)
    assert (np.isinf(z) == np.isinf(got)).all() and (np.isfinite(z) == np.isfinite(got)).all()
    same = np.isinf(z)
    assert (got[same] == z[same]).all()
    A = tuple(np.abs(np.nan_to_num(v, posinf=0, neginf=0)) for v in net)
    bound = 160 * E * _layers(A, x.astype(np.float64))[2]
    assert (np.abs(got[~same] - z[~same]) <= bound[~same]).all()
