"""The policy's matrix-core kernels at the edges of their 32-row tiles, of
their four-tile blocks and of their grids, with activations beyond the half
range (the tile then takes the float32 instructions), and with rows that
start at any half (not only at 16 bytes).

Bounds: a float32 sum of N terms is off by at most N 2^-24 times the sum of
their magnitudes.  A score is three such sums of 17, 65 and 65 terms, one
inside the other, so 160 2^-24 times the same network of magnitudes covers
them (a cut activation adds 2^-24 of its own).  A gradient adds the sigmoid
(__expf, a division: a few 2^-22 of 1), one more layer and the sum over the
rows, which one register takes at most 32 per tile: 1024 2^-24 times the
magnitudes with |dz| replaced by 1 / rows."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
E = 2.0 ** -24


def _network(seed, scale):
    from paper_1908_06418_amd.policy import init_params
    w = init_params(seed).astype(np.float64)
    w[:1088] *= scale  # W1, b1
    w[1024:1088] = np.random.default_rng(seed).normal(0, 0.1 * scale, 64)
    w = w.astype(np.float32)
    h = w.astype(np.float16).astype(np.float64)
    return w, (h[:1024].reshape(64, 16), h[1024:1088], h[1088:5184].reshape(64, 64),
               h[5184:5248], h[5248:5312], h[5312])


def _layers(net, x):
    W1, b1, W2, b2, w3, b3 = net
    a1 = x @ W1.T + b1
    a2 = np.maximum(a1, 0) @ W2.T + b2
    return a1, a2, np.maximum(a2, 0) @ w3 + b3


def _inputs(net, rows, seed):
    """Rows with no activation so near zero that float32 could cut it the
    other way."""
    rng = np.random.default_rng(seed)
    keep = []
    while sum(len(k) for k in keep) < rows:
        x = rng.random((rows + 64, 16)).astype(np.float16)
        a1, a2, _ = _layers(net, x.astype(np.float64))
        A1, A2, _ = _layers(tuple(np.abs(w) for w in net), x.astype(np.float64))
        keep.append(x[(np.abs(a1) > 64 * E * A1).all(1) & (np.abs(a2) > 256 * E * A2).all(1)])
    return np.concatenate(keep)[:rows]


def _at_any_half(x, shift):
    import torch
    flat = torch.zeros(x.size + 8, dtype=torch.float16, device="cuda")
    v = flat[shift:shift + x.size].view(x.shape)
    v.copy_(torch.from_numpy(x))
    return v


@pytest.mark.parametrize("scale", [1.0, 3e5])
@pytest.mark.parametrize("rows,shift", [(1, 0), (31, 1), (32, 0), (33, 8), (127, 0), (129, 3),
                                        (65536 + 33, 0)])
def test_scores(gpu, rows, shift, scale):
    from paper_1908_06418_amd.policy import Policy
    w, net = _network(1, scale if scale < 100 else 3000.0)
    x = np.random.default_rng(rows).random((rows, 16)).astype(np.float16)
    if scale > 100:
        x[::2] *= np.float16(100)  # some rows of a tile beyond the half range, some not
    x64 = x.astype(np.float64)
    z = _layers(net, x64)[2]
    bound = 160 * E * _layers(tuple(np.abs(v) for v in net), x64)[2]
    if scale > 100:
        assert np.abs(_layers(net, x64)[0]).max() > 65504
    got = Policy(w).forward(_at_any_half(x, shift)).cpu().numpy()
    assert (np.abs(got - z) <= bound).all()


@pytest.mark.parametrize("rows,shift", [(1, 0), (32, 5), (33, 0), (128, 0), (129, 1), (4097, 0),
                                        (33000, 0)])
def test_gradient(gpu, rows, shift):
    import torch
    from paper_1908_06418_amd.policy import Policy
    w, net = _network(2, 1.0)
    W1, b1, W2, b2, w3, b3 = net
    x = _inputs(net, rows, rows)
    y = (np.random.default_rng(rows + 1).random(rows) < 0.3).astype(np.float32)
    x64 = x.astype(np.float64)
    a1, a2, z = _layers(net, x64)
    h1, h2 = np.maximum(a1, 0), np.maximum(a2, 0)

    def grads(dz, w3, W2):
        d2 = np.outer(dz, w3) * (a2 > 0)
        d1 = (d2 @ W2) * (a1 > 0)
        return np.concatenate([(d1.T @ x64).ravel(), d1.sum(0), (d2.T @ h1).ravel(), d2.sum(0),
                               h2.T @ dz, [dz.sum()]])

    want = grads((1 / (1 + np.exp(-z)) - y) / rows, w3, W2)
    bound = 1024 * E * grads(np.full(rows, 1 / rows), np.abs(w3), np.abs(W2))
    loss, g = Policy(w).grad(_at_any_half(x, shift), torch.from_numpy(y).cuda())
    assert (np.abs(g.cpu().numpy() - want) <= bound).all()
    terms = np.maximum(z, 0) - z * y + np.log1p(np.exp(-np.abs(z)))
    assert abs(float(loss) - terms.mean()) <= 1024 * E * (np.abs(z) + 1).mean()
