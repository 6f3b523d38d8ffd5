"""fp32 layers on floats split into three bf16: operands whose parts bf16 cannot hold, above and below its range, in every tile of
the convolution kernels and both directions, and the weight gradients; gradients against 64-bit arithmetic.

The gradients are read from the momentum buffers after one step.  Bound: every product and sum in fp32, through at most
three layers in a row, 1e-5 of the sum of the absolute products (1152 products and a softmax: 2^-24 * (sqrt(1152) + 8) per layer)."""
import numpy as np
import pytest

from oracle import nets
from paper_2111_08274_amd import hadfl
from tests import torch_ref

pytestmark = pytest.mark.gpu
BOUND = 1e-5
CLASSES, HUGE = 20, 3.4e38

# (inputs of the layer, outputs, batch, replicas, tile hint): every tile of the launcher's list (tests/test_launch_checks.py)
LAYERS = [(32, 20, 16, 1, 0), (32, 20, 16, 1, 1), (32, 20, 1024, 16, 0), (32, 128, 1024, 16, 0), (32, 256, 1024, 16, 0),
          (256, 20, 1024, 16, 0), (64, 48, 16, 1, 1), (128, 128, 16, 1, 1), (64, 64, 1024, 64, 0), (132, 68, 64, 2, 0)]


def dense_net(inputs, outputs, doublings):
    """inputs of the data set -> inputs -> outputs -> doubled -> classes; no ReLU: what a feature holds is what the weights say"""
    b = nets._Builder()
    t = b.dense(b.dense(0, inputs), outputs)
    for _ in range(doublings):
        t = b.add(t, t)
    b.dense(t, CLASSES)
    return b


def gradients(builder, shape, batch, replicas, hint, w, x, y):
    cfg = hadfl.make_config(replicas, 1, net="custom", custom_ops=builder.array()[:, [0, 1, 2, 4, 5, 6, 7, 8]], batch=batch, n_samples=batch,
                            in_shape=shape, n_classes=CLASSES, lr=1e-30, momentum=0.5)
    ctx = hadfl.Context(cfg, [1] * replicas, w0=w, x=x, y=y, options={hadfl.OPT_TILE_HINT: hint})
    ctx.local_steps()
    got = [ctx.momentum(k).astype(np.float64) for k in sorted({0, replicas - 1})]
    ctx.close()
    return got


def check_dense(layer, w0, w1, b2, w2, x, y, doublings):
    """x, weights and labels of all replicas alike; biases of the first two layers zero"""
    inputs, outputs, batch, replicas, hint = layer
    w = np.concatenate([w0.ravel(), np.zeros(inputs), w1.ravel(), np.zeros(outputs), w2.ravel(), b2]).astype(np.float32)
    n = x.shape[1]
    rep = np.broadcast_to(x.reshape(1, batch, 1, 1, n), (replicas, batch, 1, 1, n)).astype(np.float32)
    got = gradients(dense_net(inputs, outputs, doublings), (1, 1, n), batch, replicas, hint, w, rep, np.broadcast_to(y, (replicas, batch)).astype(np.int32))
    x, w0, w1, w2, b2 = (v.astype(np.float32).astype(np.float64) for v in (x, w0, w1, w2, b2))
    a, s = x @ w0, 2.0 ** doublings
    out = s * (a @ w1)
    e = np.exp((out @ w2 + b2) - (out @ w2 + b2).max(1, keepdims=True))
    d2 = e / e.sum(1, keepdims=True)
    d2[np.arange(batch), y] -= 1.0
    d2 /= batch
    d1 = s * (d2 @ w2.T)
    d0 = d1 @ w1.T
    m = np.abs
    m1 = s * (m(d2) @ m(w2).T)
    m0 = m1 @ m(w1).T
    want = [x.T @ d0, d0.sum(0), a.T @ d1, d1.sum(0), out.T @ d2, d2.sum(0)]
    size = [m(x).T @ m0, m0.sum(0), (m(x) @ m(w0)).T @ m1, m1.sum(0), s * (m(x) @ m(w0) @ m(w1)).T @ m(d2), m(d2).sum(0)]
    for g in got:
        at = 0
        for what, (r, z) in enumerate(zip(want, size)):
            part = g[at:at + r.size].reshape(r.shape)
            at += r.size
            err = np.abs(part - r)
            assert np.isfinite(part).all() and (err <= BOUND * z + 1e-43).all(), (layer, what, float((err / (z + 1e-43)).max()))


@pytest.mark.parametrize("layer", LAYERS)
def test_values_above_bf16(layer):
    """A feature of 3.4e38 in one sample that meets zero weights, and a class whose weight of 3.4e38 is a zero feature's: the
    gradient that reaches that feature is 3.4e38 too, and meets zero weights.  In parts they are Inf * 0."""
    inputs, outputs, batch, replicas, hint = layer
    rng = np.random.default_rng(inputs + outputs)
    k = int(np.log2(batch))
    x = rng.standard_normal((batch, 32))
    # (activations of standard deviation 0.02 * sqrt(31) = 0.11, below 1 at 9 of them: their products with 3.4e38 stay finite)
    w0 = 0.02 * rng.standard_normal((32, inputs))
    w1 = 2.0 ** -k * rng.standard_normal((inputs, outputs))
    # (a gradient is a weight of the true class less an average of weights: below 5 * 0.1, for the same reason)
    w2, b2 = 0.1 * rng.standard_normal((outputs, CLASSES)), np.zeros(CLASSES)
    y = rng.integers(4, CLASSES, batch)
    x[:, 0] = 0.0
    x[1, 0] = HUGE
    w0[0] = 0.0
    w0[:, 5] = 0.0
    w0[0, 5], w1[5], w1[:, 7], w2[7] = 1.0, 0.0, 0.0, 0.0
    w2[7, 3], b2[3], y[2] = HUGE, -1e4, 3
    check_dense(layer, w0, w1, b2, w2, x, y, k)


@pytest.mark.parametrize("scales", [(-122, 20, 100), (20, -122, 100), (0, 60, -114)])
@pytest.mark.parametrize("layer", LAYERS)
def test_values_below_bf16(layer, scales):
    """Activations, weights and gradients around 2^-122, against the others so large that the results are ordinary numbers."""
    inputs, outputs, batch, replicas, hint = layer
    rng = np.random.default_rng(inputs + outputs)
    s0, s1, s2 = (2.0 ** v for v in scales)
    s2 *= batch / 16                              # (a gradient is divided by the batch)
    x = rng.standard_normal((batch, 32))
    check_dense(layer, 0.2 * s0 * rng.standard_normal((32, inputs)), 0.1 * s1 * rng.standard_normal((inputs, outputs)), np.zeros(CLASSES),
                0.3 * s2 * rng.standard_normal((outputs, CLASSES)), x, rng.integers(0, CLASSES, batch), 0)


@pytest.mark.parametrize("what", ["data", "activation", "gradient"])
@pytest.mark.parametrize("k,stride,batch,hint", [(3, 1, 32, 0), (3, 1, 32, 1), (3, 2, 16, 0), (1, 2, 16, 1), (5, 1, 8, 0)])
def test_convolutions_above_bf16(k, stride, batch, hint, what):
    """2^106 in the data, an activation or a gradient, against zero weights: gathered, padded, strided, with sorted positions.
    Error per tensor against the same tensor in 64 bits, of its largest element; a batch norm and two layers more than above."""
    side, huge = 8, 2.0 ** 106
    k2 = int(np.log2(batch * (side // stride) ** 2))
    b = nets._Builder()
    t = b.relu(b.bn(b.conv(0, 24, bias=False)))
    t = b.conv(t, 40, k=k, stride=stride, pad=k // 2, bias=False)
    for _ in range(k2):
        t = b.add(t, t)
    b.dense(b.gap(t), CLASSES)
    rng = np.random.default_rng(k + stride)
    x = rng.standard_normal((batch, side, side, 3))
    y = rng.integers(4, CLASSES, batch)
    w0, gamma, beta = 0.3 * rng.standard_normal((3, 3, 3, 24)), np.ones(24), 0.1 * rng.standard_normal(24)
    w1 = 2.0 ** -k2 * 0.2 * rng.standard_normal((k, k, 24, 40))
    w2, b2 = 0.3 * rng.standard_normal((40, CLASSES)), np.zeros(CLASSES)
    if what == "data":
        x[1, 2, 3, 1] = x[2, 0, 0, 1] = huge
        w0[:, :, 1] = 0.0
    elif what == "activation":
        gamma[5], beta[5] = 0.0, huge
        w1[:, :, 5] = 0.0
    else:
        w1[..., 7] = 0.0
        w2[7] = 0.0
        w2[7, 3], b2[3], y[2] = huge, -1e4, 3
    w = np.concatenate([v.ravel() for v in (w0, gamma, beta, w1, w2, b2, np.zeros(24), np.ones(24))]).astype(np.float32)
    x32 = x.astype(np.float32)
    (got,) = gradients(b, (side, side, 3), batch, 1, hint, w, x32[None], y[None].astype(np.int32))
    want = torch_ref_gradient(b.array(), (side, side, 3), w, x32, y)
    at = 0
    for shape in ((3, 3, 3, 24), (24,), (24,), (k, k, 24, 40), (40, CLASSES), (CLASSES,)):
        n = int(np.prod(shape))
        g, r = got[at:at + n].reshape(shape), want[at:at + n].reshape(shape)
        at += n
        # the huge rows of a tensor and the others are measured apart
        big = np.abs(r) > 1e20
        assert np.isfinite(g).all()
        for sel in (big, ~big):
            if sel.any():
                assert np.abs(g - r)[sel].max() <= 3e-5 * max(np.abs(r)[sel].max(), 1e-3), (shape, float(np.abs(g - r)[sel].max() / np.abs(r)[sel].max()))


def torch_ref_gradient(ops, shape, w, x, y):
    return torch_ref.loss_grad(ops, shape, w.astype(np.float64), x.astype(np.float64).reshape(len(x), -1), y)[1]
