"""fp32 networks with convolutions and without batch norm, whose sums run in one chain: the first layer's split weight gradient, added split by
split from LDS, its gathered rows, and the classifier on long rows."""
import numpy as np
import pytest

from oracle import nets
from paper_2111_08274_amd import hadfl
from tests import torch_ref

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cin,k,cout,side,batch,classes,momentum", [(3, 3, 8, 32, 64, 10, 0.9),      # 256 splits; 224 outputs
                                                                    (1, 5, 12, 16, 16, 7, 0.9),      # 32 splits, 312 outputs: no multiple of 16; odd classes
                                                                    (2, 1, 4, 20, 9, 2, 0.0),        # 12 outputs, rows and pixels that fill no slab
                                                                    (5, 3, 20, 9, 50, 16, 0.0)])     # 920 outputs; 1620 features
def test_two_steps(cin, k, cout, side, batch, classes, momentum):
    """Loss and weights after two steps on two replicas against 64-bit arithmetic.  Sums of up to 65536 products in chains of at most some
    300 and as many partial sums, 2^-24 sqrt(300) each, through two layers and two steps: 1e-5 of a tensor's largest update; and a
    rounding of its largest weight a step, 2^-24 of it, which counts where the update is a few thousandths of the weight."""
    b = nets._Builder()
    b.dense(b.relu(b.conv(0, cout, k=k, pad=k // 2)), classes)
    rng = np.random.default_rng(side + classes)
    shape = (side, side, cin)
    x = rng.standard_normal((2, 2 * batch) + shape).astype(np.float32)
    y = rng.integers(0, classes, (2, 2 * batch)).astype(np.int32)
    cfg = hadfl.make_config(2, 1, net="custom", custom_ops=b.array()[:, [0, 1, 2, 4, 5, 6, 7, 8]], batch=batch, n_samples=2 * batch,
                            in_shape=shape, n_classes=classes, lr=0.02, momentum=momentum)
    sizes = (k * k * cin * cout, cout, side * side * cout * classes, classes)
    w0 = np.concatenate([s * rng.standard_normal(n) for n, s in zip(sizes, (1 / (k * cin ** 0.5), 0.1, (side * side * cout) ** -0.5, 0.1))]).astype(np.float32)
    ctx = hadfl.Context(cfg, [2, 1], w0=w0, x=x, y=y)
    ctx.local_steps()
    got, losses = [ctx.params(r).astype(np.float64) for r in range(2)], ctx.losses()
    ctx.close()
    for r, steps in enumerate((2, 1)):
        w, buf = w0.astype(np.float64), 0.0
        for s in range(steps):
            part = slice(s * batch, (s + 1) * batch)
            want, grad, _ = torch_ref.loss_grad(b.array(), shape, w, x[r, part].astype(np.float64).reshape(batch, -1), y[r, part])
            buf = momentum * buf + grad
            w = w - 0.02 * buf
        parts = [slice(o, o + n) for o, n in zip(np.cumsum((0,) + sizes[:-1]), sizes)]
        err = [np.abs(got[r] - w)[t].max() / (np.abs(w - w0)[t].max() + 1e5 * steps * 2.0 ** -24 * np.abs(w[t]).max()) for t in parts]
        print(r, "weights", " ".join("%.1e" % e for e in err), "loss %.1e" % abs(losses[r] - want), flush=True)
        assert max(err) <= 1e-5 and abs(losses[r] - want) <= 1e-5 * max(1.0, want)


@pytest.mark.parametrize("cin,c1,c2,k,side,batch,replicas", [(3, 16, 48, 3, 9, 7, 2), (1, 32, 16, 5, 11, 33, 1), (3, 48, 36, 1, 8, 64, 3),
                                                             (2, 40, 32, 3, 10, 20, 2), (3, 32, 64, 3, 16, 64, 4), (8, 32, 16, 3, 5, 128, 5)])
def test_second_layer(cin, c1, c2, k, side, batch, replicas):
    """A step through a stride-1 layer from a patch with all channels, or (a side of it without 16-channel groups) from the tiled kernel: rows
    that fill no tile, outputs that fill no block, both tile heights, images wider and narrower than a border.  Bound as above."""
    b = nets._Builder()
    b.dense(b.gap(b.relu(b.conv(b.relu(b.conv(0, c1)), c2, k=k, pad=k // 2))), 10)
    rng = np.random.default_rng(c1 + c2 + side)
    shape = (side, side, cin)
    x = rng.standard_normal((replicas, batch) + shape).astype(np.float32)
    y = rng.integers(0, 10, (replicas, batch)).astype(np.int32)
    cfg = hadfl.make_config(replicas, 1, net="custom", custom_ops=b.array()[:, [0, 1, 2, 4, 5, 6, 7, 8]], batch=batch, n_samples=batch,
                            in_shape=shape, lr=0.1, momentum=0.0)
    sizes = (9 * cin * c1, c1, k * k * c1 * c2, c2, c2 * 10, 10)
    w0 = np.concatenate([s * rng.standard_normal(n) for n, s in zip(sizes, ((4.5 * cin) ** -0.5, 0.1, (0.5 * k * k * c1) ** -0.5, 0.1, c2 ** -0.5, 0.1))]).astype(np.float32)
    ctx = hadfl.Context(cfg, [1] * replicas, w0=w0, x=x, y=y)
    ctx.local_steps()
    got, losses = [ctx.params(r).astype(np.float64) for r in range(replicas)], ctx.losses()
    ctx.close()
    parts = [slice(o, o + n) for o, n in zip(np.cumsum((0,) + sizes[:-1]), sizes)]
    for r in range(replicas):
        want, grad, _ = torch_ref.loss_grad(b.array(), shape, w0.astype(np.float64), x[r].astype(np.float64).reshape(batch, -1), y[r])
        w = w0 - 0.1 * grad
        err = [np.abs(got[r] - w)[t].max() / (np.abs(0.1 * grad)[t].max() + 1e5 * 2.0 ** -24 * np.abs(w[t]).max()) for t in parts]
        print(r, "weights", " ".join("%.1e" % e for e in err), "loss %.1e" % abs(losses[r] - want), flush=True)
        assert max(err) <= 1e-5 and abs(losses[r] - want) <= 1e-5 * max(1.0, want)
