"""Stride-1 "same" convolutions from patches (conv_general_patch.hip), their weight gradients by position (wgrad_positions.hip), and the bf16 ones
that stay in conv_kernel (conv_bf16_fast.hip): every tile of the launchers, tiles of whole images and tiles with a border, sorted
positions, ragged channels, images and batches; and every fp32 tile on operands whose bf16 parts are not finite, in both directions."""
import numpy as np
import pytest
import torch

from oracle import nets
from paper_2111_08274_amd import hadfl
from tests import parity_metrics as pm, torch_ref
from tests.pair import Pair

pytestmark = pytest.mark.gpu
CLASSES = 5

# (image, channels in and out, k, batch, replicas, tile hint)
SHAPES = [((8, 6), 36, 132, 3, 7, 1, 0), ((8, 6), 132, 36, 3, 33, 2, 1), ((5, 7), 40, 80, 3, 50, 3, 0), ((5, 7), 40, 64, 5, 9, 2, 1),
          ((2, 2), 128, 64, 3, 32, 3, 0), ((2, 2), 64, 256, 3, 96, 2, 1), ((2, 2), 96, 64, 3, 1024, 16, 0), ((4, 4), 64, 256, 3, 32, 2, 1), ((4, 4), 160, 192, 3, 32, 2, 0),
          ((9, 63), 40, 48, 3, 2, 1, 0), ((63, 5), 48, 40, 3, 3, 2, 1), ((12, 31), 40, 48, 5, 2, 1, 1), ((16, 16), 72, 132, 3, 8, 1, 1), ((16, 16), 64, 64, 3, 32, 8, 0),
          ((10, 10), 80, 160, 3, 40, 4, 0), ((10, 10), 256, 256, 3, 16, 4, 0),
          ((4, 4), 512, 512, 3, 64, 1, 0), ((2, 2), 512, 512, 3, 64, 1, 0), ((8, 8), 256, 256, 3, 64, 1, 0),
          ((7, 9), 64, 60, 3, 50, 40, 0), ((3, 2), 192, 128, 3, 37, 6, 0), ((17, 6), 116, 64, 3, 130, 3, 0), ((16, 16), 64, 64, 3, 72, 8, 0)]

# images of one or two pixels' width or height
THIN = [((8, 1), 64, 64, 3, 50, 3, 0), ((1, 1), 64, 128, 3, 64, 2, 0), ((1, 2), 64, 64, 3, 48, 4, 0), ((2, 1), 128, 64, 3, 96, 2, 0), ((1, 8), 40, 80, 3, 32, 2, 0),
        ((1, 63), 64, 64, 3, 40, 3, 0), ((1, 9), 72, 64, 3, 130, 2, 1), ((31, 2), 64, 64, 3, 40, 4, 0), ((1, 5), 64, 64, 5, 33, 2, 0)]
THIN_BF16 = [((1, 32), 64, 64, 3, 20, 2, 0), ((1, 9), 40, 80, 3, 33, 2, 0), ((32, 2), 64, 128, 3, 18, 2, 0), ((2, 31), 64, 72, 3, 32, 2, 1), ((1, 4), 128, 128, 3, 64, 3, 0)]
# tall images: the first of either list has too many pixels for the kernel's quotients (tests/test_launch_checks.py), the second has not
TALL = [((1112, 60), 36, 40, 3, 1, 1, 0), ((1060, 60), 36, 40, 3, 1, 1, 0)]
# bf16 regular layers that the kernel does not take (wide images, large filters on 16 pixels' width, images of one pixel's width or less than
# four pixels): every tile of conv_kernel, in both directions, with sorted rows where the batch is a multiple of 32
TILED_BF16 = [((64, 64), 128, 128, 3, 2, 1, 0), ((64, 64), 128, 128, 3, 4, 8, 0), ((64, 64), 64, 64, 3, 4, 8, 0), ((16, 16), 64, 128, 5, 3, 2, 0), ((16, 16), 256, 256, 5, 2, 1, 1),
              ((16, 64), 256, 256, 3, 8, 8, 0), ((1, 1), 128, 256, 3, 64, 2, 0), ((8, 1), 256, 64, 3, 41, 2, 1), ((8, 1), 64, 128, 3, 96, 2, 0), ((16, 1), 256, 256, 3, 32, 3, 1),
              ((1, 2), 64, 64, 3, 33, 2, 0), ((4, 1), 128, 192, 5, 64, 3, 0), ((8, 1), 64, 128, 3, 1024, 16, 0), ((8, 1), 128, 64, 3, 1024, 16, 0)]
TALL_BF16 = [((2200, 31), 40, 48, 3, 1, 1, 0), ((2048, 32), 40, 48, 3, 1, 1, 0)]


def net(c, n, k):
    b = nets._Builder()
    t = b.relu(b.bn(b.conv(0, c, bias=False)))
    t = b.relu(b.bn(b.conv(t, n, k=k, pad=k // 2, bias=False)))
    t = b.relu(b.conv(t, n, k=k, pad=k // 2))
    b.dense(b.gap(t), CLASSES)
    return b


@pytest.mark.parametrize("shape", SHAPES + THIN + TALL)
def test_patch_layers(shape):
    """Gradients of one step, read from the momentum buffers, against the same network in 64 bits.  Bound: the error of a sum of
    K products in fp32, 2^-24 sqrt(K), K <= 4608 products and up to 66720 pixels, and as much again through each of two batch
    norms and a softmax: 3e-5 of a tensor's largest gradient (floored at 1e-3 of the largest of all).  Where a ReLU's input lies within that of zero its unit may open on one side and not on the other: up to a
    hundredth of a tensor's values (one filter and one column) may be off by 5e-3 for it."""
    (h, w), c, n, k, batch, replicas, hint = shape
    rng = np.random.default_rng(c + n + batch)
    x = rng.standard_normal((1, batch, h, w, 3)).astype(np.float32)
    y = rng.integers(0, CLASSES, (1, batch)).astype(np.int32)
    cfg = hadfl.make_config(replicas, 1, net="custom", custom_ops=net(c, n, k).array()[:, [0, 1, 2, 4, 5, 6, 7, 8]], batch=batch, n_samples=batch,
                            in_shape=(h, w, 3), n_classes=CLASSES, lr=1e-30, momentum=0.5)
    layout = hadfl.param_layout(cfg)
    w0 = np.zeros(max(o + m for o, m, _, _ in layout), dtype=np.float32)
    for off, cnt, kind, fan_in in layout:
        w0[off:off + cnt] = {"weight": rng.standard_normal(cnt) * np.sqrt(2.0 / max(fan_in, 1)), "bias": 0.1 * rng.standard_normal(cnt), "gamma": 1.0, "running_var": 1.0}.get(kind, 0.0)
    ctx = hadfl.Context(cfg, [1] * replicas, w0=w0, x=np.repeat(x, replicas, 0), y=np.repeat(y, replicas, 0), options={hadfl.OPT_TILE_HINT: hint})
    ctx.local_steps()
    got = [ctx.momentum(r).astype(np.float64) for r in sorted({0, replicas - 1})]
    ctx.close()
    want = torch_ref.loss_grad(net(c, n, k).array(), (h, w, 3), w0.astype(np.float64), x[0].astype(np.float64).reshape(batch, -1), y[0])[1]
    floor = 1e-3 * max(np.abs(want[o:o + m]).max() for o, m, kind, _ in layout if o + m <= got[0].size)
    for g in got:
        for off, cnt, kind, _ in layout:
            if off + cnt > g.size:
                continue
            err = np.abs(g[off:off + cnt] - want[off:off + cnt]) / max(np.abs(want[off:off + cnt]).max(), floor)
            print(shape, kind, cnt, "max %.1e median %.1e" % (err.max(), np.median(err)), flush=True)
            assert err.max() <= 5e-3 and (err > 3e-5).mean() <= 0.01, (shape, kind, float(err.max()), float((err > 3e-5).mean()))


# bf16 (image, channels in and out, k, batch, replicas, tile hint)
SHAPES_BF16 = [((8, 8), 64, 136, 3, 9, 2, 1), ((16, 32), 72, 64, 3, 5, 2, 1), ((5, 7), 40, 264, 3, 50, 1, 0), ((8, 6), 72, 200, 5, 40, 12, 0), ((16, 16), 128, 128, 3, 60, 4, 0),
               ((8, 8), 128, 256, 3, 64, 16, 0), ((10, 10), 40, 80, 3, 33, 6, 0), ((32, 32), 64, 64, 3, 17, 2, 0), ((4, 4), 256, 512, 3, 32, 1, 0), ((4, 4), 512, 512, 3, 50, 2, 0),
               ((2, 2), 256, 512, 3, 32, 1, 0), ((2, 2), 512, 512, 3, 128, 12, 0), ((2, 2), 256, 256, 3, 1024, 4, 0), ((7, 31), 48, 64, 1, 20, 2, 0), ((64, 9), 64, 64, 1, 8, 2, 0),
               ((4, 4), 64, 128, 3, 17, 3, 0), ((4, 4), 128, 64, 3, 130, 1, 0), ((4, 4), 256, 512, 3, 16, 9, 0)]         # (4 x 4: weight gradients by images, ragged sixteens, splits)


@pytest.mark.parametrize("shape", SHAPES_BF16 + THIN_BF16 + TALL_BF16 + TILED_BF16)
def test_patch_layers_bf16(shape):
    """Gradients of one step against the same network in 64 bits, in the 2-norm of a tensor.  What roundings to bf16 do to a
    tensor (units within 2^-9 of zero that open on one side only, sums that nearly cancel) is measured on the 64-bit network: the
    difference that rounding its weights to bf16 makes.  The library also rounds three activations and their gradients, so at
    most some three times as many roundings of that size: bound 4 times that difference, and 1e-2 (ten roundings of 2^-9) for what
    it misses.  A tap, channel or pixel astray is of order 1."""
    (h, w), c, n, k, batch, replicas, hint = shape
    rng = np.random.default_rng(c + n + batch)
    x = rng.standard_normal((1, batch, h, w, 3)).astype(np.float32)
    y = rng.integers(0, CLASSES, (1, batch)).astype(np.int32)
    cfg = hadfl.make_config(replicas, 1, net="custom", custom_ops=net(c, n, k).array()[:, [0, 1, 2, 4, 5, 6, 7, 8]], batch=batch, n_samples=batch,
                            in_shape=(h, w, 3), n_classes=CLASSES, lr=1e-30, momentum=0.5, bf16=1)
    layout = hadfl.param_layout(cfg)
    w0 = np.zeros(max(o + m for o, m, _, _ in layout), dtype=np.float32)
    for off, cnt, kind, fan_in in layout:
        w0[off:off + cnt] = {"weight": rng.standard_normal(cnt) * np.sqrt(2.0 / max(fan_in, 1)), "bias": 0.1 * rng.standard_normal(cnt), "gamma": 1.0, "running_var": 1.0}.get(kind, 0.0)
    ctx = hadfl.Context(cfg, [1] * replicas, w0=w0, x=np.repeat(x, replicas, 0), y=np.repeat(y, replicas, 0), options={hadfl.OPT_TILE_HINT: hint})
    ctx.local_steps()
    got = [ctx.momentum(r).astype(np.float64) for r in sorted({0, replicas - 1})]
    ctx.close()
    exact, rounded = (torch_ref.loss_grad(net(c, n, k).array(), (h, w, 3), v.astype(np.float64), x[0].astype(np.float64).reshape(batch, -1), y[0])[1]
                      for v in (w0, torch.as_tensor(w0).bfloat16().float().numpy()))
    for g in got:
        for off, cnt, kind, _ in layout:
            if off + cnt > g.size:
                continue
            part = slice(off, off + cnt)
            size = np.linalg.norm(exact[part])
            err, twin = np.linalg.norm(g[part] - exact[part]) / size, np.linalg.norm(rounded[part] - exact[part]) / size
            print(shape, kind, cnt, "%.1e (twin %.1e)" % (err, twin), flush=True)
            assert err <= 4 * twin + 1e-2, (shape, kind, off, float(err), float(twin))


# (image, channels in and out, k, batch, replicas, tile hint): every fp32 tile in both directions, and weight gradients by position
# (tests/test_launch_checks.py)
ABOVE = [((8, 8), 40, 72, 3, 32, 1, 0), ((8, 8), 40, 72, 3, 32, 1, 1), ((2, 2), 40, 72, 3, 256, 1, 0), ((7, 7), 40, 72, 3, 16, 1, 0), ((16, 16), 40, 72, 5, 16, 1, 1),
         ((32, 32), 40, 72, 3, 64, 1, 0), ((16, 16), 64, 64, 3, 50, 1, 0), ((9, 9), 64, 128, 3, 130, 1, 0), ((16, 16), 72, 132, 3, 8, 1, 1), ((4, 4), 64, 256, 3, 32, 2, 1),
         ((4, 4), 256, 64, 3, 32, 2, 1), ((5, 7), 40, 64, 5, 9, 2, 1), ((16, 16), 64, 64, 3, 32, 8, 0), ((2, 2), 96, 64, 3, 1024, 16, 0), ((2, 2), 64, 96, 3, 1024, 16, 0),
         ((8, 8), 256, 256, 3, 64, 1, 0), ((4, 4), 160, 192, 3, 32, 2, 0), ((2, 2), 512, 512, 3, 64, 1, 0), ((3, 2), 192, 128, 3, 37, 6, 0), ((17, 6), 116, 64, 3, 130, 3, 0)]


def doubled_net(c, n, k, pixels, classes):
    b = nets._Builder()
    t = b.conv(b.relu(b.bn(b.conv(0, c, bias=False))), n, k=k, pad=k // 2, bias=False)
    for _ in range(int(np.log2(pixels))):
        t = b.add(t, t)
    b.dense(b.gap(t), classes)
    return b


@pytest.mark.parametrize("what", ["activation", "gradient"])
@pytest.mark.parametrize("shape", ABOVE)
def test_patch_layers_above_bf16(shape, what):
    """2^106 in an activation or a gradient, against zero weights: as parts they are Inf * 0, and the tile of the convolution, the data
    gradient or the weight gradient is computed again from the floats.  Error as in tests/test_gpu_split_floats.py, whose layers
    are narrower: 3e-5 of a tensor's largest value, the huge ones apart."""
    (h, w_), c, n, k, batch, replicas, hint = shape
    huge, classes = 2.0 ** 106, 20
    k2 = int(np.log2(batch * h * w_))
    b = doubled_net(c, n, k, batch * h * w_, classes)
    rng = np.random.default_rng(k + h)
    x = rng.standard_normal((batch, h, w_, 3)).astype(np.float32)
    y = rng.integers(4, classes, batch)
    w0, gamma, beta = 0.3 * rng.standard_normal((3, 3, 3, c)), np.ones(c), 0.1 * rng.standard_normal(c)
    w1 = 2.0 ** -k2 * 0.2 * rng.standard_normal((k, k, c, n))
    w2, b2 = 0.3 * rng.standard_normal((n, classes)), np.zeros(classes)
    if what == "activation":
        gamma[5], beta[5] = 0.0, huge
        w1[:, :, 5] = 0.0
    else:
        w1[..., 7] = 0.0
        w2[7] = 0.0
        w2[7, 3], b2[3], y[2] = huge, -1e4, 3
    w = np.concatenate([v.ravel() for v in (w0, gamma, beta, w1, w2, b2, np.zeros(c), np.ones(c))]).astype(np.float32)
    cfg = hadfl.make_config(replicas, 1, net="custom", custom_ops=b.array()[:, [0, 1, 2, 4, 5, 6, 7, 8]], batch=batch, n_samples=batch,
                            in_shape=(h, w_, 3), n_classes=classes, lr=1e-30, momentum=0.5)
    ctx = hadfl.Context(cfg, [1] * replicas, w0=w, x=np.repeat(x[None], replicas, 0), y=np.repeat(y[None].astype(np.int32), replicas, 0), options={hadfl.OPT_TILE_HINT: hint})
    ctx.local_steps()
    all_got = [ctx.momentum(r).astype(np.float64) for r in sorted({0, replicas - 1})]
    ctx.close()
    want = torch_ref.loss_grad(b.array(), (h, w_, 3), w.astype(np.float64), x.astype(np.float64).reshape(batch, -1), y)[1]
    for got in all_got:
        at = 0
        for part in ((3, 3, 3, c), (c,), (c,), (k, k, c, n), (n, classes), (classes,)):
            m = int(np.prod(part))
            g, r = got[at:at + m], want[at:at + m]
            at += m
            assert np.isfinite(g).all(), (shape, part)
            big = np.abs(r) > 1e20
            for sel in (big, ~big):
                if sel.any():
                    err = np.abs(g - r)[sel].max() / max(np.abs(r)[sel].max(), 1e-3)
                    print(shape, what, part, "%.1e" % err, flush=True)
                    assert err <= 3e-5, (shape, part, float(err))
