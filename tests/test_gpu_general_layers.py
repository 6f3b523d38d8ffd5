"""The kernels for layers of any geometry, on floats split into three bf16 and on bf16: ragged channel counts, images, strides
and batches, each tile size of the launchers, and floats that bf16 cannot hold."""
import numpy as np
import pytest
import torch

from oracle import nets
from paper_2111_08274_amd import hadfl
from tests import parity_metrics as pm, torch_ref
from tests.pair import Pair

pytestmark = pytest.mark.gpu


def _nets():
    c = {}
    b = nets._Builder()                       # channels of 4 .. 132, stride 2 and 3, filters of 1, 3 and 5, a padded 1 x 1
    t = b.relu(b.conv(b.relu(b.conv(0, 4)), 36))
    t = b.relu(b.bn(b.conv(t, 68, stride=2, bias=False)))
    t = b.relu(b.conv(t, 132, k=5, stride=3, pad=2))
    t = b.relu(b.conv(t, 12, k=1, pad=1))
    b.dense(b.relu(b.dense(t, 20)), 5)
    c["ragged"] = (b.array(), (13, 9, 3), 7)
    b = nets._Builder()                       # a residual block whose two convolutions meet in one gradient, projection with stride 2
    t = b.relu(b.bn(b.conv(0, 40, bias=False)))
    u = b.bn(b.conv(b.relu(b.bn(b.conv(t, 80, stride=2, bias=False))), 80, bias=False))
    t = b.relu(b.add(u, b.bn(b.conv(t, 80, k=1, stride=2, pad=0, bias=False))))
    b.dense(b.gap(t), 5)
    c["residual"] = (b.array(), (10, 10, 3), 33)
    b = nets._Builder()                       # positions sorted by their taps, in both directions and the weight gradient
    t = b.relu(b.conv(b.relu(b.bn(b.conv(0, 32))), 128))
    t = b.relu(b.conv(b.maxpool(t), 96, bias=False))
    b.dense(b.gap(t), 5)
    c["tables"] = (b.array(), (8, 6, 3), 64)
    b = nets._Builder()                       # the same in groups of eight channels, for bf16
    t = b.relu(b.conv(b.relu(b.conv(0, 8)), 40))
    t = b.relu(b.bn(b.conv(t, 72, stride=2, bias=False)))
    t = b.relu(b.conv(t, 136, k=5, stride=3, pad=2))
    t = b.relu(b.conv(t, 24, k=1, pad=1))
    b.dense(b.relu(b.dense(t, 32)), 5)
    c["eights"] = (b.array(), (13, 9, 3), 7)
    b = nets._Builder()                       # a hidden layer on the (fp32) data set, contraction of 25 slabs
    b.dense(b.relu(b.dense(0, 128)), 5)
    c["dense"] = (b.array(), (1, 1, 784), 50)
    for ch, cout, pad in ((3, 20, 2), (1, 72, 0)):       # convolutions on the data set, 75 and 25 values per output: ragged slabs and rows
        b = nets._Builder()
        b.dense(b.gap(b.relu(b.bn(b.conv(b.relu(b.conv(0, cout, k=5, stride=2, pad=pad)), 8, bias=False)))), 5)
        c["first%d" % ch] = (b.array(), (11, 14, ch), 21)
    b = nets._Builder()                       # sums: of two convolutions, of a sum, without a ReLU, of one tensor twice, of a normalised tensor read twice
    t = b.relu(b.bn(b.conv(0, 16, bias=False)))
    u = b.add(b.conv(t, 16), b.conv(t, 16, k=1, pad=0))
    v = b.add(b.bn(b.conv(u, 16, bias=False)), u)
    w = b.bn(b.conv(b.relu(v), 16, bias=False))
    x = b.relu(b.add(b.add(w, w), b.bn(b.conv(w, 16, bias=False))))
    y = b.add(b.bn(b.conv(x, 16, k=1, pad=0)), b.bn(b.conv(x, 16, bias=False)))
    b.dense(b.gap(y), 5)
    c["sums"] = (b.array(), (6, 8, 3), 16)
    return c


NETS = _nets()


@pytest.mark.parametrize("hint", [0, 1])
@pytest.mark.parametrize("replicas", [2, 9])
@pytest.mark.parametrize("name,bf16", [(n, False) for n in sorted(NETS)] + [(n, True) for n in sorted(NETS) if n in ("eights", "residual", "tables", "dense", "sums")])
def test_general_layers_against_oracle(name, bf16, replicas, hint):
    """Every tensor's update of every step against the oracle.  Two and nine replicas put the launches on both sides of the
    tile rules (a few workgroups with several wave groups along K; one group), hint 1 takes the largest tiles."""
    ops, shape, batch = NETS[name]
    rng = np.random.default_rng(31)
    x = rng.standard_normal((replicas, 2 * batch) + shape).astype(np.float32)
    y = rng.integers(0, 5, size=(replicas, 2 * batch)).astype(np.int32)
    p = Pair(ops, shape, replicas, 1, x, y, batch, 0.01, 0.9, [2] + [1] * (replicas - 1), bf16=bf16, options={hadfl.OPT_TILE_HINT: hint})
    w = p.forced_steps()
    print(name, bf16, replicas, hint, pm.show(w), flush=True)
    assert w["compared"] > 0
    assert p.max_rel_diff() <= 2e-2 if bf16 else p.max_param_diff() <= 1e-4
    p.close()


def test_values_bf16_cannot_hold():
    """A dense classifier on the data set (forward in the kernel for few rows, weight gradient in the general one, whose second
    pass this reaches; the convolution kernels' is in test_gpu_split_floats.py), compared with 64-bit arithmetic where fp32 stays finite but the bf16 parts do not:
    a weight of -Inf (logit -Inf, probability 0), a weight and an input above bf16's largest number, the input against
    zero weights.  Error bound: 64 products and 24 samples in fp32, 88 * 2^-24 < 1e-5 relative."""
    d, classes, batch, lr = 64, 20, 24, 0.5
    rng = np.random.default_rng(5)
    x = rng.standard_normal((1, batch, 1, 1, d)).astype(np.float32)
    y = rng.integers(0, 7, size=(1, batch)).astype(np.int32)
    x[0, :, 0, 0, 3] = 1.0
    x[0, 2, 0, 0, 5] = 3.4e38
    b = nets._Builder()
    b.dense(0, classes)
    cfg = hadfl.make_config(1, 1, net="custom", custom_ops=b.array()[:, [0, 1, 2, 4, 5, 6, 7, 8]], batch=batch, n_samples=batch,
                            in_shape=(1, 1, d), n_classes=classes, lr=lr, momentum=0.0)
    w = (0.1 * rng.standard_normal((d, classes))).astype(np.float32)
    w[5] = 0.0
    w[3, 7] = -np.inf
    w[3, 8] = -3.4e38
    bias = np.zeros(classes, dtype=np.float32)
    ctx = hadfl.Context(cfg, [1], w0=np.concatenate([w.ravel(), bias]), x=x, y=y)
    ctx.local_steps()
    got, loss = ctx.params(0), float(ctx.losses()[0])
    ctx.close()
    xd, wd = x[0, :, 0, 0].astype(np.float64), w.astype(np.float64)
    logits = xd @ wd
    e = np.exp(logits - logits.max(1, keepdims=True))
    p = e / e.sum(1, keepdims=True)
    assert np.isfinite(loss)
    assert abs(loss + np.log(p[np.arange(batch), y[0]]).mean()) <= 1e-5
    p[np.arange(batch), y[0]] -= 1.0
    want = np.concatenate([(wd - lr * (xd.T @ (p / batch))).ravel(), -lr * p.sum(0) / batch])
    same = np.isfinite(want)
    assert np.array_equal(got[~same].astype(np.float64), want[~same]) and np.isfinite(got[same]).all()
    scale = np.concatenate([np.abs(wd) + lr * (np.abs(xd).T @ (np.abs(p) / batch)), lr * np.abs(p).sum(0)[None] / batch])
    assert (np.abs(got[same] - want[same]) <= 1e-5 * scale.ravel()[same] + 1e-30).all()


@pytest.mark.parametrize("replicas", [2, 9])
@pytest.mark.parametrize("side", [6, 8, 20])
def test_regular_layers_without_batch_norm_f32(side, replicas):
    """Convolutions of 64-multiple channels in a net without batch norm, behind and in front of layers that keep the
    kernels of such nets; 6 x 6 and 8 x 8 images have their positions sorted."""
    b = nets._Builder()
    t = b.relu(b.conv(b.relu(b.conv(0, 64)), 64))
    t = b.relu(b.conv(b.maxpool(b.relu(b.conv(t, 128, k=1, pad=0))), 64))
    u = b.relu(b.conv(t, 64, bias=False))
    b.dense(b.gap(b.relu(b.add(b.conv(u, 64), t))), 5)
    rng = np.random.default_rng(7)
    x = rng.standard_normal((replicas, 64, side, side, 3)).astype(np.float32)
    y = rng.integers(0, 5, size=(replicas, 64)).astype(np.int32)
    p = Pair(b.array(), (side, side, 3), replicas, 1, x, y, 32, 0.01, 0.9, [2] + [1] * (replicas - 1))
    w = p.forced_steps()
    print(side, replicas, pm.show(w), flush=True)
    assert w["compared"] > 0 and p.max_param_diff() <= 1e-4
    p.close()


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("batch", [256, 257, 1000])
def test_classifier_of_many_samples(batch, bf16):
    """Both sides of the rule that takes a classifier's backward pass out of its one-launch kernel."""
    b = nets._Builder()
    b.dense(b.relu(b.dense(0, 67)), 5)
    rng = np.random.default_rng(3)
    x = rng.standard_normal((3, batch, 1, 1, 33)).astype(np.float32)
    y = rng.integers(0, 5, size=(3, batch)).astype(np.int32)
    p = Pair(b.array(), (1, 1, 33), 3, 1, x, y, batch, 0.01, 0.9, [2, 1, 1], bf16=bf16)
    w = p.forced_steps()
    print(batch, bf16, pm.show(w), flush=True)
    assert w["compared"] > 0 and (p.max_rel_diff() <= 2e-2 if bf16 else p.max_param_diff() <= 1e-4)
    p.close()


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("features,cout", [(48, 128 * 28), (48, 128 * 29), (520, 128 * 42), (520, 128 * 43), (33, 128 * 43 + 5)])
def test_wide_layer_on_the_data_set(features, cout, bf16):
    """Both sides of the rule that takes a layer on the data set out of the few-rows kernel (nine replicas, 252 to 396 tiles)."""
    b = nets._Builder()
    b.dense(b.relu(b.dense(0, cout)), 5)
    rng = np.random.default_rng(3)
    x = rng.standard_normal((9, 6, 1, 1, features)).astype(np.float32)
    y = rng.integers(0, 5, size=(9, 6)).astype(np.int32)
    p = Pair(b.array(), (1, 1, features), 9, 1, x, y, 6, 0.01, 0.9, [1] * 9, bf16=bf16)
    w = p.forced_steps()
    print(features, cout, bf16, pm.show(w), flush=True)
    assert w["compared"] > 0 and (p.max_rel_diff() <= 2e-2 if bf16 else p.max_param_diff() <= 1e-4)
    p.close()


@pytest.mark.parametrize("replicas", [2, 9])
@pytest.mark.parametrize("channels,k", [(4, 3), (8, 3), (16, 1), (16, 3)])
def test_convolutions_on_a_data_set_of_many_channels(channels, k, replicas):
    """Each direction on the gathering kernel or the generic one, by the channel count."""
    b = nets._Builder()
    t = b.relu(b.bn(b.conv(0, 24, k=k, pad=k // 2)))
    b.dense(b.gap(b.relu(b.conv(t, 16, stride=2))), 5)
    rng = np.random.default_rng(9)
    x = rng.standard_normal((replicas, 66, 12, 10, channels)).astype(np.float32)
    y = rng.integers(0, 5, size=(replicas, 66)).astype(np.int32)
    p = Pair(b.array(), (12, 10, channels), replicas, 1, x, y, 33, 0.01, 0.9, [2] + [1] * (replicas - 1))
    w = p.forced_steps()
    print(channels, k, replicas, pm.show(w), flush=True)
    assert w["compared"] > 0 and p.max_param_diff() <= 1e-4
    p.close()


@pytest.mark.parametrize("cin,cout,k", [(8, 8, 3), (8, 8, 5), (8, 16, 5), (16, 8, 5)])
def test_narrow_filters_of_many_taps_bf16(cin, cout, k):
    """Both sides of the rule that leaves 8-channel layers of more than nine taps to the generic kernels."""
    b = nets._Builder()
    t = b.relu(b.conv(0, cin))
    b.dense(b.gap(b.relu(b.conv(b.relu(b.conv(t, cout, k=k, pad=k // 2)), cin, k=k, pad=k // 2))), 5)
    rng = np.random.default_rng(9)
    x = rng.standard_normal((3, 26, 12, 10, 3)).astype(np.float32)
    y = rng.integers(0, 5, size=(3, 26)).astype(np.int32)
    p = Pair(b.array(), (12, 10, 3), 3, 1, x, y, 13, 0.01, 0.9, [2, 1, 1], bf16=True)
    w = p.forced_steps()
    print(cin, cout, k, pm.show(w), flush=True)
    assert w["compared"] > 0 and p.max_rel_diff() <= 2e-2
    p.close()


def test_image_rows_of_gibibytes():
    """A filter's rows lie more than 2^31 values apart: three rows of 2^26 pixels with sixteen channels, of which a strided convolution
    reads windows of 3 x 3.  Reference: the windows side by side, in 64 bits.  Sums of 16385 values in fp32, 2^-24 sqrt(16385), in
    the average, the loss gradient behind it and the weight gradient: 3e-5 of the largest gradient of a tensor."""
    width, step, classes = 2 ** 26 + 3, 4096, 3
    n = (width - 3) // step + 1
    b, c = nets._Builder(), nets._Builder()
    for net, stride in ((b, step), (c, 3)):
        net.dense(net.gap(net.conv(0, 4, stride=stride, pad=0)), classes)
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    x = torch.zeros(1, 1, 3, width, 16, device="cuda")
    windows = torch.randn(3, n, 3, 16, device="cuda", generator=g) + 0.5
    x[0, 0, :, :(n - 1) * step].view(3, n - 1, step, 16)[:, :, :3] = windows[:, :-1]
    x[0, 0, :, (n - 1) * step:] = windows[:, -1]
    y = np.ones((1, 1), dtype=np.int32)
    w0 = (0.1 * np.random.default_rng(2).standard_normal(144 * 4 + 4 + 4 * classes + classes)).astype(np.float32)
    cfg = hadfl.make_config(1, 1, net="custom", custom_ops=b.array()[:, [0, 1, 2, 4, 5, 6, 7, 8]], batch=1, n_samples=1, in_shape=(3, width, 16),
                            n_classes=classes, lr=1e-30, momentum=0.5)
    ctx = hadfl.Context(cfg, [1], w0=w0, x=x, y=y)
    ctx.local_steps()
    got = ctx.momentum(0).astype(np.float64)
    ctx.close()
    compact = windows.reshape(1, 3, 3 * n, 16).double().cpu().numpy().reshape(1, -1)
    want = torch_ref.loss_grad(c.array(), (3, 3 * n, 16), w0.astype(np.float64), compact, y[0])[1]
    at = 0
    for size in (144 * 4, 4, 4 * classes, classes):
        err = np.abs(got[at:at + size] - want[at:at + size]).max() / np.abs(want[at:at + size]).max()
        print(size, "%.1e" % err, flush=True)
        assert err <= 3e-5
        at += size


@pytest.mark.parametrize("bf16", [False, True])
def test_layers_whose_output_nobody_reads(bf16):
    """A convolution with a ReLU, a batch norm with a pool, a sum and a dense layer beside the network: their gradient is zero, whatever
    the workspace holds (NaN here), and their parameters stay where they are."""
    b = nets._Builder()
    t = b.relu(b.bn(b.conv(0, 64)))
    b.relu(b.conv(t, 40))
    b.maxpool(b.relu(b.bn(b.conv(t, 64))))
    b.add(t, b.conv(t, 64, k=1, pad=0))
    b.dense(t, 20)
    b.dense(b.gap(b.relu(b.conv(t, 48))), 5)
    rng = np.random.default_rng(4)
    x = rng.standard_normal((2, 2 * 24, 8, 8, 3)).astype(np.float32)
    y = rng.integers(0, 5, size=(2, 2 * 24)).astype(np.int32)
    p = Pair(b.array(), (8, 8, 3), 2, 1, x, y, 24, 0.01, 0.9, [2, 1], bf16=bf16)
    # (in front: the aggregate and the momentum of two replicas; behind: small state, less than 16 KiB)
    p.gpu.scratch.view(torch.float32)[3 * p.gpu.row_stride:-4096] = float("nan")
    w = p.forced_steps()
    print(bf16, pm.show(w), flush=True)
    assert w["compared"] > 0 and (p.max_rel_diff() <= 2e-2 if bf16 else p.max_param_diff() <= 1e-4)
    p.close()
