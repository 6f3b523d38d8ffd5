"""Batch norms whose partial sums a convolution leaves, where no other batch norm of the same size sits beside them: updates of
every step against the oracle."""
import numpy as np
import pytest

from oracle import nets
from tests import parity_metrics as pm
from tests.pair import Pair
from tests.test_launch_checks import first_norm, interleaved, pooled, pre_activation, residual_stages

pytestmark = pytest.mark.gpu


def forced(builder, shape, batch, replicas, bf16):
    rng = np.random.default_rng(17)
    x = rng.standard_normal((replicas, 2 * batch) + shape).astype(np.float32)
    y = rng.integers(0, 10, size=(replicas, 2 * batch)).astype(np.int32)
    p = Pair(builder.array(), shape, replicas, 1, x, y, batch, 0.01, 0.9, [2] + [1] * (replicas - 1), bf16=bf16)
    w = p.forced_steps()
    print(batch, replicas, bf16, pm.show(w), flush=True)
    assert w["compared"] > 0
    p.close()


@pytest.mark.parametrize("batch,replicas", [(32, 2), (64, 4)])
@pytest.mark.parametrize("make", [first_norm, pre_activation, pooled])
def test_gradient_sums_of_a_lone_batch_norm_bf16(make, batch, replicas):
    """The sums from a data gradient, for a batch norm behind the first layer, a sum or a pool."""
    forced(make(), (8, 8, 3), batch, replicas, True)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("ch,side,batch,replicas", [(40, 12, 65, 2), (64, 16, 64, 1), (64, 16, 32, 9)])
def test_gradient_sums_of_residual_blocks(ch, side, batch, replicas, bf16):
    """The sums, formed with a batch norm's input, from the data gradient that completes a gradient of several parts."""
    forced(residual_stages(ch), (side, side, 3), batch, replicas, bf16)


@pytest.mark.parametrize("ch,bf16", [(40, False), (40, True), (64, False), (64, True)])
def test_layers_between_a_convolution_and_its_batch_norm(ch, bf16):
    """Batch norms whose sums another layer's have replaced by the time they run form their own."""
    forced(interleaved(ch), (8, 8, 3), 32, 3, bf16)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("side,batch,ch", [(4, 128, 40), (5, 50, 24), (2, 3, 8)])
def test_one_launch_batch_norm(side, batch, ch, bf16):
    """2048 rows, eight of a thread, the most of the kernels that keep them in registers; 1250, not a multiple; 12, fewer than threads."""
    b = nets._Builder()
    t = b.relu(b.bn(b.conv(0, ch)))
    t = b.relu(b.add(b.bn(b.conv(t, ch)), t))
    b.dense(b.gap(t), 10)
    forced(b, (side, side, 3), batch, 2, bf16)


def biased(kind):
    """A convolution with a bias in front of a batch norm of each kind: few values (one launch), many, and a pool folded in; from
    patches, and strided."""
    b = nets._Builder()
    t = b.relu(b.bn(b.conv(0, 40)))
    t = b.bn(b.conv(t, 48, stride=2) if kind == "strided" else b.conv(t, 48))
    t = b.relu(t)
    b.dense(b.gap(b.maxpool(t) if kind == "pool" else t), 10)
    return b


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("kind,side,batch,replicas", [("patch", 4, 8, 1), ("patch", 16, 64, 3), ("pool", 8, 32, 2), ("strided", 8, 16, 2), ("strided", 16, 64, 4)])
def test_bias_that_is_not_finite(kind, side, batch, replicas, value):
    """A bias of Inf or NaN in front of a batch norm reaches what the network as written makes it reach: after a step the same
    parameters and running means are not finite as in the oracle (the library's variances are clamped at zero, NaN among them).
    First layer and second, one channel."""
    rng = np.random.default_rng(5)
    x = rng.standard_normal((replicas, batch, side, side, 3)).astype(np.float32)
    y = rng.integers(0, 10, size=(replicas, batch)).astype(np.int32)
    for layer in (0, 1):
        p = Pair(biased(kind).array(), (side, side, 3), replicas, 1, x, y, batch, 0.01, 0.9, [1] * replicas)
        off, count = [(o, m) for o, m, what, _ in p.layout if what == "bias"][layer]
        for k in range(replicas):
            p.cpu.params[k][off + 3] = value
        p.share_state()
        p.gpu.local_steps()
        p.cpu.local_steps()
        for k in range(replicas):
            got, want = np.isfinite(p.gpu.params(k)), np.isfinite(p.cpu.params[k])
            differ = [(o, m, what) for o, m, what, _ in p.layout if what != "running_var" and (got[o:o + m] != want[o:o + m]).any()]
            print(kind, side, batch, replicas, value, layer, "not finite: %d of %d" % ((~want).sum(), want.size), differ, flush=True)
            assert not differ
        p.close()
