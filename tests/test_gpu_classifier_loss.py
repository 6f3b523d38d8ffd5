"""The classifier's backward kernel that forms the loss gradient itself, and the batches of the steps of one call."""
import numpy as np
import pytest

from oracle import nets
from paper_2111_08274_amd import hadfl
from tests import torch_ref

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("classes,batch,features", [(2, 1, 20), (10, 64, 784), (3, 33, 130), (16, 256, 32), (16, 257, 32), (17, 40, 36)])
def test_two_steps_of_one_call(classes, batch, features):
    """Loss and weights after two steps on two batches against 64-bit arithmetic, on both sides of the kernel's limits (16 outputs,
    256 samples).  Error of a sum of up to 784 products in fp32, 2^-24 sqrt(784), through two layers and two steps: 1e-5 of the
    largest weight update, and of the loss."""
    b = nets._Builder()
    b.dense(b.relu(b.dense(0, 64)), classes)
    rng = np.random.default_rng(batch + classes)
    x = rng.standard_normal((1, 2 * batch, 1, 1, features)).astype(np.float32)
    y = rng.integers(0, classes, (1, 2 * batch)).astype(np.int32)
    cfg = hadfl.make_config(1, 1, net="custom", custom_ops=b.array()[:, [0, 1, 2, 4, 5, 6, 7, 8]], batch=batch, n_samples=2 * batch,
                            in_shape=(1, 1, features), n_classes=classes, lr=0.1, momentum=0.0, t_sync=2)
    w0 = np.concatenate([v.ravel() for v in (rng.standard_normal((features, 64)) / np.sqrt(features), 0.1 * rng.standard_normal(64),
                                             rng.standard_normal((64, classes)) / 8, 0.1 * rng.standard_normal(classes))]).astype(np.float32)
    ctx = hadfl.Context(cfg, [1], w0=w0, x=x, y=y)
    ctx.local_steps()
    got, loss = ctx.params(0).astype(np.float64), float(ctx.losses()[0])
    ctx.close()
    w = w0.astype(np.float64)
    for step in range(2):
        part = slice(step * batch, (step + 1) * batch)
        want, grad, _ = torch_ref.loss_grad(b.array(), (1, 1, features), w, x[0, part].astype(np.float64).reshape(batch, -1), y[0, part])
        w = w - 0.1 * grad
    err = np.abs(got - w).max() / np.abs(w - w0).max()
    print(classes, batch, features, "weights %.1e loss %.1e" % (err, abs(loss - want)), flush=True)
    assert err <= 1e-5 and abs(loss - want) <= 1e-5 * max(1.0, want)
