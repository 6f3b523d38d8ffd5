"""Networks of two dense layers, whose steps run end to beginning in one kernel, at the edges of its blocks (16 features, 16 hidden units, 32
samples) and of its range."""
import numpy as np
import pytest

from oracle import nets
from paper_2111_08274_amd import hadfl, synth
from tests import torch_ref
from tests.pair import Pair

pytestmark = pytest.mark.gpu


def net(hidden, classes):
    b = nets._Builder()
    b.dense(b.relu(b.dense(0, hidden)), classes)
    return b.array()


@pytest.mark.parametrize("features,hidden,classes,batch,huge", [(128, 16, 2, 1, False), (784, 128, 10, 33, False), (144, 48, 16, 31, False),
                                                                (1024, 256, 3, 64, False), (784, 128, 10, 32, True)])
def test_steps_of_one_call(features, hidden, classes, batch, huge):
    """Three replicas with 3, 2 and 1 steps and momentum, weights and the last loss against 64-bit arithmetic.  Error of a sum of up to 1024
    products in fp32, 2^-24 sqrt(1024), through two layers and three steps: 1e-5 of the largest update.  One feature of one sample at
    2^105, where the split floats overflow: its row of the weights by itself."""
    rng = np.random.default_rng(batch + classes)
    ops, ratio, lr, mom = net(hidden, classes), [3, 1, 2], 0.1, 0.9
    x = rng.standard_normal((3, 2 * batch, 1, 1, features)).astype(np.float32)
    if huge:
        x[:, 5, 0, 0, 17] = 2.0 ** 105
    y = rng.integers(0, classes, (3, 2 * batch)).astype(np.int32)
    cfg = hadfl.make_config(3, 1, net="custom", custom_ops=ops[:, [0, 1, 2, 4, 5, 6, 7, 8]], batch=batch, n_samples=2 * batch,
                            in_shape=(1, 1, features), n_classes=classes, lr=lr, momentum=mom)
    w0 = np.concatenate([v.ravel() for v in (rng.standard_normal((features, hidden)) / np.sqrt(features), 0.1 * rng.standard_normal(hidden),
                                             rng.standard_normal((hidden, classes)) / np.sqrt(hidden), 0.1 * rng.standard_normal(classes))]).astype(np.float32)
    ctx = hadfl.Context(cfg, ratio, w0=w0, x=x, y=y)
    if huge:
        ctx.set_steps([1, 0, 1])                  # (the weights that follow are as large)
    ctx.local_steps()
    got, losses = [ctx.params(k).astype(np.float64) for k in range(3)], ctx.losses()
    ctx.close()
    for k, steps in enumerate([1, 0, 1] if huge else ratio):
        w, buf = w0.astype(np.float64), 0.0
        for s in range(steps):
            part = slice(s % 2 * batch, (s % 2 + 1) * batch)
            want, grad, _ = torch_ref.loss_grad(ops, (1, 1, features), w, x[k, part].astype(np.float64).reshape(batch, -1), y[k, part])
            buf = mom * buf + grad
            w = w - lr * buf
        if not steps:
            assert np.array_equal(got[k], w)
            continue
        row = np.zeros(w.size, bool)
        if huge:
            row[17 * hidden:18 * hidden] = True
            row[features * hidden + hidden:] = True        # (the hidden units of that sample are as large)
        for part in (row, ~row) if huge else (~row,):
            err = np.abs(got[k] - w)[part].max() / np.abs(w - w0)[part].max()
            print(k, "weights %.1e loss %.1e of %.1e" % (err, abs(losses[k] - want), want), flush=True)
            assert err <= 1e-5
        assert abs(losses[k] - want) <= 1e-5 * max(1.0, want)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("features,hidden,batch,replicas", [(784, 128, 100, 9), (160, 32, 128, 8), (784, 128, 8, 4)])
def test_against_the_oracle(features, hidden, batch, replicas, bf16):
    x, y = synth.class_shift_images(replicas, 2 * batch, (1, 1, features), 10, seed=3)
    p = Pair(net(hidden, 10), (1, 1, features), replicas, 2, x, y, batch, 0.05, 0.9, [1 + k % 3 for k in range(replicas)], bf16=bf16)
    for _ in range(2):
        p.forced_steps()
    p.local_steps(check_updates=True)
    p.close()


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("hidden,replicas,batch", [(128, 36, 32), (128, 36, 64), (192, 24, 32), (192, 42, 8), (256, 32, 16)])
def test_more_workgroups_than_run_at_once(hidden, replicas, batch, bf16):
    """288 to 512 workgroups, so that those of one replica begin at different times; one to three steps, momentum, two calls.  A replica's
    arithmetic does not depend on the others: every third one has the same data and steps, and the same bits as in a context of three
    replicas.  That one's first call is the same as test_steps_of_one_call's, with its bound (bf16: test_against_the_oracle)."""
    rng = np.random.default_rng(hidden + replicas + batch)
    ops, features, lr, mom = net(hidden, 10), 784, 0.1, 0.9
    x = rng.standard_normal((3, 2 * batch, 1, 1, features)).astype(np.float32)
    y = rng.integers(0, 10, (3, 2 * batch)).astype(np.int32)
    w0 = np.concatenate([v.ravel() for v in (rng.standard_normal((features, hidden)) / np.sqrt(features), 0.1 * rng.standard_normal(hidden),
                                             rng.standard_normal((hidden, 10)) / np.sqrt(hidden), 0.1 * rng.standard_normal(10))]).astype(np.float32)

    def calls(n):
        which = np.arange(n) % 3
        cfg = hadfl.make_config(n, 1, net="custom", custom_ops=ops[:, [0, 1, 2, 4, 5, 6, 7, 8]], batch=batch, n_samples=2 * batch,
                                in_shape=(1, 1, features), n_classes=10, lr=lr, momentum=mom, bf16=int(bf16))
        ctx = hadfl.Context(cfg, 1 + which, w0=w0, x=x[which], y=y[which])
        out = []
        for _ in range(2):
            ctx.local_steps()
            out.append(([ctx.params(k) for k in range(n)], ctx.losses()))
        ctx.close()
        return out

    few, many = calls(3), calls(replicas)
    for (w_few, l_few), (w_many, l_many) in zip(few, many):
        for k in range(replicas):
            assert np.array_equal(w_many[k], w_few[k % 3]) and l_many[k] == l_few[k % 3], k
    if bf16:
        return
    for k in range(3):
        w, buf = w0.astype(np.float64), 0.0
        for s in range(k + 1):
            part = slice(s % 2 * batch, (s % 2 + 1) * batch)
            want, grad, _ = torch_ref.loss_grad(ops, (1, 1, features), w, x[k, part].astype(np.float64).reshape(batch, -1), y[k, part])
            buf = mom * buf + grad
            w = w - lr * buf
        got, losses = few[0]
        err = np.abs(got[k] - w).max() / np.abs(w - w0).max()
        print(k, "weights %.1e loss %.1e of %.1e" % (err, abs(losses[k] - want), want), flush=True)
        assert err <= 1e-5 and abs(losses[k] - want) <= 1e-5 * max(1.0, want)
