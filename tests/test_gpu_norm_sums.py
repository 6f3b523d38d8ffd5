"""Batch norms whose partial sums a convolution leaves, where no other batch norm of the same size sits beside them: updates of
every step against the oracle."""
import numpy as np
import pytest

from tests import parity_metrics as pm
from tests.pair import Pair
from tests.test_launch_checks import first_norm, interleaved, pooled, pre_activation

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
    """The sums from a lean data gradient, for a batch norm behind the first layer, a sum or a pool."""
    forced(make(), (8, 8, 3), batch, replicas, True)


@pytest.mark.parametrize("ch,bf16", [(40, False), (40, True), (64, False), (64, True)])
def test_layers_between_a_convolution_and_its_batch_norm(ch, bf16):
    """Batch norms whose sums another layer's have replaced by the time they run form their own."""
    forced(interleaved(ch), (8, 8, 3), 32, 3, bf16)
