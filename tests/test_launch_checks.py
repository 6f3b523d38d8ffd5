"""What hadfl_local_steps asks the GPU to touch, checked without one: the library's real launch path runs on a stand-in for
the HIP runtime that holds every launch's operands to their regions (tests/native/launch_check.cpp)."""
import json
import os
import random
import subprocess
import sys

import numpy as np
import pytest

from oracle import nets

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="session")
def checked(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("hip") / "launch_check.so")
    subprocess.run(["/opt/rocm/llvm/bin/clang++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(HERE, "native", "launch_check.cpp"), "-o", so], check=True)

    def run(cases):
        r = subprocess.run([sys.executable, os.path.join(HERE, "native", "run_checked.py"), so], input=json.dumps(cases), text=True,
                           capture_output=True, cwd=os.path.dirname(HERE), env=dict(os.environ, PYTHONPATH=os.path.dirname(HERE)))
        assert r.returncode == 0, r.stderr[-3000:]
        return json.loads(r.stdout)
    return run


def case(builder, shape, batch, ratio, bf16, classes=10, **more):
    return dict(ops=builder.array()[:, [0, 1, 2, 4, 5, 6, 7, 8]].tolist(), shape=list(shape), batch=batch, ratio=ratio, bf16=int(bf16),
                classes=classes, **more)


def assert_clean(checked, cases):
    for c, r in zip(cases, checked(cases)):
        assert r["status"] == 0 and r["report"] == "", (c, r["report"])


def first_norm(ch=64, cout=64):
    """a batch norm behind the first convolution, read by one regular convolution, and no other batch norm"""
    b = nets._Builder()
    b.dense(b.gap(b.relu(b.conv(b.relu(b.bn(b.conv(0, ch))), cout))), 10)
    return b


def pre_activation(ch=64):
    """a residual block whose batch norm sits behind a sum"""
    b = nets._Builder()
    t = b.relu(b.conv(0, ch))
    u = b.add(b.conv(t, ch), t)
    v = b.conv(b.relu(b.bn(u)), ch)
    b.dense(b.gap(b.relu(b.add(v, u))), 10)
    return b


def pooled(ch=64):
    """a batch norm behind a pool and one with a pool folded into it"""
    b = nets._Builder()
    t = b.maxpool(b.relu(b.conv(0, ch)))
    t = b.maxpool(b.relu(b.bn(t)))
    b.dense(b.gap(b.relu(b.conv(t, 2 * ch))), 10)
    return b


@pytest.mark.parametrize("bf16", [1, 0])
def test_batch_norm_sums_stay_in_their_region(checked, bf16):
    """Batch norms that do not sit behind a convolution of their own size, from 64 to 131072 rows."""
    cases = []
    for make in (first_norm, pre_activation, pooled):
        for side, batch, n in ((8, 32, 2), (8, 64, 4), (16, 64, 16), (32, 32, 3), (32, 128, 2), (4, 4, 5)):
            cases.append(case(make(), (side, side, 3), batch, [2] + [1] * (n - 1), bf16))
    assert_clean(checked, cases)


def interleaved(ch=40):
    """Layers between a convolution and its batch norm, and between a batch norm and the convolution that reads it, which
    have sums of their own."""
    b = nets._Builder()
    t = b.relu(b.bn(b.conv(0, ch)))
    u, v = b.conv(t, ch), b.conv(t, ch, k=1, pad=0)
    w = b.conv(b.add(t, t), ch)
    x, y, z = b.bn(w), b.bn(v), b.relu(b.bn(u))
    p = b.relu(b.bn(b.add(x, y)))
    q = b.conv(z, ch)
    r = b.relu(b.bn(b.conv(p, ch)))
    b.dense(b.gap(b.add(b.bn(q), r)), 10)
    return b


@pytest.mark.parametrize("bf16", [1, 0])
@pytest.mark.parametrize("ch", [40, 64])
def test_batch_norm_reads_its_own_sums(checked, bf16, ch):
    assert_clean(checked, [case(interleaved(ch), (side, side, 3), 64, [1] * n, bf16) for side, n in ((8, 3), (32, 2))])


def random_net(rng):
    """Layers over the tensors at hand in any order: sums and batch norms of tensors made long before among them."""
    b = nets._Builder()
    side, widths = rng.choice([4, 6, 8, 16, 32]), rng.choice([(8, 40), (64, 128), (64, 128, 24), (16, 64)])
    live = [(b.conv(0, rng.choice(widths), bias=rng.random() < 0.5), side, None)]
    live[0] = (live[0][0], side, int(b.ops[-1][7]))
    for _ in range(rng.randint(3, 12)):
        t, s, c = rng.choice(live)
        kind = rng.choice(["conv", "conv", "bn", "bn", "relu", "pool", "add"])
        if kind == "conv":
            c, stride, k = rng.choice(widths), rng.choice([1, 1, 1, 2]), rng.choice([1, 3, 3])
            live.append((b.conv(t, c, k=k, stride=stride, pad=k // 2, bias=rng.random() < 0.5), (s + 2 * (k // 2) - k) // stride + 1, c))
        elif kind == "bn":
            live.append((b.bn(t), s, c))
        elif kind == "relu":
            live.append((b.relu(t), s, c))
        elif kind == "pool" and s % 2 == 0:
            live.append((b.maxpool(t), s // 2, c))
        elif kind == "add":
            same = [u for u in live if u[1:] == (s, c)]
            live.append((b.add(t, rng.choice(same)[0]), s, c))
    b.dense(b.gap(live[-1][0]), 10)
    return b, side


@pytest.mark.parametrize("seed", range(4))
def test_random_networks_stay_in_their_regions(checked, seed):
    rng = random.Random(seed)
    cases = []
    for _ in range(40):
        b, side = random_net(rng)
        n = rng.randint(1, 16)
        cases.append(case(b, (side, side, rng.choice([3, 3, 4, 16])), rng.choice([4, 32, 50, 64, 96]), [rng.randint(1, 2) for _ in range(n)], rng.randint(0, 1),
                          momentum=rng.choice([0.0, 0.9]), options=[(0, rng.randint(0, 1)), (1, rng.choice([0, 0, 1, 2]))]))
    assert_clean(checked, cases)


def layers_in(trace, part):
    return sum(part in name for name in trace)


def test_regular_layers_without_batch_norm_in_the_general_kernels(checked):
    """fp32 networks without batch norm: the regular layers (64-multiple channels, stride 1) in the general kernels in all three
    directions, every other layer in the kernels whose sums run in one chain (forward 2, data gradient 1, weight gradient 2)."""
    b = nets._Builder()
    t = b.relu(b.conv(b.relu(b.conv(b.relu(b.conv(0, 64)), 64)), 128))
    b.dense(b.maxpool(t), 10)
    c = nets._Builder()
    t = c.maxpool(c.relu(c.conv(c.maxpool(c.relu(c.conv(0, 32))), 64)))
    c.dense(t, 10)
    regular, narrow = (r["trace"] for r in checked([case(b, (8, 8, 3), 16, [1, 1], 0), case(c, (8, 8, 3), 16, [1, 1], 0)]))
    assert layers_in(regular, "conv_general") == 4 and layers_in(regular, "wgrad_general") == 2
    assert layers_in(narrow, "general") == 0 and layers_in(narrow, "igemm") == 2 + 2 + 3


def test_classifier_backward_route_by_batch(checked):
    """One launch up to 256 samples, data gradient, weight gradient and reduction beyond."""
    b = nets._Builder()
    b.dense(b.relu(b.dense(0, 64)), 10)
    cases = [case(b, (1, 1, 32), batch, [1], bf16) for bf16 in (0, 1) for batch in (256, 257)]
    assert [layers_in(r["trace"], "dense_small_bwd") for r in checked(cases)] == [1, 0, 1, 0]
    assert_clean(checked, cases)


def test_loss_gradient_by_the_classifier(checked):
    """Formed in the classifier's backward kernel where that is one launch; a launch of its own otherwise.  A row whose pieces are all
    updated elsewhere has no update launch, and cursors advance once a call."""
    cases = []
    for batch, classes, hidden in ((64, 10, 64), (256, 16, 64), (257, 10, 64), (64, 17, 64)):
        b = nets._Builder()
        b.dense(b.relu(b.dense(0, hidden)), classes)
        cases.append(case(b, (1, 1, 32), batch, [2, 1], 0, classes=classes))
    runs = checked(cases)
    assert [layers_in(r["trace"], "softmax_ce") for r in runs] == [0, 0, 2, 2]
    assert all(layers_in(r["trace"], "advance") == 1 for r in runs) and layers_in(runs[0]["trace"], "sgd_kernel") == 0
    assert_clean(checked, cases)


def test_wide_layer_on_the_data_set_by_launch_size(checked):
    """The few-rows kernel up to one and a half rounds of 128 x 128 tiles (bf16 with a short contraction: one), then generic tiles."""
    cases = []
    for features, bf16, tiles in ((784, 0, 384), (784, 1, 384), (100, 0, 384), (100, 1, 256), (96, 1, 256)):
        for cout in (64 * tiles, 64 * tiles + 1):
            b = nets._Builder()
            b.dense(b.relu(b.dense(0, cout)), 10)
            cases.append(case(b, (1, 1, features), 8, [1, 1], bf16))
    runs = checked(cases)
    assert [layers_in(r["trace"], "dense_rows_fwd") for r in runs] == [1, 0] * 5
    assert_clean(checked, cases)


def test_very_long_rows_on_the_data_set(checked):
    """The few-rows kernel addresses up to 32 samples by 32-bit byte offsets from the first: longer ones stay in the generic kernels."""
    cases = []
    for features, batch in ((34636830, 32), (34636834, 32), (34636834, 31), (268435458, 4), (268435458, 5), (357913952, 4)):
        b = nets._Builder()
        b.dense(0, 2)
        cases.append(case(b, (1, 1, features), batch, [1], 0, classes=2, momentum=0.0))
    for c, inside in zip(cases, (1, 0, 1, 1, 0, 0)):
        (run,) = checked([c])
        assert layers_in(run["trace"], "dense_rows_fwd") == inside and layers_in(run["trace"], "igemm") == 2 - inside, (c["shape"], c["batch"])
        assert run["status"] == 0 and run["report"] == "", run["report"]


def test_convolutions_on_the_data_set_by_channels(checked):
    """fp32: gathered where the generic kernel would gather too (channels not in sixteens forward, not in fours or at most 32
    rows in the weight gradient)."""
    want, cases = [], []
    for ch, k, forward, wgrad in ((3, 3, 1, 1), (8, 1, 1, 1), (8, 3, 1, 0), (12, 3, 1, 0), (16, 1, 0, 1), (16, 3, 0, 0), (32, 1, 0, 1), (18, 5, 1, 1)):
        b = nets._Builder()
        b.dense(b.gap(b.relu(b.bn(b.conv(0, 24, k=k, pad=k // 2)))), 10)
        cases.append(case(b, (12, 12, ch), 32, [2, 1], 0))
        want.append((2 * forward, 2 * wgrad))
    runs = checked(cases)
    assert [(layers_in(r["trace"], "conv_general"), layers_in(r["trace"], "wgrad_general")) for r in runs] == want
    assert_clean(checked, cases)


def test_narrow_layers_take_no_half_empty_tiles(checked):
    """Up to 32 outputs: 128 x 32 tiles (fp32) where the launch is large, never 128 x 64 or wider."""
    b = nets._Builder()
    b.dense(b.gap(b.relu(b.bn(b.conv(b.relu(b.bn(b.conv(0, 16))), 24)))), 10)
    r = checked([case(b, (28, 28, 3), 32, [1] * n, 0) for n in (4, 16)])
    for run in r:
        inner = [name for name in run["trace"] if "conv_general_kernelIf" in name][1:]
        assert len(inner) == 2 and all("ILi" not in name and "IfLi128ELi32E" in name for name in inner), inner


def test_eight_channels_with_many_taps_bf16(checked):
    want, cases = [], []
    for cin, cout, k, general in ((8, 8, 3, 2), (8, 8, 5, 0), (8, 16, 5, 2), (16, 8, 5, 2)):
        b = nets._Builder()
        b.dense(b.gap(b.relu(b.conv(b.relu(b.conv(0, cin)), cout, k=k, pad=k // 2))), 10)
        cases.append(case(b, (12, 12, 3), 32, [1, 1], 1))
        want.append(general)
    runs = checked(cases)
    assert [layers_in(r["trace"], "conv_general") for r in runs] == want
    assert_clean(checked, cases)


@pytest.mark.parametrize("shape", [(256, 128, 16, 64, 12), (256, 256, 16, 100, 12), (192, 320, 8, 100, 8), (512, 512, 4, 64, 3), (64, 64, 32, 32, 2)])
def test_lean_weight_gradient_splits(checked, shape):
    """The split sums of every count of active replicas stay in their region, and no launch takes 256 x 128 tiles unasked."""
    cin, cout, side, batch, n = shape
    b = nets._Builder()
    b.dense(b.gap(b.relu(b.conv(b.relu(b.conv(0, cin)), cout))), 10)
    cases = [case(b, (side, side, 3), batch, list(range(1, n + 1)), 1)]
    (run,) = checked(cases)
    assert layers_in(run["trace"], "wgrad_") > 0 and layers_in(run["trace"], "wgrad_kernelILi256ELi128E") == 0
    assert_clean(checked, cases)


def test_lean_weight_gradients_on_4_x_4_images(checked):
    """All taps, sixteen images a contraction; the split sums of every count of active replicas in their region.  Other images,
    filters and the hint that keeps to the general tiles do not go there."""
    cases = []
    for side, k, cin, cout, batch, n, hint in ((4, 3, 64, 128, 17, 3, 0), (4, 3, 512, 512, 64, 9, 0), (4, 3, 128, 64, 130, 1, 1), (2, 3, 64, 64, 64, 2, 0), (4, 5, 64, 64, 64, 2, 0), (4, 3, 64, 64, 64, 2, 2)):
        b = nets._Builder()
        b.dense(b.gap(b.relu(b.conv(b.relu(b.conv(0, cin)), cout, k=k, pad=k // 2))), 10)
        cases.append(case(b, (side, side, 3), batch, list(range(1, n + 1)), 1, options=[(1, hint)]))
    runs = checked(cases)
    assert [layers_in(r["trace"], "wgrad_images") > 0 for r in runs] == [True, True, True, False, False, False]
    assert_clean(checked, cases)


def test_lean_weight_gradients_of_nearly_4_gib(checked):
    """The all-taps kernel of 4 x 4 images takes sixteen images at a time, those beyond the batch by offsets beyond the tensor: the
    offsets have to fit 32 bits (1023 images would be 1024)."""
    cases = []
    for batch, cout in ((1008, 131072), (1023, 131072), (1024, 131008)):
        b = nets._Builder()
        b.dense(b.gap(b.conv(b.relu(b.conv(0, 64)), cout)), 2)
        cases.append(case(b, (4, 4, 3), batch, [1], 1, classes=2, momentum=0.0))
    for c, inside in zip(cases, (1, 0, 1)):
        (run,) = checked([c])
        assert layers_in(run["trace"], "wgrad_images") == inside and layers_in(run["trace"], "12wgrad_kernel") == 1 - inside, c["batch"]
        assert run["status"] == 0 and run["report"] == "", run["report"]


def test_split_float_layers_reach_every_tile(checked):
    """The dense layers of tests/test_gpu_split_floats.py between them take every tile of the fp32 launcher, in both directions."""
    from tests.test_gpu_split_floats import LAYERS, dense_net
    runs = checked([case(dense_net(c, n, 1), (1, 1, 32), batch, [1] * replicas, 0, classes=20, options=[(1, hint)])
                    for c, n, batch, replicas, hint in LAYERS])
    seen = {name.split("kernelIfLi")[1].split("EEEv")[0] for r in runs for name in r["trace"] if "conv_general_kernelIf" in name}
    tiles = ("32ELi32ELi1ELi1ELi8ELi1", "64ELi64ELi2ELi2ELi4ELi1", "64ELi64ELi2ELi2ELi2ELi1", "128ELi64ELi4ELi1ELi1ELi1", "128ELi128ELi2ELi4ELi1ELi2",
             "256ELi128ELi4ELi2ELi1ELi2", "128ELi32ELi4ELi1ELi1ELi1")
    missing = {"%sELi%dELb0" % (t, epi) for t in tiles for epi in (0, 1)} - seen
    assert not missing, missing


# fp32 tiles of conv_general_patch_kernel, for either direction
PATCH_TILES = ("4ELi1ELi4ELi1ELi4ELi1ELi%dELb0ELi1", "4ELi1ELi4ELi1ELi2ELi1ELi%dELb1ELi1", "4ELi2ELi2ELi1ELi6ELi1ELi%dELb0ELi1", "2ELi2ELi2ELi1ELi4ELi1ELi%dELb0ELi1",
               "2ELi2ELi2ELi1ELi2ELi2ELi%dELb1ELi1", "2ELi1ELi2ELi2ELi5ELi2ELi%dELb0ELi1", "2ELi1ELi2ELi4ELi5ELi2ELi%dELb0ELi1", "2ELi1ELi1ELi8ELi6ELi2ELi%dELb0ELi1",
               "2ELi1ELi1ELi8ELi4ELi2ELi%dELb1ELi1", "1ELi1ELi2ELi4ELi3ELi2ELi%dELb0ELi1")


def test_patch_layers_reach_every_tile(checked):
    """The layers of tests/test_gpu_patch_layers.py between them take every tile of that launcher, in both directions, and the
    route is theirs alone: a narrow, strided, 1 x 1 or very wide layer stays out of it."""
    from tests.test_gpu_patch_layers import SHAPES, net
    cases = [case(net(c, n, k), (h, w, 3), batch, [1] * replicas, 0, classes=5, options=[(1, hint)]) for (h, w), c, n, k, batch, replicas, hint in SHAPES]
    runs = checked(cases)
    assert all(r["status"] == 0 and r["report"] == "" and layers_in(r["trace"], "general_patch") == 4 for r in runs)
    seen = {name.split("patch_kernelIfLi")[1].split("EEEv")[0] for r in runs for name in r["trace"] if "general_patch" in name}
    missing = {t % epi for t in PATCH_TILES for epi in (0, 1)} - seen
    assert not missing, missing
    out = []
    for side, c, n, k, stride in ((8, 32, 64, 3, 1), (8, 64, 32, 3, 1), (8, 64, 64, 3, 2), (8, 64, 64, 1, 1), (64, 40, 40, 3, 1), (1, 64, 64, 3, 1)):
        b = nets._Builder()
        b.dense(b.gap(b.relu(b.conv(b.relu(b.bn(b.conv(0, c))), n, k=k, stride=stride, pad=k // 2))), 5)
        out.append(case(b, (side, side, 3), 16, [1], 0, classes=5))
    assert all(layers_in(r["trace"], "general_patch") == 0 for r in checked(out))


def test_patch_layers_reach_every_tile_bf16(checked):
    """The same for the bf16 layers: every tile in both directions; a strided, narrow or too wide layer stays out."""
    from tests.test_gpu_patch_layers import SHAPES_BF16, net
    runs = checked([case(net(c, n, k), (h, w, 3), batch, [1] * replicas, 1, classes=5, options=[(1, hint)]) for (h, w), c, n, k, batch, replicas, hint in SHAPES_BF16])
    assert all(r["status"] == 0 and r["report"] == "" and layers_in(r["trace"], "general_patch") == 4 for r in runs)
    seen = {name.split("patch_kernelIDF16bLi")[1].split("EEEv")[0] for r in runs for name in r["trace"] if "general_patch" in name}
    tiles = ("4ELi2ELi2ELi1ELi11ELi1ELi%dELb0ELi2", "4ELi2ELi2ELi1ELi11ELi1ELi%dELb0ELi1", "4ELi1ELi4ELi1ELi7ELi1ELi%dELb0ELi2",
             "2ELi2ELi2ELi1ELi7ELi1ELi%dELb0ELi2", "2ELi2ELi2ELi1ELi7ELi1ELi%dELb0ELi1", "2ELi1ELi2ELi2ELi9ELi2ELi%dELb0ELi1",
             "2ELi1ELi2ELi4ELi9ELi2ELi%dELb0ELi1", "1ELi1ELi2ELi4ELi7ELi2ELi%dELb0ELi1", "1ELi4ELi1ELi1ELi4ELi1ELi%dELb1ELi2")
    missing = {t % epi for t in tiles for epi in (0, 1)} - seen
    assert not missing, missing
    out = []
    for side, c, n, k, stride in ((8, 32, 64, 3, 1), (8, 64, 32, 3, 1), (8, 64, 64, 3, 2), (40, 64, 64, 3, 1), (16, 64, 64, 5, 1), (1, 64, 64, 3, 1)):
        b = nets._Builder()
        b.dense(b.gap(b.relu(b.conv(b.relu(b.bn(b.conv(0, c))), n, k=k, stride=stride, pad=k // 2))), 5)
        out.append(case(b, (side, side, 3), 16, [1], 1, classes=5))
    assert all(layers_in(r["trace"], "general_patch") == 0 for r in checked(out))


def test_tiled_layers_reach_every_tile_bf16(checked):
    """The regular bf16 layers that the patch kernel refuses between them take every tile of conv_kernel in both directions, with rows in
    memory order and sorted by position; all four of a network's launches are that kernel's."""
    from tests.test_gpu_patch_layers import TILED_BF16, net
    runs = checked([case(net(c, n, k), (h, w, 3), batch, [1] * replicas, 1, classes=5, options=[(1, hint)]) for (h, w), c, n, k, batch, replicas, hint in TILED_BF16])
    assert all(r["status"] == 0 and r["report"] == "" and layers_in(r["trace"], "11conv_kernel") == 4 and layers_in(r["trace"], "patch") == 0 for r in runs)
    seen = set()
    for r in runs:
        for name, after in zip(r["trace"], r["trace"][1:]):
            if "11conv_kernel" in name:
                seen.add((name.split("conv_kernelILi")[1].split("EEEv")[0], after == "(its_rows_sorted)"))
    tiles = ("256ELi256ELi2ELi4ELi2", "256ELi128ELi2ELi2ELi1", "256ELi64ELi2ELi2ELi1", "128ELi128ELi2ELi2ELi1", "128ELi64ELi2ELi2ELi1")
    missing = {("%sELi%d" % (t, epi), rows) for t in tiles for epi in (0, 1) for rows in (False, True)} - seen
    assert not missing, missing


def test_networks_of_the_bf16_tests_run_where_their_texts_say(checked):
    """Forward, data gradient and weight gradient of the second and third convolution in tests/test_gpu_train_bf16.py."""
    def net(k, *widths):
        b = nets._Builder()
        t = 0
        for c in widths:
            t = b.relu(b.conv(t, c, k=k if t else 3, pad=k // 2 if t else 1))
        b.dense(b.gap(t), 5)
        return b
    want = (((16, 16), 5, 1, 1, "conv_kernelILi256ELi256", "12wgrad_kernel", 0), ((8, 1), 3, 41, 1, "conv_kernelILi256ELi256", "12wgrad_kernel", 0),
            ((4, 1), 3, 96, 1, "conv_kernelILi256ELi256", "12wgrad_kernel", 1), ((8, 8), 3, 5, 1, "patch_kernelIDF16bLi4ELi2ELi2ELi1ELi11", "wgrad_taps", 0),
            ((2, 2), 3, 64, 0, "Lb1ELi2", "12wgrad_kernel", 0), ((4, 4), 3, 64, 0, "conv_general_patch", "wgrad_images", 0), ((32, 32), 3, 3, 0, "conv_general_patch", "wgrad_taps", 0))
    for ((h, w), k, batch, hint, forward, wgrad, rows) in want:
        wide = 128 if h == 32 else 256
        (run,) = checked([case(net(k, 64, wide, wide), (h, w, 3), batch, [1, 1, 1], 1, classes=5, options=[(1, hint)])])
        assert run["status"] == 0 and run["report"] == ""
        conv = [name for name in run["trace"] if "11conv_kernel" in name or "general_patch" in name]
        assert len(conv) == 4 and forward in conv[0] and forward in conv[1] and forward in conv[2], (h, w, conv)
        assert layers_in(run["trace"], wgrad) == 2 and (layers_in(run["trace"], "rows_sorted") > 0) == bool(rows), (h, w, run["trace"])


def test_layers_above_bf16_reach_every_second_pass(checked):
    """The layers of test_patch_layers_above_bf16 between them take every fp32 tile of the patch kernel in both directions, and the weight
    gradient by position in launches with split sums and without."""
    from tests.test_gpu_patch_layers import ABOVE, doubled_net
    runs = checked([case(doubled_net(c, n, k, batch * h * w, 20), (h, w, 3), batch, [1] * replicas, 0, classes=20, options=[(1, hint)])
                    for (h, w), c, n, k, batch, replicas, hint in ABOVE])
    assert all(r["status"] == 0 and r["report"] == "" for r in runs)
    seen = {name.split("patch_kernelIfLi")[1].split("EEEv")[0] for r in runs for name in r["trace"] if "general_patch" in name}
    missing = {t % epi for t in PATCH_TILES for epi in (0, 1)} - seen
    assert not missing, missing
    by_position = [r["trace"][i + 1] for r in runs for i, name in enumerate(r["trace"]) if "general_position" in name]
    assert {"splitk_reduce" in after for after in by_position} == {False, True}


def test_patch_layers_only_where_their_quotients_are_exact(checked):
    """The kernel divides a pixel's number by the image's size with a multiplication, umulhi(x, 2^32 / d rounded up): on images that it
    takes, every quotient of a pixel in a tile (up to 256 beyond the image) is the true one.  Tall images on either side."""
    from tests.test_gpu_patch_layers import TALL, TALL_BF16, net
    rng = random.Random(1)
    shapes = [(h, w, bf16) for bf16, tall in ((0, TALL), (1, TALL_BF16)) for (h, w), *_ in tall]
    for bf16, widest in ((0, 63), (1, 32)):
        shapes += [(rng.randint(900, 5000) * 32 // w, w, bf16) for w in (rng.randint(2, widest) for _ in range(12))] + [(2048, 32, bf16), (4096, 16, bf16)]
    runs = checked([case(net(40, 48, 3), (h, w, 3), 1, [1], bf16, classes=5) for h, w, bf16 in shapes])
    inside = [layers_in(r["trace"], "general_patch") for r in runs]
    assert {0, 4} == set(inside) and all(r["status"] == 0 and r["report"] == "" for r in runs)
    for (h, w, _), n in zip(shapes, inside):
        x = np.arange(h * w + 256, dtype=np.uint64)
        exact = all(np.array_equal((x * np.uint64(0xffffffff // d + 1)) >> np.uint64(32), x // np.uint64(d)) for d in (h * w, w))
        assert exact or n == 0, (h, w)
        assert n == 4 or h * w > 32768, (h, w)


def test_weight_gradients_by_position(checked):
    """fp32 3 x 3 stride-1 layers of (nearly) whole 64-channel tiles whose launch is large enough; every plan's split sums in their region."""
    from tests.test_gpu_patch_layers import SHAPES, THIN, net
    shapes = THIN[:4] + [s for s in SHAPES if s[0] in ((7, 9), (3, 2), (17, 6), (16, 16)) and s[3] == 3 and s[1] != 72]
    cases = [case(net(c, n, k), (h, w, 3), batch, [2] + [1] * (replicas - 1), 0, classes=5) for (h, w), c, n, k, batch, replicas, hint in shapes]
    assert len(cases) == 9 and all(layers_in(r["trace"], "general_position") > 0 for r in checked(cases))
    assert_clean(checked, cases)
    out = [case(net(c, n, k), (8, 8, 3), 64, [1] * 4, bf16, classes=5) for c, n, k, bf16 in ((64, 64, 5, 0), (80, 80, 3, 0), (64, 64, 3, 1))]
    assert all(layers_in(r["trace"], "general_position") == 0 for r in checked(out))


def test_gradient_of_a_shortcut(checked):
    """The copy of a sum's gradient to a shortcut without a convolution is left to the block's first convolution where that runs from
    patches, and to no other reader."""
    cases = []
    for ch, k in ((64, 3), (40, 3), (24, 3), (64, 1)):       # 24 channels, and 1 x 1 filters in fp32, are not for the patch kernel
        b = nets._Builder()
        t = b.relu(b.bn(b.conv(0, ch)))
        for _ in range(2):
            u = b.relu(b.bn(b.conv(t, ch, k=k, pad=k // 2)))
            t = b.relu(b.add(b.bn(b.conv(u, ch)), t))
        b.dense(b.gap(t), 10)
        cases += [case(b, (8, 8, 3), 32, [1], bf16) for bf16 in (0, 1)]
    assert [layers_in(r["trace"], "pass_grad") for r in checked(cases)] == [0, 0, 0, 0, 2, 2, 2, 0]
    assert_clean(checked, cases)


def residual_stages(ch):
    """two blocks with plain shortcuts, a strided one with a convolution in its shortcut, one more plain one, behind a first convolution"""
    b = nets._Builder()
    t = b.relu(b.bn(b.conv(0, ch)))
    for width, stride in ((ch, 1), (ch, 1), (2 * ch, 2), (2 * ch, 1)):
        u = b.relu(b.bn(b.conv(t, width, stride=stride)))
        u = b.bn(b.conv(u, width))
        t = b.relu(b.add(u, t if stride == 1 else b.bn(b.conv(t, width, k=1, stride=stride, pad=0))))
    b.dense(b.gap(t), 10)
    return b


def test_backward_sums_of_residual_blocks(checked):
    """Ten batch norms: those of the second plain block's and the last block's sums form their own, and the one under the strided
    shortcut; the others' come from the data gradient that completes their output's gradient.  Small tensors: one launch, no
    sums, but for those that a bf16 convolution forms from its mask."""
    cases = [case(residual_stages(ch), (16, 16, 3), batch, [1], bf16) for ch in (40, 64) for bf16 in (0, 1) for batch in (64, 2)]
    runs = checked(cases)
    assert [sum("bn_sums_vec_kernelILi1" in n for n in r["trace"]) for r in runs] == [3, 0] * 4
    assert [layers_in(r["trace"], "bn_small_bwd") for r in runs] == [0, 10, 0, 6] * 2
    assert_clean(checked, cases)


def test_batch_norms_that_add_their_sums_themselves(checked):
    """Up to 64 entries, and 64 MB read by all workgroups: no launch for the totals.  Sums of a stored bf16 output keep
    theirs, and a bf16 convolution in tiles of 256 pixels leaves fewer."""
    cases = []
    for side, batch, n in ((8, 64, 2), (8, 64, 40), (16, 64, 2)):
        b = nets._Builder()
        t = b.relu(b.bn(b.conv(0, 256)))
        b.dense(b.gap(b.relu(b.bn(b.conv(t, 256)))), 10)
        cases += [case(b, (side, side, 3), batch, [1] * n, bf16, options=[(1, 1)]) for bf16 in (0, 1)]
    runs = checked(cases)
    assert [sum("finalize" in name for name in r["trace"]) for r in runs] == [0, 1, 4, 3, 4, 3]
    assert_clean(checked, cases)


def test_weight_copies_of_many_layers(checked):
    """One launch writes the copies of up to 32 layers (the first layer, on the data set, needs none)."""
    def deep(n):
        b = nets._Builder()
        t = 0
        for _ in range(n):
            t = b.relu(b.bn(b.conv(t, 16)))
        b.dense(b.gap(t), 10)
        return b
    cases = [case(deep(n), (8, 8, 16), 4, [1, 1], bf16) for n in (33, 34) for bf16 in (0, 1)]
    assert [layers_in(r["trace"], "weight_copy") for r in checked(cases)] == [1, 1, 2, 2]
    assert_clean(checked, cases)


def test_batch_norms_with_a_pool_that_add_their_sums_themselves(checked):
    """The same limit of 64 entries where a max-pool is folded into the batch norm."""
    cases = []
    for side in (16, 32):
        b = nets._Builder()
        t = b.relu(b.bn(b.conv(0, 64)))
        t = b.maxpool(b.relu(b.bn(b.conv(t, 64))))
        b.dense(b.gap(t), 10)
        cases += [case(b, (side, side, 3), 16, [1, 1], bf16, options=[(1, 1)]) for bf16 in (0, 1)]
    runs = checked(cases)
    totals_here = [[any(k in name and "Lb1" in name for name in r["trace"]) for k in ("fwd_pool", "bwd_pool")] for r in runs]
    assert totals_here == [[True, True]] * 2 + [[True, False]] * 2     # (of 16 images of 32 x 32: 64 tiles of the convolution, 128 chunks)
    assert_clean(checked, cases)


def test_steps_of_two_dense_layers_exchange_through_two_buffers(checked):
    """A launch ends a step of some replicas and begins the next: its workgroups read each other's shares of the logits, and write those
    of the next step where none of them reads.  With replicas whose workgroups do not all run at once, and of one to three steps."""
    cases = []
    for hidden, n, batch in ((16, 3, 8), (128, 36, 32), (128, 36, 64), (192, 24, 32), (128, 9, 128)):
        b = nets._Builder()
        b.dense(b.relu(b.dense(0, hidden)), 10)
        cases += [case(b, (1, 1, 128), batch, [1 + k % 3 for k in range(n)], bf16, momentum=mom) for bf16 in (0, 1) for mom in (0.0, 0.9)]
    assert [layers_in(r["trace"], "dense_pair") for r in checked(cases)] == [4] * len(cases)
    assert_clean(checked, cases)


def test_profile_of_launches_for_several_layers_or_steps(checked):
    """Names carry a layer of the launch (the first whose copies it writes) and the replicas that it works for; work is counted
    once; a call without steps launches nothing but what counts them."""
    b = nets._Builder()
    t = 0
    for _ in range(4):
        t = b.relu(b.bn(b.conv(t, 16)))
    b.dense(b.gap(t), 10)
    pair = nets._Builder()
    pair.dense(pair.relu(pair.dense(0, 32)), 10)
    deep, mlp, none = checked([case(b, (8, 8, 16), 4, [2, 1], 0, profile=1), case(pair, (1, 1, 128), 8, [3, 1, 2], 0, profile=1, momentum=0.0),
                               case(pair, (1, 1, 128), 8, [3, 1, 2], 0, profile=1, steps=[0, 0, 0])])
    copies = [name for name in deep["profile"] if name.startswith("weight_prep")]
    layers = {int(name.split(":")[1][1:]) for name in copies}
    assert layers and layers <= {3, 6, 9} and {name.split(":")[2] for name in copies} == {"n2", "n1"}, copies
    assert sum(deep["profile"][name][0] for name in copies) == layers_in(deep["trace"], "weight_copy")
    assert sum(deep["profile"][name][2] for name in copies) == 3 * (2 + 1) * 16.0 * 9 * 16 * 16
    steps = {name: v for name, v in mlp["profile"].items() if name.startswith("dense_step")}
    assert {name: v[0] for name, v in steps.items()} == {"dense_step:L0:n3": 2, "dense_step:L0:n2": 1, "dense_step:L0:n1": 1}
    macs, out = 8 * (128 * 32 + 32 * 10), 8 * 32 * 10
    assert abs(sum(v[1] for v in steps.values()) - 6 * 2.0 * (2 * macs + out)) < 1.0
    assert [v[2] for name, v in mlp["profile"].items() if name.startswith("advance")] == [24.0 * 3]
    assert all(name.startswith("advance") for name in none["profile"]) and len(none["profile"]) == 1, none["profile"]


def test_two_dense_layers_in_one_launch_by_launch_size(checked):
    """Up to a workgroup a compute unit; up to two where a workgroup's batches and weights are small, of wide layers in calls of several
    steps; beyond that the layers' own kernels."""
    cases, want = [], []
    for features, hidden, n, batch, steps, pair in ((128, 256, 16, 64, 1, 1), (128, 256, 32, 8, 1, 1), (128, 256, 33, 8, 4, 0), (256, 256, 64, 16, 4, 0),
                                                    (784, 128, 32, 128, 1, 1), (784, 128, 33, 64, 2, 1), (784, 128, 33, 65, 2, 0),
                                                    (1024, 256, 32, 8, 2, 1), (1024, 256, 32, 8, 1, 0), (1024, 256, 16, 8, 1, 1),
                                                    (784, 128, 7, 64, 2, 1), (784, 128, 7, 65, 2, 0)):
        b = nets._Builder()
        b.dense(b.relu(b.dense(0, hidden)), 10)
        cases.append(case(b, (1, 1, features), batch, [1] * n, 0, steps=[steps] * n))
        want.append(pair * (steps + 1))
    assert [layers_in(r["trace"], "dense_pair") for r in checked(cases)] == want
    assert_clean(checked, cases)
