"""Gradients of training batches that span several tiles of the fused forward kernel, in both tile
lengths, and of batches past 65,535 tours.

The forward pass stores every layer's output for the backward pass, tile by tile; the weight
gradients and the masks of the backward convolutions read them. Weights have random signs, so that
the masks differ from position to position and a row stored at a wrong place shows; labels lie on
one side of the predictions, so that the tours' gradients do not cancel. Tolerance: the one of
test_nn_gpu.py for random weights (3e-3 of a tensor's norm: bfloat16 roundings that fp32 sums flip)."""
import numpy as np
import pytest

import gen
import oracle
from oracle import nn as nnref

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

N, L, Q = 200, 1000.0, 100


@pytest.fixture(scope="module")
def env():
    import paper_2511_18022_amd as sg
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    xy = gen.coords(31, N)
    ctx = sg.SplitContext(0)
    ctx.set_coords(xy)
    dem = gen.demand_uniform(31, N, 256, 0, 30)
    net = sg.SplitNN(ctx, seed=12, length_scale=L)
    net.set_scenarios(torch.from_numpy(dem).cuda(), Q)
    net.set_norm(0.0, 1.0)
    yield net, xy, dem
    net.close()
    ctx.close()


def tensors(g):
    off = 0
    for name, shape in nnref.param_shapes():
        size = int(np.prod(shape))
        yield name, np.asarray(g[off:off + size], dtype=np.float64)
        off += size


# 64-position tiles below 512 tiles of 128 positions, 128-position tiles from there on
@pytest.mark.parametrize("T,n", [(3, 64), (3, 65), (3, 129), (4, 193), (512, 65), (256, 129),
                                 (256, 193)])
def test_gradient_over_several_tiles(env, T, n):
    net, xy, dem = env
    tours = np.stack([gen.tour(31, N, n, variant=v) for v in range(T)])
    d = oracle.dist_matrix(xy)
    mu, sd = nnref.demand_stats(dem)
    Xs = [nnref.features(t, d, mu, sd, Q, L, xy=xy) for t in tours]
    p = net.params().astype(np.float64)
    y = nnref.forward(p, Xs)
    labels = (y - 1.0 - 0.5 * np.random.default_rng(n).random(T)).astype(np.float32)
    g, loss = net.gradient(torch.from_numpy(tours).cuda(), torch.from_numpy(labels).cuda())
    loss_ref, g_ref = nnref.loss_and_grad(p, Xs, labels.astype(np.float64))
    assert abs(loss - loss_ref) <= 1e-3 * (1 + loss_ref)
    for (name, a), (_, b) in zip(tensors(g), tensors(g_ref)):
        assert np.linalg.norm(a - b) <= 3e-3 * np.linalg.norm(b), name


def test_gradient_of_a_batch_past_65535_tours(env):
    # every tour but the last 65 has a residual of exactly 0, so the batch's gradient is that of the
    # 65 alone times 65 / 66,560 = 2^-10: an exact scaling, also through bfloat16. What is left is
    # the order of fp32 sums over about 500 rows: 32 additions in a row and a few partial sums,
    # under 64 roundings of 2^-24 of the terms' magnitudes, 25 times the norm or less.
    net, _, _ = env
    T, k, n = 66_560, 65, 3
    g = np.random.default_rng(8)
    tours = np.stack([g.permutation(np.arange(1, N + 1))[:n] for _ in range(T)]).astype(np.int32)
    dt = torch.from_numpy(tours).cuda()
    labels = net.predict(dt).clone()
    labels[-k:] -= 1.0
    big, loss = net.gradient(dt, labels)
    small, loss_small = net.gradient(dt[-k:].contiguous(), labels[-k:].contiguous())
    assert abs(loss * 1024 - loss_small) <= 1e-5 * loss_small
    for (name, a), (_, b) in zip(tensors(big), tensors(small)):
        assert np.linalg.norm(a * 1024 - b) <= 1e-4 * np.linalg.norm(b), name
