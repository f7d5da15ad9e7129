"""The fused forward kernel at the edges of its tiles, for prediction (64- and 128-position tiles) and
for training (which also stores every layer): predictions of one tour against those of a batch, bit for bit, and the
training pass's loss against the predictions, which go through the same layers and head."""
import numpy as np
import pytest

import gen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 127, 128, 129, 191, 193, 300])
@pytest.mark.parametrize("T", [1, 3, 520])
def test_tile_edges(n, T):
    import paper_2511_18022_amd as sg
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    if T == 520 and n > 129:
        T = 175  # 128-position tiles too (512 tiles and more)
    N = 300
    g = np.random.default_rng(n)
    ctx = sg.SplitContext(0)
    ctx.set_coords(gen.coords(5, N))
    nn = sg.SplitNN(ctx, seed=3, length_scale=1000.0)
    dem = torch.from_numpy(g.integers(1, 40, size=(N, 256), dtype=np.int16)).cuda()
    nn.set_scenarios(dem, 200)
    nn.set_norm(0.0, 1.0)
    tours = np.stack([g.permutation(np.arange(1, N + 1))[:n] for _ in range(T)]).astype(np.int32)
    dt = torch.from_numpy(tours).cuda()
    pred = nn.predict(dt)
    # one tour at a time runs in 64-position tiles: the same bits as any batch
    for t in (0, T - 1):
        assert torch.equal(nn.predict(dt[t:t + 1].contiguous()), pred[t:t + 1])
    # labels at a distance of 1: the squared errors of the training pass's own outputs (in float32;
    # its outputs equal the predictions up to the float32 rounding of the normalization)
    labels = pred + 1.0
    grad, loss = nn.gradient(dt, labels)
    want = float(((labels.double() - pred.double()) ** 2).mean())
    scale = 1.0 + float(pred.abs().max())
    assert abs(loss - want) <= 8 * 2.0 ** -24 * scale * (1.0 + T ** 0.5), (loss, want)
    assert np.isfinite(grad).all()
    ctx.close()
