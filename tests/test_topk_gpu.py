"""GPU tests of the top-k selection at the edges of its two forms: one workgroup up to 16,384
scores, digit passes over chunks of scores beyond, against a stable sort."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2511_18022_amd as sg
    c = sg.SplitContext(0)
    yield c
    c.close()


def scores_of(kind, C, rng):
    if kind == "ties":
        return np.round(rng.normal(0, 3, C), 1).astype(np.float32) + np.float32(0.05)
    if kind == "equal":
        return np.full(C, 7.25, dtype=np.float32)
    if kind == "infinite":
        s = rng.normal(60000, 3000, C).astype(np.float32)
        s[rng.integers(0, C, size=max(1, C // 9))] = np.inf
        s[rng.integers(0, C, size=max(1, C // 9))] = -np.inf
        return s
    return rng.normal(60000, 3000, C).astype(np.float32)


@pytest.mark.parametrize("kind", ["costs", "ties", "equal", "infinite"])
@pytest.mark.parametrize("C", [1, 63, 1024, 1025, 16383, 16384, 16385, 1024 * 1024,
                               1024 * 1024 + 1, 2_500_003])
def test_topk_across_its_forms(ctx, C, kind):
    import paper_2511_18022_amd as sg
    rng = np.random.default_rng(C)
    s = scores_of(kind, C, rng)
    d = torch.from_numpy(s).cuda()
    order = np.argsort(s, kind="stable")
    for K in sorted({1, max(1, C // 100), max(1, C // 2), C}):
        print(f"[topk] {kind} C={C} K={K}", flush=True)
        idx = sg.topk_smallest(ctx, d, K).cpu().numpy()
        assert np.array_equal(idx, np.sort(order[:K]))


def test_topk_of_a_misaligned_view(ctx):
    import paper_2511_18022_amd as sg
    rng = np.random.default_rng(5)
    s = rng.normal(0, 1, 40_001).astype(np.float32)
    idx = sg.topk_smallest(ctx, torch.from_numpy(s).cuda()[1:], 400).cpu().numpy()
    assert np.array_equal(idx, np.sort(np.argsort(s[1:], kind="stable")[:400]))
