"""The scenarios that the DP kernels leave to the tail kernel: in batches whose tours end inside the
chunks of its queue, with few and with all scenarios marked, for the 256-position history and for one
scenario per wavefront, and at the tour lengths where fewer wavefronts have room. Costs and moments
against the oracle, bit for bit; n_fallback against the same call in blocks of 16."""
import time

import numpy as np
import pytest

import gen
import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sg():
    import paper_2511_18022_amd as sg
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    return sg


def check(ctx, sg, tours, d, dem, Q, block=0):
    ctx.set_tuning(sg.SplitTuning(lane_block=block))
    cost, stats, status = ctx.eval_batch(tours, torch.from_numpy(dem).cuda(), Q)
    got = cost.cpu().numpy()
    assert status == [0] * len(tours)
    for t, tour in enumerate(tours):
        want = oracle.split(tour, d, dem, Q)
        assert np.array_equal(got[t], want), (t, len(tour))
        mom = oracle.moments(want)
        assert (stats[t].sum, stats[t].sumsq) == (mom["sum"], mom["sumsq"]), t
    return [s.n_fallback for s in stats]


@pytest.mark.parametrize("T,S", [(1, 64), (3, 65), (700, 130), (2000, 64), (40, 5000)])
@pytest.mark.parametrize("grid", [1000, 60_000])
def test_marks_across_tours_and_chunks(sg, T, S, grid):
    N = 300
    g = np.random.default_rng(T + S)
    xy = g.integers(0, grid, size=(N + 1, 2)).astype(np.int32)
    d = oracle.dist_matrix(xy)
    ctx = sg.SplitContext(0)
    ctx.set_coords(xy)
    dem = g.integers(1, 20, size=(N, S), dtype=np.int16)
    dem[:, S // 3] = 0                                   # one window over the whole tour
    dem[:, S // 2] = 3                                   # windows of 67
    dem[:, S - 1] = g.integers(1, 6, size=N)             # about 67
    tours = [g.permutation(np.arange(1, N + 1))[:n].astype(np.int32)
             for n in g.integers(1, N + 1, size=T)]
    tours[0] = np.arange(1, N + 1, dtype=np.int32)
    print(f"[tail] T={T} S={S} grid={grid}", flush=True)
    fb = check(ctx, sg, tours, d, dem, 200)
    assert fb[0] >= 3
    ctx.set_tuning(sg.SplitTuning(lane_block=16))
    _, stats, _ = ctx.eval_batch(tours, torch.from_numpy(dem).cuda(), 200)
    assert [s.n_fallback for s in stats] == fb
    ctx.close()


@pytest.mark.parametrize("block", [8, 16])
def test_every_scenario_left_by_the_block_length(sg, block):
    # suffix offsets past 16 bits in nearly every scenario, also where 8-state blocks hold them
    N, S = 120, 300
    g = np.random.default_rng(block)
    for grid in (9_000, 20_000, 200_000):
        xy = g.integers(0, grid, size=(N + 1, 2)).astype(np.int32)
        ctx = sg.SplitContext(0)
        ctx.set_coords(xy)
        dem = g.integers(1, 20, size=(N, S), dtype=np.int16)
        tours = [g.permutation(np.arange(1, N + 1)).astype(np.int32) for _ in range(3)]
        print(f"[tail] block={block} grid={grid}", flush=True)
        check(ctx, sg, tours, oracle.dist_matrix(xy), dem, 150, block)
        ctx.close()


def test_long_tours_leave_room_for_fewer_wavefronts(sg):
    # four wavefronts have room for tours of up to 2541 customers, three to 3388, two to 5083
    N, S = 5200, 70
    g = np.random.default_rng(11)
    xy = g.integers(0, 1000, size=(N + 1, 2)).astype(np.int32)
    d = oracle.dist_matrix(xy)
    ctx = sg.SplitContext(0)
    ctx.set_coords(xy)
    dem = g.integers(0, 3, size=(N, S), dtype=np.int16)  # windows of about 300
    dem[:, 66:] = g.integers(1, 20, size=(N, 4))         # about 30
    for n in (2541, 2542, 3388, 3389, 5083, 5084):
        tour = g.permutation(np.arange(1, N + 1))[:n].astype(np.int32)
        print(f"[tail] n={n}", flush=True)
        assert check(ctx, sg, [tour], d, dem, 300) == [66]
    ctx.close()


@pytest.mark.parametrize("S", [3, 200])
def test_many_short_tours_over_the_edges_of_small_workgroups(sg, S):
    # more tours than the prep kernel's large workgroups have places: 256 threads a tour
    N, T = 256, 600
    g = np.random.default_rng(S)
    xy = g.integers(0, 1000, size=(N + 1, 2)).astype(np.int32)
    ctx = sg.SplitContext(0)
    ctx.set_coords(xy)
    dem = g.integers(0, 20, size=(N, S), dtype=np.int16)
    lens = [1, 2, 63, 64, 65, 127, 128, 129, 191, 192, 193, 255, 256] * 47
    tours = [g.permutation(np.arange(1, N + 1))[:n].astype(np.int32) for n in lens[:T]]
    assert sum(check(ctx, sg, tours, oracle.dist_matrix(xy), dem, 100)) == 0
    ctx.close()


def test_a_few_marks_cost_little(sg):
    # four scenarios of every tour go one by one: a call of a few ms, not one of tens
    T, N, S = 256, 600, 16_384
    g = np.random.default_rng(4)
    ctx = sg.SplitContext(0)
    ctx.set_coords(gen.coords(63, N))
    dem = torch.randint(10, 30, (N, S), dtype=torch.int16, device="cuda")
    tours = [g.permutation(np.arange(1, N + 1)).astype(np.int32) for _ in range(T)]
    cost = torch.empty((T, S), dtype=torch.int32, device="cuda")

    def least_ms():
        ctx.eval_batch(tours, dem, 500, cost=cost)
        ts = []
        for _ in range(5):
            t0 = time.perf_counter()
            _, stats, _ = ctx.eval_batch(tours, dem, 500, cost=cost)
            ts.append(time.perf_counter() - t0)
        return min(ts) * 1e3, sum(s.n_fallback for s in stats)

    none, fb0 = least_ms()
    dem[:, ::S // 4] = 1
    few, fb4 = least_ms()
    print(f"[tail] no marks {none:.2f} ms, four scenarios a tour {few:.2f} ms", flush=True)
    assert fb0 == 0 and fb4 == 4 * T
    assert few <= 2 * none
    ctx.close()
