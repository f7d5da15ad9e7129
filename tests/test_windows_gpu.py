"""Window lengths around the edges of the kernels' histories: blocks of 8 states keep windows of up
to 23 positions, blocks of 16 up to 47, the long kernel up to 239. Costs and moments against the
oracle, bit for bit, and n_fallback against its definition: the scenarios whose window of some last
state of a full 16-state block (but the last block) holds more than 47 predecessors."""
import numpy as np
import pytest

import gen
import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

N, S = 700, 130


@pytest.fixture(scope="module")
def ctx():
    import paper_2511_18022_amd as sg
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    c = sg.SplitContext(0)
    c.set_coords(gen.coords(21, N))
    yield c
    c.close()


def past_history(tour, dem, Q):
    n = len(tour)
    P = np.zeros((n + 1, dem.shape[1]), dtype=np.int64)
    P[1:] = np.cumsum(dem[tour - 1], axis=0)
    hit = np.zeros(dem.shape[1], dtype=bool)
    for i in range(63, 16 * (n // 16), 16):
        hit |= P[i] - P[i - 48] <= Q
    return int(hit.sum())


def demands(window, spread, seed):
    """Windows of about `window` customers: demands of 8 each, or 8 plus or minus `spread`."""
    g = np.random.default_rng(seed)
    dem = np.full((N, S), 8, dtype=np.int16)
    if spread:
        dem += g.integers(-spread, spread + 1, size=dem.shape, dtype=np.int16)
    return dem, 8 * window


@pytest.mark.parametrize("n", [700, 641, 96, 16])
@pytest.mark.parametrize("window", [6, 17, 18, 19, 23, 24, 30, 44, 45, 46, 47, 48, 49, 90, 111, 224,
                                    238, 239, 240, 256, 690])
def test_windows_at_the_edges_of_the_histories(ctx, window, n):
    d = oracle.dist_matrix(gen.coords(21, N))
    tour = gen.tour(21, N, n, variant=3)
    for spread in (0, 7):
        dem, Q = demands(window, spread, window)
        want = oracle.split(tour, d, dem, Q)
        cost, st = ctx.eval(tour, torch.from_numpy(dem).cuda(), Q)
        assert np.array_equal(cost.cpu().numpy(), want), (window, n, spread)
        mom = oracle.moments(want)
        assert (st.sum, st.sumsq, st.mean, st.var) == (mom["sum"], mom["sumsq"], mom["mean"],
                                                      mom["var"])
        assert st.n_fallback == past_history(tour, dem, Q), (window, n, spread)


def test_tours_of_short_middling_and_long_windows_in_one_batch(ctx):
    # the classes are taken tour by tour: one demand matrix, tours over customers of small, middling
    # and large demands, and some scenarios whose windows outgrow what their tour's sample shows
    d = oracle.dist_matrix(gen.coords(21, N))
    g = np.random.default_rng(5)
    dem = np.empty((N, S), dtype=np.int16)
    dem[:200] = g.integers(1, 4, size=(200, S))     # Q / 2: windows of about 100
    dem[200:450] = g.integers(3, 12, size=(250, S))  # about 27
    dem[450:] = g.integers(14, 20, size=(250, S))    # about 12
    dem[200:, 127] = 1
    Q = 200
    ids = [np.arange(1, 201), np.arange(201, 451), np.arange(451, 701), np.arange(1, 701)]
    tours = [g.permutation(i).astype(np.int32) for i in ids]
    dt = torch.from_numpy(dem).cuda()
    graph = ctx.graph(4, 4 * N, dt, Q)
    cost, stats, status = ctx.eval_batch(tours, dt, Q)
    for t, tour in enumerate(tours):
        want = oracle.split(tour, d, dem, Q)
        assert np.array_equal(cost[t].cpu().numpy(), want), t
        assert stats[t].sum == oracle.moments(want)["sum"]
        assert stats[t].n_fallback == past_history(tour, dem, Q), t
    for _ in range(3):
        got = graph.launch(tours)
        gstats, gstatus = graph.stats()
        assert torch.equal(got, cost) and gstatus == [0] * 4
        assert [s.n_fallback for s in gstats] == [s.n_fallback for s in stats]
    graph.close()


def test_infeasible_demand_under_long_windows(ctx):
    import paper_2511_18022_amd as sg
    tour = gen.tour(21, N, 300, variant=4)
    dem, Q = demands(100, 3, 9)
    dem[int(tour[150]) - 1, 77] = Q + 1
    with pytest.raises(sg.SplitError) as ei:
        ctx.eval(tour, torch.from_numpy(dem).cuda(), Q)
    assert ei.value.status == sg.SPLIT_E_DEMAND


@pytest.mark.parametrize("block", [0, 16])
def test_two_wavefronts_per_item_over_every_remainder(ctx, block):
    # few work items of long tours run from both ends: every n mod 32 (the middle, the shift of the
    # mirrored half, the last block's tail), tours too short to be split, an asymmetric matrix
    import paper_2511_18022_amd as sg
    g = np.random.default_rng(77)
    d = g.integers(1, 1500, size=(N + 1, N + 1)).astype(np.int32)
    c = sg.SplitContext(0)
    c.set_dist(d)
    c.set_tuning(sg.SplitTuning(sg.FORM_AUTO, 0, 0, 0, block))
    lens = [*range(321, 353), 700, 1, 2, 15, 16, 17, 31, 33, 47, 48]
    tours = [g.permutation(np.arange(1, N + 1))[:n].astype(np.int32) for n in lens]
    for mean, Q in ((8, 90), (8, 200), (8, 330)):
        dem = g.integers(0, 2 * mean + 1, size=(N, S), dtype=np.int16)
        cost, stats, status = c.eval_batch(tours, torch.from_numpy(dem).cuda(), Q)
        assert status == [0] * len(tours)
        for t, tour in enumerate(tours):
            want = oracle.split(tour, d, dem, Q)
            assert np.array_equal(cost[t].cpu().numpy(), want), (lens[t], Q)
            assert stats[t].sumsq == oracle.moments(want)["sumsq"], (lens[t], Q)
            assert stats[t].n_fallback == past_history(tour, dem, Q), (lens[t], Q)
    # an infeasible demand at the customers around the middle, and at the ends
    tour = tours[0]
    for at in (0, 140, 143, 144, 145, 159, 160, 320):
        bad = dem.copy()
        bad[int(tour[at]) - 1, 99] = Q + 1
        with pytest.raises(sg.SplitError) as ei:
            c.eval(tour, torch.from_numpy(bad).cuda(), Q)
        assert ei.value.status == sg.SPLIT_E_DEMAND, at
    c.close()


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 20, 31, 32, 33])
def test_short_tours_in_one_launch(ctx, n):
    # edges of the tour length and of the workgroups' scenario counts, windows from one customer to
    # the whole tour, a demand row stride, large capacities (the lane kernel's demand bound), calls
    # after one another (the counters are left at zero), infeasible and negative demands
    import paper_2511_18022_amd as sg
    g = np.random.default_rng(n)
    d = oracle.dist_matrix(gen.coords(21, N))
    tour = g.permutation(np.arange(1, N + 1))[:n].astype(np.int32)
    for s, Q, top in ((1, 10, 10), (255, 40, 20), (256, 1000, 20), (257, 60, 60), (4099, 90, 20),
                      (32768, 45, 20), (32769, 45, 20), (300, 16383, 4000), (300, 32767, 32767)):
        dem = g.integers(0, top + 1, size=(N, s), dtype=np.int16)
        want = oracle.split(tour, d, dem, Q)
        pad = torch.zeros((N, s + 5), dtype=torch.int16, device="cuda")
        pad[:, :s] = torch.from_numpy(dem).cuda()
        mom = oracle.moments(want)
        for _ in range(2):
            cost, st = ctx.eval(tour, pad[:, :s], Q)
            assert np.array_equal(cost.cpu().numpy(), want), (n, s, Q)
            assert (st.sum, st.sumsq, st.mean, st.var) == (mom["sum"], mom["sumsq"], mom["mean"],
                                                          mom["var"])
        lane = not (n <= (32 if s <= 256 else 24 if s <= 1024 else 16 if s <= 4096 else 0)
                    or Q > 16383)
        over = 8 * np.bitwise_or.reduce(dem[tour - 1].astype(np.int64), axis=0) + Q > 32767
        assert st.n_fallback == (int(over.sum()) if lane else 0), (n, s, Q)
        for value in (Q + 1 if Q < 32767 else -1, -1):
            bad = pad.clone()
            bad[int(tour[n // 2]) - 1, s // 2] = value
            with pytest.raises(sg.SplitError) as ei:
                ctx.eval(tour, bad[:, :s], Q)
            assert ei.value.status == sg.SPLIT_E_DEMAND
