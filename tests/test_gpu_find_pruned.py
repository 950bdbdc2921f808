"""The default search of larger batches (blocks of units left out by their bounding boxes)
against the oracle, bit for bit: sizes around the edges of its leaves (32 units), blocks of
leaves (512) and blocks of those (8,192), both lane counts, and inputs for which the first
bound is poor or no bound helps."""
import numpy as np
import pytest

from parity import Pair, assert_find_equal, assert_iter_equal

pytestmark = pytest.mark.gpu


def shape(kind, n, m, seed):
    rng = np.random.default_rng(seed)
    units = rng.standard_normal((3, n)).astype(np.float32)
    sig = rng.standard_normal((3, m)).astype(np.float32)
    if kind == "grid":          # exact ties and duplicated units
        units = rng.integers(-3, 4, (3, n)).astype(np.float32)
        sig = rng.integers(-3, 4, (3, m)).astype(np.float32)
    elif kind == "clusters":    # cells with no units near the signals, far from any home
        units = (units * 1e-3 + rng.integers(0, 2, (1, n)) * 50.0).astype(np.float32)
        sig = (sig * 30.0 + 25.0).astype(np.float32)
    elif kind == "sphere":      # every unit about equally far from the signals
        units /= np.linalg.norm(units, axis=0, keepdims=True)
        sig *= np.float32(1e-7)
    elif kind == "line":        # flat boxes, one cell side of zero units
        units[1:] = 0.5
    elif kind == "overflow":    # distances past the binary32 range: all ties by index
        units *= np.float32(3e19)
        sig[:, ::3] *= np.float32(1e25)
    if kind != "sphere":
        k = min(n, m) // 3
        sig[:, :k] = units[:, n - k:]
    return units, np.ascontiguousarray(sig)


@pytest.mark.parametrize("kind", ["random", "grid", "clusters", "sphere", "line", "overflow"])
@pytest.mark.parametrize("n,m", [(2, 257), (31, 300), (32, 257), (33, 1_000), (511, 300),
                                 (513, 999), (8_192, 257), (8_193, 301), (20_011, 700),
                                 (700, 8_193)])
def test_sizes_and_shapes(kind, n, m):
    units, sig = shape(kind, n, m, n + m)
    pair = Pair(units, m_max=m)
    g, o = pair.find(sig)
    assert_find_equal(g, o, f"{kind} n={n} m={m}")


def test_units_far_from_their_place_in_the_order():
    """Units that jump onto their signals (eps_b 1) between rebuilds of the spatial order: the
    boxes are those of the present positions however old the order is, and each call's outer
    boxes are its own."""
    from paper_1503_08294_amd import gsn
    rng = np.random.default_rng(5)
    n, m = 9_000, 600
    units = rng.standard_normal((3, n)).astype(np.float32)
    pair = Pair(units, m_max=m, eps_b=1.0, eps_n=0.5, max_age=3)
    pair.net.tune(gsn.GSN_TUNE_REBUCKET, 4096)
    for t in range(12):
        sig = (rng.standard_normal((3, m)) * (1.0 + 2.0 * (t % 4))).astype(np.float32)
        g, o = pair.iterate(sig)
        assert_iter_equal(g, o, f"iteration {t}")
    pair.compare_state("end")


def test_switching_between_the_search_and_the_scans():
    """The staged scans and the search share the unit order and keep their own copies of the
    positions: alternating them on one handle changes nothing."""
    from paper_1503_08294_amd import gsn
    rng = np.random.default_rng(6)
    units = rng.standard_normal((3, 5_000)).astype(np.float32)
    pair = Pair(units, m_max=2_000, lock_mode=1)
    for t, variant in enumerate((0, 4, 0, 3, 4, 0, 0, 2, 5, 0)):
        pair.net.tune(gsn.GSN_TUNE_VARIANT, variant)
        sig = rng.standard_normal((3, 500 + 150 * t)).astype(np.float32)
        g, o = pair.iterate(sig)
        assert_iter_equal(g, o, f"call {t} variant {variant}")
    pair.compare_state("end")


@pytest.mark.parametrize("lock_mode", [0, 1, 2])
def test_records_follow_every_change_of_the_units(lock_mode):
    """The update leaves the records for the next search, so whatever else moves, adds, removes
    or replaces units must not let an older record be used: separate calls, the index, growth
    with removal, an import, small batches, a recorded loop and two finds in a row, mixed."""
    import torch
    from paper_1503_08294_amd import gsn
    rng = np.random.default_rng(40 + lock_mode)
    n, m = 3_000, 400
    units = rng.standard_normal((3, n)).astype(np.float32)
    pair = Pair(units, n_max=n + 64, e_max=8 * n, m_max=m, eps_b=0.4, eps_n=0.05, max_age=2,
                lock_mode=lock_mode)
    pair.net.tune(gsn.GSN_TUNE_REBUCKET, 7)
    lo, h, dims = [-5.0] * 3, 0.5, [20] * 3
    grid = gsn.make_grid(lo, h, dims)
    ws = pair.net.grid_workspace(grid)

    def batch(k=m):
        return rng.standard_normal((3, k)).astype(np.float32)

    for t in range(1, 31):
        what = ("fused", "steps", "grow", "small", "index", "twice", "import", "loop", "still")[
            int(rng.integers(0, 9))]
        sig = batch(60 if what == "small" else m)
        if what in ("fused", "small"):
            assert_iter_equal(*pair.iterate(sig), f"{t} {what}")
        elif what == "steps":
            assert_iter_equal(*pair.iterate(sig, calls="steps"), f"{t} {what}")
        elif what == "grow":
            assert_iter_equal(*pair.iterate(sig, t, t, True), f"{t} {what}")
        elif what == "index":
            dev = pair.to_dev(sig)
            pair.net.find_winners_grid(dev, grid, ws)
            acc = pair.net.update(dev).cpu().numpy()
            ow, osec, od1, od2 = pair.orc.find_winners_grid(sig, lo, h, dims)[:4]
            oacc = pair.orc.resolve_conflicts(ow, osec, od1)
            pair.orc.adapt(sig, ow, osec, od1, oacc)
            pair.orc.update_edges(ow, osec, oacc)
            np.testing.assert_array_equal(acc, oacc, err_msg=f"{t} {what}")
        elif what == "twice":
            for _ in range(2):
                assert_find_equal(*pair.find(batch()), f"{t} {what}")
        elif what == "still":
            for _ in range(10):
                assert_find_equal(*pair.find(batch(37)), f"{t} {what}")
        elif what == "import":
            s = pair.orc.export()
            s["xyz"] = (s["xyz"] * np.float32(1.1)).astype(np.float32)
            pair.net.import_state(torch.from_numpy(s["xyz"]), torch.from_numpy(s["err"]),
                                  torch.from_numpy(s["edges"]))
            pair.orc.import_state(s["xyz"], s["err"], s["edges"])
        else:
            sigs = [batch() for _ in range(3)]
            dev = pair.to_dev(np.stack(sigs))
            g = [x.cpu().numpy() for x in pair.net.iterate_loop(dev)]
            for x in sigs:
                o = pair.orc.iterate(x, 0, 0, False)
            assert_iter_equal(g, o, f"{t} {what}")
        pair.compare_state(f"{t} {what}")
    assert pair.net.check() == 0


@pytest.mark.parametrize("m", [64, 600])
def test_a_find_recorded_by_the_caller(m):
    """A find captured into the caller's own graph while records of the units are at hand,
    replayed after iterations that move them, between eager finds and iterations."""
    import torch
    rng = np.random.default_rng(m)
    n = 4_000
    units = rng.standard_normal((3, n)).astype(np.float32)
    pair = Pair(units, m_max=600, eps_b=0.5, eps_n=0.1, max_age=3)

    def step():
        assert_iter_equal(*pair.iterate(rng.standard_normal((3, 600)).astype(np.float32)))

    sig = pair.to_dev(rng.standard_normal((3, m)).astype(np.float32))
    for _ in range(3):
        step()
    graph = torch.cuda.CUDAGraph()
    pair.net.find_winners(sig)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, capture_error_mode="thread_local"):
        got = pair.net.find_winners(sig)
    for t in range(4):
        new = rng.standard_normal((3, m)).astype(np.float32)
        sig.copy_(pair.to_dev(new))
        graph.replay()
        torch.cuda.synchronize()
        assert_find_equal([x.cpu().numpy() for x in got], pair.orc.find_winners(new), f"{t}")
        assert_find_equal(*pair.find(new), f"{t} eager")
        step()
        step()
    pair.compare_state("end")


@pytest.mark.parametrize("lock_mode", [0, 1, 2])
@pytest.mark.parametrize("m", [64, 600])
def test_iterations_recorded_by_the_caller(m, lock_mode):
    """Two iterations in the caller's own graph move the units at each replay, without a call
    that the handle sees: finds and recorded loops in between keep no records of them."""
    import torch
    rng = np.random.default_rng(m)
    n = 4_000
    units = rng.standard_normal((3, n)).astype(np.float32)
    pair = Pair(units, m_max=600, eps_b=0.5, eps_n=0.1, max_age=3, lock_mode=lock_mode)

    def batch():
        return rng.standard_normal((3, m)).astype(np.float32)

    for _ in range(12):   # enough for small batches to take the search
        assert_iter_equal(*pair.iterate(batch()))
    sig = [pair.to_dev(batch()) for _ in range(2)]
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, capture_error_mode="thread_local"):
        for s in sig:
            pair.net.iterate(s)
    for t in range(3):
        new = [batch() for _ in sig]
        for s, b in zip(sig, new):
            s.copy_(pair.to_dev(b))
        graph.replay()
        torch.cuda.synchronize()
        for b in new:
            pair.orc.iterate(b, 0, 0, False)
        assert_find_equal(*pair.find(batch()), f"{t} eager find")
        for k in range(2):
            assert_iter_equal(*pair.iterate(batch()), f"{t} {k}")
        loop = [batch() for _ in sig]
        pair.net.iterate_loop(pair.to_dev(np.stack(loop)))
        for b in loop:
            pair.orc.iterate(b, 0, 0, False)
    pair.compare_state("end")


def prune(pair, rng, m, least=5):
    """Iterations with removal until `least` units are gone: the order keeps their places."""
    n = pair.net.sizes()[0]
    for t in range(20):
        assert_iter_equal(*pair.iterate(rng.standard_normal((3, m)).astype(np.float32), 0, 0, True),
                          f"prune {t}")
        if pair.net.sizes()[0] <= n - least:
            return
    raise AssertionError("no units removed")


@pytest.mark.parametrize("insert", [False, True])
@pytest.mark.parametrize("variant", [2, 3, 4, 5, "split"])
def test_scans_in_a_recorded_loop_after_a_removal(variant, insert):
    """A removal leaves empty places in the unit order, which only the search can read: a
    recorded loop of a scan starts from a new order, also with units appended behind them."""
    from paper_1503_08294_amd import gsn
    rng = np.random.default_rng(70)
    n, m = 3_000, 400
    pair = Pair(rng.standard_normal((3, n)).astype(np.float32), n_max=n + 64, e_max=8 * n, m_max=m,
                eps_b=0.2, eps_n=0.05, max_age=1)
    assert_iter_equal(*pair.iterate(rng.standard_normal((3, m)).astype(np.float32)))
    for call in range(2):
        pair.net.tune(gsn.GSN_TUNE_VARIANT, 0)
        pair.net.tune(gsn.GSN_TUNE_SPLIT, 0)
        prune(pair, rng, m)
        if insert:
            pair.net.grow(1, 1)
            pair.orc.grow(1, 1)
        if variant == "split":
            pair.net.tune(gsn.GSN_TUNE_SPLIT, 3)
        else:
            pair.net.tune(gsn.GSN_TUNE_VARIANT, variant)
        for again in range(2):
            sigs = rng.standard_normal((2, 3, m)).astype(np.float32)
            g = [x.cpu().numpy() for x in pair.net.iterate_loop(pair.to_dev(sigs))]
            for s in sigs:
                o = pair.orc.iterate(s, 0, 0, False)
            assert_iter_equal(g, o, f"loop {call} {again}")
            pair.compare_state(f"loop {call} {again}")
    assert pair.net.check() == 0


def record_find(pair, sig):
    import torch
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, capture_error_mode="thread_local"):
        got = pair.net.find_winners(sig)

    def replay(new):
        sig.copy_(pair.to_dev(new))
        graph.replay()
        torch.cuda.synchronize()
        return [x.cpu().numpy() for x in got]
    return replay


@pytest.mark.parametrize("variant", [0, 2, 3, 4, 5])
@pytest.mark.parametrize("places", ["none", "before", "between"])
def test_recorded_finds_and_changes_of_the_order(variant, places):
    """A recorded find keeps to its own unit order and its own counts: between its replays units
    are removed, others appended up to the same number, and eager finds make new orders of more
    or fewer places, recorded with empty places in the handle's order (before), without (none),
    and with the empty places made and filled between replays; some replays follow each other."""
    from paper_1503_08294_amd import gsn
    rng = np.random.default_rng(80)
    n, m = 3_000, 400
    pair = Pair(rng.standard_normal((3, n)).astype(np.float32), n_max=n + 64, e_max=8 * n, m_max=m,
                eps_b=0.2, eps_n=0.05, max_age=1)
    pair.net.tune(gsn.GSN_TUNE_REBUCKET, 4096)
    pair.net.tune(gsn.GSN_TUNE_VARIANT, variant)

    def batch():
        return rng.standard_normal((3, m)).astype(np.float32)

    def refill(count):
        while pair.net.sizes()[0] < count:
            pair.net.grow(1, 1)
            pair.orc.grow(1, 1)

    assert_iter_equal(*pair.iterate(batch()))
    if places == "before":
        prune(pair, rng, m)
    count = pair.net.sizes()[0]
    replay = record_find(pair, pair.to_dev(batch()))
    for t in range(4):
        if places == "between":
            # removed and appended to the recorded number (the network must hold no more)
            prune(pair, rng, m)
            refill(count)
        assert pair.net.sizes()[0] == count
        for again in range(1 + t):
            new = batch()
            assert_find_equal(replay(new), pair.orc.find_winners(new), f"{t} replay {again}")
        # eager finds: one with the order in place, then one that makes a new order
        assert_find_equal(*pair.find(batch()), f"{t} eager")
        pair.net.tune(gsn.GSN_TUNE_REBUCKET, 1)
        assert_find_equal(*pair.find(batch()), f"{t} eager, new order")
        pair.net.tune(gsn.GSN_TUNE_REBUCKET, 4096)
        new = batch()
        assert_find_equal(replay(new), pair.orc.find_winners(new), f"{t} replay, new order")
        assert_find_equal(*pair.find(batch()), f"{t} eager after it")
        pair.compare_state(f"{t}")
    assert pair.net.check() == 0


@pytest.mark.parametrize("n,holes", [(1_000, False), (1_000, True), (5_000, False), (5_000, True)])
@pytest.mark.parametrize("m", [7, 64, 256, 257, 700])
def test_signals_that_are_not_numbers(n, holes, m):
    """A signal with a NaN: a small batch refuses it (no winner, GSN_E_INVAL from the update) in
    its first call as in the later ones, which take the search; a larger one names the two units
    of lowest index, as the scans do, also with empty places in the unit order.  An infinite
    signal ties all units, so the lowest indices win.  The other signals of the batch are
    unaffected."""
    from paper_1503_08294_amd import gsn
    rng = np.random.default_rng(m)
    pair = Pair(rng.standard_normal((3, n)).astype(np.float32), m_max=700, e_max=8 * n, eps_b=0.2,
                eps_n=0.05, max_age=1 if holes else 50)
    if holes:
        assert_iter_equal(*pair.iterate(rng.standard_normal((3, 300)).astype(np.float32)))
        prune(pair, rng, n // 10, least=2)
    sig = rng.standard_normal((3, m)).astype(np.float32)
    sig[0, 2], sig[2, 4], sig[1, 5] = np.nan, -np.nan, np.inf
    bad = [2, 4]
    want = pair.orc.find_winners(sig)
    if m <= 256:
        for a in want[:2]:
            a[bad] = -1
    for call in range(12):
        g, _ = pair.find(sig)
        for a, b, name in zip(g, want, ("winner", "second", "d1", "d2")):
            np.testing.assert_array_equal(a, b, err_msg=f"call {call} {name}")
    assert pair.net.check() == 0
    if m <= 256:
        # the search's records at hand or not, an iteration refuses them
        sig[1, 5] = 0.5
        for call in range(12):
            acc = pair.net.iterate(pair.to_dev(sig))[4].cpu().numpy()
            assert not acc[bad].any(), call
            assert pair.net.check() == gsn.GSN_E_INVAL, call
        assert np.isfinite(pair.net.export()["xyz"].numpy()).all()


def centre_batch(n, m, hard, seed):
    """Units and signals on a sphere, `hard` of the signals at its centre instead, where every
    unit is about equally far and no box can be left out."""
    rng = np.random.default_rng(seed)
    units = rng.standard_normal((3, n)).astype(np.float32)
    units /= np.linalg.norm(units, axis=0, keepdims=True)
    units[:, n // 2:n // 2 + 40] = units[:, :40]    # ties by index
    sig = rng.standard_normal((3, m)).astype(np.float32)
    sig /= np.linalg.norm(sig, axis=0, keepdims=True)
    at = rng.permutation(m)[:hard]
    sig[:, at] *= np.float32(1e-7)
    sig[:, at[:hard // 8]] = 0.0
    return units, np.ascontiguousarray(sig)


@pytest.mark.parametrize("n,m,hard", [(140_003, 300, 3), (140_003, 300, 300), (131_072, 257, 9),
                                      (3_000, 8_200, 700), (140_003, 8_193, 40), (9_000, 64, 5),
                                      (3_000, 8_192, 300),
                                      (9_000, 256, 256), (70_001, 1, 1)])
def test_hard_signals(n, m, hard):
    """Signals for which the boxes leave out little, alone and among others in their workgroup,
    over more than one round of its list of blocks (131,072 units)."""
    units, sig = centre_batch(n, m, hard, n + m)
    pair = Pair(units, m_max=m)
    want = pair.orc.find_winners(sig)
    dev = pair.to_dev(sig)
    for call in range(12):   # (small batches: the scan, the search, and the scan again)
        g = [x.cpu().numpy() for x in pair.net.find_winners(dev)]
        assert_find_equal(g, want, f"call {call}")


def test_hard_signals_of_small_batches_in_loops():
    """Iterations and recorded loops of small batches go back to the scan after hard signals and
    to the search after a while, with the same results."""
    units = centre_batch(5_000, 1, 1, 90)[0]
    pair = Pair(units, m_max=40, eps_b=0.01, eps_n=0.001)
    for block in range(30):
        hard = 40 if block % 7 == 3 else 0
        sigs = np.stack([centre_batch(100, 40, hard, 100 * block + k)[1] for k in range(5)])
        g = [x.cpu().numpy() for x in pair.net.iterate_loop(pair.to_dev(sigs))]
        for s in sigs:
            o = pair.orc.iterate(s, 0, 0, False)
        assert_iter_equal(g, o, f"block {block}")
        assert_iter_equal(*pair.iterate(sigs[0]), f"block {block} eager")
        pair.compare_state(f"block {block}")
    assert pair.net.check() == 0


def test_time_of_hard_signals():
    """One signal at the centre of a sphere of 200,000 units holds up a batch of 16,384 by less
    than a scan of every pair (0.73 against 1.17 ms; a walk of its boxes one after another
    took 1.45), and small batches of such signals settle within a few times the small scan's time
    (3 times; 45 with the walk), however far the calls run ahead of the reports."""
    import torch
    from paper_1503_08294_amd import gsn

    def time_of(pair, dev, variant, calls):
        pair.net.tune(gsn.GSN_TUNE_VARIANT, variant)
        for _ in range(calls):
            pair.net.find_winners(dev)
        best = []
        for _ in range(3):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(calls):
                pair.net.find_winners(dev)
            b.record()
            torch.cuda.synchronize()
            best.append(a.elapsed_time(b) / calls)
        return min(best)

    units, sig = centre_batch(200_000, 16_384, 1, 7)
    pair = Pair(units, m_max=16_384)
    dev = pair.to_dev(sig)
    assert time_of(pair, dev, 0, 10) < 0.9 * time_of(pair, dev, 4, 10)
    units, sig = centre_batch(100_000, 64, 64, 8)
    pair = Pair(units, m_max=64)
    dev = pair.to_dev(sig)
    assert time_of(pair, dev, 0, 150) < 20 * time_of(pair, dev, 6, 150)


def test_time_and_result_with_many_appended_units():
    """Units inserted since the last order lie anywhere, so every signal visits their leaves: they
    get a new order before they outgrow the signals' lists.  A search after 4,096 insertions at
    once on 100,000 units takes as long as one in a fresh order (12.6 us a call; 90 without)."""
    import torch
    from paper_1503_08294_amd import gsn
    units, sig = centre_batch(100_000, 8_192, 0, 31)
    cloud = torch.from_numpy(np.ascontiguousarray(centre_batch(200_000, 1, 0, 32)[0])).cuda()
    pair = Pair(units, n_max=110_000, m_max=8_192)
    pair.net.tune(gsn.GSN_TUNE_REBUCKET, 4096)   # (no new order by the number of finds)
    dev = pair.to_dev(sig)

    def best_time():
        for _ in range(4):
            got = pair.net.find_winners(dev)
        out = []
        for _ in range(5):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(20):
                pair.net.find_winners(dev)
            b.record()
            torch.cuda.synchronize()
            out.append(a.elapsed_time(b) / 20)
        return min(out), [x.cpu().numpy() for x in got]

    pair.net.iterate(dev)   # (makes the order)
    pair.net.run_schedule(cloud, gsn.make_schedule(m_cap=8_192, fixed_m=8_192, insert_every=2,
                                                   max_signals=8_192))
    assert pair.net.sizes()[0] > 103_000
    appended, found = best_time()
    s = pair.net.export()
    pair.orc.import_state(*(s[k].numpy() for k in ("xyz", "err", "edges")))
    assert_find_equal(found, pair.orc.find_winners(sig), "after the insertions")
    pair.net.import_state(s["xyz"], s["err"], s["edges"])
    fresh, found = best_time()
    assert_find_equal(found, pair.orc.find_winners(sig), "after an import")
    assert appended < 2 * fresh, (appended, fresh)


@pytest.mark.parametrize("variant", [0, 4])
def test_recordings_of_several_iterations_and_finds(variant):
    """The finds of one recording share the order that its first find makes (and make another
    after GSN_TUNE_REBUCKET of them), each recording its own: two graphs recorded one after the
    other on the same stream, of six iterations and of three finds, replayed several times in a
    row and in turn, with eager calls between."""
    import torch
    from paper_1503_08294_amd import gsn
    rng = np.random.default_rng(50)
    n, m = 4_000, 500
    pair = Pair(rng.standard_normal((3, n)).astype(np.float32), n_max=n + 64, m_max=m, eps_b=0.4,
                eps_n=0.1, max_age=30)
    pair.net.tune(gsn.GSN_TUNE_VARIANT, variant)
    pair.net.tune(gsn.GSN_TUNE_REBUCKET, 4)

    def batch():
        return rng.standard_normal((3, m)).astype(np.float32)

    for _ in range(2):
        assert_iter_equal(*pair.iterate(batch()))
    runs = [pair.to_dev(batch()) for _ in range(6)]
    finds = [pair.to_dev(batch()) for _ in range(3)]
    outs = [tuple(torch.empty_like(x[:m]) for x in (pair.net.buf.winner, pair.net.buf.second,
                                                    pair.net.buf.d1, pair.net.buf.d2))
            for _ in finds]
    torch.cuda.synchronize()
    graphs = [torch.cuda.CUDAGraph() for _ in range(2)]
    with torch.cuda.graph(graphs[0], capture_error_mode="thread_local"):
        for s in runs:
            pair.net.iterate(s)
    with torch.cuda.graph(graphs[1], capture_error_mode="thread_local"):
        for s, out in zip(finds, outs):
            for a, b in zip(out, pair.net.find_winners(s)):
                a.copy_(b)

    def run():
        new = [batch() for _ in runs]
        for s, b in zip(runs, new):
            s.copy_(pair.to_dev(b))
        graphs[0].replay()
        torch.cuda.synchronize()
        for b in new:
            pair.orc.iterate(b, 0, 0, False)

    def find(where):
        new = [batch() for _ in finds]
        for s, b in zip(finds, new):
            s.copy_(pair.to_dev(b))
        graphs[1].replay()
        torch.cuda.synchronize()
        for k, (b, out) in enumerate(zip(new, outs)):
            assert_find_equal([x.cpu().numpy() for x in out], pair.orc.find_winners(b),
                              f"{where} find {k}")

    find("alone")   # (nothing of the other recording has run)
    for t in range(3):
        for again in range(t + 1):
            run()
        find(f"{t} first")
        assert_find_equal(*pair.find(batch()), f"{t} eager find")
        for k in range(2):
            assert_iter_equal(*pair.iterate(batch()), f"{t} eager {k}")
        for again in range(2):
            find(f"{t} again {again}")
        pair.compare_state(f"{t}")
    assert pair.net.check() == 0
