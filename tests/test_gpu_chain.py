"""Counting by chains over per-type lists (the default of fe_count and
fe_count_two_pass) where it can go wrong, against the CPU oracle, bit for bit:
entries with more following events than a batch holds, crowded buckets, ties
in the ticks, list lengths around a batch and a read of four, segments whose
first chains start before an earlier segment's last completion, types up to
the lists' limit and beyond it, and ticks at the ends of their range."""
import numpy as np
import pytest

import oracle
from paper_0905_2200_amd import synth
from tests.gpu_util import banner, have_gpu, oracle_counts

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not have_gpu(), reason="needs a GPU")]

EXACT, RELAXED = 0, 1
IVS = [(0, 50), (50, 100), (100, 200), (190, 200), (0, 1), (7, 9)]


@pytest.fixture(scope="module")
def fe():
    from paper_0905_2200_amd import fe as fe_mod
    return fe_mod


@pytest.fixture(scope="module")
def ctx(fe):
    c = fe.Context(0)
    yield c
    c.close()


def _check(ctx, ids_h, ticks_h, T, cand, what):
    ids, ticks = ctx.stream_tensors(ids_h, ticks_h)
    cd = ctx.cand_tensors(cand)
    seen = 0
    for mode in (EXACT, RELAXED):
        want = oracle_counts(ids_h, ticks_h, T, cand, mode)
        got = ctx.count(ids, ticks, T, cd, mode).cpu().numpy()
        bad = np.nonzero(got != want)[0]
        assert bad.size == 0, (what, mode, bad[:5], got[bad[:5]], want[bad[:5]])
        seen = max(seen, int(want.max()) if want.size else 0)
    for theta in (1, max(1, seen // 4)):
        up, ex, ns = ctx.count_two_pass(ids, ticks, T, cd, theta)
        wu, we = oracle.two_pass(ids_h, ticks_h, T, cand["types"], cand["len"], cand["lo"],
                                 cand["hi"], theta, projection=True)
        assert np.array_equal(up.cpu().numpy(), wu), (what, theta)
        assert np.array_equal(ex.cpu().numpy(), we), (what, theta)
        assert int(ns.item()) == int((wu >= theta).sum()), (what, theta)
    return seen


def _all_sizes(rng, T, M, ivs=IVS):
    return synth.pack(synth.random_episodes(rng, M, T, 8, ivs, n_min=1))


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 63, 64, 65, 66, 127, 128, 129, 191, 513, 4099])
def test_short_lists(ctx, n):
    # one and two types: lists of n and about n/2 events
    rng = np.random.default_rng(n)
    for T in (1, 2, 3):
        ids_h = rng.integers(0, T, n).astype(np.int32)
        ticks_h = np.cumsum(rng.integers(0, 30, n)).astype(np.int32)
        banner("short lists: n=%d T=%d" % (n, T))
        _check(ctx, ids_h, ticks_h, T, _all_sizes(rng, T, 200), "n=%d T=%d" % (n, T))


@pytest.mark.parametrize("gap", [0, 1, 2, 5])
def test_more_followers_than_a_batch(ctx, gap):
    # type 1 fires in runs far longer than a batch within one interval of a
    # lone type 0 event; at gap 0 the whole run shares its tick (one bucket)
    rng = np.random.default_rng(50 + gap)
    ids, ticks, t = [], [], 0
    for run in (1, 3, 4, 5, 63, 64, 65, 127, 128, 129, 200, 333):
        for first in (0, 2):
            ids += [first] + [1] * run + [2]
            ticks += [t] + list(t + 1 + gap * np.arange(run)) + [t + 2 + gap * run]
            t = ticks[-1] + int(rng.integers(0, 40))
    ids_h, ticks_h = np.array(ids, np.int32), np.array(ticks, np.int32)
    eps = [((a, b, c)[:n], (lo, lo2)[:n - 1], (hi, hi2)[:n - 1]) for n in (2, 3)
           for a in range(3) for b in range(3) for c in range(3)
           for lo, hi in ((0, 40), (0, 3000), (10, 500)) for lo2, hi2 in ((0, 2000), (3, 70))]
    banner("more followers than a batch: gap %d" % gap)
    assert _check(ctx, ids_h, ticks_h, 3, synth.pack(eps), "gap=%d" % gap) > 3


@pytest.mark.parametrize("T,mean_gap", [(2, 1), (3, 4), (5, 20), (16, 3)])
def test_dense_segments(ctx, fe, T, mean_gap):
    # a completion every few events: at most segment boundaries a chain is open
    rng = np.random.default_rng(70 + T)
    n = 40_000
    ids_h = rng.integers(0, T, n).astype(np.int32)
    ticks_h = np.cumsum(rng.integers(0, 2 * mean_gap + 1, n)).astype(np.int32)
    cand = synth.pack(synth.random_episodes(rng, 300, T, 5, IVS, n_min=1))
    banner("dense segments: T=%d gap=%d" % (T, mean_gap))
    _check(ctx, ids_h, ticks_h, T, cand, "T=%d" % T)
    assert ctx.stats()["segments_max"] >= 2
    # the whole-stream form of the same counts
    ids, ticks = ctx.stream_tensors(ids_h, ticks_h)
    keys = (fe.PARAM_CROSSOVER_A, fe.PARAM_CROSSOVER_B, fe.PARAM_CROSSOVER_A_RELAXED,
            fe.PARAM_CROSSOVER_B_RELAXED)
    saved = [ctx.get_param(p) for p in keys]
    cut = [ctx.count(ids, ticks, T, cand, m).cpu().numpy() for m in (EXACT, RELAXED)]
    try:
        for p in keys:
            ctx.set_param(p, 0)
        for m in (EXACT, RELAXED):
            assert np.array_equal(ctx.count(ids, ticks, T, cand, m).cpu().numpy(), cut[m])
            assert ctx.stats()["segments_max"] == 1
    finally:
        for p, v in zip(keys, saved):
            ctx.set_param(p, v)


@pytest.mark.parametrize("ratio", [0.1, 0.95, 1.05, 7.0, 30.0, 34.0])
@pytest.mark.parametrize("gap", [0, 1, 9])
def test_either_list_first(ctx, ratio, gap):
    # the second nodes' lists are `ratio` times the first nodes' length: walked
    # from the shorter side on, up to the lines between, with ties (gap 0, 1)
    rng = np.random.default_rng(int(10 * ratio) + gap)
    n = 12_000
    first = rng.random(n) < 1.0 / (1.0 + ratio)
    ids_h = (rng.integers(0, 2, n) + np.where(first, 0, 2)).astype(np.int32)
    ticks_h = np.cumsum(rng.integers(0, 2 * gap + 1, n) * (rng.random(n) < 0.7)).astype(np.int32)
    ivs = [(0, 1), (0, 6), (2, 40), (30, 33), (0, 500)]
    eps = []
    for _ in range(300):
        k = int(rng.integers(2, 6))
        ty = (int(rng.integers(0, 2)),) + tuple(int(x) for x in rng.integers(2, 4, k - 1))
        iv = [ivs[int(x)] for x in rng.integers(0, len(ivs), k - 1)]
        eps.append((ty, tuple(l for l, _ in iv), tuple(h for _, h in iv)))
    for nmax in (2, 3, 5):  # (tables of two, three and more nodes)
        cand = synth.pack([e for e in eps if len(e[0]) <= nmax])
        banner("lists 1:%g gap %d nmax %d" % (ratio, gap, nmax))
        _check(ctx, ids_h, ticks_h, 4, cand, "ratio=%g gap=%d nmax=%d" % (ratio, gap, nmax))


@pytest.mark.parametrize("nmax", [3, 5])
@pytest.mark.parametrize("M", [6800, 14001, 70001, 140007])
def test_survivors_in_segments(ctx, fe, M, nmax):
    # the exact pass over the segments of survivors alone, looked for among 1
    # to 16 rows a wave; tables of three and of five nodes, from too few waves
    # to fill the device on
    rng = np.random.default_rng(M)
    n = 20_000
    ids_h = rng.integers(0, 2, n).astype(np.int32)
    ticks_h = np.cumsum(rng.integers(0, 9, n)).astype(np.int32)
    eps = synth.random_episodes(rng, 211, 2, nmax, IVS, n_min=1)
    cand = synth.pack(eps)
    many = synth.pack([eps[i % len(eps)] for i in range(M)])
    up = oracle_counts(ids_h, ticks_h, 2, cand, RELAXED)
    ids, ticks = ctx.stream_tensors(ids_h, ticks_h)
    keys = (fe.PARAM_CROSSOVER_B, fe.PARAM_CROSSOVER_B_RELAXED, fe.PARAM_TARGET_WAVES)
    saved = [ctx.get_param(p) for p in keys]
    try:
        for p in keys:
            ctx.set_param(p, 1 << 22)
        for theta in (1, int(np.median(up)), int(up.max()) + 1):
            banner("survivors in segments: M=%d theta=%d" % (M, theta))
            wu, we = oracle.two_pass(ids_h, ticks_h, 2, cand["types"], cand["len"], cand["lo"],
                                     cand["hi"], theta, projection=True)
            gu, ge, ns = ctx.count_two_pass(ids, ticks, 2, many, theta)
            at = np.arange(M) % len(eps)
            assert np.array_equal(gu.cpu().numpy(), wu[at])
            assert np.array_equal(ge.cpu().numpy(), we[at])
            assert int(ns.item()) == int((wu[at] >= theta).sum())
            assert ctx.stats()["segments_max"] >= 2
    finally:
        for p, v in zip(keys, saved):
            ctx.set_param(p, v)


@pytest.mark.parametrize("T", [1000, 1025, 4096, 4097, 9000])
def test_many_types(ctx, T):
    # (beyond 4096 types the Map kernels count)
    rng = np.random.default_rng(T)
    n = 20_000
    hot = rng.choice(T, 40, replace=False)
    ids_h = np.where(rng.random(n) < 0.8, rng.choice(hot, n), rng.integers(0, T, n)).astype(np.int32)
    ticks_h = np.cumsum(rng.integers(0, 8, n)).astype(np.int32)
    eps = synth.random_episodes(rng, 300, 40, 4, IVS, n_min=1)
    eps = [(tuple(int(hot[e]) for e in ty), lo, hi) for ty, lo, hi in eps]
    eps += synth.random_episodes(rng, 100, T, 3, IVS, n_min=1)
    eps += [((T - 1,), (), ()), ((T - 1, 0), (0,), (90,))]
    banner("many types: T=%d" % T)
    _check(ctx, ids_h, ticks_h, T, synth.pack(eps), "T=%d" % T)


def test_tick_range_ends(ctx):
    # all events at either end of the tick range, and the widest hops
    top = (1 << 30) - 1
    rng = np.random.default_rng(9)
    t = np.concatenate([np.sort(rng.integers(0, 300, 500)),
                        np.sort(top - rng.integers(0, 300, 500)), [top] * 20])
    ids_h = rng.integers(0, 4, t.size).astype(np.int32)
    eps = synth.random_episodes(rng, 300, 4, 4, IVS, n_min=1)
    eps += [((a, b), (lo,), (hi,)) for a in range(4) for b in range(4)
            for lo, hi in ((0, top), (top - 300, top), (top - 1, top), (0, top - 299))]
    banner("tick range ends")
    _check(ctx, ids_h, t.astype(np.int32), 4, synth.pack(eps), "range ends")


@pytest.mark.parametrize("seed", range(8))
def test_random_streams(ctx, seed):
    # uneven rates, bursts and ties, every size and interval
    rng = np.random.default_rng(3000 + seed)
    T = int(rng.integers(2, 40))
    n = int(rng.integers(3_000, 30_000))
    w = rng.lognormal(0.0, 1.5, T)
    ids_h = rng.choice(T, n, p=w / w.sum()).astype(np.int32)
    gaps = rng.integers(0, int(rng.integers(2, 60)), n)
    gaps[rng.random(n) < 0.3 * (seed % 3)] = 0
    ticks_h = np.cumsum(gaps).astype(np.int32)
    banner("random streams: seed=%d T=%d n=%d" % (seed, T, n))
    _check(ctx, ids_h, ticks_h, T, _all_sizes(rng, T, 700), "seed=%d" % seed)


@pytest.mark.parametrize("mode", [EXACT, RELAXED])
def test_errors_write_nothing(ctx, fe, mode):
    ids, ticks = ctx.stream_tensors([0, 1, 0, 1], [0, 5, 3, 9])
    ok = ctx.stream_tensors([0, 1, 0, 1], [0, 5, 6, 9])
    out = ctx.torch.full((1,), -7, dtype=ctx.torch.int32, device=ctx.device)
    good = synth.pack([((0, 1), (0,), (10,))])
    for stream, cand, code in (((ids, ticks), good, fe.FE_EUNSORTED),
                               (ok, synth.pack([((0, 2), (0,), (10,))]), fe.FE_EINVAL),
                               ((ids + 5, ok[1]), good, fe.FE_ERANGE)):
        with pytest.raises(fe.FeError) as e:
            ctx.count(stream[0], stream[1], 2, cand, mode, out=out)
        assert e.value.code == code
        ctx.torch.cuda.synchronize()
        assert out.item() == -7
    assert ctx.count(ok[0], ok[1], 2, good, mode).item() == 2


def test_batch_of_uneven_jobs(ctx, fe):
    # recordings without events, tables without rows, one candidate, every
    # table width, and more candidates than one launch row of waves
    rng = np.random.default_rng(17)
    recs = []
    for n, T, M, nmax in ((0, 5, 40, 3), (1, 1, 1, 1), (5_000, 90, 900, 8), (20_000, 3, 300, 2),
                          (700, 64, 0, 4), (0, 2, 3, 1), (12_345, 16, 2_000, 5)):
        ids_h = rng.integers(0, T, n).astype(np.int32)
        ticks_h = np.cumsum(rng.integers(0, 12, n)).astype(np.int32)
        eps = synth.random_episodes(rng, M, T, nmax, IVS, n_min=1)
        recs.append((ids_h, ticks_h, T, synth.pack(eps, nmax=nmax), 2 if n else 1))
    dev = [{"ids": a, "ticks": b, "num_types": T, "cand": ctx.cand_tensors(c), "theta": th}
           for (i, t, T, c, th) in recs for a, b in [ctx.stream_tensors(i, t)]]
    banner("batch of uneven jobs")
    b = fe.Batch(ctx, dev)
    for _ in range(2):
        b.run()
        ctx.sync()
        for r, (i, t, T, c, th) in enumerate(recs):
            if c["M"] == 0:
                continue
            wu, we = oracle.two_pass(i, t, T, c["types"], c["len"], c["lo"], c["hi"], th,
                                     projection=True)
            assert np.array_equal(b.upper[r].cpu().numpy(), wu), r
            assert np.array_equal(b.exact[r].cpu().numpy(), we), r
    b.close()


@pytest.mark.parametrize("mode", [EXACT, RELAXED])
def test_resume_at_ties(ctx, mode):
    # every cut inside a run of equal ticks, and increments shorter than the
    # episodes' width
    rng = np.random.default_rng(23)
    T, n = 4, 3_000
    ids_h = rng.integers(0, T, n).astype(np.int32)
    ticks_h = np.cumsum(rng.integers(0, 2, n) * rng.integers(0, 25, n)).astype(np.int32)
    cand = _all_sizes(rng, T, 300)
    cd = ctx.cand_tensors(cand)
    t = ctx.torch
    cnt = t.zeros(cand["M"], dtype=t.int32, device=ctx.device)
    last = t.full((cand["M"],), -1, dtype=t.int32, device=ctx.device)
    ids, ticks = ctx.stream_tensors(ids_h, ticks_h)
    prev = 0
    banner("resume at ties")
    for cut in (1, 2, 5, 64, 65, 200, 201, 202, 900, 1500, 1510, 1511, n):
        ctx.count_resume(ids[:cut], ticks[:cut], T, cd, mode, prev, cnt, last)
        want = oracle_counts(ids_h[:cut], ticks_h[:cut], T, cand, mode)
        assert np.array_equal(cnt.cpu().numpy(), want), cut
        prev = cut


def test_served_arrays_of_different_types(ctx, fe):
    # candidates of types that an array does not have, empty windows, and
    # windows whose index passes the budget (counted event by event)
    rng = np.random.default_rng(29)
    sizes = [(3, 8_000), (40, 9_000), (40, 0)]
    arrays = [(rng.integers(0, T, n).astype(np.int32),
               np.cumsum(rng.integers(0, 9, n)).astype(np.int32)) for T, n in sizes]
    cand = synth.pack(synth.random_episodes(rng, 400, 40, 6, IVS, n_min=1))
    for budget in (1 << 30, 400 << 10):
        sv = fe.Server(ctx, cand, [T for T, _ in sizes], capacity=9_016, hbm_budget=budget,
                       max_inflight=2, max_round=5)
        for a, (i, t) in enumerate(arrays):
            sv.append(a, i, t)
        reqs = []
        for k in range(14):
            a = k % 3
            t0 = int(rng.integers(0, 30_000))
            t1 = t0 if k == 3 else t0 + int(rng.integers(1, 30_000))
            reqs.append((a, t0, t1, 1 + k % 4, sv.submit(a, t0, t1, 1 + k % 4)))
        banner("served, budget %d" % budget)
        for a, t0, t1, theta, tkt in reqs:
            res = sv.wait(tkt)
            i, t = arrays[a]
            x, y = np.searchsorted(t, t0, "left"), np.searchsorted(t, t1, "left")
            wu, we = oracle.two_pass(i[x:y], t[x:y], 40, cand["types"], cand["len"], cand["lo"],
                                     cand["hi"], theta, projection=True)
            assert res["status"] == fe.FE_OK and res["n_events"] == y - x
            assert np.array_equal(res["upper"], wu) and np.array_equal(res["exact"], we), (a, t0, t1)
        sv.close()


def test_batch_over_a_changed_recording(ctx, fe):
    # a run over events that have become invalid leaves no old counts, and
    # nothing behind for other calls of the context
    rng = np.random.default_rng(31)
    recs, host = [], []
    for n, T in ((4_000, 6), (900, 3)):
        ids_h = rng.integers(0, T, n).astype(np.int32)
        ticks_h = np.cumsum(rng.integers(0, 12, n)).astype(np.int32)
        cand = synth.pack(synth.random_episodes(rng, 150, T, 4, IVS, n_min=1))
        ids, ticks = ctx.stream_tensors(ids_h, ticks_h)
        host.append((ids_h, ticks_h, T, cand))
        recs.append({"ids": ids, "ticks": ticks, "num_types": T,
                     "cand": ctx.cand_tensors(cand), "theta": 2})
    b = fe.Batch(ctx, recs)

    def right():
        for r, (i, t, T, c) in enumerate(host):
            wu, we = oracle.two_pass(i, t, T, c["types"], c["len"], c["lo"], c["hi"], 2,
                                     projection=True)
            assert np.array_equal(b.upper[r].cpu().numpy(), wu), r
            assert np.array_equal(b.exact[r].cpu().numpy(), we), r
    banner("batch over a changed recording")
    b.run()
    ctx.sync()
    right()
    for k, at, v in (("ids", 7, 6), ("ids", 3_999, -1), ("ticks", 5, 1 << 30), ("ticks", 3_000, 0)):
        keep = int(recs[0][k][at].item())
        recs[0][k][at] = v
        ctx.torch.cuda.synchronize()
        b.run()
        ctx.sync()
        for r in range(2):
            assert (b.upper[r] == -1).all().item() and (b.exact[r] == -1).all().item(), (k, r)
        i, t, T, c = host[1]
        got = ctx.count(recs[1]["ids"], recs[1]["ticks"], T, recs[1]["cand"], EXACT)
        assert np.array_equal(got.cpu().numpy(), oracle_counts(i, t, T, c, EXACT)), k
        recs[0][k][at] = keep
        ctx.torch.cuda.synchronize()
        b.run()
        ctx.sync()
        right()
    b.close()


@pytest.mark.parametrize("rows", [1, 20_000])
def test_two_pass_errors_write_nothing(ctx, fe, rows):
    # (the survivors of small and of large tables are counted by one and by many blocks)
    t = ctx.torch
    ok = ctx.stream_tensors([0, 1, 0, 1], [0, 5, 6, 9])
    bad = ctx.stream_tensors([0, 1, 0, 1], [0, 5, 3, 9])
    good = ctx.cand_tensors(synth.pack([((0, 1), (0,), (10,))] * rows))
    wrong = ctx.cand_tensors(synth.pack([((0, 1), (0,), (10,))] * (rows - 1) +
                                        [((0, 2), (0,), (10,))]))
    up, ex = (t.full((rows,), -7, dtype=t.int32, device=ctx.device) for _ in range(2))
    ns = t.full((1,), -7, dtype=t.int32, device=ctx.device)
    for stream, cand, code in ((bad, good, fe.FE_EUNSORTED), (ok, wrong, fe.FE_EINVAL)):
        with pytest.raises(fe.FeError) as e:
            ctx.count_two_pass(stream[0], stream[1], 2, cand, 1, up, ex, ns)
        assert e.value.code == code
        t.cuda.synchronize()
        assert (up == -7).all().item() and (ex == -7).all().item() and ns.item() == -7
    ctx.count_two_pass(ok[0], ok[1], 2, good, 1, up, ex, ns)
    t.cuda.synchronize()
    assert (up == 2).all().item() and (ex == 2).all().item() and ns.item() == rows


def test_nearly_2_to_31_rows(ctx, fe):
    # one-node rows, type 1 first and last: places past 2^31 - 2^18
    t = ctx.torch
    M = (1 << 31) - 300
    if t.cuda.mem_get_info()[0] < 48 << 30:
        pytest.skip("needs 34 GB of device memory")
    ids, ticks = ctx.stream_tensors([0, 1, 0], [0, 5, 6])
    types = t.zeros((M, 1), dtype=t.int32, device=ctx.device)
    types[0] = types[-1] = 1
    one = t.ones(M, dtype=t.int32, device=ctx.device)
    hop = t.zeros((1, 1), dtype=t.int32, device=ctx.device)
    cand = {"types": types, "len": one, "lo": hop, "hi": hop, "nmax": 1, "M": M}
    banner("%d rows" % M)
    up, ex, ns = ctx.count_two_pass(ids, ticks, 2, cand, 2)
    assert ns.item() == M - 2
    for v, drop in ((up, 1), (ex, -1)):
        assert v[0].item() == drop and v[-1].item() == drop
        assert v[1].item() == 2 and v[M // 2].item() == 2 and v[-2].item() == 2
    del up, ex, types, one, cand
    t.cuda.empty_cache()


def test_batch_of_2_to_24_lists(ctx, fe):
    # 4200 recordings of 4096 types: more lists than a grid's dimension has blocks of 256
    rng = np.random.default_rng(37)
    T, n, R = 4096, 300, 4200
    ids_h = rng.integers(T - 5, T, n).astype(np.int32)
    ticks_h = np.cumsum(rng.integers(0, 12, n)).astype(np.int32)
    cand = synth.pack([((T - 1 - a, T - 1 - b), (0,), (40,)) for a in range(5) for b in range(5)])
    ids, ticks = ctx.stream_tensors(ids_h, ticks_h)
    cd = ctx.cand_tensors(cand)
    wu, we = oracle.two_pass(ids_h, ticks_h, T, cand["types"], cand["len"], cand["lo"],
                             cand["hi"], 3, projection=True)
    banner("batch of %d lists" % (R * T))
    b = fe.Batch(ctx, [{"ids": ids, "ticks": ticks, "num_types": T, "cand": cd, "theta": 3}] * R)
    b.run()
    ctx.sync()
    for r in (0, 1, R // 2, R - 105, R - 104, R - 1):
        assert np.array_equal(b.upper[r].cpu().numpy(), wu), r
        assert np.array_equal(b.exact[r].cpu().numpy(), we), r
    t = ctx.torch
    assert (t.stack(b.upper) == t.stack(b.upper)[0]).all().item()
    assert (t.stack(b.exact) == t.stack(b.exact)[0]).all().item()
    b.close()


def test_segments_whatever_the_rows(ctx, fe):
    # tables beyond the event-by-event kernels' whole-stream line keep their segments
    rng = np.random.default_rng(43)
    T, n, M, N = 64, 1_000_000, 1_050_000, 3
    ids_h = rng.integers(0, T, n).astype(np.int32)
    ticks_h = np.sort(rng.integers(0, 8 * n, n)).astype(np.int32)
    iv = rng.integers(0, len(IVS), (M, N - 1))
    lo, hi = np.array(IVS, np.int32).T
    cand = {"types": rng.integers(0, T, (M, N)).astype(np.int32), "len": np.full(M, N, np.int32),
            "lo": lo[iv], "hi": hi[iv]}
    some = rng.choice(M, 40, replace=False)
    few = dict({k: v[some] for k, v in cand.items()}, M=40, nmax=N)
    ids, ticks = ctx.stream_tensors(ids_h, ticks_h)
    cd = ctx.cand_tensors(cand)
    banner("segments of %d rows" % M)
    for mode in (EXACT, RELAXED):
        got = ctx.count(ids, ticks, T, cd, mode).cpu().numpy()
        assert ctx.stats()["segments_max"] >= 2, mode
        assert np.array_equal(got[some], oracle_counts(ids_h, ticks_h, T, few, mode)), mode


@pytest.mark.parametrize("T,n", [(4096, 300_000), (1000, 1_000_000), (600, 250_000), (600, 200_000)])
def test_long_streams_of_many_types_in_a_batch(ctx, fe, T, n):
    # (the last two on both sides of chunks of 4096 events)
    rng = np.random.default_rng(T)
    recs, want = [], []
    for k in range(2):
        ids_h = rng.integers(0, T, n + k).astype(np.int32)
        ticks_h = np.sort(rng.integers(0, n, n + k)).astype(np.int32)
        cand = synth.pack(synth.random_episodes(rng, 60, T, 3, [(0, 50), (50, 2000)], n_min=1))
        ids, ticks = ctx.stream_tensors(ids_h, ticks_h)
        recs.append({"ids": ids, "ticks": ticks, "num_types": T, "cand": ctx.cand_tensors(cand),
                     "theta": 3})
        want.append(oracle.two_pass(ids_h, ticks_h, T, cand["types"], cand["len"], cand["lo"],
                                    cand["hi"], 3, projection=True))
    banner("long streams of %d types in a batch" % T)
    b = fe.Batch(ctx, recs)
    b.run()
    ctx.sync()
    for r, (wu, we) in enumerate(want):
        assert np.array_equal(b.upper[r].cpu().numpy(), wu)
        assert np.array_equal(b.exact[r].cpu().numpy(), we)
    b.close()


def test_many_types_cost_in_a_batch(ctx, fe):
    # a batch of one takes no longer than twice the same call alone
    import time
    rng = np.random.default_rng(2)
    T, n = 4096, 1_000_000
    ids, ticks = ctx.stream_tensors(rng.integers(0, T, n).astype(np.int32),
                                    np.sort(rng.integers(0, n, n)).astype(np.int32))
    cand = ctx.cand_tensors(synth.pack(synth.random_episodes(rng, 64, T, 2, [(0, 50)], n_min=2)))
    b = fe.Batch(ctx, [{"ids": ids, "ticks": ticks, "num_types": T, "cand": cand, "theta": 5}])

    def best(call):
        t = []
        for _ in range(6):
            ctx.torch.cuda.synchronize()
            a = time.perf_counter()
            call()
            ctx.torch.cuda.synchronize()
            t.append(time.perf_counter() - a)
        return min(t)
    lone = best(lambda: ctx.count_two_pass(ids, ticks, T, cand, 5))
    both = best(b.run)
    banner("4096 types: alone %.0f us, batch %.0f us" % (lone * 1e6, both * 1e6))
    b.close()
    assert both < 2 * lone


@pytest.mark.parametrize("n", [32_767, 32_768])
@pytest.mark.parametrize("T", [1, 2, 3])
@pytest.mark.parametrize("rows", [16, 1023])
def test_relaxed_few_rows_over_dense_few_types(ctx, fe, n, T, rows):
    # few rows with long dense windows: one or two types are counted event by event
    # from a stream length on, three stay with the lists
    rng = np.random.default_rng(100 * T + rows)
    eps = synth.random_episodes(rng, 16, T, 6, [(0, 150), (30, 180)])
    cand = synth.pack(eps)
    many = synth.pack([eps[i % len(eps)] for i in range(rows)])
    ids_h = rng.integers(0, T, n).astype(np.int32)
    ticks_h = np.sort(rng.integers(0, n // T, n)).astype(np.int32)  # one of a type a tick
    ids, ticks = ctx.stream_tensors(ids_h, ticks_h)
    banner("few rows over few dense types: n=%d T=%d rows=%d" % (n, T, rows))
    ctx.set_param(fe.PARAM_TIMING, 1)
    try:
        ctx.reset_kernel_stats()
        got = ctx.count(ids, ticks, T, many, RELAXED).cpu().numpy()
        lists = "map_relaxed_chain" in ctx.kernel_stats()
    finally:
        ctx.set_param(fe.PARAM_TIMING, 0)
    want = oracle_counts(ids_h, ticks_h, T, cand, RELAXED)
    assert np.array_equal(got, want[np.arange(rows) % len(eps)])
    assert lists == (n < 32_768 or T == 3)


@pytest.mark.parametrize("T", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("rows", [1023, 1024, 8191, 8192])
def test_relaxed_rows_over_few_types(ctx, fe, T, rows):
    # sparse, dense and denser streams of few types on both sides of the rows' line
    # from which some are counted event by event
    rng = np.random.default_rng(10 * T + rows)
    n, seen = 17_000, set()
    eps = synth.random_episodes(rng, 60, T, 6, [(0, 150), (30, 180), (0, 90)], n_min=2)
    cand = synth.pack(eps)
    many = synth.pack([eps[i % len(eps)] for i in range(rows)])
    at = np.arange(rows) % len(eps)
    ctx.set_param(fe.PARAM_TIMING, 1)
    try:
        for gap in (200, 12, 1):  # mean ticks between events, times T
            ids_h = rng.integers(0, T, n).astype(np.int32)
            ticks_h = np.sort(rng.integers(0, max(1, gap * n // T), n)).astype(np.int32)
            ids, ticks = ctx.stream_tensors(ids_h, ticks_h)
            banner("relaxed rows over few types: T=%d rows=%d gap=%d" % (T, rows, gap))
            ctx.reset_kernel_stats()
            got = ctx.count(ids, ticks, T, many, RELAXED).cpu().numpy()
            assert np.array_equal(got, oracle_counts(ids_h, ticks_h, T, cand, RELAXED)[at]), gap
            seen.add("map_relaxed_chain" in ctx.kernel_stats())
    finally:
        ctx.set_param(fe.PARAM_TIMING, 0)
    if T == 5 or rows < 1024:
        assert seen == {True}
    if rows == 8192 and T <= 4:
        assert False in seen
    bad = dict(many, hi=many["lo"])
    with pytest.raises(fe.FeError) as e:
        ctx.count(ids, ticks, T, bad, RELAXED)
    assert e.value.code == fe.FE_EINVAL
    with pytest.raises(fe.FeError) as e:
        ctx.count(ids, ticks.flip(0), T, many, RELAXED)
    assert e.value.code == fe.FE_EUNSORTED
    assert np.array_equal(ctx.count(ids, ticks, T, many, RELAXED).cpu().numpy(), got)


@pytest.mark.parametrize("T,gap", [(1, 3), (2, 300), (3, 3), (4, 2), (4, 40)])
@pytest.mark.parametrize("rows", [1500, 9000])
def test_two_passes_over_few_types(ctx, T, gap, rows):
    # the relaxed pass of either kind, then the survivors: all, some and none
    rng = np.random.default_rng(100 * T + gap + rows)
    n = 17_000
    eps = synth.random_episodes(rng, 60, T, 6, [(0, 150), (30, 180), (0, 90)], n_min=2)
    cand = synth.pack(eps)
    many = synth.pack([eps[i % len(eps)] for i in range(rows)])
    at = np.arange(rows) % len(eps)
    ids_h = rng.integers(0, T, n).astype(np.int32)
    ticks_h = np.sort(rng.integers(0, gap * n // T, n)).astype(np.int32)
    ids, ticks = ctx.stream_tensors(ids_h, ticks_h)
    up = oracle_counts(ids_h, ticks_h, T, cand, RELAXED)
    for theta in (0, 1, int(np.median(up)), int(up.max()) + 1):
        banner("two passes over few types: T=%d gap=%d rows=%d theta=%d" % (T, gap, rows, theta))
        wu, we = oracle.two_pass(ids_h, ticks_h, T, cand["types"], cand["len"], cand["lo"],
                                 cand["hi"], theta, projection=True)
        gu, ge, ns = ctx.count_two_pass(ids, ticks, T, many, theta)
        assert np.array_equal(gu.cpu().numpy(), wu[at])
        assert np.array_equal(ge.cpu().numpy(), we[at])
        assert int(ns.item()) == int((wu[at] >= theta).sum())


@pytest.mark.parametrize("T,n,hot", [(300, 60_000, 1), (2000, 40_000, 2), (4096, 20_000, 1), (7, 33_000, 1)])
def test_types_of_most_events(ctx, fe, T, n, hot):
    # lists far longer than the average, whose tables several blocks fill
    rng = np.random.default_rng(T + n)
    ids_h = np.where(rng.random(n) < 0.95, rng.integers(T - hot, T, n),
                     rng.integers(0, T, n)).astype(np.int32)
    ticks_h = np.sort(rng.integers(0, 20 * n, n)).astype(np.int32)
    eps = synth.random_episodes(rng, 150, T, 4, IVS, n_min=1)
    eps += [((T - 1,) * k, (0,) * (k - 1), (30,) * (k - 1)) for k in (1, 2, 3, 4)]
    eps += [((T - 1, int(e), T - 1), (0, 5), (300, 400)) for e in rng.integers(0, T, 60)]
    cand = synth.pack(eps)
    banner("types of most events: T=%d" % T)
    _check(ctx, ids_h, ticks_h, T, cand, "T=%d" % T)
    ids, ticks = ctx.stream_tensors(ids_h, ticks_h)
    wu, we = oracle.two_pass(ids_h, ticks_h, T, cand["types"], cand["len"], cand["lo"],
                             cand["hi"], 3, projection=True)
    b = fe.Batch(ctx, [{"ids": ids, "ticks": ticks, "num_types": T,
                        "cand": ctx.cand_tensors(cand), "theta": 3}] * 3)
    b.run()
    ctx.sync()
    for r in range(3):
        assert np.array_equal(b.upper[r].cpu().numpy(), wu)
        assert np.array_equal(b.exact[r].cpu().numpy(), we)
    b.close()


def test_types_of_most_events_cost(ctx, fe):
    # the index of a stream with two types of nine tenths of its events takes no
    # more than three times that of an even one
    import time
    rng = np.random.default_rng(12)
    T, n = 1000, 1_000_000
    cand = ctx.cand_tensors(synth.pack([((3, 5), (0,), (50,))]))
    best = []
    for hot in (False, True):
        ids_h = rng.integers(0, T, n)
        if hot:
            ids_h = np.where(rng.random(n) < 0.9, rng.integers(0, 2, n), ids_h)
        ids, ticks = ctx.stream_tensors(ids_h.astype(np.int32),
                                        np.sort(rng.integers(0, 8 * n, n)).astype(np.int32))
        t = []
        for _ in range(6):
            ctx.torch.cuda.synchronize()
            a = time.perf_counter()
            ctx.count(ids, ticks, T, cand, EXACT)
            ctx.torch.cuda.synchronize()
            t.append(time.perf_counter() - a)
        best.append(min(t))
    banner("even %.0f us, uneven %.0f us" % (best[0] * 1e6, best[1] * 1e6))
    assert best[1] < 3 * best[0]
