"""Segments' results put together: streams on which a segment's own run and the
run from the segment before it meet late or never (regular gaps, dense streams),
for rows few and many, against the CPU oracle bit for bit, and what such
streams cost."""
import time

import numpy as np
import pytest

import oracle
from paper_0905_2200_amd import synth
from tests.gpu_util import banner, have_gpu, oracle_counts

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not have_gpu(), reason="needs a GPU")]

EXACT, RELAXED = 0, 1


@pytest.fixture(scope="module")
def fe():
    from paper_0905_2200_amd import fe as fe_mod
    return fe_mod


@pytest.fixture(scope="module")
def ctx(fe):
    c = fe.Context(0)
    yield c
    c.close()


def _periodic(n, T=2):
    """Every type at every tick."""
    return np.tile(np.arange(T), n // T).astype(np.int32), \
        np.repeat(np.arange(n // T), T).astype(np.int32)


def _episodes(rng, T, kind):
    if kind == "periodic":  # completions 11, 13, 24, ... ticks apart
        eps = [((a, b), (l,), (l + 1,)) for a in range(T) for b in range(T) for l in (9, 11, 22)]
        eps += [((0, 1, 0), (9, 3), (10, 4)), ((1, 1, 0, 1), (5, 7, 2), (6, 9, 3)),
                ((0,), (), ()), ((0, 0, 1), (0, 9), (1, 10))]
        return eps
    return synth.random_episodes(rng, 40, T, 6, [(0, 5), (0, 60), (20, 24), (30, 90)], n_min=2)


@pytest.mark.parametrize("kind,T,gap", [("periodic", 2, 0), ("dense", 2, 1), ("dense", 3, 2),
                                        ("dense", 4, 6)])
@pytest.mark.parametrize("rows", [1, 3, 65, 700, 8191, 8192])
def test_segments_that_do_not_meet(ctx, fe, kind, T, gap, rows):
    rng = np.random.default_rng(rows + 7 * T + gap)
    n = 9_000
    if kind == "periodic":
        ids_h, ticks_h = _periodic(n, T)
    else:
        ids_h = rng.integers(0, T, n).astype(np.int32)
        ticks_h = np.cumsum(rng.integers(0, gap + 1, n)).astype(np.int32)
    eps = _episodes(rng, T, kind)
    first = int(rng.integers(len(eps)))
    use = [eps[(first + i) % len(eps)] for i in range(min(rows, len(eps)))]
    cand = synth.pack(use)
    many = synth.pack([use[i % len(use)] for i in range(rows)])
    at = np.arange(rows) % len(use)
    want = {m: oracle_counts(ids_h, ticks_h, T, cand, m) for m in (EXACT, RELAXED)}
    theta = max(1, int(np.median(want[RELAXED])))
    wu, we = oracle.two_pass(ids_h, ticks_h, T, cand["types"], cand["len"], cand["lo"],
                             cand["hi"], theta, projection=True)
    ids, ticks = ctx.stream_tensors(ids_h, ticks_h)
    saved = ctx.get_param(fe.PARAM_TARGET_WAVES)
    try:
        # (as many segments as the rule has for so many events)
        ctx.set_param(fe.PARAM_TARGET_WAVES, 1 << 22)
        banner("segments that do not meet: %s T=%d rows=%d" % (kind, T, rows))
        for m in (EXACT, RELAXED):
            got = ctx.count(ids, ticks, T, many, m).cpu().numpy()
            assert ctx.stats()["segments_max"] >= 2
            assert np.array_equal(got, want[m][at]), m
        up, ex, ns = ctx.count_two_pass(ids, ticks, T, many, theta)
        assert np.array_equal(up.cpu().numpy(), wu[at])
        assert np.array_equal(ex.cpu().numpy(), we[at])
        assert int(ns.item()) == int((wu[at] >= theta).sum())
    finally:
        ctx.set_param(fe.PARAM_TARGET_WAVES, saved)


def test_more_segments_than_a_wave(ctx, fe):
    # 100 to 200 segments of one row: a wave puts 64 together at a time
    rng = np.random.default_rng(77)
    ids_h = rng.integers(0, 2, 200_000).astype(np.int32)
    ticks_h = np.cumsum(rng.integers(0, 3, ids_h.size)).astype(np.int32)
    eps = [((0, 1), (9,), (10,)), ((1, 0, 1), (0, 4), (30, 9)), ((0, 1), (0,), (2,)),
           ((0, 1, 1, 0), (50, 60, 70), (55, 70, 90))]
    ids, ticks = ctx.stream_tensors(ids_h, ticks_h)
    banner("more segments than a wave")
    for e in eps:
        cand = synth.pack([e])
        for m in (EXACT, RELAXED):
            want = oracle_counts(ids_h, ticks_h, 2, cand, m)
            assert np.array_equal(ctx.count(ids, ticks, 2, cand, m).cpu().numpy(), want), (e, m)
            assert ctx.stats()["segments_max"] > 64


@pytest.mark.parametrize("kind,rows", [("periodic", 64), ("dense", 64), ("dense", 1000)])
def test_segments_cost(ctx, fe, kind, rows):
    # cut into segments, a call takes no more than a few times what it takes
    # whole (rows in one wave that are put together one after the other took 30)
    rng = np.random.default_rng(5)
    if kind == "periodic":
        T = 2
        stream = _periodic(1 << 16)
        cand = synth.pack([((0, 1), (9,), (10,))] * rows)
    else:
        T = 3
        stream = (rng.integers(0, T, 300_000).astype(np.int32),
                  np.cumsum(rng.integers(0, 3, 300_000)).astype(np.int32))
        cand = synth.pack(synth.random_episodes(rng, rows, T, 3, [(0, 50), (50, 100), (100, 200)],
                                                n_min=2))
    ids, ticks = ctx.stream_tensors(*stream)
    cd = ctx.cand_tensors(cand)
    keys = (fe.PARAM_CROSSOVER_A, fe.PARAM_CROSSOVER_B, fe.PARAM_CROSSOVER_A_RELAXED,
            fe.PARAM_CROSSOVER_B_RELAXED)
    saved = [ctx.get_param(p) for p in keys]

    def best(mode):
        t = []
        for _ in range(6):
            ctx.torch.cuda.synchronize()
            a = time.perf_counter()
            ctx.count(ids, ticks, T, cd, mode)
            ctx.torch.cuda.synchronize()
            t.append(time.perf_counter() - a)
        return min(t)
    banner("segments' cost: %s, %d rows" % (kind, rows))
    cut = [best(m) for m in (EXACT, RELAXED)]
    assert ctx.stats()["segments_max"] >= 2
    try:
        for p in keys:
            ctx.set_param(p, 0)
        whole = [best(m) for m in (EXACT, RELAXED)]
        assert ctx.stats()["segments_max"] == 1
    finally:
        for p, v in zip(keys, saved):
            ctx.set_param(p, v)
    print("cut", cut, "whole", whole, flush=True)
    for c, w in zip(cut, whole):
        assert c < 5 * w + 5e-4


def _mixed_jobs(rng):
    """(ids, ticks, types, rows): few rows over long lists, which are cut, beside
    short, empty and rowless ones, which are not."""
    out = []
    for n, T, gap, rows in ((30_000, 2, 2, 40), (0, 3, 1, 5), (9_000, 3, 1, 7), (500, 4, 20, 60),
                            (24_000, 2, 0, 9), (4_000, 1, 3, 3), (700, 5, 9, 0)):
        if gap:
            ids = rng.integers(0, T, n).astype(np.int32)
            ticks = np.cumsum(rng.integers(0, gap + 1, n)).astype(np.int32)
            eps = synth.random_episodes(rng, rows, T, 6, [(0, 5), (0, 60), (20, 24), (30, 90)],
                                        n_min=1)
        else:
            ids, ticks = _periodic(n, T)
            eps = _episodes(rng, T, "periodic")[:rows]
        out.append((ids, ticks, T, synth.pack(eps, nmax=6)))
    return out


@pytest.mark.parametrize("nmax", [3, 6])
def test_batch_in_segments(ctx, fe, nmax):
    rng = np.random.default_rng(nmax)
    jobs = []
    for ids, ticks, T, cand in _mixed_jobs(rng):
        keep = cand["len"] <= nmax
        jobs.append((ids, ticks, T, {"types": cand["types"][keep, :nmax], "len": cand["len"][keep],
                                     "lo": cand["lo"][keep, :nmax - 1],
                                     "hi": cand["hi"][keep, :nmax - 1],
                                     "M": int(keep.sum()), "nmax": nmax}))
    for theta in (1, 300, 20_000):
        recs = []
        for ids, ticks, T, cand in jobs:
            i, t = ctx.stream_tensors(ids, ticks)
            recs.append({"ids": i, "ticks": t, "num_types": T, "cand": ctx.cand_tensors(cand),
                         "theta": theta})
        banner("batch in segments: nmax=%d theta=%d" % (nmax, theta))
        b = fe.Batch(ctx, recs)
        for _ in range(2):
            b.run()
            ctx.sync()
            for r, (ids, ticks, T, c) in enumerate(jobs):
                if c["M"] == 0:
                    continue
                wu, we = oracle.two_pass(ids, ticks, T, c["types"], c["len"], c["lo"], c["hi"],
                                         theta, projection=True)
                assert np.array_equal(b.upper[r].cpu().numpy(), wu), r
                assert np.array_equal(b.exact[r].cpu().numpy(), we), r
        recs[0]["ids"][5] = 99  # (no longer a valid recording)
        b.run()
        ctx.sync()
        for r in range(len(jobs)):
            assert (b.upper[r][:jobs[r][3]["M"]] == -1).all().item()
            assert (b.exact[r][:jobs[r][3]["M"]] == -1).all().item()
        b.close()


@pytest.mark.parametrize("waves", [16384, 1 << 20])
def test_served_in_segments(ctx, fe, waves):
    # (more segments than a round has room for: none)
    rng = np.random.default_rng(8)
    ids = rng.integers(0, 3, 60_000).astype(np.int32)
    ticks = np.cumsum(rng.integers(0, 3, 60_000)).astype(np.int32)
    eps = synth.random_episodes(rng, 900, 3, 4, [(0, 5), (0, 60), (20, 24), (30, 90)], n_min=1)
    cand = synth.pack(eps)
    saved = ctx.get_param(fe.PARAM_TARGET_WAVES)
    ctx.set_param(fe.PARAM_TARGET_WAVES, waves)
    try:
        sv = fe.Server(ctx, cand, [3, 3], capacity=60_000, hbm_budget=1 << 28, max_round=4)
        for a in range(2):
            sv.append(a, ids, ticks)
        cuts = [(k % 2, int(ticks[k * 900]), int(ticks[59_999 - 4_000 * k])) for k in range(9)]
        tk = [sv.submit(a, t0, t1, 40) for a, t0, t1 in cuts]
        banner("served in segments: %d waves" % waves)
        for (a, t0, t1), t in zip(cuts, tk):
            res = sv.wait(t)
            x, y = np.searchsorted(ticks, t0, "left"), np.searchsorted(ticks, t1, "left")
            wu, we = oracle.two_pass(ids[x:y], ticks[x:y], 3, cand["types"], cand["len"],
                                     cand["lo"], cand["hi"], 40, projection=True)
            assert res["status"] == fe.FE_OK
            assert np.array_equal(res["upper"], wu) and np.array_equal(res["exact"], we), (t0, t1)
        sv.close()
    finally:
        ctx.set_param(fe.PARAM_TARGET_WAVES, saved)


def test_long_batch_cost(ctx, fe):
    # few rows over one long recording: no more than three times the call alone
    rng = np.random.default_rng(4)
    T, n = 8, 4_000_000
    ids, ticks = ctx.stream_tensors(rng.integers(0, T, n).astype(np.int32),
                                    np.sort(rng.integers(0, 50 * n, n)).astype(np.int32))
    cand = ctx.cand_tensors(synth.pack(synth.random_episodes(
        rng, 16, T, 2, [(0, 50), (50, 100), (100, 200)], n_min=2)))
    b = fe.Batch(ctx, [{"ids": ids, "ticks": ticks, "num_types": T, "cand": cand, "theta": 30}])

    def best(call):
        t = []
        for _ in range(6):
            ctx.torch.cuda.synchronize()
            a = time.perf_counter()
            call()
            ctx.torch.cuda.synchronize()
            t.append(time.perf_counter() - a)
        return min(t)
    lone = best(lambda: ctx.count_two_pass(ids, ticks, T, cand, 30))
    both = best(b.run)
    banner("16 rows over 4e6 events: alone %.0f us, batch %.0f us" % (lone * 1e6, both * 1e6))
    b.close()
    assert both < 3 * lone
