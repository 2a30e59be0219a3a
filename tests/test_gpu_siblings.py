"""Mining with join siblings counted together against the oracle's miner, bit
for bit, where the masks, the pairs' entries and the columns can go wrong:
type counts around a mask word, more words than a wave takes, dense streams
(chains that start inside an earlier completion's range), ties, intervals
given twice, unsorted, narrow or wide; and both counters of every candidate
against the event-by-event kernels."""
import numpy as np
import pytest

from oracle import mine as omine
from tests.gpu_util import banner, have_gpu

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not have_gpu(), reason="needs a GPU")]


@pytest.fixture(scope="module")
def fe():
    from paper_0905_2200_amd import fe as fe_mod
    return fe_mod


@pytest.fixture(scope="module")
def ctx(fe):
    c = fe.Context(0)
    yield c
    c.close()


def _stream(rng, n, T, mean_gap, hot=None, ties=0.0):
    w = np.full(T, 1.0)
    if hot is not None:
        w[hot] = 30.0
    ids = rng.choice(T, n, p=w / w.sum()).astype(np.int32)
    gaps = rng.integers(0, 2 * mean_gap + 1, n)
    gaps[rng.random(n) < ties] = 0
    return ids, np.cumsum(gaps).astype(np.int32)


def _mine(ctx, fe, ids_h, ticks_h, T, ivs, theta, max_level, params):
    saved = {p: ctx.get_param(p) for p in params}
    ids, ticks = ctx.stream_tensors(ids_h, ticks_h)
    try:
        for p, v in params.items():
            ctx.set_param(p, v)
        return ctx.mine(ids, ticks, T, ivs, theta, max_level)
    finally:
        for p, v in saved.items():
            ctx.set_param(p, v)


def _check_oracle(got, want, theta):
    assert [lv["level"] for lv in got] == sorted(want)
    for lv in got:
        L, w = lv["level"], want[lv["level"]]
        assert lv["n_candidates"] == len(w["candidates"]), L
        g = {(tuple(t), tuple(a), tuple(b)): int(x)
             for t, a, b, x in zip(lv["types"], lv["lo"], lv["hi"], lv["exact"])}
        wf = {ep: int(w["exact"][k]) for k, ep in enumerate(w["candidates"]) if ep in w["frequent"]}
        assert g == wf, L


def _same_as_events(ctx, fe, ids_h, ticks_h, T, ivs, theta, max_level):
    for elim in (1, 0):  # both counters; the exact one alone
        base = {fe.PARAM_ELIMINATION: elim, fe.PARAM_KEEP_CANDIDATES: 1}
        a = _mine(ctx, fe, ids_h, ticks_h, T, ivs, theta, max_level, base)
        b = _mine(ctx, fe, ids_h, ticks_h, T, ivs, theta, max_level,
                  {**base, fe.PARAM_TYPE_DISPATCH: 0})
        assert [x["level"] for x in a] == [x["level"] for x in b]
        for x, y in zip(a, b):
            assert x["n_survivors"] == y["n_survivors"], x["level"]
            for k in ("types", "lo", "hi", "exact", "upper", "all_types", "all_lo", "all_hi",
                      "all_exact", "all_upper"):
                assert np.array_equal(np.asarray(x[k]), np.asarray(y[k])), (elim, x["level"], k)
    return a


@pytest.mark.parametrize("T", [3, 31, 32, 33, 64, 65, 130])
def test_type_counts(ctx, fe, T):
    rng = np.random.default_rng(T)
    hot = rng.choice(T, min(T, 5), replace=False)
    ids_h, ticks_h = _stream(rng, 9_000, T, 6, hot=hot)
    ivs, theta = [(0, 30), (30, 60)], 150 if T > 3 else 700
    banner("siblings: T=%d" % T)
    want = omine.mine(ids_h, ticks_h, T, ivs, theta, 4)
    got = _mine(ctx, fe, ids_h, ticks_h, T, ivs, theta, 4, {fe.PARAM_ELIMINATION: 0})
    assert got[-1]["level"] >= 3
    _check_oracle(got, want, theta)


@pytest.mark.parametrize("nf,n_iv", [(21, 3), (22, 3), (43, 3), (5, 13), (11, 24)])
def test_sibling_group_sizes(ctx, fe, nf, n_iv):
    # every pair frequent: each episode has nf * n_iv siblings (63, 66, 129, 65, 264)
    rng = np.random.default_rng(100 + nf)
    ids_h, ticks_h = _stream(rng, 4_000 + 150 * nf, nf, 2, ties=0.2)
    ivs = [(3 * k, 3 * k + 40) for k in range(n_iv)]
    banner("siblings: %d types x %d intervals" % (nf, n_iv))
    out = _same_as_events(ctx, fe, ids_h, ticks_h, nf, ivs, 3, 3)
    assert out[2]["n_candidates"] == nf ** 3 * n_iv ** 2


@pytest.mark.parametrize("seed,ivs", [
    (1, [(0, 20), (20, 40)]),
    (2, [(100, 200), (0, 50), (50, 100)]),      # not sorted
    (3, [(0, 40), (0, 40), (10, 60)]),          # one twice
    (4, [(190, 200), (9, 10)]),                 # narrow
    (5, [(0, 3000)]),                           # hundreds of events a window
    (6, [(5, 8), (0, 400), (399, 400)]),
])
def test_dense_streams(ctx, fe, seed, ivs):
    # few types, windows that hold many events of each: most chains start
    # inside the window of an earlier completion
    rng = np.random.default_rng(seed)
    ids_h, ticks_h = _stream(rng, 6_001, 5, 4, ties=0.15 * (seed % 3))
    banner("siblings, dense: %s" % (ivs,))
    _same_as_events(ctx, fe, ids_h, ticks_h, 5, ivs, 5, 5 if len(ivs) < 3 else 4)


def test_rule_with_samples(ctx, fe):
    # the sampled relaxed pass and both answers of the rule
    rng = np.random.default_rng(77)
    ids_h, ticks_h = _stream(rng, 8_000, 12, 5)
    ivs, theta = [(0, 30), (30, 60)], 60
    want = omine.mine(ids_h, ticks_h, 12, ivs, theta, 4)
    for cost in (0, 500, 1000):
        got = _mine(ctx, fe, ids_h, ticks_h, 12, ivs, theta, 4,
                    {fe.PARAM_ELIMINATION: 2, fe.PARAM_SAMPLE_MIN: 200, fe.PARAM_PASS1_COST: cost})
        _check_oracle(got, want, theta)
        assert cost == 1000 or any(L["sample_n"] > 0 for L in got)


@pytest.mark.parametrize("T,words", [(30, 1), (46, 2), (70, 4)])
def test_words_a_wave(ctx, fe, T, words):
    # so many frequent pairs that a wave takes one, two or four mask words
    # (the last few of them fewer), against the event-by-event kernels
    rng = np.random.default_rng(T)
    ids, ticks = _stream(rng, 60 * T, T, 1)
    ivs, theta = [(0, 50), (50, 100), (100, 200)], 12
    banner("words a wave: T=%d words=%d n=%d" % (T, words, ids.size))
    a = _mine(ctx, fe, ids, ticks, T, ivs, theta, 3, {fe.PARAM_ELIMINATION: 1})
    b = _mine(ctx, fe, ids, ticks, T, ivs, theta, 3,
              {fe.PARAM_ELIMINATION: 1, fe.PARAM_TYPE_DISPATCH: 0})
    assert len(a) == len(b) == 3
    cnt, Q = a[1]["n_frequent"], (T + 63) // 64 * 3
    assert words == 1 or cnt * -(-Q // words) >= 8192
    assert words == 4 or cnt * -(-Q // (2 * words)) < 8192
    for x, y in zip(a, b):
        for k in ("n_candidates", "n_survivors", "n_frequent"):
            assert x[k] == y[k], (x["level"], k)
        for k in ("types", "lo", "hi", "upper", "exact"):
            assert np.array_equal(x[k], y[k]), (x["level"], k)


@pytest.mark.parametrize("T,n,levels", [(3, 18_000, 5), (8, 40_000, 4), (8, 30_000, 4), (19, 90_000, 3)])
@pytest.mark.parametrize("elim", [0, 1])
def test_few_candidates_over_long_lists(ctx, fe, T, n, levels, elim):
    # few candidates row by row (lists of 4096 events and more), from more on by
    # siblings, whose pairs' entries are made then; the same sets event by event
    rng = np.random.default_rng(100 * T + n)
    ids_h, ticks_h = _stream(rng, n, T, 20, ties=0.1)
    ivs = [(0, 50), (50, 100), (100, 200)]
    theta = 3 * n // (T * T * 100)
    got = {}
    ctx.set_param(fe.PARAM_TIMING, 1)
    try:
        for room in (1 << 62, 0):
            ctx.reset_kernel_stats()
            got[room] = _mine(ctx, fe, ids_h, ticks_h, T, ivs, theta, levels,
                              {fe.PARAM_LIST_BYTES: room, fe.PARAM_ELIMINATION: elim})
            if room:
                names = set(ctx.kernel_stats())
    finally:
        ctx.set_param(fe.PARAM_TIMING, 0)
    banner("few candidates over long lists: T=%d n=%d %s" % (
        T, n, [lv["n_candidates"] for lv in got[0]]))
    a, b = got[1 << 62], got[0]
    assert len(a) == len(b)
    for x, y in zip(a, b):
        for k in ("level", "n_candidates", "n_survivors", "n_frequent", "types", "lo", "hi",
                  "upper", "exact"):
            assert np.array_equal(np.asarray(x[k]), np.asarray(y[k])), (x["level"], k)
    long_list = n // T >= 4096
    small = [lv["n_candidates"] < (1024 if lv["level"] == 2 else 16384 if elim else 4096)
             for lv in a if lv["level"] > 1]
    rows = "map_two_pass_chain" if elim else "map_exact_chain"
    assert (rows in names) == (long_list and any(small))
    assert any("pairs" in k for k in names) == (not long_list or not all(small))


def test_few_candidates_cost(ctx, fe):
    # a long recording of few types: no more than two and a half times the
    # event-by-event kernels, which cut its events into segments
    import time
    rng = np.random.default_rng(6)
    T, n = 4, 1_000_000
    ids, ticks = ctx.stream_tensors(rng.integers(0, T, n).astype(np.int32),
                                    np.sort(rng.integers(0, 100 * n, n)).astype(np.int32))
    best = {}
    for room in (1 << 62, 0):
        ctx.set_param(fe.PARAM_LIST_BYTES, room)
        t = []
        for _ in range(4):
            a = time.perf_counter()
            ctx.mine(ids, ticks, T, [(0, 50), (50, 100), (100, 200)], 20_000, 4)
            t.append(time.perf_counter() - a)
        best[room] = min(t)
    ctx.set_param(fe.PARAM_LIST_BYTES, 1 << 62)
    banner("mining 1e6 events of 4 types: %.2f ms, event by event %.2f ms" % (
        best[1 << 62] * 1e3, best[0] * 1e3))
    assert best[1 << 62] < 2.5 * best[0]
