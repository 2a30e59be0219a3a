"""Device memory: what a server, a count and the miner hold stays within what
they were given, and calls whose lists do not fit are counted all the same."""
import numpy as np
import pytest

import oracle
from paper_0905_2200_amd import synth
from tests.gpu_util import banner, have_gpu, oracle_counts

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not have_gpu(), reason="needs a GPU")]

EXACT, RELAXED = 0, 1
IVS = [(0, 50), (50, 100), (100, 200)]


@pytest.fixture(scope="module")
def fe():
    from paper_0905_2200_amd import fe as fe_mod
    return fe_mod


@pytest.fixture(scope="module")
def ctx(fe):
    c = fe.Context(0)
    yield c
    c.close()


def _free(ctx):
    ctx.torch.cuda.synchronize()
    return ctx.torch.cuda.mem_get_info()[0]


def test_server_lanes_share_the_budget(ctx, fe):
    # 8 lanes of a 2 GiB budget, buffers for windows whose lists alone are 2 GiB
    cand = synth.pack([((0, 1), (0,), (50,))])
    before = _free(ctx)
    sv = fe.Server(ctx, cand, [2], capacity=130_000_000, hbm_budget=2 << 30, max_inflight=8)
    held = before - _free(ctx)
    banner("server of 8 lanes holds %.2f GiB" % (held / 2 ** 30))
    sv.close()
    # the array (1 GiB), the lanes' shares, a quarter more of each, 1 GiB for all else
    assert held < 1.25 * (2 * 4 * 130_000_000 + (2 << 30)) + (1 << 30)


@pytest.mark.parametrize("lanes", [1, 4])
def test_windows_between_a_share_and_the_budget(ctx, fe, lanes):
    rng = np.random.default_rng(61)
    T, n = 40, 60_000
    ids = rng.integers(0, T, n).astype(np.int32)
    ticks = np.cumsum(rng.integers(0, 9, n)).astype(np.int32)
    cand = synth.pack(synth.random_episodes(rng, 64, T, 3, IVS, n_min=3))
    budget = 2 << 20
    sv = fe.Server(ctx, cand, [T], capacity=n, hbm_budget=budget, max_inflight=lanes, max_round=4)
    sv.append(0, ids, ticks)
    cuts = [(0, int(ticks[k])) for k in (500, 5_000, 20_000, 30_000, 45_000, 59_000, 200, 58_000)]
    tk = [sv.submit(0, a, b, 2) for a, b in cuts]
    banner("windows between a share and the budget: %d lanes" % lanes)
    feet = []
    for (a, b), t in zip(cuts, tk):
        r = sv.wait(t)
        k = np.searchsorted(ticks, b, "left")
        wu, we = oracle.two_pass(ids[:k], ticks[:k], T, cand["types"], cand["len"], cand["lo"],
                                 cand["hi"], 2, projection=True)
        assert r["status"] == fe.FE_OK and r["n_events"] == k
        assert np.array_equal(r["upper"], wu) and np.array_equal(r["exact"], we), k
        feet.append(r["footprint"])
    st = sv.stats()
    sv.close()
    assert st["completed"] == len(cuts) and st["rejected"] == 0
    # (the widest window's lists are about 1 MiB: within one lane's share of one,
    # not of four, where it is counted event by event)
    assert max(feet) <= budget // lanes
    assert max(feet) > budget // 4 or lanes == 4


def test_segments_of_many_rows(ctx, fe):
    # 262144 rows, as many segments as asked for: their results stay within 1 GiB
    t = ctx.torch
    M, n = 1 << 18, 1 << 21
    ids = t.zeros(n, dtype=t.int32, device=ctx.device)
    ticks = t.arange(n, dtype=t.int32, device=ctx.device)
    cand = ctx.cand_tensors({"types": np.zeros((M, 1), np.int32), "len": np.ones(M, np.int32),
                             "lo": np.zeros((M, 0), np.int32), "hi": np.zeros((M, 0), np.int32)})
    with fe.Context(0) as own:
        own.set_param(fe.PARAM_TARGET_WAVES, 1 << 30)
        before = _free(ctx)
        got = own.count(ids, ticks, 1, cand, EXACT)
        assert own.stats()["segments_max"] >= 2
        assert (got == n).all().item()
        held = before - _free(ctx)
        banner("segments of %d rows: %.2f GiB" % (M, held / 2 ** 30))
    assert held < 2 << 30


def _levels(ctx, fe, s, ivs, max_level, limit):
    """(levels, kernels' names, device bytes that limit 0 gives back) under a limit."""
    ids, ticks = ctx.stream_tensors(s["ids"], s["ticks"])
    with fe.Context(0) as own:
        if limit is not None:
            own.set_param(fe.PARAM_LIST_BYTES, limit)
        own.set_param(fe.PARAM_TIMING, 1)
        out = own.mine(ids, ticks, s["num_types"], ivs, s["theta"], max_level)
        names = set(own.kernel_stats())
        own.set_param(fe.PARAM_TIMING, 0)
        before = _free(ctx)
        own.set_param(fe.PARAM_LIST_BYTES, 0)
        back = _free(ctx) - before
        # a second run with the limit lowered, and raised again
        for lim in (0, 1 << 62):
            own.set_param(fe.PARAM_LIST_BYTES, lim)
            again = own.mine(ids, ticks, s["num_types"], ivs, s["theta"], max_level)
            _same(out, again)
    return out, names, back


def _same(a, b):
    assert len(a) == len(b)
    for x, y in zip(a, b):
        for k in ("level", "n_candidates", "n_survivors", "n_frequent", "types", "lo", "hi",
                  "upper", "exact"):
            assert np.array_equal(np.asarray(x[k]), np.asarray(y[k])), (x["level"], k)


def test_mining_within_a_limit(ctx, fe):
    # everything fits; the lists do not beside the largest level, so that they
    # are given up on the way; only the index fits; nothing does
    s = synth.config_mining(duration_s=30.0)
    T, n, n_iv = s["num_types"], s["ids"].size, len(s["intervals"])
    index = 4 * (4 * n + 40 * T) + 8 * T * (n // 512 + 1)
    # (12 B of entries a type, interval and event, 8 B of masks an interval and event, twice)
    lists = 2 * (12 * T + 8) * n_iv * (n + 5 * T) + 8 * T * T * n_iv
    banner("mining within a limit: index %d lists %d" % (index, lists))
    free, names, back = _levels(ctx, fe, s, s["intervals"], 4, None)
    assert any("siblings_n4" in k for k in names) and back > lists // 2
    want = {"mid": lambda k: any("pairs" in x for x in k) and any("_chain" in x for x in k)
            and not any("siblings_n4" in x for x in k),
            "index": lambda k: any("_chain" in x for x in k) and not any("pairs" in x for x in k),
            "none": lambda k: not any("chain" in x or "pairs" in x or "siblings" in x for x in k)}
    for key, limit in (("mid", index + lists + 64_000), ("index", 2 * index), ("none", 1)):
        got, names, back = _levels(ctx, fe, s, s["intervals"], 4, limit)
        _same(free, got)
        assert want[key](names), (key, sorted(names))
        assert back == 0, key


def test_frequent_sets_beyond_the_pinned_memory(ctx, fe):
    # nearly every pair of 2000 types with three intervals is frequent: 7e7 ints, copied
    # without the pinned staging; the same set from the event-by-event kernels
    rng = np.random.default_rng(3)
    T, n = 2000, 200_000
    ids, ticks = ctx.stream_tensors(rng.integers(0, T, n).astype(np.int32),
                                    np.sort(rng.integers(0, n // 5, n)).astype(np.int32))
    with fe.Context(0) as own:
        a = own.mine(ids, ticks, T, IVS, 1, 2)
        own.set_param(fe.PARAM_ELIMINATION, 0)
        b = own.mine(ids, ticks, T, IVS, 1, 2)
        own.set_param(fe.PARAM_LIST_BYTES, 0)
        c = own.mine(ids, ticks, T, IVS, 1, 2)
    nf = a[1]["n_frequent"]
    banner("frequent pairs: %d" % nf)
    assert nf * 6 > 64 << 20
    for k in ("types", "lo", "hi", "exact"):
        assert np.array_equal(a[1][k], b[1][k]) and np.array_equal(a[1][k], c[1][k]), k
    assert (b[1]["upper"] == -1).all()
