"""The event-by-event kernels, which take what per-type lists do not: calls
whose lists do not fit FE_PARAM_LIST_BYTES or memory, and more than 4096 types.
The tests written for them run here with no room for lists, each with a look
at which kernels ran, as the same calls are counted over lists by default."""
import numpy as np
import pytest

import oracle
from paper_0905_2200_amd import synth
from tests import test_gpu_batched as batched
from tests import test_gpu_chain as chain
from tests import test_gpu_deep as deep
from tests import test_gpu_dispatch as dispatch
from tests import test_gpu_resume as resume
from tests import test_gpu_served as served
from tests.gpu_util import banner, have_gpu

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not have_gpu(), reason="needs a GPU")]

EXACT, RELAXED = 0, 1
LISTS = ("index", "chain", "pairs", "siblings", "masks")


@pytest.fixture(scope="module")
def fe():
    from paper_0905_2200_amd import fe as fe_mod
    return fe_mod


@pytest.fixture(scope="module")
def ctx(fe):
    c = fe.Context(0)
    c.set_param(fe.PARAM_LIST_BYTES, 0)
    c.set_param(fe.PARAM_TIMING, 1)
    yield c
    c.close()


@pytest.fixture(autouse=True)
def _event_by_event(ctx):
    ctx.reset_kernel_stats()
    yield
    assert not [k for k in ctx.kernel_stats() if any(x in k for x in LISTS)]


def _ran(ctx, *parts):
    names = list(ctx.kernel_stats())
    for p in parts:
        assert any(p in k for k in names), (p, names)


def test_lists_are_the_default(fe, ctx):
    # (what the look at the kernels' names would find)
    with fe.Context(0) as own:
        own.set_param(fe.PARAM_TIMING, 1)
        ids, ticks = own.stream_tensors([0, 1, 0, 1], [0, 5, 6, 9])
        cand = own.cand_tensors(synth.pack([((0, 1), (0,), (10,))]))
        own.count(ids, ticks, 2, cand, EXACT)
        b = fe.Batch(own, [{"ids": ids, "ticks": ticks, "num_types": 2, "cand": cand, "theta": 1}])
        b.run()
        own.sync()
        names = own.kernel_stats()
        b.close()
    assert {"index", "map_exact_chain", "batch_two_pass_chain"} <= set(names)


@pytest.mark.parametrize("seg_events,wpb", [(256, 4), (2048, 1), (2048, 8), (32768, 2)])
def test_batch(ctx, fe, seg_events, wpb):
    batched.test_batch_matches_oracle(ctx, fe, seg_events, wpb)


def test_batch_autotune(ctx, fe):
    batched.test_batch_equals_alone_and_autotune(ctx, fe)


def test_batch_uneven(ctx, fe):
    chain.test_batch_of_uneven_jobs(ctx, fe)


@pytest.mark.parametrize("P", [0, 2])
def test_deep_count(ctx, P):
    deep.test_deep_hops_mixed_count(ctx, P)
    _ran(ctx, "_deep")


def test_deep_rings(ctx):
    deep.test_deep_rings_near_capacity(ctx)
    deep.test_deep_rings_bounded_by_stream_and_chunked(ctx)
    _ran(ctx, "_deep")


def test_deep_two_pass_and_resume(ctx, fe):
    deep.test_deep_two_pass_and_resume(ctx, fe)
    _ran(ctx, "map_exact_n2_deep", "resume_exact_n2_deep")


def test_deep_batched_and_served(ctx, fe):
    deep.test_deep_batched_and_served(ctx, fe)


def test_deep_mining(ctx):
    deep.test_deep_interval_in_mining(ctx)
    _ran(ctx, "map_exact_n3_deep", "map_relaxed_n3")


def test_automatic_segments(ctx, fe):
    dispatch.test_hybrid_crossover_rule(ctx, fe)
    _ran(ctx, "map_exact_n4", "map_relaxed_n4")


@pytest.mark.parametrize("elim", [1, 0])
def test_device_tiling(ctx, fe, elim):
    dispatch.test_device_tiling_same_as_host(ctx, fe, elim)
    _ran(ctx, "map_exact_n4")


def test_device_tiling_classes(ctx, fe):
    dispatch.test_device_tiling_depth_classes(ctx, fe)


def test_elimination_rule(ctx, fe):
    dispatch.test_one_pass_mining_same_result(ctx, fe)


@pytest.mark.parametrize("mode", [RELAXED, EXACT])
def test_resume(ctx, fe, mode):
    resume.test_partitions_match_whole_stream(ctx, fe, mode)
    _ran(ctx, "resume_%s_n3" % ("exact" if mode == EXACT else "relaxed"))


def test_resume_mining_stream(ctx, fe):
    resume.test_resume_on_mining_partitions(ctx, fe)


def test_served(ctx, fe):
    sv = synth.config_served(n_arrays=4, trace_s=2.0, preroll_s=8.0, M=1500, rate_req=40.0,
                             win_lo_s=0.5, win_hi_s=8.0, tag=77)
    served.test_served_requests_match_oracle_and_alone(fe, ctx, sv)


def test_served_different_types(ctx, fe):
    # (small enough for event-by-event state at both budgets)
    chain.test_served_arrays_of_different_types(ctx, fe)


@pytest.mark.parametrize("seed", range(3))
def test_random_streams(ctx, seed):
    chain.test_random_streams(ctx, seed)


def test_more_types_than_lists_take(ctx, fe):
    # 4097 and more types, with room for lists: mined and batched event by event
    from oracle import mine
    rng = np.random.default_rng(71)
    T, n = 4100, 20_000
    hot = np.sort(rng.choice(T, 6, replace=False))
    hot[-1] = T - 1
    ids_h = np.where(rng.random(n) < 0.9, rng.choice(hot, n), rng.integers(0, T, n)).astype(np.int32)
    ticks_h = np.cumsum(rng.integers(0, 8, n)).astype(np.int32)
    ctx.set_param(fe.PARAM_LIST_BYTES, 1 << 62)
    try:
        ids, ticks = ctx.stream_tensors(ids_h, ticks_h)
        banner("%d types" % T)
        got = ctx.mine(ids, ticks, T, [(0, 50), (50, 100)], 300, 3)
        to = np.zeros(T, np.int32)
        to[hot] = np.arange(6)
        keep = np.isin(ids_h, hot)
        want = mine.mine(to[ids_h[keep]], ticks_h[keep], 6, [(0, 50), (50, 100)], 300, 3)
        assert [lv["level"] for lv in got] == [1, 2, 3] == sorted(want)
        for lv in got:
            w = want[lv["level"]]
            g = {(tuple(to[t]), tuple(a), tuple(b)): (int(u), int(x))
                 for t, a, b, u, x in zip(lv["types"], lv["lo"], lv["hi"], lv["upper"],
                                          lv["exact"])}
            assert g == {ep: (int(w["upper"][k]), int(w["exact"][k]))
                         for k, ep in enumerate(w["candidates"]) if ep in w["frequent"]}
        cand = synth.pack([(tuple(int(hot[e]) for e in ty), lo, hi) for ty, lo, hi in
                           synth.random_episodes(rng, 200, 6, 4, [(0, 50), (50, 100)], n_min=1)])
        wu, we = oracle.two_pass(ids_h, ticks_h, T, cand["types"], cand["len"], cand["lo"],
                                 cand["hi"], 20, projection=True)
        b = fe.Batch(ctx, [{"ids": ids, "ticks": ticks, "num_types": T,
                            "cand": ctx.cand_tensors(cand), "theta": 20}])
        b.run()
        ctx.sync()
        assert np.array_equal(b.upper[0].cpu().numpy(), wu)
        assert np.array_equal(b.exact[0].cpu().numpy(), we)
        b.close()
    finally:
        ctx.set_param(fe.PARAM_LIST_BYTES, 0)
