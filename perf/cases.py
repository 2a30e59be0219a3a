"""The measured work of the library, one case per way a program uses it.

Sizes are this repository's own: the five synthetic workloads (plain, mining,
large array, batched, served; paper_0905_2200_amd.synth) and the shapes of its
tests, from calls of a few thousand events, where launches and waits count, to
ten million events and twenty million candidates.  Streams are Poisson spike
trains with planted cascades, ticks of 0.1 ms, hop intervals (0,5], (5,10] and
(10,20] ms unless a case says otherwise; candidate tables hold the planted
sub-episodes first and random episodes after them.

A case is a dict:
  kind       count | two_pass | resume | mine | batch | serve
  neurons, rate_hz, seconds, lognormal   the stream (events = their product)
  episodes, n_min, n_max, hops           the candidate table
  mode       exact | relaxed (count, resume)
  theta_hz   support threshold in Hz (times the duration)
  max_level  mine;  part_s  resume: length of the last partition
  recordings batch;  requests  serve
"""
from __future__ import annotations

import math

import numpy as np
import torch

TICKS_PER_S = 10000
HOPS = {
    # (0,5], (5,10], (10,20] ms
    "standard": [(0, 50), (50, 100), (100, 200)],
    # narrow intervals far from 0: (4.5,5], (9.5,10], (19,20] ms
    "narrow": [(45, 50), (95, 100), (190, 200)],
}


def _case(kind, **kw):
    c = {"kind": kind, "neurons": 64, "rate_hz": 20.0, "seconds": 20.0, "lognormal": False,
         "episodes": 0, "n_min": 2, "n_max": 4, "hops": "standard", "mode": "exact",
         "theta_hz": 0.5, "max_level": 0, "part_s": 0.0, "recordings": 0, "requests": 0}
    c.update(kw)
    return c


def listed():
    return [
        # a few episodes re-counted over a few seconds of a small array: launches and waits
        _case("count", name="count_tiny", neurons=16, seconds=6.3, episodes=61, n_min=3, n_max=3),
        # the plain workload: every ordered pair of 64 neurons over 20 s, two passes
        _case("two_pass", name="two_pass_pairs", rate_hz=15.0, seconds=20.0, episodes=4096,
              n_min=2, n_max=2, theta_hz=2.5),
        # one table of episodes of every size, more types than a 64-bit mask holds
        _case("count", name="count_mixed", neurons=200, seconds=75.0, episodes=20011, n_min=1,
              n_max=8),
        # the relaxed counter alone (upper bounds) for long episodes over a 1M-event recording
        _case("count", name="count_relaxed_long", neurons=128, seconds=400.0, episodes=5000,
              n_min=5, n_max=8, mode="relaxed"),
        # narrow delay intervals far from 0 (lists of many live windows)
        _case("count", name="count_narrow", neurons=96, seconds=50.0, episodes=3000, n_min=2,
              n_max=4, hops="narrow"),
        # the large-array workload's three-node set: log-normal rates, 1e7 events, 1e5 episodes
        _case("two_pass", name="two_pass_large", neurons=256, rate_hz=10.0, seconds=3900.0,
              lognormal=True, episodes=100000, n_min=3, n_max=3),
        # a live recording: the last 10 s of 13 minutes added to resident episodes' counts
        _case("resume", name="resume_live", seconds=780.0, part_s=10.0, episodes=20000, n_min=2,
              n_max=6),
        # mining a short recording of 26 neurons (60 s)
        _case("mine", name="mine_short", neurons=26, seconds=60.0, max_level=4),
        # mining a wide array at a high threshold (200 types)
        _case("mine", name="mine_wide", neurons=200, seconds=60.0, theta_hz=3.0, max_level=4),
        # the mining workload: 64 neurons, 13 minutes, levels 2-6
        _case("mine", name="mine_long", seconds=780.0, max_level=6),
        # a planned batch of recordings of uneven length, each with its own table
        _case("batch", name="batch_uneven", recordings=32, seconds=0.0, episodes=20000, n_min=2,
              n_max=8),
        # a burst of window requests to a server over 16 arrays with resident episodes
        _case("serve", name="serve_burst", neurons=128, seconds=120.0, requests=24,
              episodes=20000, n_min=2, n_max=6),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["count", "count", "two_pass", "two_pass", "resume", "mine", "mine", "batch",
                       "serve"])
    if kind == "mine":
        if rng.random() < 0.3:
            return _case("mine", neurons=rng.randint(65, 200), seconds=round(_log(rng, 10, 60), 2),
                         theta_hz=round(rng.uniform(3.0, 4.0), 2), max_level=rng.randint(3, 4))
        return _case("mine", neurons=rng.randint(12, 48), seconds=round(_log(rng, 15, 780), 2),
                     theta_hz=round(rng.uniform(0.5, 2.0), 2), max_level=rng.randint(2, 5))
    n_min = rng.randint(1, 6)
    c = _case(kind, neurons=rng.randint(8, 256), rate_hz=round(rng.uniform(5.0, 25.0), 1),
              lognormal=rng.random() < 0.3, n_min=n_min, n_max=rng.randint(n_min, 8),
              hops="narrow" if rng.random() < 0.15 else "standard",
              mode=rng.choice(["exact", "relaxed"]), theta_hz=round(rng.uniform(0.1, 1.0), 3))
    if kind == "batch":
        c.update(recordings=rng.randint(2, 32), seconds=0.0, lognormal=False,
                 episodes=int(_log(rng, 1000, 20000)))
        return c
    if kind == "serve":
        c.update(neurons=rng.randint(64, 256), rate_hz=20.0, lognormal=False, seconds=120.0,
                 requests=rng.randint(1, 31), episodes=int(_log(rng, 500, 20000)))
        return c
    n = _log(rng, 2e3, 1e7 if kind != "resume" else 2e6)
    # narrow hops are counted over whole streams, so those stay shorter
    if c["hops"] == "narrow":
        n = min(n, 2e5)
    M = int(min(_log(rng, 30, 1e5), 5e11 / n))
    c.update(seconds=round(n / (c["neurons"] * c["rate_hz"]), 3), episodes=max(M, 30))
    if kind == "resume":
        c["part_s"] = round(c["seconds"] * _log(rng, 0.005, 0.3), 3)
    return c


# ------------------------------------------------------------------ inputs
def _rng(case, seed, part=0):
    return np.random.default_rng([int(seed), int(part), int(case["neurons"])])


def _cascades(rng, neurons, hops, count, length_hi):
    out = []
    for _ in range(count):
        L = min(int(rng.integers(3, length_hi + 1)), neurons)
        out.append((rng.choice(neurons, size=L, replace=False).astype(np.int64),
                    rng.integers(0, len(hops), size=L - 1), float(rng.uniform(1.0, 3.0))))
    return out


def _stream(rng, neurons, rate_hz, seconds, lognormal, hops, cascades):
    """Poisson background and planted cascades, ordered by (tick, id)."""
    dur = max(int(round(seconds * TICKS_PER_S)), 1)
    rates = np.full(neurons, float(rate_hz))
    if lognormal:
        rates = rng.lognormal(math.log(rate_hz) - 0.5, 1.0, size=neurons)
    cnt = rng.poisson(rates * seconds)
    ids = [np.repeat(np.arange(neurons, dtype=np.int64), cnt)]
    tks = [(rng.random(int(cnt.sum())) * dur).astype(np.int64)]
    for nodes, hop, rate in cascades:
        t = np.sort((rng.random(rng.poisson(rate * seconds)) * dur).astype(np.int64))
        for k, e in enumerate(nodes):
            if k:
                lo, hi = hops[hop[k - 1]]
                t = t + rng.integers(lo + 1, hi + 1, size=t.size)
            keep = t < dur
            ids.append(np.full(int(keep.sum()), e, np.int64))
            tks.append(t[keep])
    key = np.concatenate(tks) * neurons + np.concatenate(ids)
    key.sort()
    return (key % neurons).astype(np.int32), (key // neurons).astype(np.int32)


def _table(rng, neurons, M, n_min, n_max, hops, cascades):
    """Planted sub-episodes first, random episodes after them."""
    los = np.array([a for a, _ in hops], np.int32)
    his = np.array([b for _, b in hops], np.int32)
    ln = rng.integers(n_min, n_max + 1, size=M).astype(np.int32)
    ty = rng.integers(0, neurons, size=(M, n_max)).astype(np.int32)
    iv = rng.integers(0, len(hops), size=(M, max(n_max - 1, 1)))
    m = 0
    for nodes, hop, _ in cascades:
        for L in range(n_min, min(n_max, len(nodes)) + 1):
            for s in range(len(nodes) - L + 1):
                if m < M // 2:
                    ln[m] = L
                    ty[m, :L] = nodes[s:s + L]
                    iv[m, :L - 1] = hop[s:s + L - 1]
                    m += 1
    lo, hi = los[iv], his[iv]
    ty[np.arange(n_max)[None, :] >= ln[:, None]] = -1
    hm = max(n_max - 1, 0)
    used = np.arange(max(hm, 1))[None, :] < (ln - 1)[:, None]
    return {"types": ty, "len": ln, "lo": np.where(used, lo, 0)[:, :hm].astype(np.int32),
            "hi": np.where(used, hi, 0)[:, :hm].astype(np.int32), "nmax": n_max, "M": M}


def _recordings(case, seed):
    """(stream, table, neurons, seconds) of each recording of a batch: 1e4 to
    3e5 events, 16 to 256 neurons, 1000 to `episodes` candidates."""
    rng = _rng(case, seed)
    shape = np.random.default_rng(case["recordings"])  # a program's arrays keep their sizes
    hops = HOPS[case["hops"]]
    out = []
    for _ in range(case["recordings"]):
        nn = int(shape.integers(16, 257))
        n = math.exp(shape.uniform(math.log(1e4), math.log(3e5)))
        sec = n / (nn * 20.0)
        ca = _cascades(rng, nn, hops, int(rng.integers(2, 5)), 8)
        st = _stream(rng, nn, 20.0, sec, False, hops, ca)
        M = int(round(math.exp(shape.uniform(math.log(min(1000, case["episodes"])),
                                             math.log(case["episodes"])))))
        out.append((st, _table(rng, nn, M, case["n_min"], case["n_max"], hops, ca), nn, sec))
    return out


def _served(case, seed):
    """16 arrays' streams, the resident table and the requested windows (1 to
    60 s, ending in the second half of the recording)."""
    rng = _rng(case, seed)
    hops = HOPS[case["hops"]]
    streams, planted = [], []
    for _ in range(16):
        nn = int(rng.integers(64, case["neurons"] + 1))
        ca = _cascades(rng, 64, hops, 4, 6)
        streams.append(_stream(rng, nn, case["rate_hz"], case["seconds"], False, hops, ca) + (nn,))
        planted.extend(ca)
    table = _table(rng, 64, case["episodes"], case["n_min"], case["n_max"], hops, planted)
    reqs = []
    for _ in range(case["requests"]):
        w = math.exp(rng.uniform(0.0, math.log(60.0)))
        end = int(rng.uniform(0.5, 1.0) * case["seconds"] * TICKS_PER_S)
        reqs.append((int(rng.integers(16)), max(0, end - int(w * TICKS_PER_S)), end,
                     int(math.ceil(case["theta_hz"] * w))))
    return streams, table, reqs


def _single(case, seed):
    rng = _rng(case, seed)
    hops = HOPS[case["hops"]]
    nn = case["neurons"]
    ca = _cascades(rng, nn, hops, min(8, max(nn // 4, 1)), 6)
    ids, ticks = _stream(rng, nn, case["rate_hz"], case["seconds"], case["lognormal"], hops, ca)
    table = None
    if case["kind"] != "mine":
        table = _table(rng, nn, case["episodes"], case["n_min"], case["n_max"], hops, ca)
    return ids, ticks, table


def _theta(case):
    return max(1, int(math.ceil(case["theta_hz"] * case["seconds"])))


# ------------------------------------------------------------------ the calls
def prepare(case, seed):
    from paper_0905_2200_amd import fe

    ctx = fe.Context(0)
    kind = case["kind"]
    st = {"case": case, "ctx": ctx, "mode": fe.FE_EXACT if case["mode"] == "exact"
          else fe.FE_RELAXED}
    if kind == "batch":
        recs = []
        for (ids, ticks), table, nn, sec in _recordings(case, seed):
            di, dt = ctx.stream_tensors(ids, ticks)
            recs.append({"ids": di, "ticks": dt, "num_types": nn, "cand": ctx.cand_tensors(table),
                         "theta": max(1, int(math.ceil(case["theta_hz"] * sec)))})
        torch.cuda.synchronize()
        st["batch"] = fe.Batch(ctx, recs)
        return st
    if kind == "serve":
        streams, table, st["reqs"] = _served(case, seed)
        cap = max(s[0].size for s in streams) + 64
        srv = fe.Server(ctx, table, [s[2] for s in streams], capacity=cap, hbm_budget=8 << 30)
        for a, (ids, ticks, _) in enumerate(streams):
            srv.append(a, ids, ticks)
        st["server"] = srv
        return st
    ids, ticks, table = _single(case, seed)
    st["ids"], st["ticks"] = ctx.stream_tensors(ids, ticks)
    st["types"], st["theta"] = case["neurons"], _theta(case)
    if table is not None:
        st["cand"] = ctx.cand_tensors(table)
    if kind == "mine":
        st["mined"] = np.full(min(4_000_000, 80 * case["neurons"] ** 3), -1, np.int32)
        st["mined_end"] = st["mined"].size
    if kind == "resume":
        # what the program carries from the partitions before the last one
        start = int(np.searchsorted(ticks, ticks[-1] - int(case["part_s"] * TICKS_PER_S)))
        cnt = torch.zeros(table["M"], dtype=torch.int32, device="cuda")
        last = torch.full((table["M"],), -1, dtype=torch.int32, device="cuda")
        if start > 0:
            ctx.count_resume(st["ids"][:start], st["ticks"][:start], st["types"], st["cand"],
                             st["mode"], 0, cnt, last)
        st.update(start=start, cnt=cnt, last=last)
    torch.cuda.synchronize()
    return st


def run(st):
    case, ctx = st["case"], st["ctx"]
    kind = case["kind"]
    if kind == "count":
        return ctx.count(st["ids"], st["ticks"], st["types"], st["cand"], st["mode"])
    if kind == "two_pass":
        return list(ctx.count_two_pass(st["ids"], st["ticks"], st["types"], st["cand"],
                                       st["theta"]))
    if kind == "resume":
        # (copies, so that the same partition can be added again)
        cnt, last = st["cnt"].clone(), st["last"].clone()
        return list(ctx.count_resume(st["ids"], st["ticks"], st["types"], st["cand"], st["mode"],
                                     st["start"], cnt, last))
    if kind == "mine":
        levels = ctx.mine(st["ids"], st["ticks"], st["types"], HOPS[case["hops"]], st["theta"],
                          case["max_level"])
        return _collect(st, levels)
    if kind == "batch":
        b = st["batch"]
        b.run()
        return list(b.upper) + list(b.exact)
    srv = st["server"]
    tickets = [srv.submit(a, b, e, theta) for a, b, e, theta in st["reqs"]]
    out = [np.zeros((len(tickets), 3), np.int32)]
    for k, t in enumerate(tickets):
        r = srv.wait(t)
        out[0][k] = r["n_events"], r["n_survivors"], r["n_frequent"]
        out += [r["upper"], r["exact"]]
        srv.release(t)
    return out


def _collect(st, levels):
    """The mined levels in the program's own array: per level its numbers of
    candidates, survivors and frequent episodes, then every level's frequent
    set with its counts, one after the other; -1 behind them."""
    buf, end = st["mined"], 32
    head = buf[:32].reshape(8, 4)
    head[:] = -1
    for k, L in enumerate(levels):
        head[k] = L["level"], L["n_candidates"], L["n_survivors"], L["n_frequent"]
        for name in ("types", "lo", "hi", "upper", "exact"):
            a = L[name].reshape(-1)[:buf.size - end]
            buf[end:end + a.size] = a
            end += a.size
    buf[end:st["mined_end"]] = -1
    st["mined_end"] = end
    return buf


def work(case):
    """Bytes each input read once and each output written once; no floating
    point is done anywhere."""
    hop = 3 * case["n_max"] - 1  # types, len, lo, hi of one table row
    n = case["neurons"] * case["rate_hz"] * case["seconds"]
    M = case["episodes"]
    kind = case["kind"]
    if kind == "mine":
        # the stream in; the frequent pairs, at least, out
        return {"bytes": 8.0 * n + 16.0 * case["neurons"] ** 2, "flops": 0.0}
    if kind == "batch":
        # log-uniform means of 1e4..3e5 events and 1e3..M episodes
        n = case["recordings"] * 2.9e5 / math.log(30.0)
        lo = min(1000, M)
        M = case["recordings"] * ((M - lo) / math.log(M / lo) if M > lo else M)
        return {"bytes": 8.0 * n + (hop + 2) * 4.0 * M, "flops": 0.0}
    if kind == "serve":
        # windows of 59/ln(60) s on average over arrays of 64..neurons neurons
        n = case["requests"] * 14.4 * case["rate_hz"] * (64 + case["neurons"]) / 2
        return {"bytes": 8.0 * n + hop * 4.0 * M + 8.0 * M * case["requests"], "flops": 0.0}
    if kind == "resume":
        # the last partition, the table, and both carry arrays in and out
        n = case["neurons"] * case["rate_hz"] * case["part_s"]
        return {"bytes": 8.0 * n + (hop + 4) * 4.0 * M, "flops": 0.0}
    outs = 2 if kind == "two_pass" else 1
    return {"bytes": 8.0 * n + (hop + outs) * 4.0 * M, "flops": 0.0}


# ------------------------------------------------------------------ reference values
def _by_type(ids, ticks, neurons):
    order = np.argsort(ids, kind="stable").astype(np.int64)
    cut = np.searchsorted(ids[order], np.arange(neurons + 1))
    t64 = ticks.astype(np.int64)
    return [(t64[order[a:b]], order[a:b]) for a, b in zip(cut[:-1], cut[1:])]


def _count_one(ev, ty, lo, hi, relaxed):
    """Size of the largest set of non-overlapped occurrences, and the index of
    the last one's final event.  Each event of node k is chained to the newest
    event of node k-1 that its delay interval allows; the chain carries its
    first event's index; completions are taken greedily."""
    t, i = ev[ty[0]]
    s = i
    for k in range(1, len(ty)):
        tk, ik = ev[ty[k]]
        if relaxed:
            j = np.searchsorted(i, ik, "left") - 1
        else:
            j = np.searchsorted(t, tk - lo[k - 1] - 1, "right") - 1
        ok = j >= 0
        if t.size:
            ok &= t[np.maximum(j, 0)] >= tk - hi[k - 1]
            s = s[j[ok]]
        else:
            s = ik[:0]
        t, i = tk[ok], ik[ok]
    if len(ty) == 1:
        return t.size, int(i[-1]) if t.size else -1
    cnt, r = 0, -1
    p = 0
    while p < s.size:
        cnt, r = cnt + 1, int(i[p])
        p = int(np.searchsorted(s, r, "right"))
    return cnt, r


def _reference(ids, ticks, neurons, table, relaxed, keep=None):
    ev = _by_type(ids, ticks, neurons)
    out = np.full((2, table["M"]), -1, np.int64)
    for m in range(table["M"]):
        if keep is None or keep[m]:
            L = int(table["len"][m])
            out[:, m] = _count_one(ev, table["types"][m, :L], table["lo"][m, :L - 1].astype(np.int64),
                                   table["hi"][m, :L - 1].astype(np.int64), relaxed)
    return out


def exact(case, seed):
    """The same outputs from numpy alone, in 64-bit integers, for tables small
    enough to be counted one episode at a time."""
    kind = case["kind"]
    if kind not in ("count", "two_pass", "resume"):
        return None
    per = case["rate_hz"] * case["seconds"]  # events a node reads
    passes = 2 if kind == "two_pass" else 1
    cost = passes * case["episodes"] * case["n_max"] * (1.5e-5 + 5e-8 * per)
    if cost > 18.0 or case["lognormal"]:
        return None
    ids, ticks, table = _single(case, seed)
    if kind == "two_pass":
        up = _reference(ids, ticks, case["neurons"], table, True)[0]
        keep = up >= _theta(case)
        ex = _reference(ids, ticks, case["neurons"], table, False, keep)[0]
        return [up, ex, np.array([int(keep.sum())])]
    out = _reference(ids, ticks, case["neurons"], table, case["mode"] == "relaxed")
    return out[0] if kind == "count" else [out[0], out[1]]
