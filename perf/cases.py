"""The work that a program using this library has it do, as cases to time.

Every case goes through the public entry points (Context, Stream, Grains and
the call sequences of pipeline.py) on device tensors that the caller owns, on
one HIP stream of its own.  Six kinds of work:

  chain   one Call over one expansion level: expand, FIFO batch of the ready
          queue (entries sealed before dispatch masked out), FIFO batch of the
          sealed list, ordered gather of every report into parent slots.
  nested  two levels: expand, batch, expand, batch, gather, gather.
  stream  one expansion whose children turn terminal wave by wave: per wave a
          FIFO batch, the wave's reports, and the emission of every parent
          that is complete now; optionally with group failures and the Call's
          barrier.
  fence   Grain phases and the generation fence: reset, dispatch, commit with
          repeated and conflicting reports, retry and dispatch of the lost
          attempts, commit of their reports among stale ones.
  pbatch  parent-bound reservation of a whole ready queue.
  ops     filter and two-level broadcast over the lower level of a nested
          expansion.

Child counts are the quantiles of the named distribution at evenly spaced
probabilities, dealt to the parents in an order drawn from the seed, so that
the size of a case does not depend on the seed.  States, record lengths, ready
orders and record bytes are drawn from the seed on the GPU.  Byte outputs have
a capacity that does not depend on the seed either, a little over what the
records need.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_2609_18703_amd as R
from paper_2609_18703_amd import pipeline as PL

SUCCESS, FAILED, SKIPPED, PENDING, GROUP_FAILED = 0, 1, 2, 3, 4
DEV = "cuda"
MEAN_BYTES = {"fixed64": 64.0, "fixed1024": 1024.0, "lognormal": 645.0, "uniform1024": 528.0, "uniform512": 288.0}


# ------------------------------------------------------------------ the cases

def listed():
    return [
        # the smallest Call in use: a thousand parents with a handful of
        # children each and fixed 64-byte records; latency and launches
        {"name": "chain-7k", "kind": "chain", "parents": 1000, "fan": "lognormal", "records": "fixed64",
         "order": "random", "failed": 0.05, "skipped": 0.0, "batch": 64, "positions": False},
        # an ordinary Call of an odd size, with the optional position of every child asked for
        {"name": "chain-1m-positions", "kind": "chain", "parents": 2431, "fan": "zipf", "records": "lognormal",
         "order": "random", "failed": 0.03, "skipped": 0.02, "batch": 256, "positions": True},
        # workers that finish in order: reports arrive in the parents' order
        {"name": "chain-4m-in-order", "kind": "chain", "parents": 10007, "fan": "zipf", "records": "uniform512",
         "order": "canonical", "failed": 0.03, "skipped": 0.02, "batch": 256, "positions": False},
        # the long-tailed fan-out of the benchmark's default workload: 41M
        # children in random ready order, 25 GB of records
        {"name": "chain-41m", "kind": "chain", "parents": 100000, "fan": "zipf", "records": "lognormal",
         "order": "random", "failed": 0.03, "skipped": 0.02, "batch": 256, "positions": False},
        # documents -> pages -> regions, a small job of a serving loop
        {"name": "docs-200", "kind": "nested", "parents": 200, "shape": "docs", "failed": 0.0, "batch": 512},
        # the same at its full size: nothing fails, so the upper level works in place
        {"name": "docs-20k", "kind": "nested", "parents": 20000, "shape": "docs", "failed": 0.0, "batch": 512},
        # videos -> clips -> frames with failed frames: the upper level moves its bytes
        {"name": "videos-1k", "kind": "nested", "parents": 1000, "shape": "videos", "failed": 0.01, "batch": 1024},
        # streaming completion, 10M children under 500,000 parents over 50 waves
        {"name": "stream-10m", "kind": "stream", "parents": 500000, "children": 10000000, "waves": 50,
         "poisoned": 0, "batch": 1024},
        # streaming with group failures: a small document set whose largest
        # documents fail at their first page and have the rest suppressed
        {"name": "stream-45k-failures", "kind": "stream", "parents": 1885, "children": 45507, "waves": 24,
         "poisoned": 99, "batch": 48},
        # reservation and commit of a large Call with lost and repeated attempts
        {"name": "fence-10m", "kind": "fence", "parents": 24400, "batch": 256},
        # parent-bound reservation of a large ready queue
        {"name": "pbatch-10m", "kind": "pbatch", "parents": 24400, "batch": 256, "skipped": 0.02},
        # filter and broadcast over the regions of the documents
        {"name": "ops-2.7m", "kind": "ops", "parents": 20000},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["chain", "chain", "chain", "nested", "nested", "stream", "stream", "fence", "pbatch", "ops"])
    batch = rng.choice([48, 64, 100, 256, 512, 1024])
    if kind == "chain":
        fan = rng.choice(["zipf", "lognormal"])
        return {"kind": kind, "parents": _log(rng, 20, 100000) if fan == "zipf" else _log(rng, 1000, 3000000),
                "fan": fan, "records": rng.choice(["fixed64", "lognormal", "uniform512", "uniform1024"]),
                "order": rng.choice(["random", "random", "canonical"]), "failed": rng.choice([0.0, 0.01, 0.03, 0.05]),
                "skipped": rng.choice([0.0, 0.02, 0.1]), "batch": batch, "positions": rng.random() < 0.3}
    if kind == "nested":
        shape = rng.choice(["docs", "videos"])
        return {"kind": kind, "parents": _log(rng, 100, 40000) if shape == "docs" else _log(rng, 10, 1000),
                "shape": shape, "failed": rng.choice([0.0, 0.001, 0.01]), "batch": batch}
    if kind == "stream":
        failures = rng.random() < 0.4
        parents = _log(rng, 500, 20000) if failures else _log(rng, 1000, 500000)
        return {"kind": kind, "parents": parents, "children": int(parents * rng.uniform(8, 24)),
                "waves": rng.randint(5, 50), "poisoned": max(1, parents // 20) if failures else 0, "batch": batch}
    if kind == "fence":
        return {"kind": kind, "parents": _log(rng, 250, 24400), "batch": batch}
    if kind == "pbatch":
        return {"kind": kind, "parents": _log(rng, 250, 24400), "batch": batch,
                "skipped": rng.choice([0.0, 0.02, 0.3])}
    return {"kind": kind, "parents": _log(rng, 400, 60000)}


# ------------------------------------------------------------------ child counts

@functools.lru_cache(maxsize=32)
def _quantiles(fan, n):
    """Counts at the probabilities (i + 1/2) / n of the distribution."""
    u = (np.arange(n) + 0.5) / n
    if fan == "zipf":                    # Zipf(1.2) truncated to [1, 10^4]
        cdf = np.cumsum(np.arange(1, 10001, dtype=np.float64) ** -1.2)
        k = 1 + np.minimum(np.searchsorted(cdf / cdf[-1], u, side="right"), 9999)
    elif fan in ("lognormal", "pages"):  # LN(1.5, 1) clipped to [1, 500]; pages LN(2.3, 0.9) in [1, 2000]
        z = torch.special.ndtri(torch.from_numpy(u)).numpy()
        k = np.clip(np.rint(np.exp(1.5 + z)), 1, 500) if fan == "lognormal" else \
            np.clip(np.rint(np.exp(2.3 + 0.9 * z)), 1, 2000)
    elif fan == "regions":               # Poisson(8) + 1
        cdf = np.cumsum(np.exp([i * math.log(8.0) - 8.0 - math.lgamma(i + 1) for i in range(40)]))
        k = 1 + np.searchsorted(cdf, u * cdf[-1], side="right")
    elif fan == "frames":                # uniform in [16, 300]
        k = 16 + np.floor(285 * u)
    else:                                # clips: Pareto(1.1, x_min 5) clipped to [1, 50000]
        k = np.clip(np.rint(5.0 * (1.0 - u) ** (-1 / 1.1)), 1, 50000)
    return k.astype(np.int64)


@functools.lru_cache(maxsize=8)
def _rank_counts(n_parents, n_children, s, hi):
    """clip(rint(C r^-s), 1, hi) over the ranks, summing to n_children."""
    w = np.arange(1, n_parents + 1, dtype=np.float64) ** -s
    lo_c, hi_c = 0.0, float(n_children) / w[-1] + 1.0
    for _ in range(70):
        mid = 0.5 * (lo_c + hi_c)
        if int(np.clip(np.rint(mid * w), 1, hi).sum()) <= n_children:
            lo_c = mid
        else:
            hi_c = mid
    k = np.clip(np.rint(lo_c * w), 1, hi).astype(np.int64)
    left = n_children - int(k.sum())
    if left > 0:
        k[np.nonzero(k < hi)[0][:left]] += 1
    return k


def _counts(case):
    """The case's top-level child counts in no particular order (host)."""
    if case["kind"] == "stream":
        s, hi = (1.0, 427) if case["poisoned"] else (1.1, 100000)
        return _rank_counts(case["parents"], case["children"], s, hi)
    if case["kind"] == "ops":
        return _quantiles("pages", case["parents"])
    if case["kind"] == "nested":
        return _quantiles("pages" if case["shape"] == "docs" else "clips", case["parents"])
    return _quantiles(case.get("fan", "zipf"), case["parents"])


# ------------------------------------------------------------------ seeded inputs

@functools.lru_cache(maxsize=1)
def _stream():
    return torch.cuda.Stream()


def _rng(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _dealt(counts, g):
    k = torch.from_numpy(counts).to(DEV)
    return k[torch.randperm(k.numel(), generator=g, device=DEV)]


def _offsets(counts):
    o = torch.zeros(counts.numel() + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(counts, 0, out=o[1:])
    return o


def _states(n, failed, skipped, g):
    u = torch.rand(n, generator=g, device=DEV)
    st = torch.zeros(n, dtype=torch.uint8, device=DEV)
    st[u < failed] = FAILED
    st[(u >= failed) & (u < failed + skipped)] = SKIPPED
    return st


def _lengths(kind, n, g):
    if kind.startswith("fixed"):
        return torch.full((n,), int(kind[5:]), dtype=torch.int64, device=DEV)
    if kind == "lognormal":              # LN(6, 1) clipped to [16, 4096]
        return torch.randn(n, generator=g, device=DEV).add_(6.0).exp_().round_().clamp_(16, 4096).to(torch.int64)
    lo, hi = {"uniform1024": (32, 1024), "uniform512": (64, 512)}[kind]
    return torch.randint(lo, hi + 1, (n,), generator=g, device=DEV, dtype=torch.int64)


def _bytes(n, g):
    """n random bytes."""
    w = torch.empty((n + 7) // 8 + 1, dtype=torch.int64, device=DEV)
    w.random_(generator=g)
    return w.view(torch.uint8)[:max(n, 1)]


def _room(n, kind, live=1.0):
    """Capacity for the bytes of the successful ones of n records: their mean
    and eight standard deviations."""
    return int(n * live * MEAN_BYTES[kind] + 8 * 1000.0 * math.sqrt(n)) + 4096


def _some(n, share, g):
    """A mask of round(n * share) random entries."""
    m = torch.zeros(n, dtype=torch.bool, device=DEV)
    m[torch.randperm(n, generator=g, device=DEV)[:int(round(n * share))]] = True
    return m


def _ready_order(n, order, g):
    if order == "canonical":
        return torch.arange(n, device=DEV)
    return torch.randperm(n, generator=g, device=DEV)


def _report_columns(order, states, lengths):
    """State and Arrow-style offsets of one report per child of `order`; only
    a successful report carries bytes."""
    st = states[order]
    ln = torch.where(st == SUCCESS, lengths[order], 0)
    return st, _offsets(ln)


def _i32(t):
    return t.to(torch.int32)


def _zeros(n, dtype):
    return torch.zeros(max(int(n), 1), dtype=dtype, device=DEV)


def _pieces(t, most=1 << 32):
    """A large byte buffer as consecutive pieces."""
    return [t] if t.numel() <= most else list(torch.split(t, most))


# ------------------------------------------------------------------ prepare

def prepare(case, seed):
    with torch.cuda.stream(_stream()):
        state = _PREPARE[case["kind"]](case, _rng(seed))
        torch.cuda.synchronize()
    return state


def run(state):
    return state["run"](state)


def _prepare_chain(case, g):
    counts = _dealt(_counts(case), g)
    n, p = int(counts.sum()), counts.numel()
    states = _states(n, case["failed"], case["skipped"], g)
    lengths = _lengths(case["records"], n, g)
    queue = _ready_order(n, case["order"], g)
    keep = states[queue] != SKIPPED
    sealed = queue[~keep]
    st, off = _report_columns(torch.cat([queue[keep], sealed]), states, lengths)
    b = PL.SingleLevelBuffers(_i32(counts), _i32(queue), keep.to(torch.uint8), _i32(sealed), st, off,
                              _bytes(int(off[-1]), g), n, n - sealed.numel(), case["batch"],
                              out_cap=_room(n, case["records"], 1 - case["failed"] - case["skipped"]))
    b.out_data.zero_()
    ctx = R.Context(_stream())
    ctx.reserve(n, p, n)
    return {"run": _run_chain, "ctx": ctx, "b": b, "pos": _zeros(n + 1, torch.int64) if case["positions"] else None}


def _run_chain(s):
    ctx, b = s["ctx"], s["b"]
    if s["pos"] is None:
        PL.single_level(ctx, b)
    else:
        n, m = b.N, b.M
        ctx.expand(b.counts, b.offsets, b.child_parent, b.child_ordinal)
        ctx.batch(b.queue, b.keep, b.offsets, b.B, None, b.rep_parent, b.rep_ordinal, b.scalars[0:1],
                  b.scalars[1:2], out_cap=m)
        if n > m:
            ctx.batch(b.sealed_ids, None, b.offsets, b.B, None, b.rep_parent[m:], b.rep_ordinal[m:],
                      b.scalars[2:3], b.scalars[3:4], q_len=n - m, out_cap=n - m)
        ctx.gather(b.rep_parent, b.rep_ordinal, b.rep_state, b.rep_off, b.data, b.offsets, b.out_off, b.out_data,
                   b.n_success, b.n_failed, b.n_skipped, b.complete, b.parent_state, n=n, out_cap=b.out_cap,
                   child_dst_off=s["pos"])
    return {"offsets": b.offsets, "child": [b.child_parent, b.child_ordinal], "tags": [b.rep_parent, b.rep_ordinal],
            "scalars": b.scalars, "slots": b.out_off, "data": _pieces(b.out_data),
            "counts": [b.n_success, b.n_failed, b.n_skipped], "complete": b.complete, "state": b.parent_state,
            "positions": s["pos"]}


def _nested_counts(case, counts1, g):
    """Second-level counts of every first-level child."""
    fan = "regions" if case.get("shape", "docs") == "docs" else "frames"
    return _dealt(_quantiles(fan, int(counts1.sum())), g)


def _prepare_nested(case, g):
    counts1 = _dealt(_counts(case), g)
    counts2 = _nested_counts(case, counts1, g)
    n1, n2, p1 = counts2.numel(), int(counts2.sum()), counts1.numel()
    states = _states(n2, case["failed"], 0.0, g)
    records = "uniform1024" if case["shape"] == "docs" else "fixed1024"
    lengths = _lengths(records, n2, g)
    queue1, queue2 = _ready_order(n1, "random", g), _ready_order(n2, "random", g)
    st, off = _report_columns(queue2, states, lengths)
    b = PL.NestedBuffers(_i32(counts1), _i32(queue1), case["batch"], _i32(counts2), _i32(queue2), case["batch"], st,
                         off, _bytes(int(off[-1]), g), n1, n2, want_data=False)
    # nothing fails: the upper level's slots are the lower ones as they lie
    b.cap = _room(n2, records, 1 - case["failed"])
    b.mid_data = _zeros(b.cap, torch.uint8)
    b.top_data = b.mid_data if case["failed"] == 0.0 else _zeros(b.cap, torch.uint8)
    ctx = R.Context(_stream())
    ctx.reserve(n2, max(n1, p1), n2)
    return {"run": _run_nested, "ctx": ctx, "b": b}


def _run_nested(s):
    b = s["b"]
    PL.nested(s["ctx"], b)
    return {"offsets": [b.offsets1, b.offsets2], "mid": [b.mid_parent, b.mid_ordinal, b.b1_parent, b.b1_ordinal],
            "leaf": [b.leaf_parent, b.leaf_ordinal, b.b2_parent, b.b2_ordinal], "scalars": b.scalars,
            "mid_slots": b.mid_off, "mid_data": _pieces(b.mid_data), "mid_counts": b.mid_cnt,
            "mid_state": [b.mid_complete, b.mid_state], "top_slots": b.top_off,
            "top_data": _pieces(b.top_data) if b.top_data is not b.mid_data else None, "top_counts": b.top_cnt,
            "top_state": [b.top_complete, b.top_state]}


def _prepare_stream(case, g):
    ranked = torch.from_numpy(_counts(case)).to(DEV)
    p, n, waves = ranked.numel(), case["children"], case["waves"]
    place = torch.randperm(p, generator=g, device=DEV)     # rank r's counts go to parent place[r]
    counts = torch.empty_like(ranked)
    counts[place] = ranked
    offsets = _offsets(counts)
    parent = torch.repeat_interleave(torch.arange(p, device=DEV), counts)
    states = _states(n, 0.0, 0.0, g)
    lengths = _lengths("uniform512", n, g)
    at = torch.randperm(n, generator=g, device=DEV)        # ready position of every child
    if case["poisoned"]:
        # a parent's children become ready in order; the largest parents fail at their first
        at = at[torch.argsort(parent * n + at)]
        states[offsets[place[:case["poisoned"]]]] = GROUP_FAILED
    queue = torch.argsort(at)
    st, off = _report_columns(queue, states, lengths)
    edges = [w * n // waves for w in range(waves + 1)]
    # what each wave can emit, which sizes its buffers: a parent is done in the
    # wave of its last child or of its group failure, with the bytes
    # committed until then
    wave_of = torch.bucketize(at, torch.tensor(edges[1:-1], device=DEV), right=True)
    done = torch.zeros(p, dtype=torch.int64, device=DEV).scatter_reduce_(0, parent, wave_of, "amax")
    stop = torch.full((p,), n, dtype=torch.int64, device=DEV)
    if case["poisoned"]:
        bad = torch.nonzero(states == GROUP_FAILED).flatten()
        stop[parent[bad]] = at[bad]
        done[parent[bad]] = wave_of[bad]
    kept = torch.where((states == SUCCESS) & (at < stop[parent]), lengths, 0)
    size = torch.zeros(p, dtype=torch.int64, device=DEV).index_add_(0, parent, kept)
    n_emit = torch.bincount(done, minlength=waves).tolist()
    n_bytes = torch.zeros(waves, dtype=torch.int64, device=DEV).index_add_(0, done, size).tolist()
    starts = [0]
    for x in n_bytes:
        starts.append(starts[-1] + -(-x // 256) * 256)
    scalars, tags = _zeros(4 * waves, torch.int64), [_zeros(n, torch.int32) for _ in range(2)]
    out = {"parent": _zeros(p, torch.int32), "slots": _zeros(p + waves, torch.int64),
           "data": _zeros(_room(n, "uniform512") + 256 * waves, torch.uint8), "counts": [_zeros(p, torch.int32) for _ in range(3)],
           "state": _zeros(p, torch.uint8), "tags": tags, "scalars": scalars,
           "offsets": _zeros(p + 1, torch.int64)}
    late = [(_i32(parent[queue]), _i32(queue - offsets[parent[queue]]))] if case["poisoned"] else None
    steps, e = [], 0
    for w in range(waves):
        a, z, m = edges[w], edges[w + 1], n_emit[w]
        steps.append({
            "n": z - a, "queue": _i32(queue[a:z]), "state": st[a:z].clone(), "off": off[a:z + 1].clone(),
            "tags": [t[a:z] for t in tags],
            # with failures in flight the reports are of entries dispatched
            # earlier, some of them of parents barred since
            "report": [late[0][0][a:z].clone(), late[0][1][a:z].clone()] if late else [t[a:z] for t in tags],
            "scalars": [scalars[4 * w + k:4 * w + k + 1] for k in range(4)],
            "parent": out["parent"][e:e + m], "slots": out["slots"][e + w:e + w + m + 1],
            "data": out["data"][starts[w]:starts[w] + n_bytes[w]], "cap": (m, n_bytes[w]),
            "counts": [t[e:e + m] for t in out["counts"]], "parent_state": out["state"][e:e + m]})
        e += m
    ctx = R.Context(_stream())
    ctx.reserve(n, p, max(s["n"] for s in steps))
    k32 = _i32(counts)
    ctx.expand(k32, out["offsets"])
    barrier = _zeros(p, torch.uint8) if case["poisoned"] else None
    return {"run": _run_stream, "ctx": ctx, "counts": k32, "st": ctx.stream(out["offsets"], n, barrier), "steps": steps,
            "data": _bytes(int(off[-1]), g), "out": out, "B": case["batch"], "barrier": barrier}


def _run_stream(s):
    ctx, st, out, data = s["ctx"], s["st"], s["out"], s["data"]
    ctx.expand(s["counts"], out["offsets"])
    st.reset()
    for w in s["steps"]:
        sc, n = w["scalars"], w["n"]
        st.batch(w["queue"], None, s["B"], None, w["tags"][0], w["tags"][1], sc[0], sc[1], q_len=n, out_cap=n)
        st.report(w["report"][0], w["report"][1], w["state"], w["off"], data, n=n)
        st.emit(w["parent"], w["slots"], w["data"], w["counts"][0], w["counts"][1], w["counts"][2],
                w["parent_state"], sc[2], sc[3], cap_parents=w["cap"][0], cap_bytes=w["cap"][1])
    return {"out": out, "barrier": s["barrier"]}


def _prepare_fence(case, g):
    counts = _dealt(_counts(case), g)
    offsets = _offsets(counts)
    n, p = int(counts.sum()), counts.numel()
    parent = torch.repeat_interleave(torch.arange(p, device=DEV), counts)
    states, lengths = _states(n, 0.03, 0.0, g), _lengths("lognormal", n, g)
    queue = _ready_order(n, "random", g)
    gone = _some(n, 0.02, g)
    lost, arrived = queue[gone], queue[~gone]
    # first copies in dispatch order, then 1% identical and 0.2% conflicting
    # repeats; half the conflicts have another state, half other bytes
    na = arrived.numel()
    first_of = torch.randperm(na, generator=g, device=DEV)[:int(round(0.012 * na))]
    rep = arrived[first_of]
    child = torch.cat([arrived, rep])
    st, off = _report_columns(child, states, lengths)
    mix = torch.rand(rep.numel(), generator=g, device=DEV) * 12
    flip = torch.nonzero(mix < 1).flatten()
    ident = torch.nonzero(mix >= 2).flatten()
    st[na + flip] = torch.where(states[rep[flip]] == FAILED, SKIPPED, FAILED).to(torch.uint8)
    data = _bytes(int(off[-1]), g)
    # an identical repeat has its first copy's bytes
    src, dst = off[:-1][first_of[ident]], off[:-1][na + ident]
    ln = off[1:][na + ident] - dst
    idx = torch.repeat_interleave(torch.arange(ident.numel(), device=DEV), ln)
    if idx.numel():
        within = torch.arange(idx.numel(), device=DEV) - (torch.cumsum(ln, 0) - ln)[idx]
        data[dst[idx] + within] = data[src[idx] + within]
    # second attempt: the lost children at generation 1 among stale
    # generation-0 reports of half of them
    stale = lost[_some(lost.numel(), 0.5, g)]
    mix = torch.randperm(lost.numel() + stale.numel(), generator=g, device=DEV)
    child1 = torch.cat([lost, stale])[mix]
    gen1 = torch.cat([torch.ones_like(lost), torch.zeros_like(stale)])[mix]
    st1, off1 = _report_columns(child1, states, lengths)

    def call(children, st_, off_, gen, bytes_):
        par = parent[children]
        return {"parent": _i32(par), "ordinal": _i32(children - offsets[par]), "state": st_, "off": off_,
                "gen": _i32(gen), "data": bytes_, "n": children.numel(),
                "out": _zeros(children.numel(), torch.uint8), "counts": _zeros(4, torch.int64)}

    ctx = R.Context(_stream())
    return {"run": _run_fence, "ctx": ctx, "grains": ctx.grains(n), "offsets": offsets, "queue": _i32(queue),
            "lost": _i32(lost), "gen": [_zeros(n, torch.int32), _zeros(lost.numel(), torch.int32)],
            "calls": [call(child, st, off, torch.zeros_like(child), data),
                      call(child1, st1, off1, gen1, _bytes(int(off1[-1]), g))]}


def _run_fence(s):
    gr = s["grains"]

    def commit(c):
        gr.commit(c["parent"], c["ordinal"], c["state"], c["off"], c["data"], c["gen"], s["offsets"], c["out"],
                  c["counts"], n=c["n"])

    gr.reset()
    gr.dispatch(s["queue"], s["gen"][0])
    commit(s["calls"][0])
    gr.retry(s["lost"])
    gr.dispatch(s["lost"], s["gen"][1], n=s["lost"].numel())
    commit(s["calls"][1])
    return {"generation": s["gen"], "outcome": [c["out"] for c in s["calls"]],
            "counts": [c["counts"] for c in s["calls"]]}


def _prepare_pbatch(case, g):
    counts = _dealt(_counts(case), g)
    offsets = _offsets(counts)
    n, p = int(counts.sum()), counts.numel()
    queue = _ready_order(n, "random", g)
    keep = ~_some(n, case["skipped"], g)
    m, nb = int(keep.sum()), int(((counts + case["batch"] - 1) // case["batch"]).sum())
    ctx = R.Context(_stream())
    ctx.reserve(n, p, n)
    return {"run": _run_pbatch, "ctx": ctx, "queue": _i32(queue), "keep": keep.to(torch.uint8), "offsets": offsets,
            "B": case["batch"], "child": _zeros(m, torch.int32), "parent": _zeros(m, torch.int32),
            "ordinal": _zeros(m, torch.int32), "batches": _zeros(nb + 1, torch.int64),
            "scalars": _zeros(2, torch.int64)}


def _run_pbatch(s):
    s["ctx"].batch_parent(s["queue"], s["keep"], s["offsets"], s["B"], s["batches"], s["child"], s["parent"],
                          s["ordinal"], s["scalars"][0:1], s["scalars"][1:2])
    return [s["child"], s["parent"], s["ordinal"], s["batches"], s["scalars"]]


def _prepare_ops(case, g):
    counts1 = _dealt(_counts(case), g)
    counts2 = _nested_counts(case, counts1, g)
    p, n1, n = counts1.numel(), counts2.numel(), int(counts2.sum())
    mix = torch.tensor([0, 0, 0, FAILED, SKIPPED, PENDING], dtype=torch.uint8, device=DEV)

    def some(k):
        return mix[torch.randint(0, 6, (k,), generator=g, device=DEV)]

    maps = [_i32(torch.repeat_interleave(torch.arange(k.numel(), device=DEV), k)) for k in (counts2, counts1)]
    return {"run": _run_ops, "ctx": R.Context(_stream()), "maps": maps, "x": some(n), "mask_state": some(n),
            "mask": (torch.rand(n, generator=g, device=DEV) < 0.5).to(torch.uint8), "top": some(p), "like": some(n),
            "filtered": _zeros(n, torch.uint8), "state": _zeros(n, torch.uint8), "ancestor": _zeros(n, torch.int32)}


def _run_ops(s):
    s["ctx"].filter(s["x"], s["mask"], s["filtered"], mask_state=s["mask_state"])
    s["ctx"].broadcast(s["maps"], s["top"], s["state"], s["ancestor"], s["like"])
    return [s["filtered"], s["state"], s["ancestor"]]


_PREPARE = {"chain": _prepare_chain, "nested": _prepare_nested, "stream": _prepare_stream, "fence": _prepare_fence,
            "pbatch": _prepare_pbatch, "ops": _prepare_ops}


# ------------------------------------------------------------------ work and tolerance

def _expand_bytes(p, n):
    return 4 * p + 8 * p + 8 * n                          # counts in; offsets and both lineage keys out


def _gather_bytes(p, n, payload):
    # tags, state and offsets in; slot offsets, counts and states out; the bytes in and out
    return 17 * n + 8 * p + 8 * p + 14 * p + 2 * payload


def work(case):
    """Each input read once and each output written once."""
    top = _counts(case)
    p, n, kind = len(top), int(top.sum()), case["kind"]
    if kind == "chain":
        live = 1.0 - case["failed"] - case["skipped"]
        by = _expand_bytes(p, n) + 5 * n + 12 * case["skipped"] * n + 8 * (1 - case["skipped"]) * n
        by += _gather_bytes(p, n, live * n * MEAN_BYTES[case["records"]]) + (8 * n if case["positions"] else 0)
    elif kind == "nested":
        leaves = n * (9 if case["shape"] == "docs" else 158)
        per, k = (MEAN_BYTES["uniform1024"], 9) if case["shape"] == "docs" else (1024.0, 158)
        low = (1 - case["failed"]) * leaves * per
        up = 0.0 if case["failed"] == 0.0 else (1 - case["failed"]) ** k * leaves * per
        by = _expand_bytes(p, n) + _expand_bytes(n, leaves) + 12 * n + 12 * leaves
        by += _gather_bytes(n, leaves, low) + _gather_bytes(p, n, up)
    elif kind == "stream":
        by = 12 * p + 12 * n + 17 * n + 2 * n * MEAN_BYTES["uniform512"] + (4 + 8 + 12 + 1) * p
    elif kind == "fence":
        repeats = 0.011 * n * 0.97
        by = 8 * n + 21 * n * 1.012 + 1 * n * 1.012 + 2 * repeats * MEAN_BYTES["lognormal"] + 16 * p
        by += 0.02 * n * (4 + 8) + 0.03 * n * 22
    elif kind == "pbatch":
        by = 5 * n + 12 * n * (1 - case["skipped"]) + 8 * p
    else:
        leaves = 9 * n
        by = 4 * leaves + (4 + 1 + 4 + 1) * leaves + 4 * n + p
    return {"bytes": float(by), "flops": 0.0}


def tolerance(case):
    """Every output is a whole number or a byte."""
    return "exact"
