"""GPU parity at the sizes where a kernel changes tile, group, unit or path,
bit-exact against the CPU oracle."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle as O  # noqa: E402
from workloads import device as D  # noqa: E402


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_18703_amd as R
    c = R.Context()
    c.reserve(1 << 21, 1 << 18, 1 << 21)
    yield c
    c.close()


def _i32(a):
    return D.to_dev(np.ascontiguousarray(a).view(np.int32))


def _zeros(n, dtype):
    return torch.zeros(max(int(n), 1), dtype=dtype, device="cuda")


def _reports(counts, lengths, states, order, lead=0, seed=0):
    """Host report columns for children in `order` (bytes only where SUCCESS)."""
    counts = np.asarray(counts, np.int64)
    parent = np.repeat(np.arange(len(counts)), counts)
    ordinal = np.arange(len(parent)) - np.repeat(np.cumsum(counts) - counts, counts)
    ln = np.where(states[order] == O.SUCCESS, lengths[order], 0).astype(np.int64)
    off = np.concatenate([[lead], lead + np.cumsum(ln)]).astype(np.int64)
    data = np.random.default_rng(seed + 99).integers(0, 256, int(off[-1]) + 1).astype(np.uint8)
    return parent[order].astype(np.uint32), ordinal[order].astype(np.uint32), states[order].astype(np.uint8), off, data


def _gather_case(ctx, counts, lengths, states, order, mis=0, lead=0):
    rp, ro, rs, off, data = _reports(counts, lengths, states, order, lead)
    offs = O.expand(np.asarray(counts, np.int32), tags=False)
    want = O.gather(rp, ro, rs, off, data, offs)
    P, N, total = len(counts), int(offs[-1]), int(want["out_off"][-1])
    out = torch.full((mis + max(total, 1) + 64,), 0xA5, dtype=torch.uint8, device="cuda")
    oo, cdst = _zeros(P + 1, torch.int64), _zeros(N + 1, torch.int64)
    ns, nf, nk = (_zeros(P, torch.int32) for _ in range(3))
    comp, pst = _zeros(P, torch.uint8), _zeros(P, torch.uint8)
    ctx.gather(_i32(rp), _i32(ro), D.to_dev(rs), D.to_dev(off), D.to_dev(data), D.to_dev(offs), oo, out[mis:],
               ns, nf, nk, comp, pst, n=len(rp), out_cap=total, child_dst_off=cdst)
    ctx.check("gather")
    assert np.array_equal(oo.cpu().numpy(), want["out_off"])
    for t, k in ((ns, "n_success"), (nf, "n_failed"), (nk, "n_skipped"), (comp, "complete"), (pst, "parent_state")):
        assert np.array_equal(t.cpu().numpy()[:P], want[k]), k
    host = out.cpu().numpy()
    assert np.array_equal(host[mis:mis + total], want["out_data"])
    assert (host[:mis] == 0xA5).all() and (host[mis + total:] == 0xA5).all()
    ln = np.zeros(N, np.int64)
    ln[order] = np.diff(off)
    assert np.array_equal(cdst.cpu().numpy(), np.concatenate([[0], np.cumsum(ln)]))


# children around a group of 64, a window of 256, a scan tile and several tiles
@pytest.mark.parametrize("n", [1, 63, 64, 65, 255, 256, 257, 1023, 1024, 1025, 4095, 4096, 4097, 20_011])
@pytest.mark.parametrize("record", ["tiny", "mixed", "large"])
def test_gather_groups_and_units(ctx, n, record):
    """Copy units from 1 KiB up to many per wave, cut anywhere in a record."""
    rng = np.random.default_rng(n)
    counts = []
    left = n
    while left > 0:
        k = int(min(left, rng.choice([0, 0, 1, 2, 3, 7, 40, 700])))
        counts.append(k)
        left -= k
    counts += [0, 0]
    hi = {"tiny": 5, "mixed": 900, "large": min(9000, 40_000_000 // n)}[record]
    lengths = rng.integers(0, hi + 1, n)
    states = rng.choice([O.SUCCESS] * 8 + [O.FAILED, O.SKIPPED], n).astype(np.uint8)
    for mis, order in ((0, rng.permutation(n)), (5, np.arange(n)), (15, rng.permutation(n))):
        _say("gather", n, record, mis)
        _gather_case(ctx, counts, lengths, states, order, mis=mis, lead=mis % 7)


# both scan tile sizes (up to 262,144 children tiles of 1,024, beyond tiles of
# 8,192), whole and ragged last tiles, parents over several tiles, empty parents
# at tile boundaries, reports missing, few reports of many children
@pytest.mark.parametrize("n, missing", [(8192, 0), (8193, 9), (131_072, 0), (131_073, 0), (139_264, 0), (139_265, 50),
                                        (150_000, 149_000), (262_144, 0), (262_145, 0), (262_145, 262_000),
                                        (300_001, 0), (1_000_003, 999_000)])
def test_gather_scan_tiles(ctx, n, missing):
    rng = np.random.default_rng(n + missing)
    counts = [0, 0, min(n // 3, 100_000), 0]
    left = n - sum(counts)
    first = 8192 - sum(counts) % 8192          # the next parents end exactly on a tile boundary
    if first < left:
        counts += [first, 0, 0, 0]
        left -= first
    while left > 0:
        k = int(min(left, rng.choice([0, 1, 1, 2, 5, 9, 64, 3000])))
        counts.append(k)
        left -= k
    counts += [0] * 5
    lengths = rng.integers(0, 20, n)
    states = rng.choice([O.SUCCESS] * 6 + [O.FAILED, O.SKIPPED], n).astype(np.uint8)
    order = rng.permutation(n)[:n - missing]
    _say("gather scan", n, missing)
    _gather_case(ctx, counts, lengths, states, order)


# A scan that follows an error runs no tiles, and its last workgroup still
# settles the call: every wave has to leave by the same way (one workgroup, a
# few, and more than one per CU, at both tile sizes).
@pytest.mark.parametrize("n", [500, 5000, 131_072, 131_073, 400_000])
def test_gather_after_an_error_runs_no_tiles(ctx, n):
    import paper_2609_18703_amd as R
    counts = np.full(n // 100 + 1, 100)
    counts[-1] = n - 100 * (n // 100)
    order = np.random.default_rng(n).permutation(n)
    lengths, states = np.full(n, 3), np.zeros(n, np.uint8)
    rp, ro, rs, off, data = _reports(counts, lengths, states, order)
    offs = D.to_dev(O.expand(counts.astype(np.int32), tags=False))
    cols = (_i32(rp), _i32(ro), D.to_dev(rs), D.to_dev(off), D.to_dev(data), offs)
    bad = rp.copy()
    bad[n // 2] = len(counts)                              # no such parent
    for k in range(20):
        _say("gather after an error", n, k)
        out = torch.full((3 * n,), 0xA5, dtype=torch.uint8, device="cuda")
        ctx.gather(_i32(bad), *cols[1:], _zeros(len(counts) + 1, torch.int64), out)
        ctx.gather(*cols, _zeros(len(counts) + 1, torch.int64), out)      # the error is still recorded
        assert ctx.status() == R.ERANGE
        assert bool((out == 0xA5).all())
    _gather_case(ctx, counts, lengths, states, order)


def _batch_case(ctx, counts, queue, keep, barrier, B):
    offs = O.expand(np.asarray(counts, np.int32), tags=False)
    P, Q = len(counts), len(queue)
    want = O.batch(queue, keep, offs, B, barrier=barrier)
    m = len(want[0])
    outs = [torch.full((Q + 3,), -1, dtype=torch.int32, device="cuda") for _ in range(3)]
    sc = _zeros(2, torch.int64)
    ctx.batch(_i32(queue), None if keep is None else D.to_dev(keep), D.to_dev(offs), B, *outs, sc[0:1], sc[1:2], q_len=Q,
              out_cap=Q, barrier=None if barrier is None else D.to_dev(barrier))
    ctx.check("batch")
    assert sc.tolist() == [m, len(want[3])]
    for t, w in zip(outs, want[:3]):
        h = t.cpu().numpy().view(np.uint32)
        assert np.array_equal(h[:m], w) and (h[m:] == 0xffffffff).all()


# queue sizes on both sides of every path (offsets searched, tiles of 1,024,
# tiles of 4,096, counted first); the reservation decides between the
# map of 64-child masks and the coarse one, or leaves children past the map
@pytest.mark.parametrize("q_len", [1023, 65_536, 65_537, 262_144, 262_145, 1_048_576, 1_048_577])
@pytest.mark.parametrize("reserve", [1000, 1 << 21, 13 << 20])
def test_batch_paths(q_len, reserve):
    import paper_2609_18703_amd as R
    rng = np.random.default_rng(q_len + reserve)
    n = q_len + 777
    pool = np.concatenate([rng.integers(0, 4, n // 3), rng.choice([0, 0, 0, 1, 64, 65, 200], n // 100),
                           [0, 5000, 0, 0, 1, 0]])
    rng.shuffle(pool)
    counts = pool[:np.searchsorted(np.cumsum(pool), n)].astype(np.int64)
    counts = np.concatenate([counts, [n - counts.sum()], [0, 0]])
    queue = rng.permutation(n)[:q_len].astype(np.uint32)
    keep = (rng.random(q_len) < 0.8).astype(np.uint8)
    barrier = (rng.random(len(counts)) < 0.1).astype(np.uint8)
    c = R.Context()
    c.reserve(reserve, len(counts), q_len)
    for k, bar in ((None, None), (keep, None), (None, barrier), (keep, barrier)):
        _say("batch paths", q_len, reserve, k is not None, bar is not None)
        _batch_case(c, counts, queue, k, bar, 256)
    c.close()


# counted queues: one tile past a group of 16 tiles, a ragged tail, arrays off
# their 16-byte alignment, mask bytes other than 1, room for a part only
@pytest.mark.parametrize("q_len", [(1 << 20) + 1, (1 << 20) + 65_536, (1 << 20) + 3 * 65_536 + 4095])
@pytest.mark.parametrize("shift", [0, 1])
def test_batch_counted(ctx, q_len, shift):
    import paper_2609_18703_amd as R
    rng = np.random.default_rng(q_len)
    offs = O.expand(np.array([3, 0, q_len - 1000, 997], np.int32), tags=False)
    queue = rng.permutation(q_len).astype(np.uint32)
    keep = rng.choice(np.array([0, 1, 0x7f, 0x80, 0xff], np.uint8), q_len)
    keep[4096:8192] = 0
    _say("batch counted", q_len, shift)
    want = O.batch(queue, keep, offs, 48)
    m = len(want[0])
    q = _i32(np.concatenate([np.zeros(shift, np.uint32), queue]))[shift:]
    k = D.to_dev(np.concatenate([np.zeros(shift, np.uint8), keep]))[shift:]
    for cap in (m, m - 1):
        outs = [torch.full((m + 8 + shift,), -1, dtype=torch.int32, device="cuda")[shift:] for _ in range(3)]
        sc = _zeros(2, torch.int64)
        ctx.batch(q, k, D.to_dev(offs), 48, *outs, sc[0:1], sc[1:2], q_len=q_len, out_cap=cap)
        assert ctx.status() == (R.OK if cap == m else R.ECAP)
        assert sc.tolist() == [m, len(want[3])]
        for t, w in zip(outs, want[:3]):
            h = t.cpu().numpy().view(np.uint32)
            assert np.array_equal(h[:cap], w[:cap]) and (h[cap:] == 0xffffffff).all()


# Counted queues over a coarse map whose tiles outnumber the workgroups: two per
# CU from 3 x 2^18 parents on and one from 2^21 on, one parent before and at each line.
@pytest.mark.parametrize("n_parents, per_cu", [((3 << 18) - 1, 0), (3 << 18, 2), ((1 << 21) - 1, 2), (1 << 21, 1)])
def test_batch_counted_in_turns(n_parents, per_cu):
    import paper_2609_18703_amd as R
    rng = np.random.default_rng(n_parents)
    counts = rng.integers(0, 3, n_parents)
    counts[n_parents // 2] = 2_500_000 - min(int(counts.sum()), 2_400_000)
    n = int(counts.sum())
    tiles = max(per_cu, 1) * torch.cuda.get_device_properties(0).multi_processor_count + 7
    q_len = max(tiles * 4096 - 1000, (1 << 20) + 1)
    assert q_len <= n
    queue = rng.permutation(n)[:q_len].astype(np.uint32)
    keep = (rng.random(q_len) < 0.8).astype(np.uint8)
    c = R.Context()
    c.reserve(13 << 20, n_parents, q_len)                  # more than 12M children and four queues: the coarse map
    _say("batch counted in turns", n_parents, n, q_len)
    _batch_case(c, counts, queue, keep, None, 256)
    c.close()


# More groups of counted tiles than every tile adds up for itself (2,048 of 65,536
# entries), by one group and with a ragged end; compared on the GPU.
@pytest.mark.parametrize("extra", [0, 1, 70_001])
def test_batch_counted_in_many_groups(extra):
    import paper_2609_18703_amd as R
    q_len = 2048 * 65_536 + extra
    offs = torch.arange(0, 1001, dtype=torch.int64, device="cuda") * 200_000
    queue = torch.arange(q_len, dtype=torch.int32, device="cuda")
    queue = torch.where(queue % 3 == 0, queue ^ 1, queue).contiguous()
    keep = (torch.arange(q_len, dtype=torch.int32, device="cuda") * 7919 % 10 < 7).to(torch.uint8)
    want = queue[keep.bool()]
    m = want.numel()
    outs = [torch.full((m + 4,), -1, dtype=torch.int32, device="cuda") for _ in range(3)]
    sc = _zeros(2, torch.int64)
    c = R.Context()
    c.reserve(1 << 20, 1000, q_len)
    _say("batch counted in many groups", q_len, m)
    torch.cuda.synchronize()
    c.batch(queue, keep, offs, 100, *outs, sc[0:1], sc[1:2], q_len=q_len, out_cap=m)
    c.check("batch")
    assert sc.tolist() == [m, -(-m // 100)]
    assert torch.equal(outs[0][:m], want)
    assert torch.equal(outs[1][:m], want // 200_000)
    assert torch.equal(outs[2][:m], want % 200_000)
    assert all(bool((t[m:] == -1).all()) for t in outs)
    c.close()


# Empty parents in long runs (in front, in the middle of a block, at a span's
# edge, behind), between all children, and in clumps of every length up to
# several steps: the walk over the parents, its jump over a run and the search
# that replaces it, and entries whose parent is searched after all.  The
# reservation decides between the mask map and the coarse one.
@pytest.mark.parametrize("shape", ["front", "middle", "spread", "clumps"])
@pytest.mark.parametrize("reserve", [100_000, 12 << 20])
def test_batch_among_empty_parents(shape, reserve):
    import paper_2609_18703_amd as R
    rng = np.random.default_rng(len(shape))
    if shape == "front":
        counts = np.concatenate([np.zeros(1_100_000, np.int64), rng.integers(1, 200, 800), np.zeros(1000, np.int64)])
    elif shape == "middle":
        empty = [np.zeros(k, np.int64) for k in (1_000_003, 63, 64, 65, 127, 128, 129, 192, 300, 5000)]
        full = [[33], [31], [64], [960], [64, 1, 1], [62], [2, 100], [924, 1024], rng.integers(1, 3, 3000), rng.integers(1, 200, 700)]
        counts = np.concatenate([np.concatenate([f, e]) for f, e in zip(full, empty)])
    elif shape == "spread":
        counts = np.zeros(900_000, np.int64)
        counts[rng.choice(len(counts), 80_000, replace=False)] = 1
    else:
        counts = np.concatenate([np.concatenate([rng.integers(1, 40, rng.integers(1, 8)), np.zeros(rng.integers(0, 400), np.int64)])
                                 for _ in range(1200)])
    n = int(counts.sum())
    q_len = min(n, 90_000)
    assert q_len > 65_536
    queue = rng.permutation(n)[:q_len].astype(np.uint32)
    keep = (rng.random(q_len) < 0.8).astype(np.uint8)
    barrier = (rng.random(len(counts)) < 0.1).astype(np.uint8)
    c = R.Context()
    c.reserve(max(reserve, n), len(counts), q_len)
    for k, bar in ((keep, None), (None, barrier), (keep, barrier)):
        _say("batch among empty parents", shape, n, len(counts), reserve, k is not None, bar is not None)
        _batch_case(c, counts, queue, k, bar, 256)
    # a million empty parents one step of 64 after another are 17,000 dependent
    # loads, 5 ms; the map takes some 15 us (the kernel is loaded by now)
    c.trace(True)
    _batch_case(c, counts, queue, keep, None, 256)
    launches, ms = c.trace_read()["batch_samples"]
    assert launches == 1 and ms < 1.0
    c.close()


def test_batch_parents_of_malformed_offsets_stay_below_the_count():
    """ro_batch does not check the offsets.  The last parent is moved to the
    first block of the last 1,024 children, so later blocks of the mask map
    count on from it: the parents looked up, at which the barrier is read, must
    still be parents.  (The barrier is followed by bytes of the same
    allocation that would suppress the entries.)"""
    import paper_2609_18703_amd as R
    P, span = 5000, 78 * 1024
    starts = np.arange(P, dtype=np.int64) * 16
    starts[4992:4998] = [span + 64 + 8, span + 64 + 24, span + 64 + 40, span + 128 + 8, span + 128 + 24, span + 128 + 40]
    starts[4998:] = [span + 192 + 5, span + 1]
    offs = np.concatenate([starts, [span + 300]])
    n, q_len = int(offs[-1]), 70_000
    queue = np.concatenate([np.arange(n - 300, n), np.arange(q_len - 300)]).astype(np.uint32)
    bar = torch.ones(P + 4096, dtype=torch.uint8, device="cuda")
    bar[:P] = 0
    c = R.Context()
    c.reserve(n, P, q_len)
    for keep in (None, torch.ones(q_len, dtype=torch.uint8, device="cuda")):
        outs = [torch.full((q_len,), -1, dtype=torch.int32, device="cuda") for _ in range(3)]
        sc = _zeros(2, torch.int64)
        _say("batch malformed offsets", keep is not None)
        c.batch(_i32(queue), keep, D.to_dev(offs), 64, *outs, sc[0:1], sc[1:2], barrier=bar[:P])
        c.check("batch")
        assert sc.tolist() == [q_len, -(-q_len // 64)]
        assert np.array_equal(outs[0].cpu().numpy().view(np.uint32), queue)
        assert int(outs[1].cpu().numpy().view(np.uint32).max()) < P
    c.close()


def test_stream_batch_parents_of_malformed_offsets_stay_below_the_count():
    """A stream reports offsets that do not start at 0, or fall, as an error, but
    builds its child -> parent map from them all the same: what a batch finds
    there before the error is read must still be parents, whose offsets are
    read."""
    import paper_2609_18703_amd as R
    n = 5000
    for what, offs in (("late start", [700, 700, 1500, 4000, n]), ("all late", [n - 1, n, n, n, n]),
                       ("falling", [0, 4000, 100, 4500, n]), ("late and falling", [3000, 200, 4000, 50, n])):
        c = R.Context()
        offsets = D.to_dev(np.array(offs, np.int64))
        _say("stream of malformed offsets", what)
        st = c.stream(offsets, n)
        for again in range(2):
            outs = [torch.full((n,), -1, dtype=torch.int32, device="cuda") for _ in range(3)]
            st.batch(_i32(np.arange(n, dtype=np.uint32)), None, 64, *outs)
            par = outs[1].cpu().numpy()
            assert par.min() >= 0 and par.max() < 4, what
            assert c.status() == R.EINVAL, what
            st.reset()
        assert c.status() == R.EINVAL, what
        st.close()
        c.close()


def test_stream_word_and_tile_edges(ctx):
    """Completion found by seen words: parents of one to many 32-child words
    at every alignment, empty parents among them, children in random order
    over waves; emissions of one and several scan tiles, select tiles of 8,192
    parents."""
    from test_gpu_stream_nested import _stream_case
    rng = np.random.default_rng(8)
    sizes = np.array([0, 1, 2, 5, 31, 32, 33, 63, 64, 65, 96, 127, 1023, 1025, 5000])
    counts = np.concatenate([rng.choice(sizes[:11], 1500), sizes, rng.integers(0, 2, 8192), [4096, 0, 0]])
    n = int(counts.sum())
    _say("stream edges", len(counts), n)
    waves = []
    for ids in np.split(rng.permutation(n), [1, n // 7, n // 2, n - 3]):
        waves.append((ids, rng.choice([O.SUCCESS] * 6 + [O.FAILED, O.SKIPPED], len(ids)),
                      rng.choice([0, 1, 15, 16, 17, 90], len(ids))))
    _stream_case(ctx, counts, waves, B=77)
    # children in order, one wave per select tile boundary
    waves = [(ids, np.zeros(len(ids), np.uint8), np.full(len(ids), 3)) for ids in np.array_split(np.arange(n), 3)]
    _stream_case(ctx, counts, waves, B=77, runs=2)


def test_stream_emission_beyond_capacity_is_emitted_later(ctx):
    """Parents an emission has no room for (RO_ECAP) stay for the next one."""
    import paper_2609_18703_amd as R
    counts = np.array([2, 0, 1, 3, 0, 1, 2, 1, 1, 1], np.int32)
    offs, par, ordi = O.expand(counts)
    n, p = len(par), len(counts)
    st = ctx.stream(D.to_dev(offs), n)
    off = np.arange(n + 1, dtype=np.int64) * 4
    data = D.to_dev(np.arange(4 * n, dtype=np.uint8))
    cols = (_i32(par), _i32(ordi), _zeros(n, torch.uint8), D.to_dev(off))
    st.report(*cols, data)
    ep, eo, ed, sc = _zeros(p, torch.int32), _zeros(p + 1, torch.int64), _zeros(4 * n, torch.uint8), _zeros(2, torch.int64)
    st.emit(ep, eo, ed, n_emitted=sc[0:1], n_bytes=sc[1:2], cap_parents=4, cap_bytes=4 * n)
    assert ctx.status() == R.ECAP
    st.emit(ep, eo, ed, n_emitted=sc[0:1], n_bytes=sc[1:2], cap_parents=p, cap_bytes=4 * n)
    ctx.check("second emission")
    assert sc.tolist() == [6, 4 * int(counts[4:].sum())]
    assert ep.tolist()[:6] == list(range(4, 10))
    assert ed.tolist()[:sc[1].item()] == list(range(4 * int(offs[4]), 4 * n))
    st.close()


# one fewer, as many and one more parents than the paths for few parents take
# (4,096, offsets in LDS), with empty parents at both ends and in between
@pytest.mark.parametrize("n_parents", [1, 2, 4095, 4096, 4097])
@pytest.mark.parametrize("fan", [2, 300])
def test_few_parents(ctx, n_parents, fan):
    rng = np.random.default_rng(n_parents + fan)
    counts = np.where(rng.random(n_parents) < 0.3, 0, rng.integers(1, 2 * fan, n_parents)).astype(np.int32)
    counts[n_parents // 2] = 5000                          # several 1,024-child spans
    if n_parents > 2:
        counts[[0, 1, -1]] = 0
    offs, par, ordi = O.expand(counts)
    n = len(par)
    _say("few parents", n_parents, fan, n)
    for shift in (0, 1):                                   # key arrays on and off their 16-byte alignment
        o = _zeros(n_parents + 1, torch.int64)
        tags = [torch.full((n + 8,), -1, dtype=torch.int32, device="cuda")[shift:shift + n] for _ in range(2)]
        ctx.expand(D.to_dev(counts), o, *tags)
        ctx.check("expand")
        assert np.array_equal(o.cpu().numpy(), offs)
        for t, w in zip(tags, (par, ordi)):
            assert np.array_equal(t.cpu().numpy().view(np.uint32), w)
    queue = rng.permutation(n).astype(np.uint32)
    keep = (rng.random(n) < 0.8).astype(np.uint8)
    barrier = (rng.random(n_parents) < 0.1).astype(np.uint8)
    for k, bar in ((None, None), (keep, None), (None, barrier), (keep, barrier)):
        _batch_case(ctx, counts, queue, k, bar, 48)


# Key arrays with room for more children than one launch takes, for as many as
# its workgroups take at once (1,024 each, one per CU), one more, more than one
# launch takes, and none at all.
@pytest.mark.parametrize("n_parents", [1, 300, 4096])
def test_expand_with_room_for_many(ctx, n_parents):
    import paper_2609_18703_amd as R
    room = 9 << 20
    here = 1024 * torch.cuda.get_device_properties(0).multi_processor_count
    tags = [torch.empty(room, dtype=torch.int32, device="cuda") for _ in range(2)]
    for n in (0, 5, here - 1, here, here + 1, (1 << 20) + 3, (8 << 20) + 5):
        counts = np.random.default_rng(n).multinomial(n, np.ones(n_parents) / n_parents).astype(np.int32)
        offs, par, ordi = O.expand(counts)
        for lo in (0, 1):                                  # on and off their 16-byte alignment
            _say("expand with room for many", n_parents, n, lo)
            o = _zeros(n_parents + 1, torch.int64)
            for t in tags:
                t.fill_(-1)
            ctx.expand(D.to_dev(counts), o, *[t[lo:] for t in tags])
            ctx.check("expand")
            assert np.array_equal(o.cpu().numpy(), offs)
            for t, w in zip(tags, (par, ordi)):
                h = t[lo:].cpu().numpy().view(np.uint32)
                assert np.array_equal(h[:n], w) and (h[n:] == 0xffffffff).all()
    for t in tags:
        t.fill_(-1)
    big = np.array([room, 1], np.int32)
    o = _zeros(3, torch.int64)
    ctx.expand(D.to_dev(big), o, *tags)
    assert ctx.status() == R.ECAP and o.tolist() == [0, room, room + 1]
    ctx.expand(D.to_dev(np.array([2 ** 31 - 1, 2 ** 31 - 1], np.int32)), o, *tags)
    assert ctx.status() == R.ECAP
    o = _zeros(4, torch.int64)
    ctx.expand(D.to_dev(np.array([2 ** 31 - 1, 2 ** 31 - 1, 2], np.int32)), o, *tags)
    assert ctx.status() == R.EOVERFLOW
    assert all(bool((t == -1).all()) for t in tags)


# The counts lie in the memory of an output: at the front, in the middle and at
# the end of a key array, or in the offsets' own memory (one tile of parents).
@pytest.mark.parametrize("n_parents", [40, 4096])
@pytest.mark.parametrize("noalloc", [False, True])
def test_expand_counts_in_an_outputs_memory(ctx, n_parents, noalloc):
    import paper_2609_18703_amd as R
    counts = np.random.default_rng(n_parents).integers(0, 200, n_parents).astype(np.int32)
    offs, par, ordi = O.expand(counts)
    n = len(par)
    for where in ("parent", "ordinal", "offsets"):
        for at in (0, (n - n_parents) // 2, n - n_parents) if where != "offsets" else (0, n_parents):
            _say("expand counts in", where, n_parents, n, at)
            o = torch.full((n_parents + 1,), -1, dtype=torch.int64, device="cuda")
            tags = {k: torch.full((n,), -1, dtype=torch.int32, device="cuda") for k in ("parent", "ordinal")}
            home = o.view(torch.int32) if where == "offsets" else tags[where]
            k = home[at:at + n_parents]
            k.copy_(torch.from_numpy(counts))
            if noalloc:
                R.expand_noalloc(k, o, tags["parent"], tags["ordinal"])
                torch.cuda.synchronize()
            else:
                ctx.expand(k, o, tags["parent"], tags["ordinal"])
                ctx.check("expand")
            assert np.array_equal(o.cpu().numpy(), offs)
            assert np.array_equal(tags["parent"].cpu().numpy().view(np.uint32), par)
            assert np.array_equal(tags["ordinal"].cpu().numpy().view(np.uint32), ordi)


def test_expand_errors_with_few_parents(ctx):
    import paper_2609_18703_amd as R
    tags = [_zeros(8, torch.int32) for _ in range(2)]
    off = _zeros(4, torch.int64)
    ctx.expand(D.to_dev(np.array([3, -1, 2], np.int32)), off, *tags)
    assert ctx.status() == R.EINVAL
    for t in tags:                                         # that call's are unspecified
        t.zero_()
    ctx.expand(D.to_dev(np.array([3, 4, 2], np.int32)), off, *tags)
    assert ctx.status() == R.ECAP and off.tolist() == [0, 3, 7, 9]
    ctx.expand(D.to_dev(np.array([2 ** 31 - 1, 2 ** 31 - 1, 2], np.int32)), off, *tags)
    assert ctx.status() == R.EOVERFLOW and off.tolist() == [0, 2 ** 31 - 1, 2 ** 32 - 2, 2 ** 32]
    assert not any(t.any() for t in tags)
