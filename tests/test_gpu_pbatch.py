"""GPU parity for parent-bound reservation against the oracle: every slot's
child, parent and ordinal and every batch boundary, bit-exact."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle as O  # noqa: E402
import workloads as W  # noqa: E402
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
    yield c
    c.close()


def _run(ctx, queue, keep, offs, B, barrier=None, out_cap=None, batch_cap=None):
    Q = len(queue)
    cap = Q if out_cap is None else out_cap
    bcap = Q + 1 if batch_cap is None else batch_cap
    q = D.to_dev(np.ascontiguousarray(queue, np.uint32).view(np.int32)) if Q else \
        torch.zeros(1, dtype=torch.int32, device="cuda")
    k = None if keep is None else (D.to_dev(np.asarray(keep, np.uint8)) if Q else
                                   torch.zeros(1, dtype=torch.uint8, device="cuda"))
    bar = None if barrier is None else D.to_dev(np.asarray(barrier, np.uint8))
    oc = torch.full((max(cap, 1),), -1, dtype=torch.int32, device="cuda")
    op = torch.full((max(cap, 1),), -1, dtype=torch.int32, device="cuda")
    oo = torch.full((max(cap, 1),), -1, dtype=torch.int32, device="cuda")
    boff = torch.full((max(bcap, 1),), -1, dtype=torch.int64, device="cuda")
    sc = torch.full((2,), -1, dtype=torch.int64, device="cuda")
    ctx.batch_parent(q, k, D.to_dev(offs), B, boff[:bcap], oc, op, oo, sc[0:1], sc[1:2], q_len=Q, out_cap=cap,
                     barrier=bar)
    return oc, op, oo, boff, sc


def _check(ctx, queue, keep, offs, B, barrier=None, what=""):
    want = O.batch(queue, keep, offs, B, barrier=barrier, parent_bound=True)
    oc, op, oo, boff, sc = _run(ctx, queue, keep, offs, B, barrier)
    ctx.check(what)
    m, nb = (int(x) for x in sc.cpu().numpy())
    assert m == len(want[0]) and nb == len(want[3]), what
    u32 = lambda t: t.cpu().numpy().view(np.uint32)[:m]
    assert np.array_equal(u32(oc), want[0]), what
    assert np.array_equal(u32(op), want[1]), what
    assert np.array_equal(u32(oo), want[2]), what
    assert np.array_equal(boff.cpu().numpy()[:nb + 1], np.concatenate([[0], np.cumsum(want[3])])), what


@pytest.mark.parametrize("P,B,seed", [(1, 4, 0), (2, 3, 1), (7, 1, 2), (300, 16, 3), (513, 5, 4), (513, 512, 5),
                                      (5000, 64, 6), (70_000, 256, 7), (70_000, 1 << 30, 8)])
def test_pbatch_random(ctx, P, B, seed):
    rng = np.random.default_rng(seed)
    counts = rng.integers(0, 9, P).astype(np.int32)
    if P > 1:
        counts[rng.integers(0, P)] = 9000                   # one parent spans several sort tiles
    offs = O.expand(counts, tags=False)
    N = int(offs[-1])
    queue = rng.permutation(N).astype(np.uint32)
    keep = (rng.random(N) < 0.9).astype(np.uint8)
    _say("pbatch", P, B, seed, "N", N)
    _check(ctx, queue, keep, offs, B, what=f"P={P} B={B} keep")
    _check(ctx, queue, None, offs, B, what=f"P={P} B={B} all")
    bar = (rng.random(P) < 0.2).astype(np.uint8)
    _check(ctx, queue, keep, offs, B, barrier=bar, what=f"P={P} B={B} barrier")


def test_pbatch_partial_queue_and_edges(ctx):
    rng = np.random.default_rng(11)
    counts = rng.integers(0, 5, 2000).astype(np.int32)
    offs = O.expand(counts, tags=False)
    N = int(offs[-1])
    q = rng.choice(N, N // 3, replace=False).astype(np.uint32)     # a queue holding some children only
    _check(ctx, q, None, offs, 7, what="partial queue")
    _check(ctx, np.zeros(0, np.uint32), None, offs, 7, what="empty queue")
    _check(ctx, q, np.zeros(len(q), np.uint8), offs, 7, what="nothing ready")
    # canonical order: every parent's entries are already together
    _check(ctx, np.arange(N, dtype=np.uint32), None, offs, 3, what="canonical order")


# one entry fewer and one more than a sort tile (4,096), a histogram span
# (8,192), a scan tile (32,768) and a bitmap word, over parent ids of one digit
# pass (up to 512 parents), two (even and odd widths) and three
@pytest.mark.parametrize("q_len", [63, 64, 65, 4095, 4097, 8191, 8193, 32_767, 32_769, 65_537])
@pytest.mark.parametrize("P", [1, 512, 513, 4097, 300_000])
def test_pbatch_tile_edges(ctx, q_len, P):
    rng = np.random.default_rng(q_len + P)
    offs = np.zeros(P + 1, np.int64)
    offs[1:] = np.cumsum(rng.multinomial(q_len + 5, rng.dirichlet(np.full(P, 0.3))) if P > 1 else [q_len + 5])
    queue = rng.permutation(q_len + 5)[:q_len].astype(np.uint32)
    _say("pbatch edges", q_len, P)
    for B in (1, 2, 100):
        _check(ctx, queue, None, offs, B, what=f"Q={q_len} P={P} B={B}")


# sizes that a byte holds, its two codes and more: a full group, remainders on
# both sides of each, and a batch that takes a whole parent
@pytest.mark.parametrize("B", [1, 252, 253, 254, 255, 256, 257, 512, 1 << 30])
def test_pbatch_group_sizes(ctx, B):
    rng = np.random.default_rng(B % 1000)
    counts = rng.permutation(np.concatenate([np.arange(248, 262), np.arange(504, 516), [0, 1, 2, 767, 1024]]))
    offs = O.expand(counts.astype(np.int32), tags=False)
    N = int(offs[-1])
    _say("pbatch group sizes", B, N)
    _check(ctx, rng.permutation(N).astype(np.uint32), None, offs, B, what=f"B={B} random")
    _check(ctx, np.arange(N, dtype=np.uint32), None, offs, B, what=f"B={B} canonical")


def test_pbatch_batches_of_one_cost_no_contention(ctx):
    """10M batches of one from one parent, whose first entries are neighbours
    in the queue.  The kernels that form the batches have 120 MB more
    of them to write than for batches of 256 and took 2.8 times as long;
    when neighbours set bits of one word, it was 7 times."""
    n = 10_000_000
    q = torch.arange(n, dtype=torch.int32, device="cuda")
    offs = torch.tensor([0, n], dtype=torch.int64, device="cuda")
    outs = [torch.zeros(n, dtype=torch.int32, device="cuda") for _ in range(3)]
    boff = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    sc = torch.zeros(2, dtype=torch.int64, device="cuda")
    ms = {}
    for B in (256, 1):
        call = lambda: ctx.batch_parent(q, None, offs, B, boff, *outs, sc[0:1], sc[1:2])
        call()
        ctx.trace(True)
        for _ in range(5):
            call()
        ms[B] = ctx.trace_read()["pbatch"][1]
        ctx.check()
        ctx.trace(False)
    _say("batches of 256 and of one:", ms)
    assert ms[1] < 4.5 * ms[256]


def test_pbatch_errors(ctx):
    import paper_2609_18703_amd as R
    offs = O.expand(np.array([3, 2], np.int32), tags=False)
    q = np.array([4, 0, 1, 3, 2], np.uint32)
    _run(ctx, q, None, offs, 2, out_cap=3)
    assert ctx.status() == R.ECAP
    _run(ctx, q, None, offs, 2, batch_cap=3)                       # 4 batches need 5 offsets
    assert ctx.status() == R.ECAP
    _run(ctx, np.array([0, 9], np.uint32), None, offs, 2)
    assert ctx.status() == R.ERANGE
    _check(ctx, q, None, offs, 2, what="after errors")


def test_pbatch_zipf_full(ctx):
    """The 41M-child Zipf workload's ready queue (sealed children masked out),
    B = 256, in full."""
    c = W.config2()
    offs = O.expand(c.counts, tags=False)
    _say("pbatch zipf full: Q", len(c.queue))
    _check(ctx, c.queue, c.keep, offs, c.batch_size, what="zipf full")
