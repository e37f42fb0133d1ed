// Streaming completion on gfx950: reports arrive wave by wave; after each
// wave, every parent whose children are now all terminal is emitted once, in
// ascending parent order, with its ordered bytes, counts and state.
//
// RayOrch (arXiv 2609.18703): a parent can finalise and proceed as soon as all
// of its required child results are terminal (Sec. 1; Sec. 4 Reduce rule);
// facts are published once and conflicting repeats are rejected (Sec. 4,
// publication rules).
//
// Per wave:   report  -> canonical slots + seen bits; the report that completes
//                        a parent sets its ready bit.
// Per emit:   select  -> ascending list of the parents whose ready bit is set
//                        and the exclusive scan of their child counts (two
//                        look-back chains in one pass over the bits): a
//                        "virtual" expansion whose children are the emitted
//                        parents' children, in order;
//             scan    -> over the virtual children: each one's canonical slot,
//                        output position and source, the emitted slot
//                        offsets and per-state counts;
//             out     -> counts, states, trailing offsets, capacity, and the
//                        emitted bytes from the per-child positions.
#include "ro_copy.h"
#include "ro_keys.h"

namespace ro {

// When a parent is complete is found by its reports themselves.  A report sets
// its child's bit in the seen bitmap with a returning atomic (which also
// detects a repeat); the one that completes the parent's share of a 32-child
// word either completes the parent (its only word) or counts that word for
// it, and the one that counts the last word completes it.  So a report adds
// to a counter only once per 32 children, and the counter of a parent of W
// words meets W additions, not one per child.  A parent of two words or more
// is the only one that holds both sides of its first inner word boundary,
// whose index names its counter.  Complete parents are bits of a bitmap,
// which the next emission reads instead of looking at every open parent
// (select 22 -> 11 us for 500,000 parents), and clears as it emits them.
int64_t stream_word_count(int64_t N) { return (N >> 5) + 2; }

__device__ __forceinline__ uint32_t word_share(int64_t w, int64_t st, int64_t en)
{
    const int64_t b0 = w << 5;
    uint32_t m = 0xffffffffu;
    if (st > b0) m &= 0xffffffffu << (st - b0);
    if (en < b0 + 32) m &= 0xffffffffu >> (b0 + 32 - en);
    return m;
}

// Validates the expansion once: offsets[0] = 0, nondecreasing, offsets[P] = N.
// Marks the parents without children complete: the first emission takes them.
// Notes the offsets and, for a reset, whether any differs from the last ones: a
// reset stream's may, and then k_stream_clear builds its child -> parent map
// again.  It finds that out without a word to be cleared in between: remap[0]
// becomes this reset's number, one more than remap[2], and remap[1] the same
// where an offset differs.
__global__ void k_stream_check(const int64_t *__restrict__ offsets, int64_t P, int64_t N, uint64_t *__restrict__ ready,
                               int64_t *__restrict__ mapped, uint32_t *__restrict__ remap, Ctl *ctl)
{
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    bool bad = (g == 0) && (offsets[0] != 0 || offsets[P] != N);
    const uint32_t run = remap ? remap[2] + 1u : 0u;
    if (remap && g == 0) remap[0] = run;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t w = g >> 6; w * 64 < P; w += nwaves) {
        const int64_t p = w * 64 + lane_id();
        const int64_t st = p < P ? offsets[p] : 0;
        const int64_t k = p < P ? offsets[p + 1] - st : 1;
        if (k < 0) bad = true;
        if (p < P && mapped[p] != st) {
            mapped[p] = st;
            if (remap) remap[1] = run;
        }
        const uint64_t m = __ballot(k == 0);
        if (lane_id() == 0) ready[w] = m;
    }
    if (bad) raise_err(ctl, RO_EINVAL);
}

// One wave of reports.  Accepted slots are tagged with the run's epoch.
// With a group-failure barrier, reports commit in order after every earlier
// wave: one of a barred parent, or one after its parent's first group
// failure in this wave, is rejected (counted into *n_rejected).
__global__ __launch_bounds__(kBlock) void k_stream_report(
    const uint32_t *__restrict__ rp, const uint32_t *__restrict__ ro_, const uint8_t *__restrict__ rs,
    const int64_t *__restrict__ roff, const uint8_t *data, int64_t n, const int64_t *__restrict__ offsets,
    int64_t P, int64_t N, Canon *__restrict__ canon, uint32_t *__restrict__ seen, uint32_t *__restrict__ words,
    uint32_t *__restrict__ ready, uint32_t run_epoch, const uint8_t *__restrict__ barrier,
    const uint64_t *__restrict__ gkey, uint32_t gf_epoch, int64_t *n_rejected, Ctl *ctl)
{
    __shared__ int64_t s_wave[kBlock / 64];
    const int64_t gtid = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t gstride = (int64_t)gridDim.x * kBlock;
    int err = 0;
    int64_t rej = 0;
    if (gtid == 0 && n > 0 && roff[0] < 0) err = RO_EINVAL;
    const int ln = lane_id();
    for (int64_t i0 = gtid - ln; i0 < n; i0 += gstride) {
        // all columns at once, then the parent's two offsets: every check that
        // stood between two loads was a trip to memory
        const int64_t i = min64(i0 + ln, n - 1);
        uint32_t s = rs[i];
        const int64_t o0 = roff[i], o1 = roff[i + 1];
        const uint32_t p = rp[i], o = ro_[i];
        if (i0 + ln >= n) s = RO_PENDING;
        const bool known = (int64_t)p < P;
        const int64_t st = known ? offsets[p] : 0, en = known ? offsets[p + 1] : 0;
        const int64_t k = en - st, c = st + (int64_t)o;
        const int64_t len = s == RO_SUCCESS ? o1 - o0 : 0;
        int bad = 0;
        bool counts = false;
        if (o1 < o0) bad = RO_EINVAL;
        else if (s > RO_PENDING && !(s == RO_GROUP_FAILED && barrier)) bad = RO_ESTATE;
        else if (s == RO_PENDING) bad = 0;
        else if (!known || (int64_t)o >= k) bad = RO_ERANGE;
        else if (st < 0 || c >= N) bad = RO_EINVAL;
        else if (len >= ((int64_t)1 << 32)) bad = RO_EOVERFLOW;
        else if (gf_rejected(barrier, gkey, gf_epoch, p, i)) ++rej;
        else counts = true;
        if (bad) err = bad;
        if (s == RO_GROUP_FAILED) s = RO_FAILED;
        // first report of this child, in this wave or any earlier one
        const uint32_t bit = 1u << (c & 31);
        const uint32_t old = change_bits<true>(seen + (c >> 5), bit, counts);
        if (!counts) continue;
        if (old & bit) { err = RO_EDUP; continue; }
        Canon e;
        e.src = reinterpret_cast<uint64_t>(data) + (uint64_t)o0;
        e.len = (uint32_t)len;
        e.tag = (run_epoch << 2) | s;
        canon[c] = e;
        const uint32_t share = word_share(c >> 5, st, st + k);
        if (((old | bit) & share) == share) {
            const int64_t nw = ((st + k - 1) >> 5) - (st >> 5) + 1;
            if (nw == 1 || (int64_t)atomicAdd(&words[(st >> 5) + 1], 1u) + 1 == nw)
                atomicOr(&ready[p >> 5], 1u << (p & 31));
        }
    }
    if (err) raise_err(ctl, err);
    if (barrier) {
        const int64_t r = block_sum(rej, s_wave);
        if (threadIdx.x == 0 && r && n_rejected)
            __hip_atomic_fetch_add(n_rejected, r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Newly complete parents, compacted in ascending order (one tile = 8192
// parents, eight per thread: one byte of the bitmap), and the exclusive scan
// of their child counts: two look-back chains, one over emitted parents and
// one over their children.  With a barrier, its bytes are read too: a barred
// parent is complete, its uncommitted children are suppressed.
// The cost is a chain of latencies, not the parents: ticket, bitmap, offsets
// of the complete ones, look-back.  So tiles are large (61 for 500,000
// parents, one round of look-back), and up to 8,192 parents need no ticket.
constexpr int kSTh = 1024;
constexpr int kSItems = 8;
constexpr int kSTile = kSTh * kSItems;

__global__ __launch_bounds__(kSTh) void k_stream_select(
    const int64_t *__restrict__ offsets, int64_t P, uint8_t *__restrict__ ready, const uint8_t *__restrict__ barrier,
    uint8_t *__restrict__ ebar, uint8_t *__restrict__ emitted, int64_t *__restrict__ ebase,
    int64_t *__restrict__ evoff, uint32_t *__restrict__ emit_parent, int32_t *__restrict__ ecnt, int64_t ecnt_stride,
    int64_t cap_parents, int64_t *n_emitted, Ctl *ctl, uint64_t *desc, uint64_t *desc_kids, int64_t desc_cap,
    int64_t ntiles)
{
    const uint32_t epoch = scan_epoch(ctl);
    __shared__ uint64_t s_w[kSTh / 64];
    __shared__ uint64_t s_b2[2];
    __shared__ int64_t s_t;
    __shared__ int32_t s_last;
    const bool single = ntiles == 1;
    const int wv = (int)(threadIdx.x >> 6), ln = lane_id();
    for (;;) {
        const int64_t t = single ? 0 : next_ticket(ctl, &s_t);
        if (t >= ntiles) break;
        const int64_t p0 = t * kSTile + (int64_t)threadIdx.x * kSItems;
        const uint32_t bits = p0 < P ? ready[p0 >> 3] : 0u;
        uint32_t fmask = bits, bmask = 0;
        if (barrier) {
#pragma unroll
            for (int k = 0; k < kSItems; ++k) {
                if (p0 + k < P && barrier[p0 + k]) {
                    bmask |= 1u << k;
                    if (!emitted[p0 + k]) fmask |= 1u << k;
                }
            }
        }
        uint32_t kk[kSItems];
        int64_t st[kSItems];
        uint64_t kids = 0;
#pragma unroll
        for (int k = 0; k < kSItems; ++k) {
            kk[k] = 0;
            st[k] = 0;
            if (fmask & (1u << k)) {
                st[k] = offsets[p0 + k];
                kk[k] = (uint32_t)(offsets[p0 + k + 1] - st[k]);
            }
        }
#pragma unroll
        for (int k = 0; k < kSItems; ++k) kids += kk[k];
        // one block scan of children << 16 | parents (a tile holds at most 8192 parents)
        const uint64_t v = kids << 16 | (uint64_t)__popc(fmask);
        const uint64_t inc = wave_incl_sum_dpp(v);
        if (ln == 63) s_w[wv] = inc;
        __syncthreads();
        uint64_t ex = inc - v, tot = 0;
#pragma unroll
        for (int i = 0; i < kSTh / 64; ++i) {
            const uint64_t x = s_w[i];
            ex += i < wv ? x : 0;
            tot += x;
        }
        uint64_t pre = 0, prek = 0;
        if (!single) tile_prefix2(desc, tot & 0xffffu, desc_kids, tot >> 16, t, epoch, s_b2, pre, prek, ctl);
        int64_t e = (int64_t)pre + (int64_t)(ex & 0xffffu);
        int64_t run = (int64_t)prek + (int64_t)(ex >> 16);
        uint32_t left = bits;                         // complete parents that stay for a later emission
        bool over = false;
#pragma unroll
        for (int k = 0; k < kSItems; ++k) {
            if (!(fmask & (1u << k))) continue;
            const int64_t p = p0 + k;
            if (e < cap_parents) {
                ebase[e] = st[k] - run;           // canonical slot of virtual child v: ebase[e] + v
                evoff[e] = run;
                ebar[e] = (bmask >> k) & 1u;
                if (emit_parent) emit_parent[e] = (uint32_t)p;
                ecnt[e] = 0;
                ecnt[ecnt_stride + e] = 0;
                ecnt[2 * ecnt_stride + e] = 0;
                emitted[p] = 1;
                left &= ~(1u << k);
            } else {
                if (e == cap_parents) {
                    // the emission stops here: its virtual children end at run
                    evoff[e] = run;
                    ctl->n_virtual = run;
                }
                over = true;
            }
            ++e;
            run += kk[k];
        }
        if (left != bits) ready[p0 >> 3] = (uint8_t)left;
        if (over) raise_err(ctl, RO_ECAP);
        if (t == ntiles - 1 && threadIdx.x == 0) {
            const int64_t E = (int64_t)pre + (int64_t)(tot & 0xffffu), V = (int64_t)prek + (int64_t)(tot >> 16);
            if (n_emitted) *n_emitted = E;
            ctl->n_items = E < cap_parents ? E : cap_parents;
            if (E <= cap_parents) {
                evoff[E] = V;
                ctl->n_virtual = V;
            }
        }
        if (single) return;
        if (ntiles <= (int64_t)gridDim.x) break;  // a tile for every workgroup
        __syncthreads();                          // s_w is written again
    }
    ticket_done(ctl, epoch, desc, desc_cap, &s_last);
}

// Byte scan over the virtual children of this emission, 4096 per tile in
// groups of 64, a group per load of a wave.  Virtual child v of emitted parent
// e lives in canonical slot ebase[e] + v; the tile's parents are in LDS, and
// every child finds its own there.  As in the gather's scan, exclusive byte
// sums and state masks per group answer any range, so after the look-back the
// work goes by parent: slot offset and counts.  Writes each child's output
// position edst[v] and source address esrc[v] for the copy.  Only as many
// workgroups as there are tiles take part; a single tile (most waves of a
// long stream) needs no ticket and no look-back.
constexpr int kETh = 1024;
constexpr int kEItems = 4;
constexpr int kETile = kETh * kEItems;

__global__ __launch_bounds__(kETh) void k_emit_scan(
    const int64_t *__restrict__ evoff, const int64_t *__restrict__ ebase, const Canon *__restrict__ canon,
    int64_t *__restrict__ edst, uint64_t *__restrict__ esrc, int64_t *__restrict__ emit_off,
    int32_t *__restrict__ ecnt, int64_t ecnt_stride, uint32_t run_epoch, Ctl *ctl, uint64_t *desc,
    int64_t desc_cap)
{
    constexpr int kG = kETile / 64;
    constexpr int kCF = 21, kCK = 42;             // a packed count: SUCCESS, FAILED << 21, SKIPPED << 42
    constexpr uint64_t kCM = (1u << kCF) - 1;
    static_assert(kG == 64, "one lane per group");
    const int64_t E = ctl->n_items;
    const int64_t V = ctl->n_virtual;
    const int64_t ntiles = (V + kETile - 1) / kETile;
    if ((int64_t)blockIdx.x >= ntiles) return;
    const uint32_t parts = (uint32_t)min64((int64_t)gridDim.x, ntiles);
    const uint32_t sepoch = scan_epoch(ctl);
    const bool single = ntiles == 1;
    __shared__ uint64_t s_pre[kETile];            // exclusive byte sum inside the child's group
    __shared__ int64_t s_base[kETile + 2];        // ebase of the tile's parents
    __shared__ int16_t s_off[kETile + 4];         // evoff of the tile's parents - vt0, clamped to [-1, kETile + 1]
    __shared__ uint64_t s_gt[kG], s_gbase[kG];
    __shared__ uint64_t s_m[3][kG + 1], s_cp[kG + 1];
    __shared__ uint64_t s_b;
    __shared__ int64_t s_t;
    __shared__ int64_t s_p[2];
    __shared__ int32_t s_last;
    const int wv = uni32((int)(threadIdx.x >> 6)), ln = lane_id();
    for (;;) {
        const int64_t t = single ? 0 : next_ticket(ctl, &s_t);
        if (t >= ntiles) break;
        const int64_t vt0 = t * kETile;
        const int nloc = (int)min64(kETile, V - vt0);
        // q0: first emitted parent starting in the tile; q1: first one after it
        if (wv < 2) {
            const int64_t x = vt0 + (wv == 0 ? 0 : nloc);
            const int64_t r = x == 0 ? 0 : wave_last_le(evoff, 0, E + 1, x - 1) + 1;
            if (ln == 0) s_p[wv] = r;
        }
        __syncthreads();
        const int64_t q0 = s_p[0], q1 = s_p[1];
        const int64_t pf = q0 > 0 ? q0 - 1 : 0;         // holds child vt0 if none starts there
        const int64_t Rp = q1 - pf;
        const bool lds_ok = Rp <= kETile;
        if (lds_ok) {
            for (int64_t j = threadIdx.x; j <= Rp; j += kETh) {
                const int64_t x = evoff[pf + j] - vt0;
                s_off[j] = (int16_t)(x < -1 ? -1 : (x > kETile + 1 ? kETile + 1 : x));
                if (j < Rp) s_base[j] = ebase[pf + j];
            }
        }
        __syncthreads();
        // every child's slot, then the slots, all in flight
        int64_t slot[kEItems];
#pragma unroll
        for (int k = 0; k < kEItems; ++k) {
            const int i = (wv * kEItems + k) * 64 + ln;
            const int rv = i < nloc ? i : nloc - 1;
            if (lds_ok) slot[k] = s_base[lds_last_le(s_off, 0, (int)Rp, rv)];
            else slot[k] = ebase[upper_bound_g(evoff, pf, q1, vt0 + rv) - 1];
            slot[k] += vt0 + rv;
        }
        Canon x[kEItems];
#pragma unroll
        for (int k = 0; k < kEItems; ++k) x[k] = canon[slot[k]];
#pragma unroll
        for (int k = 0; k < kEItems; ++k) {
            const int g = wv * kEItems + k, i = g * 64 + ln;
            const uint32_t S = (i < nloc && (x[k].tag >> 2) == run_epoch) ? x[k].tag & 3u : 4u;
            const uint64_t L = S == RO_SUCCESS ? x[k].len : 0u;
            const uint64_t m0 = __ballot(S == RO_SUCCESS), m1 = __ballot(S == RO_FAILED),
                           m2 = __ballot(S == RO_SKIPPED);
            const uint64_t inc = wave_incl_sum_dpp(L);
            s_pre[i] = inc - L;
            if (ln == 63) {
                s_gt[g] = inc;
                s_m[0][g] = m0;
                s_m[1][g] = m1;
                s_m[2][g] = m2;
            }
        }
        __syncthreads();
        if (wv == 0) {
            const uint64_t gt = s_gt[ln];
            const uint64_t gc = (uint64_t)__popcll(s_m[0][ln]) | (uint64_t)__popcll(s_m[1][ln]) << kCF |
                                (uint64_t)__popcll(s_m[2][ln]) << kCK;
            const uint64_t gi = wave_incl_sum_dpp(gt), ci = wave_incl_sum_dpp(gc);
            const uint64_t tot = (uint64_t)uni64(__shfl((long long)gi, 63, 64));
            s_gbase[ln] = gi - gt;
            s_cp[ln] = ci - gc;
            if (ln == 63) s_cp[kG] = ci;
            const uint64_t pr = single ? 0 : lookback_wave(desc, t, sepoch, tot, ctl);
            if (ln == 0) {
                s_b = pr;
                if (t == ntiles - 1) {
                    ctl->total = (int64_t)(pr + tot);
                    edst[V] = (int64_t)(pr + tot);
                    if (pr >= kSat) raise_err(ctl, RO_EOVERFLOW);
                }
            }
        }
        __syncthreads();
        const int64_t pre = (int64_t)s_b;
#pragma unroll
        for (int k = 0; k < kEItems; ++k) {
            const int g = wv * kEItems + k, i = g * 64 + ln;
            if (i < nloc) {
                edst[vt0 + i] = pre + (int64_t)(s_gbase[g] + s_pre[i]);
                esrc[vt0 + i] = (x[k].tag >> 2) == run_epoch ? x[k].src : 0;
            }
        }
        auto counts_to = [&](int y) -> uint64_t {
            const int g = y >> 6;
            const uint64_t low = (1ull << (y & 63)) - 1;
            return s_cp[g] + ((uint64_t)__popcll(s_m[0][g] & low) | (uint64_t)__popcll(s_m[1][g] & low) << kCF |
                              (uint64_t)__popcll(s_m[2][g] & low) << kCK);
        };
        auto add_counts = [&](int64_t e, uint64_t c, bool whole) {
            const int32_t cc[3] = {(int32_t)(c & kCM), (int32_t)((c >> kCF) & kCM), (int32_t)(c >> kCK)};
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                if (whole) ecnt[s * ecnt_stride + e] = cc[s];
                else if (cc[s]) atomicAdd(&ecnt[s * ecnt_stride + e], cc[s]);
            }
        };
        for (int64_t q = q0 + threadIdx.x; q < q1; q += kETh) {
            const int st = (int)(evoff[q] - vt0);
            const int64_t en = evoff[q + 1] - vt0;
            emit_off[q] = pre + (int64_t)(s_gbase[st >> 6] + s_pre[st]);
            add_counts(q, counts_to((int)min64(en, nloc)) - counts_to(st), en <= nloc);
        }
        if (threadIdx.x == kETh - 1 && vt0 > 0) {       // the parent reaching in from the tile before
            const int64_t en = min64(evoff[q0] - vt0, nloc);
            if (en > 0) add_counts(q0 - 1, counts_to((int)en), false);
        }
        if (single) return;
        if (ntiles <= (int64_t)gridDim.x) break;        // a tile for every workgroup
        __syncthreads();
    }
    ticket_done_n(ctl, sepoch, desc, desc_cap, &s_last, parts);
}

// Outputs of the emission once its scan is done: per emitted parent its
// counts, state and (for parents without children at the very end) slot
// offset; then the bytes.  The output is cut into byte units as in the
// gather's copy, kEmitMinUnit bytes or more (a unit costs a search over the
// positions, not a re-read of slot records, so small units pay here); a unit
// finds its first child by a wave search over the output positions and takes
// the children it covers 256 at a time, each clipped to the unit.
#ifndef RO_EMIT_MIN_UNIT
#define RO_EMIT_MIN_UNIT 1024
#endif
constexpr int64_t kEmitMinUnit = RO_EMIT_MIN_UNIT;
#ifndef RO_EMIT_GRID
#define RO_EMIT_GRID 4                      // emission copy workgroups per CU
#endif
#ifndef RO_EMIT_UNIT
#define RO_EMIT_UNIT (64 << 10)
#endif
constexpr int64_t kEmitUnit = RO_EMIT_UNIT;
#ifndef RO_EMIT_STEPS
#define RO_EMIT_STEPS 4
#endif

__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4))) void k_emit_out(
    int64_t *__restrict__ emit_off, const int64_t *__restrict__ evoff, const int32_t *__restrict__ ecnt,
    int64_t ecnt_stride, const uint8_t *__restrict__ ebar, int32_t *__restrict__ ns, int32_t *__restrict__ nf,
    int32_t *__restrict__ nk, uint8_t *__restrict__ pstate, int64_t *n_bytes, const int64_t *__restrict__ edst,
    const uint64_t *__restrict__ esrc, uint8_t *__restrict__ out, int64_t cap_bytes, Ctl *ctl)
{
    constexpr int kWaves = kBlock / 64;
    __shared__ int32_t s_dst_all[kWaves][kSub + 1];
    __shared__ uint64_t s_src_all[kWaves][kSub];
    __shared__ int32_t s_edge_all[kWaves][kEdgeCap];
    __shared__ int16_t s_edger_all[kWaves][kEdgeCap];
    const int64_t E = ctl->n_items;
    const int64_t V = ctl->n_virtual;
    const int64_t T = V > 0 ? ctl->total : 0;
    // parents go to the workgroups from the last one on, which have no bytes
    // to copy in a small emission
    const int64_t g = (int64_t)(gridDim.x - 1 - blockIdx.x) * blockDim.x + threadIdx.x;
    if (g == 0) {
        emit_off[E] = T;
        if (n_bytes) *n_bytes = T;
        if (out && T > cap_bytes) raise_err(ctl, RO_ECAP);
    }
    for (int64_t e = g; e < E; e += (int64_t)gridDim.x * blockDim.x) {
        if (evoff[e] >= V) emit_off[e] = T;
        const int32_t a = ecnt[e], f = ecnt[ecnt_stride + e], k = ecnt[2 * ecnt_stride + e];
        if (ns) ns[e] = a;
        if (nf) nf[e] = f;
        if (nk) nk[e] = k;
        if (pstate) pstate[e] = (f > 0 || ebar[e]) ? RO_FAILED : RO_SUCCESS;
    }
    if (out == nullptr || T <= 0 || T > cap_bytes || read_err(ctl) != 0) return;
    const uint64_t outa = reinterpret_cast<uint64_t>(out);
    const int64_t mis = (int64_t)(outa & 15);
    const int64_t nwaves = (int64_t)gridDim.x * kWaves;
    int64_t rounds = (T + nwaves * kEmitUnit / 2) / (nwaves * kEmitUnit);
    rounds = rounds < 1 ? 1 : rounds;
    int64_t G = (T + mis + nwaves * rounds - 1) / (nwaves * rounds);
    G = (G + 15) & ~(int64_t)15;
    G = G < kEmitMinUnit ? kEmitMinUnit : (G > ((int64_t)1 << 30) ? ((int64_t)1 << 30) : G);
    const int64_t nunits = (T + mis + G - 1) / G;
    const int wave = uni32((int)(threadIdx.x >> 6)), lane = lane_id();
    int32_t *s_dst = s_dst_all[wave];
    uint64_t *s_src = s_src_all[wave];
    int32_t *s_edge = s_edge_all[wave];
    int16_t *s_edger = s_edger_all[wave];
    for (int64_t u = (int64_t)blockIdx.x * kWaves + wave; u < nunits; u += nwaves) {
        const int64_t lo = max64(u * G - mis, 0);
        const int64_t hi = min64((u + 1) * G - mis, T);
        for (int64_t r0 = uni64(wave_last_le(edst, 0, V, lo)); r0 < V; r0 += kSub) {
            // children r0 .. r0 + kSub - 1, their starts clipped to [ws, we)
            const int64_t dend = edst[min64(r0 + kSub, V)];
            const int64_t ws = max64(lo, edst[r0]);
            const int64_t we = min64(hi, dend);
            if (we <= ws) {
                if (dend >= hi) break;
                continue;                          // only empty children here
            }
            // positions 64 at a time, stopping after the group that reaches
            // the window's end: a small unit covers a few children, and the
            // rest of the 256 are set empty without being read
            bool past = false;
#pragma unroll
            for (int k = 0; k < kSub / 64; ++k) {
                const int i = k * 64 + lane;
                const int64_t v = r0 + i;
                if (past) {
                    s_dst[i] = (int32_t)(we - ws);
                    s_src[i] = 0;
                    continue;
                }
                const int64_t d = v < V ? edst[v] : T;
                const int64_t cs = min64(max64(d, ws), we);
                s_dst[i] = (int32_t)(cs - ws);
                s_src[i] = (v < V ? esrc[v] : 0) + (uint64_t)(cs - d);
                past = __shfl(d, 63, 64) >= we;
            }
            if (lane == 0) s_dst[kSub] = (int32_t)(we - ws);
            __builtin_amdgcn_wave_barrier();
            copy_window_nb<RO_EMIT_STEPS>(s_dst, s_src, s_edge, s_edger, (int)(we - ws), outa, ws, lane);
            __builtin_amdgcn_wave_barrier();
            if (dend >= hi) break;
        }
    }
}

// Forgets every report and emission: seen bits, counters and emitted flags
// back to zero.  Canonical slots need no clearing, since a slot is read only
// for children of emitted parents, and those were all reported.  Builds the
// child -> parent map again if the check before found other offsets (10M
// children of 500,000 parents: 27 us a reset, 11 without; a launch of its own
// that mostly finds nothing to do took 5.5 more).
__global__ __launch_bounds__(kBlock) void k_stream_clear(uint32_t *__restrict__ seen, int64_t n_seen, uint32_t *__restrict__ words,
                               int64_t n_words, uint8_t *__restrict__ emitted, uint8_t *__restrict__ barrier,
                               int64_t n_emitted, const int64_t *__restrict__ offsets, int64_t N,
                               uint32_t *__restrict__ cpar, uint32_t *__restrict__ remap)
{
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const uint32_t run = remap[0], other = remap[1];
    if (g == 0) remap[2] = run;
    for (int64_t i = g; i < n_seen; i += stride) seen[i] = 0;
    for (int64_t i = g; i < n_words; i += stride) words[i] = 0;
    for (int64_t i = g; i < n_emitted; i += stride) {
        emitted[i] = 0;
        if (barrier) barrier[i] = 0;
    }
    if (run == other) write_keys(offsets, n_emitted, cpar, nullptr, N, -1, 1);
}

// A thread per item, up to four workgroups per CU.
static unsigned reset_grid(const Launch &L, int64_t items)
{
    const int64_t g = (items + kBlock - 1) / kBlock, most = (int64_t)L.num_cus * 4;
    return (unsigned)(g < 1 ? 1 : g < most ? g : most);
}

static hipError_t launch_stream_check(const Launch &L, StreamState &s, uint32_t *remap)
{
    RO_LAUNCH(L, RO_K_MISC, k_stream_check, dim3(reset_grid(L, s.P)), dim3(kBlock), 0, L.stream, s.offsets, s.P, s.N,
              s.ready, s.mapped, remap, L.ctl);
    return hipGetLastError();
}

// A new stream, whose state is all zero.
hipError_t launch_stream_init(const Launch &L, StreamState &s)
{
    const hipError_t e = launch_stream_check(L, s, nullptr);
    return e != hipSuccess ? e : launch_expand_tags(L, s.offsets, s.P, s.cpar, nullptr, s.N);
}

hipError_t launch_stream_reset(const Launch &L, StreamState &s)
{
    const hipError_t e = launch_stream_check(L, s, s.remap);
    if (e != hipSuccess) return e;
    RO_LAUNCH(L, RO_K_MISC, k_stream_clear, dim3(reset_grid(L, s.P + s.N / kItems)), dim3(kBlock), 0, L.stream, s.seen,
              (s.N + 31) / 32 + 1, s.words, stream_word_count(s.N), s.emitted, s.barrier, s.P, s.offsets, s.N, s.cpar,
              s.remap);
    return hipGetLastError();
}

hipError_t launch_stream_report(const Launch &L, StreamState &s, const uint32_t *rp, const uint32_t *ro,
                                const uint8_t *rs, const int64_t *roff, const uint8_t *data, int64_t n,
                                int64_t *n_rejected)
{
    if (s.barrier) {
        const hipError_t e = launch_first_gf(L, rs, rp, n, s.P, s.barrier, s.gkey, s.gf_epoch);
        if (e != hipSuccess) return e;
    }
    int64_t grid = (n + kBlock - 1) / kBlock;
    grid = grid < 1 ? 1 : (grid > (int64_t)L.num_cus * 8 ? (int64_t)L.num_cus * 8 : grid);
    RO_LAUNCH(L, RO_K_STREAM_REPORT, k_stream_report, dim3((unsigned)grid), dim3(kBlock), 0, L.stream, rp, ro,
              rs, roff, data, n, s.offsets, s.P, s.N, s.canon, s.seen, s.words,
              reinterpret_cast<uint32_t *>(s.ready), s.run_epoch, s.barrier, s.gkey, s.gf_epoch, n_rejected, L.ctl);
    if (s.barrier) return launch_gf_fold(L, rs, rp, n, s.P, s.barrier, s.gkey, s.gf_epoch);
    return hipGetLastError();
}

int64_t stream_desc_tiles(int64_t P, int64_t N)
{
    const int64_t tp = (P + kSTile - 1) / kSTile + 1, tn = (N + kETile - 1) / kETile + 1;
    return 2 * tp > tn ? 2 * tp : tn;
}

hipError_t launch_stream_emit(const Launch &L, StreamState &s, uint32_t *emit_parent, int64_t *emit_off,
                              uint8_t *emit_data, int64_t cap_parents, int64_t cap_bytes, int32_t *ns,
                              int32_t *nf, int32_t *nk, uint8_t *pstate, int64_t *n_emitted,
                              int64_t *n_bytes)
{
    const int64_t ntiles = s.P > 0 ? (s.P + kSTile - 1) / kSTile : 1;
    if (2 * ntiles > L.desc_cap || (s.N + kETile - 1) / kETile > L.desc_cap) return hipErrorInvalidValue;
    // a workgroup of select per CU at most (a tile is 8192 parents); two of the scan fit a CU's LDS
    const int64_t grid = ntiles < (int64_t)L.num_cus ? ntiles : (int64_t)L.num_cus;
    const int64_t es = s.P + 1;
    RO_LAUNCH(L, RO_K_STREAM_SELECT, k_stream_select, dim3((unsigned)grid), dim3(kSTh), 0, L.stream, s.offsets, s.P,
              reinterpret_cast<uint8_t *>(s.ready), s.barrier, s.ebar, s.emitted, s.ebase, s.evoff, emit_parent, s.ecnt,
              es, cap_parents, n_emitted, L.ctl, L.desc, L.desc + ntiles, L.desc_cap, ntiles);
    const int64_t grid_s = (int64_t)L.num_cus * 2;
    RO_LAUNCH(L, RO_K_STREAM_SCAN, k_emit_scan, dim3((unsigned)grid_s), dim3(kETh), 0, L.stream, s.evoff,
              s.ebase, s.canon, s.edst, s.esrc, emit_off, s.ecnt, es, s.run_epoch, L.ctl, L.desc, L.desc_cap);
    const int64_t grid_c = (int64_t)L.num_cus * RO_EMIT_GRID;
    RO_LAUNCH(L, RO_K_STREAM_COPY, k_emit_out, dim3((unsigned)grid_c), dim3(kBlock), 0, L.stream, emit_off,
              s.evoff, s.ecnt, es, s.ebar, ns, nf, nk, pstate, n_bytes, s.edst, s.esrc, emit_data, cap_bytes, L.ctl);
    return hipGetLastError();
}

}  // namespace ro
