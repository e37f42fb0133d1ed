// F.reduce on gfx950: ordered gather of variable-length child reports into
// parent slots, with per-parent counts and completion.
//
// RayOrch (arXiv 2609.18703), Sec. 4, Reduce rule: a parent resolves once its
// Expansion and every member outcome are terminal; dropped members are left
// out, failed members suppress the parent, present values appear in immutable
// ordinal order, and zero survivors give an empty list.  The publication
// rules of the same section reject a second, conflicting report.
//
// Three kernels:
//   scatter  : report i -> canonical slot c = offsets[p] + o (validation, one
//              16-byte store per report; the only random-access pass).
//   scan     : canonical order, decoupled look-back over the surviving byte
//              lengths -> every parent's slot offset and counts, the first
//              byte of every group of 64 children; duplicate and capacity
//              checks.
//   copy     : per parent complete / state and trailing slot offsets; then
//              the output is cut into byte ranges of equal size; per range, a
//              wave rebuilds the destination offsets of the groups it
//              overlaps and writes the range as aligned 16-byte stores;
//              sources are byte-aligned records.
// Without bytes to copy the per-parent part is a kernel of its own.
#include "ro_copy.h"

namespace ro {

// ---------------------------------------------------------------- group failure
__global__ void k_first_gf(const uint8_t *__restrict__ rs, const uint32_t *__restrict__ rp, int64_t n,
                           int64_t P, const uint8_t *__restrict__ barrier, uint64_t *__restrict__ gkey,
                           uint32_t epoch)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        if (rs[i] != RO_GROUP_FAILED) continue;
        const uint32_t p = rp[i];
        if ((int64_t)p >= P || barrier[p]) continue;
        __hip_atomic_fetch_max(&gkey[p], gf_key(epoch, i), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

__global__ void k_gf_fold(const uint8_t *__restrict__ rs, const uint32_t *__restrict__ rp, int64_t n, int64_t P,
                          uint8_t *__restrict__ barrier, const uint64_t *__restrict__ gkey, uint32_t epoch)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        if (rs[i] != RO_GROUP_FAILED) continue;
        const uint32_t p = rp[i];
        if ((int64_t)p < P && gkey[p] == gf_key(epoch, i)) barrier[p] = 1;
    }
}

hipError_t launch_first_gf(const Launch &L, const uint8_t *rs, const uint32_t *rp, int64_t n, int64_t P,
                           const uint8_t *barrier, uint64_t *gkey, uint32_t epoch)
{
    int64_t grid = (n + kBlock - 1) / kBlock;
    grid = grid < 1 ? 1 : (grid > (int64_t)L.num_cus * 8 ? (int64_t)L.num_cus * 8 : grid);
    RO_LAUNCH(L, RO_K_GATHER_SCATTER, k_first_gf, dim3((unsigned)grid), dim3(kBlock), 0, L.stream, rs, rp, n, P,
              barrier, gkey, epoch);
    return hipGetLastError();
}

hipError_t launch_gf_fold(const Launch &L, const uint8_t *rs, const uint32_t *rp, int64_t n, int64_t P,
                          uint8_t *barrier, const uint64_t *gkey, uint32_t epoch)
{
    int64_t grid = (n + kBlock - 1) / kBlock;
    grid = grid < 1 ? 1 : (grid > (int64_t)L.num_cus * 8 ? (int64_t)L.num_cus * 8 : grid);
    RO_LAUNCH(L, RO_K_STREAM_REPORT, k_gf_fold, dim3((unsigned)grid), dim3(kBlock), 0, L.stream, rs, rp, n, P,
              barrier, gkey, epoch);
    return hipGetLastError();
}

// ---------------------------------------------------------------- scatter
#ifndef RO_SCATTER_ITEMS
#define RO_SCATTER_ITEMS 2
#endif
constexpr int kScatterItems = RO_SCATTER_ITEMS;   // reports per thread and step
// With a group-failure barrier, reports commit in report order: one of a
// barred parent, or one after its parent's first group failure in this
// call, is rejected; an accepted group failure is a failed member.
__global__ __launch_bounds__(kBlock) void k_gather_scatter(
    const uint32_t *__restrict__ rp, const uint32_t *__restrict__ ro_, const uint8_t *__restrict__ rs,
    const int64_t *__restrict__ roff, const uint8_t *data, int64_t n,
    const int64_t *__restrict__ offsets, int64_t P, Canon *__restrict__ canon, int64_t canon_cap,
    int32_t *__restrict__ ns, int32_t *__restrict__ nf, int32_t *__restrict__ nk,
    const uint8_t *__restrict__ barrier, const uint64_t *__restrict__ gkey, uint32_t epoch, Ctl *ctl)
{
    __shared__ int64_t s_wave[kBlock / 64];
    const int64_t N = offsets[P];
    const bool cap_ok = N <= canon_cap;
    const int64_t gtid = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t gstride = (int64_t)gridDim.x * kBlock;
    if (gtid == 0) {
        if (!cap_ok) raise_err(ctl, RO_ECAP);
        if (n > 0 && roff[0] < 0) raise_err(ctl, RO_EINVAL);
    }
    int err = 0;
    // the Expansion must be an exclusive scan: offsets[0] = 0, nondecreasing
    if (gtid == 0 && offsets[0] != 0) err = RO_EINVAL;
    for (int64_t p = gtid; p < P; p += gstride) {
        if (ns) ns[p] = 0;
        if (nf) nf[p] = 0;
        if (nk) nk[p] = 0;
        if (offsets[p + 1] < offsets[p]) err = RO_EINVAL;
    }
    int64_t cnt = 0, rej = 0;
    constexpr int U = kScatterItems;
    // U reports per thread and step, their loads and lookups all in flight
    // before any is validated or stored
    for (int64_t b = gtid; b < n; b += U * gstride) {
        uint32_t sv[U], pv[U], ov[U];
        int64_t o0v[U], o1v[U], stv[U], env[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int64_t i = b + k * gstride;
            const bool in = i < n;
            // the report columns are read once: non-temporal loads leave L2
            // to the slots being written (workload 2's scatter 1.53 -> 1.45 ms)
            sv[k] = in ? __builtin_nontemporal_load(rs + i) : RO_PENDING;
            pv[k] = in ? __builtin_nontemporal_load(rp + i) : 0xffffffffu;
            ov[k] = in ? __builtin_nontemporal_load(ro_ + i) : 0u;
            o0v[k] = in ? __builtin_nontemporal_load(roff + i) : 0;
            o1v[k] = in ? __builtin_nontemporal_load(roff + i + 1) : 0;
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const bool ok = (int64_t)pv[k] < P;
            stv[k] = ok ? offsets[pv[k]] : 0;
            env[k] = ok ? offsets[pv[k] + 1] : 0;
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int64_t i = b + k * gstride;
            if (i >= n) continue;
            uint32_t s = sv[k];
            const int64_t o0 = o0v[k], o1 = o1v[k];
            if (o1 < o0) { err = RO_EINVAL; continue; }
            if (s > RO_PENDING && !(s == RO_GROUP_FAILED && barrier)) { err = RO_ESTATE; continue; }
            if (s == RO_PENDING) continue;
            const uint32_t p = pv[k];
            if ((int64_t)p >= P) { err = RO_ERANGE; continue; }
            const int64_t st = stv[k];
            const uint32_t o = ov[k];
            if ((int64_t)o >= env[k] - st) { err = RO_ERANGE; continue; }
            const int64_t c = st + (int64_t)o;
            if (st < 0 || c >= N) { err = RO_EINVAL; continue; }
            const int64_t len = s == RO_SUCCESS ? o1 - o0 : 0;
            if (len >= ((int64_t)1 << 32)) { err = RO_EOVERFLOW; continue; }
            if (gf_rejected(barrier, gkey, epoch, p, i)) { ++rej; continue; }
            if (s == RO_GROUP_FAILED) s = RO_FAILED;
            ++cnt;
            if (cap_ok) {
                Canon e;
                e.src = reinterpret_cast<uint64_t>(data) + (uint64_t)o0;
                e.len = (uint32_t)len;
                e.tag = (epoch << 2) | s;
                canon[c] = e;
            }
        }
    }
    if (err) raise_err(ctl, err);
    const int64_t tot = block_sum(cnt, s_wave);
    if (threadIdx.x == 0 && tot)
        __hip_atomic_fetch_add(&ctl->n_valid, tot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (barrier) {
        const int64_t r = block_sum(rej, s_wave);
        if (threadIdx.x == 0 && r)
            __hip_atomic_fetch_add(&ctl->n_rejected, r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// ---------------------------------------------------------------- scan
// One tile = kIt * kTh canonical children in groups of 64, a group per load of
// a wave, so that loads, per-child outputs and LDS accesses are all
// lane-contiguous.  Per group the wave keeps, in LDS, the exclusive byte sums
// of its children (DPP scan) and one ballot mask per state; the sums and
// popcounts over the groups then answer any range of the tile.  After the
// look-back over the tiles the work goes by parent, one per thread: a parent
// whose first child is in the tile reads its slot offset at that child and
// its counts as the difference of two positions.  A parent that lies whole in
// the tile has its counts stored; only the one crossing into the tile and the
// one leaving it add to theirs.
//
// A workgroup finishes one tile before it posts anything of the next, but it
// draws tickets two tiles ahead: as soon as a tile's slots are taken from
// their registers, the next tile's parents are searched and its slot loads
// issued, which are then in flight during the look-back and while the parents
// are written.  It takes its tiles in ascending order, so the owner of the
// smallest tile not yet posted never waits on a later one and can always
// post it.
//
// Only as many workgroups as there are tiles take part (the others return at
// once): draws from one ticket take about 12 ns each, one after another, and
// 768 workgroups drawing for two tiles took 40 us (now 11).  Where every tile
// has a workgroup of its own, each draws once.  A single tile
// needs no ticket and no look-back.  What the tiles decide together (every
// report in a slot of its own, bytes within the capacity) is settled by the
// last workgroup to finish, which also clears the call's counters.
//
// In place (the output is the report bytes themselves, as for an upper level
// whose slots are the level below's output): nothing is copied, and the scan
// checks that every surviving record already sits at its output position;
// any other would overwrite bytes still to be read (RO_EINVAL).
// Two tile sizes, chosen on the device, which alone knows the children (a gather
// may have few reports of many, and any reservation): 1,024 children up to
// kScanSmall, a tile for each of 256 CUs, and 8,192 beyond, since a look-back
// reads as many descriptors as there are tiles in flight and every tile draws a
// ticket.  1,000 children 8 us (11 as one large tile), 40,000 11.7 (15.6),
// 262,144 16.0 (15.5), 400,000 20 with small tiles and 16.3, 1M 35 and 17, 41M
// 724 and 220 (tiles of 4,096 with two workgroups of 512 threads 285, of 16,384,
// whose registers spill, 263; walked child by child in tiles of 4,096 305, and
// 1M 39).
constexpr int64_t kScanSmall = 262144;
constexpr int kScanTh = 1024, kScanIt = 8;

// LDS of a tile (sized for the larger)
struct ScanLds {
    static constexpr int kT = kScanTh * kScanIt, kG = kT / kGrp;
    uint64_t pre[kT];                           // exclusive byte sum inside the child's group
    uint64_t gt[kG];                            // byte total of each group
    uint64_t gbase[kG];                         // exclusive byte sum of the groups
    uint64_t m[3][kG + 1];                      // per state: mask of the group's children
    uint64_t cp[kG + 1];                        // exclusive packed counts of the groups
    uint64_t b;
    int64_t t;
    int64_t p[2][2];
    int32_t valid, last;                        // two words: waves still read the first when the second is set
};

template <int kIt, bool kInPlace>
__device__ __forceinline__ void scan_tiles(
    const int64_t *__restrict__ offsets, int64_t P, const Canon *__restrict__ canon, int64_t canon_cap,
    int64_t *__restrict__ out_off, int64_t out_cap, int has_data, int32_t *__restrict__ ns, int32_t *__restrict__ nf,
    int32_t *__restrict__ nk, int64_t *__restrict__ cdst, int64_t *__restrict__ sub_base, const uint8_t *out,
    int64_t *n_rejected, uint32_t epoch, Ctl *ctl, uint64_t *desc, int64_t desc_cap, int64_t N0, int64_t N, ScanLds &lds)
{
    constexpr int kTh = kScanTh;
    constexpr int kT = kTh * kIt;               // children per tile
    constexpr int kG = kT / kGrp;               // groups per tile
    constexpr int kCF = 21, kCK = 42;           // a packed count: SUCCESS, FAILED << 21, SKIPPED << 42
    constexpr uint64_t kCM = (1u << kCF) - 1;
    constexpr int kGL = kG <= 64 ? 1 : kG / 64; // groups per lane of the wave that scans them
    static_assert(kGrp == 64 && (kG <= 64 || kG % 64 == 0) && kIt <= kScanIt, "one wave load per group");
    const int64_t ntiles = (N + kT - 1) / kT;
    const uint32_t parts = ntiles > 1 ? (uint32_t)min64((int64_t)gridDim.x, ntiles) : 1u;
    if (blockIdx.x >= parts) return;
    uint64_t *s_pre = lds.pre, *s_gt = lds.gt, *s_gbase = lds.gbase, *s_cp = lds.cp;
    auto &s_m = lds.m;
    auto &s_p = lds.p;
    uint64_t &s_b = lds.b;
    int64_t &s_t = lds.t;
    int32_t &s_valid = lds.valid, &s_last = lds.last;
    const uint32_t sepoch = scan_epoch(ctl);
    const int wv = uni32((int)(threadIdx.x >> 6)), ln = lane_id();
    // an invalid Expansion found by the scatter: no tiles (one thread looks,
    // since an error may also be raised while the scan runs)
    if (threadIdx.x == 0) s_valid = read_err(ctl) == 0 ? 1 : 0;
    __syncthreads();
    const bool single = ntiles == 1;
    const bool one = ntiles <= (int64_t)gridDim.x;      // one tile and one ticket per workgroup
    int64_t t = s_valid == 0 ? ntiles : (single || ntiles == 0 ? 0 : next_ticket(ctl, &s_t));
    int64_t filled = 0;

    // Tile tt's parents, by waves 1 and 2: q0 is the first parent starting in
    // it, q1 the first one starting after it, one wave-parallel search each.
    auto prepare = [&](int64_t tt, int b) {
        if (wv == 1 || wv == 2) {
            const int64_t c = tt * kT + (wv == 1 ? 0 : min64(kT, N - tt * kT));
            const int64_t r = c == 0 ? 0 : wave_last_le(offsets, 0, P + 1, c - 1) + 1;
            if (ln == 0) s_p[b][wv - 1] = r;
        }
    };
    // The slots of tile tt, group k of the wave into ev[k]: the loads are only
    // issued here.  A slot past the expansion re-reads the tile's first one
    // and is ignored.  Out of place only the length and tag words are read.
    uint2 ev[kIt];
    uint64_t sv[kInPlace ? kIt : 1];
    auto load_slots = [&](int64_t tt) {
        const int64_t a0 = uni64(tt * kT);
        const uint32_t nloc = (uint32_t)uni64(min64(kT, N - a0));
        const uint8_t *tb = reinterpret_cast<const uint8_t *>(canon + a0);
        const uint32_t jb = (uint32_t)(wv * (64 * kIt) + ln);
#pragma unroll
        for (int k = 0; k < kIt; ++k) {
            const uint32_t j = jb + 64u * k, jj = j < nloc ? j : 0u;
            ev[k] = *reinterpret_cast<const uint2 *>(tb + offsetof(Canon, len) + jj * (uint32_t)sizeof(Canon));
            if constexpr (kInPlace) sv[k] = *reinterpret_cast<const uint64_t *>(tb + jj * (uint32_t)sizeof(Canon));
        }
    };

    int buf = 0;
    int64_t t_next = ntiles;
    if (t < ntiles) {
        prepare(t, 0);
        load_slots(t);
        if (!one) t_next = next_ticket(ctl, &s_t);
    }
    while (t < ntiles) {
        __syncthreads();                    // s_p of this tile; the previous tile's LDS is done with
        const int64_t ct0 = t * kT;
        const int nloc = (int)min64(kT, N - ct0);
        const int64_t q0 = s_p[buf][0], q1 = s_p[buf][1];
        int64_t tk = ntiles;                // the ticket after the next, awaited after the look-back
        if (threadIdx.x == 0 && !one)
            tk = (int64_t)__hip_atomic_fetch_add(&ctl->ticket, (uint64_t)1, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
        // this thread's first parent, in flight until then
        int64_t q = q0 + threadIdx.x;
        int64_t a0 = 0, a1 = 0;
        if (q < q1) {
            a0 = offsets[q];
            a1 = offsets[q + 1];
        }
        // groups: surviving lengths, state masks, exclusive byte sums
#pragma unroll
        for (int k = 0; k < kIt; ++k) {
            const int g = wv * kIt + k, i = g * 64 + ln;
            const bool in = i < nloc && (ev[k].y >> 2) == epoch;
            const uint32_t S = in ? ev[k].y & 3u : 4u;
            const uint64_t L = S == RO_SUCCESS ? ev[k].x : 0u;
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
        // the next tile's parents, and its slot loads in flight from here on;
        // meanwhile the first wave gets the tile's group sums and total and
        // does the look-back (its own slot loads follow that, since its polls
        // would wait for them)
        if constexpr (!kInPlace) {
            if (wv != 0 && t_next < ntiles) {
                prepare(t_next, buf ^ 1);
                load_slots(t_next);
            }
        }
        if (wv == 0) {
            uint64_t gt[kGL], gc[kGL], lt = 0, lc = 0;
#pragma unroll
            for (int j = 0; j < kGL; ++j) {
                const int g = ln * kGL + j;
                gt[j] = gc[j] = 0;
                if (g < kG) {
                    gt[j] = s_gt[g];
                    gc[j] = (uint64_t)__popcll(s_m[0][g]) | (uint64_t)__popcll(s_m[1][g]) << kCF |
                            (uint64_t)__popcll(s_m[2][g]) << kCK;
                }
                lt += gt[j];
                lc += gc[j];
            }
            uint64_t gi = wave_incl_sum_dpp(lt), ci = wave_incl_sum_dpp(lc);
            const uint64_t tot = (uint64_t)uni64(__shfl((long long)gi, 63, 64));
            const uint64_t ctot = (uint64_t)uni64(__shfl((long long)ci, 63, 64));
            gi -= lt;
            ci -= lc;
            filled += (int64_t)((ctot & kCM) + ((ctot >> kCF) & kCM) + (ctot >> kCK));
            const uint64_t pr = single ? 0 : lookback_wave(desc, t, sepoch, tot, ctl);
#pragma unroll
            for (int j = 0; j < kGL; ++j) {
                const int g = ln * kGL + j;
                if (g < kG) {
                    s_gbase[g] = gi;
                    s_cp[g] = ci;
                    sub_base[t * kG + g] = (int64_t)(pr + gi);      // first byte of each group
                }
                gi += gt[j];
                ci += gc[j];
            }
            if (ln == 0) {
                s_cp[kG] = ctot;
                s_b = pr;
                s_t = tk;
                if (t == ntiles - 1) {
                    __hip_atomic_store(&ctl->total, (int64_t)(pr + tot), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (pr >= kSat) raise_err(ctl, RO_EOVERFLOW);
                }
            }
        }
        __syncthreads();
        const int64_t pre = (int64_t)s_b;
        const int64_t t_after = s_t;
        if constexpr (kInPlace) {
            const uint64_t outa = reinterpret_cast<uint64_t>(out);
            bool moved = false;
#pragma unroll
            for (int k = 0; k < kIt; ++k) {
                const int g = wv * kIt + k, i = g * 64 + ln;
                const uint64_t pos = (uint64_t)pre + s_gbase[g] + s_pre[i];
                moved |= i < nloc && ev[k].y == ((epoch << 2) | RO_SUCCESS) && ev[k].x != 0 && sv[k] != outa + pos;
            }
            if (moved) raise_err(ctl, RO_EINVAL);
        }
        if (t_next < ntiles && (kInPlace || wv == 0)) {
            if constexpr (kInPlace) prepare(t_next, buf ^ 1);   // the check was the slots' last use
            load_slots(t_next);
        }
        // parents starting in this tile: slot offsets and counts
        auto counts_to = [&](int x) -> uint64_t {
            const int g = x >> 6;
            const uint64_t low = (1ull << (x & 63)) - 1;
            return s_cp[g] + ((uint64_t)__popcll(s_m[0][g] & low) | (uint64_t)__popcll(s_m[1][g] & low) << kCF |
                              (uint64_t)__popcll(s_m[2][g] & low) << kCK);
        };
        while (q < q1) {
            const int st = (int)(a0 - ct0);
            const bool whole = a1 <= ct0 + nloc;
            const uint64_t c = counts_to(whole ? (int)(a1 - ct0) : nloc) - counts_to(st);
            if (out_off) out_off[q] = pre + (int64_t)(s_gbase[st >> 6] + s_pre[st]);
            const int32_t c0 = (int32_t)(c & kCM), c1 = (int32_t)((c >> kCF) & kCM), c2 = (int32_t)(c >> kCK);
            if (whole) {
                ns[q] = c0;
                nf[q] = c1;
                nk[q] = c2;
            } else {
                if (c0) atomicAdd(&ns[q], c0);
                if (c1) atomicAdd(&nf[q], c1);
                if (c2) atomicAdd(&nk[q], c2);
            }
            q += kTh;
            if (q < q1) {
                a0 = offsets[q];
                a1 = offsets[q + 1];
            }
        }
        // the parent reaching into this tile from the one before
        if (threadIdx.x == kTh - 1 && ct0 > 0) {
            const int64_t e = min64(offsets[q0] - ct0, nloc);
            if (e > 0) {
                const uint64_t c = counts_to((int)e);
                const int32_t c0 = (int32_t)(c & kCM), c1 = (int32_t)((c >> kCF) & kCM), c2 = (int32_t)(c >> kCK);
                if (c0) atomicAdd(&ns[q0 - 1], c0);
                if (c1) atomicAdd(&nf[q0 - 1], c1);
                if (c2) atomicAdd(&nk[q0 - 1], c2);
            }
        }
        if (cdst) {
#pragma unroll
            for (int k = 0; k < kIt; ++k) {
                const int g = wv * kIt + k, i = g * 64 + ln;
                if (i < nloc) cdst[ct0 + i] = pre + (int64_t)(s_gbase[g] + s_pre[i]);
            }
        }
        t = t_next;
        t_next = t_after;
        buf ^= 1;
    }
    // the last workgroup to finish: every other one's tiles are posted (its
    // stores were waited for before it counted itself done)
    if (threadIdx.x == 0) {
        int32_t last = 1;
        if (parts > 1) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            const uint64_t o = __hip_atomic_fetch_add(&ctl->gdone, (uint64_t)1 | (uint64_t)filled << 20, __ATOMIC_RELAXED,
                                                      __HIP_MEMORY_SCOPE_AGENT);
            last = (o & 0xfffffu) == parts - 1;
            filled += (int64_t)(o >> 20);
        }
        if (last) {
            const int64_t total = N > 0 ? __hip_atomic_load(&ctl->total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
            if (out_off) out_off[P] = total;
            if (cdst && N0 <= canon_cap) cdst[N0] = total;
            if (n_rejected) *n_rejected = ctl->n_rejected;
            if (filled != ctl->n_valid) raise_err(ctl, RO_EDUP);
            if (has_data && total > out_cap) raise_err(ctl, RO_ECAP);
            // cleared for the next gather (the total is rewritten by every
            // scan with children)
            ctl->n_valid = 0;
            ctl->n_rejected = 0;
            __hip_atomic_store(&ctl->gdone, (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        s_last = last;
    }
    __syncthreads();
    if (parts > 1 && s_last) ticket_reset(ctl, sepoch, desc, desc_cap);
}

template <bool kInPlace>
__global__ __launch_bounds__(kScanTh) void k_gather_scan(
    const int64_t *__restrict__ offsets, int64_t P, const Canon *__restrict__ canon, int64_t canon_cap,
    int64_t *__restrict__ out_off, int64_t out_cap, int has_data, int32_t *__restrict__ ns, int32_t *__restrict__ nf,
    int32_t *__restrict__ nk, int64_t *__restrict__ cdst, int64_t *__restrict__ sub_base, const uint8_t *out,
    int64_t *n_rejected, uint32_t epoch, Ctl *ctl, uint64_t *desc, int64_t desc_cap)
{
    __shared__ ScanLds lds;
    const int64_t N0 = offsets[P];
    const int64_t N = N0 <= canon_cap ? N0 : 0;
    if (N <= kScanSmall)
        scan_tiles<1, kInPlace>(offsets, P, canon, canon_cap, out_off, out_cap, has_data, ns, nf, nk, cdst, sub_base, out,
                                n_rejected, epoch, ctl, desc, desc_cap, N0, N, lds);
    else
        scan_tiles<kScanIt, kInPlace>(offsets, P, canon, canon_cap, out_off, out_cap, has_data, ns, nf, nk, cdst, sub_base,
                                      out, n_rejected, epoch, ctl, desc, desc_cap, N0, N, lds);
}

// ---------------------------------------------------------------- finalize
// Complete / state of every parent from its counts, once the scan is done, and
// the slot offsets of parents with no child at or after their start.  Part of
// the copy's launch where there is one (one launch less, about 5 us of a
// small gather), else a launch of its own.  `g0` of `gn` threads.
__device__ __forceinline__ void finalize_parents(const GatherFin &f, int64_t g0, int64_t gn, int64_t N, int64_t total)
{
    for (int64_t p = g0; p < f.P; p += gn) {
        const int64_t st = f.offsets[p];
        const int64_t k = f.offsets[p + 1] - st;
        if (st >= N && f.out_off) f.out_off[p] = total;
        const int64_t a = f.ns[p], b = f.nf[p], c = f.nk[p];
        // a barred parent's uncommitted children are suppressed: it is done
        bool barred = false;
        if (f.barrier) {
            barred = f.barrier[p] || (uint32_t)(f.gkey[p] >> 32) == f.epoch;
            if (barred) f.barrier[p] = 1;
        }
        const bool done = barred || (a + b + c) == k;
        if (f.complete) f.complete[p] = done ? 1 : 0;
        if (f.pstate) f.pstate[p] = !done ? RO_PENDING : ((barred || b > 0) ? RO_FAILED : RO_SUCCESS);
    }
}

__global__ __launch_bounds__(kBlock) void k_gather_finalize(GatherFin f, const Ctl *ctl)
{
    const int64_t N0 = f.offsets[f.P];
    const int64_t N = N0 <= f.canon_cap ? N0 : 0;
    finalize_parents(f, (int64_t)blockIdx.x * kBlock + threadIdx.x, (int64_t)gridDim.x * kBlock, N,
                     N > 0 ? ctl->total : 0);
}

// ---------------------------------------------------------------- copy
// Each wave works alone on its units of output bytes, with no workgroup
// barrier.  A unit starts at the group of 64 canonical children that holds
// its first byte (a wave search over the groups' first bytes) and takes four
// groups at a time: the groups' starts are known from the scan, so each group
// needs only the exclusive sum of its own lengths, and a group past the
// unit's end is not read.  Every record is clipped to the unit's byte range
// (shifting the source start of a record that begins before it), and that
// range is written with aligned 16-byte stores.  Byte-sized units keep the
// chip busy whether the records are a few bytes or megabytes long, and few
// parents or many.
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(RO_COPY_WAVES))) void k_gather_copy(
    GatherFin fin, const Canon *__restrict__ canon, const int64_t *__restrict__ sub_base, uint8_t *__restrict__ out,
    int64_t slots, Ctl *ctl)
{
    constexpr int kWaves = kBlock / 64;
    constexpr int kGroups = kSub / kGrp;
    __shared__ int32_t s_dst_all[kWaves][kSub + 1];     // clipped destination offset of each record
    __shared__ uint64_t s_src_all[kWaves][kSub];        // source address of its first clipped byte
    __shared__ int32_t s_edge_all[kWaves][kEdgeCap];    // edge chunks of the window
    __shared__ int16_t s_edger_all[kWaves][kEdgeCap];   // the record holding each one's first byte
    const int64_t N0 = fin.offsets[fin.P];
    const int64_t N = N0 <= fin.canon_cap ? N0 : 0;
    const int64_t T = N > 0 ? ctl->total : 0;           // output bytes, from the scan
    const uint32_t epoch = fin.epoch;
    // parents go to the workgroups from the last one on, which have no unit
    // in a small copy
    finalize_parents(fin, (int64_t)(gridDim.x - 1 - blockIdx.x) * kBlock + threadIdx.x, (int64_t)gridDim.x * kBlock, N, T);
    if (T <= 0 || read_err(ctl) != 0) return;            // any recorded error: copy nothing
    const int64_t ngrp = (N + kGrp - 1) / kGrp;
    const uint64_t outa = reinterpret_cast<uint64_t>(out);
    const int64_t mis = (int64_t)(outa & 15);
    const int64_t nwaves = (int64_t)gridDim.x * kWaves;
    int64_t G, nunits;
    copy_units(T, slots, mis, G, nunits);
    const int wave = uni32((int)(threadIdx.x >> 6)), lane = lane_id();
    int32_t *s_dst = s_dst_all[wave];
    uint64_t *s_src = s_src_all[wave];
    int32_t *s_edge = s_edge_all[wave];
    int16_t *s_edger = s_edger_all[wave];
    for (int64_t u = (int64_t)blockIdx.x * kWaves + wave; u < nunits; u += nwaves) {
        const int64_t lo = max64(u * G - mis, 0);
        const int64_t hi = min64((u + 1) * G - mis, T);
        for (int64_t g = uni64(wave_last_le(sub_base, 0, ngrp, lo)); g < ngrp; g += kGroups) {
            // first bytes of the window's groups and of the one after it
            const int64_t gl = g + (lane < kGroups ? lane : kGroups);
            const int64_t dl = gl < ngrp ? sub_base[gl] : T;
            int64_t D[kGroups + 1];
#pragma unroll
            for (int k = 0; k <= kGroups; ++k) D[k] = uni64(__shfl(dl, k, 64));
            if (D[0] >= hi) break;
            // this unit's part of the window
            const int64_t ws = max64(lo, D[0]), we = min64(hi, D[kGroups]);
            if (we > ws) {
                // whole 16-byte slots, the loads of all groups in flight
                // together (a slot past the expansion re-reads the last one
                // and is ignored; a group past the unit holds nothing of it)
                uint4 ev[kGroups];
#pragma unroll
                for (int k = 0; k < kGroups; ++k) {
                    const int64_t c = (g + k) * kGrp + lane;
                    ev[k] = make_uint4(0, 0, 0, 0);
                    if (D[k] < we) ev[k] = ld16(reinterpret_cast<uint64_t>(&canon[c < N ? c : N - 1]));
                }
#pragma unroll
                for (int k = 0; k < kGroups; ++k) {
                    const int r = k * kGrp + lane;
                    if (D[k] < we) {
                        const bool ok = g * kGrp + r < N && ev[k].w == ((epoch << 2) | RO_SUCCESS);
                        const uint32_t l = ok ? ev[k].z : 0u;
                        const int64_t run = D[k] + (int64_t)wave_incl_sum_dpp(l) - l;
                        const int64_t cs = min64(max64(run, ws), we);
                        s_dst[r] = (int32_t)(cs - ws);
                        s_src[r] = (ok ? ((uint64_t)ev[k].y << 32 | ev[k].x) : 0ull) + (uint64_t)(cs - run);
                    } else {
                        s_dst[r] = (int32_t)(we - ws);
                        s_src[r] = 0;
                    }
                }
                if (lane == 0) s_dst[kSub] = (int32_t)(we - ws);
                __builtin_amdgcn_wave_barrier();
                copy_window_nb<RO_COPY_STEPS>(s_dst, s_src, s_edge, s_edger, (int)(we - ws), outa, ws, lane);
                __builtin_amdgcn_wave_barrier();
            }
            if (D[kGroups] >= hi) break;
        }
    }
}

hipError_t launch_gather(const Launch &L, const GatherArgs &a, const GatherWs &w, uint32_t epoch)
{
    if (a.barrier != nullptr && a.n > 0) {
        const hipError_t e = launch_first_gf(L, a.rs, a.rp, a.n, a.P, a.barrier, w.gkey, epoch);
        if (e != hipSuccess) return e;
    }
    const int64_t grid_r = (int64_t)L.num_cus * 8;
    RO_LAUNCH(L, RO_K_GATHER_SCATTER, k_gather_scatter, dim3((unsigned)grid_r), dim3(kBlock), 0, L.stream,
              a.rp, a.ro, a.rs, a.roff, a.data, a.n, a.offsets, a.P, w.canon, w.canon_cap, a.ns, a.nf,
              a.nk, a.barrier, w.gkey, epoch, L.ctl);
    // output aliasing the report bytes: the scan checks that nothing moves,
    // and there is nothing to copy
    const bool in_place = a.out_data != nullptr && a.out_data == a.data;
    auto scan = in_place ? k_gather_scan<true> : k_gather_scan<false>;
    RO_LAUNCH(L, RO_K_GATHER_SCAN, scan, dim3((unsigned)L.num_cus), dim3(kScanTh), 0, L.stream, a.offsets,
              a.P, w.canon, w.canon_cap, a.out_off, a.out_cap, a.out_data != nullptr ? 1 : 0, a.ns, a.nf, a.nk, a.cdst,
              w.sub_base, a.out_data, a.n_rejected, epoch, L.ctl, L.desc, L.desc_cap);
    GatherFin fin;
    fin.offsets = a.offsets;
    fin.P = a.P;
    fin.canon_cap = w.canon_cap;
    fin.out_off = a.out_off;
    fin.ns = a.ns;
    fin.nf = a.nf;
    fin.nk = a.nk;
    fin.complete = a.complete;
    fin.pstate = a.pstate;
    fin.barrier = a.barrier;
    fin.gkey = w.gkey;
    fin.epoch = epoch;
    int64_t grid_f = (a.P + kBlock - 1) / kBlock;
    grid_f = grid_f < 1 ? 1 : (grid_f > (int64_t)L.num_cus * 8 ? (int64_t)L.num_cus * 8 : grid_f);
    if (a.out_data == nullptr || in_place)
        RO_LAUNCH(L, RO_K_GATHER_FINALIZE, k_gather_finalize, dim3((unsigned)grid_f), dim3(kBlock), 0, L.stream, fin,
                  L.ctl);
    if (a.out_data != nullptr && !in_place) {
        // One unit per wave, handed out in output order as workgroups end, as
        // far as out_cap (the most the total can be) asks for them: a
        // persistent grid striding over the units was slower.
        const int64_t slots = (int64_t)L.num_cus * 4 * RO_COPY_WAVES;
        const int64_t max_c = (int64_t)L.num_cus * RO_COPY_GRID, max_s = (int64_t)L.num_cus * 32;
        const int64_t big_c = a.out_cap / (kCopyUnit * 4) + 1, small_c = a.out_cap / (kCopyMinUnit * 4) + 1;
        int64_t grid_c = small_c < max_s ? small_c : max_s;
        grid_c = big_c > grid_c ? (big_c < max_c ? big_c : max_c) : grid_c;
        grid_c = grid_c > grid_f ? grid_c : grid_f;         // and enough for the parents
        RO_LAUNCH(L, RO_K_GATHER_COPY, k_gather_copy, dim3((unsigned)grid_c), dim3(kBlock), 0, L.stream, fin, w.canon,
                  w.sub_base, a.out_data, slots, L.ctl);
    }
    return hipGetLastError();
}

}  // namespace ro
