// Grain phases and the generation fence on gfx950.
//
// RayOrch (arXiv 2609.18703), Sec. 4: a Grain goes WAITING -> READY ->
// IN-FLIGHT -> SEALED, and a retry takes IN-FLIGHT back to READY (Eq.
// grain-phase); a report commits only while its Grain is in flight at the
// report's generation (Eq. generation-fence); a repeat of a committed fact is
// idempotent and a conflicting one is rejected (publication rules).
//
// Reports and reservations come in any order, so each of them is a random
// access.  A phase is one bit in each of two words of 32 children (in flight;
// sealed), and a generation is read only where a third says that the child was
// ever retried: one 16-byte record, and one load, per 32 children, which reads
// find in cache (a 16-byte record per child took a line from memory for every
// load and every atomic).  Reserving sets the child's in-flight bit, which also
// catches a child named twice and a sealed one (sealing leaves the bit set).
//
// A commit call first validates and tests the fence, and finds the children
// with several passing reports and the first of each (in report order).  Every
// other report is accepted or stale; of those the first is accepted, another
// one's state and bytes are compared with it by 16 lanes, 16 bytes a lane and
// load.
//
// Random returning atomics reach about 26 x 10^9 a second on this chip however
// small the bitmap is (10M reservations: 387 us on 1.25 MB, 441 on records of
// 160 MB; now 108).  So a large call sorts its children into at most 512 bins of
// neighbours first, in LDS tile by tile and with coalesced stores, and one
// workgroup per bin then sets the bits in LDS (use_bins).  A commit of 10.2M
// reports with 1.2% repeats in random order takes 350 us (two passes over
// records: 1,330, of them 820 in the second, where a wave compared its lanes'
// repeats one by one, byte by byte).
//
// A smaller call goes by atomics, in two passes whose cost follows its reports
// and not the table.  A commit seals every child that passes, so a child's entry
// of `first` and its contested bit serve one commit between two resets, and only
// the reset clears them.  (Bitmaps cleared by each call took a third pass, which
// swept the table: 1,000 reports a commit 15.8 us on 100,000 children and 40 on
// 400M, now 12.9 and 20; 300,000 on 400M 90 and 57.)
#include "ro_copy.h"

namespace ro {

constexpr int kGItems = 4;

// cidx of a report that did not pass the fence, and of one that is not counted;
// kNone also in `first`, for no report
constexpr uint32_t kStale = 0xfffffffeu, kNone = 0xffffffffu;

// Every child READY at generation 0, with no report: the bitmaps and the bins'
// counts to zero, `first` to no report.
__global__ void k_grains_fill(uint4 *__restrict__ zero, int64_t n_zero, uint4 *__restrict__ first, int64_t n_first)
{
    const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = tid; i < n_zero; i += stride) zero[i] = make_uint4(0, 0, 0, 0);
    for (int64_t i = tid; i < n_first; i += stride) first[i] = make_uint4(kNone, kNone, kNone, kNone);
}

// Phase and generation of every Grain, for inspection.
__global__ void k_grains_read(GrainTab g, int64_t n, uint32_t *__restrict__ phase, uint32_t *__restrict__ gen)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t bit = 1u << (i & 31);
        const GrainBits f = g.bits[i >> 5];
        if (phase) phase[i] = (f.sealed & bit) ? RO_SEALED : ((f.inflight & bit) ? RO_IN_FLIGHT : RO_READY);
        if (gen) gen[i] = (f.retried & bit) ? g.gen[i] : 0u;
    }
}

// READY -> IN-FLIGHT; the attempt's generation goes out.
__global__ __launch_bounds__(kBlock) void k_grains_dispatch(const uint32_t *__restrict__ child, int64_t n, int64_t N,
                                                            GrainTab g, uint32_t *__restrict__ out_gen, Ctl *ctl)
{
    int err = 0;
    const int64_t span = (int64_t)kBlock * kGItems;
    for (int64_t base = (int64_t)blockIdx.x * span; base < n; base += (int64_t)gridDim.x * span) {
        uint32_t c[kGItems], retried[kGItems];
        bool ok[kGItems], set[kGItems];
#pragma unroll
        for (int k = 0; k < kGItems; ++k) {
            const int64_t i = base + k * kBlock + threadIdx.x;
            c[k] = i < n ? child[i] : 0u;
            ok[k] = i < n && (int64_t)c[k] < N;
            if (i < n && !ok[k]) err = RO_ERANGE;
        }
#pragma unroll
        for (int k = 0; k < kGItems; ++k) retried[k] = ok[k] && out_gen ? g.bits[c[k] >> 5].retried : 0u;
#pragma unroll
        for (int k = 0; k < kGItems; ++k) {
            const uint32_t bit = 1u << (c[k] & 31u);
            set[k] = (change_bits<true>(&g.bits[c[k] >> 5].inflight, bit, ok[k]) & bit) != 0;
        }
#pragma unroll
        for (int k = 0; k < kGItems; ++k) {
            if (!ok[k]) continue;
            if (set[k]) { err = RO_ESTATE; continue; }       // in flight, sealed, or named twice in this call
            if (out_gen)
                out_gen[base + k * kBlock + threadIdx.x] = ((retried[k] >> (c[k] & 31u)) & 1u) ? g.gen[c[k]] : 0u;
        }
    }
    if (err) raise_err(ctl, err);
}

// IN-FLIGHT (not sealed) -> READY at the next generation.  Only the thread
// that cleared a child's bit writes its generation.
__global__ __launch_bounds__(kBlock) void k_grains_retry(const uint32_t *__restrict__ child, int64_t n, int64_t N,
                                                         GrainTab g, Ctl *ctl)
{
    int err = 0;
    const int64_t span = (int64_t)kBlock * kGItems;
    for (int64_t base = (int64_t)blockIdx.x * span; base < n; base += (int64_t)gridDim.x * span) {
        uint32_t c[kGItems];
        GrainBits f[kGItems];
        bool ok[kGItems];
#pragma unroll
        for (int k = 0; k < kGItems; ++k) {
            const int64_t i = base + k * kBlock + threadIdx.x;
            c[k] = i < n ? child[i] : 0u;
            ok[k] = i < n && (int64_t)c[k] < N;
            if (i < n && !ok[k]) err = RO_ERANGE;
        }
#pragma unroll
        for (int k = 0; k < kGItems; ++k) f[k] = ok[k] ? g.bits[c[k] >> 5] : GrainBits{0, 0, 0, 0};
#pragma unroll
        for (int k = 0; k < kGItems; ++k) {
            const uint32_t bit = 1u << (c[k] & 31u);
            const bool open = ok[k] && !(f[k].sealed & bit);
            const bool mine = (change_bits<false>(&g.bits[c[k] >> 5].inflight, bit, open) & bit) != 0 && open;
            if (ok[k] && !mine) err = RO_ESTATE;
            const bool again = (f[k].retried & bit) != 0;
            if (mine) g.gen[c[k]] = again ? g.gen[c[k]] + 1u : 1u;
            (void)change_bits<true>(&g.bits[c[k] >> 5].retried, bit, mine && !again);
        }
    }
    if (err) raise_err(ctl, err);
}

// ---- bins
// Children c of bin b = c >> shift are neighbours, so the bits a bin sets are
// one stretch of the bitmap, which fits LDS.  A tile of children is counted per
// bin (the count at which an entry finds its bin is its rank there), gets room
// in every bin with one atomic, is put in order of bins in LDS and written out:
// with 8,192 or 16,384 entries over at most 512 bins a bin's run is mostly a
// line.
struct Bins {
    int shift, n;
};
constexpr int kMaxBinShift = 17;

// Adds one to the counter of every valid lane's bin; returns what it held
// before (a value of its own per lane).  Lanes of one bin, as in a queue in
// canonical order, add once for all.
__device__ __forceinline__ uint32_t bin_rank(uint32_t *s_cnt, uint32_t b, bool valid)
{
    const uint64_t vm = __ballot(valid);
    if (vm == 0) return 0;
    const int l0 = __ffsll((unsigned long long)vm) - 1;
    const uint32_t b0 = (uint32_t)__shfl((int)b, l0, 64);
    if (__ballot(valid && b != b0) == 0) {
        uint32_t at = 0;
        if (lane_id() == l0) at = atomicAdd(&s_cnt[b0], (uint32_t)__popcll(vm));
        at = (uint32_t)__shfl((int)at, l0, 64);
        return at + (uint32_t)__popcll(vm & ((1ull << lane_id()) - 1ull));
    }
    return valid ? atomicAdd(&s_cnt[b], 1u) : 0u;
}


// Pass 1: validation and the fence.  Per report its provisional outcome in
// state_out (its state if it passed, RO_PENDING if not) and, if it passed, its
// child in cidx.  Two reports of one child meet at its entry of `first`, which
// ends as the smaller index; the later to arrive marks the child contested.
// With bins only the reports per bin are counted.
template <bool kBins>
__global__ __launch_bounds__(kBlock) void k_grains_first(
    const uint32_t *__restrict__ rp, const uint32_t *__restrict__ ro_, const uint8_t *__restrict__ rs,
    const int64_t *__restrict__ roff, const uint32_t *__restrict__ rgen, int64_t n,
    const int64_t *__restrict__ offsets, int64_t P, int64_t N, GrainTab g, Bins bins, uint32_t *__restrict__ cidx,
    uint8_t *__restrict__ state_out, int64_t *counts, Ctl *ctl)
{
    __shared__ uint32_t s_hist[kBins ? kGrainBins : 1];
    if constexpr (kBins) {
        for (int b = threadIdx.x; b < kGrainBins; b += kBlock) s_hist[b] = 0;
        __syncthreads();
    }
    if (blockIdx.x == 0 && threadIdx.x < 4 && counts) counts[threadIdx.x] = 0;
    if (blockIdx.x == 0 && threadIdx.x < 2) g.n_list[threadIdx.x] = 0;
    int err = 0;
    const int64_t span = (int64_t)kBlock * kGItems;
    for (int64_t base = (int64_t)blockIdx.x * span; base < n; base += (int64_t)gridDim.x * span) {
        uint32_t p[kGItems], o[kGItems], s[kGItems], gen[kGItems], c[kGItems];
        int64_t o0[kGItems], o1[kGItems], st[kGItems], en[kGItems];
        GrainBits f[kGItems];
        bool ok[kGItems], met[kGItems];
#pragma unroll
        for (int k = 0; k < kGItems; ++k) {
            const int64_t i = base + k * kBlock + threadIdx.x;
            const bool in = i < n;
            s[k] = in ? rs[i] : (uint32_t)RO_PENDING;
            p[k] = in ? rp[i] : 0xffffffffu;
            o[k] = in ? ro_[i] : 0u;
            gen[k] = in ? rgen[i] : 0u;
            o0[k] = in ? roff[i] : 0;
            o1[k] = in ? roff[i + 1] : 0;
        }
#pragma unroll
        for (int k = 0; k < kGItems; ++k) {
            // both offsets with one load: a random access costs by the lane
            const v2i64 e = (int64_t)p[k] < P ? ld_pair(offsets + p[k]) : v2i64{0, 0};
            st[k] = e.x;
            en[k] = e.y;
        }
#pragma unroll
        for (int k = 0; k < kGItems; ++k) {
            ok[k] = false;
            c[k] = 0;
            if (o1[k] < o0[k]) { err = RO_EINVAL; continue; }
            if (s[k] > RO_GROUP_FAILED) { err = RO_ESTATE; continue; }
            if (s[k] == RO_PENDING) continue;
            if ((int64_t)p[k] >= P) { err = RO_ERANGE; continue; }
            if ((int64_t)o[k] >= en[k] - st[k]) { err = RO_ERANGE; continue; }
            if (st[k] < 0) { err = RO_EINVAL; continue; }         // offsets not an Expansion
            if (st[k] + (int64_t)o[k] >= N) { err = RO_ERANGE; continue; }
            c[k] = (uint32_t)(st[k] + (int64_t)o[k]);
            ok[k] = true;
        }
#pragma unroll
        for (int k = 0; k < kGItems; ++k) f[k] = ok[k] ? g.bits[c[k] >> 5] : GrainBits{0, 0, 0, 0};
#pragma unroll
        for (int k = 0; k < kGItems; ++k) {
            const uint32_t bit = 1u << (c[k] & 31u);
            ok[k] = ok[k] && (f[k].inflight & ~f[k].sealed & bit) && gen[k] == ((f[k].retried & bit) ? g.gen[c[k]] : 0u);
        }
#pragma unroll
        for (int k = 0; k < kGItems; ++k) {
            met[k] = false;
            if constexpr (kBins) {
                (void)bin_rank(s_hist, c[k] >> bins.shift, ok[k]);
            } else if (ok[k]) {
                const uint32_t i = (uint32_t)(base + k * kBlock + threadIdx.x);
                met[k] = __hip_atomic_fetch_min(&g.first[c[k]], i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != kNone;
            }
        }
#pragma unroll
        for (int k = 0; k < kGItems; ++k) {
            const int64_t i = base + k * kBlock + threadIdx.x;
            if (i >= n) continue;
            state_out[i] = ok[k] ? (uint8_t)s[k] : (uint8_t)RO_PENDING;
            if (kBins || ok[k]) cidx[i] = ok[k] ? c[k] : (s[k] == RO_PENDING ? kNone : kStale);
            if (met[k])
                __hip_atomic_fetch_or(&g.contested[c[k] >> 5], 1u << (c[k] & 31u), __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    if constexpr (kBins) {
        __syncthreads();
        for (int b = threadIdx.x; b < bins.n; b += kBlock)
            if (s_hist[b])
                __hip_atomic_fetch_add(&g.hist[b], s_hist[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (err) raise_err(ctl, err);
}

// Settles contested reports, one per lane with `have` set: report i, whose child's
// first one is first[c].  Another than that is a duplicate if state, length and (for
// SUCCESS) bytes are the same, a conflict otherwise.  Returns 0 for the first
// itself, 1 for a duplicate, 2 for a conflict, -1 without a report.  A wave looks
// at 64 reports at once, which is a chain of four loads, queues the comparisons
// in LDS, and takes four of them at a time with 16 lanes each (taking a report's
// chain by 16 lanes: 118 us for 240,000 listed reports, now 90).  The bytes go
// 16 to a lane and load, four loads of each copy in flight; the last load of a
// record overlaps the one before, so that none reads past its end.
constexpr int kCmpLanes = 16, kCmpSteps = 4;

struct CmpJobs {
    int64_t a[64], b[64], len[64];
    int32_t diff[64];
};

__device__ __forceinline__ int settle_wave(bool have, int64_t i, uint32_t c, const uint8_t *__restrict__ rs,
                                           const int64_t *__restrict__ roff, const uint8_t *__restrict__ data,
                                           const uint32_t *__restrict__ first, uint8_t *__restrict__ state_out,
                                           CmpJobs &jobs)
{
    const int lane = lane_id(), sub = lane & (kCmpLanes - 1);
    int kind = -1;
    int64_t a = 0, b = 0, len = 0;
    bool job = false;
    if (have) {
        const uint32_t s = rs[i];
        b = roff[i];
        len = roff[i + 1] - b;
        const int64_t v = first[c];
        kind = 0;
        if (v != i) {
            a = roff[v];
            const bool same = rs[v] == s && (s != RO_SUCCESS || roff[v + 1] - a == len);
            job = same && s == RO_SUCCESS && data != nullptr && len > 0;
            kind = same ? 1 : 2;
            state_out[i] = RO_PENDING;
        }
    }
    const uint64_t jm = __ballot(job);
    const int slot = (int)__popcll(jm & ((1ull << lane) - 1ull)), nj = (int)__popcll(jm);
    if (job) {
        jobs.a[slot] = a;
        jobs.b[slot] = b;
        jobs.len[slot] = len;
    }
    __builtin_amdgcn_wave_barrier();
    for (int q = lane / kCmpLanes; q < nj; q += 64 / kCmpLanes) {
        const uint8_t *pa = data + jobs.a[q], *pb = data + jobs.b[q];
        const int64_t l = jobs.len[q];
        uint32_t diff = 0;
        if (l < 16) {
            if (sub < l) diff = (uint32_t)(pa[sub] ^ pb[sub]);
        } else {
            constexpr int64_t kStep = 16 * kCmpLanes * kCmpSteps;
            for (int64_t x = (int64_t)sub * 16; x < l && diff == 0; x += kStep) {
                v4u32 A[kCmpSteps], B[kCmpSteps];
#pragma unroll
                for (int u = 0; u < kCmpSteps; ++u) {
                    const int64_t y = min64(x + u * (16 * kCmpLanes), l - 16);
                    A[u] = ld16v(reinterpret_cast<uint64_t>(pa + y));
                    B[u] = ld16v(reinterpret_cast<uint64_t>(pb + y));
                }
#pragma unroll
                for (int u = 0; u < kCmpSteps; ++u) {
                    const v4u32 d = A[u] ^ B[u];
                    diff |= d.x | d.y | d.z | d.w;
                }
            }
        }
        // lanes of this comparison that found a difference
        const uint64_t dm = __ballot(diff != 0) >> (lane & ~(kCmpLanes - 1));
        if (sub == 0) jobs.diff[q] = (dm & ((1u << kCmpLanes) - 1u)) != 0;
    }
    __builtin_amdgcn_wave_barrier();
    if (job && jobs.diff[slot]) kind = 2;
    __builtin_amdgcn_wave_barrier();
    return kind;
}

// Pass 2 of a call without bins: the children of passing reports become sealed
// (also after a bad report); a report that did not pass is stale, one of a child
// with no other report is accepted, those of contested children are settled.
__global__ __launch_bounds__(kBlock) void k_grains_decide(const uint8_t *__restrict__ rs,
                                                          const int64_t *__restrict__ roff,
                                                          const uint8_t *__restrict__ data, int64_t n, GrainTab g,
                                                          const uint32_t *__restrict__ cidx,
                                                          uint8_t *__restrict__ state_out, int64_t *counts, Ctl *ctl)
{
    __shared__ int64_t s_wave[kBlock / 64];
    __shared__ CmpJobs s_jobs[kBlock / 64];
    __shared__ int32_t s_err;
    if (threadIdx.x == 0) s_err = read_err(ctl);     // the first pass found a bad report
    __syncthreads();
    const bool bad = s_err != 0;
    int64_t cnt[4] = {0, 0, 0, 0};                   // accepted, stale, duplicate, conflict
    const int64_t span = (int64_t)kBlock * kGItems;
    for (int64_t base = (int64_t)blockIdx.x * span; base < n; base += (int64_t)gridDim.x * span) {
        uint32_t so[kGItems], s[kGItems], c[kGItems], w[kGItems];
#pragma unroll
        for (int k = 0; k < kGItems; ++k) {
            const int64_t i = base + k * kBlock + threadIdx.x;
            so[k] = i < n ? state_out[i] : (uint32_t)RO_PENDING;
            s[k] = i < n ? rs[i] : (uint32_t)RO_PENDING;
            c[k] = so[k] != RO_PENDING ? cidx[i] : 0u;
        }
#pragma unroll
        for (int k = 0; k < kGItems; ++k) w[k] = so[k] != RO_PENDING ? g.contested[c[k] >> 5] >> (c[k] & 31u) & 1u : 0u;
#pragma unroll
        for (int k = 0; k < kGItems; ++k)
            (void)change_bits<true>(&g.bits[c[k] >> 5].sealed, 1u << (c[k] & 31u), so[k] != RO_PENDING);
        if (bad) continue;
#pragma unroll
        for (int k = 0; k < kGItems; ++k) {
            const bool two = w[k] != 0;
            cnt[0] += so[k] != RO_PENDING && !two;
            cnt[1] += so[k] == RO_PENDING && s[k] != RO_PENDING;
            if (__ballot(two) == 0) continue;
            const int kind = settle_wave(two, base + k * kBlock + threadIdx.x, c[k], rs, roff, data, g.first, state_out,
                                         s_jobs[threadIdx.x >> 6]);
            cnt[0] += kind == 0;
            cnt[2] += kind == 1;
            cnt[3] += kind == 2;
        }
    }
    if (counts && !bad) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t t = block_sum(cnt[q], s_wave);
            if (threadIdx.x == 0 && t)
                __hip_atomic_fetch_add(&counts[q], t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

constexpr int kSplitTh = 1024;

// Exclusive sums of one value per thread for the first kGrainBins threads of a
// workgroup of kSplitTh; s_w holds kGrainBins / 64 entries.
__device__ __forceinline__ uint32_t bins_excl_scan(uint32_t v, uint32_t *s_w)
{
    const int wv = (int)(threadIdx.x >> 6);
    uint32_t inc = 0;
    if (threadIdx.x < kGrainBins) {
        inc = (uint32_t)wave_incl_sum_dpp(v);
        if (lane_id() == 63) s_w[wv] = inc;
    }
    __syncthreads();
    uint32_t ex = inc - v;
#pragma unroll
    for (int i = 0; i < kGrainBins / 64; ++i) ex += i < wv ? s_w[i] : 0;
    __syncthreads();
    return ex;
}

// A tile's children in order of bins, in LDS: afterwards s_k[0, total) holds
// them (and s_i their report indices), and entry j goes to place s_base[b] + j
// of the bins' array, b being its bin.  `place` gives the first place of the
// calling thread's bin for a given number of entries.
template <int kIt, bool kPairs, typename Place>
__device__ __forceinline__ uint32_t split_tile(const uint32_t (&c)[kIt], const bool (&ok)[kIt], int64_t i0, Bins bins,
                                               uint32_t *s_cnt, uint32_t *s_base, uint32_t *s_w, uint32_t *s_k,
                                               uint32_t *s_i, Place place)
{
    const int tid = (int)threadIdx.x;
    if (tid <= kGrainBins) s_cnt[tid] = 0;
    __syncthreads();
    uint32_t rank[kIt];
#pragma unroll
    for (int k = 0; k < kIt; ++k) rank[k] = bin_rank(s_cnt, c[k] >> bins.shift, ok[k]);
    __syncthreads();
    const uint32_t v = tid < kGrainBins ? s_cnt[tid] : 0u;
    const uint32_t ex = bins_excl_scan(v, s_w);
    if (tid < kGrainBins) {
        if (v) s_base[tid] = place(tid, v) - ex;
        s_cnt[tid] = ex;
        if (tid == kGrainBins - 1) s_cnt[kGrainBins] = ex + v;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kIt; ++k) {
        if (!ok[k]) continue;
        const uint32_t at = s_cnt[c[k] >> bins.shift] + rank[k];
        s_k[at] = c[k];
        if constexpr (kPairs) s_i[at] = (uint32_t)(i0 + k * kSplitTh + tid);
    }
    __syncthreads();
    return s_cnt[kGrainBins];
}

// A large reservation: generations out and the children into the bins.  A bin
// has room for each of its children once (its stretch of `room`); a child beyond
// that, in a bin where some child is named twice, sets its bit here.
constexpr int kDispIt = 16;

__global__ __launch_bounds__(kSplitTh) void k_grains_dispatch_split(const uint32_t *__restrict__ child, int64_t n,
                                                                    int64_t N, GrainTab g, Bins bins,
                                                                    uint32_t *__restrict__ out_gen, Ctl *ctl)
{
    __shared__ uint32_t s_k[kSplitTh * kDispIt];
    __shared__ uint32_t s_cnt[kGrainBins + 1], s_base[kGrainBins], s_w[kGrainBins / 64];
    int err = 0;
    const int64_t span = (int64_t)kSplitTh * kDispIt;
    for (int64_t base = (int64_t)blockIdx.x * span; base < n; base += (int64_t)gridDim.x * span) {
        uint32_t c[kDispIt];
        bool ok[kDispIt];
#pragma unroll
        for (int k = 0; k < kDispIt; ++k) {
            const int64_t i = base + k * kSplitTh + threadIdx.x;
            c[k] = i < n ? child[i] : 0u;
            ok[k] = i < n && (int64_t)c[k] < N;
            if (i < n && !ok[k]) err = RO_ERANGE;
        }
        if (out_gen) {
            uint32_t retried[kDispIt];
#pragma unroll
            for (int k = 0; k < kDispIt; ++k) retried[k] = ok[k] ? g.bits[c[k] >> 5].retried : 0u;
#pragma unroll
            for (int k = 0; k < kDispIt; ++k)
                if (ok[k])
                    out_gen[base + k * kSplitTh + threadIdx.x] =
                        ((retried[k] >> (c[k] & 31u)) & 1u) ? g.gen[c[k]] : 0u;
        }
        const uint32_t tot = split_tile<kDispIt, false>(c, ok, base, bins, s_cnt, s_base, s_w, s_k, nullptr,
                                                        [&](int b, uint32_t v) {
            return __hip_atomic_fetch_add(&g.cursor[b], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        });
        for (uint32_t j = threadIdx.x; j < tot; j += kSplitTh) {
            const uint32_t x = s_k[j], b = x >> bins.shift, at = s_base[b] + j;
            const int64_t slot = ((int64_t)b << bins.shift) + at;
            if (at < (1u << bins.shift) && slot < N) {
                g.room[slot] = x;
            } else {
                const uint32_t bit = 1u << (x & 31u);
                if (__hip_atomic_fetch_or(&g.bits[x >> 5].inflight, bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & bit)
                    err = RO_ESTATE;
            }
        }
        __syncthreads();
    }
    if (err) raise_err(ctl, err);
}

// One workgroup per bin: its children's bits in LDS, then into the bitmap.
__global__ __launch_bounds__(kSplitTh) void k_grains_dispatch_bins(int64_t N, GrainTab g, Bins bins, Ctl *ctl)
{
    extern __shared__ uint32_t s_bits[];
    const int64_t c0 = (int64_t)blockIdx.x << bins.shift;
    const int64_t room = min64((int64_t)1 << bins.shift, N - c0);
    const uint32_t mask = (1u << bins.shift) - 1u;
    const int words = 1 << (bins.shift - 5);
    const int64_t cnt = min64((int64_t)g.cursor[blockIdx.x], room);
    for (int w = threadIdx.x; w < words; w += kSplitTh) s_bits[w] = 0;
    __syncthreads();
    if (threadIdx.x == 0) g.cursor[blockIdx.x] = 0;          // for the next call
    bool twice = false;
#pragma unroll 4
    for (int64_t j = threadIdx.x; j < cnt; j += kSplitTh) {
        const uint32_t x = g.room[c0 + j] & mask, bit = 1u << (x & 31u);
        if (atomicOr(&s_bits[x >> 5], bit) & bit) twice = true;
    }
    __syncthreads();
    GrainBits *dst = g.bits + (c0 >> 5);
    for (int w = threadIdx.x; w < words; w += kSplitTh) {
        const uint32_t m = s_bits[w];
        if (m == 0) continue;
        const uint32_t old = dst[w].inflight;
        if (old & m) twice = true;                           // already in flight, or sealed
        dst[w].inflight = old | m;
    }
    if (twice) raise_err(ctl, RO_ESTATE);
}

// A large commit's second pass: the passing reports' children and indices into
// the bins, which lie one after another, sized by the first pass's counts.
constexpr int kPairIt = 8;

__global__ __launch_bounds__(kSplitTh) void k_grains_split(int64_t n, GrainTab g, Bins bins,
                                                           const uint32_t *__restrict__ cidx, uint2 *__restrict__ pair,
                                                           int64_t *counts, Ctl *ctl)
{
    __shared__ uint32_t s_k[kSplitTh * kPairIt], s_i[kSplitTh * kPairIt];
    __shared__ uint32_t s_cnt[kGrainBins + 1], s_base[kGrainBins], s_w[kGrainBins / 64];
    __shared__ uint32_t s_stale;
    const int tid = (int)threadIdx.x;
    const uint32_t start = bins_excl_scan(tid < bins.n ? g.hist[tid] : 0u, s_w);
    if (tid == 0) s_stale = 0;
    uint32_t stale = 0;
    const int64_t span = (int64_t)kSplitTh * kPairIt;
    for (int64_t base = (int64_t)blockIdx.x * span; base < n; base += (int64_t)gridDim.x * span) {
        uint32_t c[kPairIt];
        bool ok[kPairIt];
#pragma unroll
        for (int k = 0; k < kPairIt; ++k) {
            const int64_t i = base + k * kSplitTh + tid;
            c[k] = i < n ? cidx[i] : kNone;
            ok[k] = c[k] < kStale;
            stale += c[k] == kStale;
            if (!ok[k]) c[k] = 0;
        }
        const uint32_t tot = split_tile<kPairIt, true>(c, ok, base, bins, s_cnt, s_base, s_w, s_k, s_i,
                                                       [&](int b, uint32_t v) {
            return start + __hip_atomic_fetch_add(&g.cursor[b], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        });
        for (uint32_t j = tid; j < tot; j += kSplitTh) {
            const uint32_t x = s_k[j];
            pair[s_base[x >> bins.shift] + j] = make_uint2(x, s_i[j]);
        }
        __syncthreads();
    }
    if (stale) atomicAdd(&s_stale, stale);
    __syncthreads();
    if (counts && tid == 0 && s_stale && read_err(ctl) == 0)         // after a bad report nothing is counted
        __hip_atomic_fetch_add(&counts[1], (int64_t)s_stale, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Third pass, one workgroup per bin: the children become sealed; those met
// twice are contested and get neighbouring entries of `room`, and the bin is
// read again to list their reports, each with its child's entry, and to find
// the first of each there.  The list is gathered in LDS: one atomic on its
// length per wave took 980 us for 10M reports.  (120,000 contested of 10M children fill half a
// megabyte; found at the children's own places, 53 and 88 us here and in the
// last pass, now 46 and 84).
__global__ __launch_bounds__(kSplitTh) void k_grains_bins(GrainTab g, Bins bins, const uint2 *__restrict__ pair,
                                                          uint32_t *__restrict__ list, uint32_t *__restrict__ entry,
                                                          int64_t *counts, Ctl *ctl)
{
    extern __shared__ uint32_t s_bits[];
    __shared__ uint32_t s_w[kSplitTh / 64], s_buf[2 * kSplitTh], s_ent[2 * kSplitTh];
    __shared__ uint32_t s_start, s_any, s_n, s_at, s_slot;
    const int tid = (int)threadIdx.x;
    const uint32_t mask = (1u << bins.shift) - 1u;
    const int words = 1 << (bins.shift - 5);
    uint32_t *s_two = s_bits + words;
    const uint32_t cnt = g.hist[blockIdx.x];
    const uint32_t ex = bins_excl_scan(tid < bins.n ? g.hist[tid] : 0u, s_w);
    if (tid == (int)blockIdx.x) s_start = ex;
    if (tid == 0) {
        s_any = s_n = 0;
        g.cursor[blockIdx.x] = 0;                            // for the next call
    }
    for (int w = tid; w < 2 * words; w += kSplitTh) s_bits[w] = 0;
    __syncthreads();
    const uint2 *pp = pair + s_start;
    bool any = false;
    // four lanes that hold different children of one word, as neighbours come, set
    // their bits at once; the loads of four rounds together
    // (1M of 10M children in canonical order, which meet in 31 bins: 32 us, now 12)
    constexpr int kRounds = 4;
    const int quad = lane_id() & ~3;
    for (uint32_t j0 = 0; j0 < cnt; j0 += kRounds * kSplitTh) {
        uint32_t x[kRounds];
#pragma unroll
        for (int q = 0; q < kRounds; ++q) x[q] = pp[min(j0 + q * kSplitTh + tid, cnt - 1)].x & mask;
#pragma unroll
        for (int q = 0; q < kRounds; ++q) {
            const uint32_t bit = j0 + q * kSplitTh + tid < cnt ? 1u << (x[q] & 31u) : 0u;
            const uint32_t w = x[q] >> 5;
            uint32_t all = bit | quad_dpp<0xb1>(bit);
            all |= quad_dpp<0x4e>(all);
            const bool joined = (__ballot(w == quad_dpp<0x00>(w)) >> quad & 15u) == 15u && __popc(all) == 4;
            const uint32_t m = !joined ? bit : lane_id() == quad ? all : 0u;
            if (m) {
                const uint32_t met = atomicOr(&s_bits[w], m) & m;
                if (met) {
                    atomicOr(&s_two[w], met);
                    any = true;
                }
            }
        }
    }
    if (any) s_any = 1;
    __syncthreads();
    GrainBits *dst = g.bits + ((int64_t)blockIdx.x << (bins.shift - 5));
    for (int w = tid; w < words; w += kSplitTh)
        if (s_bits[w]) dst[w].sealed |= s_bits[w];
    uint32_t listed = 0;
    if (s_any) {
        __syncthreads();
        // s_bits[w]: contested children before word w, of the kWords words of a thread
        constexpr int kWords = (1 << (kMaxBinShift - 5)) / kSplitTh;
        uint32_t two[kWords], own = 0;
#pragma unroll
        for (int q = 0; q < kWords; ++q) {
            two[q] = tid * kWords + q < words ? (uint32_t)__popc(s_two[tid * kWords + q]) : 0u;
            own += two[q];
        }
        const uint32_t inc = (uint32_t)wave_incl_sum_dpp(own);
        if (lane_id() == 63) s_w[tid >> 6] = inc;
        __syncthreads();
        uint32_t before = inc - own, all = 0;
#pragma unroll
        for (int v = 0; v < kSplitTh / 64; ++v) {
            before += v < (tid >> 6) ? s_w[v] : 0u;
            all += s_w[v];
        }
        if (tid == 0) s_slot = __hip_atomic_fetch_add(g.n_list + 1, all, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int q = 0; q < kWords; ++q) {
            if (tid * kWords + q < words) s_bits[tid * kWords + q] = before;
            before += two[q];
        }
        __syncthreads();
        uint32_t *room = g.room + s_slot;
        for (uint32_t j = tid; j < all; j += kSplitTh)
            __hip_atomic_store(&room[j], kNone, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // they are set before anyone lowers them
        __syncthreads();
        for (uint32_t j0 = 0; j0 < cnt; j0 += kSplitTh) {
            const uint32_t j = j0 + tid;
            const uint2 e = j < cnt ? pp[j] : make_uint2(0, 0);
            const uint32_t x = e.x & mask, m2 = s_two[x >> 5], bit = 1u << (x & 31u);
            if (j < cnt && (m2 & bit)) {
                const uint32_t r = s_bits[x >> 5] + (uint32_t)__popc(m2 & (bit - 1u)), at = atomicAdd(&s_n, 1u);
                s_buf[at] = e.y;
                s_ent[at] = s_slot + r;
                __hip_atomic_fetch_min(&room[r], e.y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            __syncthreads();
            const uint32_t m = s_n;
            if (m > kSplitTh || j0 + kSplitTh >= cnt) {
                if (m) {
                    if (tid == 0) s_at = __hip_atomic_fetch_add(g.n_list, m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __syncthreads();
                    for (uint32_t k = tid; k < m; k += kSplitTh) {
                        list[s_at + k] = s_buf[k];
                        entry[s_at + k] = s_ent[k];
                    }
                    __syncthreads();
                }
                listed += m;
                if (tid == 0) s_n = 0;
            }
            __syncthreads();
        }
    }
    if (counts && tid == 0 && cnt > listed && read_err(ctl) == 0)
        __hip_atomic_fetch_add(&counts[0], (int64_t)(cnt - listed), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Last pass of a large call: the listed reports are settled.
__global__ __launch_bounds__(kBlock) void k_grains_settle(const uint8_t *__restrict__ rs,
                                                          const int64_t *__restrict__ roff,
                                                          const uint8_t *__restrict__ data, GrainTab g,
                                                          const uint32_t *__restrict__ list,
                                                          const uint32_t *__restrict__ entry,
                                                          uint8_t *__restrict__ state_out, int64_t *counts, Ctl *ctl)
{
    __shared__ int64_t s_wave[kBlock / 64];
    __shared__ CmpJobs s_jobs[kBlock / 64];
    if (blockIdx.x == 0)
        for (int b = threadIdx.x; b < kGrainBins; b += kBlock) g.hist[b] = 0;
    if (read_err(ctl) != 0) return;                  // a bad report: no bytes are compared
    const int64_t nl = *g.n_list;
    const int64_t tid = (int64_t)blockIdx.x * kBlock + threadIdx.x, stride = (int64_t)gridDim.x * kBlock;
    int64_t cnt[3] = {0, 0, 0};                      // accepted, duplicate, conflict
    for (int64_t j0 = tid - lane_id(); j0 < nl; j0 += stride) {
        const bool have = j0 + lane_id() < nl;
        const int64_t i = have ? list[j0 + lane_id()] : 0;
        const int kind = settle_wave(have, i, have ? entry[j0 + lane_id()] : 0u, rs, roff, data, g.room, state_out,
                                     s_jobs[threadIdx.x >> 6]);
        cnt[0] += kind == 0;
        cnt[1] += kind == 1;
        cnt[2] += kind == 2;
    }
    if (counts) {
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const int64_t t = block_sum(cnt[q], s_wave);
            if (threadIdx.x == 0 && t)
                __hip_atomic_fetch_add(&counts[q == 0 ? 0 : q + 1], t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

static int64_t grid_for(const Launch &L, int64_t n, int64_t per_block)
{
    int64_t grid = (n + per_block - 1) / per_block;
    return grid < 1 ? 1 : (grid > (int64_t)L.num_cus * 8 ? (int64_t)L.num_cus * 8 : grid);
}

// Words of each bitmap of n children, a whole number of 256-byte lines.
int64_t grain_words(int64_t n) { return ((n >> 5) + 64) & ~(int64_t)63; }

// Bins for large calls, since a bin's bitmap is swept whole and the launches have
// to be paid for.  The two bitmaps of a bin of 2^17 children take 32 KB of LDS; 512
// of those hold 67M children.
// A reservation takes them from 393,216 children and an eighth of the table on
// (1M of 1M 92 us by atomics, 30 with bins; 390,000 of 1M 25 and 29; 700,000 of
// 10M 37 and 41).  A commit by atomics makes two of them per report, so its line
// lies lower: some 12 us and 90 per million reports against 30, 20 per million
// and a half per million children (390,000 reports on 1M children 45 us and 36,
// 300,000 on 10M 39 and 37, 1M on 40M 113 and 69).
static int64_t reserve_line(int64_t N) { return N / 8 > (int64_t)3 << 17 ? N / 8 : (int64_t)3 << 17; }
static int64_t commit_line(int64_t N) { return ((int64_t)1 << 18) + N / 128; }
static bool use_bins(int64_t n, int64_t N, int64_t line, Bins &bins)
{
    bins.shift = 10;
    while (bins.shift < kMaxBinShift && (N >> bins.shift) >= kGrainBins) ++bins.shift;
    bins.n = (int)((N >> bins.shift) + 1 < kGrainBins ? (N >> bins.shift) + 1 : kGrainBins);
    return n >= line && (N >> bins.shift) < kGrainBins;
}

hipError_t launch_grains_fill(const Launch &L, const GrainTab &g, int64_t n)
{
    // four words of a record, contested; the bins' counts
    const int64_t zero = (grain_words(n) * 5 + 2 * kGrainBins) / 4, first = (n + 3) / 4;
    RO_LAUNCH(L, RO_K_GRAINS, k_grains_fill, dim3((unsigned)grid_for(L, zero > first ? zero : first, kBlock)), dim3(kBlock),
              0, L.stream, reinterpret_cast<uint4 *>(g.bits), zero, reinterpret_cast<uint4 *>(g.first), first);
    return hipGetLastError();
}

hipError_t launch_grains_read(const Launch &L, const GrainTab &g, int64_t n, uint32_t *phase, uint32_t *gen)
{
    RO_LAUNCH(L, RO_K_GRAINS, k_grains_read, dim3((unsigned)grid_for(L, n, kBlock)), dim3(kBlock), 0, L.stream, g, n,
              phase, gen);
    return hipGetLastError();
}

hipError_t launch_grains_dispatch(const Launch &L, const uint32_t *child, int64_t n, int64_t N, const GrainTab &g,
                                  uint32_t *out_gen)
{
    Bins bins;
    if (use_bins(n, N, reserve_line(N), bins)) {
        const int64_t tiles = (n + kSplitTh * kDispIt - 1) / (kSplitTh * kDispIt), most = (int64_t)L.num_cus * 2;
        RO_LAUNCH(L, RO_K_GRAINS, k_grains_dispatch_split, dim3((unsigned)(tiles < most ? tiles : most)), dim3(kSplitTh), 0,
                  L.stream, child, n, N, g, bins, out_gen, L.ctl);
        RO_LAUNCH(L, RO_K_GRAINS, k_grains_dispatch_bins, dim3((unsigned)bins.n), dim3(kSplitTh),
                  (size_t)4 << (bins.shift - 5), L.stream, N, g, bins, L.ctl);
        return hipGetLastError();
    }
    RO_LAUNCH(L, RO_K_GRAINS, k_grains_dispatch, dim3((unsigned)grid_for(L, n, kBlock * kGItems)), dim3(kBlock), 0,
              L.stream, child, n, N, g, out_gen, L.ctl);
    return hipGetLastError();
}

hipError_t launch_grains_retry(const Launch &L, const uint32_t *child, int64_t n, int64_t N, const GrainTab &g)
{
    RO_LAUNCH(L, RO_K_GRAINS, k_grains_retry, dim3((unsigned)grid_for(L, n, kBlock * kGItems)), dim3(kBlock), 0,
              L.stream, child, n, N, g, L.ctl);
    return hipGetLastError();
}

hipError_t launch_grains_commit(const Launch &L, const uint32_t *rp, const uint32_t *ro, const uint8_t *rs,
                                const int64_t *roff, const uint8_t *data, const uint32_t *rgen, int64_t n,
                                const int64_t *offsets, int64_t P, int64_t N, const GrainTab &g, uint32_t *cidx,
                                uint32_t *list, uint2 *pair, uint8_t *state_out, int64_t *counts)
{
    const int64_t grid = grid_for(L, n, kBlock * kGItems);
    Bins bins;
    if (!use_bins(n, N, commit_line(N), bins)) {
        RO_LAUNCH(L, RO_K_FENCE_FIRST, k_grains_first<false>, dim3((unsigned)grid), dim3(kBlock), 0, L.stream, rp, ro, rs,
                  roff, rgen, n, offsets, P, N, g, bins, cidx, state_out, counts, L.ctl);
        RO_LAUNCH(L, RO_K_FENCE_DECIDE, k_grains_decide, dim3((unsigned)grid), dim3(kBlock), 0, L.stream, rs, roff, data, n,
                  g, cidx, state_out, counts, L.ctl);
        return hipGetLastError();
    }
    // fewer workgroups: each adds its counts of all bins
    const int64_t most = (int64_t)L.num_cus * 4, grid_f = grid < most ? grid : most;
    RO_LAUNCH(L, RO_K_FENCE_FIRST, k_grains_first<true>, dim3((unsigned)grid_f), dim3(kBlock), 0, L.stream, rp, ro, rs,
              roff, rgen, n, offsets, P, N, g, bins, cidx, state_out, counts, L.ctl);
    const int64_t tiles = (n + kSplitTh * kPairIt - 1) / (kSplitTh * kPairIt), most_s = (int64_t)L.num_cus * 2;
    RO_LAUNCH(L, RO_K_FENCE_DECIDE, k_grains_split, dim3((unsigned)(tiles < most_s ? tiles : most_s)), dim3(kSplitTh), 0,
              L.stream, n, g, bins, cidx, pair, counts, L.ctl);
    RO_LAUNCH(L, RO_K_FENCE_DECIDE, k_grains_bins, dim3((unsigned)bins.n), dim3(kSplitTh), (size_t)8 << (bins.shift - 5),
              L.stream, g, bins, pair, list, cidx, counts, L.ctl);
    // the list may hold every report; mostly it holds a few
    RO_LAUNCH(L, RO_K_FENCE_DECIDE, k_grains_settle, dim3((unsigned)grid_for(L, n, kBlock)), dim3(kBlock), 0, L.stream, rs,
              roff, data, g, list, cidx, state_out, counts, L.ctl);
    return hipGetLastError();
}

}  // namespace ro
