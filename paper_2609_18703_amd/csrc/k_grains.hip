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
// A commit call first validates and tests the fence, then finds the children
// with several passing reports, the first of each (in report order), and lists
// their reports; every other report is settled by then, accepted or stale.  Its
// last pass takes the list, 16 lanes to a report: the first is accepted,
// another one's state and bytes are compared with it, 16 bytes a lane and load.
//
// Random returning atomics reach about 26 x 10^9 a second on this chip however
// small the bitmap is (10M reservations: 387 us on 1.25 MB, 441 on records of
// 160 MB; now 108).  So a large call sorts its children into at most 512 bins of
// neighbours first, in LDS tile by tile and with coalesced stores, and one
// workgroup per bin then sets the bits in LDS (use_bins); a smaller one sets
// them by atomics in one pass less.  A commit of 10.2M reports with 1.2% repeats
// in random order takes 350 us (two passes over records: 1,330, of them 820 in
// the second, where a wave compared its lanes' repeats one by one, byte by byte).
#include "ro_copy.h"

namespace ro {

constexpr int kGItems = 4;

// Sets the bits of the wave's children (lanes with valid set) in a bitmap whose
// words lie kStride apart, and returns whether each was set before.  Children
// that follow one another, as in a queue in canonical order, share their words:
// one atomic per word instead of one per child.  Called by all lanes of the wave.
template <int kStride>
__device__ __forceinline__ bool claim_bit(uint32_t *bits, uint32_t c, bool valid)
{
    const int lane = lane_id();
    const uint32_t c0 = (uint32_t)uni32((int32_t)c);
    if (__ballot(valid && c == c0 + (uint32_t)lane) == ~0ull) {
        const int j = (int)(c & 31u);
        const int lead = lane - (j < lane ? j : lane);
        uint32_t old = 0;
        if (lead == lane) {
            const int len = 32 - j < 64 - lane ? 32 - j : 64 - lane;
            old = __hip_atomic_fetch_or(&bits[(int64_t)(c >> 5) * kStride], (0xffffffffu >> (32 - len)) << j,
                                        __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        old = (uint32_t)__shfl((int)old, lead, 64);
        return (old >> j) & 1u;
    }
    if (!valid) return false;
    const uint32_t bit = 1u << (c & 31u);
    const uint32_t old = __hip_atomic_fetch_or(&bits[(int64_t)(c >> 5) * kStride], bit, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
    return (old & bit) != 0;
}

// Every child READY at generation 0: the bitmaps (and the call's, which are
// clear between calls) to zero.
__global__ void k_grains_fill(uint4 *__restrict__ bits, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        bits[i] = make_uint4(0, 0, 0, 0);
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
        for (int k = 0; k < kGItems; ++k) set[k] = claim_bit<4>(&g.bits->inflight, c[k], ok[k]);
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
            if (!ok[k]) continue;
            const uint32_t bit = 1u << (c[k] & 31u);
            if ((f[k].sealed & bit) ||
                !(__hip_atomic_fetch_and(&g.bits[c[k] >> 5].inflight, ~bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & bit)) {
                err = RO_ESTATE;
                continue;
            }
            if (f[k].retried & bit) {
                g.gen[c[k]] += 1u;
            } else {
                g.gen[c[k]] = 1u;
                __hip_atomic_fetch_or(&g.bits[c[k] >> 5].retried, bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
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

// cidx of a report that did not pass the fence, and of one that is not counted
constexpr uint32_t kStale = 0xfffffffeu, kNone = 0xffffffffu;

// Pass 1: validation and the fence.  Per report its provisional outcome in
// state_out (its state if it passed, RO_PENDING if not) and, if it passed, its
// child in cidx.  Two reports of one child meet at its bit of the call's
// bitmap; the later one marks the child contested and clears its entry of
// `first` for the next pass.  With bins only the reports per bin are counted.
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
    if (blockIdx.x == 0 && threadIdx.x == 0) *g.n_list = 0;
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
            if constexpr (kBins) (void)bin_rank(s_hist, c[k] >> bins.shift, ok[k]);
            met[k] = kBins ? false : claim_bit<1>(g.met, c[k], ok[k]);
        }
#pragma unroll
        for (int k = 0; k < kGItems; ++k) {
            const int64_t i = base + k * kBlock + threadIdx.x;
            if (i >= n) continue;
            state_out[i] = ok[k] ? (uint8_t)s[k] : (uint8_t)RO_PENDING;
            if (kBins || ok[k]) cidx[i] = ok[k] ? c[k] : (s[k] == RO_PENDING ? kNone : kStale);
            if (met[k]) {
                __hip_atomic_fetch_or(&g.contested[c[k] >> 5], 1u << (c[k] & 31u), __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_AGENT);
                g.first[c[k]] = 0xffffffffu;
            }
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

// Pass 2: a report that did not pass is stale, one of a child with no other
// report is accepted; those of contested children are listed, and the first of
// them recorded.  The list is gathered in LDS: one atomic on its length per
// wave took 980 us for 10M reports.
constexpr int kListBuf = 2 * kBlock * kGItems;

__device__ __forceinline__ void flush_list(uint32_t *list, uint32_t *n_list, const uint32_t *s_buf, uint32_t n,
                                           uint32_t *s_at)
{
    if (threadIdx.x == 0) *s_at = __hip_atomic_fetch_add(n_list, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    for (uint32_t j = threadIdx.x; j < n; j += blockDim.x) list[*s_at + j] = s_buf[j];
    __syncthreads();
}

__global__ __launch_bounds__(kBlock) void k_grains_decide(const uint8_t *__restrict__ rs, int64_t n, GrainTab g,
                                                          const uint32_t *__restrict__ cidx,
                                                          uint32_t *__restrict__ list,
                                                          const uint8_t *__restrict__ state_out, int64_t *counts,
                                                          Ctl *ctl)
{
    __shared__ int64_t s_wave[kBlock / 64];
    __shared__ uint32_t s_buf[kListBuf];
    __shared__ uint32_t s_n, s_at;
    __shared__ int32_t s_err;
    if (threadIdx.x == 0) {
        s_err = read_err(ctl);                       // the first pass found a bad report
        s_n = 0;
    }
    __syncthreads();
    if (s_err) return;
    int64_t accepted = 0, stale = 0;
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
        for (int k = 0; k < kGItems; ++k) w[k] = so[k] != RO_PENDING ? g.contested[c[k] >> 5] : 0u;
#pragma unroll
        for (int k = 0; k < kGItems; ++k) {
            const int64_t i = base + k * kBlock + threadIdx.x;
            if (so[k] == RO_PENDING) {
                stale += s[k] != RO_PENDING;
            } else if ((w[k] >> (c[k] & 31u)) & 1u) {
                s_buf[atomicAdd(&s_n, 1u)] = (uint32_t)i;
                __hip_atomic_fetch_min(&g.first[c[k]], (uint32_t)i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            } else {
                ++accepted;
            }
        }
        __syncthreads();
        const uint32_t m = s_n;
        if (m > kListBuf / 2) {                      // the next round might not fit
            flush_list(list, g.n_list, s_buf, m, &s_at);
            if (threadIdx.x == 0) s_n = 0;
        }
        __syncthreads();
    }
    if (s_n) flush_list(list, g.n_list, s_buf, s_n, &s_at);
    if (counts) {
        const int64_t a = block_sum(accepted, s_wave), b = block_sum(stale, s_wave);
        if (threadIdx.x == 0 && a) __hip_atomic_fetch_add(&counts[0], a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (threadIdx.x == 0 && b) __hip_atomic_fetch_add(&counts[1], b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
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
// has room for each of its children once (its stretch of `first`, which only a
// commit call uses otherwise); a child beyond that, in a bin where some child
// is named twice, sets its bit here.
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
                g.first[slot] = x;
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
        const uint32_t x = g.first[c0 + j] & mask, bit = 1u << (x & 31u);
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
                                                           int64_t *counts)
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
    if (counts && tid == 0 && s_stale)
        __hip_atomic_fetch_add(&counts[1], (int64_t)s_stale, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Third pass, one workgroup per bin: the children become sealed; those met
// twice are contested, and where there are any the bin is read again to list
// their reports and find the first of each.
__global__ __launch_bounds__(kSplitTh) void k_grains_bins(GrainTab g, Bins bins, const uint2 *__restrict__ pair,
                                                          uint32_t *__restrict__ list, int64_t *counts)
{
    extern __shared__ uint32_t s_bits[];
    __shared__ uint32_t s_w[kGrainBins / 64], s_buf[2 * kSplitTh];
    __shared__ uint32_t s_start, s_any, s_n, s_at;
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
#pragma unroll 4
    for (uint32_t j = tid; j < cnt; j += kSplitTh) {
        const uint32_t x = pp[j].x & mask, bit = 1u << (x & 31u);
        if (atomicOr(&s_bits[x >> 5], bit) & bit) {
            atomicOr(&s_two[x >> 5], bit);
            any = true;
        }
    }
    if (any) s_any = 1;
    __syncthreads();
    const int64_t c0 = (int64_t)blockIdx.x << bins.shift;
    GrainBits *dst = g.bits + (c0 >> 5);
    for (int w = tid; w < words; w += kSplitTh) {
        if (s_bits[w]) dst[w].sealed |= s_bits[w];
        for (uint32_t m = s_two[w]; m; m &= m - 1)
            __hip_atomic_store(&g.first[c0 + w * 32 + (__ffs(m) - 1)], 0xffffffffu, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
    }
    uint32_t listed = 0;
    if (s_any) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // `first` is set before anyone lowers it
        __syncthreads();
        for (uint32_t j0 = 0; j0 < cnt; j0 += kSplitTh) {
            const uint32_t j = j0 + tid;
            const uint2 e = j < cnt ? pp[j] : make_uint2(0, 0);
            const uint32_t x = e.x & mask;
            if (j < cnt && ((s_two[x >> 5] >> (x & 31u)) & 1u)) {
                s_buf[atomicAdd(&s_n, 1u)] = e.y;
                __hip_atomic_fetch_min(&g.first[e.x], e.y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            __syncthreads();
            const uint32_t m = s_n;
            if (m > kSplitTh || j0 + kSplitTh >= cnt) {
                if (m) flush_list(list, g.n_list, s_buf, m, &s_at);
                listed += m;
                if (tid == 0) s_n = 0;
            }
            __syncthreads();
        }
    }
    if (counts && tid == 0 && cnt > listed)
        __hip_atomic_fetch_add(&counts[0], (int64_t)(cnt - listed), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Last pass: in a call without bins its children become sealed and its bitmaps
// are cleared; then the listed reports are settled.  Another one than the
// child's first is a duplicate if state, length and (for SUCCESS) bytes are the
// same, a conflict otherwise.  A wave looks at 64 reports at once, which is a
// chain of four loads, queues the comparisons in LDS, and takes four of them
// at a time with 16 lanes each (taking a report's chain by 16 lanes: 118 us for
// 240,000 listed reports, now 90).  The bytes go 16 to a lane and load, four
// loads of each copy in flight; the last load of a record overlaps the one
// before, so that none reads past its end.
constexpr int kCmpLanes = 16, kCmpSteps = 4;

__global__ __launch_bounds__(kBlock) void k_grains_settle(const uint8_t *__restrict__ rs,
                                                          const int64_t *__restrict__ roff,
                                                          const uint8_t *__restrict__ data, GrainTab g, int64_t words,
                                                          const uint32_t *__restrict__ cidx,
                                                          const uint32_t *__restrict__ list,
                                                          uint8_t *__restrict__ state_out, int64_t *counts, Ctl *ctl)
{
    constexpr int kWaves = kBlock / 64;
    __shared__ int64_t s_wave[kWaves];
    __shared__ int64_t s_a[kWaves][64], s_b[kWaves][64], s_len[kWaves][64];
    __shared__ int32_t s_diff[kWaves][64];
    const int64_t tid = (int64_t)blockIdx.x * kBlock + threadIdx.x, stride = (int64_t)gridDim.x * kBlock;
    for (int64_t w = tid; w < words; w += stride) {
        const uint32_t m = g.met[w];
        if (m == 0) continue;
        g.bits[w].sealed |= m;
        g.met[w] = 0;
        if (g.contested[w]) g.contested[w] = 0;
    }
    if (blockIdx.x == 0)
        for (int b = threadIdx.x; b < kGrainBins; b += kBlock) g.hist[b] = 0;
    if (read_err(ctl) != 0) return;                  // a bad report: no bytes are compared
    const int64_t nl = *g.n_list;
    const int wv = (int)(threadIdx.x >> 6), lane = lane_id(), sub = lane & (kCmpLanes - 1);
    int64_t cnt[3] = {0, 0, 0};                      // accepted, duplicate, conflict
    for (int64_t j0 = tid - lane; j0 < nl; j0 += stride) {
        int kind = -1;
        int64_t i = 0, a = 0, b = 0, len = 0;
        bool job = false;
        if (j0 + lane < nl) {
            i = list[j0 + lane];
            const uint32_t s = rs[i];
            b = roff[i];
            len = roff[i + 1] - b;
            const int64_t v = g.first[cidx[i]];
            kind = 0;
            if (v != i) {
                a = roff[v];
                const bool same = rs[v] == s && (s != RO_SUCCESS || roff[v + 1] - a == len);
                job = same && s == RO_SUCCESS && data != nullptr && len > 0;
                kind = same ? 1 : 2;
                state_out[i] = RO_PENDING;
            }
        }
        const uint64_t jobs = __ballot(job);
        const int slot = (int)__popcll(jobs & ((1ull << lane) - 1ull)), nj = (int)__popcll(jobs);
        if (job) {
            s_a[wv][slot] = a;
            s_b[wv][slot] = b;
            s_len[wv][slot] = len;
        }
        __builtin_amdgcn_wave_barrier();
        for (int q = lane / kCmpLanes; q < nj; q += 64 / kCmpLanes) {
            const uint8_t *pa = data + s_a[wv][q], *pb = data + s_b[wv][q];
            const int64_t l = s_len[wv][q];
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
            if (sub == 0) s_diff[wv][q] = (dm & ((1u << kCmpLanes) - 1u)) != 0;
        }
        __builtin_amdgcn_wave_barrier();
        if (job && s_diff[wv][slot]) kind = 2;
        __builtin_amdgcn_wave_barrier();
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

// Bins for calls that name a good part of many children: at least an eighth of
// the table (a bin's bitmap is swept whole), and enough to pay for the launches
// (reset, reservation and commit of 289,000 children take 125 us by atomics and
// about 120 with bins, 825,000 206 and 129).  The two bitmaps
// of a bin of 2^17 children take 32 KB of LDS; 512 of those hold 67M children.
constexpr int64_t kBinCall = (int64_t)3 << 17;
constexpr int kMaxBinShift = 17;
static bool use_bins(int64_t n, int64_t N, Bins &bins)
{
    bins.shift = 10;
    while (bins.shift < kMaxBinShift && (N >> bins.shift) >= kGrainBins) ++bins.shift;
    bins.n = (int)((N >> bins.shift) + 1 < kGrainBins ? (N >> bins.shift) + 1 : kGrainBins);
    return n >= kBinCall && n >= N / 8 && (N >> bins.shift) < kGrainBins;
}

hipError_t launch_grains_fill(const Launch &L, const GrainTab &g, int64_t n)
{
    // four words of a record, met, contested; the bins' counts
    const int64_t quads = (grain_words(n) * 6 + 2 * kGrainBins) / 4;
    RO_LAUNCH(L, RO_K_GRAINS, k_grains_fill, dim3((unsigned)grid_for(L, quads, kBlock)), dim3(kBlock), 0, L.stream,
              reinterpret_cast<uint4 *>(g.bits), quads);
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
    if (use_bins(n, N, bins)) {
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
    const int64_t grid = grid_for(L, n, kBlock * kGItems), words = grain_words(N);
    Bins bins;
    if (use_bins(n, N, bins)) {
        // fewer workgroups: each adds its counts of all bins
        const int64_t most = (int64_t)L.num_cus * 4, grid_f = grid < most ? grid : most;
        RO_LAUNCH(L, RO_K_FENCE_FIRST, k_grains_first<true>, dim3((unsigned)grid_f), dim3(kBlock), 0, L.stream, rp, ro, rs,
                  roff, rgen, n, offsets, P, N, g, bins, cidx, state_out, counts, L.ctl);
        const int64_t tiles = (n + kSplitTh * kPairIt - 1) / (kSplitTh * kPairIt), most_s = (int64_t)L.num_cus * 2;
        RO_LAUNCH(L, RO_K_FENCE_DECIDE, k_grains_split, dim3((unsigned)(tiles < most_s ? tiles : most_s)), dim3(kSplitTh),
                  0, L.stream, n, g, bins, cidx, pair, counts);
        RO_LAUNCH(L, RO_K_FENCE_DECIDE, k_grains_bins, dim3((unsigned)bins.n), dim3(kSplitTh),
                  (size_t)8 << (bins.shift - 5), L.stream, g, bins, pair, list, counts);
    } else {
        RO_LAUNCH(L, RO_K_FENCE_FIRST, k_grains_first<false>, dim3((unsigned)grid), dim3(kBlock), 0, L.stream, rp, ro, rs,
                  roff, rgen, n, offsets, P, N, g, bins, cidx, state_out, counts, L.ctl);
        RO_LAUNCH(L, RO_K_FENCE_DECIDE, k_grains_decide, dim3((unsigned)grid), dim3(kBlock), 0, L.stream, rs, n, g, cidx,
                  list, state_out, counts, L.ctl);
    }
    // the list may hold every report; mostly it holds a few
    const int64_t items = n > words ? n : words;
    RO_LAUNCH(L, RO_K_FENCE_DECIDE, k_grains_settle, dim3((unsigned)grid_for(L, items, kBlock)), dim3(kBlock), 0,
              L.stream, rs, roff, data, g, words, cidx, list, state_out, counts, L.ctl);
    return hipGetLastError();
}

}  // namespace ro
