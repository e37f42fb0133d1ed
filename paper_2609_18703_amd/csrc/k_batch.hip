// Per-Call FIFO Ready Queue with elastic reservation on gfx950.
//
// RayOrch (arXiv 2609.18703), Sec. 4 "Scheduling Ready Grains": ready Grains
// sit in one FIFO queue in enqueue order; each elastic reservation removes at
// most B entries from the head and may mix parents.  Taking the reservations
// one after another until the queue is empty is a stable compaction of the
// ready entries cut into consecutive chunks of B, which is what these kernels
// compute.  A barred parent's entries (Sec. 4 "Commit, Failure, and Recovery":
// queued siblings of a group failure are suppressed before dispatch) are simply
// not ready.  Where an entry's slot comes from:
//   no mask, no barrier   the entry's own place (k_batch_all);
//   a mask                the count of set mask bytes before it, which short
//                         queues count in every tile, long ones in a launch of
//                         their own (k_batch_count, k_batch_fill) and those in
//                         between by ticket and look-back (k_batch_keep);
//   a barrier             look-back over the tiles' ready entries, after their
//                         parents are looked up (k_batch).
// Where its parent comes from: an offsets search, in LDS or memory, or one of
// two maps built for the call, or a stream's own map.
#include "ro_device.h"

namespace ro {

// Coarse child -> parent map, one 8-byte entry per block of 2^s children:
// for block j, x = the parent p0 of child j 2^s, with bit 31 set when the
// whole block lies in p0, and y = the ordinal of child j 2^s in p0.  A child
// of a one-parent block has its tags from its entry alone; any other child's
// parent lies between p0 and the next entry's parent, and the search for it
// starts from offsets[p0] = j 2^s - y without reading it.  Built for fewer
// than 2^31 parents (the flag bit); otherwise the offsets are searched whole.
// The block size follows the mean fan-out N / P (map_shift): blocks of 16
// children for small parents keep the searches short, blocks of 128 for
// large ones keep the map small enough to stay in cache (workload 2, mean
// 411: 128; the documents' levels, means 9 and 15: 16).
constexpr uint32_t kMapOne = 0x80000000u;

// Tag outputs of a queue too long for the caches are written with
// non-temporal stores: they are read once, by a later call, and kept out of
// L2 they leave the coarse map and offsets there for this kernel's lookups
// (workload 2's 41M-entry ready-queue batch 0.46 -> 0.42 ms, and the gather's
// report scatter that reads them 1.55 -> 1.53 ms).  A shorter queue's tags
// are stored normally: they then still sit in cache when the gather reads
// them (the documents' 2.7M-entry batch).
constexpr int64_t kTagNtEntries = (int64_t)8 << 20;   // 32 MB per tag array, the size of all L2s
__device__ __forceinline__ void st_tag_nt(uint32_t *p, uint32_t v) { __builtin_nontemporal_store(v, p); }

// The tile's staged outputs s_out[0, lim) to dst[base, base + lim): two
// loops, since one store with a chosen hint is folded into a plain store.
__device__ __forceinline__ void write_tags(uint32_t *__restrict__ dst, int64_t base, const uint32_t *s_out,
                                           int64_t lim, bool nt)
{
    if (nt) {
        for (int64_t j = threadIdx.x; j < lim; j += kBlock) st_tag_nt(dst + base + j, s_out[j]);
    } else {
        for (int64_t j = threadIdx.x; j < lim; j += kBlock) dst[base + j] = s_out[j];
    }
}

// log2 of the children per map block: the smallest power of two from 16 to
// 128 that is at least the mean number of children per parent.
__device__ __forceinline__ int map_shift(int64_t N, int64_t P)
{
    int s = 4;
    while (s < 7 && ((int64_t)1 << s) * P < N) ++s;
    return s;
}

// Mask map, one 16-byte entry per block of 64 children: x = the parent p0 of
// the block's first child, y = that child's ordinal, z and w = a mask with bit
// j set (j > 0) when child j of the block is the first of its parent.  A
// child's parent is p0 plus the number of mask bits up to it, its ordinal the
// distance from the last of them (or from the block's start, plus y): one
// load per lookup and no search.  Where an empty parent lies between two
// children of the block the count would miss it: bit 31 of x then says that
// children behind a mask bit search the offsets.  At N / 4 bytes it is larger
// than the coarse map for large parents, so it is used while it stays in
// every XCD's L2 (4 MB) beside the queue, or while parents are small enough
// for the coarse map to be no smaller (use_mask_map).
constexpr int kMaskShift = 6;

// The host knows the queue, the parents and the children reserved (the map has
// room for those), not the children themselves.  Measured, whole batch: 2.7M
// children under 300,000 parents 23 us with this map, 48 with the coarse one;
// 5M under 30,000 46 and 78; 8M under 20,000 91 and 107; 20M under 2.7M 238
// and 955; but 41M under 100,000 540 (a 10 MB map) against 448.  A short queue
// over a large reservation keeps the coarse map, whose build writes less.  So
// does an expansion that is mostly empty parents, which would make most
// entries search after all: more parents than children reserved, or many
// beside both the queue (a queue rarely names a child twice) and the
// reservation (100,000 children of 1M parents, 90,000 entries with a barrier:
// 28 us, 62 with this map; 1M of 4M parents 36 and 59; but 4M under 1M parents,
// 200,000 entries, 28 and 25).
constexpr int64_t kMaskChildren = (int64_t)12 << 20;
static bool use_mask_map(int64_t Q, int64_t P, int64_t reserved)
{
    if (reserved > kMaskChildren && reserved > 4 * Q) return false;
    if (P > reserved || (P > 2 * Q && 4 * P > reserved)) return false;
    return Q <= kMaskChildren || Q < 64 * P;
}

// which structure a batch kernel finds an entry's parent in
enum BatchMap { kMapSearch = 0, kMapCoarse = 1, kMapMask = 2, kMapChild = 3, kMapLds = 4 };
struct MapArgs {
    const void *map;         // coarse or mask map, or the child -> parent map
    int64_t cap;             // its entries
};

// Offsets of few parents, searched in LDS: every workgroup loads them for
// itself (P entries of 8 bytes), and a step of a search costs an LDS read
// instead of a trip to the cache.  Held in 32 bits: a child id is smaller than
// any offset that does not fit.
constexpr int kLdsParents = 4096;

template <int kMap>
__device__ __forceinline__ void load_lds_offsets(const int64_t *__restrict__ offsets, int64_t P, uint32_t *s_off,
                                                 MapArgs &map)
{
    if constexpr (kMap == kMapLds) {
        for (int p = (int)threadIdx.x; p < (int)P; p += kBlock) {
            const int64_t o = offsets[p];
            s_off[p] = o > 0xffffffffll ? 0xffffffffu : (uint32_t)(o < 0 ? 0 : o);
        }
        map.map = s_off;
        __syncthreads();
    }
}

// entries of a thread whose lookups are in flight together
#ifndef RO_BATCH_LOOKUPS
#define RO_BATCH_LOOKUPS 4
#endif

// First index i in [0, n) with a[i] > x (n if none), for K keys at once
// (n >= 1, a nondecreasing).  The halving is branch-free and its trip count
// depends on n only, so the K searches step together and each step's K loads
// are in flight at the same time.
template <int K>
__device__ __forceinline__ void upper_bound_k(const int64_t *a, int64_t n, const int64_t (&x)[K], int64_t (&r)[K])
{
    int64_t base[K];
#pragma unroll
    for (int k = 0; k < K; ++k) base[k] = 0;
    int64_t len = n;
    while (len > 1) {
        const int64_t half = len >> 1;
        int64_t v[K];
#pragma unroll
        for (int k = 0; k < K; ++k) v[k] = a[base[k] + half];
#pragma unroll
        for (int k = 0; k < K; ++k) base[k] = v[k] <= x[k] ? base[k] + half : base[k];
        len -= half;
    }
#pragma unroll
    for (int k = 0; k < K; ++k) r[k] = base[k] + (a[base[k]] <= x[k] ? 1 : 0);
}

// A wave builds 16 entries (1,024 children): the first parent starting among
// them by a wave search, then 64 parents' starts per step, each of which sets
// its bit in LDS; the parent of a block's first child is the one starting
// there, or the last one starting before.  1,024 children of parents that are
// not empty take 17 steps at most.  A run of empty parents is stepped over by a
// search (ten million of them were 156,000 dependent steps of one wave, 53 ms),
// and where empty parents still make it more than kMaskSteps every child's
// parent is searched, four blocks of children at a time: the logarithm of the
// parents left, however they lie.
constexpr int kMaskSteps = 20, kMaskSearch = 4;

__global__ __launch_bounds__(kBlock) void k_batch_mask_map(const int64_t *__restrict__ offsets, int64_t P,
                                                           uint4 *__restrict__ map, int64_t map_cap)
{
    constexpr int kB = 16, kSpan = kB << kMaskShift;
    __shared__ uint64_t s_mask[kBlock / 64][kB];
    __shared__ uint32_t s_last[kBlock / 64][kB];      // last parent starting in the block, plus 1
    __shared__ uint32_t s_at0[kBlock / 64][kB];       // parent starting at the block's first child, plus 1
    __shared__ uint32_t s_empty[kBlock / 64][kB];
    const int64_t N = offsets[P];
    int64_t nmap = (N + (1 << kMaskShift) - 1) >> kMaskShift;
    nmap = nmap < map_cap ? nmap : map_cap;
    const int w = (int)(threadIdx.x >> 6), lane = lane_id();
    const int64_t nwaves = (int64_t)gridDim.x * (kBlock / 64);
    for (int64_t wt = (int64_t)blockIdx.x * (kBlock / 64) + w; wt * kB < nmap; wt += nwaves) {
        const int64_t cb = wt * kSpan, ce = min64(cb + kSpan, N);
        if (lane < kB) {
            s_mask[w][lane] = 0;
            s_last[w][lane] = s_at0[w][lane] = s_empty[w][lane] = 0;
        }
        __builtin_amdgcn_wave_barrier();
        const int64_t q0 = cb == 0 ? 0 : wave_last_le(offsets, 0, P + 1, cb - 1) + 1;
        int steps = 0;
        bool was_idle = false;
        for (int64_t qb = q0; steps < kMaskSteps; qb += 64, ++steps) {
            const int64_t q = qb + lane;
            const int64_t st = q < P ? offsets[q] : N, en = q < P ? offsets[q + 1] : N;
            const bool here = st >= cb && st < ce, starts = here && en > st;
            if (here) {
                const int b = (int)((st - cb) >> kMaskShift), j = (int)(st & ((1 << kMaskShift) - 1));
                if (starts) {
                    if (j > 0) atomicOr((unsigned long long *)&s_mask[w][b], 1ull << j);
                    else s_at0[w][b] = (uint32_t)q + 1;
                    atomicMax(&s_last[w][b], (uint32_t)q + 1);
                } else if (j > 0) {
                    s_empty[w][b] = 1;
                }
            }
            if (__ballot(st >= ce) != 0) break;
            // 64 empty parents lie at one child; after 64 more, on to the last
            // parent there (a search as long as about six steps)
            const bool idle = __ballot(starts) == 0;
            if (idle && was_idle) {
                qb = wave_last_le(offsets, qb, P + 1, __shfl(st, 0)) - 64;
                steps += 6;
            }
            was_idle = idle;
        }
        __builtin_amdgcn_wave_barrier();
        if (steps < kMaskSteps) {
            const int64_t b = wt * kB + lane;
            if (lane < kB) {
                uint32_t before = (uint32_t)q0;           // the last parent starting before the block, plus 1
                for (int k = 0; k < lane; ++k) before = s_last[w][k] > before ? s_last[w][k] : before;
                before = s_at0[w][lane] ? s_at0[w][lane] : before;
                const uint32_t p0 = before ? before - 1 : 0u;
                const uint64_t m = s_mask[w][lane];
                if (b < nmap)
                    map[b] = make_uint4(p0 | (s_empty[w][lane] ? kMapOne : 0u),
                                        (uint32_t)((b << kMaskShift) - offsets[p0]), (uint32_t)m, (uint32_t)(m >> 32));
            }
        } else {
            // parents [lo, lo + len) hold the span's children
            const int64_t lo = q0 > 0 ? q0 - 1 : 0;
            const int64_t len = min64(wave_last_le(offsets, lo, P + 1, ce - 1) + 1, P) - lo;
#pragma unroll 1
            for (int k0 = 0; k0 < kB; k0 += kMaskSearch) {
                int64_t c[kMaskSearch], r[kMaskSearch];
#pragma unroll
                for (int k = 0; k < kMaskSearch; ++k) c[k] = min64(cb + (k0 + k) * 64 + lane, ce - 1);
                upper_bound_k<kMaskSearch>(offsets + lo, len > 0 ? len : 1, c, r);
#pragma unroll
                for (int k = 0; k < kMaskSearch; ++k) {
                    const int64_t b = wt * kB + k0 + k, p = lo + max64(r[k] - 1, 0);
                    const int64_t before = __shfl_up(p, 1);
                    const uint64_t m = __ballot(lane > 0 && p != before), e = __ballot(lane > 0 && p > before + 1);
                    if (lane == 0 && b < nmap)
                        map[b] = make_uint4((uint32_t)p | (e ? kMapOne : 0u), (uint32_t)(c[k] - offsets[p]), (uint32_t)m,
                                            (uint32_t)(m >> 32));
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
}

__global__ void k_batch_cmap(const int64_t *__restrict__ offsets, int64_t P, uint2 *__restrict__ map,
                             int64_t map_cap)
{
    const int64_t N = offsets[P];
    const int sh = map_shift(N, P);
    int64_t nmap = (N + (1 << sh) - 1) >> sh;
    nmap = nmap < map_cap ? nmap : map_cap;
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < nmap;
         j += (int64_t)gridDim.x * blockDim.x) {
        const int64_t c0 = j << sh;
        const int64_t p0 = max64(upper_bound_g(offsets, 0, P + 1, c0) - 1, 0);
        const int64_t last = c0 + (1 << sh) - 1 < N ? c0 + (1 << sh) - 1 : N - 1;
        const bool one = offsets[p0 + 1] > last;
        map[j] = make_uint2((uint32_t)p0 | (one ? kMapOne : 0u), (uint32_t)(c0 - offsets[p0]));
    }
}

// Parent and ordinal of K children at once (bit k of `live`: entry k is a
// child id below N; the others are left alone).  Every step's loads are in
// flight together: the map entries of all K, then the rounds of a lockstep
// binary search for the children of blocks that hold several parents (or
// that lie past the map).  Needs P < 2^31 and a map entry.
template <int K>
__device__ __forceinline__ void tags_of(const uint2 *__restrict__ map, int64_t nmap, int sh,
                                        const int64_t *__restrict__ offsets, int64_t P, const uint32_t (&c)[K],
                                        uint32_t live, uint32_t (&par)[K], uint32_t (&ord)[K])
{
    uint32_t l[K], h[K];
    int64_t vl[K];
    {
        // a child past the map (the map is sized by the workspace, the
        // expansion may be larger) searches all parents, from offsets[0]
        const int64_t off0 = offsets[0];
        uint2 e[K];
        uint32_t hx[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int64_t j = (int64_t)(c[k] >> sh);
            const int64_t jj = (((live >> k) & 1u) && j < nmap) ? j : 0;
            e[k] = map[jj];
            hx[k] = map[jj + 1 < nmap ? jj + 1 : jj].x;
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int64_t j = (int64_t)(c[k] >> sh);
            const uint32_t p0 = e[k].x & ~kMapOne;
            const uint32_t hi = j + 1 < nmap ? (hx[k] & ~kMapOne) : (uint32_t)(P - 1);
            if (((live >> k) & 1u) == 0) {
                l[k] = 0;
                h[k] = 1;
                vl[k] = 0;
            } else if (j >= nmap) {
                l[k] = 0;
                h[k] = (uint32_t)P;
                vl[k] = off0;
            } else {
                l[k] = p0;
                vl[k] = (j << sh) - (int64_t)e[k].y;
                h[k] = (e[k].x & kMapOne) ? p0 + 1 : hi + 1;
            }
        }
    }
    // the parent is the largest p in [l, h) with offsets[p] <= c
    for (;;) {
        bool any = false;
#pragma unroll
        for (int k = 0; k < K; ++k) any |= h[k] - l[k] > 1;
        if (!any) break;
        uint32_t mid[K];
        int64_t v[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            mid[k] = h[k] - l[k] > 1 ? (l[k] + h[k]) >> 1 : l[k];
            v[k] = offsets[mid[k]];
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (h[k] - l[k] > 1) {
                if (v[k] <= (int64_t)c[k]) {
                    l[k] = mid[k];
                    vl[k] = v[k];
                } else {
                    h[k] = mid[k];
                }
            }
        }
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        if (!((live >> k) & 1u)) continue;
        par[k] = l[k];
        ord[k] = (uint32_t)((int64_t)c[k] - vl[k]);
    }
}

// The last parent among [lo, hi) that starts at or before child c (lo - 1 if
// none does), out of line: its registers would cost the common path a wave per
// SIMD.
__device__ __noinline__ int64_t search_parent(const int64_t *offsets, int64_t lo, int64_t hi, int64_t c)
{
    return upper_bound_g(offsets, lo, hi, c) - 1;
}

// The same as tags_of with the mask map.
template <int K>
__device__ __forceinline__ void tags_of_mask(const uint4 *__restrict__ map, int64_t nmap,
                                             const int64_t *__restrict__ offsets, int64_t P, const uint32_t (&c)[K],
                                             uint32_t live, uint32_t (&par)[K], uint32_t (&ord)[K])
{
    uint4 e[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int64_t j = (int64_t)(c[k] >> kMaskShift);
        e[k] = map[((live >> k) & 1u) && j < nmap ? j : 0];
    }
    uint32_t slow = 0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int j = (int)(c[k] & ((1u << kMaskShift) - 1));
        const uint64_t m = ((uint64_t)e[k].w << 32 | e[k].z) & ((2ull << j) - 1);
        const uint32_t n = (uint32_t)__popcll(m);
        // offsets that are no expansion may hold more starts than parents follow
        // p0; the barrier is read at the result, so it stays below P
        const uint32_t p = (e[k].x & ~kMapOne) + n;
        par[k] = p < (uint32_t)P ? p : (uint32_t)P - 1u;
        ord[k] = n ? (uint32_t)(j - (63 - __clzll((long long)m))) : e[k].y + (uint32_t)j;
        if (((live >> k) & 1u) && ((n && (e[k].x & kMapOne)) || (int64_t)(c[k] >> kMaskShift) >= nmap)) slow |= 1u << k;
    }
    if (slow) {
        // the parent lies between the count and the next block's first parent;
        // a child past the map may have any
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (!((slow >> k) & 1u)) continue;
            const int64_t j = (int64_t)(c[k] >> kMaskShift);
            const int64_t lo = j < nmap ? (int64_t)par[k] : 0;
            const int64_t hi = j + 1 < nmap ? min64((int64_t)(map[j + 1].x & ~kMapOne) + 1, P) : P;
            const int64_t p = max64(search_parent(offsets, lo, hi, (int64_t)c[k]), 0);
            par[k] = (uint32_t)p;
            ord[k] = (uint32_t)((int64_t)c[k] - offsets[p]);
        }
    }
}

// Tags of K entries by whichever structure the launch chose.
template <int kMap, int K>
__device__ __forceinline__ void entry_tags(const MapArgs &m, int64_t nmap, int sh, const int64_t *__restrict__ offsets,
                                           int64_t P, const uint32_t (&c)[K], uint32_t live, uint32_t (&par)[K],
                                           uint32_t (&ord)[K])
{
    if constexpr (kMap == kMapMask) {
        tags_of_mask<K>(static_cast<const uint4 *>(m.map), nmap, offsets, P, c, live, par, ord);
    } else if constexpr (kMap == kMapChild) {
        const uint32_t *cpar = static_cast<const uint32_t *>(m.map);
        uint32_t p[K];
#pragma unroll
        for (int k = 0; k < K; ++k) p[k] = cpar[((live >> k) & 1u) ? c[k] : 0u];
        int64_t st[K];
#pragma unroll
        for (int k = 0; k < K; ++k) st[k] = offsets[p[k]];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            par[k] = p[k];
            ord[k] = (uint32_t)((int64_t)c[k] - st[k]);
        }
    } else if constexpr (kMap == kMapLds) {
        const uint32_t *so = static_cast<const uint32_t *>(m.map);
        uint32_t lo[K];
#pragma unroll
        for (int k = 0; k < K; ++k) lo[k] = 0;
        // the last parent starting at or before the child, K searches in step
        for (uint32_t len = (uint32_t)P; len > 1;) {
            const uint32_t half = len >> 1;
            uint32_t v[K];
#pragma unroll
            for (int k = 0; k < K; ++k) v[k] = so[lo[k] + half];
#pragma unroll
            for (int k = 0; k < K; ++k) lo[k] += v[k] <= c[k] ? half : 0u;
            len -= half;
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (!((live >> k) & 1u)) continue;
            par[k] = lo[k];
            ord[k] = c[k] - so[lo[k]];
        }
    } else if constexpr (kMap == kMapCoarse) {
        tags_of<K>(static_cast<const uint2 *>(m.map), nmap, sh, offsets, P, c, live, par, ord);
    } else {
        int64_t key[K], pp[K];
#pragma unroll
        for (int k = 0; k < K; ++k) key[k] = ((live >> k) & 1u) ? (int64_t)c[k] : 0;
        if (live == 0) return;
        upper_bound_k<K>(offsets, P + 1, key, pp);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (!((live >> k) & 1u)) continue;
            const int64_t p = max64(pp[k] - 1, 0);          // -1 only where the offsets do not start at 0
            par[k] = (uint32_t)p;
            ord[k] = (uint32_t)((int64_t)c[k] - offsets[p]);
        }
    }
}

// Entries of the map in use: the whole expansion's or as many as it has room for.
template <int kMap>
__device__ __forceinline__ int64_t map_entries(const MapArgs &m, int64_t N, int sh)
{
    if constexpr (kMap == kMapSearch || kMap == kMapChild || kMap == kMapLds) return 0;
    const int s = kMap == kMapMask ? kMaskShift : sh;
    const int64_t n = (N + ((int64_t)1 << s) - 1) >> s;
    return n < m.cap ? n : m.cap;
}

// A thread's kIt consecutive entries of the queue from i0 on, and the ready
// flags of its mask.
template <int kIt>
__device__ __forceinline__ void load_queue(const uint32_t *__restrict__ queue, int64_t i0, int64_t Q, int vec_ok,
                                           uint32_t (&q)[kIt])
{
    if (vec_ok && i0 + kIt <= Q) {
        const uint4 *qp = reinterpret_cast<const uint4 *>(queue + i0);
#pragma unroll
        for (int k = 0; k < kIt / 4; ++k) {
            const uint4 x = qp[k];
            q[4 * k] = x.x; q[4 * k + 1] = x.y; q[4 * k + 2] = x.z; q[4 * k + 3] = x.w;
        }
    } else {
#pragma unroll
        for (int k = 0; k < kIt; ++k) q[k] = i0 + k < Q ? queue[i0 + k] : 0u;
    }
}

template <int kIt>
__device__ __forceinline__ uint32_t load_mask(const uint8_t *__restrict__ keep, int64_t i0, int64_t Q, int vec_ok)
{
    uint32_t m = 0;
    if (vec_ok && i0 + kIt <= Q) {
        uint32_t w[kIt / 4];
#pragma unroll
        for (int k = 0; k < kIt / 4; ++k) w[k] = reinterpret_cast<const uint32_t *>(keep + i0)[k];
#pragma unroll
        for (int k = 0; k < kIt; ++k) m |= (((w[k >> 2] >> (8 * (k & 3))) & 0xffu) != 0 ? 1u : 0u) << k;
    } else {
#pragma unroll
        for (int k = 0; k < kIt; ++k)
            if (i0 + k < Q && keep[i0 + k] != 0) m |= 1u << k;
    }
    return m;
}

// Tags of a thread's kIt entries, RO_BATCH_LOOKUPS at a time with all their
// lookups in flight; entries that are not live keep 0xffffffff.
template <int kMap, int kIt>
__device__ __forceinline__ void thread_tags(const MapArgs &map, int64_t nmap, int sh, const int64_t *__restrict__ offsets,
                                            int64_t P, const uint32_t (&q)[kIt], uint32_t live, uint32_t (&par)[kIt],
                                            uint32_t (&ord)[kIt])
{
    constexpr int H = RO_BATCH_LOOKUPS;
#pragma unroll
    for (int hf = 0; hf < kIt / H; ++hf) {
        uint32_t cc[H], pp[H], oo[H];
#pragma unroll
        for (int k = 0; k < H; ++k) cc[k] = q[hf * H + k];
        entry_tags<kMap, H>(map, nmap, sh, offsets, P, cc, (live >> (hf * H)) & ((1u << H) - 1u), pp, oo);
#pragma unroll
        for (int k = 0; k < H; ++k) {
            if ((live >> (hf * H + k)) & 1u) {
                par[hf * H + k] = pp[k];
                ord[hf * H + k] = oo[k];
            }
        }
    }
}

// A tile's ready entries to its slot range: each requested array staged in
// LDS in slot order, then written with coalesced stores.
template <int kIt>
__device__ __forceinline__ void write_slots(uint32_t *out_child, uint32_t *out_parent, uint32_t *out_ordinal,
                                            const uint32_t (&q)[kIt], const uint32_t (&par)[kIt],
                                            const uint32_t (&ord)[kIt], uint32_t kmask, int ex, int64_t base,
                                            int64_t lim, uint32_t *s_out, bool nt)
{
#pragma unroll 1
    for (int which = 0; which < 3; ++which) {
        uint32_t *dst = which == 0 ? out_child : (which == 1 ? out_parent : out_ordinal);
        if (dst == nullptr) continue;
        int slot = ex;
#pragma unroll
        for (int k = 0; k < kIt; ++k) {
            if (kmask & (1u << k)) {
                s_out[slot] = which == 0 ? q[k] : (which == 1 ? par[k] : ord[k]);
                ++slot;
            }
        }
        __syncthreads();
        write_tags(dst, base, s_out, lim, nt);
        __syncthreads();
    }
}

__device__ __forceinline__ int64_t slot_room(int64_t out_cap, int64_t base, int64_t cnt)
{
    return out_cap - base < cnt ? (out_cap - base > 0 ? out_cap - base : 0) : cnt;
}

// The ready queue with a barrier (and perhaps a mask): kIt entries per thread
// and tile; a barred parent's entry is not ready, so the tags come before the
// look-back.  A queue of one tile needs neither ticket nor look-back.
template <int kMap, int kIt>
__global__ __launch_bounds__(kBlock) void k_batch(
    const uint32_t *__restrict__ queue, const uint8_t *__restrict__ keep, int64_t Q,
    const int64_t *__restrict__ offsets, int64_t P, MapArgs map, int64_t max_id, int32_t B,
    uint32_t *__restrict__ out_child, uint32_t *__restrict__ out_parent, uint32_t *__restrict__ out_ordinal,
    int64_t out_cap, int64_t *n_out, int64_t *n_batches, const uint8_t *__restrict__ barrier, Ctl *ctl,
    uint64_t *desc, int64_t desc_cap, int64_t ntiles, int vec_ok)
{
    constexpr int kT = kBlock * kIt;
    __shared__ uint32_t s_off[kMap == kMapLds ? kLdsParents : 1];
    load_lds_offsets<kMap>(offsets, P, s_off, map);
    const uint32_t epoch = scan_epoch(ctl);
    __shared__ uint32_t s_out[kT];             // one output array of a tile, in slot order
    __shared__ int64_t s_wave[kBlock / 64];
    __shared__ uint64_t s_b;
    __shared__ int64_t s_t;
    __shared__ int32_t s_last;
    const int64_t NP = offsets[P];
    const int64_t N = min64(NP, max_id);       // ids past a child map are out of range
    const int sh = map_shift(NP, P);
    const int64_t nmap = map_entries<kMap>(map, NP, sh);
    const bool want_tags = out_parent != nullptr || out_ordinal != nullptr;
    const bool nt = Q > kTagNtEntries;
    const bool single = ntiles == 1;
    for (;;) {
        const int64_t t = single ? 0 : next_ticket(ctl, &s_t);
        if (t >= ntiles) break;
        const int64_t i0 = t * kT + (int64_t)threadIdx.x * kIt;
        uint32_t q[kIt], par[kIt], ord[kIt];
        load_queue<kIt>(queue, i0, Q, vec_ok, q);
        uint32_t kmask;
        if (keep) kmask = load_mask<kIt>(keep, i0, Q, vec_ok);
        else kmask = i0 + kIt <= Q ? (uint32_t)((1ull << kIt) - 1) : (i0 < Q ? (1u << (Q - i0)) - 1u : 0u);
        bool bad_range = false;
        uint32_t live = 0;
#pragma unroll
        for (int k = 0; k < kIt; ++k) {
            par[k] = 0xffffffffu;
            ord[k] = 0xffffffffu;
            if (kmask & (1u << k)) {
                if ((int64_t)q[k] >= N) bad_range = true;
                else live |= 1u << k;
            }
        }
        // the tags are set before the barrier test, never inside it
        if (want_tags || barrier) thread_tags<kMap, kIt>(map, nmap, sh, offsets, P, q, live, par, ord);
        if (barrier) {
#pragma unroll
            for (int k = 0; k < kIt; ++k) {
                if (((live >> k) & 1u) && barrier[par[k]]) {
                    kmask &= ~(1u << k);                             // suppressed: takes no slot
                    par[k] = 0xffffffffu;
                    ord[k] = 0xffffffffu;
                }
            }
        }
        if (bad_range) raise_err(ctl, RO_ERANGE);
        int64_t tot;
        const int64_t ex = block_excl_scan(__popc(kmask), s_wave, tot);
        const int64_t base = single ? 0 : (int64_t)tile_prefix(desc, t, epoch, (uint64_t)tot, &s_b, ctl);
        if (base + tot > out_cap && threadIdx.x == 0) raise_err(ctl, RO_ECAP);
        write_slots<kIt>(out_child, out_parent, out_ordinal, q, par, ord, kmask, (int)ex, base,
                         slot_room(out_cap, base, tot), s_out, nt);
        if (t == ntiles - 1 && threadIdx.x == 0) {
            const int64_t m = base + tot;
            if (n_out) *n_out = m;
            if (n_batches) *n_batches = (m + B - 1) / B;
        }
        if (single) return;
        if (ntiles <= (int64_t)gridDim.x) break;       // a tile for every workgroup
    }
    ticket_done(ctl, epoch, desc, desc_cap, &s_last);
}

// The ready queue of kDirectQueue to kMidQueue entries with a dispatch mask and
// no barrier: an entry is ready iff its mask byte is set, so a tile's count of
// ready entries is known from the mask alone, before any lineage lookup.  A
// workgroup counts its tile, posts the count and finishes the look-back first;
// only then does it look up the tags of the ready entries and write them, staged
// in LDS, to the tile's contiguous slot range.
template <int kMap, int kIt>
__global__ __launch_bounds__(kBlock) void k_batch_keep(
    const uint32_t *__restrict__ queue, const uint8_t *__restrict__ keep, int64_t Q,
    const int64_t *__restrict__ offsets, int64_t P, MapArgs map, int32_t B,
    uint32_t *__restrict__ out_child, uint32_t *__restrict__ out_parent, uint32_t *__restrict__ out_ordinal,
    int64_t out_cap, int64_t *n_out, int64_t *n_batches, Ctl *ctl, uint64_t *desc, int64_t desc_cap,
    int64_t ntiles, int vec_ok)
{
    constexpr int kT = kBlock * kIt;
    __shared__ uint32_t s_off[kMap == kMapLds ? kLdsParents : 1];
    load_lds_offsets<kMap>(offsets, P, s_off, map);
    const uint32_t epoch = scan_epoch(ctl);
    __shared__ uint32_t s_out[kT];
    __shared__ int64_t s_wave[kBlock / 64];
    __shared__ uint64_t s_b;
    __shared__ int64_t s_t;
    __shared__ int32_t s_last;
    const int64_t N = offsets[P];
    const int sh = map_shift(N, P);
    const int64_t nmap = map_entries<kMap>(map, N, sh);
    const bool want_tags = out_parent != nullptr || out_ordinal != nullptr;
    for (;;) {
        const int64_t t = next_ticket(ctl, &s_t);
        if (t >= ntiles) break;
        const int64_t i0 = t * kT + (int64_t)threadIdx.x * kIt;
        const uint32_t km = load_mask<kIt>(keep, i0, Q, vec_ok);
        int64_t tot;
        const int64_t ex = block_excl_scan(__popc(km), s_wave, tot);
        const int64_t base = (int64_t)tile_prefix(desc, t, epoch, (uint64_t)tot, &s_b, ctl);
        if (base + tot > out_cap && threadIdx.x == 0) raise_err(ctl, RO_ECAP);
        uint32_t q[kIt], par[kIt], ord[kIt];
        load_queue<kIt>(queue, i0, Q, vec_ok, q);
        bool bad_range = false;
        uint32_t live = 0;
#pragma unroll
        for (int k = 0; k < kIt; ++k) {
            par[k] = 0xffffffffu;
            ord[k] = 0xffffffffu;
            if (km & (1u << k)) {
                if ((int64_t)q[k] >= N) bad_range = true;
                else live |= 1u << k;
            }
        }
        if (want_tags) thread_tags<kMap, kIt>(map, nmap, sh, offsets, P, q, live, par, ord);
        write_slots<kIt>(out_child, out_parent, out_ordinal, q, par, ord, km, (int)ex, base,
                         slot_room(out_cap, base, tot), s_out, false);
        if (bad_range) raise_err(ctl, RO_ERANGE);
        if (t == ntiles - 1 && threadIdx.x == 0) {
            const int64_t m = base + tot;
            if (n_out) *n_out = m;
            if (n_batches) *n_batches = (m + B - 1) / B;
        }
        if (ntiles <= (int64_t)gridDim.x) break;       // a tile for every workgroup
    }
    ticket_done(ctl, epoch, desc, desc_cap, &s_last);
}

// A long queue with a dispatch mask: counted first, then filled with no order
// between the workgroups.  Tickets and look-back hand on about one tile per
// 100 ns however many wait, so a queue of 10M entries took 81 us in 610 tiles
// (two or three workgroups per CU) and 154 in 2,441; reading the mask twice
// costs less.  k_batch_count: a wave counts the ready entries of a tile of
// 4,096, a workgroup 16 tiles, and writes each tile's place in its group and
// the group's total; k_batch_fill: a tile per workgroup adds up the totals of
// the groups before its own.  In a short queue (up to kDirectQueue entries) it
// counts the mask before its tile itself, at most 64 KB: no ticket, no look-back
// and no count at the end (7,389 entries: 10.4 us, now 7.6).
// The counts use the look-back descriptors' room (epoch field 0, which no
// look-back takes for its own).
constexpr int kFillIt = 16, kFillTile = kBlock * kFillIt, kCountGrp = 16;

__device__ __forceinline__ uint32_t nonzero_bytes(uint32_t x)
{
    return (uint32_t)__popc((x | ((x & 0x7f7f7f7fu) + 0x7f7f7f7fu)) & 0x80808080u);
}

__global__ __launch_bounds__(64 * kCountGrp) void k_batch_count(const uint8_t *__restrict__ keep, int64_t Q,
                                                                uint64_t *__restrict__ tile_at,
                                                                uint64_t *__restrict__ group_n, int vec_ok)
{
    __shared__ uint32_t s_c[kCountGrp];
    const int wv = uni32((int)(threadIdx.x >> 6)), ln = lane_id();
    const int64_t t = (int64_t)blockIdx.x * kCountGrp + wv, i0 = t * kFillTile;
    uint32_t c = 0;
    if (vec_ok && i0 + kFillTile <= Q) {
        const uint4 *k4 = reinterpret_cast<const uint4 *>(keep + i0);
        uint4 x[kFillTile / 1024];
#pragma unroll
        for (int k = 0; k < kFillTile / 1024; ++k) x[k] = k4[k * 64 + ln];
#pragma unroll
        for (int k = 0; k < kFillTile / 1024; ++k)
            c += nonzero_bytes(x[k].x) + nonzero_bytes(x[k].y) + nonzero_bytes(x[k].z) + nonzero_bytes(x[k].w);
    } else {
        for (int k = ln; k < kFillTile; k += 64) c += i0 + k < Q && keep[i0 + k] != 0;
    }
    c = wave_sum(c);
    if (ln == 0) s_c[wv] = c;
    __syncthreads();
    if (threadIdx.x < kCountGrp) {
        uint32_t at = 0, all = 0;
#pragma unroll
        for (int k = 0; k < kCountGrp; ++k) {
            at += k < (int)threadIdx.x ? s_c[k] : 0u;
            all += s_c[k];
        }
        if (((int64_t)blockIdx.x * kCountGrp + threadIdx.x) * kFillTile < Q)
            tile_at[(int64_t)blockIdx.x * kCountGrp + threadIdx.x] = at;
        if (threadIdx.x == 0) group_n[blockIdx.x] = all;
    }
}

// In a long queue every tile would add up many groups (3 x 10^9 entries: 12.7 ms,
// of them more than half for that, and 6.9 with look-back): past kGroupScan of
// them one workgroup replaces the groups' totals by what lies before each.
constexpr int64_t kGroupScan = 2048;

__global__ __launch_bounds__(64 * kCountGrp) void k_batch_groups(uint64_t *__restrict__ group_n, int64_t n)
{
    __shared__ uint64_t s_w[kCountGrp];
    const int wv = (int)(threadIdx.x >> 6);
    uint64_t sum = 0;
    for (int64_t g0 = 0; g0 < n; g0 += 64 * kCountGrp) {
        const int64_t g = g0 + threadIdx.x;
        const uint64_t v = g < n ? group_n[g] : 0, inc = wave_incl_sum_dpp(v);
        if (lane_id() == 63) s_w[wv] = inc;
        __syncthreads();
        uint64_t at = sum + inc - v;
#pragma unroll
        for (int k = 0; k < kCountGrp; ++k) {
            at += k < wv ? s_w[k] : 0;
            sum += s_w[k];
        }
        if (g < n) group_n[g] = at;
        __syncthreads();
    }
}

// kWalk: the grid is smaller than the tiles, and a workgroup strides over them.
template <int kMap, int kIt, bool kCounted, bool kWalk = false>
__global__ __launch_bounds__(kBlock) void k_batch_fill(
    const uint32_t *__restrict__ queue, const uint8_t *__restrict__ keep, int64_t Q,
    const int64_t *__restrict__ offsets, int64_t P, MapArgs map, int32_t B, uint32_t *__restrict__ out_child,
    uint32_t *__restrict__ out_parent, uint32_t *__restrict__ out_ordinal, int64_t out_cap, int64_t *n_out,
    int64_t *n_batches, const uint64_t *__restrict__ tile_at, const uint64_t *__restrict__ group_n, int scanned,
    Ctl *ctl, int vec_ok)
{
    constexpr int kT = kBlock * kIt;
    __shared__ uint32_t s_off[kMap == kMapLds ? kLdsParents : 1];
    load_lds_offsets<kMap>(offsets, P, s_off, map);
    __shared__ uint32_t s_out[kT];
    __shared__ int64_t s_wave[kBlock / 64];
    const int64_t N = offsets[P];
    const int sh = map_shift(N, P);
    const int64_t nmap = map_entries<kMap>(map, N, sh);
    const bool want_tags = out_parent != nullptr || out_ordinal != nullptr;
    const bool nt = Q > kTagNtEntries;
    const int64_t ntiles = kWalk ? (Q + kT - 1) / kT : (int64_t)gridDim.x;
    int64_t t = blockIdx.x;
    do {
        const int64_t i0 = t * kT + (int64_t)threadIdx.x * kIt;
        const uint32_t km = load_mask<kIt>(keep, i0, Q, vec_ok);
        uint32_t q[kIt], par[kIt], ord[kIt];
        load_queue<kIt>(queue, i0, Q, vec_ok, q);
        int64_t before = 0;
        if constexpr (kCounted) {
            if (threadIdx.x == 0) before = (int64_t)tile_at[t];
            // the totals of the groups before, or what lies before this one
            const int64_t at = t / kCountGrp;
            for (int64_t g = scanned * at + threadIdx.x; g < at + scanned; g += kBlock) before += (int64_t)group_n[g];
        } else if (vec_ok) {
            const uint4 *k4 = reinterpret_cast<const uint4 *>(keep);
#pragma unroll 4
            for (int64_t j = threadIdx.x; j < t * kT / 16; j += kBlock) {
                const uint4 x = k4[j];
                before += nonzero_bytes(x.x) + nonzero_bytes(x.y) + nonzero_bytes(x.z) + nonzero_bytes(x.w);
            }
        } else {
            for (int64_t j = threadIdx.x; j < t * kT; j += kBlock) before += keep[j] != 0;
        }
        bool bad_range = false;
        uint32_t live = 0;
#pragma unroll
        for (int k = 0; k < kIt; ++k) {
            par[k] = 0xffffffffu;
            ord[k] = 0xffffffffu;
            if (km & (1u << k)) {
                if ((int64_t)q[k] >= N) bad_range = true;
                else live |= 1u << k;
            }
        }
        if (want_tags) thread_tags<kMap, kIt>(map, nmap, sh, offsets, P, q, live, par, ord);
        if (bad_range) raise_err(ctl, RO_ERANGE);
        const int64_t base = block_sum(before, s_wave);
        int64_t tot;
        const int64_t ex = block_excl_scan(__popc(km), s_wave, tot);
        if (base + tot > out_cap && threadIdx.x == 0) raise_err(ctl, RO_ECAP);
        write_slots<kIt>(out_child, out_parent, out_ordinal, q, par, ord, km, (int)ex, base,
                             slot_room(out_cap, base, tot), s_out, nt);
        if (t == ntiles - 1 && threadIdx.x == 0) {
            if (n_out) *n_out = base + tot;
            if (n_batches) *n_batches = (base + tot + B - 1) / B;
        }
        t += gridDim.x;
    } while (kWalk && t < ntiles);
}

// Every queue entry is ready (no mask): the FIFO compaction is the identity,
// slot i holds queue[i], so no scan is needed and each entry is independent.
// A block takes 1024 consecutive entries, lane-contiguous, so every load and
// store instruction of a wave covers 256 contiguous bytes.
constexpr int kAllPer = 4;

template <int kMap>
__global__ __launch_bounds__(kBlock) void k_batch_all(
    const uint32_t *__restrict__ queue, int64_t Q, const int64_t *__restrict__ offsets, int64_t P, MapArgs map,
    int64_t max_id, int32_t B, uint32_t *__restrict__ out_child, uint32_t *__restrict__ out_parent,
    uint32_t *__restrict__ out_ordinal, int64_t out_cap, int64_t *n_out, int64_t *n_batches, Ctl *ctl)
{
    __shared__ uint32_t s_off[kMap == kMapLds ? kLdsParents : 1];
    load_lds_offsets<kMap>(offsets, P, s_off, map);
    const int64_t NP = offsets[P];
    const int64_t N = min64(NP, max_id);       // ids past a child map are out of range
    const int sh = map_shift(NP, P);
    const int64_t nmap = map_entries<kMap>(map, NP, sh);
    const bool want_tags = out_parent != nullptr || out_ordinal != nullptr;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (Q > out_cap) raise_err(ctl, RO_ECAP);
        if (n_out) *n_out = Q;
        if (n_batches) *n_batches = (Q + B - 1) / B;
    }
    const int64_t lim = Q < out_cap ? Q : out_cap;
    bool bad_range = false;
    for (int64_t i0 = (int64_t)blockIdx.x * (kBlock * kAllPer); i0 < Q;
         i0 += (int64_t)gridDim.x * (kBlock * kAllPer)) {
        uint32_t q[kAllPer];
        uint32_t live = 0;
#pragma unroll
        for (int k = 0; k < kAllPer; ++k) {
            const int64_t i = i0 + k * kBlock + threadIdx.x;
            q[k] = i < Q ? queue[i] : 0u;
            if (i < Q) {
                if ((int64_t)q[k] < N) live |= 1u << k;
                else bad_range = true;
            }
        }
        uint32_t par[kAllPer], ord[kAllPer];
        if (want_tags) {
            entry_tags<kMap, kAllPer>(map, nmap, sh, offsets, P, q, live, par, ord);
        }
#pragma unroll
        for (int k = 0; k < kAllPer; ++k) {
            const int64_t i = i0 + k * kBlock + threadIdx.x;
            if (i >= lim || !((live >> k) & 1u)) continue;
            if (out_child) out_child[i] = q[k];
            if (out_parent) out_parent[i] = par[k];
            if (out_ordinal) out_ordinal[i] = ord[k];
        }
    }
    if (bad_range) raise_err(ctl, RO_ERANGE);
}

// Sizes at which a queue changes path (entries):
//   up to kDirectQueue the offsets are searched, more than kLdsParents of them
//   through memory: a map is a launch and a search per block of the whole
//   expansion (65,536 masked entries under 5,000 parents 10.2 us and one more,
//   with the map, 13.8; under 1M 16.8 and 30.8; under 10M 24.7 and 97); a masked
//   queue's tiles of 1,024 count the mask before them themselves (7,389 entries:
//   7.6 us, 10.4 with tickets and look-back, 39 as one tile of 16,384);
//   up to kSmallQueue a masked queue is cut into tiles of 1,024 entries (98,000
//   entries: 18 us, 57 as 6 tiles of 16,384);
//   up to kMidQueue into tiles of 4,096 (1M entries: 29 us; 57 in 980 tiles of
//   1,024, whose tickets and look-backs queue up; 66 in 61 of 16,384, too few
//   for 256 CUs); with a barrier this is the largest tile, since the tags come
//   before the count;
//   beyond, a masked queue is counted first and needs no order between its
//   tiles (4M entries: 28 us in all, 40 with four tiles of 4,096 per ticket; 10M:
//   73 and 81; 41M: 380 and 431).
constexpr int64_t kDirectQueue = 65536, kSmallQueue = 262144, kMidQueue = 1 << 20;

// Workgroups of a counted queue's fill with the coarse map.  A lookup reads two
// of its entries and searches the offsets between, at random; where those
// outgrow the L2s, fewer lookups in flight are faster (10M entries under 10M
// parents: 663 us with all tiles at once, 626 with three workgroups per CU, 598
// with two, 506 with one; 4M under 3M parents 220, 220, 210, 207; 4M under 1M
// 152, 150, 148, 156; under 530,000 107, and 109 with two).
static int64_t fill_grid(const Launch &L, int64_t P)
{
    return P >= (int64_t)2 << 20 ? L.num_cus : (P >= (int64_t)3 << 18 ? 2 * (int64_t)L.num_cus : (int64_t)1 << 31);
}

template <int kMap>
hipError_t launch_batch_with(const Launch &L, const uint32_t *queue, const uint8_t *keep, int64_t Q,
                             const int64_t *offsets, int64_t P, MapArgs map, int64_t max_id, int32_t B,
                             uint32_t *out_child, uint32_t *out_parent, uint32_t *out_ordinal, int64_t out_cap,
                             int64_t *n_out, int64_t *n_batches, const uint8_t *barrier)
{
    const int64_t cap_grid = (int64_t)L.num_cus * 4;
    if (keep == nullptr && barrier == nullptr) {
        int64_t grid = (Q + kBlock * kAllPer - 1) / (kBlock * kAllPer);
        grid = grid < 1 ? 1 : (grid > (int64_t)L.num_cus * 8 ? (int64_t)L.num_cus * 8 : grid);
        RO_LAUNCH(L, RO_K_BATCH, k_batch_all<kMap>, dim3((unsigned)grid), dim3(kBlock), 0, L.stream, queue, Q, offsets, P,
                  map, max_id, B, out_child, out_parent, out_ordinal, out_cap, n_out, n_batches, L.ctl);
        return hipGetLastError();
    }
    const bool aligned = ((reinterpret_cast<uintptr_t>(queue) | reinterpret_cast<uintptr_t>(keep)) & 15u) == 0;
    auto tiles = [&](int64_t per) { return Q > 0 ? (Q + per - 1) / per : 1; };
    // offsets in LDS come with short queues only, a map with longer ones
    constexpr bool kShort = kMap == kMapLds || kMap == kMapSearch, kLong = kMap != kMapLds;
    const bool small = !kLong || Q <= kSmallQueue;
    const int64_t ntiles = tiles(small ? kBlock * 4 : kBlock * 16), grid_t = ntiles < cap_grid ? ntiles : cap_grid;
    if constexpr (kMap != kMapChild) {
        if (barrier == nullptr) {
            if constexpr (kLong) {
                if (Q > kMidQueue) {
                    const int64_t nt = tiles(kFillTile), ng = (nt + kCountGrp - 1) / kCountGrp;
                    if (nt + ng > L.desc_cap || nt > 0x7fffffff) return hipErrorInvalidValue;
                    RO_LAUNCH(L, RO_K_BATCH, k_batch_count, dim3((unsigned)ng), dim3(64 * kCountGrp), 0, L.stream, keep, Q,
                              L.desc, L.desc + nt, aligned ? 1 : 0);
                    if (ng > kGroupScan)
                        RO_LAUNCH(L, RO_K_BATCH, k_batch_groups, dim3(1), dim3(64 * kCountGrp), 0, L.stream, L.desc + nt, ng);
                    auto kern = k_batch_fill<kMap, kFillIt, true>;
                    int64_t grid = nt;
                    if constexpr (kMap == kMapCoarse) {
                        if (fill_grid(L, P) < nt) {
                            kern = k_batch_fill<kMap, kFillIt, true, true>;
                            grid = fill_grid(L, P);
                        }
                    }
                    RO_LAUNCH(L, RO_K_BATCH, kern, dim3((unsigned)grid), dim3(kBlock), 0, L.stream, queue, keep, Q, offsets, P,
                              map, B, out_child, out_parent, out_ordinal, out_cap, n_out, n_batches, L.desc, L.desc + nt,
                              ng > kGroupScan ? 1 : 0, L.ctl, aligned ? 1 : 0);
                    return hipGetLastError();
                }
            }
            if constexpr (kShort) {
                if (Q <= kDirectQueue) {
                    RO_LAUNCH(L, RO_K_BATCH, (k_batch_fill<kMap, 4, false>), dim3((unsigned)tiles(kBlock * 4)), dim3(kBlock),
                              0, L.stream, queue, keep, Q, offsets, P, map, B, out_child, out_parent, out_ordinal, out_cap,
                              n_out, n_batches, nullptr, nullptr, 0, L.ctl, aligned ? 1 : 0);
                    return hipGetLastError();
                }
            }
            auto kern = k_batch_keep<kMap, 4>;
            if constexpr (kLong) {
                if (!small) kern = k_batch_keep<kMap, 16>;
            }
            RO_LAUNCH(L, RO_K_BATCH, kern, dim3((unsigned)grid_t), dim3(kBlock), 0, L.stream, queue, keep, Q, offsets, P,
                      map, B, out_child, out_parent, out_ordinal, out_cap, n_out, n_batches, L.ctl, L.desc, L.desc_cap,
                      ntiles, aligned ? 1 : 0);
            return hipGetLastError();
        }
    }
    auto kern = k_batch<kMap, 4>;
    if constexpr (kLong) {
        if (!small) kern = k_batch<kMap, 16>;
    }
    RO_LAUNCH(L, RO_K_BATCH, kern, dim3((unsigned)grid_t), dim3(kBlock), 0, L.stream, queue, keep, Q, offsets, P, map,
              max_id, B, out_child, out_parent, out_ordinal, out_cap, n_out, n_batches, barrier, L.ctl, L.desc,
              L.desc_cap, ntiles, aligned ? 1 : 0);
    return hipGetLastError();
}

hipError_t launch_batch(const Launch &L, const uint32_t *queue, const uint8_t *keep,
                        int64_t Q, const int64_t *offsets, int64_t P, int32_t B,
                        uint32_t *out_child, uint32_t *out_parent, uint32_t *out_ordinal,
                        int64_t out_cap, int64_t *n_out, int64_t *n_batches, uint32_t *cmap_words,
                        int64_t cmap_words_cap, const uint8_t *barrier, const uint32_t *cpar, int64_t cpar_n)
{
    constexpr int64_t kAnyId = (int64_t)1 << 40;
    if (cpar)
        return launch_batch_with<kMapChild>(L, queue, keep, Q, offsets, P, MapArgs{cpar, cpar_n}, cpar_n, B, out_child,
                                            out_parent, out_ordinal, out_cap, n_out, n_batches, barrier);
    const bool tags = out_parent != nullptr || out_ordinal != nullptr;
    // Few parents and a short queue: the offsets in LDS.  7,389 entries under
    // 1,000 parents take 7.6 us (10.4 with a search through memory); at 1M
    // entries under 2,431 parents the batch takes 24 us, as long as with the mask
    // map and its launch, so the line lies at kSmallQueue.
    if ((tags || barrier != nullptr) && P <= kLdsParents && Q <= kSmallQueue)
        return launch_batch_with<kMapLds>(L, queue, keep, Q, offsets, P, MapArgs{nullptr, 0}, kAnyId, B, out_child,
                                          out_parent, out_ordinal, out_cap, n_out, n_batches, barrier);
    // A map costs a launch and a search per block; a short unmasked queue
    // (fewer entries than parents, such as one wave of a stream) searches
    // the offsets directly instead.  The maps' parent fields keep a flag bit.
    const bool use_map = (tags || barrier != nullptr) && cmap_words_cap >= 4 && P < ((int64_t)1 << 31) &&
                         !(keep == nullptr && barrier == nullptr && Q < P) && Q > kDirectQueue;
    if (!use_map)
        return launch_batch_with<kMapSearch>(L, queue, keep, Q, offsets, P, MapArgs{nullptr, 0}, kAnyId, B, out_child,
                                             out_parent, out_ordinal, out_cap, n_out, n_batches, barrier);
    const int64_t grid_m = (int64_t)L.num_cus * 4;
    if (use_mask_map(Q, P, cmap_words_cap * 8)) {
        uint4 *map = reinterpret_cast<uint4 *>(cmap_words);
        const int64_t cap = cmap_words_cap / 4;
        RO_LAUNCH(L, RO_K_BATCH_SAMPLES, k_batch_mask_map, dim3((unsigned)grid_m), dim3(kBlock), 0, L.stream, offsets, P,
                  map, cap);
        return launch_batch_with<kMapMask>(L, queue, keep, Q, offsets, P, MapArgs{map, cap}, kAnyId, B, out_child,
                                           out_parent, out_ordinal, out_cap, n_out, n_batches, barrier);
    }
    uint2 *map = reinterpret_cast<uint2 *>(cmap_words);
    const int64_t cap = cmap_words_cap / 2;
    RO_LAUNCH(L, RO_K_BATCH_SAMPLES, k_batch_cmap, dim3((unsigned)grid_m), dim3(256), 0, L.stream, offsets, P, map, cap);
    return launch_batch_with<kMapCoarse>(L, queue, keep, Q, offsets, P, MapArgs{map, cap}, kAnyId, B, out_child,
                                         out_parent, out_ordinal, out_cap, n_out, n_batches, barrier);
}

}  // namespace ro
