// F.expand on gfx950: child counts -> Expansion offsets (decoupled look-back
// scan) and per-child lineage keys (load-balanced over children).
//
// RayOrch (arXiv 2609.18703), Sec. 4 "Lineage State and Parent Completion":
// each parent's Expansion is its ordered child set and every child carries
// (parent, immutable zero-based ordinal).
#include "ro_keys.h"

namespace ro {

// Counts int32[P] -> offsets int64[P+1].  One tile = 4096 counts, 16 per
// thread.  Tiles come from the ticket; the exclusive prefix of each tile
// comes from the look-back.
__global__ __launch_bounds__(kBlock) void k_expand_scan(const int32_t *__restrict__ counts, int64_t P,
                                                        int64_t *__restrict__ offsets, int64_t child_cap,
                                                        int want_tags, Ctl *ctl, uint64_t *desc,
                                                        int64_t desc_cap, int64_t ntiles)
{
    const uint32_t epoch = scan_epoch(ctl);
    __shared__ int64_t s_wave[kBlock / 64];
    __shared__ uint64_t s_b;
    __shared__ int64_t s_t;
    __shared__ int32_t s_last;
    for (;;) {
        const int64_t t = next_ticket(ctl, &s_t);
        if (t >= ntiles) break;
        const int64_t i0 = t * kTile + (int64_t)threadIdx.x * kItems;
        int32_t v[kItems];
        int64_t sum = 0;
        bool bad = false;
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            const int64_t i = i0 + k;
            int32_t x = i < P ? counts[i] : 0;
            if (x < 0) { bad = true; x = 0; }
            v[k] = x;
            sum += x;
        }
        if (bad) raise_err(ctl, RO_EINVAL);
        int64_t tot;
        const int64_t ex = block_excl_scan(sum, s_wave, tot);
        const uint64_t pre = tile_prefix(desc, t, epoch, (uint64_t)tot, &s_b, ctl);
        int64_t run = (int64_t)pre + ex;
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            const int64_t i = i0 + k;
            if (i < P) offsets[i] = run;
            run += v[k];
        }
        if (t == ntiles - 1 && threadIdx.x == 0) {
            const int64_t n = (int64_t)pre + tot;
            offsets[P] = n;
            if (pre >= kSat || n >= ((int64_t)1 << 32)) raise_err(ctl, RO_EOVERFLOW);
            else if (want_tags && n > child_cap) raise_err(ctl, RO_ECAP);
        }
        if (ntiles <= (int64_t)gridDim.x) break;     // a tile for every workgroup
    }
    ticket_done(ctl, epoch, desc, desc_cap, &s_last);
}

__global__ __launch_bounds__(kBlock) void k_expand_tags(const int64_t *__restrict__ offsets, int64_t P,
                                                        uint32_t *__restrict__ child_parent,
                                                        uint32_t *__restrict__ child_ordinal,
                                                        int64_t child_cap, int64_t done_up_to, int vec_ok)
{
    write_keys(offsets, P, child_parent, child_ordinal, child_cap, done_up_to, vec_ok);
}

// Offsets and lineage keys of up to 4,096 parents (one scan tile) in one
// launch: every workgroup scans the counts for itself and keeps the offsets in
// LDS for its searches; the first one writes them.  What bounds a small
// expansion is the launches and the chain of searches through memory (1,000
// parents, 7,389 children: 5.7 and 8.9 us as two launches, now 5.9; 2,431
// parents, 1M children: 7.6 and 10.1, now 11.6), so a thread takes four children
// only (16, staged in LDS: 9.6 and 10.7).  LDS holds 32 bits per offset: more
// children than that are an error and get no keys.
//
// The scan in every workgroup and the short spans cost more than they save
// where there are many children: from 1M (4,096 parents, 4M children: 23.5 us,
// 18.0 as two launches) to 8M (100 parents, 6M: 13.8 and 17.6; 41M: 70 and 65.5),
// kSmallKeys / P in between.  The host knows the capacity and not the children:
// where that allows for more, one workgroup per CU scans, writes the offsets and
// the keys of a few children, and k_expand_tags follows, which writes the keys
// of more (4,096 parents, 4M children 16.2 us; 7,000 children of 1,000 parents
// with room for 41M 8.0, as two launches 14.2).
constexpr int64_t kSmallKeys = (int64_t)2 << 30;
static int64_t small_children(int64_t P)
{
    const int64_t n = kSmallKeys / (P > 0 ? P : 1);
    return n < (int64_t)1 << 20 ? (int64_t)1 << 20 : (n > (int64_t)8 << 20 ? (int64_t)8 << 20 : n);
}

__global__ __launch_bounds__(kBlock) void k_expand_small(const int32_t *__restrict__ counts, int64_t P,
                                                         int64_t *__restrict__ offsets,
                                                         uint32_t *__restrict__ child_parent,
                                                         uint32_t *__restrict__ child_ordinal, int64_t child_cap,
                                                         int64_t max_children, int vec_ok, Ctl *ctl)
{
    typedef uint32_t t4 __attribute__((ext_vector_type(4)));
    __shared__ uint32_t s_off[kTile + 1];
    __shared__ int64_t s_wave[kBlock / 64];
    const int64_t i0 = (int64_t)threadIdx.x * kItems;
    int32_t v[kItems];
    int64_t sum = 0;
    bool bad = false;
#pragma unroll
    for (int k = 0; k < kItems; ++k) v[k] = i0 + k < P ? counts[i0 + k] : 0;
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        if (v[k] < 0) { bad = true; v[k] = 0; }
        sum += v[k];
    }
    int64_t N;
    int64_t run = block_excl_scan(sum, s_wave, N);
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        if (i0 + k < P) {
            s_off[i0 + k] = (uint32_t)run;
            if (blockIdx.x == 0) offsets[i0 + k] = run;
        }
        run += v[k];
    }
    if (threadIdx.x == 0) s_off[P] = (uint32_t)N;
    if (blockIdx.x == 0) {
        if (bad) raise_err(ctl, RO_EINVAL);
        if (threadIdx.x == 0) {
            offsets[P] = N;
            if (N >= ((int64_t)1 << 32)) raise_err(ctl, RO_EOVERFLOW);
            else if (N > child_cap) raise_err(ctl, RO_ECAP);
        }
    }
    __syncthreads();
    if (N > child_cap || N > max_children) return;
    for (int64_t c0 = ((int64_t)blockIdx.x * kBlock + threadIdx.x) * 4; c0 < N; c0 += (int64_t)gridDim.x * kBlock * 4) {
        // the last parent starting at or before the thread's first child
        int64_t lo = 0, hi = P;
        while (hi - lo > 1) {
            const int64_t m = (lo + hi) >> 1;
            if (s_off[m] <= (uint32_t)c0) lo = m; else hi = m;
        }
        t4 par, ord;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int64_t c = c0 + k;
            if (c < N && c >= (int64_t)s_off[lo + 1]) lo = advance_parent(s_off, P, lo, c);
            par[k] = (uint32_t)lo;
            ord[k] = (uint32_t)c - s_off[lo];
        }
        if (vec_ok && c0 + 4 <= N) {
            if (child_parent) *reinterpret_cast<t4 *>(child_parent + c0) = par;
            if (child_ordinal) *reinterpret_cast<t4 *>(child_ordinal + c0) = ord;
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (c0 + k >= N) continue;
                if (child_parent) child_parent[c0 + k] = par[k];
                if (child_ordinal) child_ordinal[c0 + k] = ord[k];
            }
        }
    }
}

// done_up_to: expansions of that many children have their keys already.
static hipError_t launch_keys(const Launch &L, const int64_t *offsets, int64_t P, uint32_t *child_parent,
                              uint32_t *child_ordinal, int64_t child_cap, int64_t done_up_to)
{
    const bool aligned = ((reinterpret_cast<uintptr_t>(child_parent) |
                           reinterpret_cast<uintptr_t>(child_ordinal)) & 15u) == 0;
    const int64_t grid = (int64_t)L.num_cus * 8;
    RO_LAUNCH(L, RO_K_EXPAND_TAGS, k_expand_tags, dim3((unsigned)grid), dim3(kBlock), 0, L.stream, offsets, P,
              child_parent, child_ordinal, child_cap, done_up_to, aligned ? 1 : 0);
    return hipGetLastError();
}

hipError_t launch_expand(const Launch &L, const int32_t *counts, int64_t P,
                         int64_t *offsets, uint32_t *child_parent, uint32_t *child_ordinal,
                         int64_t child_cap)
{
    const int64_t ntiles = P > 0 ? (P + kTile - 1) / kTile : 1;
    const int want = (child_parent != nullptr || child_ordinal != nullptr);
    // every workgroup of the one-launch form reads the counts while others
    // write already: an output in the counts' memory takes the two launches,
    // of which the first reads all counts
    const int64_t key_bytes = (child_cap < (int64_t)1 << 32 ? child_cap : (int64_t)1 << 32) * 4;
    const bool apart = !overlap(counts, P * 4, child_parent, key_bytes) && !overlap(counts, P * 4, child_ordinal, key_bytes) &&
                       !overlap(counts, P * 4, offsets, (P + 1) * 8);
    if (want && P <= kTile && apart) {
        const bool aligned = ((reinterpret_cast<uintptr_t>(child_parent) |
                               reinterpret_cast<uintptr_t>(child_ordinal)) & 15u) == 0;
        // a capacity for many: only as many workgroups as there are CUs scan
        const int64_t few = small_children(P), per = kBlock * 4;
        const bool keys = child_cap > few;
        const int64_t most = keys ? (int64_t)L.num_cus : (int64_t)L.num_cus * 8, need = child_cap / per + 1;
        const int64_t here = keys ? most * per : few;
        RO_LAUNCH(L, RO_K_EXPAND_SCAN, k_expand_small, dim3((unsigned)(need < most ? need : most)), dim3(kBlock), 0, L.stream,
                  counts, P, offsets, child_parent, child_ordinal, child_cap, here, aligned ? 1 : 0, L.ctl);
        if (keys) return launch_keys(L, offsets, P, child_parent, child_ordinal, child_cap, here);
        return hipGetLastError();
    }
    const int64_t grid = ntiles < (int64_t)L.num_cus * 4 ? ntiles : (int64_t)L.num_cus * 4;
    RO_LAUNCH(L, RO_K_EXPAND_SCAN, k_expand_scan, dim3((unsigned)grid), dim3(kBlock), 0, L.stream, counts, P,
                       offsets, child_cap, want, L.ctl, L.desc, L.desc_cap, ntiles);
    if (want) return launch_keys(L, offsets, P, child_parent, child_ordinal, child_cap, -1);
    return hipGetLastError();
}

hipError_t launch_expand_tags(const Launch &L, const int64_t *offsets, int64_t P, uint32_t *child_parent,
                              uint32_t *child_ordinal, int64_t child_cap)
{
    return launch_keys(L, offsets, P, child_parent, child_ordinal, child_cap, -1);
}

}  // namespace ro
