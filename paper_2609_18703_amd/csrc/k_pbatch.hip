// Parent-bound reservation on gfx950.
//
// RayOrch (arXiv 2609.18703), Sec. 4 "Scheduling Ready Grains": a
// parent-bound reservation takes up to B siblings of the first ready parent,
// and the entries it leaves keep their order.  Run to the end of the queue,
// the reservations have a closed form that needs no sequential loop: rank
// every ready entry within its parent in queue order; the entries of ranks
// jB .. jB + B - 1 of one parent leave together (the head is always the
// earliest entry left, and it always opens such a group, since the group
// before it in its parent left whole), and the groups leave in the queue
// order of their first entries.
//
// On the GPU: the ready entries are compacted in queue order (the FIFO
// batch's compaction), sorted by parent with a stable LSD radix sort that
// carries each entry's child and queue position (so each parent's entries
// stay in queue order and an entry's rank is its distance from its parent's
// first sorted entry), every group's first entry marks its queue position
// with the group size, one scan over queue positions numbers the groups and
// gives their slot offsets, and every entry is written to its group's slot
// range.
#include "ro_device.h"

namespace ro {

constexpr int kRTh = 512;                    // threads of the scatter
constexpr int kRTile = (int)kPbTile;         // sort tile: 8 entries per thread
constexpr int kRMaxBits = 9;                 // digit width; at most 512 buckets
constexpr int kRMaxBuckets = 1 << kRMaxBits;
constexpr int kRSpan = (int)kPbSpan;          // tiles per histogram column
constexpr int64_t kRSpanLen = (int64_t)kRTile * kRSpan;
static_assert(kRMaxBuckets == kPbMaxBuckets, "histogram layout");

__device__ __forceinline__ int64_t tiles_of(int64_t m) { return (m + kRTile - 1) / kRTile; }

// Digit histograms per span of kRSpan tiles, digit-major:
// hist[d * spans_cap + st].  Spans past the ready count write zeros, so the
// scan over all spans_cap columns is the scan over the real ones.
__global__ __launch_bounds__(kBlock) void k_rs_hist(const uint32_t *__restrict__ keys, const int64_t *m_dev,
                                                   int shift, int width, int32_t *__restrict__ hist,
                                                   int64_t spans_cap)
{
    __shared__ int32_t s_h[kRMaxBuckets];
    const int64_t M = *m_dev;
    const int nb = 1 << width;
    const uint32_t mask = (uint32_t)nb - 1;
    for (int64_t st = blockIdx.x; st < spans_cap; st += gridDim.x) {
        for (int d = threadIdx.x; d < nb; d += kBlock) s_h[d] = 0;
        __syncthreads();
        const int64_t i0 = st * kRSpanLen;
        const int64_t i1 = min64(i0 + kRSpanLen, M);
        // four keys a thread at a time (a span starts 16-byte aligned)
        for (int64_t i = i0 + 4 * (int64_t)threadIdx.x; i < i1; i += 4 * kBlock) {
            if (i + 4 <= i1) {
                const uint4 k4 = *reinterpret_cast<const uint4 *>(keys + i);
                atomicAdd(&s_h[(k4.x >> shift) & mask], 1);
                atomicAdd(&s_h[(k4.y >> shift) & mask], 1);
                atomicAdd(&s_h[(k4.z >> shift) & mask], 1);
                atomicAdd(&s_h[(k4.w >> shift) & mask], 1);
            } else {
                for (int64_t j = i; j < i1; ++j) atomicAdd(&s_h[(keys[j] >> shift) & mask], 1);
            }
        }
        __syncthreads();
        for (int d = threadIdx.x; d < nb; d += kBlock) hist[(int64_t)d * spans_cap + st] = s_h[d];
        __syncthreads();
    }
}

// Stable scatter of one digit pass.  A workgroup takes a span of kRSpan
// tiles in order, starting each digit at the span's offset from the
// histogram scan.  Per tile each wave ranks its own eighth (eight rounds of 64
// entries, in order) among the eighth's entries of the same digit, with a
// wave-private running count per digit plus the lanes below with the same
// digit (one ballot per digit bit); the waves' counts give the tile's counts
// and every wave's base per digit, the tile is put in order of digits in LDS
// (values, then keys, in the same room) and written out so that consecutive
// lanes store consecutive places of a digit's run; the span's digit offsets
// then move past the tile.  Values are (child << 32 | queue position); vin ==
// nullptr: built from the compacted children and the positions.
// The runs of a digit decide the speed: 4,096 entries over 256 digits write 16
// at a time (two passes over 10M entries, 15-bit keys: 260 us with tiles of
// 2,048, digits of 9 and 6 bits and 610 workgroups of four waves; now 175).
__global__ __launch_bounds__(kRTh) void k_rs_scatter(const uint32_t *__restrict__ kin,
                                                     const uint64_t *__restrict__ vin,
                                                     const uint32_t *__restrict__ kc, uint32_t *__restrict__ kout,
                                                     uint64_t *__restrict__ vout, const int64_t *m_dev, int shift,
                                                     int width, const int64_t *__restrict__ hoff, int64_t spans_cap)
{
    constexpr int kWaves = kRTh / 64;
    constexpr int kPart = kRTile / kWaves;             // entries per wave
    constexpr int kWRounds = kPart / 64;
    static_assert(kRMaxBuckets == kRTh, "one digit per thread");
    static_assert(kRTile < 65536, "places in a tile are 16-bit");
    __shared__ int64_t s_base[kRMaxBuckets];           // place of the tile's first entry of each digit, less its place in the tile
    __shared__ uint16_t s_cnt[kWaves][kRMaxBuckets];
    __shared__ uint64_t s_v[kRTile];
    __shared__ uint32_t s_w[kWaves];
    uint32_t *s_k = reinterpret_cast<uint32_t *>(s_v);
    const int64_t M = *m_dev;
    const int64_t nspans = (M + kRSpanLen - 1) / kRSpanLen;
    const int nb = 1 << width;
    const uint32_t mask = (uint32_t)nb - 1;
    const int tid = (int)threadIdx.x, wave = uni32(tid >> 6), lane = lane_id();
    const uint64_t lt = (1ull << lane) - 1;
    uint16_t *cnt = s_cnt[wave];
    for (int64_t sp = blockIdx.x; sp < nspans; sp += gridDim.x) {
        int64_t next = tid < nb ? hoff[(int64_t)tid * spans_cap + sp] : 0;     // this thread's digit's next place
        for (int64_t t0 = sp * kRSpanLen; t0 < min64((sp + 1) * kRSpanLen, M); t0 += kRTile) {
            const int64_t i0 = t0 + (int64_t)wave * kPart;
            uint32_t key[kWRounds];
            uint64_t val[kWRounds];
            uint32_t rank[kWRounds];
#pragma unroll
            for (int r = 0; r < kWRounds; ++r) {
                const int64_t i = i0 + r * 64 + lane;
                const bool valid = i < M;
                key[r] = valid ? kin[i] : 0;
                val[r] = !valid ? 0 : (vin ? vin[i] : ((uint64_t)kc[i] << 32 | (uint64_t)i));
            }
            for (int d = lane; d < nb; d += 64) cnt[d] = 0;
            __builtin_amdgcn_wave_barrier();
            // this wave's part: ranks among its entries of the same digit
#pragma unroll
            for (int r = 0; r < kWRounds; ++r) {
                const bool valid = i0 + r * 64 + lane < M;
                const uint32_t d = (key[r] >> shift) & mask;
                uint64_t peers = __ballot(valid);
                for (int b = 0; b < width; ++b) {
                    const bool bit = (d >> b) & 1u;
                    const uint64_t m = __ballot(valid && bit);
                    peers &= bit ? m : ~m;
                }
                const uint32_t below = (uint32_t)__popcll(peers & lt);
                const uint32_t had = valid ? cnt[d] : 0u;
                rank[r] = had + below;
                __builtin_amdgcn_wave_barrier();
                if (valid && below == 0) cnt[d] = (uint16_t)(had + (uint32_t)__popcll(peers));
                __builtin_amdgcn_wave_barrier();
            }
            __syncthreads();
            // wave counts -> the tile's counts, where each digit starts in the
            // tile, and the waves' bases there
            uint32_t c[kWaves], tot = 0;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {
                c[w] = tid < nb ? s_cnt[w][tid] : 0u;
                tot += c[w];
            }
            const uint32_t inc = (uint32_t)wave_incl_sum_dpp(tot);
            if (lane == 63) s_w[wave] = inc;
            __syncthreads();
            uint32_t run = inc - tot;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) run += w < wave ? s_w[w] : 0u;
            if (tid < nb) {
                s_base[tid] = next - (int64_t)run;
                next += tot;
#pragma unroll
                for (int w = 0; w < kWaves; ++w) {
                    s_cnt[w][tid] = (uint16_t)run;
                    run += c[w];
                }
            }
            __syncthreads();
#pragma unroll
            for (int r = 0; r < kWRounds; ++r) {
                if (i0 + r * 64 + lane >= M) continue;
                rank[r] += cnt[(key[r] >> shift) & mask];
                s_k[rank[r]] = key[r];
            }
            __syncthreads();
            const int n_t = (int)min64(kRTile, M - t0);
            int64_t g[kWRounds];
#pragma unroll
            for (int r = 0; r < kWRounds; ++r) {
                const int j = r * kRTh + tid;
                g[r] = 0;
                if (j < n_t) {
                    const uint32_t k = s_k[j];
                    g[r] = s_base[(k >> shift) & mask] + j;
                    kout[g[r]] = k;
                }
            }
            __syncthreads();
#pragma unroll
            for (int r = 0; r < kWRounds; ++r)
                if (i0 + r * 64 + lane < M) s_v[rank[r]] = val[r];
            __syncthreads();
#pragma unroll
            for (int r = 0; r < kWRounds; ++r) {
                const int j = r * kRTh + tid;
                if (j < n_t) vout[g[r]] = s_v[j];
            }
            __syncthreads();
        }
    }
}

// First and end sorted index of every parent that has ready entries.  After
// an error (an id out of range leaves its entry's parent unset) the parents
// are not trusted: every kernel from here on returns at once.
__global__ void k_pb_bounds(const uint32_t *__restrict__ key, const int64_t *m_dev, int64_t P,
                            uint32_t *__restrict__ pstart, uint32_t *__restrict__ pend, uint4 *__restrict__ fmark,
                            Ctl *ctl)
{
    const int64_t M = *m_dev;
    const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t w = tid; w <= M >> 4; w += stride) fmark[w] = make_uint4(0, 0, 0, 0);   // set next, at groups' firsts (none after an error)
    if (read_err(ctl) != 0) return;
    // four keys a thread, and the one before them
    for (int64_t s0 = 4 * tid; s0 < M; s0 += 4 * stride) {
        uint32_t k[4], before = s0 > 0 ? key[s0 - 1] : 0xffffffffu;
        if (s0 + 4 <= M) {
            const uint4 x = *reinterpret_cast<const uint4 *>(key + s0);
            k[0] = x.x; k[1] = x.y; k[2] = x.z; k[3] = x.w;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) k[j] = s0 + j < M ? key[s0 + j] : 0xffffffffu;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (s0 + j < M && (s0 + j == 0 || k[j] != before)) {
                if ((int64_t)k[j] < P) pstart[k[j]] = (uint32_t)(s0 + j);
                if (s0 + j > 0 && (int64_t)before < P) pend[before] = (uint32_t)(s0 + j);
            }
            before = k[j];
        }
        if (s0 + 4 >= M) {
            const uint32_t last = key[M - 1];
            if ((int64_t)last < P) pend[last] = (uint32_t)M;
        }
    }
}

// The queue position of every group's first entry (rank a multiple of B) gets
// a byte with the group's size: a full group's and a size that a byte cannot
// hold have marks of their own.  A byte needs no atomic: bits, set 64 to a word
// by neighbouring lanes, took 584 us for one parent's 10M batches of one, the
// bytes 22.  Ranks fit 32 bits (a queue position does), so they are
// divided in 32.  Four entries a thread, the loads of each step of their
// chains together.
constexpr uint32_t kMarkFull = 255, kMarkLook = 254;
constexpr int kPbItems = 4;

__global__ __launch_bounds__(kBlock) void k_pb_firsts(const uint32_t *__restrict__ key,
                                                      const uint64_t *__restrict__ val, const int64_t *m_dev, int64_t P,
                                                      const uint32_t *__restrict__ pstart,
                                                      const uint32_t *__restrict__ pend, uint32_t B,
                                                      uint32_t *__restrict__ fsize, uint8_t *__restrict__ fmark, Ctl *ctl)
{
    if (read_err(ctl) != 0) return;
    const int64_t M = *m_dev;
    for (int64_t s0 = (int64_t)blockIdx.x * (kBlock * kPbItems) + threadIdx.x; s0 < M;
         s0 += (int64_t)gridDim.x * (kBlock * kPbItems)) {
        uint32_t p[kPbItems], st[kPbItems];
#pragma unroll
        for (int k = 0; k < kPbItems; ++k) p[k] = s0 + k * kBlock < M ? key[s0 + k * kBlock] : 0xffffffffu;
#pragma unroll
        for (int k = 0; k < kPbItems; ++k) st[k] = (int64_t)p[k] < P ? pstart[p[k]] : 0u;
#pragma unroll
        for (int k = 0; k < kPbItems; ++k) {
            const int64_t s = s0 + k * kBlock;
            if (s >= M || (int64_t)p[k] >= P) continue;
            if (((uint32_t)s - st[k]) % B != 0) continue;
            const uint32_t left = pend[p[k]] - (uint32_t)s, q = (uint32_t)val[s];
            const bool look = left < B && left >= kMarkLook;
            if (look) fsize[q] = left;
            fmark[q] = (uint8_t)(look ? kMarkLook : left < B ? left : B < kMarkLook ? B : kMarkFull);
        }
    }
}

// Groups in queue order of their first entries: one pass over the bytes of the
// queue positions, 32 a thread, with two look-back chains (groups so far,
// entries so far); sizes are read only where a byte says so.  A group's first
// position gets its batch's first slot, which is batch_off[b] of its batch
// number b; the last tile writes batch_off[n_batches] and the totals.  Tiles
// are large, since a tile costs a ticket and a look-back: 10M entries in
// 55,000 groups took 70 us in tiles of 4,096 positions that read every size,
// now 35.
constexpr int kPbScanTh = 1024, kPbScanIt = 32;
constexpr int kPbScanTile = kPbScanTh * kPbScanIt;           // positions per tile

__global__ __launch_bounds__(kPbScanTh) void k_pb_scan(const uint32_t *__restrict__ fsize,
                                                       const uint4 *__restrict__ fmark, const int64_t *m_dev,
                                                       int64_t out_cap, uint32_t B, uint32_t *__restrict__ gslot,
                                                       int64_t *__restrict__ batch_off, int64_t batch_cap,
                                                       int64_t *n_out, int64_t *n_batches, Ctl *ctl, uint64_t *desc,
                                                       uint64_t *desc_b, int64_t desc_cap)
{
    const uint32_t epoch = scan_epoch(ctl);
    __shared__ uint64_t s_w[kPbScanTh / 64];
    __shared__ uint64_t s_b2[2];
    __shared__ int64_t s_t;
    __shared__ int32_t s_last;
    const int64_t M = *m_dev;
    const int64_t ntiles = (M + kPbScanTile - 1) / kPbScanTile;
    const int wv = (int)(threadIdx.x >> 6), ln = lane_id();
    if (M > out_cap && blockIdx.x == 0 && threadIdx.x == 0) raise_err(ctl, RO_ECAP);
    if (M == 0 && blockIdx.x == 0 && threadIdx.x == 0) {
        if (batch_cap < 1) raise_err(ctl, RO_ECAP);
        else batch_off[0] = 0;
        if (n_out) *n_out = 0;
        if (n_batches) *n_batches = 0;
    }
    for (;;) {
        const int64_t t = next_ticket(ctl, &s_t);
        if (t >= ntiles) break;
        const int64_t i0 = t * kPbScanTile + (int64_t)threadIdx.x * kPbScanIt;
        // bytes at M and above are cleared up to a multiple of 16
        const uint4 none = make_uint4(0, 0, 0, 0);
        const uint4 x0 = i0 < M ? fmark[i0 >> 4] : none, x1 = i0 + 16 < M ? fmark[(i0 >> 4) + 1] : none;
        const uint32_t x[kPbScanIt / 4] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
        uint32_t f[kPbScanIt], bits = 0;
        uint64_t sum = 0;
#pragma unroll
        for (int k = 0; k < kPbScanIt; ++k) {
            const uint32_t m = x[k >> 2] >> (8 * (k & 3)) & 255u;
            f[k] = m == kMarkFull ? B : m == kMarkLook ? fsize[i0 + k] : m;
            bits |= m ? 1u << k : 0u;
        }
#pragma unroll
        for (int k = 0; k < kPbScanIt; ++k) sum += f[k];
        // one block scan of entries << 16 | groups (a tile holds at most 32,768 groups)
        const uint64_t v = sum << 16 | (uint64_t)__popc(bits);
        const uint64_t inc = wave_incl_sum_dpp(v);
        if (ln == 63) s_w[wv] = inc;
        __syncthreads();
        uint64_t ex = inc - v, tot = 0;
#pragma unroll
        for (int i = 0; i < kPbScanTh / 64; ++i) {
            const uint64_t x = s_w[i];
            ex += i < wv ? x : 0;
            tot += x;
        }
        const int64_t tc = (int64_t)(tot & 0xffffu), ts = (int64_t)(tot >> 16);
        uint64_t pc, ps;
        tile_prefix2(desc, (uint64_t)tc, desc_b, (uint64_t)ts, t, epoch, s_b2, pc, ps, ctl);
        int64_t b = (int64_t)pc + (int64_t)(ex & 0xffffu), o = (int64_t)ps + (int64_t)(ex >> 16);
        bool over = false;
#pragma unroll
        for (int k = 0; k < kPbScanIt; ++k) {
            if (!((bits >> k) & 1u)) continue;
            gslot[i0 + k] = (uint32_t)o;
            if (b < batch_cap) batch_off[b] = o;
            else over = true;
            ++b;
            o += f[k];
        }
        if (over) raise_err(ctl, RO_ECAP);
        if (t == ntiles - 1 && threadIdx.x == 0) {
            const int64_t nbat = (int64_t)pc + tc;
            if (nbat < batch_cap) batch_off[nbat] = (int64_t)ps + ts;
            else raise_err(ctl, RO_ECAP);
            if (n_out) *n_out = (int64_t)ps + ts;
            if (n_batches) *n_batches = nbat;
        }
        if (ntiles <= (int64_t)gridDim.x) break;     // a tile for every workgroup
    }
    ticket_done(ctl, epoch, desc, desc_cap, &s_last);
}

// Every entry to its group's slots: the group's first slot + rank mod B.  The
// chain of an entry (parent, first sorted entry, its group's queue position,
// the group's slot) is four loads one after another, so four entries a thread
// go through it together (10M entries: 88 us one by one, now 55).
__global__ __launch_bounds__(kBlock) void k_pb_place(
    const uint32_t *__restrict__ key, const uint64_t *__restrict__ val, const int64_t *m_dev, int64_t P,
    const uint32_t *__restrict__ pstart, uint32_t B, const uint32_t *__restrict__ gslot,
    const int64_t *__restrict__ offsets, uint32_t *__restrict__ out_child, uint32_t *__restrict__ out_parent,
    uint32_t *__restrict__ out_ordinal, int64_t out_cap, Ctl *ctl)
{
    if (read_err(ctl) != 0) return;          // a capacity error leaves the outputs unwritten
    const int64_t M = *m_dev;
    if (M > out_cap) return;
    for (int64_t s0 = (int64_t)blockIdx.x * (kBlock * kPbItems) + threadIdx.x; s0 < M;
         s0 += (int64_t)gridDim.x * (kBlock * kPbItems)) {
        uint32_t p[kPbItems], in[kPbItems], first[kPbItems], slot[kPbItems], c[kPbItems];
        int64_t off[kPbItems];
#pragma unroll
        for (int k = 0; k < kPbItems; ++k) {
            const int64_t s = s0 + k * kBlock;
            p[k] = s < M ? key[s] : 0xffffffffu;
            c[k] = s < M ? (uint32_t)(val[s] >> 32) : 0u;
        }
#pragma unroll
        for (int k = 0; k < kPbItems; ++k) {
            first[k] = (int64_t)p[k] < P ? pstart[p[k]] : 0u;
            off[k] = out_ordinal && (int64_t)p[k] < P ? offsets[p[k]] : 0;
        }
#pragma unroll
        for (int k = 0; k < kPbItems; ++k) {
            const uint32_t s = (uint32_t)(s0 + k * kBlock);
            const bool ok = s0 + k * kBlock < M && (int64_t)p[k] < P;
            in[k] = ok ? (s - first[k]) % B : 0u;
            first[k] = ok ? (uint32_t)val[s - in[k]] : 0xffffffffu;
        }
#pragma unroll
        for (int k = 0; k < kPbItems; ++k) slot[k] = s0 + k * kBlock < M && (int64_t)p[k] < P ? gslot[first[k]] + in[k] : 0u;
#pragma unroll
        for (int k = 0; k < kPbItems; ++k) {
            if (s0 + k * kBlock >= M || (int64_t)p[k] >= P) continue;
            if (out_child) out_child[slot[k]] = c[k];
            if (out_parent) out_parent[slot[k]] = p[k];
            if (out_ordinal) out_ordinal[slot[k]] = (uint32_t)((int64_t)c[k] - off[k]);
        }
    }
}

static int64_t grid_for(const Launch &L, int64_t n, int64_t per_block)
{
    int64_t grid = (n + per_block - 1) / per_block;
    return grid < 1 ? 1 : (grid > (int64_t)L.num_cus * 8 ? (int64_t)L.num_cus * 8 : grid);
}

hipError_t launch_batch_parent(const Launch &L, const uint32_t *queue, const uint8_t *keep, int64_t Q,
                               const int64_t *offsets, int64_t P, int32_t B, uint32_t *out_child,
                               uint32_t *out_parent, uint32_t *out_ordinal, int64_t out_cap, int64_t *batch_off,
                               int64_t batch_cap, int64_t *n_out, int64_t *n_batches, uint32_t *cmap,
                               int64_t cmap_cap, const uint8_t *barrier, const PbWs &w)
{
    // ready entries in queue order: children and parents, count in w.m
    hipError_t e = launch_batch(L, queue, keep, Q, offsets, P, B, w.kc, w.k[0], nullptr, Q, w.m, w.m + 1, cmap,
                                cmap_cap, barrier);
    if (e != hipSuccess) return e;
    // stable sort by parent: as few passes of at most kRMaxBits bits as the
    // parent ids need, of equal widths (fewer digits, longer runs)
    int bits = 0;
    while (bits < 32 && ((uint64_t)1 << bits) < (uint64_t)P) ++bits;
    const int passes = bits == 0 ? 1 : (bits + kRMaxBits - 1) / kRMaxBits;   // one pass of width 0 copies
    const int64_t spans_cap = (Q + kRSpanLen - 1) / kRSpanLen > 0 ? (Q + kRSpanLen - 1) / kRSpanLen : 1;
    const int64_t gsort = spans_cap < (int64_t)L.num_cus * 8 ? spans_cap : (int64_t)L.num_cus * 8;
    int cur = 0;
    const uint64_t *vals = nullptr;          // built from the compaction in the first pass
    for (int pass = 0, shift = 0; pass < passes; ++pass) {
        const int left = passes - pass, width = (bits - shift + left - 1) / left;
        RO_LAUNCH(L, RO_K_PBATCH_SORT, k_rs_hist, dim3((unsigned)gsort), dim3(kBlock), 0, L.stream, w.k[cur], w.m,
                  shift, width, w.hist, spans_cap);
        e = launch_expand(L, w.hist, (int64_t)(1 << width) * spans_cap, w.hoff, nullptr, nullptr, 0);
        if (e != hipSuccess) return e;
        RO_LAUNCH(L, RO_K_PBATCH_SORT, k_rs_scatter, dim3((unsigned)gsort), dim3(kRTh), 0, L.stream, w.k[cur],
                  vals, w.kc, w.k[1 - cur], w.v[1 - cur], w.m, shift, width, w.hoff, spans_cap);
        vals = w.v[1 - cur];
        cur = 1 - cur;
        shift += width;
    }
    const uint32_t *keys = w.k[cur];
    const int64_t g = grid_for(L, Q, kBlock * kPbItems);
    RO_LAUNCH(L, RO_K_PBATCH, k_pb_bounds, dim3((unsigned)g), dim3(kBlock), 0, L.stream, keys, w.m, P, w.pstart,
              w.pend, reinterpret_cast<uint4 *>(w.fmark), L.ctl);
    RO_LAUNCH(L, RO_K_PBATCH, k_pb_firsts, dim3((unsigned)g), dim3(kBlock), 0, L.stream, keys, vals, w.m, P,
              w.pstart, w.pend, (uint32_t)B, w.fsize, w.fmark, L.ctl);
    const int64_t ntiles = (Q + kPbScanTile - 1) / kPbScanTile > 0 ? (Q + kPbScanTile - 1) / kPbScanTile : 1;
    const int64_t gscan = ntiles < (int64_t)L.num_cus * 4 ? ntiles : (int64_t)L.num_cus * 4;
    if (2 * ntiles > L.desc_cap) return hipErrorInvalidValue;
    RO_LAUNCH(L, RO_K_PBATCH, k_pb_scan, dim3((unsigned)gscan), dim3(kPbScanTh), 0, L.stream, w.fsize,
              reinterpret_cast<const uint4 *>(w.fmark), w.m, out_cap, (uint32_t)B, w.gslot, batch_off, batch_cap, n_out, n_batches, L.ctl, L.desc, L.desc + ntiles, L.desc_cap);
    RO_LAUNCH(L, RO_K_PBATCH, k_pb_place, dim3((unsigned)g), dim3(kBlock), 0, L.stream, keys, vals, w.m, P,
              w.pstart, (uint32_t)B, w.gslot, offsets, out_child, out_parent, out_ordinal, out_cap, L.ctl);
    return hipGetLastError();
}

}  // namespace ro
