// Writing the lineage keys of an expansion.
#pragma once
#include "ro_device.h"

namespace ro {

// Lineage keys: child c -> (p, c - offsets[p]).  Each thread owns 16
// consecutive children, finds the parent of the first one by binary search
// and walks forward, so a huge parent is spread over as many threads as it
// has children/16 and never serialises a wave.
// Expansions of more children than this write their tags with
// non-temporal stores (32 MB per tag array, the size of all L2s).
constexpr int64_t kTagsNtChildren = (int64_t)8 << 20;

__device__ __forceinline__ void write_keys(const int64_t *__restrict__ offsets, int64_t P,
                                           uint32_t *__restrict__ child_parent, uint32_t *__restrict__ child_ordinal,
                                           int64_t child_cap, int64_t done_up_to, int vec_ok)
{
    constexpr int kWaveSpan = 64 * kItems;            // children per wave and step
    __shared__ alignas(16) uint32_t s_stage[kBlock / 64][kWaveSpan];
    const int64_t N = offsets[P];
    if (N > child_cap || N >= ((int64_t)1 << 32) || P == 0) return;     // reported by the scan
    if (N <= done_up_to) return;                              // the launch before has written them
    const int lane = lane_id();
    const bool nt = N > kTagsNtChildren;
    uint32_t *stage = s_stage[threadIdx.x >> 6];
    const int64_t nwaves = (int64_t)gridDim.x * (kBlock / 64);
    for (int64_t wt = (int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6); wt * kWaveSpan < N; wt += nwaves) {
        // the wave's parent range by two wave-wide searches, then each lane's
        // first parent by a search inside that range
        const int64_t cb = wt * kWaveSpan;
        const int64_t ce = cb + kWaveSpan < N ? cb + kWaveSpan : N;
        const int64_t pf = wave_last_le(offsets, 0, P + 1, cb);
        const int64_t pl = wave_last_le(offsets, 0, P + 1, ce - 1);
        const int64_t c0 = cb + (int64_t)lane * kItems;
        // (a stream's offsets are not checked yet: below the first one there is no parent)
        int64_t p = c0 < N ? max64(upper_bound_g(offsets, pf, pl + 1, c0) - 1, 0) : pl;
        int64_t start = offsets[p];
        int64_t next = offsets[p + 1];
        uint32_t par[kItems], ord[kItems];
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            const int64_t c = c0 + k;
            if (c < N && c >= next) {
                p = advance_parent(offsets, P, p, c);
                start = offsets[p];
                next = offsets[p + 1];
            }
            par[k] = (uint32_t)p;
            ord[k] = (uint32_t)(c - start);
        }
        if (vec_ok && ce - cb == kWaveSpan) {
            // staged in LDS, then written 1 KiB per store instruction
#pragma unroll 1
            for (int which = 0; which < 2; ++which) {
                uint32_t *dst = which == 0 ? child_parent : child_ordinal;
                if (dst == nullptr) continue;
                const uint32_t *v = which == 0 ? par : ord;
#pragma unroll
                for (int k = 0; k < kItems / 4; ++k)
                    *reinterpret_cast<uint4 *>(&stage[lane * kItems + 4 * k]) =
                        make_uint4(v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]);
                __builtin_amdgcn_wave_barrier();
                if (nt) {
                    // non-temporal: an expansion this large is not read back
                    // soon, and its tags would only push other data out of L2
                    typedef uint32_t t4 __attribute__((ext_vector_type(4)));
                    t4 *out = reinterpret_cast<t4 *>(dst + cb);
#pragma unroll
                    for (int k = 0; k < kItems / 4; ++k)
                        __builtin_nontemporal_store(*reinterpret_cast<const t4 *>(&stage[(k * 64 + lane) * 4]),
                                                    out + k * 64 + lane);
                } else {
                    uint4 *out = reinterpret_cast<uint4 *>(dst + cb);
#pragma unroll
                    for (int k = 0; k < kItems / 4; ++k)
                        out[k * 64 + lane] = *reinterpret_cast<const uint4 *>(&stage[(k * 64 + lane) * 4]);
                }
                __builtin_amdgcn_wave_barrier();
            }
        } else {
#pragma unroll
            for (int k = 0; k < kItems; ++k) {
                if (c0 + k < N) {
                    if (child_parent) child_parent[c0 + k] = par[k];
                    if (child_ordinal) child_ordinal[c0 + k] = ord[k];
                }
            }
        }
    }
}

}  // namespace ro
