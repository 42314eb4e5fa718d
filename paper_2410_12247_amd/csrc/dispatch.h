// Dispatch of few slots by one wave (device): the row order of the three-pass
// dispatch, for its one-launch form and for the tail of a router launch that
// is a single workgroup.
#pragma once

#include "common.h"

namespace moe {
namespace {

// Inclusive scan over a wave: DPP row_shr 1, 2, 4, 8 inside each 16-lane row
// (lanes with no source add 0), then row totals carried with readlane.
__device__ __forceinline__ int wave_inclusive_scan(int v) {
    const int lane = threadIdx.x & 63;
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);  // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);  // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);  // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);  // row_shr:8
    const int r0 = __builtin_amdgcn_readlane(v, 15);
    const int r1 = __builtin_amdgcn_readlane(v, 31);
    const int r2 = __builtin_amdgcn_readlane(v, 47);
    const int row = lane >> 4;
    v += (row > 0 ? r0 : 0) + (row > 1 ? r1 : 0) + (row > 2 ? r2 : 0);
    return v;
}

// The LDS traffic of one wave: in order, so only the compiler has to keep it.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// At most 64 NIT slots, by one wave; cnt, off: LDS of kMaxExperts ints each.
template <int NIT>
__device__ __forceinline__ void dispatch_wave(const int32_t *ids, int64_t nslots, int k,
                                              const DispatchOut &o, int *cnt, int *off) {
    const int lane = threadIdx.x & 63;
    for (int e = lane; e < o.NB; e += 64) cnt[e] = 0;
    wave_sync();
    const uint64_t lt_mask = (1ull << lane) - 1ull;
    // groups of 64 slots that hold any (the rest of the unrolled loops is
    // skipped: decode batches have one or two)
    const int nit = (int)((nslots + 63) / 64);
    int idv[NIT], bucket[NIT], rank[NIT];
#pragma unroll
    for (int it = 0; it < NIT; ++it) idv[it] = ids[min<int64_t>(it * 64 + lane, nslots - 1)];
    asm volatile("" ::: "memory");
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        bucket[it] = -1;
        rank[it] = 0;
        if (it >= nit) continue;
        const int s = it * 64 + lane;
        int e = idv[it] - o.e0;
        if (s >= nslots || e < 0 || e >= o.EL) e = -1;
        else if (o.tokens_per_stage > 0)
            e += (int)((uint32_t)s / (uint32_t)k / (uint32_t)o.tokens_per_stage) * o.EL;
        const uint32_t v = (uint32_t)(e + 1);
        uint64_t match = ~0ull;
#pragma unroll
        for (int b = 0; b < 9; ++b) {
            const bool bit = (v >> b) & 1u;
            const uint64_t bal = __ballot(bit);
            match &= bit ? bal : ~bal;
        }
        const int before = __popcll(match & lt_mask);
        bucket[it] = e;
        rank[it] = e >= 0 ? cnt[e] + before : 0;
        wave_sync();
        if (e >= 0 && before == 0) cnt[e] += __popcll(match);
        wave_sync();
    }
    int carry = 0;
    for (int b0 = 0; b0 < o.NB; b0 += 64) {
        const int e = b0 + lane;
        const int v = e < o.NB ? cnt[e] : 0;
        const int incl = wave_inclusive_scan(v);
        if (e < o.NB) {
            o.counts[e] = v;
            off[e] = carry + incl - v;
            o.offsets[e] = carry + incl - v;
        }
        carry += __builtin_amdgcn_readlane(incl, 63);
    }
    if (lane == 0) o.offsets[o.NB] = carry;
    if (o.counts_el) {  // rows per local expert over the stages
        for (int e = lane; e < o.EL; e += 64) {
            int sum = 0;
            for (int b = e; b < o.NB; b += o.EL) sum += cnt[b];
            o.counts_el[e] = sum;
        }
    }
    wave_sync();
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        const int s = it * 64 + lane;
        if (it < nit && s < nslots) {
            const int e = bucket[it];
            if (e < 0) {
                o.slot_row[s] = -1;
            } else {
                const int row = off[e] + rank[it];
                o.sorted_slot[row] = s;
                o.slot_row[s] = row;
            }
        }
    }
}

}  // namespace
}  // namespace moe
