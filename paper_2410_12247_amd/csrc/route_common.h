// Device helpers the router kernels share: cross-lane maxima and sums, top-k
// selection with softmax weights.
#pragma once

#include <type_traits>

#include "lds_dma.h"

namespace moe {
namespace {

template <int CTRL>
__device__ __forceinline__ uint32_t dpp32(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, 0xF, 0xF, false);
}

__device__ __forceinline__ uint64_t max_u64(uint64_t a, uint64_t b) { return a > b ? a : b; }

template <int CTRL>
__device__ __forceinline__ uint64_t dpp64(uint64_t v) {
    uint32_t lo = dpp32<CTRL>((uint32_t)v);
    uint32_t hi = dpp32<CTRL>((uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint64_t readlane64(uint64_t v, int l) {
    uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
    uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), l);
    return ((uint64_t)hi << 32) | lo;
}

// Wave-wide max: butterfly inside each 16-lane row (quad_perm 1032, quad_perm
// 2301, half-row mirror, row mirror), then the four row results by readlane.
__device__ __forceinline__ uint64_t wave_max_u64(uint64_t k) {
    k = max_u64(k, dpp64<0xB1>(k));
    k = max_u64(k, dpp64<0x4E>(k));
    k = max_u64(k, dpp64<0x141>(k));
    k = max_u64(k, dpp64<0x140>(k));
    return max_u64(max_u64(readlane64(k, 0), readlane64(k, 16)),
                   max_u64(readlane64(k, 32), readlane64(k, 48)));
}

__device__ __forceinline__ double dpp_f64(double v, int which) {
    uint64_t b = __builtin_bit_cast(uint64_t, v);
    uint64_t r;
    switch (which) {
        case 0: r = dpp64<0xB1>(b); break;
        case 1: r = dpp64<0x4E>(b); break;
        case 2: r = dpp64<0x141>(b); break;
        default: r = dpp64<0x140>(b); break;
    }
    return __builtin_bit_cast(double, r);
}

// Wave-wide fp64 sum; every lane combines the same pairs (commutative adds),
// so the result is identical in all lanes and from run to run.
__device__ __forceinline__ double wave_sum_f64(double v) {
#pragma unroll
    for (int i = 0; i < 4; ++i) v = v + dpp_f64(v, i);
    uint64_t b = __builtin_bit_cast(uint64_t, v);
    double r0 = __builtin_bit_cast(double, readlane64(b, 0));
    double r1 = __builtin_bit_cast(double, readlane64(b, 16));
    double r2 = __builtin_bit_cast(double, readlane64(b, 32));
    double r3 = __builtin_bit_cast(double, readlane64(b, 48));
    return (r0 + r1) + (r2 + r3);
}

__device__ __forceinline__ uint64_t logit_key(float z, int e) {
    uint32_t u = __float_as_uint(z);
    if (u == 0x80000000u) u = 0;  // -0 ranks equal to +0
    const uint32_t ord = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
    return ((uint64_t)ord << 32) | (uint32_t)(0xFFFFFFFFu - (uint32_t)e);
}

__device__ __forceinline__ float key_logit(uint64_t key) {
    const uint32_t ord = (uint32_t)(key >> 32);
    const uint32_t u = (ord & 0x80000000u) ? (ord & 0x7FFFFFFFu) : ~ord;
    return __uint_as_float(u);
}

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// Wave-wide max of an unsigned dword: inside each 16-lane row by DPP, then
// the four row results by readlane.
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
    v = max(v, dpp32<0xB1>(v));
    v = max(v, dpp32<0x4E>(v));
    v = max(v, dpp32<0x141>(v));
    v = max(v, dpp32<0x140>(v));
    const uint32_t a = __builtin_amdgcn_readlane(v, 0), b = __builtin_amdgcn_readlane(v, 16);
    const uint32_t c = __builtin_amdgcn_readlane(v, 32), d = __builtin_amdgcn_readlane(v, 48);
    return max(max(a, b), max(c, d));
}

// Lane j < k holds the j-th selected expert; those whose logit is the NaN of
// all one bits (their rounds found no other) become the lowest experts not
// taken, in order.
__device__ __forceinline__ int repick_zero_keys(int my_e, float my_z, int E, int k, int lane) {
    const uint64_t redo = __builtin_amdgcn_ballot_w64(lane < k && __float_as_uint(my_z) == ~0u);
    for (int j = redo ? __builtin_ctzll(redo) : k; j < k; ++j) {
        int e = 0;
        for (int q = 3; q >= 0; --q) {
            bool left = lane + 64 * q < E;
            for (int p = 0; p < j; ++p)
                left &= __builtin_amdgcn_readlane(my_e, p) != lane + 64 * q;
            const uint64_t m = __builtin_amdgcn_ballot_w64(left);
            if (m) e = 64 * q + __builtin_ctzll(m);
        }
        if (lane == j) my_e = e;
    }
    return my_e;
}

// Top-k and softmax weights of the N tokens t[i] (those below T) from their
// E logits zrow[i], by one wave: lane l holds experts l, l+64, l+128, l+192;
// each of the k rounds takes the wave-wide max of the logits'
// order-preserving bits and, among the lanes that hold it, the lowest expert
// (a ballot per 64 experts); the weights are fp64 softmax values rounded
// once to fp32, lane j taking the j-th selected expert's.  Several tokens
// at once hide each other's cross-lane latency.  A token's k experts are
// distinct whatever its logits (the row counts and buffers downstream rely
// on it): bits of 0 mark a taken expert but are also those of the NaN of all
// one bits, so the rounds that found nothing above 0 are done again (after
// the rounds, whose tokens a branch in them would keep apart: 65536 tokens x
// 160 experts 798 -> 807 us).
template <int N>
__device__ __forceinline__ void select_tokens(const float *const (&zrow)[N],
                                              const int64_t (&t)[N], int64_t T, int E, int k,
                                              int renorm, int lane, int32_t *__restrict__ ids,
                                              float *__restrict__ wout) {
    uint32_t ord[N][4];
    float zl[N][4];
    float my_z[N], zmax[N];
    int my_e[N];
    uint32_t last[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        my_z[i] = zmax[i] = 0.0f;
        my_e[i] = 0;
        last[i] = 1u;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int e = lane + 64 * q;
            zl[i][q] = e < E ? zrow[i][e] : 0.0f;
            ord[i][q] = e < E ? (uint32_t)(logit_key(zl[i][q], e) >> 32) : 0u;
        }
    }
    for (int j = 0; j < k; ++j) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const uint32_t best = wave_max_u32(
                max(max(ord[i][0], ord[i][1]), max(ord[i][2], ord[i][3])));
            int e = 0;
#pragma unroll
            for (int q = 3; q >= 0; --q) {
                const uint64_t m = __builtin_amdgcn_ballot_w64(ord[i][q] == best);
                if (m) e = 64 * q + __builtin_ctzll(m);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (lane + 64 * q == e) ord[i][q] = 0u;
            const float z = key_logit((uint64_t)best << 32);
            if (j == 0) zmax[i] = z;
            if (lane == j) {
                my_e[i] = e;
                my_z[i] = z;
            }
            last[i] = best;
        }
    }
#pragma unroll
    for (int i = 0; i < N; ++i)
        if (last[i] == 0u) my_e[i] = repick_zero_keys(my_e[i], my_z[i], E, k, lane);
    double ex[N], denom[N];
#pragma unroll
    for (int i = 0; i < N; ++i) ex[i] = exp((double)my_z[i] - (double)zmax[i]);
    if (renorm) {
#pragma unroll
        for (int i = 0; i < N; ++i) denom[i] = 0.0;
        for (int j = 0; j < k; ++j)
#pragma unroll
            for (int i = 0; i < N; ++i)
                denom[i] += __builtin_bit_cast(
                    double, readlane64(__builtin_bit_cast(uint64_t, ex[i]), j));
    } else {
#pragma unroll
        for (int i = 0; i < N; ++i) denom[i] = 0.0;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (64 * q < E) {
#pragma unroll
                for (int i = 0; i < N; ++i) {
                    const double p = exp((double)zl[i][q] - (double)zmax[i]);
                    if (lane + 64 * q < E) denom[i] += p;
                }
            }
#pragma unroll
        for (int i = 0; i < N; ++i) denom[i] = wave_sum_f64(denom[i]);
    }
#pragma unroll
    for (int i = 0; i < N; ++i)
        if (t[i] < T && lane < k) {
            ids[t[i] * k + lane] = my_e[i];
            wout[t[i] * k + lane] = (float)(ex[i] / denom[i]);
        }
}
__device__ __forceinline__ void select_token(const float *zrow, int64_t t, int E, int k,
                                             int renorm, int lane, int32_t *__restrict__ ids,
                                             float *__restrict__ wout) {
    const float *const z[1] = {zrow};
    const int64_t tt[1] = {t};
    select_tokens<1>(z, tt, t + 1, E, k, renorm, lane, ids, wout);
}

// Calls f(integral_constant<int, I>) for I = B .. N - 1.
template <int B, int N, class F>
__device__ __forceinline__ void lane_unroll(F &&f) {
    if constexpr (B < N) {
        f(std::integral_constant<int, B>{});
        lane_unroll<B + 1, N>(f);
    }
}

// top-k and softmax weights of one token from its E logits, by one lane
template <int EP>
__device__ __forceinline__ void select_lane(const float *zrow, int64_t t, int E, int k,
                                            int renorm, int32_t *__restrict__ ids,
                                            float *__restrict__ wout) {
    uint64_t key[EP];
    float z[EP];
#pragma unroll
    for (int e = 0; e < EP; ++e) {
        z[e] = e < E ? zrow[e] : 0.0f;
        key[e] = e < E ? logit_key(z[e], e) : 0ull;
    }
    int sel_e[kMaxTopK];
    float sel_z[kMaxTopK];
#pragma unroll
    for (int j = 0; j < kMaxTopK; ++j) {
        sel_e[j] = 0;
        sel_z[j] = 0.0f;
        if (j < k) {
            uint64_t best = key[0];
#pragma unroll
            for (int e = 1; e < EP; ++e) best = max_u64(best, key[e]);
            sel_e[j] = (int)(0xFFFFFFFFu - (uint32_t)best);
            sel_z[j] = key_logit(best);
#pragma unroll
            for (int e = 0; e < EP; ++e)
                if (key[e] == best) key[e] = 0ull;
        }
    }
    const double zmax = (double)sel_z[0];
    double denom = 0.0;
    if (renorm) {
#pragma unroll
        for (int j = 0; j < kMaxTopK; ++j)
            if (j < k) denom += exp((double)sel_z[j] - zmax);
    } else {
#pragma unroll
        for (int e = 0; e < EP; ++e)
            if (e < E) denom += exp((double)z[e] - zmax);
    }
#pragma unroll
    for (int j = 0; j < kMaxTopK; ++j) {
        if (j < k) {
            ids[t * k + j] = sel_e[j];
            wout[t * k + j] = (float)(exp((double)sel_z[j] - zmax) / denom);
        }
    }
}

}  // namespace
}  // namespace moe
