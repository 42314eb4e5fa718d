// Expert GEMMs of launches of few rows (at most 16 per expert): the GEMM is
// one pass over the weights and the time is the weight stream's.  A workgroup
// owns 16 NT weight rows of one expert over the whole of K; its eight waves
// each take an eighth of K and keep the fragments of R steps of 32 K in
// flight, loaded straight into registers in the MFMA's operand layout (no LDS
// and no barrier while the weights stream).  The waves' partial sums meet in
// LDS, are added in wave order (the same bits on every run) and the epilogue
// is applied there.  Against the tiled GEMM with a K split and its fix-up
// launch it saves the fix-up and the tiles' padding; its weight stream itself
// is no faster, so it runs where one of those weighs (stream_gateup_fits,
// stream_down_fits).  Forward, us, mean of four placements of the weights in
// memory, tiled -> this: Mixtral 1 token 70 -> 61, 4 tokens 125 -> 117; DBRX 1
// token 86 -> 78, 8 tokens 189 -> 181; 64 experts of 2048 x 1024, 1 token 59
// -> 54.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "common.h"

namespace moe {
namespace {

constexpr int SW = 8;  // waves of a workgroup (pieces of K)
// steps of 32 K in flight per wave: gate/up; down over a short and a long K
constexpr int kGateupSteps = 8, kShortSteps = 6, kLongSteps = 12;
constexpr int kStreamBufferFlags = 0x00020000;

__device__ __forceinline__ uint32_t pack2(float a, float b) {
    const uint16_t ua = __builtin_bit_cast(uint16_t, static_cast<__bf16>(a));
    const uint16_t ub = __builtin_bit_cast(uint16_t, static_cast<__bf16>(b));
    return (uint32_t)ua | ((uint32_t)ub << 16);
}
// as in the tiled GEMMs: hardware exp2 and reciprocal
__device__ __forceinline__ float silu_up(float g, float u) {
    const float e = __builtin_amdgcn_exp2f(g * -1.44269504088896341f);
    return g * __builtin_amdgcn_rcpf(1.0f + e) * u;
}

template <int B, int N, class F>
__device__ __forceinline__ void unroll(F &&f) {
    if constexpr (B < N) {
        f(std::integral_constant<int, B>{});
        unroll<B + 1, N>(f);
    }
}

// MODE 0: out = act [.][N] bf16, weight rows n0 .. + 8 NT - 1 of gate (w0)
// and up (w1); MODE 1: out = y [.][N] fp32, rows n0 .. + 16 NT - 1 of w0.
// At most 16 rows.  offsets, row_map and slot_div as in the grouped GEMM.
template <int MODE, int NT, int R>
__device__ __forceinline__ void stream_tile(float *lds, const int32_t *__restrict__ offsets,
                                            int e_first, const bf16_t *__restrict__ x,
                                            const int32_t *__restrict__ row_map, int slot_div,
                                            const bf16_t *__restrict__ w0s,
                                            const bf16_t *__restrict__ w1s, int64_t wstride,
                                            int N, int K, void *__restrict__ outp) {
    constexpr int COLS = MODE == 0 ? 8 * NT : 16 * NT;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ntile = N / COLS;
    const int e = blockIdx.x / ntile;
    const int n0 = (blockIdx.x - e * ntile) * COLS;
    const int r0 = __builtin_amdgcn_readfirstlane(offsets[e_first + e]);
    const int rows = __builtin_amdgcn_readfirstlane(offsets[e_first + e + 1]) - r0;
    if (rows <= 0) return;
    const int lr = lane & 15, q = lane >> 4;

    // weights: fragment t, MODE 0: gate rows, then up rows
    const int64_t wbase = (int64_t)(e_first + e) * wstride + (int64_t)n0 * K;
    const __amdgpu_buffer_rsrc_t wr0 = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(w0s + wbase), 0, (int)0xFFFFFFF0u, kStreamBufferFlags);
    const __amdgpu_buffer_rsrc_t wr1 =
        MODE == 0 ? __builtin_amdgcn_make_buffer_rsrc((void *)(w1s + wbase), 0, (int)0xFFFFFFF0u,
                                                      kStreamBufferFlags)
                  : wr0;
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(row_map ? x : x + (int64_t)r0 * K), 0, (int)0xFFFFFFF0u, kStreamBufferFlags);
    constexpr uint32_t DROP = 0xFFFFFFF8u;  // past the range: loads give 0
    const uint32_t woff = (uint32_t)(lr * K + q * 8) * 2u;
    const int xi = min(lr, rows - 1);  // rows past the last: repeats
    const int xsrc = row_map ? row_map[r0 + xi] / slot_div : xi;
    const uint32_t xoff = ((uint32_t)xsrc * (uint32_t)K + q * 8) * 2u;
    // this wave's steps of 32 K
    const int nk = K / 32;
    const int s0 = wave * nk / SW, s1 = (wave + 1) * nk / SW;

    u32x4 wf[R][NT], xf[R];
    auto load = [&](int s, auto slot) {
        constexpr int S = decltype(slot)::value;
        const bool on = s < s1;
        const int kb = s * 64;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const bool up = MODE == 0 && t >= NT / 2;
            const int tt = up ? t - NT / 2 : t;
            wf[S][t] = __builtin_amdgcn_raw_buffer_load_b128(
                up ? wr1 : wr0, on ? woff + (uint32_t)(tt * 32 * K) : DROP, on ? kb : 0, 0);
        }
        xf[S] = __builtin_amdgcn_raw_buffer_load_b128(xr, on ? xoff : DROP, on ? kb : 0, 0);
    };
    floatx4 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
    unroll<0, R>([&](auto i) { load(s0 + decltype(i)::value, i); });
    for (int s = s0; s < s1; s += R)
        unroll<0, R>([&](auto i) {
            constexpr int S = decltype(i)::value;
#pragma unroll
            for (int t = 0; t < NT; ++t)
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                    __builtin_bit_cast(bf16x8, wf[S][t]), __builtin_bit_cast(bf16x8, xf[S]),
                    acc[t], 0, 0, 0);
            load(s + S + R, i);
            __builtin_amdgcn_sched_barrier(0);
        });

    // partial sums: fragment t of wave w at 256 (w NT + t)
#pragma unroll
    for (int t = 0; t < NT; ++t)
        *reinterpret_cast<floatx4 *>(lds + (wave * NT + t) * 256 + lane * 4) = acc[t];
    __syncthreads();
    auto sum = [&](int t) {
        floatx4 v[SW];
#pragma unroll
        for (int w = 0; w < SW; ++w)
            v[w] = *reinterpret_cast<const floatx4 *>(lds + (w * NT + t) * 256 + lane * 4);
        floatx4 r = v[0];
#pragma unroll
        for (int w = 1; w < SW; ++w)
#pragma unroll
            for (int i = 0; i < 4; ++i) r[i] += v[w][i];
        return r;
    };
    // wave t: fragment t (or gate and up of it), whose lane holds columns
    // 4 q .. + 3 of row lr
    if (wave >= (MODE == 0 ? NT / 2 : NT) || lr >= rows) return;
    const int64_t o = (int64_t)(r0 + lr) * N + n0 + wave * 16 + q * 4;
    if (MODE == 0) {
        const floatx4 g = sum(wave), u = sum(wave + NT / 2);
        uint2 v;
        v.x = pack2(silu_up(g[0], u[0]), silu_up(g[1], u[1]));
        v.y = pack2(silu_up(g[2], u[2]), silu_up(g[3], u[3]));
        *reinterpret_cast<uint2 *>(reinterpret_cast<bf16_t *>(outp) + o) = v;
    } else {
        *reinterpret_cast<floatx4 *>(reinterpret_cast<float *>(outp) + o) = sum(wave);
    }
}

template <int MODE, int NT, int R>
__global__ __launch_bounds__(64 * SW) void stream_kernel(
    const int32_t *__restrict__ offsets, int e_first, const bf16_t *__restrict__ x,
    const int32_t *__restrict__ row_map, int slot_div, const bf16_t *__restrict__ w0s,
    const bf16_t *__restrict__ w1s, int64_t wstride, int N, int K, void *__restrict__ outp) {
    __shared__ __attribute__((aligned(16))) float lds[SW * NT * 256];
    stream_tile<MODE, NT, R>(lds, offsets, e_first, x, row_map, slot_div, w0s, w1s, wstride, N,
                             K, outp);
}

template <int MODE, int NT, int R>
hipError_t launch(const int32_t *offsets, int e_first, int e_count, const bf16_t *x,
                  const int32_t *row_map, int slot_div, const bf16_t *w0, const bf16_t *w1,
                  int64_t wstride, int N, int K, void *out, hipStream_t s) {
    constexpr int COLS = MODE == 0 ? 8 * NT : 16 * NT;
    if (N % COLS || K % 32) return hipErrorInvalidValue;
    stream_kernel<MODE, NT, R><<<(unsigned)(e_count * (N / COLS)), 64 * SW, 0, s>>>(
        offsets, e_first, x, row_map, slot_div, w0, w1, wstride, N, K, out);
    return hipGetLastError();
}

}  // namespace

// Both rules count workgroups per compute unit, two of which are resident;
// every time here is a mean over four placements of the weights in memory.
//
// Gate/up, us, tiled -> streamed.  Every expert has its workgroups, whether it
// has rows or not, and with many experts the empty ones cost more than is
// saved (256 experts of 2048 x 2048, 1 token: 34 -> 47).  A small launch, most
// of it resident at once, gains by the missing fix-up: up to 3 1/4 workgroups
// per unit where a wave's piece of K is whole rounds of its steps in flight or
// K is at most one round (4096 x 3584: 33 -> 28 at 448 workgroups, 46 -> 44 at
// 740; 2048 x 1408: 29 -> 26 at 680), else up to two (5120 x 1536, whose 20
// steps take the time of 24: 27 -> 23 at 200, 37 -> 34 at 450, 59 -> 64 at
// 800).  A larger one gains while the tiled launch leaves units idle (6144 x
// 1344: 62% full 112 -> 105, 94% 96 -> 86; 6144 x 2688, 98%: 61 -> 64), in
// whole rounds of K and, where K is one round and a workgroup soon done, at
// most 16 of them per unit (60 experts of 2048 x 1408, 21 per unit, 6 tokens
// 48 -> 57).
bool stream_gateup_fits(int64_t max_rows, double active, int experts, int H, int I, int grid) {
    constexpr int ROUND = 32 * SW * kGateupSteps, MAX_H = 2 * ROUND;
    const double cus = device_cu_count();
    const double per_cu = experts * (I / 16) / cus, live = active * (I / 16) / cus;
    if (max_rows > kStreamMaxRows || per_cu > 32.0) return false;
    const bool whole = H % ROUND == 0;
    if (live <= (H <= ROUND || (whole && H <= MAX_H) ? 3.25 : 2.0)) return true;
    const int64_t tiles = std::llround(active * ((I + 127) / 128));
    return whole && (H > ROUND || per_cu <= 16.0) && tiled_round_fill(tiles, H, grid) < 0.95;
}

// Down (where the skinny tile does not apply): one workgroup per unit, where
// the tiled launch needs its K split to fill the chip (us, tiled -> streamed:
// 4096 x 3584 22 -> 18 at 256 workgroups, 29 -> 31 at 420), or three where a
// wave's whole piece of K is in flight (2048 x 1408, 60 experts: 22 -> 16 at
// 490, 24 -> 21 at 700).
bool stream_down_fits(int64_t max_rows, double active, int experts, int H, int I) {
    const double cus = device_cu_count();
    const double per_cu = experts * (H / 32) / cus, live = active * (H / 32) / cus;
    return max_rows <= kStreamMaxRows && per_cu <= 32.0 &&
           live <= (I <= 32 * SW * kShortSteps ? 3.0 : 1.0);
}

hipError_t launch_stream_gateup(const moe_dims &d, int e_first, int e_count,
                                const int32_t *offsets, const bf16_t *x, const int32_t *row_map,
                                const bf16_t *w_gate, const bf16_t *w_up, bf16_t *act,
                                hipStream_t s) {
    if (e_count <= 0) return hipSuccess;
    return launch<0, 2, kGateupSteps>(offsets, e_first, e_count, x, row_map, d.top_k, w_gate, w_up,
                           (int64_t)d.inter * d.hidden, d.inter, d.hidden, act, s);
}

hipError_t launch_stream_down(const moe_dims &d, int e_first, int e_count,
                              const int32_t *offsets, const bf16_t *act, const bf16_t *w_down,
                              float *y, hipStream_t s) {
    if (e_count <= 0) return hipSuccess;
    const int64_t wstride = (int64_t)d.hidden * d.inter;
    // a wave's whole piece of K in flight where it is short
    if (d.inter <= 32 * SW * kShortSteps)
        return launch<1, 2, kShortSteps>(offsets, e_first, e_count, act, nullptr, 1, w_down,
                                         nullptr, wstride, d.hidden, d.inter, y, s);
    return launch<1, 2, kLongSteps>(offsets, e_first, e_count, act, nullptr, 1, w_down, nullptr,
                                    wstride, d.hidden, d.inter, y, s);
}

}  // namespace moe
