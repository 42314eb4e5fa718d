// Expert GEMMs of launches of few rows (at most 16 per expert): the GEMM is
// one pass over the weights and the time is the weight stream's.  A workgroup
// owns 16 NT weight rows of one expert over the whole of K; its eight waves
// each take an eighth of K and keep the fragments of R steps of 32 K in
// flight, loaded straight into registers in the MFMA's operand layout (no LDS
// and no barrier while the weights stream).  The waves' partial sums meet in
// LDS, are added in wave order (the same bits on every run) and the epilogue
// is applied there.  Forward, us, tiled GEMM with a K split and its fix-up
// launch -> this: Mixtral 1 token 78.5 -> 69.3, 13 tokens 163.8 -> 153.8;
// DBRX 8 tokens 174 -> 160; 64 experts of 2048 x 1024, 1 token 70 -> 55.
#include <algorithm>
#include <type_traits>

#include "common.h"

namespace moe {
namespace {

constexpr int SW = 8;  // waves of a workgroup (pieces of K)
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

bool stream_fits(int64_t max_rows, int H, int I) {
    // one fragment of rows; 32-bit byte offsets into 16 weight rows
    return max_rows <= kStreamMaxRows && H <= (1 << 20) && I <= (1 << 20);
}

hipError_t launch_stream_gateup(const moe_dims &d, int e_first, int e_count,
                                const int32_t *offsets, const bf16_t *x, const int32_t *row_map,
                                const bf16_t *w_gate, const bf16_t *w_up, bf16_t *act,
                                hipStream_t s) {
    if (e_count <= 0) return hipSuccess;
    return launch<0, 2, 8>(offsets, e_first, e_count, x, row_map, d.top_k, w_gate, w_up,
                           (int64_t)d.inter * d.hidden, d.inter, d.hidden, act, s);
}

hipError_t launch_stream_down(const moe_dims &d, int e_first, int e_count,
                              const int32_t *offsets, const bf16_t *act, const bf16_t *w_down,
                              float *y, hipStream_t s) {
    if (e_count <= 0) return hipSuccess;
    const int64_t wstride = (int64_t)d.hidden * d.inter;
    // a wave's whole piece of K in flight where it is short
    if (d.inter <= 32 * SW * 6)
        return launch<1, 2, 6>(offsets, e_first, e_count, act, nullptr, 1, w_down, nullptr,
                               wstride, d.hidden, d.inter, y, s);
    return launch<1, 2, 12>(offsets, e_first, e_count, act, nullptr, 1, w_down, nullptr, wstride,
                            d.hidden, d.inter, y, s);
}

}  // namespace moe
