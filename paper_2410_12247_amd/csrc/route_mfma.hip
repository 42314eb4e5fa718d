// Matrix-core router: fp32 logits, top-k selection and softmax weights.
//
// v_mfma_f32_16x16x4_f32 adds its four products to each accumulator one at a
// time, in ascending k, each with a single rounding
// (checked bit for bit on gfx950 against fmaf chains, denormal operands and
// results included), so a logit accumulated by it over ascending h carries
// the bits of the sequential fma chain, at twice the rate of scalar fmas
// (143-155 TFLOP/s in a probe; the vector ALU without packed fp32 reaches
// 78.6).  Bound by the matrix cores for many experts, by the x stream for 8;
// moe_route, us, against the scalar kernels it replaced: E = 160, H = 5120:
// 1027 tokens 172 -> 69, 8192 285 -> 108, 16384 421 -> 197, 65536 1478 ->
// 780 (138 TFLOP/s); E = 8, H = 4096, 16384 tokens 33 -> 24.5 (5.5 TB/s of
// x); E = 16, H = 6144, 8192 tokens 50 -> 34; in the forward with 160
// experts, 61 tokens 43 -> 28, 2048 tokens 97 -> 49.
//
// A workgroup is TW x EW waves; wave (tw, ew) owns TT blocks of 16 tokens x
// TE blocks of 16 experts (router rows are the MFMA's rows, tokens its
// columns; lane l of an operand supplies h = 4 step + l / 16 of row l % 16).
// Every wave copies its share of a stage of 64 h (bf16 x rows, fp32 router
// rows) into an LDS ring of NS stages by LDS-DMA; one barrier per stage.
//
// LDS layout: a 16-row block takes 2 KB per 128 bytes of its rows (64 h of
// x, 32 h of the router), in two requests of 8 rows (j = row / 8); 16-byte
// chunk c of row r sits at slot (c / 4) 32 + (r % 8) 4 + ((c % 4) ^ ((r / 4)
// % 4)) of its request, so that four consecutive lanes of a request fetch
// 64 contiguous bytes, the 16 rows x 4 dwords of an operand read fall on 64
// distinct banks, and steps s and s + 4 of a half stage are 512 bytes apart
// (one ds_read2st64 for both).  Operands loaded straight from global memory
// instead (64-byte pieces of 16 rows, transposed between the wave's four
// 16-lane rows by v_permlane swaps) took 296 us at 16384 tokens: the vector
// ALU work takes the matrix core's time, and rows 20 KB apart meet in few
// L2 channels.
#include <algorithm>

#include "dispatch.h"
#include "route_common.h"

namespace moe {
namespace {

constexpr int kSelectThreads = 64 * kRouteSelectTokens;

// Top-k of logits z [T][E] (any E): one wave per token.  DISP (one
// workgroup): its first wave goes on to the dispatch indices.
template <bool DISP>
__global__ __launch_bounds__(kSelectThreads) void route_select_kernel(const float *__restrict__ z,
                                                                  int64_t T, int E, int k,
                                                                  int renorm, int32_t *ids,
                                                                  float *__restrict__ wout,
                                                                  DispatchOut disp) {
    const int64_t t = (int64_t)blockIdx.x * kRouteSelectTokens + (threadIdx.x >> 6);
    if (t < T) select_token(z + t * E, t, E, k, renorm, threadIdx.x & 63, ids, wout);
    if constexpr (DISP) {
        __shared__ int cnt[kMaxExperts], off[kMaxExperts];
        static_assert(kRouteSelectTokens * kMaxTopK <= 64, "one group of slots");
        __syncthreads();  // every token's ids are out
        if (threadIdx.x < 64) dispatch_wave<1>(ids, T * k, k, disp, cnt, off);
    }
}

namespace mfma {

constexpr int HS = 64;     // h per stage
constexpr int BLK = 2048;  // LDS bytes of 16 rows x 128 bytes

template <int TT, int TE, int TW, int EW, int NS>
struct Cfg {
    static constexpr int WAVES = TW * EW;
    static constexpr int TOK = 16 * TT * TW, EP = 16 * TE * EW;
    static constexpr int XB = TT * TW * BLK, WB = TE * EW * 2 * BLK, STAGE = XB + WB;
    // requests per wave and stage: x rows, router rows
    static constexpr int XI = (XB / 1024 + WAVES - 1) / WAVES;
    static constexpr int WI = (WB / 1024 + WAVES - 1) / WAVES;
    static constexpr int PER = XI + WI;
    static constexpr int NM = 8 * TT * TE;  // MFMAs of a half stage
    static constexpr int ZLD = EP + 4;      // logits row (floats)
    static constexpr int ZBYTES = TOK * ZLD * 4;
    static constexpr int LDS = NS * STAGE > ZBYTES ? NS * STAGE : ZBYTES;
    static_assert(NS >= 2 && (NS - 1) * PER <= 63, "vmcnt range");
    static_assert(LDS <= 160 * 1024, "LDS");
};

// acc[m][n]: lane l gets token 16 m + l % 16, experts 16 n + 4 (l / 16) .. + 3
template <int TT, int TE, int TW, int EW, int NS>
__device__ __forceinline__ void logits(char *lds, floatx4 (&acc)[TT][TE],
                                       const bf16_t *__restrict__ x,
                                       const float *__restrict__ wr, int64_t tb, int64_t T,
                                       int eb, int E, int H) {
    using C = Cfg<TT, TE, TW, EW, NS>;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tw = wave / EW, ew = wave % EW;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_void_t *)lds;

    // this wave's requests of a stage, 1 KB each: XI of x rows, WI of router
    // rows (a wave without one of its own repeats the last); request rq of a
    // row block: rows 8 (rq % 2) .., 128-byte piece rq / 2
    const u32x4 xres = buf_rsrc(x + tb * H), wres = buf_rsrc(wr + (int64_t)eb * H);
    const int rr = (lane >> 2) & 7;
    uint32_t xoff[C::XI], xdst[C::XI], woff[C::WI], wdst[C::WI];
#pragma unroll
    for (int i = 0; i < C::XI; ++i) {
        const int rq = min(wave * C::XI + i, C::XB / 1024 - 1);
        const int r = rq * 8 + rr;
        const int c = (lane >> 5) * 4 + ((lane & 3) ^ ((r >> 2) & 3));
        xoff[i] = (uint32_t)min<int64_t>(r, T - 1 - tb) * (uint32_t)(H * 2) + c * 16;
        xdst[i] = lds0 + rq * 1024;
    }
#pragma unroll
    for (int i = 0; i < C::WI; ++i) {
        const int rq = min(wave * C::WI + i, C::WB / 1024 - 1);
        const int r = (rq >> 2) * 16 + (rq & 1) * 8 + rr;
        const int c = (lane >> 5) * 4 + ((lane & 3) ^ ((r >> 2) & 3));
        woff[i] = (uint32_t)min(r, E - 1 - eb) * (uint32_t)(H * 4) + ((rq >> 1) & 1) * 128 + c * 16;
        wdst[i] = lds0 + C::XB + rq * 1024;
    }
    const int nst = H / HS;
    // request i of stage st (clamped) into the slot at LDS byte offset so
    auto request = [&](auto idx, uint32_t st, uint32_t so) {
        constexpr int i = decltype(idx)::value;
        if constexpr (i < C::XI)
            buf16_to_lds(xres, xoff[i], st * (HS * 2), xdst[i] + so);
        else
            buf16_to_lds(wres, woff[i - C::XI], st * (HS * 4), wdst[i - C::XI] + so);
    };

    // Operand addresses by c % 4, one set per SPB slots (the rest of the
    // address is the instruction's offset).  The loop's only vector ALU
    // instructions widen x, once per half stage: an fp32 MFMA and the vector
    // ALU exclude each other, and every switch between them costs about 15
    // cycles (measured, ns per MFMA: 14.2 alone, 20.6 with a v_perm between
    // two, 16.5 with eight v_perm before eight MFMAs).
    constexpr int SPB = 1 + (65536 - 2 * BLK * TE) / C::STAGE, NB = (NS + SPB - 1) / SPB;
    static_assert(TT <= 2 * TE, "a wave's x rows within the offset range");
    const int row = lane & 15, q = lane >> 4;
    uint32_t xb[NB][4], wb[NB][4];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const uint32_t in_blk = (row >> 3) * 1024 + (row & 7) * 64 + ((c ^ (row >> 2)) << 4);
            xb[b][c] = lds0 + b * SPB * C::STAGE + tw * TT * BLK + in_blk;
            wb[b][c] = lds0 + b * SPB * C::STAGE + C::XB + ew * TE * 2 * BLK + in_blk + q * 4;
            asm volatile("" : "+v"(xb[b][c]), "+v"(wb[b][c]));
        }

    // picks bf16 q of two dwords into the high half of a zero dword
    const uint32_t pick = 0x01000C0Cu + (uint32_t)(q * 0x02020000);

    // Operands of a half stage: x chunk c (steps 2 c and 2 c + 1), read
    // first, then the router dwords of steps c and c + 4.
    float wo[2][8][TE];
    u32x4 xo[2][4][TT];
    constexpr int NR = 4 * (TT + TE);
    typedef __attribute__((address_space(3))) const char lds_char_t;
    // read r of half hf of slot S
    auto read = [&](auto slot, auto hf_c, auto r_c) {
        constexpr int S = decltype(slot)::value, hf = decltype(hf_c)::value;
        constexpr int r = decltype(r_c)::value, so = S % SPB * C::STAGE;
        if constexpr (r < 4 * TT) {
            constexpr int c = r / TT, m = r % TT;
            const lds_char_t *p = (const lds_char_t *)(uintptr_t)xb[S / SPB][c];
            xo[hf][c][m] = *(const __attribute__((address_space(3))) u32x4 *)(p + so + m * BLK +
                                                                            hf * 512);
        } else {
            constexpr int c = (r - 4 * TT) / TE, n = (r - 4 * TT) % TE;
            const lds_char_t *p = (const lds_char_t *)(uintptr_t)wb[S / SPB][c];
            constexpr int o = so + (n * 2 + hf) * BLK;
            wo[hf][c][n] = *(const __attribute__((address_space(3))) float *)(p + o);
            wo[hf][c + 4][n] = *(const __attribute__((address_space(3))) float *)(p + o + 512);
        }
    };
    float xf[8][TT];
    auto widen = [&](auto hf_c) {  // the half stage's x, all vector ALU work at once
        constexpr int hf = decltype(hf_c)::value;
#pragma unroll
        for (int s = 0; s < 8; ++s)
#pragma unroll
            for (int m = 0; m < TT; ++m) {
                const u32x4 v = xo[hf][s / 2][m];
                xf[s][m] = __uint_as_float(
                    __builtin_amdgcn_perm(v[2 * (s & 1) + 1], v[2 * (s & 1)], pick));
            }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto mma = [&](auto hf_c, auto i_c) {  // MFMA i of a half stage: step, token, expert block
        constexpr int hf = decltype(hf_c)::value, i = decltype(i_c)::value;
        constexpr int s = i / (TT * TE), m = i / TE % TT, n = i % TE;
        acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(wo[hf][s][n], xf[s][m], acc[m][n], 0, 0,
                                                         0);
    };
    constexpr std::integral_constant<int, 0> h0{};
    constexpr std::integral_constant<int, 1> h1{};

    lane_unroll<0, NS - 1>([&](auto s) {
        lane_unroll<0, C::PER>([&](auto i) {
            request(i, (uint32_t)min(decltype(s)::value, nst - 1),
                    decltype(s)::value * C::STAGE);
        });
    });
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 2) * C::PER) : "memory");
    __builtin_amdgcn_s_barrier();
    lane_unroll<0, NR>([&](auto r) { read(h0, h0, r); });
    auto stage = [&](int st, auto slot) {  // stage st, in slot S
        constexpr int S = decltype(slot)::value;
        constexpr int PREV = (S + NS - 1) % NS, NEXT = (S + 1) % NS;
        const uint32_t fill = (uint32_t)min(st + NS - 1, nst - 1);
        // first half: the second half's operands are read, and the slot that
        // stage st - 1 left is refilled
        widen(h0);
        lane_unroll<0, C::NM>([&](auto i_c) {
            constexpr int i = decltype(i_c)::value;
            mma(h0, i_c);
            lane_unroll<i * NR / C::NM, (i + 1) * NR / C::NM>([&](auto r) { read(slot, h1, r); });
            lane_unroll<i * C::PER / C::NM, (i + 1) * C::PER / C::NM>(
                [&](auto r) { request(r, fill, PREV * C::STAGE); });
            __builtin_amdgcn_sched_barrier(0);
        });
        // second half: once every wave holds the rest of stage st in
        // registers and its share of stage st + 1 has landed, the next
        // stage's first operands are read
        constexpr int BAR = C::NM / 4;
        widen(h1);
        lane_unroll<0, C::NM>([&](auto i_c) {
            constexpr int i = decltype(i_c)::value;
            mma(h1, i_c);
            if constexpr (i == BAR) {
                asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((NS - 2) * C::PER)
                             : "memory");
                __builtin_amdgcn_s_barrier();
            }
            if constexpr (i >= BAR)
                lane_unroll<(i - BAR) * NR / (C::NM - BAR), (i + 1 - BAR) * NR / (C::NM - BAR)>(
                    [&](auto r) { read(std::integral_constant<int, NEXT>{}, h0, r); });
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    for (int st0 = 0; st0 < nst; st0 += NS)
        lane_unroll<0, NS>([&](auto s) {
            if (st0 + decltype(s)::value < nst) stage(st0 + decltype(s)::value, s);
        });
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();  // no request in flight, no wave reads the ring any more
}

}  // namespace mfma

// ZOUT: blockIdx.y picks a group of EW * TE expert blocks and the logits
// (bias added) go to zout [T][E] for route_select_kernel; else the
// workgroup holds every expert, the logits meet in LDS and each wave selects
// its share of the tokens.
template <int TT, int TE, int TW, int EW, int NS, bool ZOUT>
__global__ __launch_bounds__(64 * TW * EW) void route_mfma_kernel(
    const bf16_t *__restrict__ x, const float *__restrict__ wr, const float *__restrict__ bias,
    int64_t T, int H, int E, int k, int renorm, int32_t *__restrict__ ids,
    float *__restrict__ wout, float *__restrict__ zout) {
    using C = mfma::Cfg<TT, TE, TW, EW, NS>;
    __shared__ __attribute__((aligned(1024))) char lds[C::LDS];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tw = wave / EW, ew = wave % EW;
    const int64_t tb = (int64_t)blockIdx.x * C::TOK;
    const int eb = ZOUT ? (int)blockIdx.y * C::EP : 0;
    floatx4 acc[TT][TE];
#pragma unroll
    for (int m = 0; m < TT; ++m)
#pragma unroll
        for (int n = 0; n < TE; ++n) acc[m][n] = floatx4{0.f, 0.f, 0.f, 0.f};
    mfma::logits<TT, TE, TW, EW, NS>(lds, acc, x, wr, tb, T, eb, E, H);

    const int tl = tw * 16 * TT + (lane & 15), el = ew * 16 * TE + 4 * (lane >> 4);
    float *zs = reinterpret_cast<float *>(lds);
#pragma unroll
    for (int n = 0; n < TE; ++n) {
        const int e = eb + el + 16 * n;
        float b[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (bias && e + i < E) b[i] = bias[e + i];
#pragma unroll
        for (int m = 0; m < TT; ++m) {
            floatx4 z = acc[m][n];
            if (bias) {
#pragma unroll
                for (int i = 0; i < 4; ++i) z[i] = z[i] + b[i];
            }
            if constexpr (ZOUT) {
                const int64_t t = tb + tl + 16 * m;
                if (t < T) {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (e + i < E) zout[t * E + e + i] = z[i];
                }
            } else {
                *reinterpret_cast<floatx4 *>(&zs[(tl + 16 * m) * C::ZLD + el + 16 * n]) = z;
            }
        }
    }
    if constexpr (!ZOUT) {
        __syncthreads();
        if constexpr (C::EP == 16) {
            if (lane < 16 * TT) {
                const int i = tw * 16 * TT + lane;
                if (tb + i < T) select_lane<16>(zs + i * C::ZLD, tb + i, E, k, renorm, ids, wout);
            }
        } else {
            constexpr int N = C::TOK / C::WAVES % 4 == 0 ? 4 : 2;  // tokens at a time
            static_assert(C::TOK % (N * C::WAVES) == 0, "tokens per wave");
            for (int i = wave * N; i < C::TOK; i += C::WAVES * N) {
                if (tb + i >= T) break;
                const float *z[N];
                int64_t t[N];
#pragma unroll
                for (int j = 0; j < N; ++j) {
                    z[j] = zs + (i + j) * C::ZLD;
                    t[j] = tb + i + j;
                }
                select_tokens<N>(z, t, T, E, k, renorm, lane, ids, wout);
            }
        }
    }
}

template <int TT, int TE, int TW, int EW, int NS>
hipError_t launch_mfma(const moe_dims &d, const bf16_t *x, const float *wr, const float *bias,
                       int32_t *ids, float *w, hipStream_t s) {
    using C = mfma::Cfg<TT, TE, TW, EW, NS>;
    route_mfma_kernel<TT, TE, TW, EW, NS, false>
        <<<(unsigned)((d.tokens + C::TOK - 1) / C::TOK), 64 * C::WAVES, 0, s>>>(
            x, wr, bias, d.tokens, d.hidden, d.experts, d.top_k, d.renormalize, ids, w, nullptr);
    return hipGetLastError();
}

template <int TT, int TE, int TW, int EW, int NS>
hipError_t launch_mfma_z(const moe_dims &d, const bf16_t *x, const float *wr, const float *bias,
                         int32_t *ids, float *w, float *z, hipStream_t s,
                         const DispatchOut *disp) {
    using C = mfma::Cfg<TT, TE, TW, EW, NS>;
    const dim3 grid((unsigned)((d.tokens + C::TOK - 1) / C::TOK),
                    (unsigned)((d.experts + C::EP - 1) / C::EP));
    route_mfma_kernel<TT, TE, TW, EW, NS, true><<<grid, 64 * C::WAVES, 0, s>>>(
        x, wr, bias, d.tokens, d.hidden, d.experts, d.top_k, d.renormalize, ids, w, z);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_route_select(d, z, ids, w, s, disp);
}

// Matrix-core router for more than 16 experts.  The time of a launch is its
// rounds of one workgroup per compute unit, each about 20 us per tile (16
// tokens x 16 experts of one wave's SIMD) at H = 5120 plus 10 us of start
// and selection (measured at E = 160: 3 tiles 69 us, 5 tiles 113, 10 tiles
// 200-205, 20 tiles 387); the shape with the lowest cost runs.  A shape
// trades operand reads per MFMA (more tiles per wave) and tokens per
// workgroup against compute units left idle.  A tile's time is proportional
// to H and the start is not; the rule keeps the two figures of H = 5120 at
// every width (only the choice of shape depends on them).
constexpr int ring_slots(int stage) { return 3 * stage <= 160 * 1024 ? 3 : 2; }
double mfma_cost(int64_t tokens, int tok, int tiles) {
    const int64_t per_round = (int64_t)tok * device_cu_count();
    return (double)((tokens + per_round - 1) / per_round) * (20.0 * tiles + 10.0);
}
// Tokens of a workgroup (16, 32, 64 or 128; the largest of equal cost) with te
// expert blocks per wave where two waves share the experts; 16 tokens spread
// them over four.
int mfma_tokens(int64_t tokens, int te) {
    const int tiles[4] = {(te + 1) / 2, te, 2 * te, 4 * te};
    int best = 0;
    for (int i = 1; i < 4; ++i)
        if (mfma_cost(tokens, 16 << i, tiles[i]) <= mfma_cost(tokens, 16 << best, tiles[best]))
            best = i;
    return 16 << best;
}
template <int TT, int TE, int TW, int EW>
hipError_t launch_mfma_ring(const moe_dims &d, const bf16_t *x, const float *wr,
                            const float *bias, int32_t *ids, float *w, hipStream_t s) {
    constexpr int STAGE = (TT * TW + 2 * TE * EW) * mfma::BLK;
    return launch_mfma<TT, TE, TW, EW, ring_slots(STAGE)>(d, x, wr, bias, ids, w, s);
}
// TE: expert blocks per wave with the experts over two waves
template <int TE>
hipError_t launch_mfma_te(const moe_dims &d, const bf16_t *x, const float *wr, const float *bias,
                          int32_t *ids, float *w, hipStream_t s) {
    switch (mfma_tokens(d.tokens, TE)) {
        case 128: return launch_mfma_ring<2, TE, 4, 2>(d, x, wr, bias, ids, w, s);
        case 64: return launch_mfma_ring<1, TE, 4, 2>(d, x, wr, bias, ids, w, s);
        case 32: return launch_mfma_ring<1, TE, 2, 2>(d, x, wr, bias, ids, w, s);
        default: return launch_mfma_ring<1, (TE + 1) / 2, 1, 4>(d, x, wr, bias, ids, w, s);
    }
}
// expert blocks, and per wave with the experts over two waves (1 .. 6 or 8)
int expert_blocks(const moe_dims &d) { return (d.experts + 15) / 16; }
int blocks_per_wave(int eb) { return eb > 12 ? 8 : (eb + 1) / 2; }
// waves of one tile each
int64_t tile_waves(const moe_dims &d) { return (d.tokens + 15) / 16 * expert_blocks(d); }
}  // namespace

hipError_t launch_route_select(const moe_dims &d, const float *z, int32_t *ids, float *w,
                               hipStream_t s, const DispatchOut *disp) {
    if (disp)
        route_select_kernel<true><<<1, kSelectThreads, 0, s>>>(
            z, d.tokens, d.experts, d.top_k, d.renormalize, ids, w, *disp);
    else
        route_select_kernel<false>
            <<<(unsigned)((d.tokens + kRouteSelectTokens - 1) / kRouteSelectTokens),
               kSelectThreads, 0, s>>>(z, d.tokens, d.experts, d.top_k, d.renormalize, ids, w,
                                       DispatchOut{});
    return hipGetLastError();
}

// Few tokens: the expert blocks over workgroups of their own (logits through
// the caller's buffer), one tile per wave; a round of a tile per SIMD takes
// 20 us, the selection kernel is in the other 10 (E = 160, us, against the
// experts in one workgroup: 61 tokens 28 against 68, 1027 tokens 31 against
// 69, 2048 tokens 49 against 70).
bool mfma_router_selects_apart(const moe_dims &d, const float *logits) {
    if (d.experts <= 16 || !logits || d.tokens > kRouteLogitsMaxTokens) return false;
    const int eb = expert_blocks(d);
    const int64_t simds = 4 * (int64_t)device_cu_count();
    const double cz = (double)((tile_waves(d) + simds - 1) / simds) * 20.0 + 10.0;
    return cz <= std::min(mfma_cost(d.tokens, 16, (eb + 3) / 4),
                          mfma_cost(d.tokens, 32, blocks_per_wave(eb)));
}

extern "C" int32_t moe_router_shape_for_tests(const moe_dims *d, int32_t *blocks) {
    const int te = blocks_per_wave(expert_blocks(*d)), tok = mfma_tokens(d->tokens, te);
    *blocks = tok == 16 ? (te + 1) / 2 : te;
    return tok;
}

hipError_t launch_mfma_router(const moe_dims &d, const bf16_t *x, const float *wr,
                              const float *bias, int32_t *ids, float *w, float *logits,
                              hipStream_t s, const DispatchOut *disp) {
    if (d.experts <= 16) {
        // one 16 x 16 tile per wave; single-wave workgroups spread up to one
        // tile per compute unit and SIMD better, above that the smaller ring
        // keeps three workgroups per compute unit (Mixtral's 8 experts, us:
        // 1000 tokens 22.3 against 24.8, 16384 tokens 46.3 against 25.9)
        if (d.tokens <= (int64_t)16 * device_cu_count())
            return launch_mfma<1, 1, 1, 1, 8>(d, x, wr, bias, ids, w, s);
        return launch_mfma<1, 1, 4, 1, 4>(d, x, wr, bias, ids, w, s);
    }
    if (mfma_router_selects_apart(d, logits)) {
        if (tile_waves(d) <= 4 * (int64_t)device_cu_count())
            return launch_mfma_z<1, 1, 1, 1, 6>(d, x, wr, bias, ids, w, logits, s, disp);
        return launch_mfma_z<1, 1, 2, 2, 3>(d, x, wr, bias, ids, w, logits, s, disp);
    }
    switch (blocks_per_wave(expert_blocks(d))) {
        case 1: return launch_mfma_te<1>(d, x, wr, bias, ids, w, s);
        case 2: return launch_mfma_te<2>(d, x, wr, bias, ids, w, s);
        case 3: return launch_mfma_te<3>(d, x, wr, bias, ids, w, s);
        case 4: return launch_mfma_te<4>(d, x, wr, bias, ids, w, s);
        case 5: return launch_mfma_te<5>(d, x, wr, bias, ids, w, s);
        case 6: return launch_mfma_te<6>(d, x, wr, bias, ids, w, s);
        default: return launch_mfma_te<8>(d, x, wr, bias, ids, w, s);
    }
}

}  // namespace moe
