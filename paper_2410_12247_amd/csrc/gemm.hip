// Expert GEMMs of the SwiGLU FFN on gfx950 bf16 MFMA (fp32 accumulation).
//
// Two launches per expert group (the paper's Gate, Up and Down GEMMs, with
// the silu activation folded into the first):
//   gate/up : act[r][j] = bf16( silu(g) * u ),  g = Wg[j].x[r], u = Wu[j].x[r]
//   down    : y[r][h]   = Wd[h].act[r]                           (fp32 out)
// Both operands are contiguous along the reduced dimension.  The MFMA is
// fed the WEIGHT rows as its first (row) operand and the TOKEN rows as its
// second (column) operand, so each lane ends up holding four consecutive
// output features of one token row, and for gate/up the matching gate and up
// values sit in the same lane, so SiLU*mul needs no data movement.  The
// outputs leave through LDS as whole row segments (tile_epilogue).
//
// Workgroup tile (the one both schedulers use): 256 weight rows x 320 token
// rows, eight waves in two groups that alternate between MFMAs and memory
// work (the "ping-pong" tile below), built from v_mfma_f32_16x16x32_bf16.
// K advances 32 per stage through four LDS stages filled by LDS-DMA loads,
// so the loads of the next three stages are in flight while a stage is
// multiplied.  16-byte chunks of each LDS row are XOR-swizzled so MFMA
// operand reads hit distinct banks.
//
// Two schedulers share that tile code and its arithmetic (so both give the
// same bits for the same rows):
//   dense : one launch per expert over host-known rows, one tile per
//           workgroup ("DenseGemm").
//   group : one persistent launch over a range of experts whose row counts
//           are read on the device; workgroups walk a tile list spanning
//           all experts ("GroupGemm").
// Both map workgroups to tiles XCD by XCD (the hardware deals workgroups
// round-robin over the 8 XCDs), so the tiles running on one XCD are
// neighbours in (m, n) and share activation and weight rows in its L2.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "lds_dma.h"

namespace moe {
namespace {

constexpr int NXCD = 8;
constexpr int GROUP_N = 8;  // n-tiles per super-column of the tile order

// XOR swizzle of the 16-byte chunk index inside an LDS row, chosen so that
// the 16 rows one MFMA operand read touches fall on distinct banks (LDS
// serves b128 reads eight lanes at a time): 128-byte rows (BK 64) use
// row & 7, 64-byte rows (BK 32) use (row >> 1) & 3.
template <int BK>
__device__ __forceinline__ int swz(int row) {
    return BK == 64 ? (row & 7) : ((row >> 1) & 3);
}

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

struct TileArgs {
    const bf16_t *w0;  // first weight row of the tile (gate rows, or down rows)
    const bf16_t *w1;  // first up row (gate/up only)
    int n_valid;       // weight rows valid from w0 (per half for gate/up)
    const bf16_t *x;   // first token row of the tile, or the token matrix
    const int32_t *rows;  // NULL: rows are contiguous from x; else tile row i
                          // is x row rows[i] / slot_div (the dispatch gather
                          // folded into the operand loads)
    int slot_div;
    int m_valid;       // token rows valid from x
    int K;             // row length of both operands (elements)
    int k0, nks;       // K stages [k0, k0 + nks) of BK elements this call covers
    void *out;         // output element (first token row, first column)
    int64_t ldo;       // output row stride in elements
    // K split: the piece's fp32 accumulators go here instead (NULL: whole K)
    float *part;
};

__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
    __bf16 ha = static_cast<__bf16>(a);
    __bf16 hb = static_cast<__bf16>(b);
    uint16_t ua = __builtin_bit_cast(uint16_t, ha);
    uint16_t ub = __builtin_bit_cast(uint16_t, hb);
    return (uint32_t)ua | ((uint32_t)ub << 16);
}

// silu(g) * u = g * u / (1 + e^-g), with the hardware's exp2 and
// reciprocal (about 1 ulp each; the result is rounded to bf16 next):
// e^-g = 2^(-g log2 e).  An IEEE-rounded reciprocal costs a ten-instruction
// division sequence per value, and the gate/up epilogue evaluates 80 of
// them per lane with every wave of the workgroup in its epilogue at once.
// Large |g| behaves: e^-g -> inf gives 0 (silu -> 0), e^-g -> 0 gives g.
__device__ __forceinline__ float silu_mul(float g, float u) {
    const float e = __builtin_amdgcn_exp2f(g * -1.44269504088896341f);
    return g * __builtin_amdgcn_rcpf(1.0f + e) * u;
}

// ---------------------------------------------------------------------------
// Eight-wave ping-pong variant.  256 (weights) x BM (tokens) output tile,
// eight waves in two groups of four, one wave of each group on every SIMD.
// Each wave owns a 128 x BM/4 accumulator block.  The groups alternate
// between a compute phase (MFMAs on fragments already in registers) and a
// memory phase (its share of the LDS-DMA for stage k+NS-1 and the fragment
// reads of its next stage), separated by workgroup barriers, so every SIMD
// always has one wave issuing MFMAs while the other feeds LDS.  Stage s
// lives in LDS buffer s % NS (NS = 4 stages of 32 K, or 3 of 64 K).
//   group A (waves 0-3, token rows 0..BM/2-1):  compute(k) | mem: frags(k+1), DMA(k+NS-1)
//   group B (waves 4-7, token rows BM/2..BM-1): mem: frags(k), DMA(k+NS-1) | compute(k)
// LDS traffic per MFMA falls as the wave tile grows: BM = 320 (wave tile
// 128 x 80, 40 MFMAs per 13 fragment reads, 160 accumulator registers, four
// 36 KiB stages) is the largest that fits 256 registers and 160 KiB of LDS.
// ---------------------------------------------------------------------------
// K per LDS stage of the ping-pong tile of bm token rows: 64 for the
// 128-row tile (decode-sized launches, bound by the weight stream, read 128
// contiguous bytes of each weight row per stage instead of 64: about 10%
// faster on 64-token decode), 32 for the taller, MFMA-bound tiles
__host__ __device__ constexpr int pp_stage_k(int bm) { return bm == 128 ? 64 : 32; }
// buffer resource word 3 for raw (untyped, unswizzled) access on gfx9 parts
constexpr int kBufferFlags = 0x00020000;

template <int MODE, int BM_>
struct PPCfg {
    static constexpr int BN = 256, BM = BM_, WAVES = 8;
    static constexpr int BK = pp_stage_k(BM_);
    static constexpr int NS = BK == 64 ? 3 : 4;  // ring within 144 KB of LDS
    static constexpr int KH = BK / 32;  // MFMA K-steps per stage
    static constexpr int WTN = 128, WTM = BM / 4;  // wave tile (weights x tokens)
    static constexpr int TN = WTN / 16, TM = WTM / 16;
    static_assert(WTM % 16 == 0, "token rows per wave: whole 16-row fragments");
    static constexpr int CPR = BK / 8;          // 16-byte chunks per LDS row
    static constexpr int RPI = 64 / CPR;        // rows one LDS-DMA instruction fills
    static constexpr int W_INSTR = BN / 8 / RPI;
    // token rows: BM / RPI instructions, group A's waves take X_INSTR_A
    // each, group B's the rest
    static constexpr int X_TOTAL = BM / RPI;
    static constexpr int X_INSTR_A = (X_TOTAL + 7) / 8;
    static constexpr int X_INSTR_B = (X_TOTAL - 4 * X_INSTR_A) / 4;
    static_assert(4 * X_INSTR_A + 4 * X_INSTR_B == X_TOTAL, "token rows split over waves");
    static constexpr int LPS_A = W_INSTR + X_INSTR_A;  // DMA instructions per wave per stage
    static constexpr int LPS_B = W_INSTR + X_INSTR_B;
    static constexpr int STAGE_W = BN * BK, STAGE_X = BM * BK, STAGE = STAGE_W + STAGE_X;
    // the epilogue's scratch (one 16 x 64 block of outputs per wave, rows
    // padded by 16 bytes) starts at the ring's last buffer: the next tile's
    // first stages land in the others meanwhile
    static constexpr int SCRATCH_ROW = (MODE == 0 ? 64 * 2 : 64 * 4) + 16;  // bytes
    static constexpr int SCRATCH_WAVE = 16 * SCRATCH_ROW;
    static constexpr int SCRATCH = (NS - 1) * STAGE * 2;  // byte offset
    static constexpr int LDS_BYTES = NS * STAGE * 2 > SCRATCH + 8 * SCRATCH_WAVE
                                         ? NS * STAGE * 2
                                         : SCRATCH + 8 * SCRATCH_WAVE;
    static constexpr int LDS_ELEMS = LDS_BYTES / 2;
    static_assert(LDS_BYTES <= 144 * 1024, "ring within 144 KB of LDS");
    // output stores of a whole tile per wave (fixed, whatever rows are valid)
    static constexpr int STORES = MODE == 0 ? 2 * TM : 8 * TM;
    static_assert(NS >= 3 && (NS - 2) * LPS_A + STORES <= 63, "vmcnt range");
    static constexpr int BNOUT = MODE == 0 ? BN / 2 : BN;
    static constexpr int PART_ELEMS = BN * BM;  // fp32 accumulators of one tile
    static constexpr int PART_BYTES = PART_ELEMS * 4;
    static constexpr int WAVE_BYTES = TN * TM * 1024;  // one wave's block of them
};

// Epilogue of a ping-pong tile (or of the sum of its K pieces), one 16x16
// output fragment at a time; the lane holds output columns col..col+3 of
// token row `row`.  gate/up: fragment (p, m) of wave (wn, wm) from the
// matching gate and up accumulators, stored as bf16(silu(g) * u).
template <class C>
__device__ __forceinline__ void store_gateup(const floatx4 &g, const floatx4 &u, int p, int m,
                                             int wn, int wm, int lane, bf16_t *out, int64_t ldo,
                                             int m_valid, int n_valid) {
    const int row = wm * C::WTM + m * 16 + (lane & 15);
    const int col = wn * (C::WTN / 2) + p * 16 + (lane >> 4) * 4;
    if (row < m_valid && col < n_valid) {
        uint2 v;
        v.x = pack_bf16x2(silu_mul(g[0], u[0]), silu_mul(g[1], u[1]));
        v.y = pack_bf16x2(silu_mul(g[2], u[2]), silu_mul(g[3], u[3]));
        *reinterpret_cast<uint2 *>(out + row * ldo + col) = v;
    }
}
// down: fragment (t, m) of wave (wn, wm), the fp32 values.
template <class C>
__device__ __forceinline__ void store_down(const floatx4 &v, int t, int m, int wn, int wm,
                                           int lane, float *out, int64_t ldo, int m_valid,
                                           int n_valid) {
    const int row = wm * C::WTM + m * 16 + (lane & 15);
    const int col = wn * C::WTN + t * 16 + (lane >> 4) * 4;
    if (row < m_valid && col < n_valid) *reinterpret_cast<floatx4 *>(out + row * ldo + col) = v;
}

// K split: the piece stores its accumulators (each wave its own block,
// one 1 KiB store per fragment, through a buffer resource so the
// fragment offsets are scalars); split_fixup_kernel adds the pieces and
// runs the epilogue
template <class C>
__device__ __forceinline__ void tile_store_piece(const floatx4 (&acc)[C::TN][C::TM], int wave,
                                                 const TileArgs &a) {
    const int wm = wave >> 1, lane = threadIdx.x & 63;
    const __amdgpu_buffer_rsrc_t pres =
        __builtin_amdgcn_make_buffer_rsrc(a.part, 0, -1, kBufferFlags);
    const int loff = lane * 16;
    // fragment rows wholly past the valid edge are never stored, so
    // their partial sums are neither written nor read back (decode-sized
    // tiles hold one or two valid rows of 320)
#pragma unroll
    for (int m = 0; m < C::TM; ++m) {
        if (wm * C::WTM + m * 16 >= a.m_valid) break;
#pragma unroll
        for (int t = 0; t < C::TN; ++t)
            __builtin_amdgcn_raw_buffer_store_b128(
                __builtin_bit_cast(u32x4, acc[t][m]), pres, loff,
                wave * C::WAVE_BYTES + (t * C::TM + m) * 1024, 0);
    }
}

// Outputs of a whole tile.  A fragment leaves the MFMA with four columns of
// 16 rows per lane; stored as it is, a request would scatter 16-byte (down)
// or 8-byte (gate/up) pieces over 16 rows, each its own trip to the L2.  So
// 16 x 64 blocks go through the wave's LDS scratch and leave as whole row
// segments (256 or 128 bytes).  With another tile's stages requested before
// (more), every store is issued, whatever rows are valid, since the waits
// count them: lanes without a valid row get an offset past the resource's
// range, which drops them; the workgroup's last tile leaves its empty blocks
// out (dense FFN of 1 row x 4096 x 2048: 53.8 -> 52.2 us).  Down GEMM us,
// scattered stores after the K loop -> this, with the next tile's first
// stages requested before (PPTile): DBRX 8192 tokens 632 -> 576, Mixtral
// 16384 tokens 864 -> 831; dense FFN of 3001 rows x 5120 x 3072 229 -> 217;
// non-temporal stores: within 1%.
template <int MODE, class C>
__device__ __forceinline__ void tile_epilogue(const floatx4 (&acc)[C::TN][C::TM], bf16_t *smem,
                                              int wave, const TileArgs &a, bool more) {
    const int wn = wave & 1, wm = wave >> 1;
    // (an opaque lane index: addresses computed from it are not hoisted
    // over the K loop, which has no register to spare for them)
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));
    char *sc = reinterpret_cast<char *>(smem) + C::SCRATCH + wave * C::SCRATCH_WAVE;
    constexpr uint32_t RANGE = 0xFFFFFFF0u, DROP = 0xFFFFFFF8u;
    const __amdgpu_buffer_rsrc_t ores =
        __builtin_amdgcn_make_buffer_rsrc(a.out, 0, (int)RANGE, kBufferFlags);
    const int row_w = (lane & 15) * C::SCRATCH_ROW;  // write: row lane % 16
    if (MODE == 0) {
        const int rr = lane >> 3, rc = lane & 7;  // read: 8 rows x 8 chunks of 16 bytes
        const uint32_t colb = (uint32_t)(wn * 64 + rc * 8) * 2u;
        const bool cols = wn * 64 < a.n_valid;
#pragma unroll
        for (int m = 0; m < C::TM; ++m) {
            if (!more && wm * C::WTM + m * 16 >= a.m_valid) break;
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                const floatx4 g = acc[p][m], u = acc[p + 4][m];
                uint2 v;
                v.x = pack_bf16x2(silu_mul(g[0], u[0]), silu_mul(g[1], u[1]));
                v.y = pack_bf16x2(silu_mul(g[2], u[2]), silu_mul(g[3], u[3]));
                *reinterpret_cast<uint2 *>(sc + row_w + p * 32 + (lane >> 4) * 8) = v;
            }
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const u32x4 v = *reinterpret_cast<const u32x4 *>(
                    sc + (i * 8 + rr) * C::SCRATCH_ROW + rc * 16);
                const int row = wm * C::WTM + m * 16 + i * 8 + rr;
                const uint32_t off = cols && row < a.m_valid
                                         ? (uint32_t)(row * a.ldo) * 2u + colb
                                         : DROP;
                __builtin_amdgcn_raw_buffer_store_b128(v, ores, off, 0, 0);
            }
            __builtin_amdgcn_wave_barrier();
        }
    } else {
        const int rr = lane >> 4, rc = lane & 15;  // read: 4 rows x 16 chunks
#pragma unroll
        for (int m = 0; m < C::TM; ++m) {
            if (!more && wm * C::WTM + m * 16 >= a.m_valid) break;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const bool cols = wn * 128 + h * 64 < a.n_valid;
                const uint32_t colb = (uint32_t)(wn * 128 + h * 64 + rc * 4) * 4u;
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    *reinterpret_cast<floatx4 *>(sc + row_w + t * 64 + (lane >> 4) * 16) =
                        acc[h * 4 + t][m];
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const u32x4 v = *reinterpret_cast<const u32x4 *>(
                        sc + (i * 4 + rr) * C::SCRATCH_ROW + rc * 16);
                    const int row = wm * C::WTM + m * 16 + i * 4 + rr;
                    const uint32_t off = cols && row < a.m_valid
                                             ? (uint32_t)(row * a.ldo) * 4u + colb
                                             : DROP;
                    __builtin_amdgcn_raw_buffer_store_b128(v, ores, off, 0, 0);
                }
                __builtin_amdgcn_wave_barrier();
            }
        }
    }
}

// A workgroup's walk over its tiles: bind (operand addresses of a tile),
// prologue (its first NS - 1 stages requested), kloop, epilogue.  The next
// tile is bound and its prologue issued before the current tile's epilogue,
// so its first stages land while the outputs are written, and the waits of
// its first stages leave the stores, which are younger, in flight (loads and
// stores share one in-order vmcnt).
//
// SINGLE: the tile is the workgroup's only one, so nothing is sent behind its
// last stages: the loop then requests a whole share in every stage (the last
// stage again past the end) and waits for the same count, without a tail.  In
// launches of few rows, bound by how fast requests go out, its fragment
// reads also go before the requests; with many tiles per workgroup the
// requests go first.  Dense FFN us, one workgroup per tile, loop with tail
// and requests first -> this: 4096 x 2048, 1 row 55.3 -> 53.8; 3008 x 3008,
// 200 rows 73.8 -> 68.7; 6144 x 1024, 700 rows 91.2 -> 86.3; 320-row tiles
// the other way round: 5120 x 3072, 3001 rows 228 against 232.
template <int MODE, int BM_, bool SINGLE>
struct PPTile {
    using C = PPCfg<MODE, BM_>;
    static constexpr int BK = C::BK, NS = C::NS;
    bf16_t *smem;
    uint32_t lds0;
    int lane, wave, grp, wn, wm;
    int k0, nk;       // K stages of the tile
    bool active;
    u32x4 wres, xres;  // buffer resources over the weight rows and the token rows
    uint32_t woff[C::W_INSTR], xoff[C::X_INSTR_A];
    floatx4 acc[C::TN][C::TM];

    __device__ __forceinline__ explicit PPTile(bf16_t *sm) : smem(sm) {
        lds0 = (uint32_t)(uintptr_t)(lds_void_t *)sm;
        lane = threadIdx.x & 63;
        wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        grp = wave >> 2;  // 0 = A, 1 = B
        wn = wave & 1;    // weight half
        wm = wave >> 1;   // token block
    }

    // first token row of this wave's LDS-DMA share
    __device__ __forceinline__ int x_row0() const {
        return grp == 0 ? wave * C::X_INSTR_A * C::RPI
                        : 4 * C::X_INSTR_A * C::RPI + (wave - 4) * C::X_INSTR_B * C::RPI;
    }

    // LDS-DMA share of this wave: BN/8 weight rows and a slice of the token
    // rows (group A's waves taking the larger slices when they do not divide
    // evenly); a 32-bit per-lane row offset, the stage's k offset is scalar
    __device__ __forceinline__ void bind(const TileArgs &a) {
        k0 = a.k0;
        nk = a.nks;
        // a wave whose token rows or weight rows all lie past the valid edge
        // of a partial tile skips its MFMAs (its outputs are never stored);
        // it still takes its share of the loads and barriers
        active = wm * C::WTM < a.m_valid &&
                 (MODE == 0 ? wn * (C::WTN / 2) : wn * C::WTN) < a.n_valid;
        int lane = threadIdx.x & 63;  // opaque, as in the epilogue
        asm volatile("" : "+v"(lane));
        const int drow = lane / C::CPR;
        const int dchunk = ((lane % C::CPR) ^ swz<BK>(drow)) * 8;
        int wrow0;
        if (MODE == 0) {  // waves 0..3 copy gate rows, 4..7 up rows
            wres = buf_rsrc(wave >= 4 ? a.w1 : a.w0);
            wrow0 = (wave & 3) * (C::BN / 8);
        } else {
            wres = buf_rsrc(a.w0);
            wrow0 = wave * (C::BN / 8);
        }
        xres = buf_rsrc(a.x);
#pragma unroll
        for (int i = 0; i < C::W_INSTR; ++i) {
            const int r = min(wrow0 + i * C::RPI + drow, a.n_valid - 1);
            woff[i] = (uint32_t)(r * a.K + dchunk) * 2u;
        }
#pragma unroll
        for (int i = 0; i < C::X_INSTR_A; ++i) {
            const int r = min(x_row0() + i * C::RPI + drow, a.m_valid - 1);
            const int64_t src = a.rows ? (int64_t)(a.rows[r] / a.slot_div) : r;
            xoff[i] = (uint32_t)((src * a.K + dchunk) * 2);
        }
    }

    // this wave's share of stage ks (nx: its token-row instruction count,
    // the group's) into the stage's buffer
    template <class NX>
    __device__ __forceinline__ void issue(int ks, NX) {
        const uint32_t sb = lds0 + (uint32_t)((ks % NS) * C::STAGE * 2);
        const uint32_t kb = (uint32_t)((k0 + (SINGLE ? min(ks, nk - 1) : ks)) * BK * 2);
#pragma unroll
        for (int i = 0; i < C::W_INSTR; ++i)
            buf16_to_lds(wres, woff[i], kb, sb + (wave * (C::BN / 8) + i * C::RPI) * BK * 2);
#pragma unroll
        for (int i = 0; i < NX::value; ++i)
            buf16_to_lds(xres, xoff[i], kb,
                         sb + C::STAGE_W * 2 + (x_row0() + i * C::RPI) * BK * 2);
    }
    using nxa = std::integral_constant<int, C::X_INSTR_A>;
    using nxb = std::integral_constant<int, C::X_INSTR_B>;

    // stages 0 .. NS-2 requested (a shorter tile repeats its last stage)
    __device__ __forceinline__ void prologue() {
#pragma unroll
        for (int s = 0; s < NS - 1; ++s) {
            // (the copy of stage nk-1 goes to a buffer nothing reads)
            const int back = SINGLE ? 0 : max(s - (nk - 1), 0);
            k0 -= back;
            if (grp == 0) issue(s, nxa{}); else issue(s, nxb{});
            k0 += back;
        }
    }

    // What this wave sent after the prologue's requests.
    enum After { NOTHING, STORES, PIECE };

    // The K loop; every wave leaves it with the ring free and no request in
    // flight.
    __device__ __forceinline__ void kloop(After after) {
#pragma unroll
        for (int t = 0; t < C::TN; ++t)
#pragma unroll
            for (int m = 0; m < C::TM; ++m) acc[t][m] = floatx4{0.f, 0.f, 0.f, 0.f};
        // stage 0 landed (a piece's stores vary in number: everything landed)
        if (after == PIECE)
            wait_vmcnt<0>();
        else if (after == STORES && grp == 0)
            wait_vmcnt<(NS - 2) * C::LPS_A + C::STORES>();
        else if (after == STORES)
            wait_vmcnt<(NS - 2) * C::LPS_B + C::STORES>();
        else if (grp == 0)
            wait_vmcnt<(NS - 2) * C::LPS_A>();
        else
            wait_vmcnt<(NS - 2) * C::LPS_B>();
        __builtin_amdgcn_s_barrier();
        // the two groups' loops, with or without the MFMAs; each is straight
        // code (no branch around the MFMA block inside the loop)
        using on = std::integral_constant<bool, true>;
        using off = std::integral_constant<bool, false>;
        const bool stored = after == STORES;
        if (grp == 0) {
            if (active) loop_a(stored, on{}); else loop_a(stored, off{});
        } else {
            if (active) loop_b(stored, on{}); else loop_b(stored, off{});
        }
        if (SINGLE) {  // the repeated requests
            wait_vmcnt<0>();
            __builtin_amdgcn_s_barrier();
        }
    }

    // fragments of this wave: the chunk holding K 32 h + 8 (lane / 16) .. + 7
    // of a row, K-step h
    struct Frags {
        bf16x8 a[C::KH][C::TN], b[C::KH][C::TM];
    };
    __device__ __forceinline__ void load_frags(Frags &f, int ks) {
        const bf16_t *sw = smem + (ks % NS) * C::STAGE;
        const bf16_t *sx = sw + C::STAGE_W;
        const int lrow = lane & 15;
#pragma unroll
        for (int h = 0; h < C::KH; ++h) {
            const int chunk = ((h * 4 + (lane >> 4)) ^ swz<BK>(lrow)) * 8;
#pragma unroll
            for (int t = 0; t < C::TN; ++t) {
                const int arow = MODE == 0 ? (t < C::TN / 2
                                                  ? wn * (C::WTN / 2) + t * 16
                                                  : C::BN / 2 + wn * (C::WTN / 2) +
                                                        (t - C::TN / 2) * 16)
                                           : wn * C::WTN + t * 16;
                f.a[h][t] = *reinterpret_cast<const bf16x8 *>(sw + (arow + lrow) * BK + chunk);
            }
#pragma unroll
            for (int m = 0; m < C::TM; ++m)
                f.b[h][m] = *reinterpret_cast<const bf16x8 *>(
                    sx + (wm * C::WTM + m * 16 + lrow) * BK + chunk);
        }
    }
    __device__ __forceinline__ void mfmas(const Frags &f) {  // K-steps in ascending order
#pragma unroll
        for (int h = 0; h < C::KH; ++h)
#pragma unroll
            for (int m = 0; m < C::TM; ++m)
#pragma unroll
                for (int t = 0; t < C::TN; ++t)
                    acc[t][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.a[h][t], f.b[h][m],
                                                                        acc[t][m], 0, 0, 0);
    }

    // Both loops: the stages that send a request run without a branch, the
    // last ones in a loop of their own (branches around request and wait in
    // one loop: 85 ns per 64-K stage, 128-row tiles).
    template <class W>
    __device__ __forceinline__ void loop_a(bool stored, W) {
        Frags f;
        load_frags(f, 0);
        auto compute = [&] {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_setprio(1);
            if constexpr (W::value) mfmas(f);
            __builtin_amdgcn_s_setprio(0);
        };
        // compute phase: stage k; then stage k+1 landed before the barrier:
        // this wave's requests for stages k+2 .. k+NS-2 (and, older than
        // those from the loop itself, the previous tile's stores) may stay in
        // flight.  Memory phase: this wave's share of stage k+NS-1, fragments
        // of stage k+1 (stale but in bounds past the end).
        int k = 0;
        for (; SINGLE ? k < nk : k + NS - 1 < nk; ++k) {
            compute();
            if (!SINGLE && stored && k <= NS - 3)
                wait_vmcnt<(NS - 3) * C::LPS_A + C::STORES>();
            else
                wait_vmcnt<(NS - 3) * C::LPS_A>();
            __builtin_amdgcn_s_barrier();
            if (!SINGLE) issue(k + NS - 1, nxa{});
            load_frags(f, k + 1);
            if (SINGLE) issue(k + NS - 1, nxa{});
            __builtin_amdgcn_s_barrier();
        }
        if (SINGLE) return;
        for (; k < nk; ++k) {
            compute();
            if (stored && k <= NS - 3 && k + NS - 1 <= nk)
                wait_vmcnt<(NS - 3) * C::LPS_A + C::STORES>();
            else if (k + NS - 1 <= nk)
                wait_vmcnt<(NS - 3) * C::LPS_A>();
            else
                wait_vmcnt<0>();
            __builtin_amdgcn_s_barrier();
            load_frags(f, k + 1);
            __builtin_amdgcn_s_barrier();
        }
    }
    template <class W>
    __device__ __forceinline__ void loop_b(bool stored, W) {
        Frags f;
        auto compute = [&] {
            __builtin_amdgcn_s_barrier();
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_setprio(1);
            if constexpr (W::value) mfmas(f);
            __builtin_amdgcn_s_setprio(0);
            __builtin_amdgcn_s_barrier();
        };
        // memory phase: this wave's share of stage k+NS-1, fragments of stage
        // k; then stage k+1 landed: this wave's requests for stages k+2 ..
        // k+NS-1 (the last just issued) may stay in flight.  Compute phase:
        // stage k.
        int k = 0;
        for (; SINGLE ? k < nk : k + NS <= nk; ++k) {
            if (!SINGLE) issue(k + NS - 1, nxb{});
            load_frags(f, k);
            if (SINGLE) issue(k + NS - 1, nxb{});
            if (!SINGLE && stored && k <= NS - 3)
                wait_vmcnt<(NS - 2) * C::LPS_B + C::STORES>();
            else
                wait_vmcnt<(NS - 2) * C::LPS_B>();
            compute();
        }
        if (SINGLE) return;
        for (; k < nk; ++k) {
            load_frags(f, k);
            if (NS > 3 && k + NS == nk + 1 && k > NS - 3)
                wait_vmcnt<(NS - 3) * C::LPS_B>();
            else
                wait_vmcnt<0>();
            compute();
        }
    }

    __device__ __forceinline__ void store_piece(const TileArgs &a) {
        tile_store_piece<C>(acc, wave, a);
    }
    __device__ __forceinline__ void epilogue(const TileArgs &a, bool more) {
        tile_epilogue<MODE, C>(acc, smem, wave, a, more);
    }
};

// Tile order inside one expert: super-columns of GROUP_N n-tiles, walked
// row by row, so consecutive tiles share token rows and weight rows.
__device__ __forceinline__ void decode_tile(int tau, int MT, int NT, int &mt, int &nt) {
    const int per_sc = GROUP_N * MT;
    const int sc = tau / per_sc;
    const int r = tau - sc * per_sc;
    const int width = min(GROUP_N, NT - sc * GROUP_N);
    mt = r / width;
    nt = sc * GROUP_N + (r - mt * width);
}

// Tile policy shared by the two schedulers.
template <int MODE, int BM_>
struct PingPong {
    using C = PPCfg<MODE, BM_>;  // also read by split_fixup_kernel
    template <bool SINGLE> using Tile = PPTile<MODE, BM_, SINGLE>;
    static constexpr int THREADS = 64 * C::WAVES;
    static constexpr int BM = C::BM;
    static constexpr int BNOUT = C::BNOUT;
    static constexpr int LDS_ELEMS = C::LDS_ELEMS;
    static constexpr int KSTEP = C::BK;
    static constexpr int PART_ELEMS = C::PART_ELEMS;
};

template <int MODE, class TP>
__global__ __launch_bounds__(TP::THREADS) void dense_kernel(const bf16_t *__restrict__ x,
                                                            int64_t rows, const bf16_t *w0,
                                                            const bf16_t *w1, int N, int K,
                                                            void *out, int64_t ldo, int MT,
                                                            int NT) {
    constexpr int BM = TP::BM;
    __shared__ __attribute__((aligned(16))) bf16_t smem[TP::LDS_ELEMS];
    const int per = gridDim.x / NXCD;
    const int tau = (blockIdx.x % NXCD) * per + blockIdx.x / NXCD;
    if (tau >= MT * NT) return;
    int mt, nt;
    decode_tile(tau, MT, NT, mt, nt);
    TileArgs a;
    const int64_t n0 = (int64_t)nt * TP::BNOUT;
    const int64_t m0 = (int64_t)mt * BM;
    a.w0 = w0 + n0 * K;
    a.w1 = MODE == 0 ? w1 + n0 * K : nullptr;
    a.n_valid = (int)(N - n0);
    a.x = x + m0 * K;
    a.rows = nullptr;
    a.slot_div = 1;
    a.m_valid = (int)min<int64_t>(BM, rows - m0);
    a.K = K;
    a.k0 = 0;
    a.nks = K / TP::KSTEP;
    a.ldo = ldo;
    a.part = nullptr;
    if (MODE == 0)
        a.out = reinterpret_cast<bf16_t *>(out) + m0 * ldo + n0;
    else
        a.out = reinterpret_cast<float *>(out) + m0 * ldo + n0;
    using Tile = typename TP::template Tile<TP::BM == 128>;
    Tile tile(smem);
    tile.bind(a);
    tile.prologue();
    tile.kloop(Tile::NOTHING);
    tile.epilogue(a, false);
}

template <int MODE, class TP>
__global__ __launch_bounds__(TP::THREADS) void group_kernel(
    const int32_t *__restrict__ offsets, int e_first, int e_count, const bf16_t *__restrict__ x,
    const int32_t *__restrict__ row_map, int slot_div, const bf16_t *w0s, const bf16_t *w1s,
    int64_t wstride, int N, int K, void *out, int64_t ldo, float *__restrict__ parts,
    int32_t *__restrict__ split_meta, int rows_one) {
    constexpr int BM = TP::BM;
    // one LDS object (stage buffers, then the per-expert offsets and tile
    // prefix sums): the compiler then does not make fragment reads wait for
    // the LDS-DMA in flight
    __shared__ __attribute__((aligned(16))) bf16_t smem[TP::LDS_ELEMS + 4 * (kMaxExperts + 1)];
    int *s_off = reinterpret_cast<int *>(smem + TP::LDS_ELEMS);
    int *s_pre = s_off + (kMaxExperts + 1);
    const int tid = threadIdx.x;
    const int NT = (N + TP::BNOUT - 1) / TP::BNOUT;

    // offsets NULL: one expert of rows_one rows (known on the host)
    for (int i = tid; i <= e_count; i += TP::THREADS)
        s_off[i] = offsets ? offsets[e_first + i] : (i == 0 ? 0 : rows_one);
    __syncthreads();
    // tiles per expert, then an inclusive scan (Hillis-Steele over <= 256)
    int mine = 0;
    if (tid < e_count) mine = ((s_off[tid + 1] - s_off[tid] + BM - 1) / BM) * NT;
    if (tid < kMaxExperts) s_pre[tid + 1] = mine;
    if (tid == 0) s_pre[0] = 0;
    __syncthreads();
    for (int d = 1; d < kMaxExperts; d <<= 1) {
        int v = 0;
        if (tid < kMaxExperts && tid >= d) v = s_pre[tid + 1 - d];
        __syncthreads();
        if (tid < kMaxExperts) s_pre[tid + 1] += v;
        __syncthreads();
    }
    const int total = __builtin_amdgcn_readfirstlane(s_pre[e_count]);

    const int G = gridDim.x;  // multiple of NXCD
    const int slot = (blockIdx.x % NXCD) * (G / NXCD) + blockIdx.x / NXCD;
    const int nk = K / TP::KSTEP;
    // Tiles [0, full) fill whole rounds of the grid.  The rem < G tiles left
    // would occupy rem workgroups for one more tile time while the others
    // idle.  With a split buffer the tail is cut along K:
    //  - rem <= G/2: each tail tile j = tau - full into S equal pieces
    //    (slots [S*j, S*j + S));
    //  - a launch that is one partial round of more than G/2 tiles (full ==
    //    0): its W = rem * nk K stages, the tail tiles laid end to end, are
    //    spread evenly over P <= G units (stream-K): unit u takes stages
    //    [u*W/P, (u+1)*W/P), so it ends one tile and starts the next, and its
    //    segment of tile j goes to slot u + j (unique: a unit that reaches
    //    into tile j + 1 is the last of tile j).  Only for tiles of 192 or
    //    more token rows (their MFMA work, done for every row of the tile,
    //    bounds them; a round of 128-row tiles is bound by the weight
    //    stream, which fewer workgroups already saturate), at most half
    //    full on average (each piece writes and the fixup re-reads the
    //    partial sums of the valid rows: for fuller tiles that traffic
    //    outweighs the shorter round), and when the round gets at least a
    //    quarter shorter.
    // The pieces store fp32 partial sums; split_fixup_kernel, launched next,
    // adds each tile's pieces in K order and writes the outputs.
    // split_meta: [0] tail tiles cut (0: none), [1] S (0: stream-K), [2] P,
    // [3] nk, then per tail tile its first output row, first output column
    // and valid rows and columns.
    const int full = total - total % G;
    const int rem = total - full;
    const int64_t W = (int64_t)rem * nk;
    int S = 1, P = 0;
    if (parts != nullptr && rem > 0 && rem <= kSplitMaxTail) {
        if (full == 0 && 2 * rem > G && BM >= 192) {
            // mean valid rows per tile: all rows over the m-tiles
            const int64_t rows_all =
                __builtin_amdgcn_readfirstlane(s_off[e_count] - s_off[0]);
            if (2 * rows_all * NT <= (int64_t)BM * total) {
                P = (int)min<int64_t>(min(G, kSplitSlots - rem), W / kSplitMinStagesAlone);
                if (4 * rem > 3 * P) P = 0;
            }
        } else {
            S = min(min(kSplitMaxPieces, G / rem),
                    min(nk / (full == 0 ? kSplitMinStagesAlone : kSplitMinStages),
                        kSplitSlots / rem));
        }
    }
    if (S < 2) S = 1;
    if (split_meta != nullptr && slot == 0 && tid == 0) {
        split_meta[0] = S > 1 || P > 0 ? rem : 0;
        split_meta[1] = P > 0 ? 0 : S;
        split_meta[2] = P;
        split_meta[3] = nk;
    }

    // tile tau over K stages [k0, k0 + nks); part: the slot of its partial
    // sums (NULL: the whole K range, outputs written); j >= 0: the tail tile
    // whose record this call writes (the call that starts at stage 0)
    auto tile_args = [&](int tau, int k0, int nks, float *part, int j) {
        // expert: last e with s_pre[e] <= tau (LDS values as scalars: the
        // tile's addresses then stay out of the vector registers)
        auto lds = [](const int &v) { return __builtin_amdgcn_readfirstlane(v); };
        int lo = 0, hi = e_count - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (lds(s_pre[mid]) <= tau) lo = mid; else hi = mid - 1;
        }
        const int e = lo;
        const int row0 = lds(s_off[e]);
        const int cnt = lds(s_off[e + 1]) - row0;
        const int MT = (cnt + BM - 1) / BM;
        int mt, nt;
        decode_tile(tau - lds(s_pre[e]), MT, NT, mt, nt);
        const int64_t n0 = (int64_t)nt * TP::BNOUT;
        const int64_t r0 = (int64_t)row0 + (int64_t)mt * BM;
        TileArgs a;
        const int64_t woffe = (int64_t)(e_first + e) * wstride;
        a.w0 = w0s + woffe + n0 * K;
        a.w1 = MODE == 0 ? w1s + woffe + n0 * K : nullptr;
        a.n_valid = (int)(N - n0);
        a.x = row_map ? x : x + r0 * K;
        a.rows = row_map ? row_map + r0 : nullptr;
        a.slot_div = slot_div;
        a.m_valid = min(BM, cnt - mt * BM);
        a.K = K;
        a.k0 = k0;
        a.nks = nks;
        a.ldo = ldo;
        if (MODE == 0)
            a.out = reinterpret_cast<bf16_t *>(out) + r0 * ldo + n0;
        else
            a.out = reinterpret_cast<float *>(out) + r0 * ldo + n0;
        a.part = part;
        if (j >= 0 && tid == 0) {
            int32_t *md = split_meta + 4 + 4 * j;
            md[0] = (int32_t)r0;
            md[1] = (int32_t)n0;
            md[2] = a.m_valid;
            md[3] = a.n_valid;
        }
        return a;
    };
    // The workgroup's work, in order: `u` counts its whole tiles and equal
    // pieces (slot, slot + G, ..: at most one piece, the last); in the
    // stream-K form the stages [g, g1) of its unit, one tile's segment at a
    // time.
    const int end = S > 1 ? full : total;
    const int units = P > 0 ? 0 : S > 1 ? full + rem * S : total;
    int u = slot;
    int64_t g = 0, g1 = 0;
    if (P > 0 && slot < P) {
        g = (int64_t)slot * W / P;
        g1 = (int64_t)(slot + 1) * W / P;
    }
    auto take = [&](TileArgs &a) {
        if (P > 0) {
            if (g >= g1) return false;
            const int j = (int)(g / nk);
            const int64_t t0 = (int64_t)j * nk, stop = min<int64_t>(g1, t0 + nk);
            a = tile_args(j, (int)(g - t0), (int)(stop - g),
                          parts + (size_t)(slot + j) * TP::PART_ELEMS, g == t0 ? j : -1);
            g = stop;
            return true;
        }
        if (u >= units) return false;
        if (u < end) {
            a = tile_args(u, 0, nk, nullptr, -1);
        } else {
            // piece p of S covers stages [p*nk/S, (p+1)*nk/S)
            const int j = (u - full) / S, piece = (u - full) % S;
            const int k0 = piece * nk / S;
            a = tile_args(full + j, k0, (piece + 1) * nk / S - k0,
                          parts + (size_t)(j * S + piece) * TP::PART_ELEMS, piece == 0 ? j : -1);
        }
        u += G;
        return true;
    };
    using Tile = typename TP::template Tile<false>;
    Tile tile(smem);
    TileArgs a;
    if (!take(a)) return;
    tile.bind(a);
    tile.prologue();
    typename Tile::After after = Tile::NOTHING;
    while (true) {
        tile.kloop(after);
        TileArgs next;
        const bool more = take(next);
        if (more) {
            tile.bind(next);
            tile.prologue();
        }
        if (a.part != nullptr) {
            tile.store_piece(a);
            after = Tile::PIECE;
        } else {
            tile.epilogue(a, more);
            after = Tile::STORES;
        }
        if (!more) break;
        a = next;
    }
}

// The fragment rows of one (GEMM wave, fragment-row pair) of a tail tile
// cut into S pieces: each fragment's S pieces are loaded together and added
// in piece order, one fragment row at a time.
template <int MODE, class C, int S>
__device__ __forceinline__ void fixup_rows(__amdgpu_buffer_rsrc_t pres, int loff, int wave, int p,
                                           void *o, int64_t ldo, int m_valid, int n_valid) {
    static_assert(S >= 2 && S <= kSplitMaxPieces, "piece count");
    constexpr int NP = C::TN / 2;
#pragma unroll 1
    for (int m = 0; m < C::TM; ++m) {
        // fragment rows wholly past the valid edge: no partials were stored
        if ((wave >> 1) * C::WTM + m * 16 >= m_valid) break;
        floatx4 sum[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int f = wave * C::WAVE_BYTES + ((p + h * NP) * C::TM + m) * 1024;
            floatx4 v[S];
#pragma unroll
            for (int q = 0; q < S; ++q)
                v[q] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(
                                                       pres, loff, q * C::PART_BYTES + f, 0));
            floatx4 r = v[0];
#pragma unroll
            for (int q = 1; q < S; ++q) {
                r[0] += v[q][0];
                r[1] += v[q][1];
                r[2] += v[q][2];
                r[3] += v[q][3];
            }
            sum[h] = r;
        }
        const int lane = threadIdx.x & 63;
        if (MODE == 0) {
            store_gateup<C>(sum[0], sum[1], p, m, wave & 1, wave >> 1, lane,
                            reinterpret_cast<bf16_t *>(o), ldo, m_valid, n_valid);
        } else {
            store_down<C>(sum[0], p, m, wave & 1, wave >> 1, lane, reinterpret_cast<float *>(o),
                          ldo, m_valid, n_valid);
            store_down<C>(sum[1], p + NP, m, wave & 1, wave >> 1, lane,
                          reinterpret_cast<float *>(o), ldo, m_valid, n_valid);
        }
    }
}

// Sum of the K pieces of the grouped GEMM's tail tiles, then the tile
// epilogue.  Work unit = (tail tile, GEMM wave), taken grid-stride by
// workgroups of four waves, one wave per fragment-row pair of that GEMM
// wave: it loads a fragment's S pieces together, adds them in piece order
// (p0 + p1 + ...), so the result is the same whichever piece finished first,
// and stores the pair as the GEMM's own epilogue would.  With no tail tiles
// (the host does not know the count) every workgroup returns at once.
template <int MODE, class TP>
__global__ __launch_bounds__(256) void split_fixup_kernel(const float *__restrict__ parts,
                                                         const int32_t *__restrict__ meta,
                                                         void *out, int64_t ldo) {
    using C = typename TP::C;
    constexpr int NP = C::TN / 2;  // fragment-row pairs per wave
    static_assert(NP * 64 == 256, "one wave per fragment-row pair");
    const int ntail = meta[0];
    const int S_eq = meta[1];  // equal pieces per tile, or 0: stream-K over P units
    const int P = meta[2], nk = meta[3];
    const int64_t W = (int64_t)ntail * nk;
    const int p = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    for (int unit = blockIdx.x; unit < ntail * C::WAVES; unit += gridDim.x) {
        const int j = unit / C::WAVES;
        const int wave = unit % C::WAVES;
        // the tile's pieces sit in consecutive slots [first, first + S), in K order
        int first, S;
        if (S_eq > 0) {
            first = j * S_eq;
            S = S_eq;
        } else {
            // units holding the tile's first and last stage (the unit of
            // stage s is the last u with u * W / P <= s)
            const int u0 = (int)((((int64_t)j * nk + 1) * P - 1) / W);
            const int u1 = (int)(((int64_t)(j + 1) * nk * P - 1) / W);
            first = u0 + j;
            S = u1 - u0 + 1;
        }
        const int32_t *md = meta + 4 + 4 * j;
        const int64_t r0 = md[0], n0 = md[1];
        const int m_valid = md[2], n_valid = md[3];
        const __amdgpu_buffer_rsrc_t pres = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float *>(parts) + (size_t)first * C::PART_ELEMS, 0, -1, kBufferFlags);
        const int loff = lane * 16;
        void *o = MODE == 0 ? (void *)(reinterpret_cast<bf16_t *>(out) + r0 * ldo + n0)
                            : (void *)(reinterpret_cast<float *>(out) + r0 * ldo + n0);
        switch (S) {  // a static piece count: loads and sums stay unrolled
            case 2: fixup_rows<MODE, C, 2>(pres, loff, wave, p, o, ldo, m_valid, n_valid); break;
            case 3: fixup_rows<MODE, C, 3>(pres, loff, wave, p, o, ldo, m_valid, n_valid); break;
            case 4: fixup_rows<MODE, C, 4>(pres, loff, wave, p, o, ldo, m_valid, n_valid); break;
            case 5: fixup_rows<MODE, C, 5>(pres, loff, wave, p, o, ldo, m_valid, n_valid); break;
            case 6: fixup_rows<MODE, C, 6>(pres, loff, wave, p, o, ldo, m_valid, n_valid); break;
            case 7: fixup_rows<MODE, C, 7>(pres, loff, wave, p, o, ldo, m_valid, n_valid); break;
            case 8: fixup_rows<MODE, C, 8>(pres, loff, wave, p, o, ldo, m_valid, n_valid); break;
            default: break;
        }
    }
}

// Tile policy of each scheduler: the ping-pong tile, 256 weight rows by BM
// token rows.  The grouped launch knows its experts' host row counts or
// only a bound on them (the tokens); the launch-cost model picks its height
// (group_launch_rows) up to the smallest that holds that bound, with 320
// rows (fewest LDS bytes per MFMA) above 256; a dense launch knows its
// expert's rows and takes the height whose tile count fills the grid best
// (dense_tile_rows).
constexpr int kTokenTile = 320;
template <int MODE, int BM = kTokenTile> using TileOf = PingPong<MODE, BM>;
template <int MODE> using GroupTile = TileOf<MODE>;

// ---------------------------------------------------------------------------
// Skinny down tile for decode-sized grouped launches: every expert of the
// launch has at most 64 rows, so its down GEMM is one row of tiles that
// streams the expert's weights once.  A workgroup is one wave and owns SK_BN
// output columns (weight rows) by the expert's rows over the whole K range:
// no K split, no fixup.  The height (16, 32 or 64 rows) is the workgroup's
// own, from its expert's row count: a launch of 61 tokens over 160 experts
// has one or two experts above 16 rows, and a height taken from the upper
// bound would make every other tile read and multiply padding (us, one
// height for the launch -> per expert: DeepSeekV2 61 tokens 62 -> 51, DBRX 64
// 50.9 -> 49.0, 64 tokens over 64 experts of 2048 x 1024 20.5 -> 19.3).
// Weight and act rows stream through a ring of LDS stages of SK_BK K by
// LDS-DMA, all but one stage ahead, as many stages as the launch's LDS holds
// (sk_ring), the 16-byte chunks of each row XOR-placed as in the ping-pong
// tile.  The MFMA (16x16x32 bf16, the weight fragment as the A
// operand, K ascending from 0) and the fragment contents are the ping-pong
// tile's, so the outputs carry the same bits as every other tile height in
// exact order.  The fragment reads and their wait are one assembly block:
// the compiler would otherwise wait for all LDS-DMA in flight before
// reading LDS and drain the ring every stage.
constexpr int SK_BN = 64;  // weight rows (output columns) per tile
// K per ring stage: 64, so each stage reads 128 contiguous bytes of every
// weight row.  With 32 (64-byte pieces of rows 3-12 KB apart) the weight
// stream ran 13-27% slower, even where the wider stages leave fewer tiles
// resident per compute unit.
constexpr int SK_BK = 64;
constexpr int SK_NS_MAX = 16;             // ring stages at most
constexpr size_t SK_LDS_MAX = 64 * 1024;  // dynamic LDS of one workgroup at most

// stages a wave can keep ahead: vmcnt counts at most 63 requests
__host__ __device__ constexpr int sk_ahead_max(int lps) {
    return SK_NS_MAX - 1 < 63 / lps ? SK_NS_MAX - 1 : 63 / lps;
}
// LDS-DMA requests per stage (64 lanes x 16 bytes each)
__host__ __device__ constexpr int sk_lps(int bm) { return (SK_BN + bm) * SK_BK * 2 / 1024; }

// LDS bytes of a workgroup with a ring of ns stages: the ring plus
// room for the act-fragment reads a tile of fewer than 64 rows does not use
__host__ __device__ constexpr size_t sk_lds_bytes(int bm, int ns) {
    return (size_t)ns * (SK_BN + bm) * SK_BK * 2 + (size_t)(4 - bm / 16) * 16 * SK_BK * 2;
}
// stages of a tile of bm rows in `lds` bytes, as many as vmcnt can count
__host__ __device__ constexpr int sk_ring(int bm, size_t lds) {
    int ns = sk_ahead_max(sk_lps(bm)) + 1;
    while (ns > 1 && sk_lds_bytes(bm, ns) > lds) --ns;
    return ns;
}
// LDS of a launch's workgroups: SK_LDS_MAX, two resident per compute unit;
// or, three resident, four stages of up to 32 rows, where every tile that may
// have rows is then resident at once.  us, two -> three: 700 tiles (2.7 per
// unit) of 6144 x 1344 28.0 -> 26.4, of 6144 x 10752 176 -> 161; but 3.6 per
// unit of 4096 x 6400 132 -> 160.
constexpr size_t SK_LDS_THREE = sk_lds_bytes(32, 4);
static_assert(3 * SK_LDS_THREE <= 160 * 1024, "three resident");

// one K-step's fragments: 4 weight fragments from wa, 4 act fragments from
// xa (a tile of fewer rows reads the first ones; the others land in the
// next slot or the padding after the ring), F bytes (16 LDS rows) apart
template <int F>
__device__ __forceinline__ void sk_read_frags(bf16x8 (&f)[8], uint32_t wa, uint32_t xa) {
    asm volatile(
        "ds_read_b128 %0, %8\n\t"
        "ds_read_b128 %1, %8 offset:%10\n\t"
        "ds_read_b128 %2, %8 offset:%11\n\t"
        "ds_read_b128 %3, %8 offset:%12\n\t"
        "ds_read_b128 %4, %9\n\t"
        "ds_read_b128 %5, %9 offset:%10\n\t"
        "ds_read_b128 %6, %9 offset:%11\n\t"
        "ds_read_b128 %7, %9 offset:%12\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(f[0]), "=&v"(f[1]), "=&v"(f[2]), "=&v"(f[3]), "=&v"(f[4]), "=&v"(f[5]),
          "=&v"(f[6]), "=&v"(f[7])
        : "v"(wa), "v"(xa), "i"(F), "i"(2 * F), "i"(3 * F)
        : "memory");
}

// s_waitcnt vmcnt(LPS * n), 0 <= n <= K
template <int LPS, int K = sk_ahead_max(LPS)>
__device__ __forceinline__ void sk_wait(int n) {
    if (n == K) {
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(K * LPS) : "memory");
    } else if constexpr (K > 0) {
        sk_wait<LPS, K - 1>(n);
    }
}

// One tile: y columns n0 .. n0 + 63 of the `rows` <= BM rows from r0 on; w:
// the expert's weights; ns ring stages.
template <int BM>
__device__ __forceinline__ void skinny_tile(bf16_t *smem, int ns, int r0, int rows, int n0,
                                            const bf16_t *__restrict__ act,
                                            const bf16_t *__restrict__ w, int N, int K,
                                            float *__restrict__ y) {
    constexpr int TN = SK_BN / 16, TM = BM / 16, BK = SK_BK;
    static_assert(TM <= 4, "at most 4 act fragments per K-step");
    constexpr int CPR = BK / 8;    // 16-byte chunks per LDS row
    constexpr int RPI = 64 / CPR;  // rows one LDS-DMA request fills
    constexpr int WI = SK_BN / RPI, XI = BM / RPI;
    constexpr int LPS = WI + XI;
    static_assert(LPS == sk_lps(BM), "requests per stage");
    constexpr int STAGE = (SK_BN + BM) * BK;  // bf16 elements
    constexpr int F = 16 * BK * 2;            // bytes of 16 LDS rows
    constexpr int KH = BK / 32;               // MFMA K-steps per stage
    const int lane = threadIdx.x;

    // LDS-DMA sources: lane i fetches row (i / CPR) of an RPI-row request,
    // the 16-byte chunk (i % CPR) ^ swz(row) of the stage's BK K, into
    // place i % CPR
    const int drow = lane / CPR;
    const int dchunk = ((lane % CPR) ^ swz<BK>(drow)) * 8;
    const bf16_t *src[LPS];
#pragma unroll
    for (int i = 0; i < WI; ++i) src[i] = w + (int64_t)(n0 + i * RPI + drow) * K + dchunk;
#pragma unroll
    for (int i = 0; i < XI; ++i) {
        const int j = min(i * RPI + drow, rows - 1);  // rows past the expert's: repeats
        src[WI + i] = act + (int64_t)(r0 + j) * K + dchunk;
    }
    const int nk = K / BK;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_void_t *)smem;
    auto issue = [&](int kt, int slot) {
#pragma unroll
        for (int i = 0; i < LPS; ++i)
            dma16_to_lds(src[i] + kt * BK, lds0 + (slot * STAGE + i * RPI * BK) * 2);
    };

    // fragment addresses in ring slot 0, K-step h of the stage: weight row
    // t * 16 + lrow and act row m * 16 + lrow, the chunk holding K
    // 32 h + 8 (lane / 16) .. + 7
    const int lrow = lane & 15;
    uint32_t wa0[KH], xa0[KH];
#pragma unroll
    for (int h = 0; h < KH; ++h) {
        const int chunk = ((h * 4 + (lane >> 4)) ^ swz<BK>(lrow)) * 8;
        wa0[h] = lds0 + (uint32_t)((lrow * BK + chunk) * 2);
        xa0[h] = wa0[h] + (uint32_t)(SK_BN * BK * 2);
    }

    floatx4 acc[TN][TM];
#pragma unroll
    for (int t = 0; t < TN; ++t)
#pragma unroll
        for (int m = 0; m < TM; ++m) acc[t][m] = floatx4{0.f, 0.f, 0.f, 0.f};

    // stage kt goes to ring slot kt % ns
    const int ahead = ns - 1;
    for (int kt = 0; kt < min(ahead, nk); ++kt) issue(kt, kt);
    int wslot = ahead, rslot = 0;  // slots of stages kt + ahead and kt
    for (int kt = 0; kt < nk; ++kt) {
        // stage kt + ahead into the slot read at kt - 1
        if (kt + ahead < nk) issue(kt + ahead, wslot);
        wslot = wslot + 1 == ns ? 0 : wslot + 1;
        sk_wait<LPS>(min(ahead, nk - 1 - kt));  // stage kt landed
        const uint32_t so = (uint32_t)(rslot * STAGE * 2);
        rslot = rslot + 1 == ns ? 0 : rslot + 1;
#pragma unroll
        for (int h = 0; h < KH; ++h) {
            bf16x8 f[8];
            sk_read_frags<F>(f, wa0[h] + so, xa0[h] + so);
#pragma unroll
            for (int m = 0; m < TM; ++m)
#pragma unroll
                for (int t = 0; t < TN; ++t)
                    acc[t][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[t], f[4 + m],
                                                                        acc[t][m], 0, 0, 0);
        }
    }

    // epilogue: the lane holds output columns t * 16 + 4 (lane / 16) .. + 3
    // of row m * 16 + (lane % 16)
    const int ocol = (lane >> 4) * 4;
#pragma unroll
    for (int m = 0; m < TM; ++m) {
        const int row = m * 16 + lrow;
        if (row >= rows) continue;
        float *o = y + (int64_t)(r0 + row) * N + n0;
#pragma unroll
        for (int t = 0; t < TN; ++t) *reinterpret_cast<floatx4 *>(o + t * 16 + ocol) = acc[t][m];
    }
}

// y[r0 + r][n0 .. n0 + 63] = w_down[e_first + e][n0 ..] . act[r0 + r] for
// the r < rows of expert e (offsets indexed by e_first + e, as in the other
// launches); grid = e_count * (N / SK_BN).  The expert's rows, read on the
// device, pick the tile's height (every expert's may be far below the
// launch's bound, the tokens): against one height for the launch, us,
// DeepSeekV2 61 tokens 62 -> 51, Zipf 64 tokens 20.5 -> 19.3, DBRX 64 tokens
// 50.9 -> 49.0.
template <size_t LDS>
__global__ __launch_bounds__(64) void skinny_down_kernel(const int32_t *__restrict__ offsets,
                                                         int e_first, int e_count,
                                                         const bf16_t *__restrict__ act,
                                                         const bf16_t *__restrict__ w,
                                                         int64_t wstride, int N, int K,
                                                         float *__restrict__ y) {
    extern __shared__ __attribute__((aligned(16))) bf16_t smem[];
    const int NT = N / SK_BN;
    const int e = blockIdx.x / NT;
    const int n0 = (blockIdx.x - e * NT) * SK_BN;
    if (e >= e_count) return;
    const int r0 = __builtin_amdgcn_readfirstlane(offsets[e_first + e]);
    const int rows = __builtin_amdgcn_readfirstlane(offsets[e_first + e + 1]) - r0;
    if (rows <= 0) return;  // (rows <= 64: the launcher's bound)
    const bf16_t *we = w + (int64_t)(e_first + e) * wstride;
    if (rows <= 16)
        skinny_tile<16>(smem, sk_ring(16, LDS), r0, rows, n0, act, we, N, K, y);
    else if (rows <= 32)
        skinny_tile<32>(smem, sk_ring(32, LDS), r0, rows, n0, act, we, N, K, y);
    else
        skinny_tile<64>(smem, sk_ring(64, LDS), r0, rows, n0, act, we, N, K, y);
}

int round_grid(int64_t tiles) { return (int)(((tiles + NXCD - 1) / NXCD) * NXCD); }

// Fixup launch after a grouped GEMM that was given a split buffer: fewer
// than grid tail tiles can be cut (each into two or more pieces), 8 work
// units each; one workgroup per compute unit at most, so an empty fixup is
// cheap to dispatch.
template <int MODE, class TP>
hipError_t launch_split_fixup(int grid, const float *parts, const int32_t *meta, void *out,
                              int64_t ldo, hipStream_t s) {
    const int max_tail = std::min(grid, kSplitMaxTail);
    const int blocks = std::min(max_tail * TP::C::WAVES, device_cu_count());
    split_fixup_kernel<MODE, TP><<<blocks, 256, 0, s>>>(parts, meta, out, ldo);
    return hipGetLastError();
}

template <int MODE, class TP>
hipError_t group_launch(const int32_t *offsets, int e_first, int e_count, const bf16_t *x,
                        const int32_t *row_map, int slot_div, const bf16_t *w0s,
                        const bf16_t *w1s, int64_t wstride, int N, int K, void *out,
                        int64_t ldo, int grid, float *parts, int32_t *split_meta, int rows_one,
                        hipStream_t s) {
    const bool split = parts != nullptr && split_meta != nullptr;
    group_kernel<MODE, TP><<<grid, TP::THREADS, 0, s>>>(
        offsets, e_first, e_count, x, row_map, slot_div, w0s, w1s, wstride, N, K, out, ldo,
        split ? parts : nullptr, split ? split_meta : nullptr, rows_one);
    if (split) return launch_split_fixup<MODE, TP>(grid, parts, split_meta, out, ldo, s);
    return hipGetLastError();
}

template <int MODE>
hipError_t group_launch_bm(int bm, const int32_t *offsets, int e_first, int e_count,
                           const bf16_t *x, const int32_t *row_map, int slot_div,
                           const bf16_t *w0s, const bf16_t *w1s, int64_t wstride, int N, int K,
                           void *out, int64_t ldo, int grid, float *parts, int32_t *split_meta,
                           int rows_one, hipStream_t s) {
#define MOE_GROUP_LAUNCH(BMV)                                                                   \
    return group_launch<MODE, TileOf<MODE, BMV>>(offsets, e_first, e_count, x, row_map,       \
                                                 slot_div, w0s, w1s, wstride, N, K, out, ldo, \
                                                 grid, parts, split_meta, rows_one, s)
    switch (bm) {
        case 128: MOE_GROUP_LAUNCH(128);
        case 192: MOE_GROUP_LAUNCH(192);
        case 256: MOE_GROUP_LAUNCH(256);
        default: MOE_GROUP_LAUNCH(320);
    }
#undef MOE_GROUP_LAUNCH
}

template <int MODE, class TP>
hipError_t dense_launch(int64_t rows, const bf16_t *x, const bf16_t *w0, const bf16_t *w1, int N,
                        int K, void *out, int64_t ldo, hipStream_t s) {
    const int MT = (int)((rows + TP::BM - 1) / TP::BM);
    const int NT = (N + TP::BNOUT - 1) / TP::BNOUT;
    dense_kernel<MODE, TP><<<round_grid((int64_t)MT * NT), TP::THREADS, 0, s>>>(
        x, rows, w0, w1, N, K, out, ldo, MT, NT);
    return hipGetLastError();
}

template <int MODE>
hipError_t dense_launch_bm(int bm, int64_t rows, const bf16_t *x, const bf16_t *w0,
                           const bf16_t *w1, int N, int K, void *out, int64_t ldo, hipStream_t s) {
    switch (bm) {
        case 128: return dense_launch<MODE, TileOf<MODE, 128>>(rows, x, w0, w1, N, K, out, ldo, s);
        case 192: return dense_launch<MODE, TileOf<MODE, 192>>(rows, x, w0, w1, N, K, out, ldo, s);
        case 256: return dense_launch<MODE, TileOf<MODE, 256>>(rows, x, w0, w1, N, K, out, ldo, s);
        default: return dense_launch<MODE, TileOf<MODE, 320>>(rows, x, w0, w1, N, K, out, ldo, s);
    }
}

// ---- launch cost model (host) ---------------------------------------------
// Device time of one launch of the persistent scheduler, from per-tile costs
// of each tile height measured on MI355X (microseconds):
//   tile time = K / 32 * step(MODE, BM) + epi(MODE, BM)
// (step: the cost of 32 K, whatever the tile's stage depth).  Tiles run in rounds of G
// workgroups; a partial round of rem tiles takes the fraction
// kPartialRound[MODE] + (1 - kPartialRound) * busy of a full round's K loop
// (busy = the fraction of workgroups with work: fewer active compute units
// run each tile faster), then the epilogue.  With the K split, a partial
// last round of rem <= G/2 tiles is cut into S pieces as the scheduler does
// (S = min(8, G/rem, stages/32, slots/rem)): its K loop is S times shorter, and
// the fixup costs a fixed time plus a time per partial-sum block (its bytes
// grow with BM).  Each launch pays a fixed start-up and drain time.
struct TileCost {
    int bm;
    double step_us[2];  // 32 K of a 256 x BM tile: gate/up, down
    double epi_us[2];   // a tile's epilogue: gate/up (bf16 SiLU*mul), down (fp32)
};
// Fitted by least squares (4.0% rms gate/up, 4.5% down, 14% worst) to one
// expert's dense launches at 512 .. 32768 rows on the DeepSeekV2 (H 5120,
// I 1536) and Mixtral (H 4096, I 3584) expert shapes, every tile height,
// with and without the K split (bench.py --tile-study), of tiles that ran
// their epilogue after the K loop and branched in it.  On the present tiles
// the same study reads 6.6% rms gate/up, 8.2% down, 18% worst (priced 4 and
// 6% high on average); the height picked is the fastest at 24 of 27 points
// and at most 5% off at the others.  Streaming and skinny launches are not
// in the model.
constexpr TileCost kTileCosts[] = {
    {320, {0.896, 1.004}, {13.0, 12.3}},
    {256, {0.750, 0.839}, {14.6, 12.8}},
    {192, {0.607, 0.715}, {10.7, 9.3}},
    {128, {0.441, 0.471}, {6.2, 7.7}},
};
constexpr double kLaunchUs[2] = {12.9, 6.4};     // start-up + drain: gate/up, down
constexpr double kPartialRound[2] = {0.69, 0.71};
constexpr double kFixupUs[2] = {0.0, 2.3};       // fixup launch with work
constexpr double kFixupBlockUs[2] = {0.0994, 0.0864};  // per 256 x 320 partial block

const TileCost &tile_cost(int bm) {
    for (const TileCost &c : kTileCosts)
        if (c.bm == bm) return c;
    return kTileCosts[0];
}

// Equal K pieces that group_kernel cuts the rem tiles of a partial last round
// into, after full_rounds whole ones, nk K stages each.
int split_pieces(int64_t rem, int64_t full_rounds, int nk, int grid) {
    if (2 * rem > grid) return 1;
    return (int)std::max<int64_t>(
        1, std::min<int64_t>(
               std::min<int64_t>(kSplitMaxPieces, grid / rem),
               std::min<int64_t>(nk / (full_rounds == 0 ? kSplitMinStagesAlone : kSplitMinStages),
                                 kSplitSlots / rem)));
}

}  // namespace

double tiled_round_fill(int64_t tiles, int K, int grid) {
    if (tiles <= 0) return 0.0;
    const int64_t full = tiles / grid, rem = tiles % grid;
    double rounds = (double)full;
    if (rem > 0) rounds += 1.0 / split_pieces(rem, full, K / pp_stage_k(128), grid);
    return (double)tiles / (grid * rounds);
}

double gemm_launch_us(int mode, int bm, int64_t tiles, int K, int grid, bool split) {
    if (tiles <= 0) return 0.0;
    const TileCost &c = tile_cost(bm);
    const int md = mode ? 1 : 0;
    const double loop_us = K / 32 * c.step_us[md];
    const int nk = K / pp_stage_k(bm);  // the tile's K stages, as the kernel cuts them
    const int64_t full_rounds = tiles / grid;
    const int64_t rem = tiles % grid;
    double us = kLaunchUs[md] + full_rounds * (loop_us + c.epi_us[md]);
    if (rem > 0) {
        // (a round of more than half the grid that the kernel spreads
        // stream-K, for tall tiles at most half full, is priced unsplit: an
        // upper bound)
        const int S = split ? split_pieces(rem, full_rounds, nk, grid) : 1;
        const double busy = (double)std::min<int64_t>(grid, rem * S) / grid;
        const double part = kPartialRound[md] + (1.0 - kPartialRound[md]) * busy;
        if (S >= 2)
            us += loop_us / S * part + c.epi_us[md] + kFixupUs[md] +
                  kFixupBlockUs[md] * (double)(rem * S) * bm / 320.0;
        else
            us += loop_us * part + c.epi_us[md];
    }
    return us;
}

int64_t gemm_tiles(int mode, int bm, int64_t rows, int N) {
    const int bnout = mode == 0 ? 128 : 256;
    return ((rows + bm - 1) / bm) * ((N + bnout - 1) / bnout);
}

double ffn_expert_us(int bm, int64_t rows, int H, int I, int grid, bool split) {
    return gemm_launch_us(0, bm, gemm_tiles(0, bm, rows, I), H, grid, split) +
           gemm_launch_us(1, bm, gemm_tiles(1, bm, rows, H), I, grid, split);
}

int dense_tile_rows(int64_t rows, int H, int I, int grid, bool split) {
    int best = kTokenTile;
    double best_us = 0.0;
    for (const TileCost &c : kTileCosts) {
        const double us = ffn_expert_us(c.bm, rows, H, I, grid, split);
        if (best_us == 0.0 || us < best_us) {
            best = c.bm;
            best_us = us;
        }
    }
    return best;
}

int group_tile_rows(int64_t max_rows) {
    // below the tallest tile, the smallest height that still holds every
    // expert's rows in one tile: fewer padded rows, never more tiles
    if (max_rows <= 128) return 128;
    if (max_rows <= 192) return 192;
    if (max_rows <= 256) return 256;
    return kTokenTile;
}

namespace {

constexpr int kTileHeights[4] = {128, 192, 256, 320};

// Expected m-tiles of one expert for each tile height, E[ceil(min(r, cap)
// / bm)], where its row count r ~ Binomial(tokens, p): every token picks
// the expert with probability p (top_k distinct of E experts, uniform).
// The probabilities are walked out from the mode by the ratio of
// neighbouring terms until they fall below 1e-12 of the mode's.
void expected_mtiles(int64_t tokens, double p, int64_t cap, double out[4]) {
    for (int i = 0; i < 4; ++i) out[i] = 0.0;
    if (tokens <= 0 || cap <= 0 || p <= 0.0) return;
    auto add = [&](int64_t r, double pr) {
        const int64_t rr = std::min(r, cap);
        for (int i = 0; i < 4; ++i) out[i] += pr * (double)((rr + kTileHeights[i] - 1) / kTileHeights[i]);
    };
    if (p >= 1.0) {
        add(tokens, 1.0);
        return;
    }
    const double q = 1.0 - p, n = (double)tokens;
    const int64_t mode = std::min<int64_t>(tokens, (int64_t)((n + 1.0) * p));
    const double m = (double)mode;
    const double pm = std::exp(std::lgamma(n + 1.0) - std::lgamma(m + 1.0) -
                               std::lgamma(n - m + 1.0) + m * std::log(p) + (n - m) * std::log(q));
    double total = pm, pr = pm;
    add(mode, pm);
    for (int64_t r = mode; r < tokens; ++r) {
        pr *= (double)(tokens - r) / (double)(r + 1) * (p / q);
        if (pr < 1e-12 * pm) break;
        add(r + 1, pr);
        total += pr;
    }
    pr = pm;
    for (int64_t r = mode; r > 0; --r) {
        pr *= (double)r / (double)(tokens - r + 1) * (q / p);
        if (pr < 1e-12 * pm) break;
        add(r - 1, pr);
        total += pr;
    }
    for (int i = 0; i < 4; ++i) out[i] /= total;
}

}  // namespace

int group_launch_rows(int64_t max_rows, const int32_t *rows, int n_experts, int64_t tokens,
                      double p, int H, int I, int grid, bool split) {
    const int cap = group_tile_rows(max_rows);
    if (n_experts <= 0 || cap == kTileHeights[0]) return cap;
    double mt[4];
    if (rows == nullptr) expected_mtiles(tokens, p, max_rows, mt);
    double us[4] = {0.0, 0.0, 0.0, 0.0};
    int best = -1, icap = 0;
    for (int i = 0; i < 4 && kTileHeights[i] <= cap; ++i) {
        const int bm = kTileHeights[i];
        int64_t tiles_gu = 0, tiles_dn = 0;
        if (rows != nullptr) {
            for (int e = 0; e < n_experts; ++e) {
                tiles_gu += gemm_tiles(0, bm, rows[e], I);
                tiles_dn += gemm_tiles(1, bm, rows[e], H);
            }
        } else {
            const double m = n_experts * mt[i];
            tiles_gu = std::llround(m * (double)gemm_tiles(0, bm, bm, I));
            tiles_dn = std::llround(m * (double)gemm_tiles(1, bm, bm, H));
        }
        us[i] = gemm_launch_us(0, bm, tiles_gu, H, grid, split) +
                gemm_launch_us(1, bm, tiles_dn, I, grid, split);
        if (best < 0 || us[i] < us[best]) best = i;
        icap = i;
    }
    // another height only for a predicted gain above the model's error
    return us[best] < (1.0 - kGroupRowsMinGain) * us[icap] ? kTileHeights[best] : cap;
}

bool valid_tile_rows(int bm) {
    return bm == 128 || bm == 192 || bm == 256 || bm == 320;
}

hipError_t launch_dense_gateup(int64_t rows, int H, int I, const bf16_t *x, const bf16_t *w_gate,
                               const bf16_t *w_up, bf16_t *act, int bm, hipStream_t s) {
    if (rows <= 0) return hipSuccess;
    return dense_launch_bm<0>(bm, rows, x, w_gate, w_up, I, H, act, I, s);
}

hipError_t launch_dense_down(int64_t rows, int H, int I, const bf16_t *act,
                             const bf16_t *w_down, float *y, int bm, hipStream_t s) {
    if (rows <= 0) return hipSuccess;
    return dense_launch_bm<1>(bm, rows, act, w_down, nullptr, H, I, y, H, s);
}

size_t gemm_split_bytes() {
    // the tallest tile has the largest block of partial sums
    const size_t e = std::max(GroupTile<0>::PART_ELEMS, GroupTile<1>::PART_ELEMS);
    return e * sizeof(float) * kSplitSlots;
}

hipError_t launch_group_gateup(const moe_dims &d, int e_first, int e_count,
                               const int32_t *offsets, const bf16_t *x_rows,
                               const int32_t *row_map, const bf16_t *w_gate,
                               const bf16_t *w_up, bf16_t *act, int grid, float *parts,
                               int32_t *split_meta, int bm, hipStream_t s, int64_t rows_one) {
    if (e_count <= 0) return hipSuccess;
    if (!offsets && (e_count != 1 || rows_one < 0 || rows_one > INT32_MAX))
        return hipErrorInvalidValue;
    return group_launch_bm<0>(bm, offsets, e_first, e_count, x_rows, row_map, d.top_k, w_gate,
                              w_up, (int64_t)d.inter * d.hidden, d.inter, d.hidden, act,
                              d.inter, grid, parts, split_meta, (int)rows_one, s);
}

hipError_t launch_group_down(const moe_dims &d, int e_first, int e_count,
                             const int32_t *offsets, const bf16_t *act,
                             const bf16_t *w_down, float *y_perm, int grid, float *parts,
                             int32_t *split_meta, int bm, hipStream_t s, int64_t rows_one) {
    if (e_count <= 0) return hipSuccess;
    if (!offsets && (e_count != 1 || rows_one < 0 || rows_one > INT32_MAX))
        return hipErrorInvalidValue;
    return group_launch_bm<1>(bm, offsets, e_first, e_count, act, nullptr, 1, w_down, nullptr,
                              (int64_t)d.hidden * d.inter, d.hidden, d.inter, y_perm, d.hidden,
                              grid, parts, split_meta, (int)rows_one, s);
}

bool skinny_down_fits(int64_t max_rows, int64_t active_experts, int N) {
    return max_rows <= kSkinnyMaxRows &&
           active_experts * (N / SK_BN) >= 2 * (int64_t)device_cu_count();
}

hipError_t launch_skinny_down(const moe_dims &d, int e_first, int e_count,
                              const int32_t *offsets, const bf16_t *act, const bf16_t *w_down,
                              float *y_perm, int64_t max_rows, int64_t active_experts,
                              hipStream_t s) {
    if (e_count <= 0) return hipSuccess;
    const int N = d.hidden, K = d.inter;
    if (max_rows > kSkinnyMaxRows) return hipErrorInvalidValue;
    static_assert(kDimAlign % SK_BN == 0 && kDimAlign % SK_BK == 0, "whole tiles and stages");
    static_assert(sk_ring(64, SK_LDS_THREE) >= 2, "ring depth");
    const int64_t active = std::min<int64_t>(e_count, std::max<int64_t>(1, active_experts));
    const int64_t tiles = active * (N / SK_BN), cus = device_cu_count();
    const unsigned blocks = (unsigned)(e_count * (N / SK_BN));
    if (max_rows <= 32 && tiles > 2 * cus && tiles <= 3 * cus)
        skinny_down_kernel<SK_LDS_THREE><<<blocks, 64, SK_LDS_THREE, s>>>(
            offsets, e_first, e_count, act, w_down, (int64_t)N * K, N, K, y_perm);
    else
        skinny_down_kernel<SK_LDS_MAX><<<blocks, 64, SK_LDS_MAX, s>>>(
            offsets, e_first, e_count, act, w_down, (int64_t)N * K, N, K, y_perm);
    return hipGetLastError();
}

}  // namespace moe
