// Per-example weight gradients of 3x3, pad-1 convolutions of stride 1 and 2 (bf16) from raw image rows.
//
// Same contraction as the general kernel (H1 of the path; per example i
//     dW_i[co, ci, kh, kw] = sum_{oh, ow} dY_i[co, oh, ow] * Xpad_i[ci, s oh + kh - 1, s ow + kw - 1]),
// but the nine taps of one input channel are nine shifted views of the SAME rows of X, so a
// workgroup fetches each row once and builds all nine MFMA operands from it:
//
//   * a workgroup owns 64 output channels x 64 input channels x 9 taps of one example (four
//     waves, each 32 co x 32 ci x 9 taps = nine 32x32 accumulator tiles) and walks stages of a few rows (C3Cfg);
//   * rows travel global -> LDS as they lie in memory (16-byte LDS-direct loads), in rings: no registers, no masks, no shifts on the way;
//   * a K step is eight columns of a pair of rows (the two halves of a wave hold one row each).  Stride 1: a run of X, and the same run one column
//     to the left and to the right, meets dY of the row below it (kh = 0), of its own (kh = 1) and of the row above (kh = 2): nine MFMAs from one
//     16-byte read of X, two of dY (the third is the first one of the pair before) and eight funnel shifts.  Stride 2: the even and the odd
//     columns of two rows of X are put together by byte permutes, 24 for nine MFMAs.  What lies outside the image is zeros: a row is
//     read from a few bytes of zeros, columns behind a row's end are cleared in registers, the column before it is a zero shifted in.
//     Zeros times what is not finite are no numbers.  Which rows lie outside decides where that shows in an example whose norm is not finite either way: a value of X
//     in the first (stride 1) or last row that is not finite makes the taps kh = 2 or kh = 0 of its channel NaN, which do not read it (they meet zeros of dY); one of
//     dY there leaves the taps alone that do not read it (no row of X above the image is walked, below it one where the height is odd).  Clearing X for those taps instead
//     costs 24 instructions for nine MFMAs in the rows concerned: 2-9 % of this kernel, ResNet-50's step of 8 x 32 6455 -> 6530 us.
//   * a workgroup that is done with a row of results (an example's, or a clipping unit's) stores it and goes on with the next one, whose rows
//     are on their way meanwhile.
//
// Bound by the matrix units where two workgroups share a compute unit (the best calls below reach 900-950 TFLOP/s of dense bf16's 2500; a whole launch of
// ResNet-50's layers, whose 56-wide ones leave the chip half empty, 670); by the stores where blocks are stored and K is short.  One call, us and TFLOP/s, before (rows staged through registers, nine operands
// built from three rows of X per K step: 13-25 vector instructions per MFMA) and now: 64 -> 64 at 56 x 56, 128 examples, 135 (219) -> 48 (616);
// 128 -> 128 at 28 x 28, 128, 56 (532) -> 33 (899); 256 -> 256 at 14 x 14, 256, 93 (634) -> 68 (866), stored 185 -> 156 (3.9 TB/s), clip-weighted
// 142 (416) -> 96 (616); 128 -> 128 at 16 x 16, 256, 47 (415) -> 20 (947); 128 -> 128 stride 2 onto 28 x 28, 64, 76 (195) -> 27 (559).
//
// K may be sliced over workgroups (few tiles, long K): slices store their accumulators in the
// workspace and a second kernel adds them in slice order, so results are run-to-run identical.
#include "internal.h"
#include "group.h"
#include "pieces.h"

#include <algorithm>
#include <atomic>
#include <cstdio>
#include <utility>

namespace dp {

namespace {

constexpr int C3_THREADS = 256;

struct C3Args {
    const void *x, *dy;
    int x_tab, dy_tab;                // Geo::x_tab / dy_tab: the operand pointers are arrays of example addresses
    float *out_w;                     // per-example gradients (may be null) or, weighted, the accumulator
    size_t out_stride;
    float *partials;                  // [n, tiles] partial squared norms
    float *ws_part;                   // sliced K / example ranges: accumulators in register layout
    const float *group_sqnorm;        // weighted: [n]
    float clip_c;
    int n, cin, cout, h;              // h: OUTPUT height (= input height for stride 1)
    int hin;                          // input height
    int tiles_co, tiles_ci;
    int stages;                       // of an example (C3Cfg)
    int ksplit, stages_per_split;     // per-example mode: K slices, in stages (C3Cfg)
    int ex_per_split;                 // weighted mode: examples per workgroup (ksplit = example ranges)
    int variant;                      // which body conv3x3_any_kernel runs for this layer (C3_ANY_* below)
    int rows, unit;                   // per-example modes: rows of results, examples of each (Geo::unit)
    int rows_per_wg;                  // per-example mode, not sliced: rows of results that a workgroup makes
    int total;                        // workgroups that have something to do
    int slice_ex;                     // per-example mode, sliced: > 0: the slices are ranges of this many examples of a unit
};

constexpr int C3_RP = 292;                           // floats per row staged by the store epilogue: 288 + 4
constexpr int C3_ADD_LDS = 4 * 8 * C3_RP * 4;        // bytes that adding to the accumulator needs: 4 waves x 8 rows
constexpr int C3_STORE_LDS = 4 * 2 * C3_RP * 4;      // and storing a block: 4 waves x 2 rows, beside the rings (they fill while it runs)

// How a layer's rows lie in LDS.  A workgroup walks STAGES of RPS output rows: the RPS rows of dY and the STRIDE * RPS rows of X below
// them, for its 64 channels of each.  A stage is SG groups, a group is RPG consecutive rows of 64 channels: in memory one run of bytes per
// channel, in LDS the 16-byte pieces of a run one after the other, channels PA (PX) pieces apart.  The odd pitches make the operand
// reads of 16 channels touch 16 different 16-byte bank groups, and 64 channels a whole number of LDS-direct wave instructions: PA of them.
// (Rows of 7 values may start between two dwords: their pieces are counted from the dword that the run starts in.)
// D stages are in flight ahead of the one whose products run; the rings are what two workgroups of a compute unit have room for.
template <int W, int STRIDE> struct C3Cfg {
    static constexpr int XW = W * STRIDE;                    // row length of X
    static constexpr int ROW_A = 2 * W, ROW_X = 2 * XW;      // bytes
    static constexpr int PPR = (W + 7) / 8;                  // K steps of a pair of output rows: 8 columns of either
    static constexpr bool ODD = W % 2 != 0;                  // rows of dY (stride 1: X too) start between dwords
    static constexpr bool ODD_X = XW % 2 != 0;
    static constexpr int RPG = STRIDE == 2 ? (W == 28 ? 2 : 4) : (W == 56 ? 1 : (W >= 28 ? 2 : (W >= 14 ? 4 : 8)));
    static constexpr int SG = (STRIDE == 1 && W == 56) ? 2 : 1;
    static constexpr int RPS = RPG * SG, PAIRS = RPS / 2;
    static constexpr int GB_A = RPG * ROW_A, GB_X = RPG * STRIDE * ROW_X;      // bytes of a channel's run
    static constexpr int NA = (GB_A + (ODD ? 2 : 0) + 15) / 16, NX = (GB_X + (ODD_X ? 2 : 0) + 15) / 16;
    static constexpr int PA = NA | 1, PX = NX | 1;
    static constexpr int GROUP_A = PA * 1024, GROUP_X = PX * 1024;
    static constexpr int STAGE_A = SG * GROUP_A, STAGE_X = SG * GROUP_X;
    static constexpr int D = STRIDE == 2 ? (PX > 15 ? 1 : 2) : (SG == 2 ? 1 : (PA == 7 ? 3 : 2));
    static constexpr int QX = SG * PX, QA = SG * PA;         // wave instructions of a stage
    static constexpr int UB = (QX + QA + 3) / 4;             // that a wave issues for X of a stage and dY of the next one together
    static constexpr int DUMP_SIZE = (QX + QA) % 4 ? 1024 : 0;           // (so that all waves issue the same number: what the last ones fetch lands here)
    static constexpr int ZEROS = 128;                        // bytes of zeros at the start: rows outside the image
    static constexpr int RING_X = ZEROS, RING_A = ZEROS + (D + 1) * STAGE_X;
    static constexpr int DUMP = RING_A + (D + 2) * STAGE_A, END = DUMP + DUMP_SIZE;      // dY one stage further: its next row meets this stage's last row of X
    static constexpr bool STREAMS = END + C3_STORE_LDS <= 81920 - 256;       // several rows of results by a workgroup, one after the other
    static constexpr int STORE = STREAMS ? END : 0;
    static constexpr int LDS = STREAMS ? END + C3_STORE_LDS : END;
    static constexpr bool PARTIAL_A = ROW_A % 16 != 0, PARTIAL_X = ROW_X % 16 != 0;     // a tensor may end inside a piece
    // where local row r (of a stage) of the first channel starts, for rows that start at a dword
    static constexpr int at_a(int r) { return (r / RPG) * GROUP_A + (r % RPG) * ROW_A; }
    static constexpr int at_x(int r) { return (r / (RPG * STRIDE)) * GROUP_X + (r % (RPG * STRIDE)) * ROW_X; }
    static_assert(RPS % 2 == 0, "pairs of rows");
    static_assert(LDS <= 81920 - 256, "two workgroups per CU");
    static_assert(END >= C3_ADD_LDS, "room for the epilogues");
    static_assert(PPR * 16 * STRIDE <= ZEROS, "a row of zeros");
};

constexpr int c3_rows_per_stage(int ow, int stride) { return stride == 2 ? (ow == 28 ? 2 : 4) : (ow >= 28 ? 2 : (ow >= 14 ? 4 : 8)); }
constexpr bool c3_streams(int ow, int stride) { return stride == 1 || ow == 7; }
static_assert(C3Cfg<56, 1>::STREAMS && C3Cfg<32, 1>::STREAMS && C3Cfg<28, 1>::STREAMS && C3Cfg<16, 1>::STREAMS && C3Cfg<14, 1>::STREAMS && C3Cfg<8, 1>::STREAMS &&
              C3Cfg<7, 1>::STREAMS && C3Cfg<7, 2>::STREAMS, "what the host plans");
static_assert(C3Cfg<56, 1>::RPS == c3_rows_per_stage(56, 1) && C3Cfg<32, 1>::RPS == c3_rows_per_stage(32, 1) && C3Cfg<28, 1>::RPS == c3_rows_per_stage(28, 1) &&
              C3Cfg<16, 1>::RPS == c3_rows_per_stage(16, 1) && C3Cfg<14, 1>::RPS == c3_rows_per_stage(14, 1) && C3Cfg<8, 1>::RPS == c3_rows_per_stage(8, 1) &&
              C3Cfg<7, 1>::RPS == c3_rows_per_stage(7, 1) && C3Cfg<28, 2>::RPS == c3_rows_per_stage(28, 2) && C3Cfg<14, 2>::RPS == c3_rows_per_stage(14, 2) &&
              C3Cfg<7, 2>::RPS == c3_rows_per_stage(7, 2), "what the host plans");

// Finished accumulators (all of K of one row of results): this wave's share of the squared norm of the 64 x 64 x 9 block, in lane 63.
__device__ __forceinline__ float c3_squares(const f32x16 (&acc)[9], const C3Args &a, int co0, int ci0, int wm, int wn, int lane)
{
    asm volatile("" : "+v"(lane), "+s"(co0), "+s"(ci0));             // (nothing of this is worth a register during the products)
    float ss = 0.0f;
    const bool ci_there = ci0 + wn * 32 + (lane & 31) < a.cin;
    const int co_there = a.cout - (co0 + wm * 32 + (lane >> 5) * 4);
#pragma unroll
    for (int r = 0; r < 16; ++r) {                    // (what stands for channels beyond the layer does not count)
        float s = 0.0f;
#pragma unroll
        for (int t = 0; t < 9; ++t) s += acc[t][r] * acc[t][r];
        ss += ci_there && (r >> 2) * 8 + (r & 3) < co_there ? s : 0.0f;
    }
    return wave_sum_last_lane(ss);
}

// The block in the framework's [Cout, Cin, 3, 3] order; returns whether this wave issued all of its 48 stores.
//
// In the accumulator layout a lane holds, per tap, one input channel and sixteen output channels,
// so a direct store writes 4 bytes every 36.  When the layer's channel counts allow it the block
// goes through LDS instead (`buf`, this wave's own): the wave lays down two output-channel
// rows of 32 ci x 9 taps = 288 consecutive floats of the gradient, and reads them
// back as 16-byte pieces that leave as fully coalesced 1152-byte row segments.
__device__ __forceinline__ bool c3_store(const f32x16 (&acc)[9], const C3Args &a, int i, int co0, int ci0, int wm, int wn, int lane, float *buf)
{
    asm volatile("" : "+v"(lane), "+s"(co0), "+s"(ci0), "+s"(i));    // (as above)
    float *out = a.out_w + (size_t)i * a.out_stride;
    // wave-uniform: whole 32-channel blocks, 16-byte aligned rows
    if ((a.cin % 32 == 0) && (a.out_stride % 4 == 0) && ((reinterpret_cast<uintptr_t>(a.out_w) & 15u) == 0)) {
        const int cil = lane & 31, half = lane >> 5;
        const int cib = ci0 + wn * 32;                                // first input channel of this wave
        const int left = cib < a.cin ? a.cout - co0 - wm * 32 : 0;    // output channels there are
#pragma unroll
        for (int r = 0; r < 16; ++r) {                                // (a wave's LDS instructions run in order: no waits between the passes)
#pragma unroll
            for (int t = 0; t < 9; ++t) buf[half * C3_RP + cil * 9 + t] = acc[t][r];
            const int co = (r >> 2) * 8 + (r & 3);                    // and co + 4
#pragma unroll
            for (int it = 0; it < 3; ++it) {
                const int f4 = it * 64 + lane;                        // 2 rows x 72 pieces
                if (it < 2 || f4 < 144) {
                    const int row = f4 >= 72 ? 1 : 0, c4 = f4 - row * 72;
                    const float4 v = *reinterpret_cast<const float4 *>(buf + row * C3_RP + c4 * 4);
                    if (co + row * 4 < left)
                        *reinterpret_cast<float4 *>(out + ((size_t)(co0 + wm * 32 + co + row * 4) * a.cin + cib) * 9 + c4 * 4) = v;
                }
            }
        }
        return left >= 32;
    }
    const int ci = ci0 + wn * 32 + (lane & 31);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int co = co0 + wm * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
        const bool ok = co < a.cout && ci < a.cin;
        const size_t base = ((size_t)co * a.cin + ci) * 9;
#pragma unroll
        for (int t = 0; t < 9; ++t)
            if (ok) out[base + t] = acc[t][r];
    }
    return false;
}

// Weighted sum of one tile over all examples: acc[co, ci, tap] += block, through LDS in the same
// coalesced row form as the store above (eight rows a wave) when the shapes allow, else element by element.
__device__ __forceinline__ void c3_add_to_accumulator(const f32x16 (&acc)[9], const C3Args &a, int co0, int ci0,
                                                      int wm, int wn, int lane, char *lds)
{
    float *out = a.out_w;
    const bool via_lds = (a.cin % 32 == 0) && ((reinterpret_cast<uintptr_t>(a.out_w) & 15u) == 0);
    if (via_lds) {
        float *buf = reinterpret_cast<float *>(lds) + (threadIdx.x >> 6) * (8 * C3_RP);
        const int cil = lane & 31, half = lane >> 5;
        const int cib = ci0 + wn * 32;
        __syncthreads();                              // the rings are no longer read
#pragma unroll
        for (int q = 0; q < 4; ++q) {
#pragma unroll
            for (int rr = 0; rr < 4; ++rr)
#pragma unroll
                for (int t = 0; t < 9; ++t) buf[(half * 4 + rr) * C3_RP + cil * 9 + t] = acc[t][q * 4 + rr];
#pragma unroll
            for (int it = 0; it < 9; ++it) {
                const int f4 = it * 64 + lane;
                const int row = f4 / 72, c4 = f4 - row * 72;
                const int co = co0 + wm * 32 + q * 8 + row;
                const float4 v = *reinterpret_cast<const float4 *>(buf + row * C3_RP + c4 * 4);
                if (co < a.cout && cib < a.cin) {
                    float4 *dst = reinterpret_cast<float4 *>(out + ((size_t)co * a.cin + cib) * 9 + c4 * 4);
                    float4 o = *dst;
                    o.x += v.x; o.y += v.y; o.z += v.z; o.w += v.w;
                    *dst = o;
                }
            }
        }
    } else {
        const int ci = ci0 + wn * 32 + (lane & 31);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int co = co0 + wm * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
            const bool ok = co < a.cout && ci < a.cin;
            const size_t base = ((size_t)co * a.cin + ci) * 9;
#pragma unroll
            for (int t = 0; t < 9; ++t)
                if (ok) out[base + t] += acc[t][r];
        }
    }
}

// MODE 0: one workgroup = all of K of one (example, tile); 1: a K slice of it (accumulators to the
// workspace); 2: clip-weighted sum over a range of examples for one tile (dY scaled by f_i while it
// is staged; added to the accumulator, or to the workspace when the examples are split into ranges).
enum { C3_FULL = 0, C3_SLICED = 1, C3_WEIGHTED = 2 };

// One 16-byte piece of an LDS row as the MFMA operand it is: columns 8j .. 8j + 7 of a row, those at or beyond the row's end zero.
// `row`: the row's first byte; rows of 7 values: the dword it starts in, `bits` 16 where that is its high half.
template <int W, int J>
__device__ __forceinline__ uint4 c3_piece(const char *row, unsigned bits)
{
    constexpr int LEFT = W - 8 * J;                  // columns there are
    const char *p = row + 16 * J;
    if constexpr (W % 8 == 0) {
        return *reinterpret_cast<const uint4 *>(p);
    } else if constexpr (W % 2 != 0) {
        static_assert(W == 7, "one piece");
        const uint32_t *d = reinterpret_cast<const uint32_t *>(p);
        const uint32_t d0 = d[0], d1 = d[1], d2 = d[2], d3 = d[3];
        return make_uint4(funnel(d1, d0, bits), funnel(d2, d1, bits), funnel(d3, d2, bits), (bits ? d3 >> 16 : d3) & 0xFFFFu);
    } else if constexpr (W % 4 == 0) {
        const uint2 a = *reinterpret_cast<const uint2 *>(p);
        if constexpr (LEFT <= 4) return make_uint4(a.x, a.y, 0u, 0u);
        const uint2 b = *reinterpret_cast<const uint2 *>(p + 8);
        return make_uint4(a.x, a.y, b.x, b.y);
    } else {
        const uint32_t *d = reinterpret_cast<const uint32_t *>(p);
        return make_uint4(d[0], LEFT > 2 ? d[1] : 0u, LEFT > 4 ? d[2] : 0u, LEFT > 6 ? d[3] : 0u);
    }
}

// f(0), f(1), ... with constants
template <int... J, typename F>
__device__ __forceinline__ void c3_each(std::integer_sequence<int, J...>, F f) { (f(std::integral_constant<int, J>{}), ...); }

// the high (low) halves of two dwords side by side
__device__ __forceinline__ uint32_t c3_high(uint32_t second, uint32_t first) { return __builtin_amdgcn_perm(second, first, 0x07060302u); }
__device__ __forceinline__ uint32_t c3_low(uint32_t second, uint32_t first) { return __builtin_amdgcn_perm(second, first, 0x05040100u); }

// the three taps of kernel row kh
__device__ __forceinline__ void c3_taps(f32x16 (&acc)[9], int kh, uint4 dy, uint4 b0, uint4 b1, uint4 b2)
{
    const bf16x8 va = __builtin_bit_cast(bf16x8, dy);
    acc[kh * 3 + 0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, __builtin_bit_cast(bf16x8, b0), acc[kh * 3 + 0], 0, 0, 0);
    acc[kh * 3 + 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, __builtin_bit_cast(bf16x8, b1), acc[kh * 3 + 1], 0, 0, 0);
    acc[kh * 3 + 2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, __builtin_bit_cast(bf16x8, b2), acc[kh * 3 + 2], 0, 0, 0);
}

struct C3Row { unsigned at, bits; };       // where a row lies in LDS; rows of 7: how far into its first dword it starts

// What one workgroup does; `bid` is its number within its layer.
template <int W, int MODE, int STRIDE>
__device__ __forceinline__ void conv3x3_body(const C3Args &a, const unsigned bid)
{
    constexpr bool WEIGHTED = MODE == C3_WEIGHTED;
    using C = C3Cfg<W, STRIDE>;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    __shared__ float red[2][4];

    // consecutive hardware workgroup ids rotate over the 8 XCDs; give each XCD a run of
    // consecutive logical ids (the slices and tiles of the same examples share its L2)
    const int total = a.total, per_xcd = (total + 7) >> 3;
    const unsigned wg = (bid & 7u) * (unsigned)per_xcd + (bid >> 3);
    if ((int)wg >= total) return;
    // full: some rows of results, one after the other, of a tile; sliced: a slice of a row's tile; weighted: a range of examples of a tile
    const unsigned tiles = a.tiles_co * a.tiles_ci;
    const unsigned pick = MODE == C3_SLICED ? wg / (unsigned)a.ksplit : wg;
    const int group = __builtin_amdgcn_readfirstlane(pick / tiles), tile = __builtin_amdgcn_readfirstlane(pick % tiles);
    const int split = MODE == C3_FULL ? 0 : (WEIGHTED ? group : __builtin_amdgcn_readfirstlane(wg % (unsigned)a.ksplit));
    const int row0 = MODE == C3_FULL ? group * a.rows_per_wg : (WEIGHTED ? 0 : group);
    const int per_row = a.unit;                       // examples that add up to a row
    const int row1 = MODE == C3_FULL ? min(a.rows, row0 + a.rows_per_wg) : row0 + 1;
    const int i_first = WEIGHTED ? split * a.ex_per_split : row0 * a.unit + (MODE == C3_SLICED ? split * a.slice_ex : 0);
    const int i_last = WEIGHTED ? min(a.n, i_first + a.ex_per_split) : (MODE == C3_SLICED ? i_first + max(1, a.slice_ex) : row1 * a.unit);
    const int tco = __builtin_amdgcn_readfirstlane((unsigned)tile / (unsigned)a.tiles_ci), tci = tile - tco * a.tiles_ci;
    const int co0 = tco * 64, ci0 = tci * 64;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int half = lane >> 5;
    const int H = a.h, hin = a.hin;
    const int cin = a.cin, cout = a.cout;

    // Stages of an example: all of them, or a slice [k_begin, k_end).  A slice that starts inside the image has the stage before it as
    // well, which gives its first rows their upper neighbours in dY and no products; its last rows need the stage behind it of dY.
    const int n_stages = a.stages;
    const bool cut = MODE == C3_SLICED && a.slice_ex == 0;
    const int k_begin = cut ? split * a.stages_per_split : 0, k_end = cut ? min(n_stages, k_begin + a.stages_per_split) : n_stages;
    const int s_begin = STRIDE == 1 && k_begin > 0 ? k_begin - 1 : k_begin;
    const int a_end = min(n_stages, cut ? k_end + 1 : k_end);
    const int T = (i_last - i_first) * (k_end - s_begin);

    // ---- global -> LDS.  A bundle is X of a stage and dY of the next one of the stream; its wave instruction q moves pieces 64 q .. 64 q + 63 of X, or
    // from QX on of dY, and belongs to wave q % 4.
    // Pieces that hold nothing (padding, channels beyond the layer, rows below the image) fetch something of the same example, which
    // no product reads or no result shows.  The piece that an example's end cuts ends with it instead; the values move to their place
    // in LDS when they are there (mend).
    const int x_chan = hin * C::XW, a_chan = H * W;                // elements of a channel
    const unsigned x_ex = (unsigned)cin * (unsigned)x_chan, a_ex = (unsigned)cout * (unsigned)a_chan;         // and of an example: below 2^31
    struct Operand { int c0, channels, chan; unsigned ex; };
    const Operand ox{ci0, cin, x_chan, x_ex}, oa{co0, cout, a_chan, a_ex};
    struct Where { unsigned off, last; int cut; };                 // byte offset from the dword that the example's stage starts in; the same in an example's
                                                                   // last stage, and values that it was moved back by there
    // lane's piece of wave instruction q.  odd: the example starts in the high half of its first dword
    auto where = [&](auto is_x, int q, unsigned odd) {
        constexpr bool X = decltype(is_x)::value;
        constexpr unsigned pitch = X ? C::PX : C::PA;
        constexpr int run = X ? C::GB_X : C::GB_A;
        constexpr bool shifted = X ? C::ODD_X : C::ODD;
        const Operand &o = X ? ox : oa;
        const unsigned g = (unsigned)q / pitch, id = ((unsigned)q - g * pitch) * 64 + lane, ch = id / pitch, pc = id - ch * pitch;
        unsigned e = (unsigned)min(o.c0 + (int)ch, o.channels - 1) * (unsigned)o.chan + odd;
        const int pieces = shifted ? (run + 2 * (int)(e & 1u) + 15) / 16 : (X ? C::NX : C::NA);
        const int in_run = (int)g * run + min((int)pc, pieces - 1) * 16;
        if constexpr (shifted) e &= ~1u;
        Where w{2u * e + (unsigned)in_run, 0u, 0};
        const int before = (n_stages - 1) * C::SG * (run / 2);     // elements of a channel above its last stage
        const int over = (int)(e + (unsigned)(in_run / 2 + before + 8) - (o.ex + odd));
        w.last = w.off;
        if (in_run / 2 >= o.chan - before + (shifted ? 1 : 0) || over >= 8) {
            w.last = 0u;
        } else if (over > 0) {
            if (shifted && ((o.ex + odd) & 1)) {
                w.last = 0u;                                       // (an example of an odd number of values may end inside a dword: mend_odd)
            } else {
                w.last = w.off - 2u * (unsigned)over;
                w.cut = o.c0 + (int)ch < o.channels ? over : 0;
            }
        }
        return w;
    };
    typedef std::true_type is_x;
    typedef std::false_type is_a;
    // instruction u of this wave: always X, always dY, or either
    auto kind = [&](auto uu) {
        constexpr int u = decltype(uu)::value;
        return 4 * u + 3 < C::QX ? true : (4 * u >= C::QX ? false : wave + 4 * u < C::QX);
    };
    using bundle_t = std::make_integer_sequence<int, C::UB>;
    unsigned off[C::UB], off_last[C::UB];
    int x_cut = 0, a_cut = 0;                                      // at most one piece of a lane: 16 u + values
    c3_each(bundle_t{}, [&](auto uu) {
        constexpr int u = decltype(uu)::value;
        const int q = wave + 4 * u;
        const bool x = kind(uu);
        const Where w = x ? where(is_x{}, q, 0u) : where(is_a{}, min(q - C::QX, C::QA - 1), 0u);
        x_cut |= C::PARTIAL_X && x && w.cut ? 16 * u + w.cut : 0;
        a_cut |= C::PARTIAL_A && !x && w.cut && q < C::QX + C::QA ? 16 * u + w.cut : 0;
        off[u] = w.off;
        off_last[u] = w.last;
    });
    const bool x_cuts = C::PARTIAL_X && __ballot(x_cut != 0) != 0, a_cuts = C::PARTIAL_A && __ballot(a_cut != 0) != 0;
    const bool odd_x_ex = C::ODD_X && (x_ex & 1), odd_a_ex = C::ODD && (a_ex & 1);
    const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(size_t)lds);
    const unsigned long long x_ptr = reinterpret_cast<unsigned long long>(a.x), a_ptr = reinterpret_cast<unsigned long long>(a.dy);
    const int x_tab = a.x_tab, a_tab = a.dy_tab;
    // (by scalar loads: a wait for a vector load would wait for everything that is on its way to LDS)
    auto x_at = [&](int i) { return x_tab ? scalar_load<unsigned long long>(x_ptr, (size_t)i * x_tab) : x_ptr + 2ull * x_ex * (unsigned)i; };
    auto a_at = [&](int i) { return a_tab ? scalar_load<unsigned long long>(a_ptr, (size_t)i * a_tab) : a_ptr + 2ull * a_ex * (unsigned)i; };
    // The next bundle to fetch: stages (and their examples) of X and dY, where they come from and go.  Past the end of the stream the last stages are
    // fetched again, into slots that nobody reads any more: counts of what is on its way stay the same to the end.
    unsigned long long fx_base = x_at(i_first), fa_base = a_at(i_first);
    int fx_i = i_first, fx_s = s_begin, fa_i = i_first, fa_s = s_begin;
    unsigned fx_dst = lds0 + C::RING_X, fa_dst = lds0 + C::RING_A;
    auto fetch = [&](auto uu) {
        constexpr int u = decltype(uu)::value;
        const bool x = kind(uu);
        const int q = wave + 4 * u;
        const bool last = (x ? fx_s : fa_s) == n_stages - 1;
        const unsigned long long base = x ? fx_base : fa_base;
        const unsigned odd = (x ? odd_x_ex : odd_a_ex) ? (unsigned)(base >> 1) & 1u : 0u;
        const unsigned long long b = ((x ? C::ODD_X : C::ODD) ? base & ~3ull : base) + (unsigned)(x ? fx_s * (C::SG * C::GB_X) : fa_s * (C::SG * C::GB_A));
        unsigned dst = x ? fx_dst + q * 1024 : fa_dst + (q - C::QX) * 1024;
        if (4 * u + 3 >= C::QX + C::QA && q >= C::QX + C::QA) dst = lds0 + C::DUMP;
        unsigned o = last ? off_last[u] : off[u];
        if (odd) {
            const Where w = x ? where(is_x{}, q, 1u) : where(is_a{}, min(q - C::QX, C::QA - 1), 1u);
            o = last ? w.last : w.off;
        }
        lds_direct_16(b, o, dst);
    };
    auto fetched_x = [&]() {
        fx_dst = fx_dst == lds0 + C::RING_X + C::D * C::STAGE_X ? lds0 + C::RING_X : fx_dst + C::STAGE_X;
        if (++fx_s == k_end) {
            if (fx_i + 1 < i_last) { fx_s = s_begin; fx_base = x_at(++fx_i); }
            else --fx_s;
        }
    };
    auto fetched_a = [&]() {
        fa_dst = fa_dst == lds0 + C::RING_A + (C::D + 1) * C::STAGE_A ? lds0 + C::RING_A : fa_dst + C::STAGE_A;
        if (++fa_s == a_end) {
            if (fa_i + 1 < i_last) { fa_s = s_begin; fa_base = a_at(++fa_i); }
            else --fa_s;
        }
    };
    // by the lane that fetched the piece, after that has landed
    auto mend = [&](int gone, char *piece) {
        if (gone) {
            ulonglong2 *p = reinterpret_cast<ulonglong2 *>(piece);
            ulonglong2 v = *p;
            const int bits = 16 * gone;
            v.x = bits < 64 ? (v.x >> bits) | (v.y << (64 - bits)) : v.y >> (bits - 64);
            v.y = bits < 64 ? v.y >> bits : 0ull;
            *p = v;
        }
    };
    // the same in examples of an odd number of values: value by value from memory
    auto mend_odd = [&](auto which, unsigned long long base, char *stage) {
        constexpr bool X = decltype(which)::value;
        constexpr unsigned pitch = X ? C::PX : C::PA, run = (X ? C::GB_X : C::GB_A) / 2;
        const Operand &o = X ? ox : oa;
        const unsigned odd = (unsigned)(base >> 1) & 1u;
        const uint16_t *src = reinterpret_cast<const uint16_t *>(base & ~3ull);
        const unsigned end = o.ex + odd;
#pragma unroll 1
        for (int u = 0; u < C::UB; ++u) {
            const int q = wave + 4 * u - (X ? 0 : C::QX);
            if (q < 0 || q >= (X ? C::QX : C::QA)) continue;
            const unsigned g = (unsigned)q / pitch, id = ((unsigned)q - g * pitch) * 64 + lane, ch = id / pitch, pc = id - ch * pitch;
            if (o.c0 + (int)ch != o.channels - 1 || pc >= (unsigned)(X ? C::NX : C::NA)) continue;
            const unsigned e = (((unsigned)(o.channels - 1) * (unsigned)o.chan + odd) & ~1u) + (unsigned)(n_stages - 1) * (C::SG * run) + g * run + pc * 8;
            uint16_t *dst = reinterpret_cast<uint16_t *>(stage + q * 1024 + lane * 16);
#pragma unroll 1
            for (unsigned k = 0; k < 8 && e + k < end; ++k) dst[k] = src[e + k];
        }
    };
    // ---- what has to be done to the pieces of a stage that this wave fetched, once they have landed and before the barrier that shows them to the
    // others: a piece that an example's end cut; dY in the clip-weighted form: times the example's factor, rounded to bf16
    auto touch_x = [&](int i, int s, int slot) {
        if (C::PARTIAL_X && s == n_stages - 1 && i < i_last) {
            if (odd_x_ex) { if (ci0 + 64 >= cin) mend_odd(is_x{}, x_at(i), lds + C::RING_X + slot * C::STAGE_X); }
            else if (x_cuts) mend(x_cut & 15, lds + C::RING_X + slot * C::STAGE_X + (wave + 4 * (x_cut >> 4)) * 1024 + lane * 16);
        }
    };
    auto touch_a = [&](int i, int s, int slot) {
        if (C::PARTIAL_A && s == n_stages - 1 && i < i_last) {
            if (odd_a_ex) { if (co0 + 64 >= cout) mend_odd(is_a{}, a_at(i), lds + C::RING_A + slot * C::STAGE_A); }
            else if (a_cuts) mend(a_cut & 15, lds + C::RING_A + slot * C::STAGE_A + (wave + 4 * (a_cut >> 4) - C::QX) * 1024 + lane * 16);
        }
    };
    // the factors of 64 examples, one a lane
    const float *sqnorms = WEIGHTED ? a.group_sqnorm : nullptr;
    float factors = 1.0f;
    int factors_at = i_first;
    auto load_factors = [&](int from) {
        factors_at = from;
        if (sqnorms) factors = clip_factor(sqnorms[min(from + lane, i_last - 1)], a.clip_c);
    };
    constexpr int US = C::QX / 4;                     // a wave's first instruction that may be dY's
    struct Scaled { uint4 v[C::UB - US]; };
    auto scale_at = [&](auto uu, int slot) {          // where what instruction u fetched lies, if it is dY's
        constexpr int u = decltype(uu)::value;
        const int q = wave + 4 * u;
        const bool here = (4 * u >= C::QX || q >= C::QX) && (4 * u + 3 < C::QX + C::QA || q < C::QX + C::QA);
        return here ? lds + C::RING_A + slot * C::STAGE_A + (q - C::QX) * 1024 + lane * 16 : lds + C::DUMP + lane * 16;
    };
    auto scale_read = [&](int slot) {
        Scaled o;
        c3_each(std::make_integer_sequence<int, C::UB - US>{}, [&](auto k) {
            o.v[k.value] = *reinterpret_cast<const uint4 *>(scale_at(std::integral_constant<int, US + decltype(k)::value>{}, slot));
        });
        return o;
    };
    auto scale_write = [&](Scaled &o, float f, int slot) {
        c3_each(std::make_integer_sequence<int, C::UB - US>{}, [&](auto k) {
            uint32_t t[4] = {o.v[k.value].x, o.v[k.value].y, o.v[k.value].z, o.v[k.value].w};
            scale_regs<true, 4>(t, f);
            *reinterpret_cast<uint4 *>(scale_at(std::integral_constant<int, US + decltype(k)::value>{}, slot)) = make_uint4(t[0], t[1], t[2], t[3]);
        });
    };
    static_assert(!WEIGHTED || C::DUMP + 1024 <= C::LDS, "a place for what is not dY's");

    f32x16 acc[9];
    auto clear = [&]() {
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[t][r] = 0.0f;
    };

    // ---- dY of stage 0, then bundles 0 .. D - 1; bundle t + D is issued during stage t, into what stage t - 1 has left
    c3_each(bundle_t{}, [&](auto uu) {
        if (!kind(uu) && wave + 4 * decltype(uu)::value < C::QX + C::QA) fetch(uu);
    });
    fetched_a();
#pragma unroll
    for (int k = 0; k < C::D; ++k) {
        c3_each(bundle_t{}, fetch);
        fetched_x();
        fetched_a();
    }
    clear();
    if (threadIdx.x < C::ZEROS / 16) *reinterpret_cast<uint4 *>(lds + threadIdx.x * 16) = make_uint4(0u, 0u, 0u, 0u);

    // operand reads: lane -> channel (lane & 31) of its 32, and the upper or lower one of a pair of rows
    const unsigned lane_x = (unsigned)((wn * 32 + (lane & 31)) * (C::PX * 16)), lane_a = (unsigned)((wm * 32 + (lane & 31)) * (C::PA * 16));
    const int x_odd_chan = C::ODD_X ? ((ci0 + wn * 32 + (lane & 31)) * x_chan) & 1 : 0;
    const int a_odd_chan = C::ODD ? ((co0 + wm * 32 + (lane & 31)) * a_chan) & 1 : 0;

    int ci = i_first, cs = s_begin, x_slot = 0, a_slot = 0;        // the stage whose products run
    int na_i = i_first, na_s = s_begin, na_slot = 0;               // the stage of dY that is touched next
    auto touched_a = [&]() {
        na_slot = na_slot == C::D + 1 ? 0 : na_slot + 1;
        if (++na_s == a_end) { na_s = s_begin; ++na_i; }
    };
    auto factor_of = [&](int i) {
        if (i - factors_at >= 64) load_factors(i);
        return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, factors), i - factors_at));
    };
    auto slot_after = [](int slot, int slots) { return slot + 1 == slots ? 0 : slot + 1; };
    // this lane's one of rows r and r + 1 of dY, counted from the first one of the stage at hand, of which the image has `below` from there on:
    // those below it are zeros
    int below = 0;
    unsigned odd_x = 0, odd_a = 0, xs = 0, as = 0, an = 0;
    auto row_a = [&](int r) {
        C3Row o{0u, 0u};
        if constexpr (C::ODD) {
            const int lr = r + half;
            const unsigned e = odd_a + 7u * (unsigned)(lr < C::RPS ? lr : 0);
            o.at = (lr < C::RPS ? as : an) + (e >> 1) * 4u;
            o.bits = (e & 1u) * 16u;
        } else {
            o.at = half ? (r + 1 < C::RPS ? as + C::at_a(r + 1) : an) : as + C::at_a(r);
        }
        if (r + 1 >= below && r + half >= below) o.at = 0u;
        return o;
    };
    auto row_x = [&](int r) {                         // stride 1: rows r and r + 1 of X; stride 2: 2 r and 2 r + 2
        C3Row o{0u, 0u};
        if constexpr (C::ODD_X) {
            const unsigned e = odd_x + 7u * (unsigned)(r + half);
            o.at = xs + (e >> 1) * 4u;
            o.bits = (e & 1u) * 16u;
        } else {
            o.at = xs + (half ? C::at_x(STRIDE * (r + 1)) : C::at_x(STRIDE * r));
        }
        if (r + 1 >= below && r + half >= below) o.at = 0u;
        return o;
    };
    auto begin = [&]() {                              // a stage begins: everyone's pieces are there, those of the stage before have been read
        __syncthreads();
        odd_x = C::ODD_X ? (unsigned)(x_odd_chan + (odd_x_ex ? (int)((x_at(ci) >> 1) & 1) : 0)) & 1u : 0u;
        odd_a = C::ODD ? (unsigned)(a_odd_chan + (odd_a_ex ? (int)((a_at(ci) >> 1) & 1) : 0)) & 1u : 0u;
        xs = C::RING_X + x_slot * C::STAGE_X + lane_x;
        as = C::RING_A + a_slot * C::STAGE_A + lane_a;
        an = C::RING_A + slot_after(a_slot, C::D + 2) * C::STAGE_A + lane_a;
        below = H - cs * C::RPS;
    };
    int stores = 0;                                   // for how many more waits the stores of a row of results are younger than what is waited for
    // this wave's pieces of what the next stage reads (bundle t + 1) have landed: as many bundles as were issued after it are on their way
    auto landed = [&](auto young) {
        constexpr int n = decltype(young)::value * C::UB;
        if (MODE == C3_FULL && stores > 0) { wait_vmcnt<n + 48 < 63 ? n + 48 : 63>(); --stores; }
        else wait_vmcnt<n>();
    };
    Scaled scaled;
    float f = 1.0f;
    auto prepare = [&](auto young) {
        landed(young);
        touch_a(na_i, na_s, na_slot);
        touch_x(ci + (cs + 1 == k_end ? 1 : 0), cs + 1 == k_end ? s_begin : cs + 1, slot_after(x_slot, C::D + 1));
        if constexpr (WEIGHTED) {
            scaled = scale_read(na_slot);
            f = factor_of(min(na_i, i_last - 1));
        }
    };
    auto prepared = [&]() {
        if constexpr (WEIGHTED) scale_write(scaled, f, na_slot);
        touched_a();
    };
    auto leave = [&]() {
        x_slot = slot_after(x_slot, C::D + 1);
        a_slot = slot_after(a_slot, C::D + 2);
        if (++cs == k_end) { cs = s_begin; ++ci; }
    };
    using pieces_t = std::make_integer_sequence<int, C::PPR>;
    uint4 carry[STRIDE == 1 ? C::PPR : 1];            // dY rows 2 q - 1 and 2 q, from the pair of rows before
    auto carry_from = [&](const C3Row o) {
        c3_each(pieces_t{}, [&](auto j) { if constexpr (STRIDE == 1) carry[j.value] = c3_piece<W, j.value>(lds + o.at, o.bits); });
    };
    // the operands of a K step: a piece of the rows of X and of both pairs of rows of dY
    struct Ops { uint4 x[STRIDE == 1 ? 1 : 4], a0, a1; };
    struct Rows { C3Row x, y0, y1; };
    auto rows_of = [&](int p) { return Rows{row_x(2 * p), row_a(2 * p + 1), row_a(2 * p)}; };
    auto load = [&](const Rows &r, auto jj) {
        constexpr int j = decltype(jj)::value;
        Ops o;
        if constexpr (STRIDE == 1) {
            o.x[0] = c3_piece<W, j>(lds + r.x.at, r.x.bits);
        } else {
#pragma unroll
            for (int k = 0; k < 2; ++k) {             // row 2 oh of X, then 2 oh + 1
                const char *row = lds + r.x.at + (r.x.at ? k * C::ROW_X : 0);
                o.x[2 * k] = c3_piece<C::XW, 2 * j>(row, 0u);
                if constexpr (16 * j + 8 < C::XW) o.x[2 * k + 1] = c3_piece<C::XW, 2 * j + 1>(row, 0u);
                else o.x[2 * k + 1] = make_uint4(0u, 0u, 0u, 0u);
            }
        }
        o.a1 = c3_piece<W, j>(lds + r.y1.at, r.y1.bits);
        o.a0 = c3_piece<W, j>(lds + r.y0.at, r.y0.bits);
        return o;
    };
    // Work that is not products is dealt out between them, three MFMAs at a time, so that the matrix units have something meanwhile: the next bundle's
    // loads in the first half of a stage's first pair of rows, then the wait for the bundle before and the factors.
    constexpr int SLOTS = 3 * C::PPR;
    auto between = [&](auto kk) {
        constexpr int k = decltype(kk)::value;
        c3_each(bundle_t{}, [&](auto uu) { if constexpr (decltype(uu)::value * ((SLOTS + 1) / 2) / C::UB == k) fetch(uu); });
        if constexpr (k == (SLOTS - 1) / 2) { fetched_x(); fetched_a(); }
        if constexpr (C::D > 1 && k == (SLOTS + 1) / 2) prepare(std::integral_constant<int, C::D - 1>{});
        if constexpr (C::D > 1 && k == SLOTS - 1) prepared();
    };

    // ---- the first bundle
    if constexpr (WEIGHTED) load_factors(i_first);
    wait_vmcnt<(C::D - 1) * C::UB>();
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        touch_a(na_i, na_s, na_slot);
        if constexpr (WEIGHTED) {
            Scaled o = scale_read(na_slot);
            scale_write(o, factor_of(min(na_i, i_last - 1)), na_slot);
        }
        touched_a();
    }
    touch_x(ci, cs, 0);
    int t = 0;
    if (STRIDE == 1 && cut && s_begin < k_begin) {    // the stage above a slice: its last row and the next stage's first
        begin();
        carry_from(row_a(C::RPS - 1));
        c3_each(bundle_t{}, fetch);
        fetched_x();
        fetched_a();
        prepare(std::integral_constant<int, C::D - 1>{});
        prepared();
        leave();
        ++t;
    }
    int row = row0, in_row = 0, half_red = 0;
    for (; t < T; ++t) {
        begin();
        if (MODE == C3_FULL && row > row0 && in_row == 0 && cs == s_begin && threadIdx.x == 0) {       // (the barrier has just shown the waves' shares)
            const float *r = red[half_red ^ 1];
            a.partials[(row - 1) * tiles + tile] = r[0] + r[1] + r[2] + r[3];
        }
        if constexpr (STRIDE == 1) {
            // the pair above the first one: row -1 is zeros, row 0 this stage's first
            if (cs == 0) carry_from(half ? C3Row{as + (odd_a >> 1) * 4u, odd_a * 16u} : C3Row{0u, 0u});
        }
        Rows rows = rows_of(0);
        Ops next = load(rows, std::integral_constant<int, 0>{});
        c3_each(std::make_integer_sequence<int, C::PAIRS>{}, [&](auto pp) {
            constexpr int p = decltype(pp)::value;
            if (p > 0 && 2 * p >= below) return;      // uniform
            uint32_t left[2] = {0u, 0u};              // the two columns before the piece
            const Rows rows2 = p + 1 < C::PAIRS ? rows_of(p + 1) : rows;
            c3_each(pieces_t{}, [&](auto jj) {
                constexpr int j = decltype(jj)::value;
                auto gap = [&](auto g) {
                    if constexpr (p == 0) between(std::integral_constant<int, 3 * j + decltype(g)::value>{});
                };
                // the operands of the step after this one are read while its products run
                const Ops o = next;
                if constexpr (j + 1 < C::PPR) next = load(rows, std::integral_constant<int, j + 1>{});
                else if constexpr (p + 1 < C::PAIRS) next = load(rows2, std::integral_constant<int, 0>{});
                if constexpr (STRIDE == 1) {
                    const uint4 b1 = o.x[0];
                    const uint32_t right = j + 1 < C::PPR ? next.x[0].x : 0u;
                    // the same run of columns one to the left and one to the right
                    const uint32_t o0 = funnel(b1.x, left[0], 16), o1 = funnel(b1.y, b1.x, 16), o2 = funnel(b1.z, b1.y, 16), o3 = funnel(b1.w, b1.z, 16),
                                   o4 = funnel(right, b1.w, 16);
                    const uint4 b0 = make_uint4(o0, o1, o2, o3), b2 = make_uint4(o1, o2, o3, o4);
                    c3_taps(acc, 1, o.a1, b0, b1, b2);
                    gap(std::integral_constant<int, 0>{});
                    c3_taps(acc, 0, o.a0, b0, b1, b2);
                    gap(std::integral_constant<int, 1>{});
                    c3_taps(acc, 2, carry[j], b0, b1, b2);
                    gap(std::integral_constant<int, 2>{});
                    carry[j] = o.a0;
                    left[0] = b1.w;
                } else {
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        const uint4 v = o.x[2 * k], w = o.x[2 * k + 1];
                        const uint4 b0 = make_uint4(c3_high(v.x, left[k]), c3_high(v.z, v.y), c3_high(w.x, v.w), c3_high(w.z, w.y)),       // X[2 ow - 1]
                                    b1 = make_uint4(c3_low(v.y, v.x), c3_low(v.w, v.z), c3_low(w.y, w.x), c3_low(w.w, w.z)),             // X[2 ow]
                                    b2 = make_uint4(c3_high(v.y, v.x), c3_high(v.w, v.z), c3_high(w.y, w.x), c3_high(w.w, w.z));         // X[2 ow + 1]
                        left[k] = w.w;
                        if (k == 0) {
                            c3_taps(acc, 1, o.a1, b0, b1, b2);
                            gap(std::integral_constant<int, 0>{});
                        } else {
                            c3_taps(acc, 2, o.a1, b0, b1, b2);
                            gap(std::integral_constant<int, 1>{});
                            c3_taps(acc, 0, o.a0, b0, b1, b2);
                            gap(std::integral_constant<int, 2>{});
                        }
                    }
                }
            });
            rows = rows2;
        });
        if constexpr (C::D == 1) {
            prepare(std::integral_constant<int, 0>{});
            prepared();
        }
        leave();
        if constexpr (MODE == C3_FULL) {
            if (cs == s_begin && ++in_row == per_row) {
                // a row of results: its share of the norm, its gradient; the next row's stages are on their way meanwhile
                in_row = 0;
                const float ss = c3_squares(acc, a, co0, ci0, wm, wn, lane);
                if (lane == 63) red[half_red][wave] = ss;
                half_red ^= 1;
                if (a.out_w) {
                    if (!C::STREAMS) { wait_vmcnt<0>(); __syncthreads(); }       // (one row alone: the rings are free)
                    const bool all = c3_store(acc, a, row, co0, ci0, wm, wn, lane, reinterpret_cast<float *>(lds + C::STORE) + wave * (2 * C3_RP));
                    stores = all ? C::D - 1 : 0;
                }
                ++row;
                clear();
            }
        }
    }
    wait_vmcnt<0>();                                  // (the stages that were fetched again)

    if constexpr (MODE == C3_FULL) {
        __syncthreads();
        if (threadIdx.x == 0) {
            const float *r = red[half_red ^ 1];
            a.partials[(row - 1) * tiles + tile] = r[0] + r[1] + r[2] + r[3];
        }
    } else if (WEIGHTED && a.ksplit == 1) {
        c3_add_to_accumulator(acc, a, co0, ci0, wm, wn, lane, lds);
    } else {
        const size_t slot = (size_t)(WEIGHTED ? (unsigned)tile : pick) * a.ksplit + split;
        float *mine_part = a.ws_part + slot * (9 * 16 * C3_THREADS);
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) mine_part[(t * 16 + r) * C3_THREADS + threadIdx.x] = acc[t][r];
    }
}

template <int W, int MODE, int STRIDE>
__global__ void __launch_bounds__(C3_THREADS, 2) conv3x3_kernel(const Grouped<C3Args> grp)
{
    unsigned bid;
    const C3Args &a = grp.a[group_pick(grp, bid)];
    conv3x3_body<W, MODE, STRIDE>(a, bid);
}

// The variants a ResNet of 224 x 224 images needs, in ONE kernel that dispatches on the layer's variant, so that all
// 3x3 layers of a batch call share a launch: at most four kernels run at a time on the chip, and the few workgroups of
// a narrow layer cost none of those four when they sit inside a wide launch.  Two sets (a body that is not needed is
// not compiled in: registers and LDS are those of the largest body of a set): set 0 for micro-steps of one or two
// examples (sliced variants: every launch is a few dozen workgroups and costs more than its work), set 1, every variant,
// for larger micro-steps.  The finely sliced 56-wide body, which micro-steps of 32 examples take when clip units of four
// are formed, fits in set 1's registers without a spill: ResNet-50's step with such units 3.70 -> 3.68 ms against a launch
// of its own.
enum { C3_ANY_56_SLICED = 0, C3_ANY_28_SLICED, C3_ANY_28_FULL, C3_ANY_14_FULL, C3_ANY_14_SLICED, C3_ANY_7_FULL,
       C3_ANY_14S2_SLICED, C3_ANY_14S2_FULL, C3_ANY_7S2_FULL, C3_ANY_56_FULL, C3_ANY_28_WEIGHTED, C3_ANY_14_WEIGHTED,
       C3_ANY_7_WEIGHTED, C3_ANY_28S2_FULL, C3_ANY_28S2_SLICED, C3_ANY_COUNT };

constexpr bool c3_any_in_set(int variant, int set)
{
    if (variant < 0) return false;
    return set == 1 || variant <= C3_ANY_7S2_FULL;
}

template <int SET>
__global__ void __launch_bounds__(C3_THREADS, 2) conv3x3_any_kernel(const Grouped<C3Args> grp)
{
    unsigned bid;
    const C3Args &a = grp.a[group_pick(grp, bid)];
    const int v = __builtin_amdgcn_readfirstlane(a.variant);
#define C3_ANY_CASE(ID, W, MODE, STRIDE)                                                  \
    if constexpr (c3_any_in_set(ID, SET)) {                                               \
        if (v == ID) { conv3x3_body<W, MODE, STRIDE>(a, bid); return; }               \
    }
    C3_ANY_CASE(C3_ANY_56_SLICED, 56, C3_SLICED, 1)
    C3_ANY_CASE(C3_ANY_28_SLICED, 28, C3_SLICED, 1)
    C3_ANY_CASE(C3_ANY_28_FULL, 28, C3_FULL, 1)
    C3_ANY_CASE(C3_ANY_14_FULL, 14, C3_FULL, 1)
    C3_ANY_CASE(C3_ANY_14_SLICED, 14, C3_SLICED, 1)
    C3_ANY_CASE(C3_ANY_7_FULL, 7, C3_FULL, 1)
    C3_ANY_CASE(C3_ANY_14S2_SLICED, 14, C3_SLICED, 2)
    C3_ANY_CASE(C3_ANY_14S2_FULL, 14, C3_FULL, 2)
    C3_ANY_CASE(C3_ANY_7S2_FULL, 7, C3_FULL, 2)
    C3_ANY_CASE(C3_ANY_56_FULL, 56, C3_FULL, 1)
    C3_ANY_CASE(C3_ANY_28_WEIGHTED, 28, C3_WEIGHTED, 1)
    C3_ANY_CASE(C3_ANY_14_WEIGHTED, 14, C3_WEIGHTED, 1)
    C3_ANY_CASE(C3_ANY_7_WEIGHTED, 7, C3_WEIGHTED, 1)
    C3_ANY_CASE(C3_ANY_28S2_FULL, 28, C3_FULL, 2)
    C3_ANY_CASE(C3_ANY_28S2_SLICED, 28, C3_SLICED, 2)
#undef C3_ANY_CASE
}

constexpr int c3_max(int a, int b) { return a > b ? a : b; }
constexpr int C3_ANY_LDS = c3_max(c3_max(c3_max(C3Cfg<56, 1>::LDS, C3Cfg<28, 1>::LDS), c3_max(C3Cfg<14, 1>::LDS, C3Cfg<7, 1>::LDS)),
                                  c3_max(C3Cfg<28, 2>::LDS, c3_max(C3Cfg<14, 2>::LDS, C3Cfg<7, 2>::LDS)));

template <int W, int MODE, int STRIDE> constexpr int c3_any_variant()
{
    if (STRIDE == 1) {
        if (W == 56) return MODE == C3_SLICED ? C3_ANY_56_SLICED : (MODE == C3_FULL ? C3_ANY_56_FULL : -1);
        if (W == 28) return MODE == C3_SLICED ? C3_ANY_28_SLICED : (MODE == C3_FULL ? C3_ANY_28_FULL : C3_ANY_28_WEIGHTED);
        if (W == 14) return MODE == C3_SLICED ? C3_ANY_14_SLICED : (MODE == C3_FULL ? C3_ANY_14_FULL : C3_ANY_14_WEIGHTED);
        if (W == 7) return MODE == C3_FULL ? C3_ANY_7_FULL : (MODE == C3_WEIGHTED ? C3_ANY_7_WEIGHTED : -1);
        return -1;
    }
    if (W == 14) return MODE == C3_SLICED ? C3_ANY_14S2_SLICED : (MODE == C3_FULL ? C3_ANY_14S2_FULL : -1);
    if (W == 28) return MODE == C3_SLICED ? C3_ANY_28S2_SLICED : (MODE == C3_FULL ? C3_ANY_28S2_FULL : -1);
    if (W == 7 && MODE == C3_FULL) return C3_ANY_7S2_FULL;
    return -1;
}

// Slices of one (example, tile) meet here.  The sum is elementwise, so it is spread over many
// small workgroups: one per (example, tile, tap t, four of the tap's sixteen accumulator
// registers); each thread adds its four values in slice order with eight slices in flight, then
// squares / stores them like the unsliced epilogue.
constexpr int C3_FIX_R = 4, C3_FIX_PARTS = 16 / C3_FIX_R;

template <bool WEIGHTED>
__global__ void __launch_bounds__(C3_THREADS) conv3x3_fixup_kernel(const Grouped<C3Args> grp)
{
    __shared__ float red[4];
    unsigned bid;
    const C3Args &a = grp.a[group_pick(grp, bid)];
    const int tiles = a.tiles_co * a.tiles_ci;
    const int part = bid % C3_FIX_PARTS;
    const int t = (bid / C3_FIX_PARTS) % 9;
    const int unit = bid / (C3_FIX_PARTS * 9);                    // (example, tile); weighted: tile
    const int i = WEIGHTED ? 0 : unit / tiles, tile = unit - i * tiles;
    const int tco = tile / a.tiles_ci, tci = tile - tco * a.tiles_ci;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const size_t slice = (size_t)9 * 16 * C3_THREADS;
    const float *base = a.ws_part + (size_t)unit * a.ksplit * slice + (size_t)(t * 16 + part * C3_FIX_R) * C3_THREADS + threadIdx.x;
    float v[C3_FIX_R];
#pragma unroll
    for (int r = 0; r < C3_FIX_R; ++r) v[r] = 0.0f;
    int s = 0;
    for (; s + 8 <= a.ksplit; s += 8) {
        float tmp[8][C3_FIX_R];
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
            for (int r = 0; r < C3_FIX_R; ++r) tmp[u][r] = base[(size_t)(s + u) * slice + r * C3_THREADS];
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
            for (int r = 0; r < C3_FIX_R; ++r) v[r] += tmp[u][r];
    }
    for (; s < a.ksplit; ++s) {
        float tmp[C3_FIX_R];
#pragma unroll
        for (int r = 0; r < C3_FIX_R; ++r) tmp[r] = base[(size_t)s * slice + r * C3_THREADS];
#pragma unroll
        for (int r = 0; r < C3_FIX_R; ++r) v[r] += tmp[r];
    }
    const int ci = tci * 64 + wn * 32 + (lane & 31);
    float *out = WEIGHTED ? a.out_w : a.out_w + (size_t)i * a.out_stride;
    float ss = 0.0f;
#pragma unroll
    for (int rr = 0; rr < C3_FIX_R; ++rr) {
        const int r = part * C3_FIX_R + rr;
        const int co = tco * 64 + wm * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
        const bool ok = co < a.cout && ci < a.cin;
        const size_t idx = ((size_t)co * a.cin + ci) * 9 + t;
        if constexpr (WEIGHTED) {
            if (ok) out[idx] += v[rr];
        } else {
            if (ok) ss += v[rr] * v[rr];
            if (a.out_w && ok) out[idx] = v[rr];
        }
    }
    if constexpr (!WEIGHTED) {
        const float tot = block_sum<4>(ss, red);
        if (threadIdx.x == 0) a.partials[bid] = tot;
    }
}

// ------------------------------------------------------------------------------------ host

struct C3Plan {
    int stage_rows;                    // output rows of a stage (C3Cfg)
    int tiles_co, tiles_ci, chunks;    // chunks: a unit of work that slices of K are planned in, about 224 output positions (not what the kernel walks in)
    int ksplit, stages_per_split;      // per-example modes: K slices; weighted: example ranges
    int ex_per_split;                  // weighted
    int slice_ex;                      // per-example modes: examples per slice of a clipping unit, or 0
    int rows_per_wg;                   // per-example modes, not sliced: rows of results per workgroup
};

int rows_of_width(int ow, int stride)
{
    const int owp = (ow + 7) / 8 * 8;
    if (stride == 2) return owp == 16 ? 5 : (owp == 32 ? 3 : 8);
    return owp == 8 ? 8 : 224 / owp;
}

// plans inside a batch call (the launch is shared with other layers) differ; workspace sizes cover both
thread_local int c3_forced_crowd = -1;
int c3_plan_crowd() { return c3_forced_crowd >= 0 ? c3_forced_crowd : crowd_hint(); }
int c3_launch_crowd() { return c3_forced_crowd >= 0 ? c3_forced_crowd : crowd3_hint(); }         // of this kernel's launch alone

C3Plan c3_plan_slices(const Geo &g, int mode)
{
    C3Plan p;
    p.tiles_co = (g.cout + 63) / 64;
    p.tiles_ci = (g.cin + 63) / 64;
    p.chunks = (g.oh + rows_of_width(g.ow, g.stride) - 1) / rows_of_width(g.ow, g.stride);
    p.ksplit = 1;
    p.stage_rows = c3_rows_per_stage(g.ow, g.stride);
    p.stages_per_split = 0;
    p.ex_per_split = g.n;
    p.slice_ex = 0;
    p.rows_per_wg = 1;
    const long long tiles = (long long)p.tiles_co * p.tiles_ci;
    // inside a batch call: chunks per workgroup to plan for (a chunk here is about eight 128x128x64 chunks of work, but
    // slices cost a second pass over partial blocks: only very long walks are cut)
    int crowd = c3_plan_crowd(), tgt = crowd ? (crowd / 2 > 1 ? crowd / 2 : 1) : 0;
    // a layer that is small even chunk by chunk (micro-steps of one or two examples): a chunk per workgroup, the
    // walk of a workgroup is what such a launch waits for
    if (crowd && mode != MODE_WEIGHTED && (long long)g.n * tiles * p.chunks <= 128) tgt = 1;
    if (mode == MODE_WEIGHTED) {
        // Example ranges, partial blocks in the workspace kept below ~100 MB.  A layer alone: about 256 workgroups.
        long long want = (256 + tiles - 1) / tiles;
        if (crowd) {
            // In a launch shared with other layers ranges are long: without partial blocks and slice-sum launch a narrow launch that the other streams
            // of a replayed step overlap beats one that fills the chip (ResNet-50, 32 examples, crowd 32: one range per tile 6690 us a step, two
            // for the 14-wide layers, 16 tiles, 6850, four 7030).  But no longer than the launch is worth: `crowd` (of this kernel's launch, not of the whole
            // call, whose other kernels wait for it) grows with its work, and a walk has about four stages per unit of it (that range of 32 examples
            // is 128 stages), and 48 chunks.  A layer of few tiles brings 32 workgroups, and so does one on 7 x 7 or 8 x 8 maps, whose stages take longest.
            // Two such layers by themselves, us, with the 48 chunks alone / so: 64 -> 64 at 14 x 14, 48 examples, 241 / 25; at 28 x 28, 32, 169 / 32; 256 -> 256 at
            // 14 x 14, 48, 240 / 78; four of 128 -> 128 at 28 x 28, 16, 129 / 62; beside another kernel's layer 256 -> 64 at 7 x 7, 32, 538 / 484 the two.
            // (Sixteen tiles and more on larger maps keep their one range in small launches too: 256 -> 256 at 14 x 14, 4 examples, 33; two ranges 40.)
            const long long stages = (long long)g.n * ((g.oh + p.stage_rows - 1) / p.stage_rows);
            crowd = c3_launch_crowd();
            want = std::max((stages + 4 * crowd - 1) / (4 * crowd), ((long long)g.n * p.chunks + 47) / 48);
            if ((tiles <= 8 || g.ow <= 8) && want * tiles < 32) want = (32 + tiles - 1) / tiles;
        }
        const long long cap = (long long)(96.0e6 / (4.0 * 9 * 16 * C3_THREADS * (double)tiles));
        if (want > cap) want = cap;
        if (want > g.n) want = g.n;
        if (want < 1) want = 1;
        p.ex_per_split = (int)((g.n + want - 1) / want);
        p.ksplit = (g.n + p.ex_per_split - 1) / p.ex_per_split;
        return p;
    }
    const long long units = (long long)(g.n / g.unit) * tiles;
    if (g.unit > 1) {
        // clipping units are sliced by examples; few blocks that walk long are cut too (ResNet-50, 8 units of 4 examples: the three
        // 56-wide layers are 24 blocks of 56 chunks, 0.6 ms where the rest of the phase needs as long together)
        const long long walk = (long long)p.chunks * g.unit;
        long long want = 1;
        if (crowd ? walk > 3 * tgt : units < 128) want = crowd ? (walk + tgt - 1) / tgt : (128 + units - 1) / units;
        if (units < 64 && walk >= 16 && want < 64 / units) want = 64 / units;
        int k = 1;
        while (k < g.unit && (k < want || g.unit % k)) ++k;                       // slices of equal size
        if (k > 1) { p.ksplit = k; p.slice_ex = g.unit / k; }
        return p;
    }
    // (measured in the replayed step, where other streams fill the compute units a narrow launch leaves free: the 56-wide
    // layers run 14 chunks per workgroup unsliced rather than in three slices + a slice-sum launch)
    if (p.chunks > 1 && (crowd ? p.chunks > 3 * tgt : units < 128)) {
        long long want = (128 + units - 1) / units;
        if (crowd) want = (p.chunks + tgt - 1) / tgt;
        if (want > p.chunks) want = p.chunks;
        const int stages = (g.oh + p.stage_rows - 1) / p.stage_rows;
        if (want > stages) want = stages;
        p.stages_per_split = (int)((stages + want - 1) / want);
        p.ksplit = (stages + p.stages_per_split - 1) / p.stages_per_split;
    }
    return p;
}

C3Plan c3_plan(const Geo &g, int mode)
{
    C3Plan p = c3_plan_slices(g, mode);
    if (mode == MODE_WEIGHTED || p.ksplit > 1 || !c3_streams(g.ow, g.stride)) return p;
    // Starting a workgroup costs as much as three stages: one that walks fewer than sixteen takes several rows of results in a row, as long as the launch (of
    // which this layer's work is a share) has two workgroups left for every compute unit, and a layer of a shared one a workgroup for every second one.  Where they are
    // stored, at most four: of more the last workgroups' stores are left alone at the end (512 -> 512 at 7 x 7, us for at most 16 / 8 / 4 / 2 / 1: two layers of 48
    // examples 205 / 189 / 183 / 178 / 187, four of 8 59 / 59 / 59 / 63 / 71, one of 128 249 / 242 / 237 / 233 / 249, of 32 60 / 60 / 60 / 64 / 69; 512 -> 64 at
    // 8 x 8, 48 examples, beside a 1x1 layer, 3 / 1, 38 / 31).
    const long long stages = (long long)g.unit * ((g.oh + p.stage_rows - 1) / p.stage_rows), rows = g.n / g.unit, tiles = (long long)p.tiles_co * p.tiles_ci;
    long long k = 16 / stages, most = rows * tiles / 512;
    if (c3_launch_crowd()) most = std::min(rows * tiles / 128, (long long)((double)(rows * tiles) * std::max(1.0, macs3_hint() / conv_macs(g)) / 512.0));
    if (k > most) k = most;
    if (k > rows) k = rows;
    if (mode == MODE_MATERIALISE && k > 4) k = 4;
    if (k > 1) p.rows_per_wg = (int)k;
    return p;
}

size_t c3_align16(size_t b) { return (b + 15) & ~(size_t)15; }

// partial squared norms per (example, tile): one, or one per fixup workgroup when K is sliced
size_t c3_partials_per_unit(const C3Plan &p) { return p.ksplit > 1 ? 9 * C3_FIX_PARTS : 1; }

template <int W, int MODE, int STRIDE>
dp_status c3_launch_mode(const C3Args &a, unsigned blocks, hipStream_t s)
{
    using C = C3Cfg<W, STRIDE>;
    constexpr int any = c3_any_variant<W, MODE, STRIDE>();
    const int set = fuse_hint() == 2 ? 0 : 1;
    if (fuse_hint() && (set == 0 ? c3_any_in_set(any, 0) : c3_any_in_set(any, 1))) {
        // inside a batch call: every row width in one launch
        const void *fn = set == 0 ? reinterpret_cast<const void *>(&conv3x3_any_kernel<0>) : reinterpret_cast<const void *>(&conv3x3_any_kernel<1>);
        static std::atomic<bool> any_attr_done[2];
        if (!any_attr_done[set].load()) {
            if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, C3_ANY_LDS) != hipSuccess)
                return fail(DP_ERR_DEVICE, "conv3x3: cannot reserve %d bytes of LDS", C3_ANY_LDS);
            any_attr_done[set].store(true);
        }
        C3Args b = a;
        b.variant = any;
        return submit_main<C3Args>(fn, b, blocks, C3_THREADS, C3_ANY_LDS, s, "conv3x3");
    }
    const void *fn = reinterpret_cast<const void *>(&conv3x3_kernel<W, MODE, STRIDE>);
    static std::atomic<bool> attr_done;              // zero-initialised; setting the attribute twice is harmless
    if (!attr_done.load()) {
        if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS) != hipSuccess)
            return fail(DP_ERR_DEVICE, "conv3x3: cannot reserve %d bytes of LDS", C::LDS);
        attr_done.store(true);
    }
    return submit_main<C3Args>(fn, a, blocks, C3_THREADS, C::LDS, s, "conv3x3");
}

template <int W, int STRIDE>
dp_status c3_launch_w(const C3Args &a, bool weighted, unsigned blocks, hipStream_t s)
{
    if constexpr (STRIDE == 1) {
        if (weighted) return c3_launch_mode<W, C3_WEIGHTED, STRIDE>(a, blocks, s);
    }
    if (a.ksplit > 1) return c3_launch_mode<W, C3_SLICED, STRIDE>(a, blocks, s);
    return c3_launch_mode<W, C3_FULL, STRIDE>(a, blocks, s);
}

}  // namespace

void c3_set_forced_crowd(int v) { c3_forced_crowd = v; }

bool conv3x3_applicable(const Geo &g, int mode)
{
    if (!g.bf16 || g.has_bias || (mode == MODE_WEIGHTED && g.blocks)) return false;
    if (g.kh != 3 || g.kw != 3 || g.pad != 1) return false;
    if (g.cin < 64 || g.cout < 64) return false;
    if (g.stride == 1) {
        switch (g.w) {
        case 7: case 8: case 14: case 16: case 28: case 32: case 56: break;
        default: return false;
        }
    } else if (g.stride == 2) {
        // even images only (a row of dY meets two whole rows of X), and the widths and forms that there are bodies for
        if (g.h % 2 || g.w % 2 || g.oh * 2 != g.h || g.ow * 2 != g.w) return false;
        if (mode == MODE_WEIGHTED || (g.ow != 7 && g.ow != 14 && g.ow != 28)) return false;
        // Calls of one and two examples onto 28 columns stay with the kernel that gathers its operands, although this one is faster there by now (us, gathered /
        // this: two layers of 128 -> 128, one example 25 / 21, two 28 / 26, alone 20 / 21; ResNet-50, sixteen micro-steps of one example by themselves
        // 3270 / 3087): its slices take up to twice the workspace, and the entry point with built-in scratch would refuse layers that it takes.
        if (g.ow == 28 && g.n <= 2) return false;
    } else {
        return false;
    }
    // 32-bit element offsets inside the whole tensor
    return (long long)g.n * g.cin * g.h * g.w < (1ll << 31) && (long long)g.n * g.cout * g.h * g.w < (1ll << 31);
}

static size_t conv3x3_ws_bytes_plan(const Geo &g, int mode);

size_t conv3x3_ws_bytes(const Geo &g, int mode)
{
    const int saved = c3_forced_crowd;
    c3_forced_crowd = 0;
    const size_t alone = conv3x3_ws_bytes_plan(g, mode);
    // the smallest target that a batch call with this layer can have: most slices
    c3_forced_crowd = mode == MODE_WEIGHTED ? crowd_of(conv_macs(g)) : 4;
    const size_t shared = conv3x3_ws_bytes_plan(g, mode);
    c3_forced_crowd = saved;
    return alone > shared ? alone : shared;
}

// What the layers are counted with that the entry point with built-in scratch takes: layers of stride 2 with a copy of X besides, its rows split by
// column parity, that their kernel once read.
size_t conv3x3_scratch_bytes(const Geo &g)
{
    const size_t columns = 2 * (size_t)((g.ow + 7) / 8 * 8) + 8;
    return conv3x3_ws_bytes(g, MODE_MATERIALISE) + (g.stride == 2 ? c3_align16((size_t)g.n * g.cin * g.h * columns * sizeof(uint16_t)) : 0);
}

static size_t conv3x3_ws_bytes_plan(const Geo &g, int mode)
{
    const C3Plan p = c3_plan(g, mode);
    const size_t tiles = (size_t)p.tiles_co * p.tiles_ci;
    if (mode == MODE_WEIGHTED) return p.ksplit > 1 ? tiles * p.ksplit * 9 * 16 * C3_THREADS * sizeof(float) : 0;
    const size_t units = (size_t)(g.n / g.unit) * tiles;
    size_t b = c3_align16(units * c3_partials_per_unit(p) * sizeof(float));
    if (p.ksplit > 1) b += units * p.ksplit * 9 * 16 * C3_THREADS * sizeof(float);
    return b;
}

size_t conv3x3_norm_partial_count(const Geo &g)
{
    const C3Plan p = c3_plan(g, MODE_NORM);
    return (size_t)p.tiles_co * p.tiles_ci * c3_partials_per_unit(p);
}

const char *conv3x3_variant_name(const Geo &g, int mode)
{
    static const int widths[7] = {7, 8, 14, 16, 28, 32, 56};
    struct Names {
        char v[2][2][7][56];
        Names()
        {
            for (int st = 0; st < 2; ++st)
                for (int wt = 0; wt < 2; ++wt)
                    for (int k = 0; k < 7; ++k)
                        snprintf(v[st][wt][k], 56, "conv3x3_rows<bf16,w%d%s,%s>", widths[k], st ? ",s2" : "",
                                 wt ? "weighted" : "per_example");
        }
    };
    static const Names names;               // initialised once, thread-safe
    int slot = 6;
    for (int k = 0; k < 7; ++k)
        if (widths[k] == g.ow) slot = k;
    return names.v[g.stride == 2 ? 1 : 0][mode == MODE_WEIGHTED ? 1 : 0][slot];
}

dp_status launch_conv3x3(const Geo &g, int mode, const void *x, const void *dy, float *out_w, size_t out_stride,
                         float *sqnorm, const float *group_sqnorm, float clip_c, void *ws, hipStream_t s)
{
    const bool weighted = mode == MODE_WEIGHTED;
    const C3Plan p = c3_plan(g, mode);
    C3Args a;
    a.variant = -1;
    a.rows = g.n / g.unit; a.unit = g.unit; a.slice_ex = p.slice_ex; a.rows_per_wg = p.rows_per_wg;
    a.x = x; a.dy = dy; a.x_tab = g.x_tab; a.dy_tab = g.dy_tab;
    a.out_w = out_w;
    a.out_stride = out_stride ? out_stride : g.pw;
    a.group_sqnorm = group_sqnorm; a.clip_c = clip_c;
    a.n = g.n; a.cin = g.cin; a.cout = g.cout; a.h = g.oh; a.hin = g.h;
    a.tiles_co = p.tiles_co; a.tiles_ci = p.tiles_ci; a.stages = (g.oh + p.stage_rows - 1) / p.stage_rows;
    a.ksplit = p.ksplit; a.stages_per_split = p.stages_per_split;
    a.ex_per_split = p.ex_per_split;
    const size_t tiles = (size_t)p.tiles_co * p.tiles_ci;
    const size_t units = weighted ? tiles : (size_t)a.rows * tiles;
    char *w = static_cast<char *>(ws);
    a.partials = nullptr;
    if (!weighted) {
        a.partials = reinterpret_cast<float *>(w);
        w += c3_align16(units * c3_partials_per_unit(p) * sizeof(float));
    }
    a.ws_part = p.ksplit > 1 ? reinterpret_cast<float *>(w) : nullptr;
    const long long total = weighted || p.ksplit > 1 ? (long long)units * p.ksplit : (long long)((a.rows + p.rows_per_wg - 1) / p.rows_per_wg) * tiles;
    const unsigned blocks = (unsigned)(((total + 7) / 8) * 8);
    a.total = (int)total;
    dp_status st;
    if (g.stride == 2) {
        if (g.ow == 7) st = c3_launch_w<7, 2>(a, weighted, blocks, s);
        else if (g.ow == 28) st = c3_launch_w<28, 2>(a, weighted, blocks, s);
        else st = c3_launch_w<14, 2>(a, weighted, blocks, s);
    } else {
        switch (g.w) {
        case 7: st = c3_launch_w<7, 1>(a, weighted, blocks, s); break;
        case 8: st = c3_launch_w<8, 1>(a, weighted, blocks, s); break;
        case 14: st = c3_launch_w<14, 1>(a, weighted, blocks, s); break;
        case 16: st = c3_launch_w<16, 1>(a, weighted, blocks, s); break;
        case 28: st = c3_launch_w<28, 1>(a, weighted, blocks, s); break;
        case 32: st = c3_launch_w<32, 1>(a, weighted, blocks, s); break;
        default: st = c3_launch_w<56, 1>(a, weighted, blocks, s); break;
        }
    }
    if (st != DP_OK) return st;
    // what follows the main kernel: at once, or after the grouped launch of a batch call
    if (p.ksplit > 1) {
        const unsigned fix_blocks = (unsigned)(units * 9 * C3_FIX_PARTS);
        const void *fix = weighted ? reinterpret_cast<const void *>(&conv3x3_fixup_kernel<true>)
                                   : reinterpret_cast<const void *>(&conv3x3_fixup_kernel<false>);
        st = submit_kernel<C3Args>(TIER_POST, fix, a, fix_blocks, C3_THREADS, 0, s, "conv3x3_fixup");
        if (st != DP_OK) return st;
    }
    if (weighted || !sqnorm) return DP_OK;
    const int n = a.rows, per_example = p.tiles_co * p.tiles_ci * (int)c3_partials_per_unit(p);
    const float *partials = a.partials;
    return submit_post([=]() -> dp_status { return launch_sum_partials(partials, n, per_example, sqnorm, s); });
}

}  // namespace dp
