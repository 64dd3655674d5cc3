// Per-example weight gradients of 3x3, stride-1, pad-1 convolutions (bf16) from raw image rows.
//
// Same contraction as the general kernel (H1 of the path; per example i
//     dW_i[co, ci, kh, kw] = sum_{oh, ow} dY_i[co, oh, ow] * Xpad_i[ci, oh + kh - 1, ow + kw - 1]),
// but the nine taps of one input channel are nine shifted views of the SAME rows of X, so a
// workgroup stages each row once and builds all nine MFMA operands from it:
//
//   * a workgroup owns 64 output channels x 64 input channels x 9 taps of one example (four
//     waves, each 32 co x 32 ci x 9 taps = nine 32x32 accumulator tiles) and walks chunks of R
//     output rows;
//   * per chunk it stages dY[64 co][R rows] (K-contiguous, rows padded to OWP = W rounded up to
//     8) and X[64 ci][R + 2 rows][WP = OWP + 8 columns] into LDS; X is stored with column
//     c = iw + 1, zeros for iw = -1, iw >= W and rows outside the image, so every tap reads
//     plain in-range LDS;
//   * per 16 values of K a lane reads 16 bytes of dY and, per kernel row kh, 20 bytes of X
//     starting at column ow0: tap kw = 0 is dwords 0..3, kw = 1 the same five dwords shifted by
//     one element, kw = 2 dwords 1..4 -- nine MFMAs from four LDS reads.
//
// Against the general kernel this cuts global/L2 reads of X by ~9x (each row is fetched once
// per workgroup instead of once per tap) and LDS reads per MFMA by ~3x.
//
// K may be sliced over workgroups (few tiles, long K): slices store their accumulators in the
// workspace and a second kernel adds them in slice order, so results are run-to-run identical.
#include "internal.h"
#include "group.h"
#include "pieces.h"

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
    int ksplit, stages_per_split;     // per-example mode: K slices, in stages (C3Cfg)
    int ex_per_split;                 // weighted mode: examples per workgroup (ksplit = example ranges)
    int variant;                      // which body conv3x3_any_kernel runs for this layer (C3_ANY_* below)
    int rows, unit;                   // per-example modes: rows of results, examples of each (Geo::unit)
    int slice_ex;                     // per-example mode, sliced: > 0: the slices are ranges of this many examples of a unit
};

constexpr int C3_RP = 292;                           // floats per row staged by the store epilogue: 288 + 4
constexpr int C3_STORE_LDS = 4 * 8 * C3_RP * 4;      // bytes the store epilogue needs: 4 waves x 8 rows

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
    static constexpr int ZEROS = 128;                        // bytes of zeros at the start: rows outside the image
    static constexpr int RING_X = ZEROS, RING_A = ZEROS + (D + 1) * STAGE_X;
    static constexpr int END = RING_A + (D + 2) * STAGE_A;   // dY one stage further: its next row meets this stage's last row of X
    static constexpr int LDS = END > C3_STORE_LDS ? END : C3_STORE_LDS;
    static constexpr int QX = SG * PX, QA = SG * PA;         // wave instructions of a stage
    static constexpr int UX = (QX + 3) / 4, UA = (QA + 3) / 4;
    static constexpr int BUNDLE = (QX + QA + 3) / 4;         // most of them that a wave issues per stage
    static constexpr bool PARTIAL_A = ROW_A % 16 != 0, PARTIAL_X = ROW_X % 16 != 0;     // a tensor may end inside a piece
    // where local row r (of a stage) of the first channel starts, for rows that start at a dword
    static constexpr int at_a(int r) { return (r / RPG) * GROUP_A + (r % RPG) * ROW_A; }
    static constexpr int at_x(int r) { return (r / (RPG * STRIDE)) * GROUP_X + (r % (RPG * STRIDE)) * ROW_X; }
    static_assert(RPS % 2 == 0, "pairs of rows");
    static_assert(LDS <= 81920 - 256, "two workgroups per CU");
    static_assert(PPR * 16 * STRIDE <= ZEROS, "a row of zeros");
};

constexpr int c3_rows_per_stage(int ow, int stride) { return stride == 2 ? (ow == 28 ? 2 : 4) : (ow >= 28 ? 2 : (ow >= 14 ? 4 : 8)); }
static_assert(C3Cfg<56, 1>::RPS == c3_rows_per_stage(56, 1) && C3Cfg<32, 1>::RPS == c3_rows_per_stage(32, 1) && C3Cfg<28, 1>::RPS == c3_rows_per_stage(28, 1) &&
              C3Cfg<16, 1>::RPS == c3_rows_per_stage(16, 1) && C3Cfg<14, 1>::RPS == c3_rows_per_stage(14, 1) && C3Cfg<8, 1>::RPS == c3_rows_per_stage(8, 1) &&
              C3Cfg<7, 1>::RPS == c3_rows_per_stage(7, 1) && C3Cfg<28, 2>::RPS == c3_rows_per_stage(28, 2) && C3Cfg<14, 2>::RPS == c3_rows_per_stage(14, 2) &&
              C3Cfg<7, 2>::RPS == c3_rows_per_stage(7, 2), "what the host plans");

// What a workgroup does with finished accumulators (all of K of one example): squared norm of
// its 64 x 64 x 9 block and the optional store in the framework's [Cout, Cin, 3, 3] order.
//
// In the accumulator layout a lane holds, per tap, one input channel and sixteen output channels,
// so a direct store writes 4 bytes every 36.  When the layer's channel counts allow it the block
// goes through LDS instead (`lds`, free once the MFMAs are done): each wave lays down eight
// output-channel rows of 32 ci x 9 taps = 288 consecutive floats of the gradient, and reads them
// back as 16-byte pieces that leave as fully coalesced 1152-byte row segments.
__device__ __forceinline__ void c3_epilogue(const f32x16 (&acc)[9], const C3Args &a, int i, int unit, int co0, int ci0,
                                            int wm, int wn, int lane, float *red, char *lds)
{
    float ss = 0.0f;
    const bool store = a.out_w != nullptr;
    float *out = a.out_w + (size_t)i * a.out_stride;
    const bool ci_there = ci0 + wn * 32 + (lane & 31) < a.cin;
    const int co_there = a.cout - (co0 + wm * 32 + (lane >> 5) * 4);
#pragma unroll
    for (int r = 0; r < 16; ++r) {                    // (what stands for channels beyond the layer does not count)
        float s = 0.0f;
#pragma unroll
        for (int t = 0; t < 9; ++t) s += acc[t][r] * acc[t][r];
        ss += ci_there && (r >> 2) * 8 + (r & 3) < co_there ? s : 0.0f;
    }
    // wave-uniform: whole 32-channel blocks, 16-byte aligned rows
    const bool via_lds = store && lds != nullptr && (a.cin % 32 == 0) && (a.out_stride % 4 == 0) &&
                         ((reinterpret_cast<uintptr_t>(a.out_w) & 15u) == 0);
    if (via_lds) {
        float *buf = reinterpret_cast<float *>(lds) + (threadIdx.x >> 6) * (8 * C3_RP);
        const int cil = lane & 31, half = lane >> 5;
        const int cib = ci0 + wn * 32;                                // first input channel of this wave
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            __syncthreads();                                          // previous pass read / MFMAs done with LDS
#pragma unroll
            for (int rr = 0; rr < 4; ++rr)
#pragma unroll
                for (int t = 0; t < 9; ++t) buf[(half * 4 + rr) * C3_RP + cil * 9 + t] = acc[t][q * 4 + rr];
            __syncthreads();
#pragma unroll
            for (int it = 0; it < 9; ++it) {
                const int f4 = it * 64 + lane;                        // 8 rows x 72 pieces
                const int row = f4 / 72, c4 = f4 - row * 72;
                const int co = co0 + wm * 32 + q * 8 + row;
                const float4 v = *reinterpret_cast<const float4 *>(buf + row * C3_RP + c4 * 4);
                if (co < a.cout && cib < a.cin)
                    *reinterpret_cast<float4 *>(out + ((size_t)co * a.cin + cib) * 9 + c4 * 4) = v;
            }
        }
    } else if (store) {
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
    }
    const float tot = block_sum<4>(ss, red);
    if (threadIdx.x == 0) a.partials[unit] = tot;
}

// Weighted sum of one tile over all examples: acc[co, ci, tap] += block, through LDS in the same
// coalesced row form as the store above when the shapes allow, else element by element.
__device__ __forceinline__ void c3_add_to_accumulator(const f32x16 (&acc)[9], const C3Args &a, int co0, int ci0,
                                                      int wm, int wn, int lane, char *lds)
{
    float *out = a.out_w;
    const bool via_lds = (a.cin % 32 == 0) && ((reinterpret_cast<uintptr_t>(a.out_w) & 15u) == 0);
    if (via_lds) {
        float *buf = reinterpret_cast<float *>(lds) + (threadIdx.x >> 6) * (8 * C3_RP);
        const int cil = lane & 31, half = lane >> 5;
        const int cib = ci0 + wn * 32;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            __syncthreads();
#pragma unroll
            for (int rr = 0; rr < 4; ++rr)
#pragma unroll
                for (int t = 0; t < 9; ++t) buf[(half * 4 + rr) * C3_RP + cil * 9 + t] = acc[t][q * 4 + rr];
            __syncthreads();
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
    using pieces_t = std::make_integer_sequence<int, C::PPR>;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    __shared__ float red[4];

    // consecutive hardware workgroup ids rotate over the 8 XCDs; give each XCD a run of
    // consecutive logical ids (the slices and tiles of the same examples share its L2)
    const int tiles = a.tiles_co * a.tiles_ci;
    const int total = (WEIGHTED ? 1 : a.rows) * tiles * a.ksplit;
    const int per_xcd = (total + 7) >> 3;
    const int wg = (int)(bid & 7u) * per_xcd + (int)(bid >> 3);
    if (wg >= total) return;
    const int split = wg % a.ksplit;
    const int unit = wg / a.ksplit;                   // (example, tile); weighted: tile
    const int result = WEIGHTED ? 0 : unit / tiles;   // row of results
    const int i_first = __builtin_amdgcn_readfirstlane(WEIGHTED ? split * a.ex_per_split : result * a.unit + (MODE == C3_SLICED ? split * a.slice_ex : 0));
    const int i_last = __builtin_amdgcn_readfirstlane(WEIGHTED ? min(a.n, i_first + a.ex_per_split) : i_first + (MODE == C3_SLICED ? max(1, a.slice_ex) : a.unit));
    const int tile = unit - result * tiles;
    const int tco = tile / a.tiles_ci, tci = tile - tco * a.tiles_ci;
    const int co0 = __builtin_amdgcn_readfirstlane(tco * 64), ci0 = __builtin_amdgcn_readfirstlane(tci * 64);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int half = lane >> 5;
    const int H = a.h, hin = a.hin;
    const int cin = a.cin, cout = a.cout;

    // Stages of an example: all of them, or a slice [k_begin, k_end).  A slice that starts inside the image has the stage before it as
    // well, which gives its first rows their upper neighbours in dY and no products; its last rows need the stage behind it of dY.
    const int n_stages = (H + C::RPS - 1) / C::RPS;
    const bool cut = MODE == C3_SLICED && a.slice_ex == 0;
    const int k_begin = cut ? split * a.stages_per_split : 0, k_end = cut ? min(n_stages, k_begin + a.stages_per_split) : n_stages;
    const int s_begin = __builtin_amdgcn_readfirstlane(STRIDE == 1 && k_begin > 0 ? k_begin - 1 : k_begin);
    const int x_stages = k_end - s_begin, a_stages = min(n_stages, k_end + 1) - s_begin;
    const int T = (i_last - i_first) * x_stages, TA = (i_last - i_first) * a_stages;

    // ---- global -> LDS.  Wave instruction q of a stage moves pieces 64 q .. 64 q + 63; X's are dealt to the waves from the first, dY's from the last.
    // Pieces that hold nothing (padding, channels beyond the layer, rows below the image) fetch something of the same example, which
    // no product reads or no result shows; so does a piece that the example's end cuts (mend() below fills it in).
    const int x_chan = hin * C::XW, a_chan = H * W;                // elements of a channel
    const size_t x_ex = (size_t)cin * x_chan, a_ex = (size_t)cout * a_chan;
    const int first_x = wave, first_a = 3 - wave;
    struct Piece { int ch, sub, pc; };
    auto piece = [&](int q, int pitch) {
        const int g = q / pitch, id = (q - g * pitch) * 64 + lane;
        return Piece{id / pitch, g, id % pitch};
    };
    // byte offset of a lane's piece from the dword that its example's stage starts in; LAST: the example's last stage (at most
    // that many rows of it are there).  odd: the example starts in the high half of that dword
    auto off_x = [&](int u, unsigned odd, bool last) {
        const Piece p = piece(first_x + 4 * u, C::PX);
        const int c = min(ci0 + p.ch, cin - 1);
        unsigned e = (unsigned)c * (unsigned)x_chan + odd;
        const int pieces = C::ODD_X ? (C::GB_X + 2 * (int)(e & 1u) + 15) / 16 : C::NX;
        const int in_run = p.sub * C::GB_X + min(p.pc, pieces - 1) * 16;
        if constexpr (C::ODD_X) e &= ~1u;
        const unsigned off = 2u * e + (unsigned)in_run;
        if (!last) return off;
        const int before = (n_stages - 1) * C::SG * C::GB_X;       // bytes of a channel above its last stage
        const bool there = in_run < 2 * x_chan - before + (C::ODD_X ? 2 : 0);
        return there && (size_t)off + before + 16 <= 2 * (x_ex + odd) ? off : 0u;
    };
    auto off_a = [&](int u, unsigned odd, bool last) {
        const Piece p = piece(first_a + 4 * u, C::PA);
        const int c = min(co0 + p.ch, cout - 1);
        unsigned e = (unsigned)c * (unsigned)a_chan + odd;
        const int pieces = C::ODD ? (C::GB_A + 2 * (int)(e & 1u) + 15) / 16 : C::NA;
        const int in_run = p.sub * C::GB_A + min(p.pc, pieces - 1) * 16;
        if constexpr (C::ODD) e &= ~1u;
        const unsigned off = 2u * e + (unsigned)in_run;
        if (!last) return off;
        const int before = (n_stages - 1) * C::SG * C::GB_A;
        const bool there = in_run < 2 * a_chan - before + (C::ODD ? 2 : 0);
        return there && (size_t)off + before + 16 <= 2 * (a_ex + odd) ? off : 0u;
    };
    unsigned xo[C::UX], xl[C::UX], ao[C::UA], al[C::UA];
#pragma unroll
    for (int u = 0; u < C::UX; ++u) { xo[u] = off_x(u, 0u, false); xl[u] = off_x(u, 0u, true); }
#pragma unroll
    for (int u = 0; u < C::UA; ++u) { ao[u] = off_a(u, 0u, false); al[u] = off_a(u, 0u, true); }
    const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(size_t)lds);
    auto x_at = [&](int i) { return reinterpret_cast<unsigned long long>(example_at_uniform<uint16_t>(a.x, a.x_tab, i, x_ex)); };
    auto a_at = [&](int i) { return reinterpret_cast<unsigned long long>(example_at_uniform<uint16_t>(a.dy, a.dy_tab, i, a_ex)); };
    struct Stream { unsigned long long base; int i, s, slot; };
    auto fetch_x = [&](Stream &f) {
        const bool last = f.s == n_stages - 1;
        const unsigned odd = C::ODD_X ? (unsigned)(f.base >> 1) & 1u : 0u;
        const unsigned long long b = (f.base & ~3ull) + (unsigned long long)f.s * (C::SG * C::GB_X);
        const unsigned dst = lds0 + C::RING_X + f.slot * C::STAGE_X;
#pragma unroll
        for (int u = 0; u < C::UX; ++u) {
            const int q = first_x + 4 * u;
            if ((C::QX % 4 == 0 || u < C::UX - 1 || q < C::QX)) {
                const unsigned off = C::ODD_X && odd ? off_x(u, odd, last) : (last ? xl[u] : xo[u]);
                lds_direct_16(b, off, dst + q * 1024);
            }
        }
        f.slot = f.slot == C::D ? 0 : f.slot + 1;
        if (++f.s == k_end) {
            f.s = s_begin;
            if (++f.i < i_last) f.base = x_at(f.i);
        }
    };
    auto fetch_a = [&](Stream &f) {
        const bool last = f.s == n_stages - 1;
        const unsigned odd = C::ODD ? (unsigned)(f.base >> 1) & 1u : 0u;
        const unsigned long long b = (f.base & ~3ull) + (unsigned long long)f.s * (C::SG * C::GB_A);
        const unsigned dst = lds0 + C::RING_A + f.slot * C::STAGE_A;
#pragma unroll
        for (int u = 0; u < C::UA; ++u) {
            const int q = first_a + 4 * u;
            if ((C::QA % 4 == 0 || u < C::UA - 1 || q < C::QA)) {
                const unsigned off = C::ODD && odd ? off_a(u, odd, last) : (last ? al[u] : ao[u]);
                lds_direct_16(b, off, dst + q * 1024);
            }
        }
        f.slot = f.slot == C::D + 1 ? 0 : f.slot + 1;
        if (++f.s == s_begin + a_stages) {
            f.s = s_begin;
            if (++f.i < i_last) f.base = a_at(f.i);
        }
    };
    // the piece of an example's last channel that the example's end cuts: its values one by one (by the lane that fetched the rest of its
    // wave instruction, after that has landed)
    auto mend_x = [&](int i, int slot) {
        const unsigned long long base = x_at(i);
        const unsigned odd = C::ODD_X ? (unsigned)(base >> 1) & 1u : 0u;
        const uint16_t *src = reinterpret_cast<const uint16_t *>(base & ~3ull);
        const size_t end = x_ex + odd;
#pragma unroll 1
        for (int u = 0; u < C::UX; ++u) {
            const int q = first_x + 4 * u;
            const Piece p = piece(q, C::PX);
            if (q >= C::QX || ci0 + p.ch != cin - 1 || p.pc >= C::NX) continue;
            const int in_run = p.sub * (C::GB_X / 2) + p.pc * 8;
            size_t e = (size_t)(cin - 1) * x_chan + odd;
            if (C::ODD_X) e &= ~(size_t)1;
            e += (size_t)(n_stages - 1) * (C::SG * C::GB_X / 2) + in_run;
            if (e >= end || e + 8 <= end) continue;
            uint16_t *dst = reinterpret_cast<uint16_t *>(lds + C::RING_X + slot * C::STAGE_X + q * 1024 + lane * 16);
#pragma unroll 1
            for (int k = 0; e + k < end; ++k) dst[k] = src[e + k];
        }
    };
    auto mend_a = [&](int i, int slot) {
        const unsigned long long base = a_at(i);
        const unsigned odd = C::ODD ? (unsigned)(base >> 1) & 1u : 0u;
        const uint16_t *src = reinterpret_cast<const uint16_t *>(base & ~3ull);
        const size_t end = a_ex + odd;
#pragma unroll 1
        for (int u = 0; u < C::UA; ++u) {
            const int q = first_a + 4 * u;
            const Piece p = piece(q, C::PA);
            if (q >= C::QA || co0 + p.ch != cout - 1 || p.pc >= C::NA) continue;
            const int in_run = p.sub * (C::GB_A / 2) + p.pc * 8;
            size_t e = (size_t)(cout - 1) * a_chan + odd;
            if (C::ODD) e &= ~(size_t)1;
            e += (size_t)(n_stages - 1) * (C::SG * C::GB_A / 2) + in_run;
            if (e >= end || e + 8 <= end) continue;
            uint16_t *dst = reinterpret_cast<uint16_t *>(lds + C::RING_A + slot * C::STAGE_A + q * 1024 + lane * 16);
#pragma unroll 1
            for (int k = 0; e + k < end; ++k) dst[k] = src[e + k];
        }
    };
    const bool mends_x = C::PARTIAL_X && ci0 + 64 >= cin, mends_a = C::PARTIAL_A && co0 + 64 >= cout;
    // clip-weighted form: a wave multiplies the pieces of dY that it fetched by the example's factor, rounded to bf16
    auto scale_a = [&](int i, int slot) {
        const float f = a.group_sqnorm ? clip_factor(a.group_sqnorm[i], a.clip_c) : 1.0f;
#pragma unroll
        for (int u = 0; u < C::UA; ++u) {
            const int q = first_a + 4 * u;
            if ((C::QA % 4 == 0 || u < C::UA - 1 || q < C::QA)) {
                uint4 *p = reinterpret_cast<uint4 *>(lds + C::RING_A + slot * C::STAGE_A + q * 1024 + lane * 16);
                const uint4 v = *p;
                uint32_t t[4] = {v.x, v.y, v.z, v.w};
                scale_regs<true, 4>(t, f);
                *p = make_uint4(t[0], t[1], t[2], t[3]);
            }
        }
    };

    f32x16 acc[9];
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t][r] = 0.0f;

    if (threadIdx.x < C::ZEROS / 16) *reinterpret_cast<uint4 *>(lds + threadIdx.x * 16) = make_uint4(0u, 0u, 0u, 0u);
    Stream fx{x_at(i_first), i_first, s_begin, 0}, fa{a_at(i_first), i_first, s_begin, 0};
    int x_issued = 0, a_issued = 0;
    fetch_a(fa);
    a_issued = 1;
#pragma unroll
    for (int k = 0; k < C::D; ++k) {
        if (x_issued < T) { fetch_x(fx); ++x_issued; }
        if (a_issued < TA) { fetch_a(fa); ++a_issued; }
    }

    // operand reads: lane -> channel (lane & 31) of its 32, and the upper or lower one of a pair of rows
    const unsigned lane_x = (unsigned)((wn * 32 + (lane & 31)) * (C::PX * 16)), lane_a = (unsigned)((wm * 32 + (lane & 31)) * (C::PA * 16));
    const int x_odd_chan = C::ODD_X ? ((ci0 + wn * 32 + (lane & 31)) * x_chan) & 1 : 0;
    const int a_odd_chan = C::ODD ? ((co0 + wm * 32 + (lane & 31)) * a_chan) & 1 : 0;

    int ci = i_first, cs = s_begin;                   // stage whose products run
    int ni = i_first, ns = s_begin;                   // the stage of dY behind it in the stream
    auto next_a = [&]() {
        if (++ns == s_begin + a_stages) { ns = s_begin; ++ni; }
    };
    int x_slot = 0, a_slot = 0;
    uint4 carry[STRIDE == 1 ? C::PPR : 1];            // dY rows 2 q - 1 and 2 q, from the pair of rows before

    // stage t of the stream: its rows are there, the loads that the rings have room for are on their way
    int a_next = 1;
    auto arrive = [&](int t) {
        // X of this stage and dY of the next one are bundle t; up to D - 1 younger bundles may still be on their way
        {
            const int mine = (C::QX - first_x + 3) / 4 + (C::QA - first_a + 3) / 4;
            const int young = min(C::D - 1, T - 2 - t);
            if (young <= 0) wait_vmcnt<0>();
            else if (young == 1) { if (mine == C::BUNDLE) wait_vmcnt<C::BUNDLE>(); else wait_vmcnt<C::BUNDLE - 1>(); }
            else { if (mine == C::BUNDLE) wait_vmcnt<2 * C::BUNDLE>(); else wait_vmcnt<2 * C::BUNDLE - 2>(); }
        }
        a_next = a_slot == C::D + 1 ? 0 : a_slot + 1;
        if (t == 0) {
            if (mends_a && ns == n_stages - 1) mend_a(ni, a_slot);
            if constexpr (WEIGHTED) scale_a(ni, a_slot);
            next_a();
        }
        if (t + 1 < TA) {
            if (mends_a && ns == n_stages - 1) mend_a(ni, a_next);
            if constexpr (WEIGHTED) scale_a(ni, a_next);
            next_a();
        }
        if (mends_x && cs == n_stages - 1) mend_x(ci, x_slot);
        __syncthreads();                              // everyone's pieces are there; the stage before has been read
        if (x_issued < T) { fetch_x(fx); ++x_issued; }
        if (a_issued < TA) { fetch_a(fa); ++a_issued; }
    };
    auto leave = [&]() {
        x_slot = x_slot == C::D ? 0 : x_slot + 1;
        a_slot = a_next;
        if (++cs == k_end) { cs = s_begin; ++ci; }
    };
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
    auto rows_here = [&]() {
        odd_x = C::ODD_X ? (unsigned)(x_odd_chan + ((x_ex & 1) ? (int)((x_at(ci) >> 1) & 1) : 0)) & 1u : 0u;
        odd_a = C::ODD ? (unsigned)(a_odd_chan + ((a_ex & 1) ? (int)((a_at(ci) >> 1) & 1) : 0)) & 1u : 0u;
        xs = C::RING_X + x_slot * C::STAGE_X + lane_x;
        as = C::RING_A + a_slot * C::STAGE_A + lane_a;
        an = C::RING_A + a_next * C::STAGE_A + lane_a;
        below = H - cs * C::RPS;
    };
    int t = 0;
    if (STRIDE == 1 && cut && s_begin < k_begin) {    // the stage above a slice: its last row and the next stage's first
        arrive(t++);
        rows_here();
        const C3Row o = row_a(C::RPS - 1);
        c3_each(pieces_t{}, [&](auto j) { if constexpr (STRIDE == 1) carry[j.value] = c3_piece<W, j.value>(lds + o.at, o.bits); });
        leave();
    }
    for (; t < T; ++t) {
        arrive(t);
        rows_here();
        if constexpr (STRIDE == 1) {
            if (cs == 0) {                            // the pair above the first one: row -1 is zeros, row 0 this stage's first
                C3Row o{0u, 0u};
                if (half) o = C3Row{as + (odd_a >> 1) * 4u, odd_a * 16u};
                c3_each(pieces_t{}, [&](auto j) { carry[j.value] = c3_piece<W, j.value>(lds + o.at, o.bits); });
            }
        }
#pragma unroll
        for (int p = 0; p < C::PAIRS; ++p) {
            if (p > 0 && 2 * p >= below) continue;                    // uniform
            const C3Row x = row_x(2 * p), y1 = row_a(2 * p), y0 = row_a(2 * p + 1);
            if constexpr (STRIDE == 1) {
                uint32_t left = 0u;                                   // the two columns before the piece
                uint4 b1 = c3_piece<W, 0>(lds + x.at, x.bits);
                c3_each(pieces_t{}, [&](auto jj) {
                    constexpr int j = jj.value;
                    uint4 ahead = make_uint4(0u, 0u, 0u, 0u);
                    if constexpr (j + 1 < C::PPR) ahead = c3_piece<W, j + 1>(lds + x.at, x.bits);
                    const uint4 a0 = c3_piece<W, j>(lds + y0.at, y0.bits), a1 = c3_piece<W, j>(lds + y1.at, y1.bits);
                    // the same run of columns one to the left and one to the right
                    const uint32_t o0 = funnel(b1.x, left, 16), o1 = funnel(b1.y, b1.x, 16), o2 = funnel(b1.z, b1.y, 16), o3 = funnel(b1.w, b1.z, 16),
                                   o4 = funnel(ahead.x, b1.w, 16);
                    const uint4 b0 = make_uint4(o0, o1, o2, o3), b2 = make_uint4(o1, o2, o3, o4);
                    c3_taps(acc, 1, a1, b0, b1, b2);
                    c3_taps(acc, 0, a0, b0, b1, b2);
                    c3_taps(acc, 2, carry[j], b0, b1, b2);
                    carry[j] = a0;
                    left = b1.w;
                    b1 = ahead;
                });
            } else {
                uint32_t left[2] = {0u, 0u};
                c3_each(pieces_t{}, [&](auto jj) {
                    constexpr int j = jj.value;
                    const uint4 a1 = c3_piece<W, j>(lds + y1.at, y1.bits), a0 = c3_piece<W, j>(lds + y0.at, y0.bits);
#pragma unroll
                    for (int odd_row = 0; odd_row < 2; ++odd_row) {   // row 2 oh of X, then 2 oh + 1
                        const char *row = lds + x.at + (x.at ? odd_row * C::ROW_X : 0);
                        const uint4 v = c3_piece<C::XW, 2 * j>(row, 0u);
                        uint4 w = make_uint4(0u, 0u, 0u, 0u);
                        if constexpr (16 * j + 8 < C::XW) w = c3_piece<C::XW, 2 * j + 1>(row, 0u);
                        const uint4 b0 = make_uint4(c3_high(v.x, left[odd_row]), c3_high(v.z, v.y), c3_high(w.x, v.w), c3_high(w.z, w.y)),     // X[2 ow - 1]
                                    b1 = make_uint4(c3_low(v.y, v.x), c3_low(v.w, v.z), c3_low(w.y, w.x), c3_low(w.w, w.z)),                 // X[2 ow]
                                    b2 = make_uint4(c3_high(v.y, v.x), c3_high(v.w, v.z), c3_high(w.y, w.x), c3_high(w.w, w.z));             // X[2 ow + 1]
                        left[odd_row] = w.w;
                        if (odd_row == 0) {
                            c3_taps(acc, 1, a1, b0, b1, b2);
                        } else {
                            c3_taps(acc, 2, a1, b0, b1, b2);
                            c3_taps(acc, 0, a0, b0, b1, b2);
                        }
                    }
                });
            }
        }
        leave();
    }

    if constexpr (MODE == C3_FULL) {
        c3_epilogue(acc, a, result, unit, co0, ci0, wm, wn, lane, red, lds);
    } else if (WEIGHTED && a.ksplit == 1) {
        c3_add_to_accumulator(acc, a, co0, ci0, wm, wn, lane, lds);
    } else {
        const size_t slot = (size_t)unit * a.ksplit + split;
        float *mine = a.ws_part + slot * (9 * 16 * C3_THREADS);
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) mine[(t * 16 + r) * C3_THREADS + threadIdx.x] = acc[t][r];
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
// not compiled in: registers and LDS are those of the largest body of a set, and the finely sliced 56-wide body
// spills a few registers): set 0 for micro-steps of one or two examples (sliced variants: every launch is a few dozen
// workgroups and costs more than its work), set 1 for larger micro-steps (unsliced and clip-weighted variants).
enum { C3_ANY_56_SLICED = 0, C3_ANY_28_SLICED, C3_ANY_28_FULL, C3_ANY_14_FULL, C3_ANY_14_SLICED, C3_ANY_7_FULL,
       C3_ANY_14S2_SLICED, C3_ANY_14S2_FULL, C3_ANY_7S2_FULL, C3_ANY_56_FULL, C3_ANY_28_WEIGHTED, C3_ANY_14_WEIGHTED,
       C3_ANY_7_WEIGHTED, C3_ANY_28S2_FULL, C3_ANY_28S2_SLICED, C3_ANY_COUNT };

constexpr bool c3_any_in_set(int variant, int set)
{
    if (variant < 0) return false;
    if (set == 0) return variant <= C3_ANY_7S2_FULL || variant >= C3_ANY_28S2_FULL;
    return variant != C3_ANY_56_SLICED;
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
    int tiles_co, tiles_ci, chunks;    // chunks: what the plans count work in, about 224 output positions
    int ksplit, stages_per_split;      // per-example modes: K slices; weighted: example ranges
    int ex_per_split;                  // weighted
    int slice_ex;                      // per-example modes: examples per slice of a clipping unit, or 0
};

int rows_of_width(int ow, int stride)
{
    const int owp = (ow + 7) / 8 * 8;
    if (stride == 2) return owp == 16 ? 5 : (owp == 32 ? 3 : 8);
    return owp == 8 ? 8 : 224 / owp;
}

// The stride-2 form needs no copy of X (it once read one with rows split by column parity).  What is reported stays: callers size buffers
// by it, and the entry point with built-in scratch refuses layers by it.
size_t c3_reported_copy(const Geo &g)
{
    if (g.stride != 2) return 0;
    const int owp = (g.ow + 7) / 8 * 8;
    return ((size_t)g.n * g.cin * g.h * (2 * owp + 8) * sizeof(uint16_t) + 15) & ~(size_t)15;
}

// plans inside a batch call (the launch is shared with other layers) differ; workspace sizes cover both
thread_local int c3_forced_crowd = -1;
int c3_plan_crowd() { return c3_forced_crowd >= 0 ? c3_forced_crowd : crowd_hint(); }

C3Plan c3_plan(const Geo &g, int mode)
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
    const long long tiles = (long long)p.tiles_co * p.tiles_ci;
    // inside a batch call: chunks per workgroup to plan for (a chunk here is about eight 128x128x64 chunks of work, but
    // slices cost a second pass over partial blocks: only very long walks are cut)
    int crowd = c3_plan_crowd(), tgt = crowd ? (crowd / 2 > 1 ? crowd / 2 : 1) : 0;
    // a layer that is small even chunk by chunk (micro-steps of one or two examples): a chunk per workgroup, the
    // walk of a workgroup is what such a launch waits for
    if (crowd && mode != MODE_WEIGHTED && (long long)g.n * tiles * p.chunks <= 128) tgt = 1;
    if (mode == MODE_WEIGHTED) {
        // example ranges: about 256 workgroups, partial blocks in the workspace kept below ~100 MB; in a launch
        // shared with other layers, ranges of at most 48 chunks
        long long want = (256 + tiles - 1) / tiles;
        // (measured in the replayed step: one range -- no partial blocks, no slice-sum launch, a narrow launch that the
        // other streams overlap -- beats four ranges by 4 % of the whole step; a walk is still capped at 48 chunks)
        // and a layer of few tiles still brings 32 workgroups
        if (crowd) {
            want = ((long long)g.n * p.chunks + 47) / 48;
            if (want * tiles < 32) want = (32 + tiles - 1) / tiles;
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
        // even images only (rows split by column parity, output exactly half the size)
        if (g.h % 2 || g.w % 2 || g.oh * 2 != g.h || g.ow * 2 != g.w) return false;
        // measured: worthwhile for the per-example calls on 14- and 7-wide outputs, and on 28-wide ones (chunks of
        // three rows) once a micro-step holds more than two examples: the layer then rides in the launch of the other
        // 3x3 layers (+ 0.4 % for the step; - 0.9 % with one example per micro-step); the clip-weighted form does
        // better in the general kernel / on packed operands
        if (mode == MODE_WEIGHTED || (g.ow != 7 && g.ow != 14 && g.ow != 28)) return false;
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
    c3_forced_crowd = 4;                             // smallest target: most slices
    const size_t shared = conv3x3_ws_bytes_plan(g, mode);
    c3_forced_crowd = saved;
    return alone > shared ? alone : shared;
}

static size_t conv3x3_ws_bytes_plan(const Geo &g, int mode)
{
    const C3Plan p = c3_plan(g, mode);
    const size_t tiles = (size_t)p.tiles_co * p.tiles_ci;
    if (mode == MODE_WEIGHTED) return c3_reported_copy(g) + (p.ksplit > 1 ? tiles * p.ksplit * 9 * 16 * C3_THREADS * sizeof(float) : 0);
    const size_t units = (size_t)(g.n / g.unit) * tiles;
    size_t b = c3_align16(units * c3_partials_per_unit(p) * sizeof(float));
    if (p.ksplit > 1) b += units * p.ksplit * 9 * 16 * C3_THREADS * sizeof(float);
    return b + c3_reported_copy(g);
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
    a.rows = g.n / g.unit; a.unit = g.unit; a.slice_ex = p.slice_ex;
    a.x = x; a.dy = dy; a.x_tab = g.x_tab; a.dy_tab = g.dy_tab;
    a.out_w = out_w;
    a.out_stride = out_stride ? out_stride : g.pw;
    a.group_sqnorm = group_sqnorm; a.clip_c = clip_c;
    a.n = g.n; a.cin = g.cin; a.cout = g.cout; a.h = g.oh; a.hin = g.h;
    a.tiles_co = p.tiles_co; a.tiles_ci = p.tiles_ci;
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
    const long long total = (long long)units * p.ksplit;
    const unsigned blocks = (unsigned)(((total + 7) / 8) * 8);
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
