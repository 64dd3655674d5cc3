// Per-example weight gradients of fp32 convolutions with square odd kernels (3, 5; padding (k - 1) / 2, stride 1 or 2), H1 of
// the path, from raw image rows:
//     dW_i[co, ci, kh, kw] = sum_{oh, ow} dY_i[co, oh, ow] * Xpad_i[ci, s oh + kh - p, s ow + kw - p].
// The fp32 matrix rate (157 TFLOP/s) bounds these layers in any kernel that multiplies fp32 numbers as they are, and an im2col column per
// (ci, kh, kw) stages every element of X k * k times.  Here rows of dY and X go to LDS once per chunk of output rows, all k * k taps
// are read from them, and the products run on the bf16 matrix units, which are sixteen times as fast: every staged number, times 2^24, is split
// into three bf16 numbers whose sum it is, bit for bit (its nearest bf16, the nearest one to what that leaves, and the rest; the smallest fp32 number
// is 2^-149, the smallest normal bf16 2^-126), and a product of two numbers
// is the six products of their parts that reach 2^-24 of it,
//     a b ~ ah bh + (ah bm + am bh) + (am bm + ah bl + al bh),
// each exact in fp32 and added up in fp32.  What is left out is below 2^-23 of the product, and a sum of 32 of them is rounded a handful of
// times where the fp32 instruction rounds at every step.  Relative error of the gradient against 64 bits (2-norm), fp32 instruction ->
// this: 64 -> 64 3x3 on 56 x 56 5.0e-7 -> 1.3e-7, 16 -> 16 on 32 x 32 2.8e-7 -> 0.9e-7, 64 -> 64 on 8 x 8 1.3e-7 -> 0.5e-7, 40 -> 72 5x5 stride 2 on
// 45 x 37 2.6e-7 -> 0.8e-7.
// An infinity or a NaN has no such parts (and its sums are not finite), nor has a number from 2^104 on, and a sum from 2^80 on has no room for the factor:
// a block with a sum that is not finite is computed again with the fp32
// instruction, a row of the output at a time (no reads ahead: it is rare).  us per call, no example broken / one / all: 64 examples of 64 -> 64 3x3 on
// 56 x 56 112 / 482 / 508, 256 of 16 -> 16 on 32 x 32 21 / 75 / 81, 40 of 40 -> 72 5x5 stride 2 on 45 x 37 79 / 160 / 258.
//
// A workgroup owns one block of at most 32 x 32 channels (32 x 16 for 5 x 5) of one example (several examples in a row, so that the set-up is
// paid once and loads run ahead across examples).  K is cut into runs of eight output columns of one row.  Wave (kh, q) keeps the
// k taps of kernel row kh as k accumulators per 16 x 16 channels and takes every q-th group of four runs: in
// v_mfma_f32_16x16x32_bf16 the four lane groups of an operand are eight consecutive K values each, so lane group t holds run t -- eight
// consecutive numbers of dY, one 16-byte read per part, and the sixteen numbers of X around them, 32 bytes per part, from which
// the k shifted operands are cut.  Stride 2: the rows of X are staged as their even and their odd columns, so that every tap is again a
// run of consecutive numbers.  Columns beyond a row's end and runs beyond the chunk are zeros in dY (and finite in X).
//
// The next chunk's rows are loaded into registers before the MFMAs.  Where LDS has room for two chunks (a lone workgroup on a
// compute unit), half of the waves split and write the next chunk before their MFMAs and half after them, so that the vector and the
// matrix units work side by side; where it has not, workgroups overlap one another.  A finished block is
// added up over q in LDS in a fixed order, 16 rows at a time, and leaves as contiguous rows of the gradient; its square goes to one partial
// norm per (example, block).
// A SIMD gives MFMAs and vector instructions their turns (a 16x16x32 MFMA takes 18.8 cycles, every vector instruction beside it 2.6 more), so what
// bounds a full chip is their sum: 3.2 us per chunk of two rows of 64 -> 64 on 56 wide maps, half of it MFMAs.
// MI355X, per-example call alone, fp32 instruction -> this: 64 examples of 64 -> 64 3x3 with a bias on 56 x 56: 194 -> 100 us (154 TFLOP/s), 256:
// 800 -> 433; 256 of 16 -> 16 on 32 x 32: 30 -> 20; 40 of 40 -> 72 5x5 stride 2 with a bias on 45 x 37: 105 -> 80.  Where it is chosen: rows_choice.
#include "group.h"
#include "internal.h"
#include "pieces.h"
#include "rows_plan.h"

#include <atomic>
#include <cstring>

namespace dp {

namespace {

typedef float r_f32x4 __attribute__((ext_vector_type(4)));

constexpr int CR_LEFT = 4;                      // zeros in front of a staged image row (padding <= 2; keeps pieces of four on 8 bytes)
// Where tap kw of a run is: in which columns of the row (stride 2: 0 the even, 1 the odd ones), and how many numbers behind the run's window
constexpr int cr_parity(int k, int s, int kw) { return s == 1 ? 0 : (kw - (k - 1) / 2) & 1; }
constexpr int cr_shift(int k, int s, int kw) { return CR_LEFT + (s == 1 ? kw - (k - 1) / 2 : (kw - (k - 1) / 2 - cr_parity(k, s, kw)) / 2); }

typedef __bf16 r_bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t r_u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t r_u32x2 __attribute__((ext_vector_type(2)));

struct RowsArgs {
    const void *x, *dy;             // [n][cin][H][W], [n][cout][OH][OW]
    int x_tab, dy_tab;              // Geo::x_tab / dy_tab
    float *out_w, *out_b;           // rows of out_stride floats per example, or null
    size_t out_stride_w, out_stride_b;
    float *partials;                // [n][tiles_m * tiles_n]
    int n, cin, cout, h, w, oh, ow;
    int tiles_m, tiles_n, ex_per_wg;
    int unit;                       // Geo::unit
    int q;                          // waves that share the runs of a kernel row
    int rows, chunks;               // output rows per chunk, chunks per example
    int rpr;                        // runs per output row
    int xp, cha, chx;               // LDS pitches in dwords: a staged image row, a channel of dY, a channel of X
    int tail;                       // RowsPlan::tail
    int waves_a;                    // waves that stage dY (the others stage X)
    int bufs;                       // chunks in LDS (1 or 2)
    int bias;
    int ragged, narrow;             // rows of dY or X are no multiple of four; are shorter than four
};

__device__ __forceinline__ int cr_small_div(int a, int d) { return (int)(((float)a + 0.5f) * __builtin_amdgcn_rcpf((float)d)); }   // a, d < 2^15, quotient exact: the distance to an integer is at least 1 / (2 d)

// The three bf16 parts of a pair of numbers, packed: the number rounded to the nearest bf16, what that leaves of it rounded likewise, and what is
// then left, which has no more than eight significant bits.
__device__ __forceinline__ void cr_split(float v0, float v1, uint32_t (&part)[3])
{
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        part[p] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{v0, v1}), bf16x2));
        if (p < 2) {
            v0 -= __uint_as_float(part[p] << 16);
            v1 -= __uint_as_float(part[p] & 0xFFFF0000u);
        }
    }
}

constexpr float CR_UP = 0x1p24f, CR_DOWN = 0x1p-24f;     // what a number is scaled by before it is split, and back (sums: twice)
constexpr unsigned CR_NOWHERE = 0xFFFFFFF0u;     // a byte beyond every example: the load gives zeros

// NM x NN blocks of 16 x 16 channels
template <int K, int S, int NM, int NN>
__global__ void __launch_bounds__(64 * K * cr_qmax(K)) conv_rows_kernel(const Grouped<RowsArgs> grp)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t rows_lds[];
    constexpr int PT = CR_PIECES, PAD = (K - 1) / 2, CO = 16 * NM, CI = 16 * NN;
    unsigned bid;
    const RowsArgs &a = grp.a[group_pick(grp, bid)];
    const int tiles = a.tiles_m * a.tiles_n;
    const int batches = (a.n + a.ex_per_wg - 1) / a.ex_per_wg;
    // the blocks of an example read the same rows: one after the other behind the L2 of one XCD
    const int per_xcd = (batches * tiles + 7) >> 3, wg = (int)(bid & 7u) * per_xcd + (int)(bid >> 3);
    if (wg >= batches * tiles) return;
    const int batch = wg / tiles, tile = wg - batch * tiles;
    const int i_begin = batch * a.ex_per_wg, i_end = min(a.n, i_begin + a.ex_per_wg);
    const int m0 = (tile / a.tiles_n) * CO, n0 = (tile - (tile / a.tiles_n) * a.tiles_n) * CI;
    const int cm = min(CO, a.cout - m0), cn = min(CI, a.cin - n0);       // live channels
    const int tid = (int)threadIdx.x, nthreads = 64 * K * a.q, nwaves = K * a.q;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kh = wave / a.q, q = wave - kh * a.q;
    const int OH = a.oh, OW = a.ow, H = a.h, W = a.w, R = a.rows, RPR = a.rpr;
    const int lines = (R - 1) * S + K;
    const int groups = (R * RPR + 3) / 4;

    // LDS: per chunk dY, [channel][run][part][8 numbers], and X, [channel][row][8 columns of a parity][parity][part]; then the runs' offsets.
    // (Parts of eight numbers side by side: every read of a run has a constant offset.)  The epilogue uses the chunks' place, and may need more of
    // it than they do; the table is written once for all examples of the workgroup.
    const int chunk_x = CO * a.cha, chunk_dwords = chunk_x + CI * a.chx;
    int *tab = reinterpret_cast<int *>(rows_lds + a.tail);
    float *red = reinterpret_cast<float *>(tab + groups * 4);
    float *epi = reinterpret_cast<float *>(rows_lds);
    const int EP = CI * K * K + 2;                     // pitch of a gradient row in LDS (spreads the lane groups over the banks)

    // per run: where its X starts inside a channel
    for (int t = tid; t < groups * 4; t += nthreads) {
        const int r = cr_small_div(t, RPR), c = t - r * RPR;
        tab[t] = t < R * RPR ? r * S * a.xp + 12 * S * c : 0;
    }
    // What this thread moves per chunk: the first waves_a waves pieces of dY, the others pieces of X.  Byte offset at output row 0 of the
    // example, and packed: LDS dword, row of the chunk, elements (0: no piece).
    const bool is_x = wave >= a.waves_a;
    const int apr = (OW + 3) / 4, xpr = (W + 3) / 4, a_threads = 64 * a.waves_a;
    unsigned off[PT];
    int meta[PT];
#pragma unroll
    for (int u = 0; u < PT; ++u) {
        if (!is_x) {
            const int idx = tid + a_threads * u;
            const int row = cr_small_div(idx, apr), pc = idx - row * apr, ch = cr_small_div(row, R), r = row - ch * R;
            off[u] = 4u * (unsigned)(((m0 + ch) * OH + r) * OW + (a.narrow ? 4 * pc : min(4 * pc, OW - 4)));
            meta[u] = idx < cm * R * apr ? (ch * a.cha + (r * RPR + pc / 2) * 12 + (pc & 1) * 2) | (r << 16) | (min(4, OW - 4 * pc) << 24) : 0;
        } else {
            const int idx = tid - a_threads + (nthreads - a_threads) * u;
            const int row = cr_small_div(idx, xpr), pc = idx - row * xpr, ch = cr_small_div(row, lines), k = row - ch * lines;
            const int d = (CR_LEFT + 4 / S * pc) / 2;  // dword of the row (of one parity)
            off[u] = 4u * (unsigned)(((n0 + ch) * H + k - PAD) * W + (a.narrow ? 4 * pc : min(4 * pc, W - 4)));
            meta[u] = idx < cn * lines * xpr ? (chunk_x + ch * a.chx + k * a.xp + (d / 4) * (12 * S) + d % 4) | (k << 16) | (min(4, W - 4 * pc) << 24) : 0;
        }
    }
    r_f32x4 raw[PT];
    int f_i = i_begin, f_c = 0;                        // next chunk to fetch
    __amdgpu_buffer_rsrc_t rsrc;
    auto fetch = [&]() {
        if (f_i >= i_end) return;
        const int row0 = is_x ? f_c * R * S - PAD : f_c * R, rows = is_x ? H : OH;
        const unsigned step = 4u * (unsigned)(is_x ? f_c * R * S * W : f_c * R * OW);
        if (f_c == 0) {
            const unsigned bytes = 4u * (unsigned)(is_x ? a.cin * H * W : a.cout * OH * OW);
            const float *ex = example_at_uniform<float>(is_x ? a.x : a.dy, is_x ? a.x_tab : a.dy_tab, f_i, bytes / 4u);
            rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(ex), 0, bytes, 0x00020000);
        }
        if (++f_c == a.chunks) { f_c = 0; ++f_i; }
#pragma unroll
        for (int u = 0; u < PT; ++u) {
            int mt = meta[u];
            asm volatile("" : "+v"(mt));               // unpacked anew for every chunk: kept unpacked, it is three registers a piece
            const bool there = mt && (unsigned)(row0 + ((mt >> 16) & 0xff)) < (unsigned)rows;
            const unsigned at = there ? off[u] + step : CR_NOWHERE;
            if (a.narrow) {                            // rows of fewer than four numbers
                const int count = mt >> 24;
#pragma unroll
                for (int e = 0; e < 4; ++e) raw[u][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc, there && e < count ? at + 4 * e : CR_NOWHERE, 0, 0));
            } else {
                raw[u] = __builtin_bit_cast(r_f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, at, 0, 0));
            }
        }
    };
    const bool has_bias = a.bias && n0 == 0;
    float bsum[PT];                                    // of the numbers of dY that this thread staged
    auto stage = [&](int buf) {
        uint32_t *const chunk = rows_lds + buf * chunk_dwords;
        if (a.ragged) {
            // the end of a row that is no multiple of four was fetched as the row's last four numbers: the first `count` places get the last ones
            asm volatile("");
#pragma unroll
            for (int u = 0; u < PT; ++u)
#pragma unroll
                for (int c = 3; c > 0; --c) raw[u] = meta[u] >> 24 <= c ? r_f32x4{raw[u].y, raw[u].z, raw[u].w, 0.0f} : raw[u];
        }
#pragma unroll
        for (int u = 0; u < PT; ++u)
            if (int mt = meta[u]) {
                asm volatile("" : "+v"(mt));
                uint32_t lo[3], hi[3];
                const r_f32x4 r = raw[u], v = r * CR_UP;
                uint32_t *dst = chunk + (mt & 0xffff);
                if (S == 1 || !is_x) {
                    if (has_bias) bsum[u] += (r.x + r.y) + (r.z + r.w);
                    cr_split(v.x, v.y, lo);
                    cr_split(v.z, v.w, hi);
#pragma unroll
                    for (int p = 0; p < 3; ++p) *reinterpret_cast<r_u32x2 *>(dst + 4 * p) = r_u32x2{lo[p], hi[p]};
                } else {                               // even columns and odd columns
                    cr_split(v.x, v.z, lo);
                    cr_split(v.y, v.w, hi);
#pragma unroll
                    for (int p = 0; p < 3; ++p) { dst[4 * p] = lo[p]; dst[4 * p + 12] = hi[p]; }
                }
            }
    };

    r_f32x4 acc[NM][NN][K];
    const int kq = lane >> 4;
    // the MFMAs of a chunk's runs
    auto multiply = [&](int buf, int live) {
        const uint32_t *pa = rows_lds + buf * chunk_dwords + (lane & 15) * a.cha;
        const uint32_t *px = rows_lds + buf * chunk_dwords + chunk_x + (lane & 15) * a.chx + kh * a.xp;
#pragma unroll 1
        for (int g = q; g < live; g += a.q) {
            const int t = 4 * g + kq, at = tab[t];
            r_bf16x8 av[NM][3];
#pragma unroll
            for (int b = 0; b < NM; ++b)
#pragma unroll
                for (int p = 0; p < 3; ++p) av[b][p] = __builtin_bit_cast(r_bf16x8, *reinterpret_cast<const r_u32x4 *>(pa + b * 16 * a.cha + 12 * t + 4 * p));
#pragma unroll
            for (int by = 0; by < NN * S; ++by) {
                const int b = by / S, y = by % S;
                asm volatile("" ::: "memory");           // one block's X (of one parity) at a time in registers
                uint32_t w[3][8];
#pragma unroll
                for (int p = 0; p < 3; ++p) {
                    const uint32_t *src = px + b * 16 * a.chx + at + 12 * y + 4 * p;
                    const r_u32x4 v = *reinterpret_cast<const r_u32x4 *>(src);
                    const r_u32x4 e = *reinterpret_cast<const r_u32x4 *>(src + 12 * S);
                    w[p][0] = v.x; w[p][1] = v.y; w[p][2] = v.z; w[p][3] = v.w; w[p][4] = e.x; w[p][5] = e.y; w[p][6] = e.z; w[p][7] = e.w;
                }
#pragma unroll
                for (int kw = 0; kw < K; ++kw) {
                    if (cr_parity(K, S, kw) != y) continue;
                    const int sh = cr_shift(K, S, kw), d = sh / 2;
                    r_bf16x8 xv[3];
#pragma unroll
                    for (int p = 0; p < 3; ++p) {
                        r_u32x4 v;
                        if (sh & 1)
                            v = r_u32x4{funnel(w[p][d + 1], w[p][d], 16), funnel(w[p][d + 2], w[p][d + 1], 16),
                                        funnel(w[p][d + 3], w[p][d + 2], 16), funnel(w[p][d + 4], w[p][d + 3], 16)};
                        else
                            v = r_u32x4{w[p][d], w[p][d + 1], w[p][d + 2], w[p][d + 3]};
                        xv[p] = __builtin_bit_cast(r_bf16x8, v);
                    }
                    // The six products of 32 K values, small ones first, are a sum of their own, which is then added to the block: it is much smaller
                    // than the block, and so is what the six instructions round off.
                    constexpr int pairs[6][2] = {{2, 0}, {0, 2}, {1, 1}, {1, 0}, {0, 1}, {0, 0}};
                    r_f32x4 sum[NM];
#pragma unroll
                    for (int e = 0; e < 6; ++e)
#pragma unroll
                        for (int m = 0; m < NM; ++m)
                            sum[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[m][pairs[e][0]], xv[pairs[e][1]], e ? sum[m] : r_f32x4{0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0);
#pragma unroll
                    for (int m = 0; m < NM; ++m) acc[m][b][kw] += sum[m];
                }
            }
        }
    };

    const bool early = a.bufs == 2 && ((wave >> 2) & 1) == 0;      // waves 0 .. 3 are on different SIMDs
    const int steps = a.chunks * a.unit;
    fetch();
    for (int row_i = i_begin / a.unit; row_i * a.unit < i_end; ++row_i) {
        // margins, dead channels and the runs beyond a chunk's last one are never written
        for (int t = tid; t < a.bufs * chunk_dwords; t += nthreads) rows_lds[t] = 0u;
#pragma unroll
        for (int m = 0; m < NM; ++m)
#pragma unroll
            for (int b = 0; b < NN; ++b)
#pragma unroll
                for (int k = 0; k < K; ++k) acc[m][b][k] = r_f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int u = 0; u < PT; ++u) bsum[u] = 0.0f;
        __syncthreads();
        stage(0);
        fetch();                                       // (the last chunk's: of the next example)
        __syncthreads();
        int c = 0;
        for (int step = 0; step < steps; ++step) {
            const bool more = step + 1 < steps;
            const int buf = a.bufs == 2 ? step & 1 : 0;
            if (early && more) { stage(buf ^ 1); fetch(); }
            const int live = (min(R, OH - c * R) * RPR + 3) / 4;
            multiply(buf, live);
            if (++c == a.chunks) c = 0;
            if (!early && more) {
                if (a.bufs == 1) __syncthreads();      // everyone has read this chunk
                stage(a.bufs == 1 ? 0 : buf ^ 1);
                fetch();
            }
            __syncthreads();
        }
        float odd = 0.0f;
#pragma unroll
        for (int m = 0; m < NM; ++m)
#pragma unroll
            for (int b = 0; b < NN; ++b)
#pragma unroll
                for (int k = 0; k < K; ++k)
#pragma unroll
                    for (int r = 0; r < 4; ++r) odd = fmaf(acc[m][b][k][r], 0.0f, odd);
        const bool plain = __syncthreads_or(odd != 0.0f) != 0;        // (true for NaN)
        if (plain) {
            // Not every sum is finite: the block again with the fp32 instruction, a row of the output at a time (dY and the K rows of X that it meets lie
            // in the chunks' place as they are; lane group t has column t of four).  Both operands of a position outside the image are zero.
            // (The opaque copies keep what is worked out from them here: hoisted out of the loop over examples, it costs the products above their registers.)
            int ow_n = OW, w_n = W, oh_n = OH, h_n = H, id = tid, rows_a = cm, rows_x = cn * K;
            asm volatile("" : "+s"(ow_n), "+s"(w_n), "+s"(oh_n), "+s"(h_n), "+s"(rows_a), "+s"(rows_x));
            asm volatile("" : "+v"(id));
            const int pitch_a = ow_n | 1, pitch_x = (K * w_n) | 1, col = id & 15, four = (id >> 4) & 3;
            float *const sx = epi + CO * pitch_a;
#pragma unroll
            for (int m = 0; m < NM; ++m)
#pragma unroll
                for (int b = 0; b < NN; ++b)
#pragma unroll
                    for (int k = 0; k < K; ++k) acc[m][b][k] = r_f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 1
            for (int i = row_i * a.unit; i < (row_i + 1) * a.unit; ++i) {
                const float *dy_ex = example_at_uniform<float>(a.dy, a.dy_tab, i, (size_t)a.cout * oh_n * ow_n) + (size_t)m0 * oh_n * ow_n;
                const float *x_ex = example_at_uniform<float>(a.x, a.x_tab, i, (size_t)a.cin * h_n * w_n) + (size_t)n0 * h_n * w_n;
#pragma unroll 1
                for (int oh = 0; oh < oh_n; ++oh) {
                    __syncthreads();                   // everyone has read the row before
#pragma unroll 1
                    for (int t = id; t < rows_a * ow_n; t += nthreads) {
                        const int ch = t / ow_n, c = t - ch * ow_n;
                        epi[ch * pitch_a + c] = dy_ex[((size_t)ch * oh_n + oh) * ow_n + c];
                    }
#pragma unroll 1
                    for (int t = id; t < rows_x * w_n; t += nthreads) {
                        const int row = t / w_n, c = t - row * w_n, ch = row / K, k = row - ch * K, ih = oh * S + k - PAD;
                        sx[ch * pitch_x + k * w_n + c] = (unsigned)ih < (unsigned)h_n ? x_ex[((size_t)ch * h_n + ih) * w_n + c] : 0.0f;
                    }
                    __syncthreads();
                    if ((unsigned)(oh * S + kh - PAD) >= (unsigned)h_n) continue;        // (the same in every lane of a wave)
#pragma unroll 1
                    for (int g = q; 4 * g < ow_n; g += a.q) {
                        const int ow = 4 * g + four;
#pragma unroll
                        for (int k = 0; k < K; ++k) {
                            const int iw = ow * S + k - PAD;
                            const bool there = ow < ow_n && (unsigned)iw < (unsigned)w_n;
                            float d[NM];
#pragma unroll
                            for (int m = 0; m < NM; ++m) d[m] = there ? epi[(m * 16 + col) * pitch_a + ow] : 0.0f;
#pragma unroll
                            for (int b = 0; b < NN; ++b) {
                                const float v = there ? sx[(b * 16 + col) * pitch_x + kh * w_n + iw] : 0.0f;
#pragma unroll
                                for (int m = 0; m < NM; ++m) acc[m][b][k] = __builtin_amdgcn_mfma_f32_16x16x4f32(d[m], v, acc[m][b][k], 0, 0, 0);
                            }
                        }
                    }
                }
            }
            __syncthreads();
        }
        const float down = plain ? 1.0f : CR_DOWN;
        float ss = 0.0f;
        // the block, 16 rows at a time: summed over q in order, squared, stored
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            if (m * 16 >= cm) break;
            float *mine = epi + (q * 16 + kq * 4) * EP + ((lane & 15) * K + kh) * K;
#pragma unroll
            for (int b = 0; b < NN; ++b)
#pragma unroll
                for (int k = 0; k < K; ++k)
#pragma unroll
                    for (int r = 0; r < 4; ++r) mine[r * EP + b * 16 * K * K + k] = acc[m][b][k][r] * down;
            __syncthreads();
            const int len = cn * K * K;
            for (int r = wave; r < min(16, cm - m * 16); r += nwaves) {
                const int co = m0 + m * 16 + r;
                float *dst = a.out_w ? a.out_w + (size_t)row_i * a.out_stride_w + ((size_t)co * a.cin + n0) * (K * K) : nullptr;
                for (int t = lane; t < len; t += 64) {
                    float v = epi[r * EP + t];
                    for (int part = 1; part < a.q; ++part) v += epi[(part * 16 + r) * EP + t];
                    v *= down;
                    ss += v * v;
                    if (dst) __builtin_nontemporal_store(v, dst + t);
                }
            }
            __syncthreads();                           // epi is free again
        }
        if (has_bias) {
            // a channel's pieces are R * apr threads' in a row (in PT rounds): one thread adds them up
#pragma unroll
            for (int u = 0; u < PT; ++u)
                if (!is_x) epi[tid + a_threads * u] = bsum[u];
            __syncthreads();
            if (tid < cm) {
                float v = 0.0f;
                for (int t = 0; t < R * apr; ++t) v += epi[tid * R * apr + t];
                ss += v * v;
                if (a.out_b) a.out_b[(size_t)row_i * a.out_stride_b + m0 + tid] = v;
            }
            __syncthreads();
        }
        ss = wave_sum(ss);
        if (lane == 0) red[wave] = ss;
        __syncthreads();
        if (tid == 0) {
            float t = 0.0f;
            for (int k = 0; k < nwaves; ++k) t += red[k];
            a.partials[(size_t)row_i * tiles + tile] = t;
        }
    }
}

size_t cr_align16(size_t b) { return (b + 15) & ~(size_t)15; }

template <int K, int S> const void *rows_fn(int nm, int nn)
{
    if constexpr (K == 3)
        if (nn == 2) return nm == 2 ? reinterpret_cast<const void *>(&conv_rows_kernel<K, S, 2, 2>) : reinterpret_cast<const void *>(&conv_rows_kernel<K, S, 1, 2>);
    return nm == 2 ? reinterpret_cast<const void *>(&conv_rows_kernel<K, S, 2, 1>) : reinterpret_cast<const void *>(&conv_rows_kernel<K, S, 1, 1>);
}

// What the sizes decide, kept for the sizes seen last (a call asks several times): the plan, and whether the kernel is the faster one.
struct RowsChoice {
    int key[10];
    bool use;
    RowsPlan plan;
};

const RowsChoice &rows_choice(const Geo &g)
{
    static thread_local RowsChoice kept[64];
    const bool shared = crowd_hint() > 0;
    const int key[10] = {g.n, g.unit, g.cin, g.cout, g.h, g.w, g.kh, g.stride, 1 + g.has_bias, shared};
    unsigned at = 0;
    for (int v : key) at = at * 31u + (unsigned)v;
    RowsChoice &c = kept[(at ^ at >> 6) % 64];
    if (std::memcmp(c.key, key, sizeof(key)) != 0) {
        c.plan = rows_plan(g, false);
        // Both times estimated (the general kernel's holds 3 us that only calls outside a graph pay), a margin of 12 % to the general kernel.  On
        // 181 layers in and around the networks here (3x3 and 5x5, strides 1 and 2, 3 to 160 channels, 7 to 56 rows, 8 to 512 examples, with and
        // without a bias) all together take 0.74 of the general kernel's time, where the faster of the two each time would be 0.73; a
        // margin of 5 % took 8 that are slower by more than 5 %, this one takes 3.  us, general / this: 64 -> 64 3x3 on 56 x 56,
        // 64 examples with a bias 385 / 94, 256 without 795 / 403; 16 -> 16 on 32 x 32, 256: 97 / 20; 128 -> 128 on 28 x 28, 64:
        // 231 / 127; 32 -> 64 stride 2 on 16 x 16, 256: 22 / 31; 5x5, 40 -> 72 stride 2 on 45 x 37 with a bias, 40: 120 / 78.
        c.use = c.plan.ok && c.plan.us + 3.0 < 0.88 * conv_general_f32_us(g);
        if (shared && c.use) c.plan = rows_plan(g, true);
        std::memcpy(c.key, key, sizeof(key));
    }
    return c;
}

}  // namespace

bool conv_rows_applicable(const Geo &g, int mode)
{
    if (mode == MODE_WEIGHTED || g.bf16) return false;
    if (g.kh != g.kw || (g.kh != 3 && g.kh != 5) || g.pad != (g.kh - 1) / 2 || g.stride < 1 || g.stride > 2) return false;
    // offsets inside an example (rows above and below the image included) fit 31 bits; quotients of the set-up stay exact
    if ((size_t)g.cin * (g.h + 8) * g.w >= ((size_t)1 << 29) || (size_t)g.cout * (g.oh + 64) * g.ow >= ((size_t)1 << 29)) return false;
    if (g.w > 4096 || (double)g.n * conv_rows_norm_partial_count(g) >= 1.0e9) return false;
    return rows_choice(g).use;
}

size_t conv_rows_norm_partial_count(const Geo &g)
{
    const int co = 16 * rows_nm(g), ci = 16 * rows_nn(g);
    return (size_t)((g.cout + co - 1) / co) * ((g.cin + ci - 1) / ci);
}

size_t conv_rows_ws_bytes(const Geo &g) { return cr_align16((size_t)(g.n / g.unit) * conv_rows_norm_partial_count(g) * sizeof(float)); }

const char *conv_rows_variant_name(const Geo &g)
{
    // (kernel size, stride, blocks of output and of input channels: the kernels that share a launch)
#define DP_ROWS_NAMES(KS) {{{"conv_rows<f32," KS ",16x16,per_example>", "conv_rows<f32," KS ",16x32,per_example>"}, \
                            {"conv_rows<f32," KS ",32x16,per_example>", "conv_rows<f32," KS ",32x32,per_example>"}}, \
                           {{"conv_rows<f32," KS ",s2,16x16,per_example>", "conv_rows<f32," KS ",s2,16x32,per_example>"}, \
                            {"conv_rows<f32," KS ",s2,32x16,per_example>", "conv_rows<f32," KS ",s2,32x32,per_example>"}}}
    static const char *const names[2][2][2][2] = {DP_ROWS_NAMES("3x3"), DP_ROWS_NAMES("5x5")};
#undef DP_ROWS_NAMES
    return names[g.kh / 2 - 1][g.stride - 1][rows_nm(g) - 1][rows_nn(g) - 1];
}

dp_status launch_conv_rows(const Geo &g, const void *x, const void *dy, float *out_w, float *out_b, size_t out_stride, float *sqnorm,
                           void *ws, hipStream_t s)
{
    const RowsPlan p = rows_choice(g).plan;
    RowsArgs a;
    a.x = x; a.dy = dy; a.x_tab = g.x_tab; a.dy_tab = g.dy_tab;
    a.out_w = out_w; a.out_b = out_b;
    a.out_stride_w = out_stride ? out_stride : g.pw;
    a.out_stride_b = out_stride ? out_stride : g.pb;
    a.partials = static_cast<float *>(ws);
    a.n = g.n; a.cin = g.cin; a.cout = g.cout; a.h = g.h; a.w = g.w; a.oh = g.oh; a.ow = g.ow;
    a.tiles_m = p.tiles_m; a.tiles_n = p.tiles_n; a.ex_per_wg = p.ex_per_wg; a.unit = g.unit; a.q = p.q;
    a.rows = p.rows; a.chunks = p.chunks; a.rpr = p.rpr; a.xp = p.xp; a.cha = p.cha; a.chx = p.chx; a.bufs = p.bufs; a.tail = p.tail; a.waves_a = p.waves_a;
    a.bias = g.has_bias ? 1 : 0;
    a.narrow = g.w < 4 || g.ow < 4;
    a.ragged = !a.narrow && (g.w % 4 || g.ow % 4);
    const void *fn = g.kh == 3 ? (g.stride == 2 ? rows_fn<3, 2>(p.nm, p.nn) : rows_fn<3, 1>(p.nm, p.nn))
                               : (g.stride == 2 ? rows_fn<5, 2>(p.nm, p.nn) : rows_fn<5, 1>(p.nm, p.nn));
    static std::atomic<bool> attr_done[2][2][2][2];     // zero-initialised; setting the attribute twice is harmless
    std::atomic<bool> &done = attr_done[g.kh / 2 - 1][g.stride - 1][p.nm - 1][p.nn - 1];
    if (!done.load()) {
        if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, 156 * 1024) != hipSuccess)
            return fail(DP_ERR_DEVICE, "conv_rows: cannot reserve LDS");
        done.store(true);
    }
    const long long total = (long long)((g.n + p.ex_per_wg - 1) / p.ex_per_wg) * p.tiles_m * p.tiles_n;
    const dp_status st = submit_main<RowsArgs>(fn, a, (unsigned)((total + 7) / 8 * 8), (unsigned)(64 * g.kh * p.q), p.lds, s, "conv_rows");
    if (st != DP_OK || !sqnorm) return st;
    const float *parts = a.partials;
    const int n = g.n / g.unit, count = (int)conv_rows_norm_partial_count(g);
    return submit_post([=]() -> dp_status { return launch_sum_partials(parts, n, count, sqnorm, s); });
}

}  // namespace dp
