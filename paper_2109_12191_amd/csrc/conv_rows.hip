// Per-example weight gradients of fp32 convolutions with square odd kernels (3, 5; padding (k - 1) / 2, stride 1 or 2), H1 of
// the path, from raw image rows:
//     dW_i[co, ci, kh, kw] = sum_{oh, ow} dY_i[co, oh, ow] * Xpad_i[ci, s oh + kh - p, s ow + kw - p].
// What bounds these layers is the fp32 matrix rate (157 TFLOP/s, 256 flop per cycle and compute unit): an im2col column per
// (ci, kh, kw) fetches and stages every element of X k * k times, which costs the general kernel more cycles than its MFMAs (35
// TFLOP/s on 64 -> 64 at 56 x 56; and 64 x 64 tiles of a 16-channel layer are three quarters padding).  Here rows of dY and X go to LDS
// once per chunk of output rows and all k * k taps are read from them.
//
// A workgroup owns one block of at most 32 x 32 channels (32 x 16 for 5 x 5) of one example (several examples in a row, so that the set-up is
// paid once and loads run ahead across examples).  K is cut into runs of four output columns of one row.  Wave (kh, q) keeps the
// k taps of kernel row kh as k accumulators per 16 x 16 channels and takes every q-th group of four runs: in
// v_mfma_f32_16x16x4_f32 the four lane groups of an operand are the four K values, so lane group t holds run t -- four
// consecutive floats of dY, one 16-byte read, and the 4 s + k - s floats of X behind them, two to four aligned 16-byte reads --
// and MFMA (j, kw) multiplies column j of each run with X shifted by kw.  12 k or more MFMAs of 32 cycles follow a handful
// of LDS reads, so neither LDS nor the vector unit is near its rate.  Columns beyond a row's end and runs beyond the
// chunk are masked in both operands, as no element outside the image may reach a sum (0 * inf).
//
// The next chunk's rows are loaded into registers before the MFMAs and written to LDS after them.  A finished block is
// added up over q in LDS in a fixed order, 16 rows at a time, and leaves as contiguous rows of the gradient; its square goes to one partial
// norm per (example, block).
// MI355X, per-example call alone, general kernel -> this: 64 examples of 64 -> 64 3x3 with a bias on 56 x 56: 378 -> 202 us (73 TFLOP/s);
// 40 of 40 -> 72 5x5 stride 2 with a bias on 45 x 37: 126 -> 109 us.  Where it is chosen: rows_choice.
#include "group.h"
#include "internal.h"
#include "pieces.h"

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>

namespace dp {

namespace {

typedef float r_f32x4 __attribute__((ext_vector_type(4)));
typedef r_f32x4 r_f32x4_a4 __attribute__((aligned(4)));

constexpr int CR_CH = 32;                       // output channels of a block
constexpr int cr_cin(int k) { return k == 5 ? 16 : 32; }                // its input channels (5 accumulators a block of 16 x 16: registers)
constexpr int CR_LEFT = 4;                      // zeros in front of a staged image row (padding <= 2; keeps pieces on 16 bytes)
constexpr int cr_qmax(int k) { return k == 5 ? 2 : 4; }
constexpr int cr_pieces(int k) { return k == 3 ? 7 : 8; }               // 16-byte pieces a thread moves per chunk
// 16-byte reads that cover X of a run: the first starts at the multiple of four at or below the run's first element
constexpr int cr_first(int k) { return (CR_LEFT - (k - 1) / 2) % 4; }   // where the run's first element is in them
constexpr int cr_reads(int k, int s) { return (cr_first(k) + 3 * s + k + 3) / 4; }

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
    int xp, cha, chx;               // LDS pitches in floats: an image row, a channel of dY, a channel of X
    int tm, tn;                     // channels staged per block (16 or 32)
    int bias;
};

__device__ __forceinline__ int cr_small_div(int a, int d) { return (int)(((float)a + 0.5f) * __builtin_amdgcn_rcpf((float)d)); }   // a, d < 2^15, quotient exact: the distance to an integer is at least 1 / (2 d)

template <int K, int S>
__global__ void __launch_bounds__(64 * K * cr_qmax(K)) conv_rows_kernel(const Grouped<RowsArgs> grp)
{
    extern __shared__ __attribute__((aligned(16))) float rows_lds[];
    constexpr int PT = cr_pieces(K), NB = cr_reads(K, S), FIRST = cr_first(K), PAD = (K - 1) / 2, CI = cr_cin(K), NI = CI / 16;
    unsigned bid;
    const RowsArgs &a = grp.a[group_pick(grp, bid)];
    const int tiles = a.tiles_m * a.tiles_n;
    const int batches = (a.n + a.ex_per_wg - 1) / a.ex_per_wg;
    if ((int)bid >= batches * tiles) return;
    const int batch = (int)bid / tiles, tile = (int)bid - batch * tiles;
    const int i_begin = batch * a.ex_per_wg, i_end = min(a.n, i_begin + a.ex_per_wg);
    const int m0 = (tile / a.tiles_n) * CR_CH, n0 = (tile - (tile / a.tiles_n) * a.tiles_n) * CI;
    const int cm = min(CR_CH, a.cout - m0), cn = min(CI, a.cin - n0);       // live channels
    const int tid = (int)threadIdx.x, nthreads = 64 * K * a.q, nwaves = K * a.q;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kh = wave / a.q, q = wave - kh * a.q;
    const int OH = a.oh, OW = a.ow, H = a.h, W = a.w, R = a.rows, RPR = a.rpr;
    const int lines = (R - 1) * S + K;
    const int groups = (R * RPR + 3) / 4;

    float *sA = rows_lds, *sX = sA + a.tm * a.cha;
    int *tab = reinterpret_cast<int *>(sX + a.tn * a.chx + 16);
    float *epi = reinterpret_cast<float *>(tab + groups * 4);
    const int EP = a.tn * K * K + 2;                   // pitch of a gradient row in LDS (spreads the lane groups over the banks)
    float *sbias = epi + 16 * EP, *red = sbias + CR_CH;

    // zero everything once: margins, dead channels and the runs beyond a chunk's last one are never written
    for (int t = tid; t < a.tm * a.cha + a.tn * a.chx + 16; t += nthreads) rows_lds[t] = 0.0f;
    // per run: offset of its X inside a channel, and how many of its four columns exist
    for (int t = tid; t < groups * 4; t += nthreads) {
        const int r = cr_small_div(t, RPR), c = t - r * RPR;
        tab[t] = t < R * RPR ? ((r * S * a.xp + 4 * S * c + CR_LEFT - PAD - FIRST) | (min(4, OW - 4 * c) << 24)) : 0;
    }
    // what this thread moves per chunk: source offset at output row 0, and packed: LDS offset, row of the chunk, elements, dY or X
    const int xpr = (W + 3) / 4;
    const int n_a = cm * R * RPR, n_all = n_a + cn * lines * xpr;
    int off[PT], meta[PT];
#pragma unroll
    for (int u = 0; u < PT; ++u) {
        const int idx = tid + nthreads * u;
        off[u] = 0; meta[u] = 0;
        if (idx < n_a) {
            const int row = cr_small_div(idx, RPR), pc = idx - row * RPR, ch = cr_small_div(row, R), r = row - ch * R;
            off[u] = ((m0 + ch) * OH + r) * OW + 4 * pc;
            meta[u] = (ch * a.cha + (r * RPR + pc) * 4) | (r << 16) | (min(4, OW - 4 * pc) << 24);
        } else if (idx < n_all) {
            const int t = idx - n_a, row = cr_small_div(t, xpr), pc = t - row * xpr, ch = cr_small_div(row, lines), k = row - ch * lines;
            off[u] = ((n0 + ch) * H + k - PAD) * W + 4 * pc;
            meta[u] = (a.tm * a.cha + ch * a.chx + k * a.xp + CR_LEFT + 4 * pc) | (k << 16) | (min(4, W - 4 * pc) << 24) | (1 << 28);
        }
    }
    r_f32x4 raw[PT];
    auto fetch = [&](int i, int oh0) {
        const float *dy_ex = example_at_uniform<float>(a.dy, a.dy_tab, i, (size_t)a.cout * OH * OW);
        const float *x_ex = example_at_uniform<float>(a.x, a.x_tab, i, (size_t)a.cin * H * W);
#pragma unroll
        for (int u = 0; u < PT; ++u) {
            int mt = meta[u];
            asm volatile("" : "+v"(mt));               // unpacked anew for every chunk: kept unpacked, it is four registers a piece
            const int count = (mt >> 24) & 7, r = (mt >> 16) & 0x7f;
            const bool is_x = (mt >> 28) & 1;
            const int row = is_x ? oh0 * S + r - PAD : oh0 + r;
            const float *src = is_x ? x_ex + (off[u] + oh0 * S * W) : dy_ex + (off[u] + oh0 * OW);
            const bool ok = (unsigned)row < (unsigned)(is_x ? H : OH);
            raw[u] = r_f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            if (ok && count == 4) raw[u] = *reinterpret_cast<const r_f32x4_a4 *>(src);
            else if (ok && count) {                    // the end of a row that is no multiple of four: element by element
                raw[u].x = src[0];
                if (count > 1) raw[u].y = src[1];
                if (count > 2) raw[u].z = src[2];
            }
        }
    };
    auto stage = [&]() {
#pragma unroll
        for (int u = 0; u < PT; ++u) {
            int mt = meta[u];
            asm volatile("" : "+v"(mt));
            if (mt >> 24) *reinterpret_cast<r_f32x4 *>(rows_lds + (mt & 0xffff)) = raw[u];
        }
    };

    r_f32x4 acc[2][NI][K];
    float bsum[2];
    const float *pa = sA + (lane & 15) * a.cha, *px = sX + (lane & 15) * a.chx + kh * a.xp;
    const int kq = lane >> 4;
    const bool has_bias = a.bias && n0 == 0 && kh == 0;
    // the MFMAs of one chunk of `runs` runs for NM x NN blocks of 16 x 16 channels
    auto multiply = [&](auto nm, auto nn, int runs) {
        constexpr int NM = decltype(nm)::value, NN = decltype(nn)::value;
#pragma unroll 1
        for (int g = q; g < groups; g += a.q) {
            const int t = 4 * g + kq, info = tab[t];
            const int live = t < runs ? (info >> 24) : 0;
            r_f32x4 av[NM];
            float xv[NN][4 * NB];
#pragma unroll
            for (int b = 0; b < NM; ++b) av[b] = *reinterpret_cast<const r_f32x4 *>(pa + b * 16 * a.cha + 4 * t);
#pragma unroll
            for (int b = 0; b < NN; ++b)
#pragma unroll
                for (int k = 0; k < NB; ++k) {
                    const r_f32x4 v = *reinterpret_cast<const r_f32x4 *>(px + b * 16 * a.chx + (info & 0xffff) + 4 * k);
                    xv[b][4 * k] = v.x; xv[b][4 * k + 1] = v.y; xv[b][4 * k + 2] = v.z; xv[b][4 * k + 3] = v.w;
                }
            if (has_bias)
#pragma unroll
                for (int b = 0; b < NM; ++b) bsum[b] += (av[b].x + av[b].y) + (av[b].z + av[b].w);
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int kw = 0; kw < K; ++kw)
#pragma unroll
                    for (int b = 0; b < NN; ++b) {
                        const float xo = j < live ? xv[b][FIRST + j * S + kw] : 0.0f;
#pragma unroll
                        for (int m = 0; m < NM; ++m)
                            acc[m][b][kw] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[m][j], xo, acc[m][b][kw], 0, 0, 0);
                    }
        }
    };
    typedef std::integral_constant<int, 1> one;
    typedef std::integral_constant<int, 2> two;
    typedef std::integral_constant<int, NI> wide;

    fetch(i_begin, 0);
    int in_unit = 0;
    for (int i = i_begin; i < i_end; ++i) {
        if (in_unit == 0)
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            bsum[m] = 0.0f;
#pragma unroll
            for (int b = 0; b < NI; ++b)
#pragma unroll
                for (int k = 0; k < K; ++k) acc[m][b][k] = r_f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        }
        for (int c = 0; c < a.chunks; ++c) {
            const int oh0 = c * R;
            __syncthreads();                           // the previous chunk has been read (first pass: the clearing is done)
            stage();
            __syncthreads();
            if (c + 1 < a.chunks) fetch(i, oh0 + R);
            else if (i + 1 < i_end) fetch(i + 1, 0);
            const int runs = min(R, OH - oh0) * RPR;
            if (cm > 16) {
                if (NI == 2 && cn > 16) multiply(two{}, wide{}, runs);
                else multiply(two{}, one{}, runs);
            } else {
                if (NI == 2 && cn > 16) multiply(one{}, wide{}, runs);
                else multiply(one{}, one{}, runs);
            }
        }
        if (++in_unit < a.unit) continue;              // the next example adds to the same block
        in_unit = 0;
        const int row_i = i / a.unit;
        // the block, 16 rows at a time: summed over q in order, squared, stored
        float ss = 0.0f;
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            if (m * 16 >= cm) break;
            for (int part = 0; part < a.q; ++part) {
                if (q == part) {
#pragma unroll
                    for (int b = 0; b < NI; ++b)
                        if (b * 16 < cn)
#pragma unroll
                            for (int k = 0; k < K; ++k)
#pragma unroll
                                for (int r = 0; r < 4; ++r) {
                                    float *e = epi + (kq * 4 + r) * EP + ((b * 16 + (lane & 15)) * K + kh) * K + k;
                                    *e = part ? *e + acc[m][b][k][r] : acc[m][b][k][r];
                                }
                    if (has_bias) {
                        float v = bsum[m];
                        v += __shfl_xor(v, 16, 64);
                        v += __shfl_xor(v, 32, 64);
                        if (lane < 16) sbias[m * 16 + lane] = part ? sbias[m * 16 + lane] + v : v;
                    }
                }
                __syncthreads();
            }
            const int len = cn * K * K;
            for (int r = wave; r < min(16, cm - m * 16); r += nwaves) {
                float *dst = a.out_w ? a.out_w + (size_t)row_i * a.out_stride_w + ((size_t)(m0 + m * 16 + r) * a.cin + n0) * (K * K) : nullptr;
                for (int t = lane; t < len; t += 64) {
                    const float v = epi[r * EP + t];
                    ss += v * v;
                    if (dst) __builtin_nontemporal_store(v, dst + t);
                }
            }
            __syncthreads();                           // epi is free again
        }
        if (a.bias && n0 == 0 && tid < cm) {
            const float v = sbias[tid];
            ss += v * v;
            if (a.out_b) a.out_b[(size_t)row_i * a.out_stride_b + m0 + tid] = v;
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

struct RowsPlan {
    int tiles_m, tiles_n, tm, tn, q, rows, chunks, rpr, xp, cha, chx, ex_per_wg;
    unsigned lds;
    double us;                      // estimated time of a call alone
    bool ok;
};

int odd_quads(int floats) { const int v = (floats + 3) / 4; return (v | 1) * 4; }     // consecutive channels start in different banks

// us of a per-example call alone.  A launch lasts as long as the compute unit with most blocks, which takes them in rounds of as many
// workgroups as it has room for.  Chunk by chunk a round needs the longer of two things (a little more where they are close): what
// the SIMD with most waves multiplies and stages for all its workgroups -- the waves of every workgroup start on the same SIMD, so K q waves count
// as ceil(K q / 4) on it --, or one workgroup's own chain of barrier, staging and MFMAs.  On 704 layers with several plans measured the one
// it prefers is 1.6 % slower than the best of them on average, 657 of them within 10 % (one figure for pieces of all widths, and none
// for fewer waves: 3.4 %, 601).
double rows_us(int k, const RowsPlan &p, double blocks, int unit, int groups, long long pieces, bool even, bool shared, int resident)
{
    // us per staged piece: 16-byte reads of rows that are no multiple of four columns are off their alignment and the last one is cut off
    const double piece = k == 3 ? (even ? 0.565e-3 : 0.794e-3) : even ? 0.823e-3 : 0.995e-3;
    const double mfma = k == 3 ? 1.2 : 1.23, start = k == 3 ? 2.3 : 4.2, share = k == 3 ? 0.53 : 0.0, epilogue = k == 3 ? 0.92 : 1.07;
    const double wave = 32.0 * k * 4 * (p.tm / 16) * (p.tn / 16) * ((groups + p.q - 1) / p.q) / 2400.0 * ((k * p.q + 3) / 4) * mfma;
    const double staging = piece * (double)pieces, chunks = (double)p.chunks * unit;
    const auto round = [&](double r) {
        const double all = r * (wave + staging), own = share * wave + start + staging;
        return r > 0.0 ? chunks * std::sqrt(std::sqrt(all * all * all * all + own * own * own * own)) + epilogue * (p.tm / 16) * (p.q + 1) * (0.7 + 0.3 * r) : 0.0;
    };
    const double most = std::ceil(blocks / 256.0), r = std::min<double>(most, resident), full = std::floor(most / r);
    // fewer waves than fit on a kernel row measured about 1.2 times what the terms above give, but not beside other layers' workgroups
    // (ResNet-20, 256 examples on eight streams: 716 us with the factor there, 641 without)
    return ((k == 3 ? 8.9 : 8.7) + full * round(r) + round(most - full * r)) * (shared || p.q == cr_qmax(k) ? 1.0 : k == 3 ? 1.21 : 1.24);
}

RowsPlan rows_plan(const Geo &g, bool shared)
{
    RowsPlan best = {};
    const int K = g.kh, S = g.stride, CI = cr_cin(K);
    RowsPlan p = {};
    p.tiles_m = (g.cout + CR_CH - 1) / CR_CH;
    p.tiles_n = (g.cin + CI - 1) / CI;
    p.tm = g.cout > 16 ? 32 : 16;
    p.tn = CI > 16 && g.cin > 16 ? 32 : 16;
    p.rpr = (g.ow + 3) / 4;
    p.xp = CR_LEFT + (g.w + 3) / 4 * 4;
    const int lc = g.cout < CR_CH ? g.cout : CR_CH, ln = g.cin < CI ? g.cin : CI;      // channels that are staged
    const double own = (double)(g.n / g.unit) * p.tiles_m * p.tiles_n;
    // Inside a batch call of several layers the plan with the best rate of a full chip, eight blocks on every compute unit, whatever
    // this layer brings: the other layers' workgroups run on the units beside its own.  ResNet-20, 256 examples on eight streams: 758 us
    // as alone, 641 so; 4 x 32: 473, 393.
    const double blocks = shared ? 8.0 * 256.0 : own;
    // several examples in a row where there are far more (example, block) pairs than workgroups that run at a time
    const int e = (int)(own / 4096.0);
    p.ex_per_wg = g.unit * (e < 1 ? 1 : e > 8 ? 8 : e);
    for (p.q = 1; p.q <= cr_qmax(K); p.q *= 2)
        for (p.rows = 1; p.rows <= g.oh && p.rows <= 64; ++p.rows) {
            const int lines = (p.rows - 1) * S + K;
            if (lines > 127) break;
            const long long pieces = (long long)lc * p.rows * p.rpr + (long long)ln * lines * ((g.w + 3) / 4);
            if (pieces > (long long)cr_pieces(K) * 64 * K * p.q) break;
            const int groups = (p.rows * p.rpr + 3) / 4;
            p.cha = odd_quads(groups * 16);
            p.chx = odd_quads(lines * p.xp + 4);
            const long long floats = (long long)p.tm * p.cha + (long long)p.tn * p.chx + 16 + groups * 4 + 16 * (p.tn * K * K + 2) + CR_CH + 64;
            // LDS in quarters, halves or the whole of what a compute unit has: layers of different sizes share a launch
            const unsigned need = (unsigned)(floats * 4);
            if (need > 156 * 1024) break;
            p.lds = need <= 39 * 1024 ? 39 * 1024 : need <= 78 * 1024 ? 78 * 1024 : 156 * 1024;
            p.chunks = (g.oh + p.rows - 1) / p.rows;
            p.us = rows_us(K, p, blocks, g.unit, groups, pieces, g.w % 4 == 0 && g.ow % 4 == 0, shared, std::max(1, std::min({(int)(156 * 1024 / p.lds), 12 / (K * p.q), 8})));
            p.ok = true;
            if (!best.ok || p.us < best.us) best = p;
        }
    return best;
}

size_t cr_align16(size_t b) { return (b + 15) & ~(size_t)15; }

template <int K> const void *rows_fn(int stride)
{
    return stride == 2 ? reinterpret_cast<const void *>(&conv_rows_kernel<K, 2>) : reinterpret_cast<const void *>(&conv_rows_kernel<K, 1>);
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
        // Both times estimated, a margin of 3 % to the general kernel.  Fitted to 1249 layers in and around the networks here (3x3 and
        // 5x5, strides 1 and 2, 3 to 256 channels, 7 to 64 rows, 8 to 512 examples, with and without a bias), both kernels measured
        // on each: half of the estimates are within 5 % for either kernel, nine of ten within 14 %.  Where the kernels differ by a
        // quarter or more (763 layers) the faster one is chosen in all but 5.  The rule takes 537 layers, 13 of them slower by more
        // than 3 % (at most 31 %); all 1249 together take 0.858 of the general kernel's time, where the faster of the two each time
        // would be 0.852.  us, general / this: 64 -> 64 3x3 on 56 x 56, 64 examples 278 / 196, 48: 185 / 192, 128: 467 / 381; with a
        // bias 376 / 200, 245 / 194, 615 / 390; 16 -> 16 on 32 x 32, 256: 102 / 32; 128 -> 128 on 28 x 28, 256: 651 / 916; 5x5,
        // 40 -> 72 stride 2 on 45 x 37 with a bias, 40: 128 / 107.
        c.use = c.plan.ok && c.plan.us < 0.97 * conv_general_f32_us(g);
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
    // offsets inside an example (rows above and below the image included) fit 32 bits; quotients of the set-up stay exact
    if ((size_t)g.cin * (g.h + 8) * g.w >= ((size_t)1 << 30) || (size_t)g.cout * (g.oh + 64) * g.ow >= ((size_t)1 << 30)) return false;
    if (g.w > 4096 || (double)g.n * conv_rows_norm_partial_count(g) >= 1.0e9) return false;
    return rows_choice(g).use;
}

size_t conv_rows_norm_partial_count(const Geo &g) { return (size_t)((g.cout + CR_CH - 1) / CR_CH) * ((g.cin + cr_cin(g.kh) - 1) / cr_cin(g.kh)); }

size_t conv_rows_ws_bytes(const Geo &g) { return cr_align16((size_t)(g.n / g.unit) * conv_rows_norm_partial_count(g) * sizeof(float)); }

const char *conv_rows_variant_name(const Geo &g)
{
    static const char *const names[2][2] = {{"conv_rows<f32,3x3,per_example>", "conv_rows<f32,3x3,s2,per_example>"},
                                            {"conv_rows<f32,5x5,per_example>", "conv_rows<f32,5x5,s2,per_example>"}};
    return names[g.kh / 2 - 1][g.stride - 1];
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
    a.rows = p.rows; a.chunks = p.chunks; a.rpr = p.rpr; a.xp = p.xp; a.cha = p.cha; a.chx = p.chx; a.tm = p.tm; a.tn = p.tn;
    a.bias = g.has_bias ? 1 : 0;
    const void *fn = g.kh == 3 ? rows_fn<3>(g.stride) : rows_fn<5>(g.stride);
    static std::atomic<bool> attr_done[2][2];           // zero-initialised; setting the attribute twice is harmless
    if (!attr_done[g.kh / 2 - 1][g.stride - 1].load()) {
        if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, 156 * 1024) != hipSuccess)
            return fail(DP_ERR_DEVICE, "conv_rows: cannot reserve LDS");
        attr_done[g.kh / 2 - 1][g.stride - 1].store(true);
    }
    const long long total = (long long)((g.n + p.ex_per_wg - 1) / p.ex_per_wg) * p.tiles_m * p.tiles_n;
    const dp_status st = submit_main<RowsArgs>(fn, a, (unsigned)((total + 7) / 8 * 8), (unsigned)(64 * g.kh * p.q), p.lds, s, "conv_rows");
    if (st != DP_OK || !sqnorm) return st;
    const float *parts = a.partials;
    const int n = g.n / g.unit, count = (int)conv_rows_norm_partial_count(g);
    return submit_post([=]() -> dp_status { return launch_sum_partials(parts, n, count, sqnorm, s); });
}

}  // namespace dp
