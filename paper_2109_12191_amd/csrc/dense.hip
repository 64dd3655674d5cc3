// Per-example gradients of dense layers:  dW_i[o,k] = sum_t dY_i[t,o] X_i[t,k];  db_i[o] = sum_t dY_i[t,o].
//
// Both operands are stored with the contraction index (the token t) outermost, so neither is in the K-contiguous order
// the convolution kernels read.  Four kernels:
//   dense_outer_kernel       one token, gradients stored: the rank-one product dy_i (x) x_i, a streaming outer product
//   dense_rank1_norm_kernel  one token, norm only: |dy_i|^2 |x_i|^2 (+ |dy_i|^2)
//   dense_tokens_kernel      bf16, several tokens: bf16 MFMA; an 8 x 4 block (tokens x features) per thread is transposed in
//                            registers on its way into LDS
//   dense_rows_kernel        fp32 MFMA on operands that stay as they lie ([t][feature]: the operand order of the
//                            32x32x2 instruction): fp32 inputs, and the clip-weighted sum of bf16 layers with fewer than 16
//                            tokens, whose K runs over (example, token) with dY scaled in fp32
#include "internal.h"
#include "group.h"
#include "pieces.h"

#include <algorithm>
#include <atomic>

namespace dp {

namespace {

struct DenseArgs {
    const void *x, *dy;
    int x_tab, dy_tab;              // Geo::x_tab / dy_tab: the operand pointers are arrays of example addresses
    float *out_w, *out_b;
    size_t out_stride_w, out_stride_b;
    float *partials;                // per-example kernels: [n, partial count]
    const float *group_sqnorm;      // weighted: [n]
    float clip_c;
    int n, tokens, cin, cout, has_bias;
    int tiles_k, tiles_o;
};

// ------------------------------------------------------------------------------------------
// One token, gradients stored.  Workgroup tile: OUTER_ROWS rows (o) x 256 columns (k); a thread owns one column, so x loads
// and gradient stores are coalesced along k and dy values are wave-uniform.  Bound by the stores.
constexpr int OUTER_ROWS = 16;

template <bool BF16>
__global__ void __launch_bounds__(256) dense_outer_kernel(const Grouped<DenseArgs> grp)
{
    typedef typename In<BF16>::type E;
    __shared__ float red[4];
    unsigned bid;
    const DenseArgs &a = grp.a[group_pick(grp, bid)];
    const int tiles = a.tiles_k * a.tiles_o;
    const int i = (int)(bid / (unsigned)tiles), tile = (int)(bid - (unsigned)i * (unsigned)tiles);
    const int tile_o = tile / a.tiles_k, tile_k = tile - tile_o * a.tiles_k;
    const int k = tile_k * 256 + threadIdx.x, o0 = tile_o * OUTER_ROWS;
    const E *xi = example_at_uniform<E>(a.x, a.x_tab, (int)i, a.cin);
    const E *dyi = example_at_uniform<E>(a.dy, a.dy_tab, (int)i, a.cout);
    const float xv = k < a.cin ? In<BF16>::ld(xi + k) : 0.0f;
    float *out = a.out_w + (size_t)i * a.out_stride_w + (size_t)o0 * a.cin + k;
    float ss = 0.0f;
#pragma unroll
    for (int r = 0; r < OUTER_ROWS; ++r) {
        const float v = (o0 + r < a.cout ? In<BF16>::ld(dyi + o0 + r) : 0.0f) * xv;
        ss += v * v;
        if (k < a.cin && o0 + r < a.cout) out[(size_t)r * a.cin] = v;
    }
    if (a.has_bias && tile_k == 0 && threadIdx.x < OUTER_ROWS && o0 + (int)threadIdx.x < a.cout) {
        const float v = In<BF16>::ld(dyi + o0 + threadIdx.x);
        ss += v * v;
        a.out_b[(size_t)i * a.out_stride_b + o0 + threadIdx.x] = v;
    }
    const float tot = block_sum<4>(ss, red);
    if (threadIdx.x == 0) a.partials[(size_t)i * tiles + tile] = tot;
}

// One token per example: the gradient is the rank-one product dy_i (x) x_i (plus db_i = dy_i), so
// its squared Frobenius norm is |dy_i|^2 |x_i|^2 (+ |dy_i|^2) -- the same number H2 defines, from
// two short reductions instead of Cout*Cin products.  One workgroup per example.
template <bool BF16>
__global__ void __launch_bounds__(256) dense_rank1_norm_kernel(const Grouped<DenseArgs> grp)
{
    typedef typename In<BF16>::type E;
    __shared__ float red[4];
    unsigned i;
    const DenseArgs &a = grp.a[group_pick(grp, i)];
    const E *xi = example_at_uniform<E>(a.x, a.x_tab, (int)i, a.cin);
    const E *dyi = example_at_uniform<E>(a.dy, a.dy_tab, (int)i, a.cout);
    float sx = 0.0f, sd = 0.0f;
    for (int k = threadIdx.x; k < a.cin; k += 256) { const float v = In<BF16>::ld(xi + k); sx += v * v; }
    for (int o = threadIdx.x; o < a.cout; o += 256) { const float v = In<BF16>::ld(dyi + o); sd += v * v; }
    sx = block_sum<4>(sx, red);
    sd = block_sum<4>(sd, red);
    if (threadIdx.x == 0) a.partials[i] = sd * sx + (a.has_bias ? sd : 0.0f);
}

// ------------------------------------------------------------------------------------------
// What the two MFMA kernels share.  A workgroup owns a 64 (o) x 64 (k) tile of the gradient; `G` groups of four waves (each
// wave a 32 x 32 block) take every G-th step of K, so that the few tiles of a weighted call, whose K is the whole micro-step,
// are not one long serial chain each; the groups' blocks are added in group order through LDS (same bits on every run).
//
// Result of a tile in the MFMA accumulator layout of the first group's waves: stored and squared, or added to the accumulator.
constexpr int DT = 64;

template <bool WEIGHTED>
__device__ __forceinline__ void dense_tile_out(const f32x16 &acc, const f32x16 &accb, const DenseArgs &a, int i, int tile, int tiles,
                                               int o0, int k0, int wm, int wn, int lane, bool bias_here, float *red, bool first_group)
{
    float ss = 0.0f;
    if (first_group) {
        const int col = k0 + wn * 32 + (lane & 31), row0 = o0 + wm * 32 + (lane >> 5) * 4;
        float *out = a.out_w ? a.out_w + (WEIGHTED ? 0 : (size_t)i * a.out_stride_w) : nullptr;
        float old[16];
        if constexpr (WEIGHTED) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {                            // all loads before the first add
                const int row = row0 + (r >> 2) * 8 + (r & 3);
                old[r] = (row < a.cout && col < a.cin) ? out[(size_t)row * a.cin + col] : 0.0f;
            }
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int row = row0 + (r >> 2) * 8 + (r & 3);
            if (row < a.cout && col < a.cin) {
                ss += acc[r] * acc[r];
                if constexpr (WEIGHTED) out[(size_t)row * a.cin + col] = old[r] + acc[r];
                else if (out) out[(size_t)row * a.cin + col] = acc[r];
            }
        }
        if (bias_here && (lane & 31) == 0) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = row0 + (r >> 2) * 8 + (r & 3);
                if (row < a.cout) {
                    ss += accb[r] * accb[r];
                    if constexpr (WEIGHTED) a.out_b[row] += accb[r];
                    else if (out) a.out_b[(size_t)i * a.out_stride_b + row] = accb[r];
                }
            }
        }
    }
    if constexpr (!WEIGHTED) {
        const float tot = block_sum<4>(ss, red);
        if (threadIdx.x == 0) a.partials[(size_t)i * tiles + tile] = tot;
    }
}

// Blocks of groups 1 .. G-1 added to group 0's, in order.  `buf` holds 64 * 64 floats per group after the first
// (plus 64 for the bias).
template <int G>
__device__ __forceinline__ void dense_add_groups(f32x16 &acc, f32x16 &accb, float *buf, int group, int t, bool bias_here)
{
    if constexpr (G > 1) {
        __syncthreads();                                             // everyone is done with the operands in LDS
        constexpr int PER = 2 * 16 * 256;
        if (group > 0) {
            float *mine = buf + (group - 1) * PER;
#pragma unroll
            for (int r = 0; r < 16; ++r) mine[r * 256 + t] = acc[r];
            if (bias_here) {
#pragma unroll
                for (int r = 0; r < 16; ++r) mine[(16 + r) * 256 + t] = accb[r];
            }
        }
        __syncthreads();
        if (group == 0) {
#pragma unroll 1
            for (int g = 1; g < G; ++g) {
                const float *theirs = buf + (g - 1) * PER;
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[r] += theirs[r * 256 + t];
                if (bias_here) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) accb[r] += theirs[(16 + r) * 256 + t];
                }
            }
        }
    }
}

// ------------------------------------------------------------------------------------------
// bf16, several tokens.  A step is 64 tokens of one example: per operand a thread loads 8 features of 4 consecutive tokens
// (8 threads cover 128 bytes of a row; with 4 features a thread and 16 threads a row the loads took 1.6 x as long, with
// neighbouring threads in different rows 2.7 x), transposes the block with byte permutes and writes eight 8-byte runs of K
// into LDS rows of 128 bytes.  The 16-byte piece p of row r lies in slot p ^ f(r), f(r) = (r >> 1 ^ r >> 3) & 7: the operand
// reads (16 rows at one K) touch 16 different bank groups, the writes (rows 8 apart) 8.  The next step's loads are in flight
// during the MFMAs; double-buffered LDS, one barrier per step.
// Weighted: the finished block of an example is scaled by its clip factor in fp32 and added to a second set of accumulators.
// 16 x 128 tokens, 768 -> 768 with bias: norm-only call 454 -> 17 us, weighted 2634 -> 24 us against one scalar multiply-add
// kernel for both; bound by the rate at which a compute unit takes in pieces of 128 bytes (about 28 bytes a clock).
typedef uint32_t u32x4_b4 __attribute__((ext_vector_type(4), aligned(4)));   // 16 bytes, dword aligned
constexpr int DTK = 64, DT_PITCH = 128, DT_STAGE = 2 * DT * DT_PITCH;

template <bool WEIGHTED, int G>
__global__ void __launch_bounds__(256 * G, G == 1 ? 2 : 4) dense_tokens_kernel(const Grouped<DenseArgs> grp)
{
    extern __shared__ __attribute__((aligned(16))) char dense_lds[];
    __shared__ float red[4];
    unsigned bid;
    const DenseArgs &a = grp.a[group_pick(grp, bid)];
    const int tiles = a.tiles_k * a.tiles_o;
    const int ex = WEIGHTED ? 0 : (int)(bid / (unsigned)tiles);
    const int tile = (int)(bid - (unsigned)ex * (unsigned)tiles);
    const int tile_o = tile / a.tiles_k, tile_k = tile - tile_o * a.tiles_k;
    const int o0 = tile_o * DT, k0 = tile_k * DT;
    const int group = (int)(threadIdx.x >> 8), t = threadIdx.x & 255, lane = t & 63, wave = t >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    char *lds = dense_lds + group * (2 * DT_STAGE);

    // this thread's block of a step: operand, eight features, four tokens.  An element lies at a wave-uniform base (example,
    // step, row within the block) plus `off`, which never changes and is even, so the parity of a row that starts on an odd
    // element is uniform too.  Features beyond the layer read the last ones again (never stored, not in the norm).
    const bool is_x = __builtin_amdgcn_readfirstlane(t >> 7) != 0;
    const int cb = t & 7, tb = (t & 127) >> 3;
    const int C = is_x ? a.cin : a.cout, col = min((is_x ? k0 : o0) + cb * 8, (C - 1) & ~7);
    const unsigned off = 2u * ((unsigned)tb * 4u * (unsigned)C + (unsigned)col);
    const void *const operand = is_x ? a.x : a.dy;
    const int tab = is_x ? a.x_tab : a.dy_tab;
    const bool even = (C & 1) == 0;
    char *dst = lds + ((is_x ? DT : 0) + cb * 8) * DT_PITCH + (tb & 1) * 8;
    const int slot0 = (tb >> 1) ^ cb ^ ((cb & 1) << 2);                      // slot of feature c of the block: slot0 ^ (c >> 1)

    const int tokens = a.tokens, cpe = (tokens + DTK - 1) / DTK, n_ex = a.n;
    const unsigned long long ex_elems = (unsigned long long)tokens * (unsigned)C;
    const int first_ex = WEIGHTED ? __builtin_amdgcn_readfirstlane(group) : ex, ex_step = G;
    const int mine = WEIGHTED ? (n_ex - first_ex + G - 1) / G * cpe : cpe;    // steps of this group
    const int all = WEIGHTED ? (n_ex + G - 1) / G * cpe : cpe;                // steps of the longest group

    uint32_t raw[4][5];
    int f_ex = first_ex, f_c = 0;                                             // next step to fetch
    int r_valid = 0;                                                          // of the fetched step: tokens that exist,
    uint32_t r_odd = 0;                                                       //   rows that start on an odd element,
    const uint16_t *r_slow = nullptr;                                         //   or where to stage it from element by element
    auto fetch = [&]() {
        // elements count from the start of the tensor, or from the dword an example with an address of its own starts in
        const char *src = static_cast<const char *>(operand);
        unsigned long long e0 = f_ex * ex_elems, total = n_ex * ex_elems;
        if (tab) {
            const unsigned long long at = reinterpret_cast<unsigned long long>(example_at_uniform<uint16_t>(operand, tab, f_ex, 0));
            src = reinterpret_cast<const char *>(at & ~3ull);
            e0 = (at >> 1) & 1u;
            total = e0 + ex_elems;
        }
        e0 += (unsigned long long)(unsigned)(f_c * DTK) * (unsigned)C;
        const int valid = min(tokens - f_c * DTK, DTK);
        r_valid = valid;
        r_odd = 0;
        // the last block of a row reads up to seven elements beyond it, an odd row two more: not at the tensor's very end
        r_slow = ((C & 7) && e0 + (unsigned long long)valid * (unsigned)C + 9 > total) ? reinterpret_cast<const uint16_t *>(src) + e0 : nullptr;
        if (++f_c == cpe) { f_c = 0; f_ex += ex_step; }
        if (r_slow) return;
        if (valid == DTK) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const unsigned long long e = e0 + (unsigned)(r * C);
                const char *p = src + (e >> 1) * 4 + off;
                const u32x4_b4 v = *reinterpret_cast<const u32x4_b4 *>(p);
                raw[r][0] = v.x; raw[r][1] = v.y; raw[r][2] = v.z; raw[r][3] = v.w;
                if (!even) {
                    raw[r][4] = *reinterpret_cast<const uint32_t *>(p + 16);
                    r_odd |= (uint32_t)(e & 1) << r;
                }
            }
        } else {                                                              // rows beyond the last token read that one again
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const unsigned long long e = e0 + ((unsigned)min(tb * 4 + r, valid - 1) * (unsigned)C + (unsigned)col);
                const char *p = src + (e >> 1) * 4;
                const u32x4_b4 v = *reinterpret_cast<const u32x4_b4 *>(p);
                raw[r][0] = v.x; raw[r][1] = v.y; raw[r][2] = v.z; raw[r][3] = v.w;
                if (!even) {                                                  // (here the parity differs from lane to lane)
                    raw[r][4] = *reinterpret_cast<const uint32_t *>(p + 16);
                    r_odd |= (uint32_t)(e & 1) << r;
                }
            }
        }
    };
    auto stage = [&](int buf) {
        char *d = dst + buf * DT_STAGE;
        if (r_slow) {
#pragma unroll 1
            for (int q = 0; q < 32; ++q) {
                const int r = q & 3, c = q >> 2;
                const bool there = tb * 4 + r < r_valid && col + c < C;
                *reinterpret_cast<uint16_t *>(d + c * DT_PITCH + (slot0 ^ (c >> 1)) * 16 + r * 2) = there ? r_slow[(size_t)(tb * 4 + r) * C + col + c] : (uint16_t)0;
            }
            return;
        }
        if (!even) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const uint32_t bits = ((r_odd >> r) & 1u) * 16u;
#pragma unroll
                for (int j = 0; j < 4; ++j) raw[r][j] = funnel(raw[r][j + 1], raw[r][j], bits);
            }
        }
        if (!is_x && r_valid < DTK) {                                         // zeros of dY meet whatever X holds there
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (tb * 4 + r >= r_valid) raw[r][0] = raw[r][1] = raw[r][2] = raw[r][3] = 0u;
        }
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const uint32_t sel = (c & 1) ? 0x07060302u : 0x05040100u;         // high or low halves of two dwords
            *reinterpret_cast<uint2 *>(d + c * DT_PITCH + (slot0 ^ (c >> 1)) * 16) =
                make_uint2(__builtin_amdgcn_perm(raw[1][c >> 1], raw[0][c >> 1], sel), __builtin_amdgcn_perm(raw[3][c >> 1], raw[2][c >> 1], sel));
        }
    };

    f32x16 acc, accb, tot, totb;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = accb[r] = tot[r] = totb[r] = 0.0f;
    const bool bias_here = a.has_bias && tile_k == 0 && wn == 0;

    // byte offset of K step 0 in this lane's operand rows (K step ks: exclusive or with 32 ks)
    auto first_slot = [&](int row) { return ((lane >> 5) ^ (((row >> 1) ^ (row >> 3)) & 7)) * 16; };
    const int slot_a = first_slot(wm * 32 + (lane & 31)), slot_b = first_slot(wn * 32 + (lane & 31));

    if (mine > 0) { fetch(); stage(0); }
    __syncthreads();
    int c_ex = first_ex, c_c = 0;
    for (int s = 0; s < all; ++s) {
        if (s + 1 < mine) fetch();
        if (s < mine) {
            const char *pa = lds + (s & 1) * DT_STAGE + (wm * 32 + (lane & 31)) * DT_PITCH;
            const char *pb = lds + (s & 1) * DT_STAGE + (DT + wn * 32 + (lane & 31)) * DT_PITCH;
            const int ksteps = (min(a.tokens - c_c * DTK, DTK) + 15) >> 4;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                if (ks < ksteps) {
                    const bf16x8 va = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(pa + (slot_a ^ (ks * 32))));
                    const bf16x8 vb = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(pb + (slot_b ^ (ks * 32))));
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, vb, acc, 0, 0, 0);
                    if (bias_here) {
                        const uint4 one = make_uint4(0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u);
                        accb = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, __builtin_bit_cast(bf16x8, one), accb, 0, 0, 0);
                    }
                }
            }
            if (++c_c == cpe) {
                c_c = 0;
                if constexpr (WEIGHTED) {
                    const float f = clip_factor(a.group_sqnorm[c_ex], a.clip_c);
                    // an example whose gradient overflows has factor 0: it adds nothing, and no 0 * inf.  (Rare: cleared first, the additions
                    // below as without it.  16 x 128 tokens, 768 -> 768: 24.36 us without, 24.41 so, 24.8 with a branch around the additions)
                    if (__builtin_expect(f == 0.0f, 0)) {
#pragma unroll
                        for (int r = 0; r < 16; ++r) acc[r] = accb[r] = 0.0f;
                    }
#pragma unroll
                    for (int r = 0; r < 16; ++r) { tot[r] += f * acc[r]; acc[r] = 0.0f; }
                    if (bias_here) {
#pragma unroll
                        for (int r = 0; r < 16; ++r) { totb[r] += f * accb[r]; accb[r] = 0.0f; }
                    }
                    c_ex += ex_step;
                }
            }
        }
        if (s + 1 < mine) stage((s + 1) & 1);
        __syncthreads();
    }
    if constexpr (WEIGHTED) {
        dense_add_groups<G>(tot, totb, reinterpret_cast<float *>(dense_lds), group, t, bias_here);
        dense_tile_out<true>(tot, totb, a, 0, tile, tiles, o0, k0, wm, wn, lane, bias_here, red, group == 0);
    } else {
        dense_tile_out<false>(acc, accb, a, ex, tile, tiles, o0, k0, wm, wn, lane, bias_here, red, true);
    }
}

// ------------------------------------------------------------------------------------------
// fp32 MFMA on rows as they lie: a step is 32 rows (tokens of an example; weighted: rows (example, token) of the whole
// micro-step, dY scaled by its example's factor in fp32 while it is staged) of 64 features of either operand, in LDS rows of
// 68 floats (an operand is 32 consecutive floats of two rows).  bf16 inputs are widened on the way.
constexpr int DRK = 32, DR_PITCH = 68, DR_STAGE = 2 * DRK * DR_PITCH;         // floats

template <bool BF16, bool WEIGHTED, int G>
__global__ void __launch_bounds__(256 * G, G == 1 ? 2 : 4) dense_rows_kernel(const Grouped<DenseArgs> grp)
{
    typedef typename In<BF16>::type E;
    extern __shared__ __attribute__((aligned(16))) char dense_lds[];
    __shared__ float red[4];
    unsigned bid;
    const DenseArgs &a = grp.a[group_pick(grp, bid)];
    const int tiles = a.tiles_k * a.tiles_o;
    const int ex = WEIGHTED ? 0 : (int)(bid / (unsigned)tiles);
    const int tile = (int)(bid - (unsigned)ex * (unsigned)tiles);
    const int tile_o = tile / a.tiles_k, tile_k = tile - tile_o * a.tiles_k;
    const int o0 = tile_o * DT, k0 = tile_k * DT;
    const int group = (int)(threadIdx.x >> 8), t = threadIdx.x & 255, lane = t & 63, wave = t >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    float *lds = reinterpret_cast<float *>(dense_lds) + group * (2 * DR_STAGE);

    // row `rb + 8 u` of a step, four features: a wave-uniform base (step, u) plus offsets that never change.  Features beyond the
    // layer read the last one again (never stored, not in the norm), rows beyond the last one that row (zeros of dY meet it).
    const bool is_x = __builtin_amdgcn_readfirstlane(t >> 7) != 0;
    const int cb = t & 15, rb = (t & 127) >> 4;
    const int C = is_x ? a.cin : a.cout, col = (is_x ? k0 : o0) + cb * 4;
    const bool aligned = (C & 3) == 0;
    unsigned off[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) off[c] = (unsigned)sizeof(E) * ((unsigned)rb * (unsigned)C + (unsigned)min(col + c, C - 1));
    if (aligned) off[0] = (unsigned)sizeof(E) * ((unsigned)rb * (unsigned)C + (unsigned)min(col, C - 4));
    const void *const operand = is_x ? a.x : a.dy;
    const int tab = is_x ? a.x_tab : a.dy_tab;
    const char *src = reinterpret_cast<const char *>(WEIGHTED ? static_cast<const E *>(operand) : example_at_uniform<E>(operand, tab, ex, (size_t)a.tokens * C));
    float *dst = lds + (is_x ? DRK * DR_PITCH : 0) + rb * DR_PITCH + cb * 4;
    const int tokens = a.tokens;
    const long long rows = WEIGHTED ? (long long)a.n * tokens : tokens;
    const int all = (int)((rows + DRK * G - 1) / (DRK * G));                   // steps of every group (the last may be empty)

    float v[4][4], f[4];
    long long f_row = __builtin_amdgcn_readfirstlane(group) * DRK;
    auto fetch = [&]() {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const long long over = max(0ll, f_row + 8 * u + rb - (rows - 1));
            const char *p = src + ((f_row + 8 * u) * C - over * C) * (long long)sizeof(E);
            if (WEIGHTED && tab) {                                             // the row's example has an address of its own
                const long long row = f_row + 8 * u + rb - over, i = row / tokens;
                p = reinterpret_cast<const char *>(example_at<E>(operand, tab, (int)i, 0)) + ((row - i * tokens) * C - (long long)rb * C) * (long long)sizeof(E);
            }
            if (aligned) {
                if constexpr (BF16) {
                    const uint2 w = *reinterpret_cast<const uint2 *>(p + off[0]);
                    v[u][0] = __uint_as_float(w.x << 16); v[u][1] = __uint_as_float(w.x & 0xFFFF0000u);
                    v[u][2] = __uint_as_float(w.y << 16); v[u][3] = __uint_as_float(w.y & 0xFFFF0000u);
                } else {
                    const float4 w = *reinterpret_cast<const float4 *>(p + off[0]);
                    v[u][0] = w.x; v[u][1] = w.y; v[u][2] = w.z; v[u][3] = w.w;
                }
            } else {
#pragma unroll
                for (int c = 0; c < 4; ++c) v[u][c] = In<BF16>::ld(reinterpret_cast<const E *>(p + off[c]));
            }
            f[u] = over > 0 ? -1.0f : 0.0f;                                    // (a negative norm: factor 0)
            if (WEIGHTED && !is_x && over == 0) {
                const long long row = f_row + 8 * u + rb;
                const long long i = tokens == 1 ? row : (rows >> 32 ? row / tokens : (long long)((unsigned)row / (unsigned)tokens));
                f[u] = a.group_sqnorm[i];
            }
        }
    };
    auto stage = [&](int buf) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (!is_x) {
                const float fu = WEIGHTED ? clip_factor(f[u], a.clip_c) : 1.0f + f[u];
                if (fu == 0.0f) v[u][0] = v[u][1] = v[u][2] = v[u][3] = 0.0f;
                else if (WEIGHTED) { v[u][0] *= fu; v[u][1] *= fu; v[u][2] *= fu; v[u][3] *= fu; }
            }
            *reinterpret_cast<float4 *>(dst + buf * DR_STAGE + 8 * u * DR_PITCH) = make_float4(v[u][0], v[u][1], v[u][2], v[u][3]);
        }
        f_row += G * DRK;
    };

    f32x16 acc, accb;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = accb[r] = 0.0f;
    const bool bias_here = a.has_bias && tile_k == 0 && wn == 0;
    fetch();
    stage(0);
    __syncthreads();
    for (int s = 0; s < all; ++s) {
        const int left = (int)max(0ll, min((long long)DRK, rows - ((long long)s * G + group) * DRK));     // rows of this step that exist
        if (s + 1 < all) fetch();
        const float *pa = lds + (s & 1) * DR_STAGE + (lane >> 5) * DR_PITCH + wm * 32 + (lane & 31);
        const float *pb = lds + (s & 1) * DR_STAGE + (DRK + (lane >> 5)) * DR_PITCH + wn * 32 + (lane & 31);
        auto mul = [&](int kk) {
            const float va = pa[2 * kk * DR_PITCH], vb = pb[2 * kk * DR_PITCH];
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(va, vb, acc, 0, 0, 0);
            if (bias_here) accb = __builtin_amdgcn_mfma_f32_32x32x2f32(va, 1.0f, accb, 0, 0, 0);
        };
        if (left == DRK) {
#pragma unroll
            for (int kk = 0; kk < DRK / 2; ++kk) mul(kk);
        } else {
#pragma unroll 1
            for (int kk = 0; 2 * kk < left; ++kk) mul(kk);
        }
        if (s + 1 < all) stage((s + 1) & 1);
        __syncthreads();
    }
    dense_add_groups<G>(acc, accb, reinterpret_cast<float *>(dense_lds), group, t, bias_here);
    dense_tile_out<WEIGHTED>(acc, accb, a, ex, tile, tiles, o0, k0, wm, wn, lane, bias_here, red, group == 0);
}

// ------------------------------------------------------------------------------------------
enum DenseRoute { DENSE_NORM1, DENSE_OUTER, DENSE_TOKENS, DENSE_ROWS };

// Which kernel: with one token there is nothing to contract per example.  The clip-weighted sum of bf16 layers needs at least
// 16 tokens to fill an MFMA of an example's own (its factor is applied to the finished block, in fp32).
DenseRoute dense_route(const Geo &g, int mode)
{
    if (g.h == 1 && mode == MODE_NORM) return DENSE_NORM1;
    if (g.h == 1 && mode == MODE_MATERIALISE) return DENSE_OUTER;
    return g.bf16 && (mode != MODE_WEIGHTED || g.h >= 16) ? DENSE_TOKENS : DENSE_ROWS;
}

size_t mfma_tiles(const Geo &g) { return (size_t)((g.cin + DT - 1) / DT) * ((g.cout + DT - 1) / DT); }

}  // namespace

size_t dense_norm_partial_count(const Geo &g, int mode)
{
    switch (dense_route(g, mode)) {
    case DENSE_NORM1: return 1;                       // rank-one closed form: one value per example
    case DENSE_OUTER: return (size_t)((g.cin + 255) / 256) * ((g.cout + OUTER_ROWS - 1) / OUTER_ROWS);
    default: return mfma_tiles(g);
    }
}

// A slot for every OUTER_ROWS x 256 of the gradient: the layers that the entry point with built-in scratch takes
size_t dense_scratch_bytes(const Geo &g)
{
    return (size_t)g.n * ((g.cin + 255) / 256) * ((g.cout + OUTER_ROWS - 1) / OUTER_ROWS) * sizeof(float);
}

size_t dense_ws_bytes(const Geo &g, int mode)
{
    if (mode == MODE_WEIGHTED) return 0;
    const size_t need = (size_t)g.n * dense_norm_partial_count(g, MODE_MATERIALISE) * sizeof(float);      // (norm-only calls: no more)
    return std::max(need, dense_scratch_bytes(g));
}

dp_status launch_dense(const Geo &g, int mode, const void *x, const void *dy, float *out_w, float *out_b,
                       size_t out_stride, float *sqnorm, const float *group_sqnorm, float clip_c, void *ws,
                       hipStream_t s)
{
    DenseArgs a;
    a.x = x; a.dy = dy; a.x_tab = g.x_tab; a.dy_tab = g.dy_tab; a.out_w = out_w; a.out_b = out_b;
    a.out_stride_w = out_stride ? out_stride : g.pw;
    a.out_stride_b = out_stride ? out_stride : g.pb;
    a.partials = static_cast<float *>(ws);
    a.group_sqnorm = group_sqnorm; a.clip_c = clip_c;
    a.n = g.n; a.tokens = g.h; a.cin = g.cin; a.cout = g.cout; a.has_bias = g.has_bias;
    a.tiles_k = (g.cin + DT - 1) / DT;
    a.tiles_o = (g.cout + DT - 1) / DT;
    const bool weighted = mode == MODE_WEIGHTED;
    const void *fn = nullptr;
    unsigned threads = 256, lds = 0;
    long long blocks = weighted ? (long long)a.tiles_k * a.tiles_o : (long long)g.n * a.tiles_k * a.tiles_o;
    const DenseRoute route = dense_route(g, mode);
    if (route == DENSE_NORM1) {
        blocks = g.n;
        if (sqnorm) a.partials = sqnorm;                 // the one partial of an example is its norm
        fn = g.bf16 ? reinterpret_cast<const void *>(&dense_rank1_norm_kernel<true>) : reinterpret_cast<const void *>(&dense_rank1_norm_kernel<false>);
    } else if (route == DENSE_OUTER) {
        a.tiles_k = (g.cin + 255) / 256;
        a.tiles_o = (g.cout + OUTER_ROWS - 1) / OUTER_ROWS;
        blocks = (long long)g.n * a.tiles_k * a.tiles_o;
        fn = g.bf16 ? reinterpret_cast<const void *>(&dense_outer_kernel<true>) : reinterpret_cast<const void *>(&dense_outer_kernel<false>);
    } else {
        // four groups of waves share a tile's K when the tiles alone leave compute units idle and K is more than a step long
        const bool tok = route == DENSE_TOKENS;
        const long long steps = tok ? (long long)g.n * ((g.h + DTK - 1) / DTK) : ((long long)g.n * g.h + DRK - 1) / DRK;
        const bool split = weighted && blocks < 512 && steps > 1;
        threads = split ? 1024 : 256;
        lds = (split ? 4u : 1u) * 2u * (tok ? (unsigned)DT_STAGE : (unsigned)DR_STAGE * 4u);
        if (tok) {
            if (!weighted) fn = reinterpret_cast<const void *>(&dense_tokens_kernel<false, 1>);
            else fn = split ? reinterpret_cast<const void *>(&dense_tokens_kernel<true, 4>) : reinterpret_cast<const void *>(&dense_tokens_kernel<true, 1>);
        } else if (g.bf16) {                              // weighted, fewer than 16 tokens
            fn = split ? reinterpret_cast<const void *>(&dense_rows_kernel<true, true, 4>) : reinterpret_cast<const void *>(&dense_rows_kernel<true, true, 1>);
        } else if (!weighted) {
            fn = reinterpret_cast<const void *>(&dense_rows_kernel<false, false, 1>);
        } else {
            fn = split ? reinterpret_cast<const void *>(&dense_rows_kernel<false, true, 4>) : reinterpret_cast<const void *>(&dense_rows_kernel<false, true, 1>);
        }
        static std::atomic<bool> attr_done[2][2];         // [tokens][bf16]: the split kernels; setting it twice is harmless
        if (split && !attr_done[tok][g.bf16 ? 1 : 0].load()) {
            if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
                return fail(DP_ERR_DEVICE, "dense: cannot reserve %u bytes of LDS", lds);
            attr_done[tok][g.bf16 ? 1 : 0].store(true);
        }
    }
    if (blocks > 0x7FFFFFFFll) return fail(DP_ERR_UNSUPPORTED, "dense: layer too large");
    // (TIER_PRE: the timing aid brackets convolutions only)
    const dp_status st = submit_kernel<DenseArgs>(TIER_PRE, fn, a, (unsigned)blocks, threads, lds, s, "dense");
    if (st != DP_OK || weighted || !sqnorm || route == DENSE_NORM1) return st;
    const float *partials = a.partials;
    const int n = g.n, count = (int)dense_norm_partial_count(g, mode);
    return submit_post([=]() -> dp_status { return launch_sum_partials(partials, n, count, sqnorm, s); });
}

}  // namespace dp
