// Per-example gradients of GroupNorm affine parameters: two reductions over each channel of x and dy.
#include "internal.h"
#include "group.h"

namespace dp {

size_t gn_norm_partial_count(const Geo &g) { return (size_t)g.gn_groups; }

// ------------------------------------------------------------------------------------------
// GroupNorm affine, groups of more than GN_CMAX channels: one workgroup per (example, group).  Mean
// and biased variance of the group's (C/G)*H*W elements in two passes (the group is L2-resident
// after the first), then
// each wave takes channels of the group in turn and reduces sum dy*xhat and sum dy with
// shuffles.
struct GnArgs {
    const void *x, *dy;
    int x_tab, dy_tab;              // Geo::x_tab / dy_tab: the operand pointers are arrays of example addresses
    float *out_w, *out_b;           // [n, stride] rows of dgamma / dbeta (may be null)
    size_t out_stride_w, out_stride_b;
    float *partials;                // [n, groups]
    int n, c, hw, groups;
    float eps;
    int vec, team, waves;           // one-sweep kernel: elements per load, lanes per channel, waves per group (gn_plan)
};

template <bool BF16>
__global__ void __launch_bounds__(256) gn_affine_3pass_kernel(const Grouped<GnArgs> launch)
{
    typedef typename In<BF16>::type E;
    __shared__ float red[4];
    unsigned bid;
    const GnArgs &a = launch.a[group_pick(launch, bid)];
    const int i = bid / a.groups, grp = bid - i * a.groups;
    const int cg = a.c / a.groups;
    const size_t ex = (size_t)a.c * a.hw, first = (size_t)grp * cg * a.hw;
    const int cnt = cg * a.hw;
    const E *xg = example_at_uniform<E>(a.x, a.x_tab, i, ex) + first;
    const E *dyg = example_at_uniform<E>(a.dy, a.dy_tab, i, ex) + first;

    // the mean is taken about the group's first element, so that a group far from zero keeps its spread
    const float k = In<BF16>::ld(xg);
    float s = 0.0f;
    for (int p = threadIdx.x; p < cnt; p += 256) s += In<BF16>::ld(xg + p) - k;
    const float m1 = block_sum<4>(s, red) / (float)cnt;              // mean - k
    float v = 0.0f;
    for (int p = threadIdx.x; p < cnt; p += 256) {
        const float d = (In<BF16>::ld(xg + p) - k) - m1;
        v += d * d;
    }
    const float var = block_sum<4>(v, red) / (float)cnt;
    const float rstd = 1.0f / sqrtf(var + a.eps);

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    float ss = 0.0f;
    for (int cl = wave; cl < cg; cl += 4) {
        const E *xc = xg + (size_t)cl * a.hw, *dc = dyg + (size_t)cl * a.hw;
        float sg = 0.0f, sb = 0.0f;
        for (int p = lane; p < a.hw; p += 64) {
            const float d = In<BF16>::ld(dc + p);
            sg += d * (((In<BF16>::ld(xc + p) - k) - m1) * rstd);
            sb += d;
        }
        sg = wave_sum(sg);
        sb = wave_sum(sb);
        if (lane == 0) {
            const int c = grp * cg + cl;
            ss += sg * sg + sb * sb;
            if (a.out_w) {
                a.out_w[(size_t)i * a.out_stride_w + c] = sg;
                a.out_b[(size_t)i * a.out_stride_b + c] = sb;
            }
        }
    }
    const float tot = block_sum<4>(ss, red);
    if (threadIdx.x == 0) a.partials[(size_t)i * a.groups + grp] = tot;
}

// One sweep over x and dy (groups of at most GN_CMAX channels): with k = the group's first element as
// a shift (so that the variance does not cancel) every channel's team of lanes accumulates
//     sum (x-k), sum (x-k)^2 for the group statistics,   sum dy (x-k), sum dy for the channel;
// then dgamma_c = rstd (sum dy (x-k) - (mean-k) sum dy), dbeta_c = sum dy.
//
// HBM-bound (x and dy are read once, 2 c floats written per example), but a layer alone is too small to get there:
// all layers of a batch call share a launch, and the work is laid out so that a lane always has several wide loads in
// flight.  A channel belongs to a team of `team` lanes (a power of two, about four vectors per lane), a group to
// `waves` waves of the workgroup, so that narrow groups do not leave waves idle; a vector is the widest piece (16 .. 2
// bytes) that divides the channel's row.  Kernel time per optimiser step beside the other layers' kernels, against one
// launch per layer and one wave per channel with 2- or 4-byte loads: ResNet-18-GN, 8 x 32 examples, 20 layers: 1377 ->
// 606 us (160 -> 16 launches; whole step 2.67 -> 2.07 ms); ResNet-20 in fp32, 256 examples: 963 -> 429 us.
//
// A group of a few kilobytes is a wave's work for a microsecond, of which its sums were the longer part: with the sums in
// registers (below), the example found by a 32-bit scalar division instead of one in 64 bits per lane, and no barriers
// where a wave has its group for itself, ResNet-18-GN's whole step of 64 examples went from 1.31 to 1.27 ms, that of
// 200 x 200 images, 36 examples, from 1.77 to 1.74 ms.
constexpr int GN_CMAX = 256;
constexpr int GN_WIDE_HW = 1024;             // maps of so many values, a multiple of four, are read four at a time
constexpr int GN_SHIFTED = 9;                // GnArgs::vec: vectors of eight bf16 values that need not start with a channel

// Sums over the lanes of a wave, and over its aligned teams of a power of two of lanes (in every lane of the team), by data-parallel-primitive moves as far as
// rows of sixteen lanes go.  (Shuffles through LDS took a wave longer than its loads on small groups.)
__device__ __forceinline__ float gn_wave_sum(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, wave_sum_last_lane(v)), 63));
}
template <int CTRL>
__device__ __forceinline__ float gn_moved(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ void gn_team_sum(float &a, float &b, int team)
{
    if (team == 64) { a = gn_wave_sum(a); b = gn_wave_sum(b); return; }
    if (team > 1) { a += gn_moved<0xB1>(a); b += gn_moved<0xB1>(b); }         // quad_perm 1 0 3 2
    if (team > 2) { a += gn_moved<0x4E>(a); b += gn_moved<0x4E>(b); }         // quad_perm 2 3 0 1
    if (team > 4) { a += gn_moved<0x141>(a); b += gn_moved<0x141>(b); }       // row_half_mirror
    if (team > 8) { a += gn_moved<0x140>(a); b += gn_moved<0x140>(b); }       // row_mirror
    if (team > 16) { a += __shfl_xor(a, 16, 64); b += __shfl_xor(b, 16, 64); }
}

template <bool BF16, int V>
__device__ __forceinline__ void gn_load(const typename In<BF16>::type *p, float (&o)[V])
{
    if constexpr (!BF16) {
        if constexpr (V == 4) { const float4 v = *reinterpret_cast<const float4 *>(p); o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w; }
        else if constexpr (V == 2) { const float2 v = *reinterpret_cast<const float2 *>(p); o[0] = v.x; o[1] = v.y; }
        else o[0] = *p;
    } else if constexpr (V == 1) {
        o[0] = bf16_bits_to_float(*p);
    } else {
        uint32_t d[V / 2];
        if constexpr (V == 8) { const uint4 v = *reinterpret_cast<const uint4 *>(p); d[0] = v.x; d[1] = v.y; d[2] = v.z; d[3] = v.w; }
        else if constexpr (V == 4) { const uint2 v = *reinterpret_cast<const uint2 *>(p); d[0] = v.x; d[1] = v.y; }
        else d[0] = *reinterpret_cast<const uint32_t *>(p);
#pragma unroll
        for (int e = 0; e < V / 2; ++e) {
            o[2 * e] = __uint_as_float(d[e] << 16);
            o[2 * e + 1] = __uint_as_float(d[e] & 0xFFFF0000u);
        }
    }
}

// SHIFTED: channels that do not start on 16 bytes (odd maps) are read in the aligned vectors that cover them.  The first and the last
// of these hold values of the neighbours, which are masked; a last one that reaches beyond the tensor is read value by value.  The vectors of X
// and dY have to start at the same value: an example whose two addresses differ modulo 16 (tensors of odd examples, calls by address)
// is read value by value, a vector placed by the other tensor would lie askew and reach out of its own.
template <bool BF16, int V, bool SHIFTED = false>
__device__ __forceinline__ void gn_affine_body(const GnArgs &a, unsigned bid, float *s_dx, float *s_d, float *red)
{
    typedef typename In<BF16>::type E;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int waves = a.waves, team = a.team;
    const int shift = waves == 4 ? 2 : waves - 1;                     // (waves: 1, 2 or 4)
    const int per_wg = 4 >> shift;                                    // groups per workgroup
    const int sub = wave >> shift, wv = wave & (waves - 1);
    const long long gid = (long long)bid * per_wg + sub, all = (long long)a.n * a.groups;
    const bool live = gid < all;                                      // the last workgroup may hold fewer groups
    int i = 0;
    if (live) i = all < (1ll << 31) ? (int)((unsigned)gid / (unsigned)a.groups) : (int)(gid / a.groups);
    i = __builtin_amdgcn_readfirstlane(i);
    const int grp = live ? (int)(gid - (long long)i * a.groups) : 0;
    const int cg = a.c / a.groups;
    const size_t ex = (size_t)a.c * a.hw, first = (size_t)grp * cg * a.hw;
    const E *xg = example_at_uniform<E>(a.x, a.x_tab, i, ex) + first;
    const E *dyg = example_at_uniform<E>(a.dy, a.dy_tab, i, ex) + first;
    // end of the tensor that the example lies in, as far as it is known
    const uintptr_t x_end = reinterpret_cast<uintptr_t>(xg - first) + ex * sizeof(E) * (size_t)(a.x_tab ? 1 : a.n - i);
    // (the same in every lane of a wave)
    const bool apart = SHIFTED && ((reinterpret_cast<uintptr_t>(xg) ^ reinterpret_cast<uintptr_t>(dyg)) & 15u) != 0;
    const float k = In<BF16>::ld(xg);
    s_dx += sub * cg;
    s_d += sub * cg;

    const int hw = a.hw, tl = lane & (team - 1), teams = 64 / team;
    float sx = 0.0f, sxx = 0.0f;
    for (int cl = wv * teams + lane / team; cl < cg; cl += waves * teams) {
        const E *xc = xg + (size_t)cl * a.hw, *dc = dyg + (size_t)cl * a.hw;
        int nv = hw / V, off = 0, last = 0;                           // whole vectors of the channel
        if constexpr (SHIFTED) {
            off = (int)((reinterpret_cast<uintptr_t>(xc) & 15u) / sizeof(E));      // values before the channel in its first vector
            last = (off + hw + V - 1) / V - 1;
            nv = last - 1;                                            // those between the first and the last
            xc += V - off;
            dc += V - off;
        }
        float dx[V], d1[V], x1[V], x2[V];
#pragma unroll
        for (int e = 0; e < V; ++e) dx[e] = d1[e] = x1[e] = x2[e] = 0.0f;
        auto add = [&](const float (&xv)[V], const float (&dv)[V]) {
#pragma unroll
            for (int e = 0; e < V; ++e) {
                const float xs = xv[e] - k;
                dx[e] += dv[e] * xs; d1[e] += dv[e]; x1[e] += xs; x2[e] += xs * xs;
            }
        };
        if (apart) {
#pragma unroll 1
            for (int p = tl; p < hw; p += team) {
                const float xs = In<BF16>::ld(xg + (size_t)cl * hw + p) - k, dv = In<BF16>::ld(dyg + (size_t)cl * hw + p);
                dx[0] += dv * xs; d1[0] += dv; x1[0] += xs; x2[0] += xs * xs;
            }
            nv = 0;
        }
        constexpr int U = SHIFTED ? 3 : 4;                            // vectors in flight (a fourth costs the kernel a wave per SIMD)
        int p = tl;
        for (; p + (U - 1) * team < nv; p += U * team) {
            float xv[U][V], dv[U][V];
#pragma unroll
            for (int u = 0; u < U; ++u) { gn_load<BF16, V>(xc + (size_t)(p + u * team) * V, xv[u]); gn_load<BF16, V>(dc + (size_t)(p + u * team) * V, dv[u]); }
#pragma unroll
            for (int u = 0; u < U; ++u) add(xv[u], dv[u]);
        }
        if (!SHIFTED || nv > 0) {                                     // the vectors that are left, loaded together
            float xv[U - 1][V], dv[U - 1][V];
#pragma unroll
            for (int u = 0; u < U - 1; ++u) {
                const int at = min(p + u * team, nv - 1);
                gn_load<BF16, V>(xc + (size_t)at * V, xv[u]);
                gn_load<BF16, V>(dc + (size_t)at * V, dv[u]);
            }
#pragma unroll
            for (int u = 0; u < U - 1; ++u)
                if (p + u * team < nv) add(xv[u], dv[u]);
        }
        if constexpr (SHIFTED) {
#pragma unroll 1
            for (int edge = 0; edge < 2; ++edge) {
                if (apart || tl != (edge ? team - 1 : 0)) continue;
                const int e0 = edge ? last * V - off : -off;          // the channel's value that the vector starts at
                const E *xe = xc + (off - V) + e0, *de = dc + (off - V) + e0;
                float xv[V], dv[V];
                if (reinterpret_cast<uintptr_t>(xe + V) <= x_end) {
                    gn_load<BF16, V>(xe, xv);
                    gn_load<BF16, V>(de, dv);
                } else {
#pragma unroll
                    for (int e = 0; e < V; ++e) {
                        const bool in = e0 + e >= 0 && e0 + e < hw;
                        xv[e] = in ? In<BF16>::ld(xe + e) : k;
                        dv[e] = in ? In<BF16>::ld(de + e) : 0.0f;
                    }
                }
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    const bool in = e0 + e >= 0 && e0 + e < hw;
                    xv[e] = in ? xv[e] : k;
                    dv[e] = in ? dv[e] : 0.0f;
                }
                add(xv, dv);
            }
        }
        float sdx = 0.0f, sd = 0.0f;
#pragma unroll
        for (int e = 0; e < V; ++e) { sdx += dx[e]; sd += d1[e]; sx += x1[e]; sxx += x2[e]; }
        gn_team_sum(sdx, sd, team);
        if (tl == 0 && live) { s_dx[cl] = sdx; s_d[cl] = sd; }
    }
    sx = gn_wave_sum(sx);
    sxx = gn_wave_sum(sxx);
    if (waves > 1) {
        if (lane == 0) { red[wave] = sx; red[4 + wave] = sxx; }
        __syncthreads();                                              // also makes s_dx / s_d visible
        sx = sxx = 0.0f;
        for (int w = sub * waves; w < (sub + 1) * waves; ++w) { sx += red[w]; sxx += red[4 + w]; }
    } else {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");        // (a wave's own s_dx / s_d: its LDS instructions run in order)
        __builtin_amdgcn_wave_barrier();
    }
    const float inv = 1.0f / (float)(cg * a.hw);
    const float m1 = sx * inv, var = fmaxf(sxx * inv - m1 * m1, 0.0f);
    const float rstd = 1.0f / sqrtf(var + a.eps);
    float ss = 0.0f;
    if (live) {
        for (int cl = wv * 64 + lane; cl < cg; cl += waves * 64) {
            const float sg = rstd * (s_dx[cl] - m1 * s_d[cl]), sb = s_d[cl];
            const int c = grp * cg + cl;
            ss += sg * sg + sb * sb;
            if (a.out_w) {
                a.out_w[(size_t)i * a.out_stride_w + c] = sg;
                a.out_b[(size_t)i * a.out_stride_b + c] = sb;
            }
        }
    }
    ss = gn_wave_sum(ss);
    if (waves > 1) {
        __syncthreads();
        if (lane == 0) red[wave] = ss;
        __syncthreads();
        ss = 0.0f;
        for (int w = sub * waves; w < (sub + 1) * waves; ++w) ss += red[w];
    }
    if (lane == 0 && wv == 0 && live) a.partials[(size_t)i * a.groups + grp] = ss;
}

template <bool BF16>
__global__ void __launch_bounds__(256, 4) gn_affine_kernel(const Grouped<GnArgs> grp)
{
    __shared__ float s_dx[GN_CMAX], s_d[GN_CMAX], red[8];
    unsigned bid;
    const GnArgs &a = grp.a[group_pick(grp, bid)];
    if constexpr (BF16) {
        if (a.vec == 8) { gn_affine_body<true, 8>(a, bid, s_dx, s_d, red); return; }
        if (a.vec == GN_SHIFTED) { gn_affine_body<true, 8, true>(a, bid, s_dx, s_d, red); return; }
    }
    if (a.vec == 4) gn_affine_body<BF16, 4>(a, bid, s_dx, s_d, red);
    else if (a.vec == 2) gn_affine_body<BF16, 2>(a, bid, s_dx, s_d, red);
    else gn_affine_body<BF16, 1>(a, bid, s_dx, s_d, red);
}

// How the lanes of gn_affine_kernel are dealt to channels and groups.
static void gn_plan(GnArgs &a, bool bf16)
{
    const int cg = a.c / a.groups;
    a.vec = bf16 ? 8 : 4;
    while (a.hw % a.vec) a.vec >>= 1;
    int nv = a.hw / a.vec;
    // maps that are no multiple of eight values: eight at a time all the same.  us per call, narrower vectors / this: 1024 channels on
    // 13 x 13, 36 examples 25.4 / 15.1; 2048 on 7 x 7, 64 examples 21.3 / 12.7; 512 on 25 x 25, 36 25.4 / 23.0; 256 on 14 x 14, 128 14.8 / 12.3.
    // All layers of ResNet-50-GN at 200 x 200, 36 examples: 599 / 422.  Multiples of four values keep vectors of four from GN_WIDE_HW values on: a channel's
    // two ends cost more than they bring (256 on 50 x 50, 36 examples: 26.1 / 28.7).
    if (bf16 && a.vec < 8 && a.hw >= 16 && (a.vec < 4 || a.hw < GN_WIDE_HW)) { a.vec = GN_SHIFTED; nv = (a.hw + 14) / 8; }
    a.team = 1;
    while (a.team < 64 && a.team * 4 < nv) a.team <<= 1;              // about four vectors per lane,
    while (a.team < 64 && (64 / a.team) / 2 >= cg) a.team <<= 1;      // and no more teams in a wave than the group has channels
    a.waves = 4;
    while (a.waves > 1 && a.waves * (64 / a.team) > cg && a.waves * 32 >= cg) a.waves >>= 1;     // (4 / waves) * cg channels fit in LDS
}

size_t gn_ws_bytes(const Geo &g, int mode)
{
    size_t b = (size_t)g.n * g.gn_groups * sizeof(float);
    b = (b + 15) & ~(size_t)15;
    if (mode == MODE_WEIGHTED) b += (size_t)g.n * 2 * g.cin * sizeof(float);
    return b;
}

dp_status launch_gn(const Geo &g, int mode, const void *x, const void *dy, float *out_w, float *out_b,
                    size_t out_stride, float *sqnorm, const float *group_sqnorm, float clip_c, void *ws,
                    hipStream_t s)
{
    GnArgs a;
    a.x = x; a.dy = dy; a.x_tab = g.x_tab; a.dy_tab = g.dy_tab;
    a.partials = static_cast<float *>(ws);
    a.n = g.n; a.c = g.cin; a.hw = g.h * g.w; a.groups = g.gn_groups; a.eps = g.gn_eps;
    const bool weighted = mode == MODE_WEIGHTED;
    float *gw = out_w, *gb = out_b;
    if (weighted) {
        const size_t head = (((size_t)g.n * g.gn_groups * sizeof(float)) + 15) & ~(size_t)15;
        gw = reinterpret_cast<float *>(static_cast<char *>(ws) + head);
        gb = gw + (size_t)g.n * g.cin;
        a.out_stride_w = a.out_stride_b = (size_t)g.cin;
    } else {
        a.out_stride_w = out_stride ? out_stride : g.pw;
        a.out_stride_b = out_stride ? out_stride : g.pb;
    }
    a.out_w = gw; a.out_b = gb;
    const bool one_sweep = g.cin / g.gn_groups <= GN_CMAX;
    const void *fn;
    long long blocks = (long long)g.n * g.gn_groups;
    if (one_sweep) {
        gn_plan(a, g.bf16);
        blocks = (blocks + 4 / a.waves - 1) / (4 / a.waves);
        fn = g.bf16 ? reinterpret_cast<const void *>(&gn_affine_kernel<true>) : reinterpret_cast<const void *>(&gn_affine_kernel<false>);
    } else {
        fn = g.bf16 ? reinterpret_cast<const void *>(&gn_affine_3pass_kernel<true>) : reinterpret_cast<const void *>(&gn_affine_3pass_kernel<false>);
    }
    if (blocks > 0x7FFFFFFFll) return fail(DP_ERR_UNSUPPORTED, "GroupNorm: more than 2^31 groups in a call");
    // (TIER_PRE: the timing aid brackets contractions only)
    dp_status st = submit_kernel<GnArgs>(TIER_PRE, fn, a, (unsigned)blocks, 256, 0, s, "gn_affine");
    if (st != DP_OK) return st;
    const int n = g.n, c = g.cin, groups = g.gn_groups;
    if (weighted)
        return submit_post([=]() -> dp_status {
            const dp_status sw = launch_clip_accumulate(gw, (size_t)c, group_sqnorm, clip_c, n, (size_t)c, out_w, s);
            return sw != DP_OK ? sw : launch_clip_accumulate(gb, (size_t)c, group_sqnorm, clip_c, n, (size_t)c, out_b, s);
        });
    if (!sqnorm) return st;
    const float *partials = a.partials;
    return submit_post([=]() -> dp_status { return launch_sum_partials(partials, n, groups, sqnorm, s); });
}

// Clipping units: rows[u*unit .. (u+1)*unit) of the per-example scale / shift gradients are added (in example
// order), stored if wanted, and squared.  One workgroup per (256 channels, unit).
struct UnitRowsArgs {
    const float *gw, *gb;          // [n, c] per-example gradients
    float *out_w, *out_b;          // unit sums (may be null)
    size_t out_stride_w, out_stride_b;
    float *partials;               // [units, gridDim.x]
    int c, unit;
};

__global__ void __launch_bounds__(256) unit_rows_kernel(const UnitRowsArgs a)
{
    __shared__ float red[4];
    const int c = blockIdx.x * 256 + threadIdx.x, u = blockIdx.y;
    float sw = 0.0f, sb = 0.0f;
    if (c < a.c) {
        for (int e = 0; e < a.unit; ++e) {
            const size_t row = (size_t)(u * a.unit + e) * a.c + c;
            sw += a.gw[row];
            sb += a.gb[row];
        }
        if (a.out_w) {
            a.out_w[(size_t)u * a.out_stride_w + c] = sw;
            a.out_b[(size_t)u * a.out_stride_b + c] = sb;
        }
    }
    const float tot = block_sum<4>(sw * sw + sb * sb, red);
    if (threadIdx.x == 0) a.partials[(size_t)u * gridDim.x + blockIdx.x] = tot;
}

static size_t gn_unit_head(const Geo &g) { return gn_ws_bytes(g, MODE_WEIGHTED); }

size_t gn_unit_ws_bytes(const Geo &g, int unit)
{
    return gn_unit_head(g) + (size_t)(g.n / unit) * ((g.cin + 255) / 256) * sizeof(float);
}

const float *gn_unit_partials(const Geo &g, const void *ws) { return reinterpret_cast<const float *>(static_cast<const char *>(ws) + gn_unit_head(g)); }
size_t gn_unit_norm_partial_count(const Geo &g) { return (size_t)((g.cin + 255) / 256); }

dp_status launch_gn_units(const Geo &g, int unit, const void *x, const void *dy, float *out_w, float *out_b,
                          size_t out_stride, float *sqnorm, void *ws, hipStream_t s)
{
    // per-example gradients into the workspace (where the clip-weighted call keeps them), then the unit sums
    const size_t head = (((size_t)g.n * g.gn_groups * sizeof(float)) + 15) & ~(size_t)15;
    float *gw = reinterpret_cast<float *>(static_cast<char *>(ws) + head);
    float *gb = gw + (size_t)g.n * g.cin;
    dp_status st = launch_gn(g, MODE_MATERIALISE, x, dy, gw, gb, (size_t)g.cin, nullptr, nullptr, 0.0f, ws, s);
    if (st != DP_OK) return st;
    UnitRowsArgs a;
    a.gw = gw; a.gb = gb; a.out_w = out_w; a.out_b = out_b;
    a.out_stride_w = out_stride ? out_stride : g.pw;
    a.out_stride_b = out_stride ? out_stride : g.pb;
    a.partials = reinterpret_cast<float *>(static_cast<char *>(ws) + gn_unit_head(g));
    a.c = g.cin; a.unit = unit;
    const int blocks = (g.cin + 255) / 256, units = g.n / unit;
    return submit_post([=]() -> dp_status {
        hipLaunchKernelGGL(unit_rows_kernel, dim3(blocks, units), dim3(256), 0, s, a);
        const dp_status su = check_launch("unit_rows");
        return (su != DP_OK || !sqnorm) ? su : launch_sum_partials(a.partials, units, blocks, sqnorm, s);
    });
}

}  // namespace dp
