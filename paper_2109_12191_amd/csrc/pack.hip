// Operand packing for the clip-weighted contraction (the recomputation form of H4):
//     acc[co, j] += sum_i f_i sum_k dY_i[co, k] * Xcol_i[j, k],   f_i = min(1, C / |g_i|)
// is one GEMM whose K axis runs over (example, output position).  For layers with small
// feature maps the operands are first rewritten K-contiguous and 16-byte aligned:
//     dYp[grp][co][e * SP + k] = bf16(f_i * dY_i[co, k])            i = grp * EG + e
//     Xp [grp][j ][e * SP + k] = Xpad_i[ci, oh*s + kh - p, ow*s + kw - p]   (im2col row j = (ci,kh,kw))
// with SP = S rounded up to 8 and zeros in the padding, so that the contraction kernel streams
// plain aligned pieces with no masks, gathers or per-example scaling, whatever the stride, kernel
// size or parity of S.  The clip factor is applied here, in fp32, and rounded to bf16 once
// (nearest even) -- the same arithmetic the in-kernel scaling performs.
// `grp` splits the examples into ranges that different workgroups contract (the K slices).
// Without norms the operands are copied as they are (rows of 64 per example: the contraction scales each example's finished block).
#include "group.h"
#include "internal.h"
#include "pieces.h"

namespace dp {

namespace {

struct PackArgs {
    const void *x, *dy;
    int x_tab, dy_tab;              // Geo::x_tab / dy_tab: the operand pointers are arrays of example addresses
    uint16_t *xp, *dyp;
    const float *group_sqnorm;      // null: dY is not scaled
    float clip_c;
    int n, cin, cout, h, w, kh, kw, stride, pad, oh, ow;
    int S, SP, J;
    int groups, eg;                 // example ranges and examples per range
    int kg8;                        // pieces per packed row: eg * SP / 8
    long long x_pieces, dy_pieces;
};

__global__ void __launch_bounds__(256) pack_weighted_kernel(const Grouped<PackArgs> layers)
{
    unsigned bid;
    const PackArgs &a = layers.a[group_pick(layers, bid)];
    const long long q = (long long)bid * 256 + threadIdx.x;
    uint32_t out[4] = {0u, 0u, 0u, 0u};
    if (q < a.x_pieces) {
        const int kk8 = (int)(q % a.kg8);
        const long long row = q / a.kg8;
        const int j = (int)(row % a.J), grp = (int)(row / a.J);
        const int kk = kk8 * 8;
        const int e = kk / a.SP, k0 = kk - e * a.SP;
        const int i = grp * a.eg + e;
        if (i < a.n && k0 < a.S) {
            const int taps = a.kh * a.kw;
            const int ci = j / taps, t = j - ci * taps;
            const int kh = t / a.kw, kw = t - kh * a.kw;
            const size_t ex_elems = (size_t)a.cin * a.h * a.w;
            const uint16_t *ex = example_at<uint16_t>(a.x, a.x_tab, i, ex_elems);
            const uint16_t *src = ex + (size_t)ci * a.h * a.w;
            if (taps == 1 && a.stride == 1 && a.pad == 0) {
                // 1x1 stride 1: the im2col row is the channel itself -- eight consecutive elements from whole dwords
                // (the run may start on an odd element), element by element only where that window would leave the tensor
                const uintptr_t at = reinterpret_cast<uintptr_t>(src + k0), word = at & ~(uintptr_t)3;
                const int hi = min(8, a.S - k0);
                if (word + 20 <= reinterpret_cast<uintptr_t>(ex + ex_elems * (size_t)(a.x_tab ? 1 : a.n - i))) {     // the tensor's end
                    const Raw<5> raw = piece_load_words(reinterpret_cast<const uint32_t *>(word));
                    piece_finish<true, 1>(out, raw, (uint32_t)(at >> 1) & 1u, 0, hi);
                } else {
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const uint32_t v = (k0 + u < a.S) ? src[k0 + u] : 0u;
                        out[u >> 1] |= v << ((u & 1) * 16);
                    }
                }
                *reinterpret_cast<uint4 *>(a.xp + q * 8) = make_uint4(out[0], out[1], out[2], out[3]);
                return;
            }
            int oh = k0 / a.ow, ow = k0 - oh * a.ow;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                uint32_t v = 0u;
                if (k0 + u < a.S) {
                    const int ih = oh * a.stride + kh - a.pad, iw = ow * a.stride + kw - a.pad;
                    if (ih >= 0 && ih < a.h && iw >= 0 && iw < a.w) v = src[ih * a.w + iw];
                }
                out[u >> 1] |= v << ((u & 1) * 16);
                if (++ow == a.ow) { ow = 0; ++oh; }
            }
        }
        *reinterpret_cast<uint4 *>(a.xp + q * 8) = make_uint4(out[0], out[1], out[2], out[3]);
        return;
    }
    const long long qd = q - a.x_pieces;
    if (qd >= a.dy_pieces) return;
    const int kk8 = (int)(qd % a.kg8);
    const long long row = qd / a.kg8;
    const int co = (int)(row % a.cout), grp = (int)(row / a.cout);
    const int kk = kk8 * 8;
    const int e = kk / a.SP, k0 = kk - e * a.SP;
    const int i = grp * a.eg + e;
    if (i < a.n) {
        const float f = a.group_sqnorm ? clip_factor(a.group_sqnorm[i], a.clip_c) : 1.0f;     // (times 1: the same bits)
        const size_t ex_elems = (size_t)a.cout * a.S;
        const uint16_t *ex = example_at<uint16_t>(a.dy, a.dy_tab, i, ex_elems);
        const uint16_t *src = ex + (size_t)co * a.S;
        const uintptr_t at = reinterpret_cast<uintptr_t>(src + k0), word = at & ~(uintptr_t)3;
        const int hi = min(8, a.S - k0);
        if (hi > 0 && word + 20 <= reinterpret_cast<uintptr_t>(ex + ex_elems * (size_t)(a.dy_tab ? 1 : a.n - i))) {
            const Raw<5> raw = piece_load_words(reinterpret_cast<const uint32_t *>(word));
            piece_finish<true, 1>(out, raw, (uint32_t)(at >> 1) & 1u, 0, hi);
            scale_regs<true, 4>(out, f);                 // f * dY in fp32, rounded to bf16 once (nearest even)
        } else {
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                uint32_t v = 0u;
                if (k0 + u < a.S) v = float_to_bf16_bits(bf16_bits_to_float(src[k0 + u]) * f);
                out[u >> 1] |= v << ((u & 1) * 16);
            }
        }
    }
    *reinterpret_cast<uint4 *>(a.dyp + qd * 8) = make_uint4(out[0], out[1], out[2], out[3]);
}

// X of layers with taps whose planes fit into LDS (small maps, which is what is packed): a workgroup takes some examples of some channels, whose planes
// are contiguous in memory, into LDS once and writes their rows (all taps) from there, consecutive examples side by side.  The kernel above
// reads a value once per tap, and neighbouring threads read different examples.  Us a launch, both
// operands there / X here and dY there: ResNet-18-GN, 256 examples, 202 / 82 + 40; ResNet-50-GN at 200 x 200, 36 examples, 222 / 100 + 67; 64 examples of
// ResNet-50 for finished blocks 155 / 60 + 82.  Twice the LDS and pieces per workgroup: ResNet-50, 32 examples on one stream, 2312 -> 2337 us a step of two
// (a layer alone is too few workgroups).
struct PackStaged {
    const void *in;
    uint16_t *out;
    int tab, n, channels, h, w;     // Geo::x_tab; planes of an example
    int taps, kw, stride, pad, ow;
    int S, SP, eg, kg;              // positions, values of an example in a packed row, examples of a range, values of a packed row
    int cb, eb;                     // channels and examples of a workgroup
    unsigned c_blocks, e_blocks;    // workgroups of a range
    unsigned by_ed, by_rp, by_p8, by_taps, by_kw, by_ow;             // divisors as factors (pack_div)
};
// It is one more launch, of workgroups that take longer: only where a layer's copies, or those of a batch call's layers together, are worth that.  Us of a clip-weighted call, all in the kernel
// above / so, on both sides of the line.  A layer alone: 128 -> 128 stride 2 on 56 x 56, 8 examples (14 MB) 38 / 43, 16 (29 MB) 50 / 48, 32 (58 MB) 96 / 69; 64 -> 64
// stride 2 on 80 x 80, 8 (15 MB) 40 / 47, 16 (29 MB) 55 / 49; at two examples and less 13 / 24.  Batch calls: two of 5x5, 16 -> 32 stride 2 on 80 x 80, 8 examples
// (20 MB) 57 / 69, 16 (40 MB) 73 / 70; two of 64 -> 64 stride 2 on 32 x 32, 64 (38 MB) 76 / 59; four of 290 -> 64 stride 2 on 18 x 18, 16 (29 MB) 53 / 45; six of
// 512 -> 64 stride 2 on 11 x 64, 4 (42 MB) 53 / 41; ten of 64 -> 256 on 36 x 37, 4 (61 MB) 106 / 93; one of 243 -> 64 stride 2 on 32 x 32, 16 (18 MB), beside
// 119 -> 64 stride 2 on 21 x 21 (4 MB) 71 / 57.
constexpr size_t PACK_STAGED = (size_t)24 << 20, PACK_STAGED_SHARED = (size_t)12 << 20;         // (alone or together; one layer in a batch call)
// And where a workgroup's planes are not much to write (of 24 MB there are as many as compute units then): few large planes are.  The first convolution (3 -> 64 7x7 stride 2 on
// 112 x 112: a workgroup a plane, each of which writes 300 KB), alone, 48 examples, 82 / 130 us; in a batch call with another layer, 16 examples, 75 / 146; ten
// of 64 -> 55 5x5 on 25 x 25, 3 examples (192 workgroups each that write 32 KB), 67 / 61.
constexpr size_t PACK_STAGED_WRITES = (size_t)96 << 10;
constexpr int PACK_LDS = 12 * 1024, PACK_PLANE = 32 * 1024, PACK_EB = 16;

// x / d for x * d < 2^32; by = ceil(2^32 / d), 0 for d = 1
__device__ __forceinline__ unsigned pack_div(unsigned x, unsigned by) { return by ? __umulhi(x, by) : x; }

__global__ void __launch_bounds__(256) pack_staged_kernel(const Grouped<PackStaged> layers)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t words[];
    __shared__ unsigned odd[PACK_EB];
    unsigned bid;
    const PackStaged &a = layers.a[group_pick(layers, bid)];
    const unsigned per_range = a.c_blocks * a.e_blocks, grp = bid / per_range, r = bid - grp * per_range;
    const unsigned cblk = r / a.e_blocks, eblk = r - cblk * a.e_blocks;
    const int e0 = (int)eblk * a.eb, ne = min(a.eb, a.eg - e0), i0 = (int)grp * a.eg + e0, c0 = (int)cblk * a.cb, nc = min(a.cb, a.channels - c0);
    const int plane = a.h * a.w, count = nc * plane;
    const unsigned ed = (unsigned)(a.cb * plane + 3) / 2;            // dwords of an example in LDS
    const size_t ex_elems = (size_t)a.channels * plane;
    const int there = min(ne, a.n - i0);                             // examples of this workgroup that there are (a last range may be short)
    if (threadIdx.x < (unsigned)max(there, 0)) {
        const int i = i0 + (int)threadIdx.x;
        odd[threadIdx.x] = (unsigned)(reinterpret_cast<uintptr_t>(example_at<uint16_t>(a.in, a.tab, i, ex_elems) + (size_t)c0 * plane) >> 1) & 1u;
    }
    // whole dwords around an example's planes, a last half dword by itself (it may be the tensor's last value)
    const unsigned total_in = there > 0 ? (unsigned)there * ed : 0u;
    for (unsigned q0 = threadIdx.x; q0 < total_in; q0 += 1024) {
        uint32_t v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const unsigned q = q0 + 256u * k, e = pack_div(q, a.by_ed), d = q - e * ed;
            v[k] = 0u;
            if (q < total_in) {
                const uintptr_t at = reinterpret_cast<uintptr_t>(example_at<uint16_t>(a.in, a.tab, i0 + (int)e, ex_elems) + (size_t)c0 * plane);
                const int left = count - (int)(2 * d - ((at >> 1) & 1u));            // values from this dword's first half on
                const uintptr_t word = (at & ~(uintptr_t)3) + 4ull * d;
                if (left >= 2) v[k] = *reinterpret_cast<const uint32_t *>(word);
                else if (left == 1) v[k] = *reinterpret_cast<const uint16_t *>(word);
            }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (q0 + 256u * k < total_in) words[q0 + 256u * k] = v[k];
    }
    __syncthreads();
    const uint16_t *halves = reinterpret_cast<const uint16_t *>(words);
    const unsigned p8 = (unsigned)a.SP / 8, rp = (unsigned)a.eb * p8, total = (unsigned)(nc * a.taps) * rp;
    for (unsigned p = threadIdx.x; p < total; p += 256) {
        const unsigned row = pack_div(p, a.by_rp), q = p - row * rp, e = pack_div(q, a.by_p8), k8 = q - e * p8;
        if ((int)e >= ne) continue;
        const unsigned ci = pack_div(row, a.by_taps), t = row - ci * (unsigned)a.taps;
        const int k0 = (int)k8 * 8;
        uint32_t out[4] = {0u, 0u, 0u, 0u};
        if ((int)e < there && k0 < a.S) {
            const unsigned base = e * ed * 2 + odd[e] + ci * (unsigned)plane;
            const int kh = (int)pack_div(t, a.by_kw), kw = (int)t - kh * a.kw;
            const int oh = (int)pack_div((unsigned)k0, a.by_ow);
            int ow = k0 - oh * a.ow, ih = oh * a.stride + kh - a.pad, iw = ow * a.stride + kw - a.pad;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                uint32_t v = 0u;
                if (k0 + u < a.S && (unsigned)ih < (unsigned)a.h && (unsigned)iw < (unsigned)a.w) v = halves[base + (unsigned)(ih * a.w + iw)];
                out[u >> 1] |= v << ((u & 1) * 16);
                iw += a.stride;
                if (++ow == a.ow) { ow = 0; iw = kw - a.pad; ih += a.stride; }
            }
        }
        const size_t at = ((size_t)grp * ((size_t)a.channels * a.taps) + (size_t)(c0 * a.taps) + row) * (size_t)a.kg + (size_t)(e0 + (int)e) * a.SP + k0;
        *reinterpret_cast<uint4 *>(a.out + at) = make_uint4(out[0], out[1], out[2], out[3]);
    }
}

// Rows of another length (launch_widen): what the raw-row, LDS-direct and stem kernels are not built for is brought to the next length
// that they are, with zeros behind the values (zeros add nothing to a contraction).  Bound by memory: every value is read and written
// once.  One thread per 16 bytes of output, from whole dwords where it lies in one row or its halves do; else value by value, and
// its eight values may end one row and begin the next.  The layers of ResNet-50-GN at 200 x 200, 36 examples: 547 us value by value,
// 338 with dwords.
struct WidenArgs {
    const void *in;
    int in_tab, channels;           // Geo::x_tab; planes of an example
    uint16_t *out;
    unsigned total;                 // values of the copy
    int n, plane, w, rows, cols, step, dw, row;
};

__global__ void __launch_bounds__(256) widen_kernel(const Grouped<WidenArgs> grp)
{
    unsigned bid;
    const WidenArgs &a = grp.a[group_pick(grp, bid)];
    const unsigned e = (bid * 256u + threadIdx.x) * 8u;
    if (e >= a.total) return;
    unsigned ch = e / (unsigned)a.row;                               // plane of the whole copy
    int k = (int)(e - ch * (unsigned)a.row);
    int r = k / a.dw, c = k - r * a.dw;
    const unsigned i = ch / (unsigned)a.channels;
    unsigned in_ex = ch - i * (unsigned)a.channels;
    const size_t ex_elems = (size_t)a.channels * a.plane;
    const uint16_t *ex = example_at<uint16_t>(a.in, a.in_tab, (int)i, ex_elems);
    unsigned next = i + 1;
    const uint16_t *src = ex + (size_t)in_ex * a.plane;
    uint32_t out[4] = {0u, 0u, 0u, 0u};
    const uintptr_t end = reinterpret_cast<uintptr_t>(ex + ex_elems * (size_t)(a.in_tab ? 1u : (unsigned)a.n - i));     // the tensor's
    if (a.step == 1 && a.dw % 8 == 0) {
        // a piece lies in one row: whole dwords around it (the run may start on an odd value), what is beyond the row masked
        const int hi = r < a.rows ? min(8, a.cols - c) : 0;
        const uintptr_t at = reinterpret_cast<uintptr_t>(src + (size_t)r * a.w + c), word = at & ~(uintptr_t)3;
        if (hi <= 0 || word + 20 <= end) {
            if (hi > 0) {
                const Raw<5> raw = piece_load_words(reinterpret_cast<const uint32_t *>(word));
                piece_finish<true, 1>(out, raw, (uint32_t)(at >> 1) & 1u, 0, hi);
            }
            *reinterpret_cast<uint4 *>(a.out + e) = make_uint4(out[0], out[1], out[2], out[3]);      // (rows of whole pieces: so is the copy)
            return;
        }
    } else if (a.step == 1 && a.dw % 4 == 0 && a.total % 8 == 0) {
        // the same with two halves of four values, each in one row
        bool inside = true;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int hi = r < a.rows ? min(4, a.cols - c) : 0;
            const uintptr_t at = reinterpret_cast<uintptr_t>(src + (size_t)r * a.w + c), word = at & ~(uintptr_t)3;
            inside = inside && (hi <= 0 || word + 12 <= end);
            if (hi > 0 && word + 12 <= end) {
                const uint32_t *d = reinterpret_cast<const uint32_t *>(word);
                const uint32_t odd = (uint32_t)(at >> 1) & 1u, d0 = d[0], d1 = d[1], d2 = d[2];
                const uint32_t lo = funnel(d1, d0, odd * 16), up = funnel(d2, d1, odd * 16);
                out[2 * half] = hi >= 2 ? lo : lo & 0xFFFFu;
                out[2 * half + 1] = hi >= 4 ? up : (hi == 3 ? up & 0xFFFFu : 0u);
            }
            if (half == 0) {
                c += 4; k += 4;
                if (c == a.dw) { c = 0; ++r; }
                if (k == a.row) {
                    k = r = c = 0;
                    if (++in_ex == (unsigned)a.channels) break;      // the next example: value by value
                    src = ex + (size_t)in_ex * a.plane;
                }
            }
        }
        if (inside && in_ex < (unsigned)a.channels) {
            *reinterpret_cast<uint4 *>(a.out + e) = make_uint4(out[0], out[1], out[2], out[3]);
            return;
        }
        in_ex = ch - i * (unsigned)a.channels;
        k = (int)(e - ch * (unsigned)a.row);
        r = k / a.dw; c = k - r * a.dw;
        src = ex + (size_t)in_ex * a.plane;
        out[0] = out[1] = out[2] = out[3] = 0u;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        if (e + u < a.total) {
            const uint32_t v = (r < a.rows && c < a.cols) ? src[(size_t)(r * a.step) * a.w + c * a.step] : 0u;
            out[u >> 1] |= v << ((u & 1) * 16);
        }
        ++k;
        if (++c == a.dw) { c = 0; ++r; }
        if (k == a.row) {                                            // the next plane
            k = r = c = 0;
            if (++in_ex == (unsigned)a.channels) {
                in_ex = 0;
                if (e + u + 1 < a.total) ex = example_at<uint16_t>(a.in, a.in_tab, (int)next, ex_elems);
                ++next;
            }
            src = ex + (size_t)in_ex * a.plane;
        }
    }
    uint16_t *dst = a.out + e;
    if (e + 8u <= a.total) *reinterpret_cast<uint4 *>(dst) = make_uint4(out[0], out[1], out[2], out[3]);
    else
        for (unsigned u = 0; e + u < a.total; ++u) dst[u] = (uint16_t)(out[u >> 1] >> ((u & 1) * 16));
}

// Strided 1x1 convolutions only look at every stride-th row and column of X: this copies those
// into a compact [n*cin][OH*OW] tensor so that the contraction runs its plain aligned loader on
// half (a quarter, with both strides) of the bytes.  One thread per pair of output elements.
struct SubArgs {
    const void *x;
    int x_tab, cin;                 // Geo::x_tab; rows (channels) of an example
    uint16_t *out;
    long long rows;
    int h, w, oh, ow, stride;
};

__global__ void __launch_bounds__(256) subsample_kernel(const Grouped<SubArgs> grp)
{
    unsigned bid;
    const SubArgs &a = grp.a[group_pick(grp, bid)];
    uint16_t *__restrict__ out = a.out;
    const long long rows = a.rows;
    const int w = a.w, ow = a.ow, stride = a.stride;
    const int S = a.oh * ow, pairs = (S + 1) / 2;
    const long long t = (long long)bid * 256 + threadIdx.x;
    if (t >= rows * pairs) return;
    const long long row = t / pairs;
    const int k = (int)(t - row * pairs) * 2;
    const uint16_t *src;
    if (a.x_tab) {
        const int i = (int)((unsigned)row / (unsigned)a.cin);       // (rows < 2^31: the copy is at most 96 MB)
        src = example_at<uint16_t>(a.x, a.x_tab, i, 0) + (size_t)(row - (long long)i * a.cin) * a.h * w;
    } else {
        src = static_cast<const uint16_t *>(a.x) + (size_t)row * a.h * w;
    }
    const int r0 = k / ow, c0 = k - r0 * ow;
    const uint32_t lo = src[(size_t)r0 * stride * w + c0 * stride];
    uint16_t *dst = out + (size_t)row * S + k;
    if (k + 1 < S) {
        const int k1 = k + 1, r1 = k1 / ow, c1 = k1 - r1 * ow;
        const uint32_t hi = src[(size_t)r1 * stride * w + c1 * stride];
        if (((size_t)row * S) % 2 == 0) *reinterpret_cast<uint32_t *>(dst) = lo | (hi << 16);
        else { dst[0] = (uint16_t)lo; dst[1] = (uint16_t)hi; }
    } else {
        dst[0] = (uint16_t)lo;
    }
}

}  // namespace

namespace {

// Channels-last inputs: [n][positions][channels] -> [n][channels][positions], 32 x 32 tiles through LDS (both the
// reads and the writes are runs of 32 consecutive elements).  One workgroup of 256 threads per tile.
struct TrArgs {
    const void *in;
    void *out;
    int positions, channels, tiles_p, tiles_c;
};

template <typename T>
__global__ void __launch_bounds__(256) channels_first_kernel(const Grouped<TrArgs> layers)
{
    __shared__ T tile[32][33];
    unsigned bid;
    const TrArgs &a = layers.a[group_pick(layers, bid)];
    const int per_ex = a.tiles_p * a.tiles_c;
    const int i = (int)(bid / (unsigned)per_ex), t = (int)(bid - (unsigned)i * (unsigned)per_ex);
    const int tc = t / a.tiles_p, tp = t - tc * a.tiles_p;
    const size_t ex = (size_t)i * a.positions * a.channels;
    const T *in = static_cast<const T *>(a.in) + ex;
    T *out = static_cast<T *>(a.out) + ex;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
#pragma unroll
    for (int r = ty; r < 32; r += 8) {
        const int p = tp * 32 + r, c = tc * 32 + tx;
        if (p < a.positions && c < a.channels) tile[r][tx] = in[(size_t)p * a.channels + c];
    }
    __syncthreads();
#pragma unroll
    for (int r = ty; r < 32; r += 8) {
        const int c = tc * 32 + r, p = tp * 32 + tx;
        if (p < a.positions && c < a.channels) out[(size_t)c * a.positions + p] = tile[tx][r];
    }
}

}  // namespace

dp_status launch_to_channels_first(const void *in, void *out, int n, int positions, int channels, int elem_bytes, hipStream_t s)
{
    TrArgs a;
    a.in = in; a.out = out; a.positions = positions; a.channels = channels;
    a.tiles_p = (positions + 31) / 32; a.tiles_c = (channels + 31) / 32;
    const long long blocks = (long long)n * a.tiles_p * a.tiles_c;
    if (blocks > 0x7FFFFFFFll) return fail(DP_ERR_UNSUPPORTED, "channels-last input too large");
    const void *fn = elem_bytes == 2 ? reinterpret_cast<const void *>(&channels_first_kernel<uint16_t>)
                                     : reinterpret_cast<const void *>(&channels_first_kernel<uint32_t>);
    return submit_kernel<TrArgs>(TIER_LAYOUT, fn, a, (unsigned)blocks, 256, 0, s, "channels_first");
}

dp_status launch_widen(const void *in, int tab, void *out, int n, int channels, int h, int w, int rows, int cols, int step, int dw, int row,
                       hipStream_t s)
{
    const long long total = (long long)n * channels * row;
    if (total >= (1ll << 31)) return fail(DP_ERR_UNSUPPORTED, "widen: layer too large");
    WidenArgs a;
    a.in = in; a.in_tab = tab; a.channels = channels; a.out = static_cast<uint16_t *>(out); a.total = (unsigned)total; a.n = n;
    a.plane = h * w; a.w = w; a.rows = rows; a.cols = cols; a.step = step; a.dw = dw; a.row = row;
    return submit_kernel<WidenArgs>(TIER_ROWS, reinterpret_cast<const void *>(&widen_kernel), a, (unsigned)((total + 2047) / 2048), 256, 0, s, "widen");
}

dp_status launch_subsample(const Geo &g, const void *x, void *out, hipStream_t s)
{
    const long long rows = (long long)g.n * g.cin;
    const long long threads = rows * ((g.oh * g.ow + 1) / 2);
    const long long blocks = (threads + 255) / 256;
    if (blocks > 0x7FFFFFFFll) return fail(DP_ERR_UNSUPPORTED, "subsample: layer too large");
    SubArgs a;
    a.x = x; a.x_tab = g.x_tab; a.cin = g.cin; a.out = static_cast<uint16_t *>(out); a.rows = rows;
    a.h = g.h; a.w = g.w; a.oh = g.oh; a.ow = g.ow; a.stride = g.stride;
    return submit_kernel<SubArgs>(TIER_PRE, reinterpret_cast<const void *>(&subsample_kernel), a, (unsigned)blocks, 256, 0,
                                  s, "subsample");
}

PackPlan pack_plan(const Geo &g, int groups, int row)
{
    PackPlan p;
    p.S = g.oh * g.ow;
    p.SP = row ? row : (p.S + 7) / 8 * 8;
    p.J = g.cin * g.kh * g.kw;
    p.groups = groups;
    p.eg = (g.n + groups - 1) / groups;
    p.groups = (g.n + p.eg - 1) / p.eg;          // no empty trailing range
    p.kg = p.eg * p.SP;
    p.x_bytes = (size_t)p.groups * p.J * p.kg * 2;
    p.dy_bytes = (size_t)p.groups * g.cout * p.kg * 2;
    return p;
}

static unsigned pack_by(unsigned d) { return d > 1 ? (unsigned)(((1ull << 32) + d - 1) / d) : 0u; }

bool pack_staged_fits(const Geo &g) { return g.kh * g.kw > 1 && g.h * g.w * 2 <= PACK_PLANE; }

// X through pack_staged_kernel, if a plane of it fits and it pays; `done` says whether.  (Operands without taps stay with the kernel above: staged, ResNet-50 at 32
// examples was as fast alone and 2 % slower beside other kernels, which its LDS keeps off a compute unit.)
static dp_status launch_pack_staged(const Geo &g, const PackPlan &p, const void *in, void *out, hipStream_t s, bool &done)
{
    const int channels = g.cin;
    const int plane = g.h * g.w, taps = g.kh * g.kw, p8 = p.SP / 8;
    done = pack_staged_fits(g) && (p.x_bytes >= (crowd_hint() ? PACK_STAGED_SHARED : PACK_STAGED) || taps_hint() >= PACK_STAGED);
    if (!done) return DP_OK;
    PackStaged a;
    a.in = in; a.out = static_cast<uint16_t *>(out);
    a.tab = g.x_tab; a.n = g.n; a.channels = channels; a.h = g.h; a.w = g.w;
    a.taps = taps; a.kw = g.kw; a.stride = g.stride; a.pad = g.pad; a.ow = g.ow;
    a.S = p.S; a.SP = p.SP; a.eg = p.eg; a.kg = p.kg;
    // examples: runs of half a kilobyte in a row of the copy; channels: what LDS and about 2300 pieces have room for
    int eb = 1;
    while (eb < PACK_EB && eb * p.SP * 2 < 512 && (eb * 2) * plane * 2 <= PACK_LDS && eb < p.eg) eb *= 2;
    int cb = PACK_LDS / (eb * plane * 2);
    if (cb > 2304 / (taps * eb * p8)) cb = 2304 / (taps * eb * p8);
    if (cb > channels) cb = channels;
    if (cb < 1) cb = 1;
    a.cb = cb; a.eb = eb;
    a.c_blocks = (unsigned)((channels + cb - 1) / cb);
    a.e_blocks = (unsigned)((p.eg + eb - 1) / eb);
    const unsigned ed = (unsigned)(cb * plane + 3) / 2, rp = (unsigned)(eb * p8);
    a.by_ed = pack_by(ed); a.by_rp = pack_by(rp); a.by_p8 = pack_by((unsigned)p8); a.by_taps = pack_by((unsigned)taps); a.by_kw = pack_by((unsigned)g.kw); a.by_ow = pack_by((unsigned)g.ow);
    // (pack_div: what is divided is below 2^32 / the divisor)
    const unsigned long long most = (unsigned long long)cb * taps * rp;
    if ((unsigned long long)eb * ed * ed >= (1ull << 32) || most * rp >= (1ull << 32)) { done = false; return DP_OK; }
    const unsigned long long blocks = (unsigned long long)p.groups * a.c_blocks * a.e_blocks;
    if (p.x_bytes > blocks * PACK_STAGED_WRITES) { done = false; return DP_OK; }
    if (blocks > 0x7FFFFFFFull) return fail(DP_ERR_UNSUPPORTED, "pack: layer too large");
    // (layers share a launch if they ask for the same LDS; a piece is read from up to five dwords, which may lie behind the planes)
    return submit_kernel<PackStaged>(TIER_PRE, reinterpret_cast<const void *>(&pack_staged_kernel), a, (unsigned)blocks, 256,
                                     (plane * 2 <= PACK_LDS ? PACK_LDS : PACK_PLANE) + 256, s, "pack_staged");
}

dp_status launch_pack_weighted(const Geo &g, const PackPlan &p, const void *x, const void *dy,
                               const float *group_sqnorm, float clip_c, void *xp, void *dyp, hipStream_t s)
{
    PackArgs a;
    a.x = x; a.dy = dy; a.x_tab = g.x_tab; a.dy_tab = g.dy_tab;
    a.xp = static_cast<uint16_t *>(xp);
    a.dyp = static_cast<uint16_t *>(dyp);
    a.group_sqnorm = group_sqnorm; a.clip_c = clip_c;
    a.n = g.n; a.cin = g.cin; a.cout = g.cout; a.h = g.h; a.w = g.w; a.kh = g.kh; a.kw = g.kw;
    a.stride = g.stride; a.pad = g.pad; a.oh = g.oh; a.ow = g.ow;
    a.S = p.S; a.SP = p.SP; a.J = p.J; a.groups = p.groups; a.eg = p.eg; a.kg8 = p.kg / 8;
    a.x_pieces = (long long)p.groups * p.J * a.kg8;
    a.dy_pieces = (long long)p.groups * g.cout * a.kg8;
    if (g.kh * g.kw > 1) {
        bool done;
        const dp_status st = launch_pack_staged(g, p, x, xp, s, done);
        if (st != DP_OK) return st;
        if (done) a.x_pieces = 0;
    }
    const long long blocks = (a.x_pieces + a.dy_pieces + 255) / 256;
    if (blocks > 0x7FFFFFFFll) return fail(DP_ERR_UNSUPPORTED, "pack: layer too large");
    return submit_kernel<PackArgs>(TIER_PRE, reinterpret_cast<const void *>(&pack_weighted_kernel), a, (unsigned)blocks,
                                   256, 0, s, "pack_weighted");
}

}  // namespace dp
