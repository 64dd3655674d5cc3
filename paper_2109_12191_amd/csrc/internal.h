// Internal declarations shared by the translation units of libdp_privatise (gfx950 only).
#pragma once

#include <type_traits>
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/dp_privatise.h"

namespace dp {

// ---- error reporting (api.hip) ---------------------------------------------------------
dp_status fail(dp_status code, const char *fmt, ...);
dp_status check_launch(const char *what);

// ---- benchmark timing aid (api.hip): events armed by dp_profile_next_contraction.  A contraction
// launcher calls profile_begin(s) right before and profile_end(s) right after its main kernel.
void profile_begin(hipStream_t s);
void profile_end(hipStream_t s);

// ---- geometry of a validated descriptor ------------------------------------------------
struct Geo {
    int kind, bf16, n;
    int cin, cout, h, w, kh, kw, stride, pad, oh, ow;
    int has_bias, gn_groups;
    float gn_eps;
    int nhwc;               // conv / GroupNorm inputs arrive channels-last; the kernels read a transposed copy
    size_t pw, pb;          // weight / bias parameter counts
    size_t x_elems, dy_elems;   // per example
    // Where the examples of x / dy are.  0: one after the other from the given pointer.  k > 0: the pointer is a device array of
    // example addresses and example i starts at entry i * k (the micro-steps of a step, each in tensors of its own, contracted in
    // one launch; k > 1: the unit of a dense layer whose units are read as examples).
    int x_tab, dy_tab;
    // Per-example calls of convolutions: consecutive examples whose gradients are added up to one row of results (clipping units; K
    // then runs over the positions of all of them).  1 otherwise; n is a multiple of it.
    int unit;
    // Calls of bf16 layers on finished fp32 blocks.  Clip-weighted ones: the factors meet those (conv_scales_blocks), never an operand that is
    // rounded again.  Per-example ones: a squared norm is a sum of squares, never one of products that may cancel (gram.hip).
    int blocks;
    // Per-example batch calls: the workspace has room for operands whose rows get another length (dp_batch_workspace_bytes).
    int copies;
};

// Contraction modes of the conv / dense kernels.
enum Mode { MODE_NORM = 0, MODE_MATERIALISE = 1, MODE_WEIGHTED = 2 };

size_t conv_ws_bytes(const Geo &g, int mode);
const char *conv_variant_name(const Geo &g, int mode, bool shared);
// which launch of a batch call a convolution shares with others of its kind
enum { CONV_OTHER = 0, CONV_ROWS3 = 1, CONV_WHOLE_ROWS = 2 };
int conv_shared_launch(const Geo &g, int mode);
// bytes of the copy of X that a clip-weighted call of this layer packs by way of LDS, if that pays, or 0
size_t conv_staged_copy(const Geo &g);
bool pack_staged_fits(const Geo &g);
// multiply-adds of a call, and the work per workgroup (LaunchQueue::crowd) of a batch call whose convolutions have that many together
inline double conv_macs(const Geo &g) { return (double)g.n * g.cout * g.cin * g.kh * g.kw * g.oh * g.ow; }
int crowd_of(double macs);
constexpr double CROWD_UNIT = 768.0 * 128.0 * 128.0 * 64.0;
void c3_set_forced_crowd(int v);      // conv3x3.hip: plan as alone (0), as in a shared launch (1), or by the open batch (-1)
dp_status launch_conv(const Geo &g, int mode, const void *x, const void *dy, float *out_w, float *out_b,
                      size_t out_stride, float *sqnorm, const float *group_sqnorm, float clip_c, void *ws,
                      hipStream_t s);

// 3x3 stride-1 pad-1 bf16 convolutions staged from raw image rows (conv3x3.hip); launch_conv,
// conv_ws_bytes and conv_variant_name route to these when conv3x3_applicable() says so.
bool conv_scales_blocks(const Geo &g);
bool conv3x3_applicable(const Geo &g, int mode);
size_t conv3x3_ws_bytes(const Geo &g, int mode);
size_t conv3x3_scratch_bytes(const Geo &g);
const char *conv3x3_variant_name(const Geo &g, int mode);
dp_status launch_conv3x3(const Geo &g, int mode, const void *x, const void *dy, float *out_w, size_t out_stride,
                         float *sqnorm, const float *group_sqnorm, float clip_c, void *ws, hipStream_t s);

// Clipping units of normalisation layers: sums of the per-example gradients over `unit` consecutive examples (n a multiple of
// unit), and their squared norms [n / unit]; out_w / out_b rows are units.  (Convolutions: Geo::unit; dense layers read
// a unit as one example.)
const float *gn_unit_partials(const Geo &g, const void *ws);
size_t gn_unit_norm_partial_count(const Geo &g);
size_t gn_unit_ws_bytes(const Geo &g, int unit);
dp_status launch_gn_units(const Geo &g, int unit, const void *x, const void *dy, float *out_w, float *out_b,
                          size_t out_stride, float *sqnorm, void *ws, hipStream_t s);

// Packed operands of the clip-weighted contraction (pack.hip): K-contiguous, aligned, dY
// pre-scaled by the clip factors; `groups` example ranges of `eg` examples, rows of `kg` elements.
struct PackPlan {
    int S, SP, J, groups, eg, kg;
    size_t x_bytes, dy_bytes;
};
PackPlan pack_plan(const Geo &g, int groups, int row = 0);        // row: values of an example in a packed row (0: S rounded up to 8)
dp_status launch_pack_weighted(const Geo &g, const PackPlan &p, const void *x, const void *dy,
                               const float *group_sqnorm, float clip_c, void *xp, void *dyp, hipStream_t s);

// Partial squared norms per example that a per-example call leaves at the start of its workspace
// ([n, count] floats) when it is told not to reduce them (sqnorm == nullptr).
size_t conv_norm_partial_count(const Geo &g, int mode);
size_t conv3x3_norm_partial_count(const Geo &g);
size_t dense_norm_partial_count(const Geo &g, int mode);
size_t gn_norm_partial_count(const Geo &g);

// [n][positions][channels] -> [n][channels][positions], elements of 2 or 4 bytes (pack.hip): channels-last inputs
dp_status launch_to_channels_first(const void *in, void *out, int n, int positions, int channels, int elem_bytes, hipStream_t s);

// copy of an operand whose rows get another length (pack.hip): per example `channels` planes of dh x dw values, row-major, `row` values
// from one plane to the next; value (r, c) is in[r * step][c * step] of a plane of h x w where r < rows and c < cols, zero elsewhere
dp_status launch_widen(const void *in, int tab, void *out, int n, int channels, int h, int w, int rows, int cols, int step, int dw, int row,
                       hipStream_t s);

// compact copy of the rows / columns a strided 1x1 convolution reads: out[n*cin][OH*OW] (pack.hip)
dp_status launch_subsample(const Geo &g, const void *x, void *out, hipStream_t s);

// Norm-only calls of 1x1 convolutions on small feature maps through two Gram matrices (gram.hip).
// the network's first convolution (7x7, stride 2, pad 3, few input channels): stem.hip
bool stem_applicable(const Geo &g, int mode);
size_t stem_ws_bytes(const Geo &g);
size_t stem_norm_partial_count(void);
dp_status launch_stem(const Geo &g, const void *x, const void *dy, float *out_w, size_t out_stride, float *sqnorm, void *ws,
                      hipStream_t s);
// fp32 convolutions with square odd kernels from raw image rows, where that is faster than the general kernel: conv_rows.hip
double conv_general_f32_us(const Geo &g);
bool conv_rows_applicable(const Geo &g, int mode);
size_t conv_rows_ws_bytes(const Geo &g);
size_t conv_rows_norm_partial_count(const Geo &g);
const char *conv_rows_variant_name(const Geo &g);
dp_status launch_conv_rows(const Geo &g, const void *x, const void *dy, float *out_w, float *out_b, size_t out_stride, float *sqnorm,
                           void *ws, hipStream_t s);
bool gram_norm_applicable(const Geo &g, int mode);
size_t gram_ws_bytes(const Geo &g);
size_t gram_norm_partial_count(void);
dp_status launch_gram_norm(const Geo &g, const void *x, const void *dy, float *sqnorm, void *ws, hipStream_t s);

size_t dense_ws_bytes(const Geo &g, int mode);
size_t dense_scratch_bytes(const Geo &g);
dp_status make_geo(const dp_layer_desc *d, Geo &g);      // api.hip: validates a descriptor and derives its geometry
dp_status launch_dense(const Geo &g, int mode, const void *x, const void *dy, float *out_w, float *out_b,
                       size_t out_stride, float *sqnorm, const float *group_sqnorm, float clip_c, void *ws,
                       hipStream_t s);

size_t gn_ws_bytes(const Geo &g, int mode);
dp_status launch_gn(const Geo &g, int mode, const void *x, const void *dy, float *out_w, float *out_b,
                    size_t out_stride, float *sqnorm, const float *group_sqnorm, float clip_c, void *ws,
                    hipStream_t s);

// streaming kernels (stream_kernels.hip)
dp_status launch_sum_partials(const float *partials, int n, int per_example, float *sqnorm, hipStream_t s);
dp_status launch_norms(const float *layer_sqnorm, const int32_t *group_of_layer, int n_layers, int n,
                       int n_groups, float *group_sqnorm, hipStream_t s);
dp_status launch_norms_from_partials(const float *const *partials, const int32_t *counts, const int32_t *group_of_layer,
                                     int n_layers, int n, int n_groups, float *group_sqnorm, hipStream_t s);
dp_status launch_layer_norms(const float *const *partials, const int32_t *counts, float *const *out, int n_layers, int n,
                             hipStream_t s);
dp_status launch_clip_factors(const float *sqnorm, float clip_c, int n, float *f, hipStream_t s);
dp_status launch_clip_accumulate(const float *g, size_t stride, const float *sqnorm, float clip_c, int n,
                                 size_t p, float *acc, hipStream_t s);
dp_status launch_example_addresses(const void *const *tensors, const size_t *example_bytes, int n_operands, int n_tensors,
                                   int per_tensor, uint64_t *table, hipStream_t s);
dp_status launch_clip_accumulate_segments(const float *g, size_t stride, const float *group_sqnorm, const size_t *seg_begin,
                                          const size_t *seg_acc, const int32_t *seg_group, const float *seg_clip, int n_seg, int n, int run,
                                          size_t p, float *acc, hipStream_t s);
dp_status launch_noise_finalize(const float *acc, float *out, size_t p, float sigma, float clip_total,
                                uint64_t total_batch, uint64_t seed, uint64_t step, uint32_t tensor_id,
                                hipStream_t s);
dp_status launch_example_noise(float *acc, size_t p, float sigma, float clip_total, uint64_t total_batch, uint64_t seed,
                               uint64_t step, uint32_t tensor_id, uint64_t first_example, int count,
                               const uint64_t *step_dev, hipStream_t s);
dp_status launch_noise_finalize_update(const float *acc, float *theta, float *vbuf, float *out, size_t p, float sigma,
                                       float clip_total, uint64_t total_batch, uint64_t seed, uint64_t step,
                                       uint32_t tensor_id, float lr, float momentum, hipStream_t s);
dp_status launch_noise_finalize_flat(const float *acc, float *out, float *theta, float *vbuf, const uint64_t *seg_begin,
                                     const uint64_t *seg_size, const uint32_t *seg_tensor_id, int n_seg, float sigma,
                                     float clip_total, uint64_t total_batch, uint64_t seed, uint64_t step,
                                     const uint64_t *step_dev, float lr, float momentum, hipStream_t s);
dp_status launch_philox_raw(uint32_t *raw, size_t p, uint64_t seed, uint64_t step, uint32_t tensor_id,
                            hipStream_t s);

// ---- device helpers --------------------------------------------------------------------
#if defined(__HIP_DEVICE_COMPILE__) || defined(__HIPCC__)

// min(1, C / sqrt(n2)); 1 for a zero gradient or an infinite bound; 0 for a squared norm that is
// NaN or negative (a broken example contributes nothing instead of passing unclipped).
__device__ __forceinline__ float clip_factor(float n2, float clip_c)
{
    if (n2 == 0.0f) return 1.0f;
    const float r = clip_c / sqrtf(n2);     // +inf / x = +inf -> 1
    return r < 1.0f ? r : (r >= 1.0f ? 1.0f : 0.0f);
}

__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// The same sum by data-parallel-primitive moves (no trip through LDS), valid in lane 63 only: an inclusive scan inside
// each row of 16 lanes (shifts by 1, 2, 4, 8 with zeros shifted in), then lane 15 of rows 0 and 2 added into rows 1 and 3,
// then lane 31 into rows 2 and 3.  Fixed order: the same bits every run.
__device__ __forceinline__ float wave_sum_last_lane(float v)
{
    auto moved = [](float x, auto ctrl, auto rows) {
        return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(ctrl)::value,
                                                                     decltype(rows)::value, 0xf, true));
    };
    typedef std::integral_constant<int, 0xf> all_rows;
    v += moved(v, std::integral_constant<int, 0x111>{}, all_rows{});         // row_shr:1
    v += moved(v, std::integral_constant<int, 0x112>{}, all_rows{});         // row_shr:2
    v += moved(v, std::integral_constant<int, 0x114>{}, all_rows{});         // row_shr:4
    v += moved(v, std::integral_constant<int, 0x118>{}, all_rows{});         // row_shr:8
    v += moved(v, std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xa>{});   // row_bcast:15 into rows 1, 3
    v += moved(v, std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xc>{});   // row_bcast:31 into rows 2, 3
    return v;
}

// Sum over a workgroup of `NW` waves; result valid in every thread.  `red` holds NW floats.
template <int NW>
__device__ __forceinline__ float block_sum(float v, float *red)
{
    v = wave_sum(v);
    const int wave = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[wave] = v;
    __syncthreads();
    float t = 0.0f;
#pragma unroll
    for (int i = 0; i < NW; ++i) t += red[i];
    return t;
}

__device__ __forceinline__ float bf16_bits_to_float(uint16_t b)
{
    return __uint_as_float(((uint32_t)b) << 16);
}

// Start of example i of an operand (Geo::x_tab / dy_tab) of `elems` elements per example.
template <typename E>
__device__ __forceinline__ const E *example_at(const void *p, int tab, int i, size_t elems)
{
    if (tab) return reinterpret_cast<const E *>(static_cast<const unsigned long long *>(p)[(size_t)i * tab]);
    return static_cast<const E *>(p) + (size_t)i * elems;
}

// The same where i is the same in every lane: the address stays in scalar registers (a value read from memory would not).
template <typename E>
__device__ __forceinline__ const E *example_at_uniform(const void *p, int tab, int i, size_t elems)
{
    const unsigned long long v = reinterpret_cast<unsigned long long>(example_at<E>(p, tab, i, elems));
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v), hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
    return reinterpret_cast<const E *>(((unsigned long long)hi << 32) | lo);
}

// Element i of an array that nothing writes while the kernel runs, by a scalar load (i and the address are the same in every lane).
template <typename E>
__device__ __forceinline__ E scalar_load(unsigned long long array, size_t i)
{
    typedef const E __attribute__((address_space(4))) *constant;
    return reinterpret_cast<constant>(array)[i];
}

// one element of an input tensor as fp32
template <bool BF16> struct In;
template <> struct In<true> {
    typedef uint16_t type;
    static __device__ __forceinline__ float ld(const uint16_t *p) { return bf16_bits_to_float(*p); }
};
template <> struct In<false> {
    typedef float type;
    static __device__ __forceinline__ float ld(const float *p) { return *p; }
};

// round to nearest, ties to even (finite inputs)
__device__ __forceinline__ uint16_t float_to_bf16_bits(float f)
{
    const uint32_t u = __float_as_uint(f);
    return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

#endif

}  // namespace dp
