// dp_per_example_grad_static: dp_per_example_grad for callers that cannot hand over (or allocate) a
// workspace -- code under HIP graph capture, tight serving loops, harnesses that forbid hipMalloc.
// The workspace is a file-scope device array of a fixed, modest size; every GPU the library runs on
// holds its own copy until the process ends.  In host code the array's name is only a stand-in: its
// device address is asked for once per device (hipGetSymbolAddress, with that device current) and
// that pointer, never the name, is what the kernels get.
#include "internal.h"

#include <mutex>

namespace {

constexpr size_t SCRATCH_BYTES = (size_t)32 << 20;
__device__ __align__(256) unsigned char scratch[SCRATCH_BYTES];

constexpr int MAX_DEVICES = 64;
void *g_scratch_ptr[MAX_DEVICES];       // device address of `scratch` on each device, once resolved
std::mutex g_scratch_mutex;

// Address of this device's copy of the array (resolved on the first call on that device).
dp_status scratch_of_current_device(void **out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return dp::fail(DP_ERR_DEVICE, "hipGetDevice failed: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= MAX_DEVICES) return dp::fail(DP_ERR_UNSUPPORTED, "device %d beyond the %d this build tracks", dev, MAX_DEVICES);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return dp::fail(DP_ERR_DEVICE, "hipGetSymbolAddress(scratch) failed on device %d: %s", dev, hipGetErrorString(e));
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return DP_OK;
}

}  // namespace

extern "C" {

size_t dp_static_scratch_bytes(void) { return SCRATCH_BYTES; }

dp_status dp_per_example_grad_static(const dp_layer_desc *desc, const void *x, const void *dy, float *g_w, float *g_b,
                                     size_t g_stride, float *sqnorm, dp_stream stream)
{
    size_t need = dp_workspace_bytes(desc, DP_WS_PER_EXAMPLE_GRAD);           // 0 on a bad descriptor: reported below
    // A dense layer of several tokens may need more (a slot for every 64 x 64 of the gradient) than what decides whether it is
    // taken: then its examples go through the scratch a piece at a time, which changes none of their numbers.
    int piece = need ? desc->n : 0;
    dp::Geo g;
    if (need && dp::make_geo(desc, g) == DP_OK && g.kind == DP_CONV2D && dp::conv3x3_applicable(g, dp::MODE_MATERIALISE) && dp::conv3x3_scratch_bytes(g) > need)
        need = dp::conv3x3_scratch_bytes(g);
    if (need > SCRATCH_BYTES && dp::make_geo(desc, g) == DP_OK && g.kind == DP_DENSE && dp::dense_scratch_bytes(g) <= SCRATCH_BYTES)
        piece = (int)(SCRATCH_BYTES / (need / (size_t)desc->n)) & ~7;          // (eight examples keep every address 16-byte aligned)
    if (need > SCRATCH_BYTES && (piece == desc->n || piece < 8))
        return dp::fail(DP_ERR_WORKSPACE, "this layer needs %zu bytes of workspace, the built-in scratch holds %zu; "
                        "use dp_per_example_grad with a caller-owned workspace", need, SCRATCH_BYTES);
    void *ws = nullptr;
    dp_status st = scratch_of_current_device(&ws);
    if (st != DP_OK) return st;
    if (need <= SCRATCH_BYTES) return dp_per_example_grad(desc, x, dy, g_w, g_b, g_stride, sqnorm, ws, SCRATCH_BYTES, stream);
    const size_t es = g.bf16 ? 2 : 4, row_w = g_stride ? g_stride : g.pw, row_b = g_stride ? g_stride : g.pb;
    for (int i = 0; i < g.n; i += piece) {
        dp_layer_desc part = *desc;
        part.n = g.n - i < piece ? g.n - i : piece;
        st = dp_per_example_grad(&part, x ? static_cast<const char *>(x) + i * g.x_elems * es : nullptr,
                                 dy ? static_cast<const char *>(dy) + i * g.dy_elems * es : nullptr, g_w ? g_w + i * row_w : nullptr,
                                 g_b ? g_b + i * row_b : nullptr, g_stride, sqnorm ? sqnorm + i : nullptr, ws, SCRATCH_BYTES, stream);
        if (st != DP_OK) return st;
    }
    return DP_OK;
}

}  // extern "C"
