// C ABI of the SCC library: argument validation, window arithmetic, kernel selection.
// Every check except the launch status happens on the host before any HIP call.
#include "scc.h"
#include "scc_common.h"

#include <algorithm>
#include <cmath>
#include <limits>
#include <mutex>

// Scratch of scc_backward_weight_static: the K-split partials of grad-weight live here instead of in a
// caller-supplied workspace.  One copy per GPU, held until the process ends.  In host code the name is only a
// handle for hipGetSymbolAddress; the device address it resolves to is what the kernels get.
static __device__ __align__(256) unsigned char scratch[SCC_STATIC_SCRATCH_BYTES];

namespace {

using scc::Problem;

long long gcd_ll(long long a, long long b)
{
    while (b) {
        long long t = a % b;
        a = b;
        b = t;
    }
    return a;
}

// Algorithm 1 in closed form.  Returns SCC_OK or the status that rejects the arguments.
int make_problem(int N, int Cin, int Cout, int H, int W, int cg, double co, Problem* out)
{
    if (N <= 0 || Cin <= 0 || Cout <= 0 || H <= 0 || W <= 0 || cg < 1) return SCC_ERR_SHAPE;
    if (Cin % cg != 0) return SCC_ERR_SHAPE;
    if (!std::isfinite(co) || co < 0.0 || co > 1.0) return SCC_ERR_OVERLAP;
    const long long HW = (long long)H * W;
    const long long lim = std::numeric_limits<int>::max();
    // the kernels index columns, planes of one sample and the weight matrix with 32-bit ints
    if (HW > lim || HW * N > lim || HW * Cin > lim || HW * Cout > lim) return SCC_ERR_SHAPE;
    const int L = Cin / cg;
    if ((long long)Cout * L > lim) return SCC_ERR_SHAPE;
    const int ov = (int)(co * (double)L);  // truncation of the double product, as Algorithm 1 writes it
    const int stride = (L - ov) % Cin;     // L - ov == Cin only for cg == 1 with no overlap
    Problem p;
    p.N = N;
    p.Cin = Cin;
    p.Cout = Cout;
    p.HW = (int)HW;
    p.L = L;
    p.stride = stride;
    p.period = stride == 0 ? 1 : (int)(Cin / gcd_ll(stride, Cin));
    p.NQ = HW * N;
    *out = p;
    return SCC_OK;
}

bool dtype_ok(scc_dtype d) { return d == SCC_F32 || d == SCC_BF16; }

int launch_status(hipError_t e) { return e == hipSuccess ? SCC_OK : SCC_ERR_LAUNCH; }

// The launchers report hipGetLastError(), which also returns (and clears) an error an EARLIER, unrelated call of
// the process left behind.  Every entry point that launches drops such a leftover first, so that SCC_ERR_LAUNCH
// always speaks of this call's own kernels.
void drop_stale_error() { (void)hipGetLastError(); }

// Device address of `scratch` on the current device, resolved once per device (each GPU holds its own copy
// of the array at its own address).
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices];

int scratch_of_current_device(void** out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return SCC_ERR_LAUNCH;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress((void**)&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return SCC_ERR_LAUNCH;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return SCC_OK;
}

// f(T()) with T the storage type of `dtype`
template <typename F>
int with_type(scc_dtype dtype, F&& f)
{
    return dtype == SCC_F32 ? f(float()) : f(scc::bf16_t());
}

// SCC_FORWARD_*, or SCC_ERR_WORKSPACE.  bf16 layers that gain from it keep their weights in registers and leave a workspace they are
// given alone; else, with a workspace, the layers that packed_workspace names take the product with packed weights.
int forward_path(const Problem& p, int es, const void* y, const void* workspace, size_t workspace_bytes)
{
    const size_t need = workspace ? scc::packed_workspace<true>(p, es) : 0;
    if (need > 0 && (workspace_bytes < need || ((uintptr_t)workspace & 255u) != 0)) return SCC_ERR_WORKSPACE;
    if (scc::forward_resident_preferred(p, es, y, workspace != nullptr)) return SCC_FORWARD_RESIDENT;
    if (need > 0) return SCC_FORWARD_PACKED;
    return scc::forward_mfma_eligible(p) ? SCC_FORWARD_TILE : SCC_FORWARD_ANY;
}

template <typename T>
int run_forward(const T* x, const T* w, T* y, const Problem& p, void* workspace, size_t workspace_bytes, hipStream_t st)
{
    const int path = forward_path(p, (int)sizeof(T), y, workspace, workspace_bytes);
    if (path < 0) return path;
    drop_stale_error();
    if constexpr (sizeof(T) == 2) {
        if (path == SCC_FORWARD_RESIDENT) return launch_status(scc::launch_forward_resident(x, w, y, p, st));
    }
    if (path == SCC_FORWARD_PACKED) return launch_status(scc::launch_packed<T, true>(x, w, y, workspace, p, st));
    if (path == SCC_FORWARD_TILE) return launch_status(scc::launch_forward_mfma(x, w, y, p, st));
    return launch_status(scc::launch_forward_generic(x, w, y, p, st));
}

// Grad-input: with a workspace, the layers that packed_workspace names take the product with packed weights; without one, and
// every other layer, the kernels that need none.
template <typename T>
int run_backward_input(const T* dy, const T* w, T* dx, const Problem& p, void* workspace, size_t workspace_bytes, hipStream_t st)
{
    const size_t need = workspace ? scc::packed_workspace<false>(p, (int)sizeof(T)) : 0;
    if (need > 0 && (workspace_bytes < need || ((uintptr_t)workspace & 255u) != 0)) return SCC_ERR_WORKSPACE;
    drop_stale_error();
    if (need > 0) return launch_status(scc::launch_packed<T, false>(dy, w, dx, workspace, p, st));
    if (scc::backward_input_mfma_eligible(p)) return launch_status(scc::launch_backward_input_mfma(dy, w, dx, p, st));
    return launch_status(scc::launch_backward_input_generic(dy, w, dx, p, st));
}

int size_of(scc_dtype dtype) { return dtype == SCC_F32 ? 4 : 2; }

// Whether a call may use `need` bytes of its workspace.
bool holds(size_t need, const void* workspace, size_t workspace_bytes)
{
    return need == 0 || (workspace && workspace_bytes >= need && ((uintptr_t)workspace & 255u) == 0);
}

// Grad-weight: the kernel that shares its operands between filter tiles on the layers that gain from it (`shared`) where
// the workspace holds its partial sums, else the one with a tile per wavefront, else the one for any shape.  A workspace of
// weight_least bytes is what a call cannot do without.
size_t weight_least(const Problem& p)
{
    return scc::backward_weight_mfma_eligible(p) ? scc::backward_weight_mfma_workspace(p) : 0;
}

size_t weight_shared_need(const Problem& p, scc_dtype dtype)   // 0: not a layer for that kernel
{
    const int es = size_of(dtype);
    return scc::backward_weight_shared_preferred(p, es) ? scc::backward_weight_shared_workspace(p, es) : 0;
}

// SCC_WEIGHT_*, or SCC_ERR_WORKSPACE.
int weight_path(const Problem& p, scc_dtype dtype, const void* workspace, size_t workspace_bytes)
{
    if (!holds(weight_least(p), workspace, workspace_bytes)) return SCC_ERR_WORKSPACE;
    const size_t need = weight_shared_need(p, dtype);
    if (need > 0 && holds(need, workspace, workspace_bytes)) return SCC_WEIGHT_SHARED;
    return scc::backward_weight_mfma_eligible(p) ? SCC_WEIGHT_TILE : SCC_WEIGHT_ANY;
}

int run_weight(const void* x, const void* dy, void* dw, const Problem& p, scc_dtype dtype, int path, void* workspace,
               hipStream_t st)
{
    drop_stale_error();
    return with_type(dtype, [&](auto t) {
        typedef const decltype(t)* In;
        if (path == SCC_WEIGHT_SHARED)
            return launch_status(scc::launch_backward_weight_shared((In)x, (In)dy, (float*)dw, (float*)workspace, p, st));
        if (path == SCC_WEIGHT_TILE)
            return launch_status(scc::launch_backward_weight_mfma((In)x, (In)dy, (float*)dw, (float*)workspace, p, st));
        return launch_status(scc::launch_backward_weight_generic((In)x, (In)dy, (float*)dw, p, st));
    });
}

size_t align256(size_t v) { return (v + 255) / 256 * 256; }

}  // namespace

extern "C" {

int scc_window_params(int Cin, int Cout, int cg, double co, int* L, int* stride, int* period)
{
    Problem p;
    const int rc = make_problem(1, Cin, Cout, 1, 1, cg, co, &p);
    if (rc != SCC_OK) return rc;
    if (L) *L = p.L;
    if (stride) *stride = p.L - (int)(co * (double)p.L);
    if (period) *period = p.period < Cout ? p.period : Cout;
    return SCC_OK;
}

size_t scc_forward_workspace_bytes(int N, int Cin, int Cout, int H, int W, int cg, double co, scc_dtype dtype)
{
    Problem p;
    if (make_problem(N, Cin, Cout, H, W, cg, co, &p) != SCC_OK || !dtype_ok(dtype)) return 0;
    return scc::packed_workspace<true>(p, dtype == SCC_F32 ? 4 : 2);
}

int scc_forward_ws(const void* x, const void* w, void* y, int N, int Cin, int Cout, int H, int W, int cg, double co,
                   scc_dtype dtype, void* workspace, size_t workspace_bytes, void* stream)
{
    if (!x || !w || !y) return SCC_ERR_NULL;
    Problem p;
    const int rc = make_problem(N, Cin, Cout, H, W, cg, co, &p);
    if (rc != SCC_OK) return rc;
    if (!dtype_ok(dtype)) return SCC_ERR_DTYPE;
    return with_type(dtype, [&](auto t) {
        typedef decltype(t) T;
        return run_forward<T>((const T*)x, (const T*)w, (T*)y, p, workspace, workspace_bytes, (hipStream_t)stream);
    });
}

int scc_forward_path(int N, int Cin, int Cout, int H, int W, int cg, double co, scc_dtype dtype, size_t workspace_bytes)
{
    Problem p;
    const int rc = make_problem(N, Cin, Cout, H, W, cg, co, &p);
    if (rc != SCC_OK) return rc;
    if (!dtype_ok(dtype)) return SCC_ERR_DTYPE;
    return forward_path(p, dtype == SCC_F32 ? 4 : 2, nullptr, workspace_bytes ? (const void*)256 : nullptr, workspace_bytes);   // aligned addresses
}

int scc_forward(const void* x, const void* w, void* y, int N, int Cin, int Cout, int H, int W, int cg, double co,
                scc_dtype dtype, void* stream)
{
    return scc_forward_ws(x, w, y, N, Cin, Cout, H, W, cg, co, dtype, nullptr, 0, stream);
}

size_t scc_backward_input_workspace_bytes(int N, int Cin, int Cout, int H, int W, int cg, double co, scc_dtype dtype)
{
    Problem p;
    if (make_problem(N, Cin, Cout, H, W, cg, co, &p) != SCC_OK || !dtype_ok(dtype)) return 0;
    return scc::packed_workspace<false>(p, dtype == SCC_F32 ? 4 : 2);
}

int scc_backward_input_ws(const void* dy, const void* w, void* dx, int N, int Cin, int Cout, int H, int W, int cg,
                          double co, scc_dtype dtype, void* workspace, size_t workspace_bytes, void* stream)
{
    if (!dy || !w || !dx) return SCC_ERR_NULL;
    Problem p;
    const int rc = make_problem(N, Cin, Cout, H, W, cg, co, &p);
    if (rc != SCC_OK) return rc;
    if (!dtype_ok(dtype)) return SCC_ERR_DTYPE;
    return with_type(dtype, [&](auto t) {
        typedef decltype(t) T;
        return run_backward_input<T>((const T*)dy, (const T*)w, (T*)dx, p, workspace, workspace_bytes, (hipStream_t)stream);
    });
}

int scc_backward_input(const void* dy, const void* w, void* dx, int N, int Cin, int Cout, int H, int W, int cg,
                       double co, scc_dtype dtype, void* stream)
{
    return scc_backward_input_ws(dy, w, dx, N, Cin, Cout, H, W, cg, co, dtype, nullptr, 0, stream);
}

size_t scc_backward_weight_workspace_bytes(int N, int Cin, int Cout, int H, int W, int cg, double co, scc_dtype dtype)
{
    Problem p;
    if (make_problem(N, Cin, Cout, H, W, cg, co, &p) != SCC_OK || !dtype_ok(dtype)) return 0;
    return std::max(weight_least(p), weight_shared_need(p, dtype));
}

int scc_backward_weight(const void* x, const void* dy, void* dw, int N, int Cin, int Cout, int H, int W, int cg,
                        double co, scc_dtype dtype, void* workspace, size_t workspace_bytes, void* stream)
{
    if (!x || !dy || !dw) return SCC_ERR_NULL;
    Problem p;
    const int rc = make_problem(N, Cin, Cout, H, W, cg, co, &p);
    if (rc != SCC_OK) return rc;
    if (!dtype_ok(dtype)) return SCC_ERR_DTYPE;
    const int path = weight_path(p, dtype, workspace, workspace_bytes);
    if (path < 0) return path;
    return run_weight(x, dy, dw, p, dtype, path, workspace, (hipStream_t)stream);
}

// scc_backward: what a call cannot do without, whichever of the kernels that follow runs (tensors that are not aligned to
// 16 bytes keep a layer from the fused one), and what the launch of both shared kernels takes (0: not a layer for it).
static size_t backward_least(const Problem& p, scc_dtype dtype)
{
    const size_t least = weight_least(p);
    return dtype == SCC_F32 && scc::backward_fused_eligible(p) ? std::max(least, scc::backward_fused_workspace(p)) : least;
}

static size_t backward_shared_need(const Problem& p, scc_dtype dtype)
{
    if (dtype == SCC_F32 && scc::backward_fused_eligible(p)) return 0;
    return scc::backward_shared_workspace(p, size_of(dtype));
}

// SCC_BACKWARD_*, or SCC_ERR_WORKSPACE.
static int backward_path(const Problem& p, scc_dtype dtype, bool aligned, const void* workspace, size_t workspace_bytes)
{
    if (!holds(backward_least(p, dtype), workspace, workspace_bytes)) return SCC_ERR_WORKSPACE;
    if (dtype == SCC_F32 && aligned && scc::backward_fused_eligible(p)) return SCC_BACKWARD_FUSED;
    const size_t shared = backward_shared_need(p, dtype);
    if (shared > 0 && holds(shared, workspace, workspace_bytes)) return SCC_BACKWARD_SHARED;
    // layers both per-tile kernels take: their two grids as one launch
    const bool merged = with_type(dtype, [&](auto t) { return (int)scc::backward_merged_applicable<decltype(t)>(p); });
    return merged ? SCC_BACKWARD_MERGED : SCC_BACKWARD_TWO_PASSES;
}

int scc_backward_weight_path(int N, int Cin, int Cout, int H, int W, int cg, double co, scc_dtype dtype, size_t workspace_bytes)
{
    Problem p;
    const int rc = make_problem(N, Cin, Cout, H, W, cg, co, &p);
    if (rc != SCC_OK) return rc;
    if (!dtype_ok(dtype)) return SCC_ERR_DTYPE;
    return weight_path(p, dtype, workspace_bytes ? (const void*)256 : nullptr, workspace_bytes);   // any aligned address
}

int scc_backward_path(int N, int Cin, int Cout, int H, int W, int cg, double co, scc_dtype dtype, size_t workspace_bytes)
{
    Problem p;
    const int rc = make_problem(N, Cin, Cout, H, W, cg, co, &p);
    if (rc != SCC_OK) return rc;
    if (!dtype_ok(dtype)) return SCC_ERR_DTYPE;
    return backward_path(p, dtype, true, workspace_bytes ? (const void*)256 : nullptr, workspace_bytes);
}

static size_t backward_need(const Problem& p, scc_dtype dtype)
{
    size_t most = backward_shared_need(p, dtype);
    const bool two_passes = most == 0 && !(dtype == SCC_F32 && scc::backward_fused_eligible(p)) &&
                            !with_type(dtype, [&](auto t) { return (int)scc::backward_merged_applicable<decltype(t)>(p); });
    if (two_passes) most = weight_shared_need(p, dtype);
    return std::max(backward_least(p, dtype), most);
}

size_t scc_backward_workspace_bytes(int N, int Cin, int Cout, int H, int W, int cg, double co, scc_dtype dtype)
{
    Problem p;
    if (make_problem(N, Cin, Cout, H, W, cg, co, &p) != SCC_OK || !dtype_ok(dtype)) return 0;
    return backward_need(p, dtype);
}

int scc_backward(const void* x, const void* dy, const void* w, void* dx, void* dw, int N, int Cin, int Cout, int H,
                 int W, int cg, double co, scc_dtype dtype, void* workspace, size_t workspace_bytes, void* stream)
{
    if (!x || !dy || !w || !dx || !dw) return SCC_ERR_NULL;
    Problem p;
    const int rc = make_problem(N, Cin, Cout, H, W, cg, co, &p);
    if (rc != SCC_OK) return rc;
    if (!dtype_ok(dtype)) return SCC_ERR_DTYPE;
    const bool aligned = (((uintptr_t)x | (uintptr_t)dy | (uintptr_t)dx) & 15u) == 0;
    const int path = backward_path(p, dtype, aligned, workspace, workspace_bytes);
    if (path < 0) return path;
    drop_stale_error();
    const hipStream_t st = (hipStream_t)stream;
    if (path == SCC_BACKWARD_FUSED)
        return launch_status(scc::launch_backward_fused((const float*)x, (const float*)dy, (const float*)w, (float*)dx,
                                                        (float*)dw, (float*)workspace, p, st));
    if (path == SCC_BACKWARD_SHARED || path == SCC_BACKWARD_MERGED)
        return with_type(dtype, [&](auto t) {
            typedef decltype(t) T;
            return launch_status(path == SCC_BACKWARD_SHARED
                                     ? scc::launch_backward_shared((const T*)x, (const T*)dy, (const T*)w, (T*)dx, (float*)dw,
                                                                   workspace, p, st)
                                     : scc::launch_backward_merged((const T*)x, (const T*)dy, (const T*)w, (T*)dx, (float*)dw,
                                                                   (float*)workspace, p, st));
        });
    // every other layer: the two passes one after the other
    const int r1 = scc_backward_input(dy, w, dx, N, Cin, Cout, H, W, cg, co, dtype, stream);
    if (r1 != SCC_OK) return r1;
    return scc_backward_weight(x, dy, dw, N, Cin, Cout, H, W, cg, co, dtype, workspace, workspace_bytes, stream);
}

// Geometry of the depthwise stage; SCC_ERR_SHAPE for a stride below 1 or maps too large for 32-bit pixel indices.
static int make_dw_geom(int C, int H, int W, int dw_stride, scc::DwGeom* g)
{
    if (C <= 0 || H <= 0 || W <= 0 || dw_stride < 1) return SCC_ERR_SHAPE;
    if ((long long)H * W * C > std::numeric_limits<int>::max()) return SCC_ERR_SHAPE;
    g->H = H;
    g->W = W;
    g->s = dw_stride;
    g->Ho = (H - 1) / dw_stride + 1;
    g->Wo = (W - 1) / dw_stride + 1;
    return SCC_OK;
}

int scc_depthwise3x3_out(int size, int dw_stride)
{
    if (size <= 0 || dw_stride < 1) return SCC_ERR_SHAPE;
    return (size - 1) / dw_stride + 1;
}

int scc_depthwise3x3_forward(const void* x, const void* kdw, void* z, int N, int C, int H, int W, int dw_stride,
                             scc_dtype dtype, void* stream)
{
    if (!x || !kdw || !z) return SCC_ERR_NULL;
    scc::DwGeom g;
    if (N <= 0) return SCC_ERR_SHAPE;
    const int rc = make_dw_geom(C, H, W, dw_stride, &g);
    if (rc != SCC_OK) return rc;
    if ((long long)N * H * W > std::numeric_limits<int>::max()) return SCC_ERR_SHAPE;
    if (!dtype_ok(dtype)) return SCC_ERR_DTYPE;
    drop_stale_error();
    if (dtype == SCC_F32)
        return launch_status(
            scc::launch_depthwise3x3((const float*)x, (const float*)kdw, (float*)z, N, C, g, (hipStream_t)stream));
    return launch_status(scc::launch_depthwise3x3((const scc::bf16_t*)x, (const scc::bf16_t*)kdw, (scc::bf16_t*)z, N, C,
                                                  g, (hipStream_t)stream));
}

size_t scc_depthwise3x3_backward_workspace_bytes(int N, int C, int H, int W, int dw_stride, scc_dtype dtype)
{
    scc::DwGeom g;
    if (N <= 0 || make_dw_geom(C, H, W, dw_stride, &g) != SCC_OK || !dtype_ok(dtype)) return 0;
    return scc::depthwise3x3_backward_workspace(N, C, g);
}

int scc_depthwise3x3_backward(const void* x, const void* kdw, const void* dz, void* dx, void* dkdw, int N, int C, int H,
                              int W, int dw_stride, scc_dtype dtype, void* workspace, size_t workspace_bytes,
                              void* stream)
{
    if (!dz || (!dx && !dkdw) || (dx && !kdw) || (dkdw && !x)) return SCC_ERR_NULL;
    scc::DwGeom g;
    if (N <= 0) return SCC_ERR_SHAPE;
    const int rc = make_dw_geom(C, H, W, dw_stride, &g);
    if (rc != SCC_OK) return rc;
    if ((long long)N * H * W > std::numeric_limits<int>::max()) return SCC_ERR_SHAPE;
    if (!dtype_ok(dtype)) return SCC_ERR_DTYPE;
    const size_t need = dkdw ? scc::depthwise3x3_backward_workspace(N, C, g) : 0;
    if (need > 0 && (!workspace || workspace_bytes < need || ((uintptr_t)workspace & 255u) != 0))
        return SCC_ERR_WORKSPACE;
    drop_stale_error();
    if (dtype == SCC_F32)
        return launch_status(scc::launch_depthwise3x3_backward((const float*)x, (const float*)kdw, (const float*)dz,
                                                               (float*)dx, (float*)dkdw, (float*)workspace, N, C, g,
                                                               (hipStream_t)stream));
    return launch_status(scc::launch_depthwise3x3_backward((const scc::bf16_t*)x, (const scc::bf16_t*)kdw,
                                                           (const scc::bf16_t*)dz, (scc::bf16_t*)dx, (float*)dkdw,
                                                           (float*)workspace, N, C, g, (hipStream_t)stream));
}

// Problem of the SCC behind the depthwise stage (it sees the Ho x Wo map) and the stage's geometry.
static int make_dw_problem(int N, int Cin, int Cout, int H, int W, int dw_stride, int cg, double co, Problem* p,
                           scc::DwGeom* g)
{
    if (N <= 0) return SCC_ERR_SHAPE;
    int rc = make_dw_geom(Cin, H, W, dw_stride, g);
    if (rc != SCC_OK) return rc;
    if ((long long)N * H * W > std::numeric_limits<int>::max()) return SCC_ERR_SHAPE;
    return make_problem(N, Cin, Cout, g->Ho, g->Wo, cg, co, p);
}

// The depthwise stage's output, or nothing where one kernel keeps it on chip by the library's own choice.
static size_t dw_forward_need(const Problem& p, const scc::DwGeom& g, scc_dtype dtype)
{
    if (dtype == SCC_F32 && scc::dw_forward_fused_preferred(p, g)) return 0;
    return (size_t)p.NQ * p.Cin * size_of(dtype);
}

size_t scc_dw_forward_workspace_bytes(int N, int Cin, int Cout, int H, int W, int dw_stride, int cg, double co,
                                      scc_dtype dtype)
{
    Problem p;
    scc::DwGeom g;
    if (make_dw_problem(N, Cin, Cout, H, W, dw_stride, cg, co, &p, &g) != SCC_OK || !dtype_ok(dtype)) return 0;
    return dw_forward_need(p, g, dtype);
}

int scc_dw_forward_fusable(int N, int Cin, int Cout, int H, int W, int dw_stride, int cg, double co, scc_dtype dtype)
{
    Problem p;
    scc::DwGeom g;
    const int rc = make_dw_problem(N, Cin, Cout, H, W, dw_stride, cg, co, &p, &g);
    if (rc != SCC_OK) return rc;
    if (!dtype_ok(dtype)) return SCC_ERR_DTYPE;
    return dtype == SCC_F32 && scc::dw_forward_fused_eligible(p) ? 1 : 0;
}

// SCC_DW_FORWARD_*, or SCC_ERR_WORKSPACE.  keep: a workspace that two stages would run in holds the depthwise output afterwards.
static int dw_forward_path(const Problem& p, const scc::DwGeom& g, scc_dtype dtype, bool keep, const void* workspace,
                           size_t workspace_bytes)
{
    const size_t need = dw_forward_need(p, g, dtype);
    const bool room = workspace && workspace_bytes >= need && ((uintptr_t)workspace & 255u) == 0;
    // without a workspace the fused kernel runs wherever it can, also where the two stages would be faster; from kFusedPixels on a workspace
    // that does not do is none
    const bool fused = dtype == SCC_F32 && (need == 0 || (scc::dw_forward_fused_eligible(p) &&
                                                          (!workspace || (!room && p.NQ >= scc::kFusedPixels))));
    if (!fused && !room) return SCC_ERR_WORKSPACE;
    if ((fused || !keep) && scc::dw_forward_few_preferred(p, g, size_of(dtype), fused)) return SCC_DW_FORWARD_FEW;   // touches no workspace
    return fused ? SCC_DW_FORWARD_FUSED : SCC_DW_FORWARD_TWO_STAGES;
}

static int dw_forward_path_of(int N, int Cin, int Cout, int H, int W, int dw_stride, int cg, double co, scc_dtype dtype, bool keep,
                              size_t workspace_bytes)
{
    Problem p;
    scc::DwGeom g;
    const int rc = make_dw_problem(N, Cin, Cout, H, W, dw_stride, cg, co, &p, &g);
    if (rc != SCC_OK) return rc;
    if (!dtype_ok(dtype)) return SCC_ERR_DTYPE;
    return dw_forward_path(p, g, dtype, keep, workspace_bytes ? (const void*)256 : nullptr, workspace_bytes);   // any aligned address
}

int scc_dw_forward_path(int N, int Cin, int Cout, int H, int W, int dw_stride, int cg, double co, scc_dtype dtype,
                        size_t workspace_bytes)
{
    return dw_forward_path_of(N, Cin, Cout, H, W, dw_stride, cg, co, dtype, true, workspace_bytes);
}

int scc_dw_forward_scratch_path(int N, int Cin, int Cout, int H, int W, int dw_stride, int cg, double co, scc_dtype dtype,
                                size_t workspace_bytes)
{
    return dw_forward_path_of(N, Cin, Cout, H, W, dw_stride, cg, co, dtype, false, workspace_bytes);
}

static int dw_forward(const void* x, const void* kdw, const void* w, void* y, int N, int Cin, int Cout, int H, int W,
                      int dw_stride, int cg, double co, scc_dtype dtype, void* workspace, size_t workspace_bytes,
                      void* stream, bool keep)
{
    if (!x || !kdw || !w || !y) return SCC_ERR_NULL;
    Problem p;
    scc::DwGeom g;
    const int rc = make_dw_problem(N, Cin, Cout, H, W, dw_stride, cg, co, &p, &g);
    if (rc != SCC_OK) return rc;
    if (!dtype_ok(dtype)) return SCC_ERR_DTYPE;
    const int path = dw_forward_path(p, g, dtype, keep, workspace, workspace_bytes);
    if (path < 0) return path;
    drop_stale_error();
    if (path == SCC_DW_FORWARD_FEW) {
        return with_type(dtype, [&](auto t) {
            typedef decltype(t) T;
            return launch_status(scc::launch_dw_forward_few((const T*)x, (const T*)kdw, (const T*)w, (T*)y, p, g,
                                                            (hipStream_t)stream));
        });
    }
    if (path == SCC_DW_FORWARD_FUSED)
        return launch_status(scc::launch_dw_forward_fused((const float*)x, (const float*)kdw, (const float*)w, (float*)y,
                                                          p, g, (hipStream_t)stream));
    // every other layer: the depthwise stage into the workspace, then the SCC forward on it
    const int r1 = scc_depthwise3x3_forward(x, kdw, workspace, N, Cin, H, W, dw_stride, dtype, stream);
    if (r1 != SCC_OK) return r1;
    return scc_forward(workspace, w, y, N, Cin, Cout, g.Ho, g.Wo, cg, co, dtype, stream);
}

int scc_dw_forward(const void* x, const void* kdw, const void* w, void* y, int N, int Cin, int Cout, int H, int W,
                   int dw_stride, int cg, double co, scc_dtype dtype, void* workspace, size_t workspace_bytes,
                   void* stream)
{
    return dw_forward(x, kdw, w, y, N, Cin, Cout, H, W, dw_stride, cg, co, dtype, workspace, workspace_bytes, stream, true);
}

int scc_dw_forward_scratch(const void* x, const void* kdw, const void* w, void* y, int N, int Cin, int Cout, int H, int W,
                           int dw_stride, int cg, double co, scc_dtype dtype, void* workspace, size_t workspace_bytes,
                           void* stream)
{
    return dw_forward(x, kdw, w, y, N, Cin, Cout, H, W, dw_stride, cg, co, dtype, workspace, workspace_bytes, stream, false);
}

// The workspace of scc_dw_backward: the depthwise output, its gradient, then the scratch of whichever stage runs.
static size_t dw_backward_plane_bytes(const Problem& p, scc_dtype dtype)
{
    return align256((size_t)p.NQ * p.Cin * (dtype == SCC_F32 ? 4 : 2));
}

// What a call that adds each gradient's slices right behind its stage cannot do without.
static size_t dw_backward_least(const Problem& p, const scc::DwGeom& g, scc_dtype dtype)
{
    return 2 * dw_backward_plane_bytes(p, dtype) +
           std::max(backward_need(p, dtype), scc::depthwise3x3_backward_workspace(p.N, p.Cin, g));
}

// What one that adds them together at the end takes: the scratch of both at once and, where the gradients leave rounded, both in
// binary32.
static size_t dw_backward_whole(const Problem& p, const scc::DwGeom& g, scc_dtype dtype, scc_dtype grad)
{
    const size_t wide = grad == SCC_BF16 ? align256((size_t)p.Cout * p.L * 4) + align256((size_t)p.Cin * 9 * 4) : 0;
    return 2 * dw_backward_plane_bytes(p, dtype) + align256(backward_need(p, dtype)) +
           align256(scc::depthwise3x3_backward_workspace(p.N, p.Cin, g)) + wide;
}

size_t scc_dw_backward_as_workspace_bytes(int N, int Cin, int Cout, int H, int W, int dw_stride, int cg, double co,
                                          scc_dtype dtype, scc_dtype grad)
{
    Problem p;
    scc::DwGeom g;
    if (make_dw_problem(N, Cin, Cout, H, W, dw_stride, cg, co, &p, &g) != SCC_OK || !dtype_ok(dtype) || !dtype_ok(grad)) return 0;
    return dw_backward_whole(p, g, dtype, grad);
}

size_t scc_dw_backward_workspace_bytes(int N, int Cin, int Cout, int H, int W, int dw_stride, int cg, double co,
                                       scc_dtype dtype)
{
    Problem p;
    scc::DwGeom g;
    if (make_dw_problem(N, Cin, Cout, H, W, dw_stride, cg, co, &p, &g) != SCC_OK || !dtype_ok(dtype)) return 0;
    return dw_backward_least(p, g, dtype);
}

int scc_dw_backward_as(const void* x, const void* kdw, const void* w, const void* dy, void* dx, void* dkdw, void* dw, int N,
                       int Cin, int Cout, int H, int W, int dw_stride, int cg, double co, scc_dtype dtype, scc_dtype grad,
                       void* workspace, size_t workspace_bytes, void* stream)
{
    if (!x || !kdw || !w || !dy || !dx || !dkdw || !dw) return SCC_ERR_NULL;
    Problem p;
    scc::DwGeom g;
    const int rc = make_dw_problem(N, Cin, Cout, H, W, dw_stride, cg, co, &p, &g);
    if (rc != SCC_OK) return rc;
    if (!dtype_ok(dtype) || !dtype_ok(grad)) return SCC_ERR_DTYPE;
    const size_t whole = dw_backward_whole(p, g, dtype, grad);
    const bool together = workspace && holds(whole, workspace, workspace_bytes);
    if (!together && (grad != SCC_F32 || !workspace || !holds(dw_backward_least(p, g, dtype), workspace, workspace_bytes)))
        return SCC_ERR_WORKSPACE;
    const size_t plane = dw_backward_plane_bytes(p, dtype);
    char* z = (char*)workspace;
    char* dz = z + plane;
    char* rest = dz + plane;
    int r;
    if (!together) {
        r = scc_depthwise3x3_forward(x, kdw, z, N, Cin, H, W, dw_stride, dtype, stream);
        if (r != SCC_OK) return r;
        r = scc_backward(z, dy, w, dz, dw, N, Cin, Cout, g.Ho, g.Wo, cg, co, dtype, rest, workspace_bytes - 2 * plane, stream);
        if (r != SCC_OK) return r;
        return scc_depthwise3x3_backward(x, kdw, dz, dx, dkdw, N, Cin, H, W, dw_stride, dtype, rest, workspace_bytes - 2 * plane,
                                         stream);
    }
    const hipStream_t st = (hipStream_t)stream;
    const size_t need = backward_need(p, dtype);
    char* part_k = rest + align256(need);
    char* wide = part_k + align256(scc::depthwise3x3_backward_workspace(N, Cin, g));
    // where the kernels put a gradient of one slice
    float* to_w = grad == SCC_F32 ? (float*)dw : (float*)wide;
    float* to_k = grad == SCC_F32 ? (float*)dkdw : (float*)(wide + align256((size_t)Cout * p.L * 4));
    scc::SliceSum sum_w = {to_w, Cout * p.L, 1}, sum_k = {to_k, Cin * 9, 1};
    const bool aligned = ((uintptr_t)dy & 15u) == 0;                       // z and dz are
    const int path = backward_path(p, dtype, aligned, rest, need);
    if (path < 0) return path;
    drop_stale_error();
    r = with_type(dtype, [&](auto t) {
        typedef decltype(t) T;
        const T *tx = (const T*)x, *tk = (const T*)kdw, *tw = (const T*)w, *ty = (const T*)dy;
        if (path == SCC_BACKWARD_MERGED && scc::block_backward_applicable<T>(p, g))
            return launch_status(scc::launch_block_backward(tx, tk, tw, ty, (T*)dx, to_k, to_w, (T*)z, (T*)dz, (float*)rest,
                                                            (float*)part_k, &sum_w, &sum_k, p, g, st));
        int e = scc_depthwise3x3_forward(x, kdw, z, N, Cin, H, W, dw_stride, dtype, stream);
        if (e != SCC_OK) return e;
        if (path == SCC_BACKWARD_FUSED)
            e = launch_status(scc::launch_backward_fused((const float*)z, (const float*)dy, (const float*)w, (float*)dz, to_w,
                                                         (float*)rest, p, st, &sum_w));
        else if (path == SCC_BACKWARD_SHARED)
            e = launch_status(scc::launch_backward_shared((const T*)z, ty, tw, (T*)dz, to_w, rest, p, st, &sum_w));
        else if (path == SCC_BACKWARD_MERGED)
            e = launch_status(scc::launch_backward_merged((const T*)z, ty, tw, (T*)dz, to_w, (float*)rest, p, st, &sum_w));
        else
            e = scc_backward(z, dy, w, dz, to_w, N, Cin, Cout, g.Ho, g.Wo, cg, co, dtype, rest, need, stream);
        if (e != SCC_OK) return e;
        return launch_status(scc::launch_depthwise3x3_backward(tx, tk, (const T*)dz, (T*)dx, to_k, (float*)part_k, N, Cin, g, st,
                                                               &sum_k));
    });
    if (r != SCC_OK) return r;
    if (grad == SCC_F32) return launch_status(scc::launch_gradient_sums(sum_w, (float*)dw, sum_k, (float*)dkdw, st));
    return launch_status(scc::launch_gradient_sums(sum_w, (scc::bf16_t*)dw, sum_k, (scc::bf16_t*)dkdw, st));
}

int scc_dw_backward(const void* x, const void* kdw, const void* w, const void* dy, void* dx, void* dkdw, void* dw, int N,
                    int Cin, int Cout, int H, int W, int dw_stride, int cg, double co, scc_dtype dtype, void* workspace,
                    size_t workspace_bytes, void* stream)
{
    return scc_dw_backward_as(x, kdw, w, dy, dx, dkdw, dw, N, Cin, Cout, H, W, dw_stride, cg, co, dtype, SCC_F32, workspace,
                              workspace_bytes, stream);
}

int scc_backward_weight_static(const void* x, const void* dy, void* dw, int N, int Cin, int Cout, int H, int W, int cg,
                               double co, scc_dtype dtype, void* stream)
{
    if (!x || !dy || !dw) return SCC_ERR_NULL;
    Problem p;
    const int rc = make_problem(N, Cin, Cout, H, W, cg, co, &p);
    if (rc != SCC_OK) return rc;
    if (!dtype_ok(dtype)) return SCC_ERR_DTYPE;
    const size_t need = std::max(weight_least(p), weight_shared_need(p, dtype));
    if (need > (size_t)SCC_STATIC_SCRATCH_BYTES) return SCC_ERR_SCRATCH;
    void* ptr = nullptr;
    if (need > 0) {
        const int sc = scratch_of_current_device(&ptr);
        if (sc != SCC_OK) return sc;
    }
    return run_weight(x, dy, dw, p, dtype, weight_path(p, dtype, ptr, need), ptr, (hipStream_t)stream);
}

const char* scc_status_string(int status)
{
    switch (status) {
        case SCC_OK: return "SCC_OK";
        case SCC_ERR_NULL: return "SCC_ERR_NULL: a required pointer is NULL";
        case SCC_ERR_SHAPE: return "SCC_ERR_SHAPE: non-positive dimension, cg < 1, Cin not divisible by cg, or tensor too large";
        case SCC_ERR_OVERLAP: return "SCC_ERR_OVERLAP: co must be finite and within [0, 1]";
        case SCC_ERR_DTYPE: return "SCC_ERR_DTYPE: dtype must be SCC_F32 or SCC_BF16";
        case SCC_ERR_WORKSPACE: return "SCC_ERR_WORKSPACE: workspace missing, misaligned or too small";
        case SCC_ERR_LAUNCH: return "SCC_ERR_LAUNCH: the HIP runtime refused the kernel launch";
        case SCC_ERR_SCRATCH:
            return "SCC_ERR_SCRATCH: the problem needs more scratch than the library's static buffer holds";
        default: return "unknown scc status";
    }
}

}  // extern "C"
