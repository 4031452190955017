// Grad-weight with both operands shared by four filter tiles (see scc_shared_bww_kernel.h): launchers.
#include "scc_shared_bww_kernel.h"

namespace scc {

using namespace shared_bww;

namespace {

template <typename T_, int PT>
__global__ __launch_bounds__(256, 3) void weight_product(const T_* __restrict__ x, const T_* __restrict__ dy,
                                                         float* __restrict__ out, Problem P, WeightTiling T)
{
    extern __shared__ __attribute__((aligned(16))) char lds_w[];
    weight_body<T_, PT>(x, dy, out, P, T, (int)blockIdx.x, lds_w);
}

template <typename T_, int PT>
hipError_t launch_tile(const T_* x, const T_* dy, float* out, const Problem& p, const WeightTiling& t, hipStream_t st)
{
    constexpr int kLds = weight_lds((int)sizeof(T_), PT);
    static const hipError_t allowed = hipFuncSetAttribute((const void*)weight_product<T_, PT>,
                                                          hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
    if (allowed != hipSuccess) return allowed;
    weight_product<T_, PT><<<dim3((unsigned)(8 * t.chunk)), dim3(256), kLds, st>>>(x, dy, out, p, t);
    return hipGetLastError();
}

}  // namespace

// Used where the per-tile kernel fetches at least 1.4 times the planes this one does, and enough of them.  The pass alone, us,
// per-tile kernel against this one: 128 x 128 -> 512 on 32x32, cg 2, co 0.33: f32 155 -> 96, bf16 66 -> 40; 128 x 256 -> 256 on
// 16x16, cg 1: f32 51 -> 43, bf16 22 -> 23 (not taken); 30 x 640 -> 640 on 32x32, cg 4, co 0: 138 -> 72; 128 x 256 -> 256, cg 2: 31 -> 32
// (50e6 fetches, not taken); 882 x 256 -> 128, cg 4, co 0: 70 -> 77 (0.75 times the fetches, not taken).
bool backward_weight_shared_preferred(const Problem& p, int es)
{
    if (!weight_eligible(p, es) || backward_weight_shared_workspace(p, es) > (size_t)SCC_STATIC_SCRATCH_BYTES) return false;
    double there, here;
    weight_fetches(p, es, &there, &here);
    return there >= (es == 2 ? 105e6 : 90e6) && there >= 1.4 * here;
}

size_t backward_weight_shared_workspace(const Problem& p, int es)
{
    int pt;
    const WeightTiling t = make_weight_tiling(p, es, &pt);
    return (size_t)t.KS * p.Cout * p.L * sizeof(float);
}

template <typename T_>
hipError_t launch_backward_weight_shared(const T_* x, const T_* dy, float* dw, float* workspace, const Problem& p,
                                         hipStream_t st)
{
    int pt;
    const WeightTiling t = make_weight_tiling(p, (int)sizeof(T_), &pt);
    const hipError_t e = pt == 2   ? launch_tile<T_, 2>(x, dy, workspace, p, t, st)
                         : pt == 3 ? launch_tile<T_, 3>(x, dy, workspace, p, t, st)
                                   : launch_tile<T_, 4>(x, dy, workspace, p, t, st);
    if (e != hipSuccess) return e;
    return launch_weight_reduce(workspace, dw, p.Cout * p.L, t.KS, st);
}

template hipError_t launch_backward_weight_shared<float>(const float*, const float*, float*, float*, const Problem&, hipStream_t);
template hipError_t launch_backward_weight_shared<bf16_t>(const bf16_t*, const bf16_t*, float*, float*, const Problem&, hipStream_t);

}  // namespace scc
