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
    constexpr int kLds = weight_lds(PT);
    static const hipError_t allowed = hipFuncSetAttribute((const void*)weight_product<T_, PT>,
                                                          hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
    if (allowed != hipSuccess) return allowed;
    weight_product<T_, PT><<<dim3((unsigned)(8 * t.chunk)), dim3(256), kLds, st>>>(x, dy, out, p, t);
    return hipGetLastError();
}

}  // namespace

// Used where the per-tile kernel fetches at least 1.4 times the planes this one does, and enough of them, and, binary32, where
// this one's matrix time is at most 1.1 times the other's.  The pass alone, us, per-tile kernel against this one: 128 x 128 -> 512 on
// 32x32, cg 2, co 0.33: f32 148 -> 134, bf16 66 -> 45; 37 x 336 -> 330 on 20x41, cg 1: f32 150 -> 97, bf16 74 -> 34; 64 x 2048 -> 2048 on 7x7, cg 2: f32
// 153 -> 140, bf16 78 -> 54; 22 fp32 layers below 1.1 gain 1.04 to 2.4 times, nine from 1.27 on lose 1.1 to 1.5 times (150 x 288 -> 429 on
// 16x16, cg 2: 89 -> 106).  Too few fetches: 128 x 256 -> 256 on 16x16, cg 1 (101e6): f32 53 -> 54, bf16 23 -> 23.
bool backward_weight_shared_preferred(const Problem& p, int es)
{
    if (!weight_eligible(p, es)) return false;
    int pt;
    const WeightTiling t = make_weight_tiling(p, es, &pt);
    if (t.KS == 0) return false;
    const WeightCost c = weight_cost(p, es, t, pt, false);
    return c.there >= 105e6 && c.there >= 1.4 * c.here && (es == 2 || c.matrix <= 1.1);
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
    if (t.KS == 0) return hipErrorInvalidValue;
    const hipError_t e = pt == 2   ? launch_tile<T_, 2>(x, dy, workspace, p, t, st)
                         : pt == 3 ? launch_tile<T_, 3>(x, dy, workspace, p, t, st)
                                   : launch_tile<T_, 4>(x, dy, workspace, p, t, st);
    if (e != hipSuccess) return e;
    return launch_weight_reduce(workspace, dw, p.Cout * p.L, t.KS, st);
}

template hipError_t launch_backward_weight_shared<float>(const float*, const float*, float*, float*, const Problem&, hipStream_t);
template hipError_t launch_backward_weight_shared<bf16_t>(const bf16_t*, const bf16_t*, float*, float*, const Problem&, hipStream_t);

}  // namespace scc
