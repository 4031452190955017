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
// this one's matrix time is not longer.  The pass alone, us, per-tile kernel against this one: 128 x 128 -> 512 on 32x32, cg 2,
// co 0.33: f32 160 -> 130, bf16 66 -> 40; 40 x 272 -> 270 on 28x29, cg 1: f32 114 -> 74, bf16 56 -> 29; 253 x 112 -> 56 on 28x28, cg 1, co 0.75:
// f32 84 -> 74.  Not taken: 150 x 288 -> 429 on 16x16, cg 2: f32 89 -> 100 (1.33 times the matrix time); 128 x 256 -> 256 on 16x16, cg 1
// (101e6 fetches): f32 53 -> 54, bf16 23 -> 23; 882 x 256 -> 128, cg 4, co 0 (0.75 times the fetches): f32 70 -> 81, bf16 43 -> 43.
bool backward_weight_shared_preferred(const Problem& p, int es)
{
    if (!weight_eligible(p, es) || backward_weight_shared_workspace(p, es) > (size_t)SCC_STATIC_SCRATCH_BYTES) return false;
    const WeightCost c = weight_cost(p, es);
    return c.there >= 105e6 && c.there >= 1.4 * c.here && (es == 2 || c.matrix <= 1.15);
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
