// Both gradients of one SCC layer in ONE launch, for the layers the fused backward kernel (scc_lds_bwd.hip) does
// not take: the workgroups of the grad-weight kernel (scc_mfma_bww_kernel.h) and those of the grad-input kernel
// (scc_mfma_bwi_kernel.h) are two ranges of one grid and run side by side.
//
//   dx[n,c,p] = sum over filters k covering c of w[k,(c-s_k) mod Cin] * dy[n,k,p]    (Section 4.2, input-centric)
//   dw[k,j]   = sum_{n,p} dy[n,k,p] * x[n,(s_k+j) mod Cin,p]
//
// Nothing about either computation changes: same tiles, same arithmetic, same summation order, so the results
// are bitwise those of the two separate passes (one exception: a split of the columns into only two slices is
// dropped here, see bww::make_tiling, so dw is then one summation chain instead of two).  What changes is time: one launch instead of two, no drained
// chip between them, and on layers with few columns (where each pass alone leaves most of the chip waiting on
// latencies) the two passes overlap.  The grad-weight range comes first in the grid (its partial sums still have
// to be reduced by a second kernel, so it should not finish last); both ranges are a multiple of 8 workgroups,
// which keeps workgroup index mod 8 = XCD true inside each of them.
#include "scc_mfma_bwi_kernel.h"
#include "scc_mfma_bww_kernel.h"

namespace scc {

namespace {

// Wavefronts per SIMD that a variant's registers have to leave room for.  Unbounded, the compiler keeps accumulators apart from
// the other registers and copies between the two: with the four accumulators of grad-weight's narrow tiles (NPT 1) a SIMD then
// holds two wavefronts instead of three (11 x 320 -> 1280 on 16x16, cg 2, f32: 42 us, with this bound 37.5), with three position
// tiles as well, and with a contraction shared by four wavefronts (S 4) one instead of two (64 x 512 -> 1024 on 7x7, cg 2,
// co 0.33, f32: 57 -> 47; 128 x 512 -> 512 on 4x4, cg 2, bf16: 17.6 -> 12.5).  1: as it is; no more would fit, or nothing is gained
// (882 x 256 -> 128 on 16x16, cg 4, f32: 133 us, 136 with a bound of two).
template <typename T_, int CT, int S, int NPT, bool SMALL>
constexpr int least_waves()
{
    if (SMALL) return 1;
    if (CT == 4) return S == 4 ? 2 : sizeof(T_) == 2 ? 3 : 1;
    return NPT == 2 ? 1 : 3;
}

template <typename T_, int CT, int S, int NPT, bool SMALL>
__global__ __launch_bounds__(256, (least_waves<T_, CT, S, NPT, SMALL>())) void backward_merged(
    const T_* __restrict__ x, const T_* __restrict__ dy, const T_* __restrict__ w, T_* __restrict__ dx, float* __restrict__ out,
    Problem P, bwi::BwiTiling TI, bww::BwwTiling TW, int nbww)
{
    // the dynamic LDS is the grad-weight range's staging area; the grad-input range, which a workgroup never is at
    // the same time, adds its shared tiles' partial sums in it
    extern __shared__ __attribute__((aligned(16))) float lds_dyn[];
    const int bid = (int)blockIdx.x;
    if (bid < nbww)
        bww::backward_weight_body<T_, NPT, true, SMALL>(x, dy, out, P, TW, bid);
    else
        bwi::backward_input_body<T_, CT, 8, S, 4, true>(dy, w, dx, P, TI, bid - nbww, lds_dyn);
}

template <typename T_, int CT, int S, int NPT, bool SMALL = false>
hipError_t launch_variant(const T_* x, const T_* dy, const T_* w, T_* dx, float* out, const Problem& p,
                          const bwi::BwiTiling& ti, long long nbwi, const bww::BwwTiling& tw, hipStream_t st)
{
    constexpr size_t kNeedW = bww::lds_bytes_of(NPT, (int)sizeof(T_)), kNeedI = bwi::reduce_bytes<CT, S, 4>();
    constexpr size_t kLds = kNeedW > kNeedI ? kNeedW : kNeedI;
    if (kLds > 48 * 1024) {
        // more than 64 KiB of LDS per workgroup has to be allowed once
        static const hipError_t allowed = hipFuncSetAttribute((const void*)backward_merged<T_, CT, S, NPT, SMALL>,
                                                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLds);
        if (allowed != hipSuccess) return allowed;
    }
    const long long nbww = (long long)8 * tw.chunk;
    bwi::BwiTiling beside = ti;
    beside.deal = in_eighths(ti.deal);
    backward_merged<T_, CT, S, NPT, SMALL><<<dim3((unsigned)(nbww + nbwi)), dim3(256), kLds, st>>>(x, dy, w, dx, out, p, beside,
                                                                                               tw, (int)nbww);
    return hipGetLastError();
}

}  // namespace

// Layers the merged launch takes: both passes on the matrix-core kernels, planes of at least 4 pixels, and the grad-input variant with 4 wavefronts
// per workgroup (the 8-wavefront variant is for grids the fused backward kernel takes anyway).
template <typename T_>
bool backward_merged_applicable(const Problem& p)
{
    if (!backward_input_mfma_eligible(p) || !backward_weight_mfma_eligible(p) || p.HW < 4) return false;
    bool four = false;
    bwi::select_backward_input<T_>(p, [&](auto, auto, auto wpb, const bwi::BwiTiling&, long long) {
        four = decltype(wpb)::value == 4;
    });
    return four && (long long)8 * bww::make_tiling(p, true).chunk < (1ll << 30);
}

template <typename T_>
hipError_t launch_backward_merged(const T_* x, const T_* dy, const T_* w, T_* dx, float* dw, float* workspace,
                                  const Problem& p, hipStream_t st, SliceSum* later)
{
    const bww::BwwTiling tw = bww::make_tiling(p, true);
    float* out = tw.KS > 1 ? workspace : dw;
    hipError_t e = hipErrorInvalidValue;
    bwi::select_backward_input<T_>(p, [&](auto ct, auto s, auto wpb, const bwi::BwiTiling& ti, long long nbwi) {
        constexpr int CT = decltype(ct)::value, S = decltype(s)::value, WPB = decltype(wpb)::value;
        if constexpr (WPB == 4) {
            if constexpr (sizeof(T_) == 4)
                if (p.NQ < 256) {
                    e = launch_variant<T_, CT, S, 1, true>(x, dy, w, dx, out, p, ti, nbwi, tw, st);
                    return;
                }
            if (tw.NPT == 1)
                e = launch_variant<T_, CT, S, 1>(x, dy, w, dx, out, p, ti, nbwi, tw, st);
            else if (tw.NPT == 2)
                e = launch_variant<T_, CT, S, 2>(x, dy, w, dx, out, p, ti, nbwi, tw, st);
            else
                e = launch_variant<T_, CT, S, 3>(x, dy, w, dx, out, p, ti, nbwi, tw, st);
        }
    });
    if (later) *later = {out, p.Cout * p.L, tw.KS};
    if (e != hipSuccess || tw.KS == 1 || later) return e;
    return launch_weight_reduce(workspace, dw, p.Cout * p.L, tw.KS, st);
}

template bool backward_merged_applicable<float>(const Problem&);
template bool backward_merged_applicable<bf16_t>(const Problem&);
template hipError_t launch_backward_merged<float>(const float*, const float*, const float*, float*, float*, float*,
                                                  const Problem&, hipStream_t, SliceSum*);
template hipError_t launch_backward_merged<bf16_t>(const bf16_t*, const bf16_t*, const bf16_t*, bf16_t*, float*, float*,
                                                   const Problem&, hipStream_t, SliceSum*);

}  // namespace scc
