// The backward of a DW + SCC block in two launches and a sum, for layers whose SCC gradients come from the per-tile kernels:
//
//   first    dz = SCC grad-input of (dy, w)            beside   z = the depthwise stage of (x, kdw), recomputed
//   second   dw = SCC grad-weight of (z, dy)           beside   dk and dx, the depthwise gradients of (x, dz)
//   sum      the slices of dw and dk, where either has more than one
//
// Each launch is ranges of one grid.  The stages one after the other (z; both SCC gradients; both depthwise gradients; two
// sums) are five launches of kernels that, on the small maps of a network's later blocks, take about as long as a launch and
// leave most of the chip waiting on latencies: there the matrix work of one range runs beside the memory work of the other.
// The bodies are those of the stages' own kernels and so are the results, bit for bit.
#include "scc_dw_bwd_kernel.h"
#include "scc_mfma_bwi_kernel.h"
#include "scc_mfma_bww_kernel.h"

namespace scc {

namespace {

// The depthwise gradients as two ranges of workgroups: dk (channel fastest, then slice), then dx.
enum { kInputStage, kInputS2, kInputGather };

struct DwGrads {
    int filter;        // strips: 8 * stride + rows of a strip; columns: rows of a column; planes: 32 + stride; 0: pixel by pixel
    int slices, per;   // slices of the samples, samples of a slice
    uint32_t nfilter;  // workgroups of the first range
    int input;         // kInput*
    dw::Stage stage;   // kInputStage: the stage on dz with its filters turned
    long long items;   // kInputS2, kInputGather: work items
    uint32_t blocks;   // workgroups of the second range
};

template <typename T_>
DwGrads plan_gradients(const T_* x, const T_* dz, const T_* dx, int N, int C, const DwGeom& g)
{
    DwGrads d;
    d.slices = dw::filter_slices(N, C, g);
    d.per = (N + d.slices - 1) / d.slices;
    d.filter = dw::filter_on_strips(x, dz, g, d.per) ? 8 * g.s + dw::strip_rows_of(g)
               : dw::filter_on_columns(g, d.per) ? dw::strip_rows_of(g) : 0;
    uint32_t channels = (uint32_t)C;                  // or groups of them
    if (dw::filter_on_planes(g)) {
        d.filter = 32 + g.s;
        channels = (channels + dw::kPlaneChannels - 1) / dw::kPlaneChannels;
    }
    d.nfilter = channels * (uint32_t)d.slices;
    d.stage = dw::plan_stage(dz, dx, N, C, g, true);
    d.items = 0;
    if (g.s == 1) {
        d.input = kInputStage;
        d.blocks = d.stage.blocks;
        return d;
    }
    d.input = dw::input_on_s2(dz, dx, N, C, g) ? kInputS2 : kInputGather;
    d.items = d.input == kInputS2 ? (long long)N * C * g.Ho * (g.Wo / 2) : (long long)N * C * g.H * g.W;
    const long long blocks = (d.items + 255) / 256;
    d.blocks = (uint32_t)(blocks < (1ll << 20) ? blocks : 1ll << 20);   // the bodies stride over what is left
    return d;
}

template <typename T_>
__device__ __forceinline__ void gradients_body(const T_* __restrict__ x, const T_* __restrict__ kdw, const T_* __restrict__ dz,
                                               T_* __restrict__ dx, float* __restrict__ part, int N, int C, const DwGeom& G,
                                               const DwGrads& D, uint32_t bid, float* lds)
{
    if (bid < D.nfilter) {
        if (D.filter > 32) {
            const uint32_t groups = (uint32_t)(C + dw::kPlaneChannels - 1) / dw::kPlaneChannels;
            const int group = (int)(bid % groups), part_of = (int)(bid / groups);
            if (D.filter == 32 + 1) return dw::filter_planes_body<T_, 1>(x, dz, part, N, C, D.per, group, part_of, lds);
            return dw::filter_planes_body<T_, 2>(x, dz, part, N, C, D.per, group, part_of, lds);
        }
        const int a = (int)(bid % (uint32_t)C), slice = (int)(bid / (uint32_t)C);
        switch (D.filter) {
            case 8 + 1: return dw::filter_strips_body<T_, 1, 1>(x, dz, part, N, C, G, D.per, a, slice);
            case 8 + 2: return dw::filter_strips_body<T_, 1, 2>(x, dz, part, N, C, G, D.per, a, slice);
            case 8 + 4: return dw::filter_strips_body<T_, 1, 4>(x, dz, part, N, C, G, D.per, a, slice);
            case 16 + 1: return dw::filter_strips_body<T_, 2, 1>(x, dz, part, N, C, G, D.per, a, slice);
            case 16 + 2: return dw::filter_strips_body<T_, 2, 2>(x, dz, part, N, C, G, D.per, a, slice);
            case 16 + 4: return dw::filter_strips_body<T_, 2, 4>(x, dz, part, N, C, G, D.per, a, slice);
            case 1: return dw::filter_columns_body<T_, 1>(x, dz, part, N, C, G, D.per, a, slice);
            case 2: return dw::filter_columns_body<T_, 2>(x, dz, part, N, C, G, D.per, a, slice);
            case 4: return dw::filter_columns_body<T_, 4>(x, dz, part, N, C, G, D.per, a, slice);
            default: return dw::filter_pixels_body<T_>(x, dz, part, N, C, G, D.per, a, slice);
        }
    }
    bid -= D.nfilter;
    if (D.input == kInputStage)
        dw::stage_body<T_>(dz, kdw, dx, C, G, D.stage, bid);
    else if (D.input == kInputS2)
        dw::input_s2_body<T_, 2>(dz, kdw, dx, C, G, (uint32_t)D.items, bid, D.blocks);
    else
        dw::input_gather_body<T_>(dz, kdw, dx, C, G, D.items, bid, D.blocks);
}

// Bounds of the registers as in scc_mfma_bwi.hip.
template <typename T_, int CT, int S>
__global__ __launch_bounds__(256, CT == 4 && S == 4 ? 2 : 1) void block_backward_first(
    const T_* __restrict__ x, const T_* __restrict__ kdw, const T_* __restrict__ dy, const T_* __restrict__ w,
    T_* __restrict__ z, T_* __restrict__ dz, Problem P, bwi::BwiTiling TI, int nbwi, DwGeom G, dw::Stage D)
{
    const int bid = (int)blockIdx.x;
    if (bid < nbwi)
        bwi::backward_input_body<T_, CT, 8, S, 4>(dy, w, dz, P, TI, bid);
    else
        dw::stage_body<T_>(x, kdw, z, P.Cin, G, D, (uint32_t)(bid - nbwi));
}

template <typename T_, int NPT, bool SMALL>
__global__ __launch_bounds__(256, SMALL ? 2 : NPT == 2 && sizeof(T_) == 4 ? 1 : 3) void block_backward_second(
    const T_* __restrict__ x, const T_* __restrict__ kdw, const T_* __restrict__ dy, const T_* __restrict__ z,
    const T_* __restrict__ dz, T_* __restrict__ dx, float* __restrict__ part_k, float* __restrict__ part_w, Problem P,
    bww::BwwTiling TW, int nbww, DwGeom G, DwGrads D)
{
    extern __shared__ __attribute__((aligned(16))) float lds_dyn[];    // grad-weight's staging area, or the filter gradient's sums
    static_assert(bww::lds_bytes_of(NPT, (int)sizeof(T_)) >= dw::kPlanesLds, "the first range's LDS holds the second's");
    const int bid = (int)blockIdx.x;
    if (bid < nbww)
        bww::backward_weight_body<T_, NPT, true, SMALL>(z, dy, part_w, P, TW, bid);
    else
        gradients_body<T_>(x, kdw, dz, dx, part_k, P.N, P.Cin, G, D, (uint32_t)(bid - nbww), lds_dyn);
}

template <typename T_>
__global__ __launch_bounds__(256) void block_backward_sum(const float* __restrict__ part_w, T_* __restrict__ dw, int count_w,
                                                          int slices_w, int nw, const float* __restrict__ part_k,
                                                          T_* __restrict__ dk, int count_k, int slices_k)
{
    const int bid = (int)blockIdx.x;
    if (bid < nw)
        bww::weight_reduce_body(part_w, dw, count_w, slices_w, bid);
    else
        dw::filter_reduce_body(part_k, dk, count_k, slices_k, (uint32_t)(bid - nw));
}

template <typename T_, int NPT, bool SMALL = false>
hipError_t launch_second(const T_* x, const T_* kdw, const T_* dy, const T_* z, const T_* dz, T_* dx, float* part_k,
                         float* part_w, const Problem& p, const bww::BwwTiling& tw, const DwGeom& g, const DwGrads& d,
                         hipStream_t st)
{
    constexpr size_t kLds = bww::lds_bytes_of(NPT, (int)sizeof(T_));
    if (kLds > 48 * 1024) {
        // more than 64 KiB of LDS per workgroup has to be allowed once
        static const hipError_t allowed = hipFuncSetAttribute((const void*)block_backward_second<T_, NPT, SMALL>,
                                                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLds);
        if (allowed != hipSuccess) return allowed;
    }
    const int nbww = 8 * tw.chunk;
    block_backward_second<T_, NPT, SMALL><<<dim3((unsigned)nbww + d.nfilter + d.blocks), dim3(256), kLds, st>>>(
        x, kdw, dy, z, dz, dx, part_k, part_w, p, tw, nbww, g, d);
    return hipGetLastError();
}

}  // namespace

// Layers that gain: those small enough that launches and latencies count.  The depthwise ranges share the matrix kernels' registers and
// LDS and so run with fewer wavefronts than in kernels of their own, which larger maps feel, and the matrix ranges wait for one another's
// workgroups, which long binary32 contractions feel.  One stage after the other (sums in one launch) / paired over 3415 drawn layers, geometric mean
// and least, by the depthwise range: stride 2 on even maps and 2x2 maps, taken up to 2^23 values of x and z (rows of 4 pixels; 2^22 others) f32 1.12
// (0.87), bf16 1.17 (0.94); rows of 4 at stride 1, f32, taken up to 150e6 multiply-adds and 2^22 values 1.09 (0.86), on one group of 4 pixels per row
// with more up to 3 x 2^20 values 1.02 (0.93; 128 x 512 -> 512 on 4x4 1.03), left 0.96; bf16, up to 2^23
// values, 1.11 (0.82); columns, f32, up to 250e6 and 2^21 1.12 (0.79), left 0.94; bf16, up to 3 x 2^20, 1.21 (0.89), left 1.00; the gather of odd
// maps, f32, up to 15e6 and 2^20 1.18 (0.84), left 0.92; bf16, up to 2^21, 1.21 (1.00).
template <typename T_>
bool block_backward_applicable(const Problem& p, const DwGeom& g)
{
    const long long values = (long long)p.Cin * p.N * ((long long)g.H * g.W + p.HW);
    const double products = (double)p.NQ * p.Cout * p.L;
    const bool wide = sizeof(T_) == 4, fours = g.Wo % 4 == 0;
    const bool sized = (g.s == 1 || g.s == 2) && g.H == g.s * g.Ho && g.W == g.s * g.Wo;
    long long most;
    if (sized && (dw::filter_on_planes(g) || (g.s == 2 && g.Wo % 2 == 0)))
        most = fours ? 1ll << 23 : 1ll << 22;
    else if (sized && fours)
        most = !wide ? 1ll << 23 : products <= 150e6 ? 1ll << 22 : g.Wo == 4 ? 3ll << 20 : 0;
    else if (g.s == 1)
        most = !wide ? 3ll << 20 : products <= 250e6 ? 1ll << 21 : 0;
    else
        most = !wide ? 1ll << 21 : products <= 15e6 ? 1ll << 20 : 0;
    return values <= most && backward_merged_applicable<T_>(p);
}

template <typename T_>
hipError_t launch_block_backward(const T_* x, const T_* kdw, const T_* w, const T_* dy, T_* dx, float* dk, float* dw, T_* z,
                                 T_* dz, float* part_w, float* part_k, SliceSum* later_w, SliceSum* later_k, const Problem& p,
                                 const DwGeom& g, hipStream_t st)
{
    hipError_t e = hipErrorInvalidValue;
    const dw::Stage stage = dw::plan_stage(x, (const T_*)z, p.N, p.Cin, g, false);
    bwi::select_backward_input<T_>(p, [&](auto ct, auto s, auto wpb, const bwi::BwiTiling& ti, long long nbwi) {
        if constexpr (decltype(wpb)::value == 4) {
            block_backward_first<T_, decltype(ct)::value, decltype(s)::value>
                <<<dim3((unsigned)nbwi + stage.blocks), dim3(256), 0, st>>>(x, kdw, dy, w, z, dz, p, ti, (int)nbwi, g, stage);
            e = hipGetLastError();
        }
    });
    if (e != hipSuccess) return e;
    const bww::BwwTiling tw = bww::make_tiling(p, true);
    const DwGrads d = plan_gradients(x, (const T_*)dz, (const T_*)dx, p.N, p.Cin, g);
    if (tw.KS == 1) part_w = dw;
    if (d.slices == 1) part_k = dk;
    *later_w = {part_w, p.Cout * p.L, tw.KS};
    *later_k = {part_k, p.Cin * 9, d.slices};
    if (sizeof(T_) == 4 && p.NQ < 256)
        e = launch_second<T_, 1, sizeof(T_) == 4>(x, kdw, dy, z, dz, dx, part_k, part_w, p, tw, g, d, st);
    else if (tw.NPT == 1)
        e = launch_second<T_, 1>(x, kdw, dy, z, dz, dx, part_k, part_w, p, tw, g, d, st);
    else if (tw.NPT == 2)
        e = launch_second<T_, 2>(x, kdw, dy, z, dz, dx, part_k, part_w, p, tw, g, d, st);
    else
        e = launch_second<T_, 3>(x, kdw, dy, z, dz, dx, part_k, part_w, p, tw, g, d, st);
    return e;
}

template <typename T_>
hipError_t launch_gradient_sums(const SliceSum& w, T_* dw, const SliceSum& k, T_* dk, hipStream_t st)
{
    const bool done_w = w.slices == 1 && (const void*)w.part == (const void*)dw, done_k = k.slices == 1 && (const void*)k.part == (const void*)dk;
    const int nw = done_w ? 0 : (w.count + 63) / 64, nk = done_k ? 0 : (k.count + 255) / 256;
    if (nw + nk == 0) return hipSuccess;
    block_backward_sum<T_><<<dim3((unsigned)(nw + nk)), dim3(256), 0, st>>>(w.part, dw, w.count, w.slices, nw, k.part, dk, k.count,
                                                                          k.slices);
    return hipGetLastError();
}

template bool block_backward_applicable<float>(const Problem&, const DwGeom&);
template bool block_backward_applicable<bf16_t>(const Problem&, const DwGeom&);
template hipError_t launch_block_backward<float>(const float*, const float*, const float*, const float*, float*, float*, float*,
                                                 float*, float*, float*, float*, SliceSum*, SliceSum*, const Problem&, const DwGeom&,
                                                 hipStream_t);
template hipError_t launch_block_backward<bf16_t>(const bf16_t*, const bf16_t*, const bf16_t*, const bf16_t*, bf16_t*, float*,
                                                  float*, bf16_t*, bf16_t*, float*, float*, SliceSum*, SliceSum*, const Problem&,
                                                  const DwGeom&, hipStream_t);
template hipError_t launch_gradient_sums<float>(const SliceSum&, float*, const SliceSum&, float*, hipStream_t);
template hipError_t launch_gradient_sums<bf16_t>(const SliceSum&, bf16_t*, const SliceSum&, bf16_t*, hipStream_t);

}  // namespace scc
