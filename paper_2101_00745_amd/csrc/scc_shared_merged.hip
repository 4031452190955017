// Both gradients of the layers whose tiles share their planes, in ONE launch behind the packing of the weights: the workgroups
// of the shared grad-weight (scc_shared_bww_kernel.h) and those of the packed grad-input (scc_packed_kernel.h) are two ranges
// of one grid.  Nothing about either computation changes (dw sums other slices than scc_backward_weight does).  Grad-weight
// comes first, with one (bf16) or two (binary32) workgroups per CU that stay for the whole launch; grad-input's pass through
// what is left of the CUs, so that one range's matrix instructions run beside the other's loads and stores, and both read the
// same eighth of the columns on an XCD, where part of dy is still on the chip for the second of them.
// us, the per-tile kernels' merged launch -> this one: 128 x 128 -> 512, 32x32, cg 2, co 0.33: f32 251 -> 214, bf16 118 -> 63; 128 x 256 -> 256,
// 16x16, cg 1: f32 78 -> 75, bf16 35 -> 31; 37 x 336 -> 330, 20x41, cg 1: f32 179 -> 130, bf16 88 -> 47; 64 x 2048 -> 2048, 7x7, cg 2: f32 262 -> 213,
// bf16 132 -> 95.
#include "scc_packed_kernel.h"
#include "scc_shared_bww_kernel.h"

namespace scc {

namespace {

template <typename T_, int CT, int PT>
__global__ __launch_bounds__(256, 3) void backward_shared(const T_* __restrict__ x, const T_* __restrict__ dy,
                                                          const char* __restrict__ packed_w, T_* __restrict__ dx,
                                                          float* __restrict__ part, Problem P, packed::Packed TI,
                                                          shared_bww::WeightTiling TW, int nweight)
{
    extern __shared__ __attribute__((aligned(16))) char lds_b[];
    const int bid = (int)blockIdx.x;
    if (bid < nweight)
        shared_bww::weight_body<T_, PT>(x, dy, part, P, TW, bid, lds_b);
    else
        packed::packed_body<T_, CT, false, false>(dy, packed_w, dx, P, TI, bid - nweight, lds_b);
}

template <typename T_, int CT, int PT>
hipError_t launch_variant(const T_* x, const T_* dy, const char* packed_w, T_* dx, float* part, const Problem& p,
                          const packed::Packed& ti, const shared_bww::WeightTiling& tw, hipStream_t st)
{
    constexpr int kW = shared_bww::weight_lds(PT), kI = packed::lds_bytes((int)sizeof(T_), CT);
    constexpr int kMost = kI + packed::kMaxGroups * 16 * 4 > kW ? kI + packed::kMaxGroups * 16 * 4 : kW;
    static const hipError_t allowed = hipFuncSetAttribute((const void*)backward_shared<T_, CT, PT>,
                                                          hipFuncAttributeMaxDynamicSharedMemorySize, kMost);
    if (allowed != hipSuccess) return allowed;
    const int need = kI + ti.nround * 16 * ti.KG * 4, nweight = 8 * tw.chunk;
    backward_shared<T_, CT, PT><<<dim3((unsigned)(nweight + 8 * ti.deal.chunk)), dim3(256), need > kW ? need : kW, st>>>(
        x, dy, packed_w, dx, part, p, ti, tw, nweight);
    return hipGetLastError();
}

size_t partial_bytes(const Problem& p, const shared_bww::WeightTiling& t)
{
    return ((size_t)t.KS * p.Cout * p.L * sizeof(float) + 255) / 256 * 256;
}

}  // namespace

// Taken where sharing saves enough plane fetches over the per-tile kernels of both passes (grad-weight's and grad-input's
// together) and, binary32, where grad-weight's matrix time is at most 1.1 times theirs.  Against their merged launch: bf16, of 110
// layers the 99 above the lines run 0.88 to 2.9 times as fast, median 1.3, the 11 below 0.76 to 1.36, median 1.0 (uneven layers, on which
// the per-tile kernels lose more, have a line of their own); fp32, 34 above 0.98 to 1.7, median 1.16, nine below 0.76 (53 x 960 ->
// 1437 on 9x6, cg 8: 48 -> 64 us) to 1.19, median 1.0, and with longer matrix times down to 0.8 (186 x 416 -> 208 on 14x14, cg 2: 101 -> 116).
size_t backward_shared_workspace(const Problem& p, int es)
{
    const int ct = packed::tile_width<false>(p, es);
    if (ct == 0 || !shared_bww::weight_eligible(p, es)) return 0;
    const Band b = make_band(p);
    int pt;
    const shared_bww::WeightTiling t = shared_bww::make_weight_tiling(p, es, &pt, true);
    if (t.KS == 0) return 0;
    double again;
    const shared_bww::WeightCost c = shared_bww::weight_cost(p, es, t, pt, true);
    if (es == 4 && c.matrix > 1.1) return 0;
    double saved = c.there - c.here;
    saved += packed::fetches_without_sharing<false>(p, b, &again);
    for (int c0 = 0; c0 < p.Cin; c0 += 128) {
        int first, len;
        packed::walk_of<false>(p, b, p.Cin, c0 / 128, first, len);
        saved -= (double)len * p.NQ;
    }
    if (saved < (es == 4 ? 80e6 : packed::uneven(p, b) ? 45e6 : 65e6)) return 0;
    return partial_bytes(p, t) + packed::make_packed<false>(p, es, ct).bytes;
}

template <typename T_>
hipError_t launch_backward_shared(const T_* x, const T_* dy, const T_* w, T_* dx, float* dw, void* workspace,
                                  const Problem& p, hipStream_t st, SliceSum* later)
{
    constexpr int es = (int)sizeof(T_);
    int pt;
    const shared_bww::WeightTiling tw = shared_bww::make_weight_tiling(p, es, &pt, true);
    const int ct = packed::tile_width<false>(p, es);
    if (ct == 0 || tw.KS == 0) return hipErrorInvalidValue;
    packed::Packed ti = packed::make_packed<false>(p, es, ct);
    ti.deal = in_eighths(ti.deal);
    float* part = (float*)workspace;
    char* packed_w = (char*)workspace + partial_bytes(p, tw);
    hipError_t e = pack_only<T_, false>(w, packed_w, p, ct, st);
    if (e != hipSuccess) return e;
    auto with_ct = [&](auto c) {
        constexpr int CT = decltype(c)::value;
        return pt == 2   ? launch_variant<T_, CT, 2>(x, dy, packed_w, dx, part, p, ti, tw, st)
               : pt == 3 ? launch_variant<T_, CT, 3>(x, dy, packed_w, dx, part, p, ti, tw, st)
                         : launch_variant<T_, CT, 4>(x, dy, packed_w, dx, part, p, ti, tw, st);
    };
    e = ct == 4 ? with_ct(std::integral_constant<int, 4>{}) : with_ct(std::integral_constant<int, 2>{});
    if (later) *later = {part, p.Cout * p.L, tw.KS > 1 ? tw.KS : 1};
    if (e != hipSuccess || later) return e;
    return launch_weight_reduce(part, dw, p.Cout * p.L, tw.KS, st);
}

template hipError_t launch_backward_shared<float>(const float*, const float*, const float*, float*, float*, void*,
                                                  const Problem&, hipStream_t, SliceSum*);
template hipError_t launch_backward_shared<bf16_t>(const bf16_t*, const bf16_t*, const bf16_t*, bf16_t*, float*, void*,
                                                   const Problem&, hipStream_t, SliceSum*);

}  // namespace scc
