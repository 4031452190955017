// Gradients of the depthwise 3x3 stage (Eq. 2 of the paper) that precedes the SCC in a DW + SCC block:
//
//   z[n,a,m,q]  = sum_{i,j<3} kdw[a,i,j] * x[n,a, s*m+i-1, s*q+j-1]          (forward, zero outside the map)
//   dx[n,a,r,c] = sum over (i,j,m,q) with s*m+i-1 = r, s*q+j-1 = c of kdw[a,i,j] * dz[n,a,m,q]
//   dk[a,i,j]   = sum_{n,m,q} dz[n,a,m,q] * x[n,a, s*m+i-1, s*q+j-1]
//
// (the paper trains DW + SCC blocks end to end and gives no formula for these; they are the derivatives of Eq. 2).
// At stride 1 the grad-input is the stage itself applied to dz with every filter turned by 180 degrees, and runs on
// the forward's kernels; other strides gather per input pixel.  The filter gradient is nine dot products per
// channel over all samples and pixels: workgroups take (channel, slice of the samples), every thread keeps nine
// sums, a workgroup adds its threads' sums through LDS in a fixed order and writes one partial per slice, and a
// second kernel adds the slices in order: no atomics, bitwise reproducible.
#include "scc_common.h"
#include "scc_dw_bwd_kernel.h"

#include <type_traits>

namespace scc {

namespace {

using dw::kDkThreads;

template <typename T_>
__global__ __launch_bounds__(256) void depthwise3x3_backward_input_gather(const T_* __restrict__ dz,
                                                                          const T_* __restrict__ kdw,
                                                                          T_* __restrict__ dx, int C, DwGeom G,
                                                                          long long items)
{
    dw::input_gather_body<T_>(dz, kdw, dx, C, G, items, blockIdx.x, gridDim.x);
}

template <typename T_>
__global__ __launch_bounds__(256) void depthwise3x3_backward_input_s2(const T_* __restrict__ dz, const T_* __restrict__ kdw,
                                                                      T_* __restrict__ dx, int C, DwGeom G, uint32_t items)
{
    dw::input_s2_body<T_, 2>(dz, kdw, dx, C, G, items, blockIdx.x, gridDim.x);
}

template <typename T_, int S, int RB>
__global__ __launch_bounds__(kDkThreads) void depthwise3x3_backward_filter_strips(const T_* __restrict__ x,
                                                                                  const T_* __restrict__ dz,
                                                                                  float* __restrict__ part, int N, int C,
                                                                                  DwGeom G, int per)
{
    dw::filter_strips_body<T_, S, RB>(x, dz, part, N, C, G, per, (int)blockIdx.x, (int)blockIdx.y);
}

// Both gradients in one launch where both run on strips: the filter's workgroups (channel fastest) are the first range of the
// grid, grad-input's the second.  Neither computation changes; small maps, whose kernels take about as long as a launch, gain
// most (13-block stack at batch 128, training step: kernels 810 -> 737 us with the sums and slices above, 11 of 13 blocks take it).
// RBX: rows of grad-input's strips; at stride 2, outputs of a row under which a thread writes.
template <typename T_, int S, int RB, int RBX>
__global__ __launch_bounds__(256) void depthwise3x3_backward_strips(const T_* __restrict__ x, const T_* __restrict__ kdw,
                                                                    const T_* __restrict__ dz, T_* __restrict__ dx,
                                                                    float* __restrict__ part, int N, int C, DwGeom G, int per,
                                                                    uint32_t nfilter, long long items)
{
    const uint32_t bid = blockIdx.x;
    if (bid < nfilter)
        dw::filter_strips_body<T_, S, RB>(x, dz, part, N, C, G, per, (int)(bid % (uint32_t)C), (int)(bid / (uint32_t)C));
    else if constexpr (S == 1)
        dw::strips_body<T_, 1, RBX>(dz, kdw, dx, C, G, items, 1, bid - nfilter, gridDim.x - nfilter);
    else
        dw::input_s2_body<T_, RBX>(dz, kdw, dx, C, G, (uint32_t)items, bid - nfilter, gridDim.x - nfilter);
}

template <typename T_>
__global__ __launch_bounds__(kDkThreads) void depthwise3x3_backward_filter_generic(const T_* __restrict__ x,
                                                                                   const T_* __restrict__ dz,
                                                                                   float* __restrict__ part, int N, int C,
                                                                                   DwGeom G, int per)
{
    dw::filter_pixels_body<T_>(x, dz, part, N, C, G, per, (int)blockIdx.x, (int)blockIdx.y);
}

template <typename T_, int RB>
__global__ __launch_bounds__(kDkThreads) void depthwise3x3_backward_filter_columns(const T_* __restrict__ x,
                                                                                   const T_* __restrict__ dz,
                                                                                   float* __restrict__ part, int N, int C,
                                                                                   DwGeom G, int per)
{
    dw::filter_columns_body<T_, RB>(x, dz, part, N, C, G, per, (int)blockIdx.x, (int)blockIdx.y);
}

template <typename T_, int S>
__global__ __launch_bounds__(kDkThreads) void depthwise3x3_backward_filter_planes(const T_* __restrict__ x,
                                                                                  const T_* __restrict__ dz,
                                                                                  float* __restrict__ part, int N, int C, int per)
{
    __shared__ float red[dw::kPlanesLds / sizeof(float)];
    dw::filter_planes_body<T_, S>(x, dz, part, N, C, per, (int)blockIdx.x, (int)blockIdx.y, red);
}

__global__ __launch_bounds__(256) void depthwise3x3_filter_reduce(const float* __restrict__ part, float* __restrict__ dk,
                                                                  int count, int slices)
{
    dw::filter_reduce_body(part, dk, count, slices, blockIdx.x);
}

template <typename T, int S>
void launch_filter_strips(const T* x, const T* dz, float* part, int N, int C, const DwGeom& g, int slices, int per,
                          hipStream_t st)
{
    const dim3 grid((unsigned)C, (unsigned)slices), block(kDkThreads);
    if (g.Ho % 4 == 0)
        depthwise3x3_backward_filter_strips<T, S, 4><<<grid, block, 0, st>>>(x, dz, part, N, C, g, per);
    else if (g.Ho % 2 == 0)
        depthwise3x3_backward_filter_strips<T, S, 2><<<grid, block, 0, st>>>(x, dz, part, N, C, g, per);
    else
        depthwise3x3_backward_filter_strips<T, S, 1><<<grid, block, 0, st>>>(x, dz, part, N, C, g, per);
}

template <typename T>
void launch_filter_columns(const T* x, const T* dz, float* part, int N, int C, const DwGeom& g, int slices, int per,
                           hipStream_t st)
{
    const dim3 grid((unsigned)C, (unsigned)slices), block(kDkThreads);
    const int rb = dw::strip_rows_of(g);
    if (rb == 4)
        depthwise3x3_backward_filter_columns<T, 4><<<grid, block, 0, st>>>(x, dz, part, N, C, g, per);
    else if (rb == 2)
        depthwise3x3_backward_filter_columns<T, 2><<<grid, block, 0, st>>>(x, dz, part, N, C, g, per);
    else
        depthwise3x3_backward_filter_columns<T, 1><<<grid, block, 0, st>>>(x, dz, part, N, C, g, per);
}

// One launch for both gradients; false where the layer does not run on strips throughout.
template <typename T, int S>
bool launch_both_strips(const T* x, const T* kdw, const T* dz, T* dx, float* part, int N, int C, const DwGeom& g, int slices,
                        int per, hipStream_t st)
{
    long long items, blocks;
    int rbx = dw::strip_rows(N, C, g, &items, &blocks);
    if (S == 2) {
        // no strips on that side.  bf16: stores of 16 bytes, and half the workgroups to go through beside the filter's, from 3072 of them on.
        // Both gradients, us, two outputs / four: 128 x 128 on 32x32 24.6 / 20.9 (4.0 TB/s), 100 x 96 on 64x64 51.6 / 41.1, 64 x 128 on 40x40
        // 23.8 / 21.7; the same or slower with fewer workgroups (128 x 256 on 16x16 15.0 / 15.4, 128 x 256 on 14x24 19.9 / 22.2), and alone
        // (128 x 128 on 32x32 9.9 / 10.3)
        rbx = sizeof(T) == 2 && (long long)N * C * g.Ho * (g.Wo / 4) >= 3072 * 256 ? 4 : 2;
        items = (long long)N * C * g.Ho * (g.Wo / rbx);
        blocks = (items + 255) / 256;
        if (blocks > (1ll << 20)) blocks = 1ll << 20;
    }
    const long long nfilter = (long long)C * slices;
    if (items >= (1ll << 31) || nfilter + blocks >= (1ll << 31)) return false;
    const int rb = dw::strip_rows_of(g);
    auto go = [&](auto r, auto q) {
        depthwise3x3_backward_strips<T, S, decltype(r)::value, decltype(q)::value>
            <<<dim3((unsigned)(nfilter + blocks)), dim3(kDkThreads), 0, st>>>(x, kdw, dz, dx, part, N, C, g, per,
                                                                              (uint32_t)nfilter, items);
    };
    auto with_rb = [&](auto r) {                              // stride 1: rbx divides rb
        constexpr int RB = decltype(r)::value;
        if constexpr (S == 2) {
            if constexpr (sizeof(T) == 2)
                if (rbx == 4) return go(r, std::integral_constant<int, 4>{});
            return go(r, std::integral_constant<int, 2>{});
        }
        if constexpr (S == 1 && RB >= 4)
            if (rbx == 4) return go(r, std::integral_constant<int, 4>{});
        if constexpr (S == 1 && RB >= 2)
            if (rbx == 2) return go(r, std::integral_constant<int, 2>{});
        if constexpr (S == 1) go(r, std::integral_constant<int, 1>{});
    };
    rb == 4 ? with_rb(std::integral_constant<int, 4>{})
    : rb == 2 ? with_rb(std::integral_constant<int, 2>{}) : with_rb(std::integral_constant<int, 1>{});
    return true;
}

}  // namespace

size_t depthwise3x3_backward_workspace(int N, int C, const DwGeom& g)
{
    const int slices = dw::filter_slices(N, C, g);
    return slices > 1 ? (size_t)slices * C * 9 * sizeof(float) : 0;
}

template <typename T>
hipError_t launch_depthwise3x3_backward(const T* x, const T* kdw, const T* dz, T* dx, float* dk, float* workspace, int N,
                                        int C, const DwGeom& g, hipStream_t st, SliceSum* later)
{
    const int slices = dw::filter_slices(N, C, g);
    const int per = (N + slices - 1) / slices;
    float* part = slices > 1 ? workspace : dk;
    const bool strips = dw::filter_on_strips(x, dz, g, per);
    bool both = false;
    if (dx && dk && strips && ((uintptr_t)dx & (4 * sizeof(T) - 1)) == 0)
        both = g.s == 1 ? launch_both_strips<T, 1>(x, kdw, dz, dx, part, N, C, g, slices, per, st)
                        : launch_both_strips<T, 2>(x, kdw, dz, dx, part, N, C, g, slices, per, st);
    if (dx && !both) {
        if (g.s == 1) {
            // the stage applied to dz (an Ho x Wo = H x W map) with the filters turned by 180 degrees
            DwGeom gz = g;
            const hipError_t e = launch_depthwise3x3(dz, kdw, dx, N, C, gz, st, true);
            if (e != hipSuccess) return e;
        } else if (dw::input_on_s2(dz, dx, N, C, g)) {
            const long long items = (long long)N * C * g.Ho * (g.Wo / 2);
            long long blocks = (items + 255) / 256;
            if (blocks > (1ll << 20)) blocks = 1ll << 20;
            depthwise3x3_backward_input_s2<T><<<dim3((unsigned)blocks), dim3(256), 0, st>>>(dz, kdw, dx, C, g, (uint32_t)items);
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        } else {
            const long long items = (long long)N * C * g.H * g.W;
            long long blocks = (items + 255) / 256;
            if (blocks > (1ll << 20)) blocks = 1ll << 20;   // the kernel strides over what is left
            depthwise3x3_backward_input_gather<T><<<dim3((unsigned)blocks), dim3(256), 0, st>>>(dz, kdw, dx, C, g, items);
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
    }
    if (dk) {
        if (both)
            ;                                                 // launched above
        else if (strips && g.s == 1)
            launch_filter_strips<T, 1>(x, dz, part, N, C, g, slices, per, st);
        else if (strips)
            launch_filter_strips<T, 2>(x, dz, part, N, C, g, slices, per, st);
        else if (dw::filter_on_planes(g)) {
            const dim3 grid((unsigned)((C + dw::kPlaneChannels - 1) / dw::kPlaneChannels), (unsigned)slices);
            if (g.s == 1)
                depthwise3x3_backward_filter_planes<T, 1><<<grid, dim3(kDkThreads), 0, st>>>(x, dz, part, N, C, per);
            else
                depthwise3x3_backward_filter_planes<T, 2><<<grid, dim3(kDkThreads), 0, st>>>(x, dz, part, N, C, per);
        } else if (dw::filter_on_columns(g, per))
            launch_filter_columns<T>(x, dz, part, N, C, g, slices, per, st);
        else
            depthwise3x3_backward_filter_generic<T><<<dim3((unsigned)C, (unsigned)slices), dim3(kDkThreads), 0, st>>>(
                x, dz, part, N, C, g, per);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        if (later) *later = {part, C * 9, slices};
        if (slices > 1 && !later) {
            depthwise3x3_filter_reduce<<<dim3((unsigned)((C * 9 + 255) / 256)), dim3(256), 0, st>>>(part, dk, C * 9, slices);
            e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
    }
    return hipSuccess;
}

template hipError_t launch_depthwise3x3_backward<float>(const float*, const float*, const float*, float*, float*, float*,
                                                        int, int, const DwGeom&, hipStream_t, SliceSum*);
template hipError_t launch_depthwise3x3_backward<bf16_t>(const bf16_t*, const bf16_t*, const bf16_t*, bf16_t*, float*,
                                                         float*, int, int, const DwGeom&, hipStream_t, SliceSum*);

}  // namespace scc
