// Forward and grad-input as a product with packed weights (see scc_packed_kernel.h): the packing kernel and the launchers.
#include "scc_packed_kernel.h"

namespace scc {

using namespace packed;

namespace {

// One wavefront per (row group, K group, tile).
template <typename T_, bool FWD>
__global__ __launch_bounds__(256) void pack_weights(const T_* __restrict__ w, char* __restrict__ ws, Problem P, Packed T)
{
    const int nkg = T.nround * T.KG;
    const int unit = (int)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (unit >= T.NG * nkg * kTiles) return;
    const int tile = unit % kTiles, kg = unit / kTiles % nkg, ng = unit / kTiles / nkg;
    const int lane = threadIdx.x & 63, f = lane & 31, h = lane >> 5;
    int first, len;
    walk_of<FWD>(P, T.b, T.rows, ng, first, len);

    const int row = (ng * kTiles + tile) * 32 + f;
    int k_row = -1, s_row = 0;
    if (FWD && row < T.rows) {
        k_row = filter_of(T.b, row / T.b.F, row % T.b.F, P.Cout);
        s_row = T.b.g * (row / T.b.F);
    }
    // Indexes first, then 8 loads without a condition, then the masks: a load behind a condition each is a branch and a wait each.
    // Grad-input walks on from the lane's first position instead of dividing for every one.
    float v[8];
    bool any = false;
    uint32_t at[8], in8 = 0;
    const int pos0 = 16 * kg + 8 * h;
    int mm = FWD ? 0 : pos0 / T.b.F, i = FWD ? 0 : pos0 - mm * T.b.F, m = 0, r = 0;
    if (!FWD) {
        m = (first + mm) % T.b.P;
        m += m < 0 ? T.b.P : 0;
        r = (int)(((uint32_t)m * (uint32_t)T.b.inv) % (uint32_t)T.b.P);
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int pos = pos0 + e;
        int k = k_row, s = s_row, c = row;
        if (FWD) {
            c = first + pos;                       // first < Cin and pos < Cin where it counts
            c -= c >= P.Cin ? P.Cin : 0;
        } else {
            k = r + T.b.P * i;
            k = k < P.Cout ? k : -1;
            s = T.b.g * m;
            ++i;                                   // the next filter of window m, or the first of the next window
            const bool next = i == T.b.F;
            i = next ? 0 : i;
            int rn = r + T.b.inv, mn = m + 1;
            rn -= rn >= T.b.P ? T.b.P : 0;
            mn -= mn >= T.b.P ? T.b.P : 0;
            r = next ? rn : r;
            m = next ? mn : m;
        }
        int j = c - s;
        j += j < 0 ? P.Cin : 0;
        const bool in = (pos < len) & (row < T.rows) & (k >= 0) & (j < P.L);
        const uint32_t idx = (uint32_t)k * (uint32_t)P.L + (uint32_t)j;
        at[e] = in ? idx : 0u;
        in8 |= in ? 1u << e : 0u;
    }
    T_ raw[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) raw[e] = w[at[e]];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = (in8 >> e) & 1u ? to_f32(raw[e]) : 0.f;
    any = in8 != 0;
    constexpr int NP = sizeof(T_) == 2 ? 1 : 3;
    char* dst = ws + T.a_at + ((size_t)((ng * nkg + kg) * kTiles + tile) * NP) * 1024 + lane * 16;
    if constexpr (NP == 3) {
        uint32_t hi[4], mid[4], lo[4];
        split3<8>([&](int e) { return v[e]; }, hi, mid, lo);
        *(u32x4*)dst = u32x4{hi[0], hi[1], hi[2], hi[3]};
        *(u32x4*)(dst + 1024) = u32x4{mid[0], mid[1], mid[2], mid[3]};
        *(u32x4*)(dst + 2048) = u32x4{lo[0], lo[1], lo[2], lo[3]};
    } else {
        uint32_t o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e)                // bf16 values widened above: their upper halves are all there is
            o[e] = (__float_as_uint(v[2 * e]) >> 16) | (__float_as_uint(v[2 * e + 1]) & 0xffff0000u);
        *(u32x4*)dst = u32x4{o[0], o[1], o[2], o[3]};
    }
    const bool some = __any(any);
    if (lane == 0) *(uint8_t*)(ws + T.act_at + (ng * kTiles + tile) * kMaxGroups + kg) = some ? 1 : 0;

    // plane offsets of this K group, written by tile 0's wavefront
    uint32_t* tab = (uint32_t*)ws + (size_t)ng * T.tab_group;
    if (tile == 0 && lane < 16) {
        const int pos = 16 * kg + lane;
        int plane = 0;
        if (pos < len) {
            if (FWD) {
                plane = first + pos;
                plane -= plane >= P.Cin ? P.Cin : 0;
            } else {
                const int mm = pos / T.b.F;
                int m = (first + mm) % T.b.P;
                m += m < 0 ? T.b.P : 0;
                const int k = filter_of(T.b, m, pos - mm * T.b.F, P.Cout);
                plane = k < 0 ? 0 : k;
            }
        }
        tab[pos] = (uint32_t)plane * (uint32_t)P.HW * (uint32_t)sizeof(T_);
    }
}

template <typename T_, int CT, bool FWD>
__global__ __launch_bounds__(256, 2) void packed_product(const T_* __restrict__ src, const char* __restrict__ ws,
                                                         T_* __restrict__ out, Problem P, Packed T)
{
    extern __shared__ __attribute__((aligned(16))) char lds_p[];
    packed_body<T_, CT, FWD>(src, ws, out, P, T, (int)blockIdx.x, lds_p);
}

template <typename T_, bool FWD>
void launch_pack(const T_* w, char* ws, const Problem& p, const Packed& t, hipStream_t st)
{
    const int units = t.NG * t.nround * t.KG * kTiles;
    pack_weights<T_, FWD><<<dim3((unsigned)((units + 3) / 4)), dim3(256), 0, st>>>(w, ws, p, t);
}

template <typename T_, int CT, bool FWD>
hipError_t launch_variant(const T_* src, const T_* w, T_* out, char* ws, const Problem& p, hipStream_t st)
{
    const Packed t = make_packed<FWD>(p, (int)sizeof(T_), CT);
    const int lds = lds_bytes((int)sizeof(T_), CT) + t.nround * 16 * t.KG * 4;
    static const hipError_t allowed = hipFuncSetAttribute((const void*)packed_product<T_, CT, FWD>,
                                                          hipFuncAttributeMaxDynamicSharedMemorySize,
                                                          lds_bytes((int)sizeof(T_), CT) + kMaxGroups * 16 * 4);
    if (allowed != hipSuccess) return allowed;
    launch_pack<T_, FWD>(w, ws, p, t, st);
    packed_product<T_, CT, FWD><<<dim3((unsigned)(8 * t.deal.chunk)), dim3(256), lds, st>>>(src, ws, out, p, t);
    return hipGetLastError();
}

}  // namespace

template <bool FWD>
size_t packed_workspace(const Problem& p, int es)
{
    const int ct = choose<FWD>(p, es);
    return ct ? make_packed<FWD>(p, es, ct).bytes : 0;
}

template <typename T_, bool FWD>
hipError_t launch_packed(const T_* src, const T_* w, T_* out, void* workspace, const Problem& p, hipStream_t st)
{
    switch (choose<FWD>(p, (int)sizeof(T_))) {
        case 4: return launch_variant<T_, 4, FWD>(src, w, out, (char*)workspace, p, st);
        case 2: return launch_variant<T_, 2, FWD>(src, w, out, (char*)workspace, p, st);
        default: return hipErrorInvalidValue;
    }
}

// the packing launch alone, for a launch that runs packed_body with tiles of 32*ct columns beside something else
template <typename T_, bool FWD>
hipError_t pack_only(const T_* w, void* workspace, const Problem& p, int ct, hipStream_t st)
{
    launch_pack<T_, FWD>(w, (char*)workspace, p, make_packed<FWD>(p, (int)sizeof(T_), ct), st);
    return hipGetLastError();
}

template hipError_t pack_only<float, false>(const float*, void*, const Problem&, int, hipStream_t);
template hipError_t pack_only<bf16_t, false>(const bf16_t*, void*, const Problem&, int, hipStream_t);
template size_t packed_workspace<true>(const Problem&, int);
template size_t packed_workspace<false>(const Problem&, int);
template hipError_t launch_packed<float, true>(const float*, const float*, float*, void*, const Problem&, hipStream_t);
template hipError_t launch_packed<float, false>(const float*, const float*, float*, void*, const Problem&, hipStream_t);
template hipError_t launch_packed<bf16_t, true>(const bf16_t*, const bf16_t*, bf16_t*, void*, const Problem&, hipStream_t);
template hipError_t launch_packed<bf16_t, false>(const bf16_t*, const bf16_t*, bf16_t*, void*, const Problem&, hipStream_t);

}  // namespace scc
