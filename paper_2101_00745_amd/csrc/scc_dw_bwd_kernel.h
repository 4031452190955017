// Bodies of the depthwise stage's gradients (formulas in scc_dw_bwd.hip), for its own kernels and for the ranges of a block's
// backward (scc_block_bwd.hip).
#pragma once
#include "scc_common.h"
#include "scc_dw_strip.h"

namespace scc {

namespace dw {

// ---- grad-input, any stride: one thread per input pixel pulls from the outputs whose taps reach it ---------------
template <typename T_>
__device__ __forceinline__ void input_gather_body(const T_* __restrict__ dz, const T_* __restrict__ kdw, T_* __restrict__ dx, int C,
                                                  const DwGeom& G, long long items, uint32_t bid, uint32_t blocks)
{
    const long long HWo = (long long)G.Ho * G.Wo;
    for (long long e = (long long)bid * 256 + threadIdx.x; e < items; e += (long long)blocks * 256) {
        const int c = (int)(e % G.W);
        long long t = e / G.W;
        const int r = (int)(t % G.H);
        t /= G.H;                                  // t = n*C + a
        const int a = (int)(t % C);
        const T_* go = dz + t * HWo;
        float out = 0.f;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const int rr = r + 1 - i;              // = s*m
            if (rr < 0 || rr % G.s != 0 || rr / G.s >= G.Ho) continue;
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const int cc = c + 1 - j;          // = s*q
                if (cc < 0 || cc % G.s != 0 || cc / G.s >= G.Wo) continue;
                out += to_f32(kdw[a * 9 + i * 3 + j]) * to_f32(go[(long long)(rr / G.s) * G.Wo + cc / G.s]);
            }
        }
        dx[e] = from_f32<T_>(out);
    }
}

// ---- grad-input at stride 2 on even maps (H = 2*Ho, W = 2*Wo, Q dividing Wo, tensors aligned to 4 values): the taps
// that reach input pixel (r, c) are fixed by the parities of r and c, so a thread writes the 2 x 2Q input pixels
// under Q neighbouring outputs (m, q0) ... (m, q0+Q-1) from the 2 x (Q+1) outputs around them:
//   dx[2m  ][2q  ] = k11*g[m][q]                      dx[2m  ][2q+1] = k10*g[m][q+1] + k12*g[m][q]
//   dx[2m+1][2q  ] = k01*g[m+1][q] + k21*g[m][q]      dx[2m+1][2q+1] = k00*g[m+1][q+1] + k02*g[m+1][q] + k20*g[m][q+1] + k22*g[m][q]
template <typename T_, int Q>
__device__ __forceinline__ void input_s2_body(const T_* __restrict__ dz, const T_* __restrict__ kdw, T_* __restrict__ dx, int C,
                                              const DwGeom& G, uint32_t items, uint32_t bid, uint32_t blocks)
{
    typedef T_ ovec __attribute__((ext_vector_type(2 * Q), aligned(4 * sizeof(T_))));
    typedef T_ gvec __attribute__((ext_vector_type(Q)));
    const uint32_t WQ = G.Wo / Q;
    const size_t HWi = (size_t)G.H * G.W, HWo = (size_t)G.Ho * G.Wo;
    for (uint32_t e = bid * 256u + threadIdx.x; e < items; e += blocks * 256u) {
        const int q0 = (int)(e % WQ) * Q;
        uint32_t t = e / WQ;
        const int m = (int)(t % (uint32_t)G.Ho);
        t /= (uint32_t)G.Ho;                        // t = n*C + a
        const int a = (int)(t % (uint32_t)C);
        float k[9];
        load_taps(kdw, a, false, k);
        const T_* g0 = dz + t * HWo + (size_t)m * G.Wo + q0;
        const bool down = m + 1 < G.Ho, right = q0 + Q < G.Wo;
        const T_* g1 = down ? g0 + G.Wo : g0;
        const gvec a01 = *(const gvec*)g0, b01 = *(const gvec*)g1;
        // under two outputs behind a branch: without it 128 x 256 on 14x24, bf16, both gradients, 20.9 us against 19.9
        const float araw = Q > 2 ? to_f32(g0[right ? Q : 0]) : right ? to_f32(g0[Q]) : 0.f, braw = to_f32(g1[right ? Q : 0]);
        float ga[Q + 1], gb[Q + 1];
#pragma unroll
        for (int j = 0; j < Q; ++j) {
            ga[j] = to_f32((T_)a01[j]);
            gb[j] = down ? to_f32((T_)b01[j]) : 0.f;
        }
        ga[Q] = right ? araw : 0.f;
        gb[Q] = (down && right) ? braw : 0.f;
        ovec r0, r1;
#pragma unroll
        for (int j = 0; j < Q; ++j) {
            // spelled out, as in columns_body: three kernels hold this body and their results are the same bit for bit
            r0[2 * j] = from_f32<T_>(k[4] * ga[j]);
            r0[2 * j + 1] = from_f32<T_>(__builtin_fmaf(k[5], ga[j], k[3] * ga[j + 1]));
            r1[2 * j] = from_f32<T_>(__builtin_fmaf(k[7], ga[j], k[1] * gb[j]));
            const float up = __builtin_fmaf(k[2], gb[j], k[0] * gb[j + 1]);
            r1[2 * j + 1] = from_f32<T_>(__builtin_fmaf(k[8], ga[j], __builtin_fmaf(k[6], ga[j + 1], up)));
        }
        T_* o = dx + t * HWi + (size_t)(2 * m) * G.W + 2 * q0;
        __builtin_nontemporal_store(r0, (ovec*)o);
        __builtin_nontemporal_store(r1, (ovec*)(o + G.W));
    }
}

// ---- grad-filter ----------------------------------------------------------------------------------------------
constexpr int kDkThreads = 256;

// the workgroup's nine sums: a tree over the lanes of each wavefront, then thread t < 9 adds the four wavefronts in order.
// (One thread per sum adding 256 values from LDS one after the other was half of the kernel on small maps.)
__device__ __forceinline__ void reduce_nine(const float (&s)[9], float* out9)
{
    __shared__ float part[kDkThreads / 64][9];
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        float v = s[t];
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d, 64);
        if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6][t] = v;
    }
    __syncthreads();
    if (threadIdx.x < 9)
        out9[threadIdx.x] = ((part[0][threadIdx.x] + part[1][threadIdx.x]) + part[2][threadIdx.x]) + part[3][threadIdx.x];
}

// On strips (stride S = 1 or 2, output rows of whole column quads, input maps of exactly S times the output size,
// RB dividing the output rows, tensors aligned to 4 values): a thread reads the strip's RB rows of dz and its
// S*(RB-1)+3 rows of x once (strip_row) and adds their products to its nine sums.
// Workgroup (a, slice) walks the strips of channel a in samples [slice*per, slice*per + per).
template <typename T_, int S, int RB>
__device__ __forceinline__ void filter_strips_body(const T_* __restrict__ x, const T_* __restrict__ dz,
                                                   float* __restrict__ part, int N, int C, const DwGeom& G, int per, int a,
                                                   int slice)
{
    typedef T_ tvec __attribute__((ext_vector_type(4)));
    constexpr int NR = S * (RB - 1) + 3;
    const int n0 = slice * per, n1 = n0 + per < N ? n0 + per : N;
    const uint32_t W4 = G.Wo / 4, SB = G.Ho / RB, spp = W4 * SB;             // strips per plane
    const uint32_t items = (uint32_t)(n1 > n0 ? n1 - n0 : 0) * spp;
    const size_t HWi = (size_t)G.H * G.W, HWo = (size_t)G.Ho * G.Wo;
    const uint32_t lane = threadIdx.x & 63;
    float s[9] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    // all lanes of a wavefront run the same number of trips (strip_row shuffles between lanes); lanes past the end
    // read strip 0 again and add nothing
    for (uint32_t e0 = 0; e0 < items; e0 += kDkThreads) {
        const uint32_t ee = e0 + threadIdx.x;
        const bool live = ee < items;
        const uint32_t e = live ? ee : 0;
        const int cw = (int)(e % W4) * 4;
        uint32_t t = e / W4;
        const int r0 = (int)(t % SB) * RB;
        const size_t plane = (size_t)(n0 + t / SB) * C + a;
        const T_* xc = x + plane * HWi + (size_t)(S * r0) * G.W + S * cw;
        const T_* gz = dz + plane * HWo + (size_t)r0 * G.Wo + cw;
        float g[RB][4];
#pragma unroll
        for (int rr = 0; rr < RB; ++rr) {
            const tvec m = *(const tvec*)(gz + rr * G.Wo);
#pragma unroll
            for (int i = 0; i < 4; ++i) g[rr][i] = live ? to_f32(m[i]) : 0.f;
        }
        const uint32_t rowmask = strip_rowmask<S, RB>(r0, G.Ho);
#pragma unroll
        for (int tr = 0; tr < NR; ++tr) {
            float v[4 * S + 2];
            strip_row<S>(xc, G.W, tr, rowmask, cw > 0, cw + 4 < G.Wo, lane == 0, lane == 63 || ee + 1 >= items, v);
#pragma unroll
            for (int rr = 0; rr < RB; ++rr) {
                const int di = tr - S * rr;      // tap row that pairs this input row with output row rr
                if (di < 0 || di > 2) continue;
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 3; ++j) s[di * 3 + j] += g[rr][i] * v[S * i + j];
            }
        }
    }
    reduce_nine(s, part + ((size_t)slice * C + a) * 9);
}

// On columns (stride 1, rows of any length, RB dividing the rows): a thread owns one column of RB rows of dz, consecutive lanes
// consecutive pixels, and the pixels left and right of its own x are its neighbours' (lane shuffle), as in columns_body: 2 + 2/RB
// loads per output where the body below takes ten (both gradients of 64 x 256 on 14x14, f32: see scc_dw_bwd.hip).
template <typename T_, int RB>
__device__ __forceinline__ void filter_columns_body(const T_* __restrict__ x, const T_* __restrict__ dz, float* __restrict__ part,
                                                    int N, int C, const DwGeom& G, int per, int a, int slice)
{
    const int n0 = slice * per, n1 = n0 + per < N ? n0 + per : N;
    const uint32_t W = (uint32_t)G.W, SB = (uint32_t)G.H / RB;
    const uint32_t items = (uint32_t)(n1 > n0 ? n1 - n0 : 0) * (W * SB);
    const size_t HW = (size_t)G.H * G.W;
    const uint32_t lane = threadIdx.x & 63;
    float s[9] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    // all lanes of a wavefront run the same number of trips (they shuffle); lanes past the end redo item 0 and add nothing
    for (uint32_t e0 = 0; e0 < items; e0 += kDkThreads) {
        const uint32_t ee = e0 + threadIdx.x;
        const bool live = ee < items;
        const uint32_t e = live ? ee : 0;
        uint32_t t = e / W;
        const int c = (int)(e - t * W);
        const uint32_t n = t / SB;
        const int r0 = (int)(t - n * SB) * RB;
        const size_t at = ((size_t)(n0 + n) * C + a) * HW + (size_t)r0 * W + c;
        const T_ *xc = x + at, *gz = dz + at;
        float g[RB];
#pragma unroll
        for (int rr = 0; rr < RB; ++rr) {
            const float v = to_f32(gz[rr * (int)W]);
            g[rr] = live ? v : 0.f;
        }
        const bool left = c > 0, right = c + 1 < (int)W;
        const bool lo = lane == 0, hi = lane == 63 || ee + 1 >= items;
#pragma unroll
        for (int tr = 0; tr < RB + 2; ++tr) {
            const int r = r0 - 1 + tr;
            const bool ok = r >= 0 && r < G.H;
            const T_* row = ok ? xc + (tr - 1) * (int)W : xc;
            const float mid = to_f32(row[0]);
            float lv = __shfl_up(mid, 1, 64), rv = __shfl_down(mid, 1, 64);
            if (lo && left) lv = to_f32(row[-1]);
            if (hi && right) rv = to_f32(row[1]);
            const float v[3] = {(ok && left) ? lv : 0.f, ok ? mid : 0.f, (ok && right) ? rv : 0.f};
#pragma unroll
            for (int rr = 0; rr < RB; ++rr) {
                const int di = tr - rr;              // tap row that pairs this row of x with row rr of dz
                if (di < 0 || di > 2) continue;
#pragma unroll
                for (int j = 0; j < 3; ++j) s[di * 3 + j] += g[rr] * v[j];
            }
        }
    }
    reduce_nine(s, part + ((size_t)slice * C + a) * 9);
}

// On planes (output maps of 2 x 2 read from maps of S times that): a lane owns one channel, whose planes are 16 (16 * S * S) bytes
// next to its neighbours'.  Lanes on samples of one channel, as in the bodies above, fetch a cache line for every 16 bytes here.
// A workgroup takes eight channels, a cache line of binary32 planes, and its 32 groups of eight lanes share the samples: there are
// C / 8 workgroups per slice, and no more than 1024 / C slices.  (64 channels per workgroup leave 16 to 32 workgroups whatever the
// batch.)  The filter gradient, us, lanes on samples / 64 channels per workgroup / 8: f32 1024 channels, batch 128 13.8 / 6.3 / 3.5, batch 1024 55 /
// 32 / 9.0 and at stride 2 76 / 142 / 24; 512 channels, batch 1024, stride 2 40 / 50 / 12; bf16 1024 channels, batch 1024 49 / 74 / 12; 64 channels,
// batch 16 7.2 / 5.1 / 5.1; 16 channels, one sample 4.6 / 2.7 / 3.0.
// kBatch samples are in flight, each with sums of its own, added as a tree behind the loop.
// `red`: kPlanesLds bytes of LDS.
constexpr int kPlaneChannels = 8, kPlaneShares = kDkThreads / kPlaneChannels;
constexpr size_t kPlanesLds = kDkThreads * 9 * sizeof(float);

inline __host__ __device__ bool filter_on_planes(const DwGeom& g)
{
    return (g.s == 1 || g.s == 2) && g.Ho == 2 && g.Wo == 2 && g.H == 2 * g.s && g.W == 2 * g.s;
}

template <typename T_, int S>
__device__ __forceinline__ void filter_planes_body(const T_* __restrict__ x, const T_* __restrict__ dz, float* __restrict__ part,
                                                   int N, int C, int per, int group, int slice, float* red)
{
    typedef T_ plane4 __attribute__((ext_vector_type(4), aligned(sizeof(T_))));
    constexpr int kBatch = S == 1 ? 8 : 4, W = 2 * S;
    const int a0 = group * kPlaneChannels, own_a = a0 + (int)(threadIdx.x % kPlaneChannels);
    const int a = own_a < C ? own_a : C - 1;           // past the end: the last one again, not stored
    const int n0 = slice * per, n1 = n0 + per < N ? n0 + per : N;
    float s[kBatch][9];
#pragma unroll
    for (int u = 0; u < kBatch; ++u)
#pragma unroll
        for (int t = 0; t < 9; ++t) s[u][t] = 0.f;
    for (int n = n0 + (int)(threadIdx.x / kPlaneChannels); n < n1; n += kPlaneShares * kBatch) {
        plane4 gv[kBatch], xv[kBatch][S * S];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int nu = n + kPlaneShares * u;
            const size_t plane = (size_t)(nu < n1 ? nu : n) * C + a;
            gv[u] = *(const plane4*)(dz + plane * 4);
#pragma unroll
            for (int q = 0; q < S * S; ++q) xv[u][q] = *(const plane4*)(x + plane * (W * W) + 4 * q);
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const bool live = n + kPlaneShares * u < n1;
            float own[9] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int o = 0; o < 4; ++o)
#pragma unroll
                for (int i = 0; i < 3; ++i)
#pragma unroll
                    for (int j = 0; j < 3; ++j) {
                        const int rr = S * (o / 2) + i - 1, cc = S * (o % 2) + j - 1;
                        if (rr < 0 || rr >= W || cc < 0 || cc >= W) continue;
                        const int e = rr * W + cc;
                        own[3 * i + j] += to_f32((T_)gv[u][o]) * to_f32((T_)xv[u][e / 4][e % 4]);
                    }
#pragma unroll
            for (int t = 0; t < 9; ++t) s[u][t] += live ? own[t] : 0.f;
        }
    }
#pragma unroll
    for (int d = 1; d < kBatch; d *= 2)
#pragma unroll
        for (int u = 0; u + d < kBatch; u += 2 * d)
#pragma unroll
            for (int t = 0; t < 9; ++t) s[u][t] += s[u + d][t];
#pragma unroll
    for (int t = 0; t < 9; ++t) red[threadIdx.x * 9 + t] = s[0][t];
    __syncthreads();
    const int count = ((a0 + kPlaneChannels < C ? a0 + kPlaneChannels : C) - a0) * 9;
    if ((int)threadIdx.x < count) {
        constexpr int kStep = 9 * kPlaneChannels;
        float sum[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < kPlaneShares; w += 4)
#pragma unroll
            for (int u = 0; u < 4; ++u) sum[u] += red[(w + u) * kStep + threadIdx.x];
        part[((size_t)slice * C + a0) * 9 + threadIdx.x] = (sum[0] + sum[1]) + (sum[2] + sum[3]);
    }
}

// Any stride and map size: a thread takes output pixels one by one.  The batch's pixels fit 32 bits (64-bit divisions in every
// lane cost more than the nine products).
template <typename T_>
__device__ __forceinline__ void filter_pixels_body(const T_* __restrict__ x, const T_* __restrict__ dz, float* __restrict__ part,
                                                   int N, int C, const DwGeom& G, int per, int a, int slice)
{
    const int n0 = slice * per, n1 = n0 + per < N ? n0 + per : N;
    const uint32_t HWo = (uint32_t)G.Ho * (uint32_t)G.Wo, Wo = (uint32_t)G.Wo;
    const size_t HWi = (size_t)G.H * G.W;
    const uint32_t items = (uint32_t)(n1 > n0 ? n1 - n0 : 0) * HWo;
    float s[9] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (uint32_t e = threadIdx.x; e < items; e += kDkThreads) {
        const uint32_t n = e / HWo, px = e - n * HWo;
        const int m = (int)(px / Wo), q = (int)(px - (uint32_t)m * Wo);
        const size_t plane = (size_t)(n0 + n) * C + a;
        const float g = to_f32(dz[plane * HWo + px]);
        const T_* xc = x + plane * HWi;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const int rr = G.s * m + i - 1;
            if (rr < 0 || rr >= G.H) continue;
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const int cc = G.s * q + j - 1;
                if (cc < 0 || cc >= G.W) continue;
                s[i * 3 + j] += g * to_f32(xc[(size_t)rr * G.W + cc]);
            }
        }
    }
    reduce_nine(s, part + ((size_t)slice * C + a) * 9);
}

// dk[e] = sum over slices of part[slice][e], in slice order
template <typename T_>
__device__ __forceinline__ void filter_reduce_body(const float* __restrict__ part, T_* __restrict__ dk, int count, int slices,
                                                   uint32_t bid)
{
    const int e = (int)bid * 256 + (int)threadIdx.x;
    if (e >= count) return;
    float s = 0.f;
    int sl = 0;
    for (; sl + 8 <= slices; sl += 8) {          // 8 loads in flight, added in order
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = part[(size_t)(sl + u) * count + e];
#pragma unroll
        for (int u = 0; u < 8; ++u) s += v[u];
    }
    for (; sl < slices; ++sl) s += part[(size_t)sl * count + e];
    dk[e] = from_f32<T_>(s);
}

// slices of the samples per channel: about 1024 workgroups of one channel in all (128 of eight on planes), at least one sample for each and,
// on strips, one strip per thread; at most 65535.  Maps of 4x4 at batch 128 have 128 strips per channel: with two slices three quarters of the
// threads had none and the slices' sums took another launch (512 channels: 10.4 + 3.9 us, 9.6 with one).
inline int filter_slices(int N, int C, const DwGeom& g)
{
    int sl = (1024 + C - 1) / C;
    if ((g.s == 1 || g.s == 2) && g.Wo % 4 == 0 && g.H == g.s * g.Ho && g.W == g.s * g.Wo) {
        const int rb = g.Ho % 4 == 0 ? 4 : g.Ho % 2 == 0 ? 2 : 1;
        const long long full = ((long long)N * (g.Wo / 4) * (g.Ho / rb) + kDkThreads - 1) / kDkThreads;
        if (sl > full) sl = (int)full;
    }
    if (sl > N) sl = N;
    if (sl > 65535) sl = 65535;
    return sl < 1 ? 1 : sl;
}

// Whether the filter gradient runs on strips (rows of a strip: strip_rows_of), `per` samples to a slice.
template <typename T_>
inline bool filter_on_strips(const T_* x, const T_* dz, const DwGeom& g, int per)
{
    return (g.s == 1 || g.s == 2) && g.Wo % 4 == 0 && g.H == g.s * g.Ho && g.W == g.s * g.Wo &&
           (((uintptr_t)x | (uintptr_t)dz) & (4 * sizeof(T_) - 1)) == 0 && (long long)per * g.Ho * (g.Wo / 4) < (1ll << 31);
}

inline int strip_rows_of(const DwGeom& g) { return g.Ho % 4 == 0 ? 4 : g.Ho % 2 == 0 ? 2 : 1; }

// Whether the filter gradient of a layer that does not run on strips (or planes) runs on columns (rows of a column: strip_rows_of),
// `per` samples to a slice, and not pixel by pixel: where a workgroup has 350 pixels, on maps of two rows and columns.  With fewer, its threads
// have a pixel or two each, and a column's rows one after another cost what the loads save; a map of one row or column has no neighbours
// to share.  Over 5252 layers of 1 to 32 rows of 1 to 30 pixels, both types, pixels / columns, geometric mean and least: the layers this takes
// 1.41 (0.92), the others 0.96 (0.61).
inline bool filter_on_columns(const DwGeom& g, int per)
{
    return g.s == 1 && g.H > 1 && g.W > 1 && (long long)per * g.H * g.W >= 350;
}

// Whether grad-input at stride 2 runs on input_s2_body.
template <typename T_>
inline bool input_on_s2(const T_* dz, const T_* dx, int N, int C, const DwGeom& g)
{
    return g.s == 2 && g.H == 2 * g.Ho && g.W == 2 * g.Wo && g.Wo % 2 == 0 &&
           (((uintptr_t)dz | (uintptr_t)dx) & (4 * sizeof(T_) - 1)) == 0 && (long long)N * C * g.Ho * (g.Wo / 2) < (1ll << 31);
}

}  // namespace dw

}  // namespace scc
