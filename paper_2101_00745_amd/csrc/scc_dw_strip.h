// Strips of the depthwise 3x3 stage (Eq. 2 of the paper): the unit of work of the stand-alone stage, of the fused
// DW + SCC forward and of the stage's gradients.
#pragma once
#include "scc_common.h"

namespace scc {

namespace dw {

// The nine taps of channel a's filter as binary32, tap t of the result taking weight 8 - t when `flip` is set (the
// filter turned by 180 degrees).  A vector memory instruction costs the same address-processing time whatever
// its width, and the taps are a third to a half of a strip's instructions: binary32 taps are fetched with two
// 16-byte loads and one 4-byte load, bf16 taps with a 16-byte and a 2-byte one (the address is only aligned to a value, which global
// loads allow; nine 2-byte loads: grad-input of 128 x 256 on 16x16, stride 2, 6.35 us, 6.13 so).
template <typename T_>
__device__ __forceinline__ void load_taps(const T_* kdw, int a, bool flip, float (&k)[9])
{
    float raw[9];
    if constexpr (sizeof(T_) == 4) {
        typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
        const float* src = (const float*)kdw + a * 9;
        const f32x4u lo = *(const f32x4u*)src, hi = *(const f32x4u*)(src + 4);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            raw[i] = lo[i];
            raw[4 + i] = hi[i];
        }
        raw[8] = src[8];
    } else {
        typedef T_ t8u __attribute__((ext_vector_type(8), aligned(sizeof(T_))));
        const T_* src = kdw + a * 9;
        const t8u lo = *(const t8u*)src;
#pragma unroll
        for (int i = 0; i < 8; ++i) raw[i] = to_f32((T_)lo[i]);
        raw[8] = to_f32(src[8]);
    }
#pragma unroll
    for (int i = 0; i < 9; ++i) k[i] = flip ? raw[8 - i] : raw[i];
}

// Input rows of a strip: RB consecutive output rows x 4 consecutive output columns of one channel at spatial stride
// S (1 or 2) need NR = S*(RB-1)+3 input rows of 4*S+2 pixels each; pixel e of row t is input pixel
// (S*r0 - 1 + t, S*cw - 1 + e).  Each row is read once: 4*S pixels from the strip's first input column on (one or
// two 16-byte loads for binary32, one load for bf16); the pixel left of them and, for S == 1, the pixel right of them are the last
// and first pixel of what the NEIGHBOURING LANES loaded for the same row: lane l-1 must own the strip to the left and
// lane l+1 the strip to the right (same channel, same rows) whenever `left` / `right` is set and `lo` / `hi` is
// not; they are fetched with a lane shuffle (single misaligned 4-byte loads measured 40 % of the whole stage).
//   xc       input pixel (S*r0, S*cw) of the channel: centre of the strip's first output
//   W        pixels per input row
//   rowmask  bit t set: input row S*r0 - 1 + t lies inside the map (bit 1 always is)
//   left     the input column left of the strip exists; right (S == 1): the column right of it exists
//   lo, hi   the lane has no lane below / above it in the wavefront that owns the neighbouring strip: it loads
//            the edge pixel itself
// Rows and columns outside the map are read at an address inside it and replaced by zero.  Every lane of the
// wavefront must call this together (the shuffles are wavefront-wide).
template <int S, typename T_>
__device__ __forceinline__ void strip_row(const T_* xc, int W, int t, uint32_t rowmask, bool left, bool right, bool lo,
                                          bool hi, float (&v)[4 * S + 2])
{
    constexpr int kLoad = sizeof(T_) == 4 ? 4 : 4 * S;      // values per load
    typedef T_ tvec __attribute__((ext_vector_type(kLoad), aligned(4 * sizeof(T_))));
    const bool ok = (rowmask >> t) & 1u;
    const T_* row = ok ? xc + (t - 1) * W : xc;
    float raw[4 * S];
#pragma unroll
    for (int h = 0; h < 4 * S; h += kLoad) {
        const tvec m = *(const tvec*)(row + h);
#pragma unroll
        for (int e = 0; e < kLoad; ++e) raw[h + e] = to_f32((T_)m[e]);
    }
    float lv = __shfl_up(raw[4 * S - 1], 1, 64);
    if (lo && left) lv = to_f32(row[-1]);
    v[0] = (ok && left) ? lv : 0.f;
#pragma unroll
    for (int e = 0; e < 4 * S; ++e) v[1 + e] = ok ? raw[e] : 0.f;
    if constexpr (S == 1) {
        float rv = __shfl_down(raw[0], 1, 64);
        if (hi && right) rv = to_f32(row[4]);
        v[5] = (ok && right) ? rv : 0.f;
    } else {
        v[4 * S + 1] = 0.f;   // never used: the last tap of the last output reads v[S*3 + 2] = v[8]
    }
}

// The strip's outputs: out[rr][i] = sum over taps (di, dj) of k[di*3 + dj] * pixel (S*rr + di, S*i + dj) of the rows above.
template <int S, int RB, typename T_>
__device__ __forceinline__ void dw_strip(const T_* xc, int W, const float (&k)[9], uint32_t rowmask, bool left, bool right,
                                         bool lo, bool hi, float (&out)[RB][4])
{
    constexpr int NR = S * (RB - 1) + 3;
#pragma unroll
    for (int rr = 0; rr < RB; ++rr)
#pragma unroll
        for (int i = 0; i < 4; ++i) out[rr][i] = 0.f;
#pragma unroll
    for (int t = 0; t < NR; ++t) {
        float v[4 * S + 2];
        strip_row<S>(xc, W, t, rowmask, left, right, lo, hi, v);
#pragma unroll
        for (int rr = 0; rr < RB; ++rr) {
            const int di = t - S * rr;   // tap row of output row rr that this input row feeds
            if (di < 0 || di > 2) continue;
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 3; ++j) out[rr][i] += k[di * 3 + j] * v[S * i + j];
        }
    }
}

// Input rows a strip of output rows [r0, r0 + RB) has inside the map, as the mask strip_row takes.
template <int S, int RB>
__device__ __forceinline__ uint32_t strip_rowmask(int r0, int Ho)
{
    uint32_t m = (1u << (S * (RB - 1) + 3)) - 1;
    if (r0 == 0) m &= ~1u;
    if (S == 1 && r0 + RB == Ho) m &= ~(1u << (RB + 1));
    return m;
}

// Stand-alone depthwise stage on strips (see above): stride 1 or 2, input maps of exactly S times the
// output size, RB dividing the output rows, output rows of whole quads of pixels, tensors aligned to 4 values.
// Workgroup `bid` of `blocks`.
template <typename T_, int S, int RB>
__device__ __forceinline__ void strips_body(const T_* __restrict__ x, const T_* __restrict__ kdw, T_* __restrict__ z, int C,
                                            const DwGeom& G, long long items, int flip, uint32_t bid, uint32_t blocks)
{
    typedef T_ tvec __attribute__((ext_vector_type(4)));
    const size_t HWi = (size_t)G.H * G.W, HWo = (size_t)G.Ho * G.Wo;
    const uint32_t W4 = G.Wo / 4, SB = G.Ho / RB;
    // 32-bit index arithmetic (the launcher sends fewer than 2^31 strips here): 64-bit divisions in every lane
    // cost more than the stencil itself.  All lanes of a wavefront run the same number of trips (the strip
    // routine shuffles between lanes); lanes past the end compute strip 0 again and store nothing.
    const uint32_t lane = threadIdx.x & 63;
    for (uint32_t e0 = bid * 256u; e0 < (uint32_t)items; e0 += blocks * 256u) {
        const uint32_t ee = e0 + threadIdx.x;
        const bool live = ee < (uint32_t)items;
        const uint32_t e = live ? ee : 0;
        const int cw = (int)(e % W4) * 4;
        uint32_t t = e / W4;
        const int r0 = (int)(t % SB) * RB;
        t /= SB;                          // t = n*C + a
        const int a = (int)(t % (uint32_t)C);
        float k[9];
        load_taps(kdw, a, flip != 0, k);
        const uint32_t rowmask = strip_rowmask<S, RB>(r0, G.Ho);
        float out[RB][4];
        // consecutive strips of a row are consecutive lanes; the first and last lane of the wavefront and the
        // last live one have no neighbour to ask
        dw_strip<S, RB>(x + t * HWi + (size_t)(S * r0) * G.W + S * cw, G.W, k, rowmask, cw > 0, cw + 4 < G.Wo, lane == 0,
                        lane == 63 || ee + 1 >= (uint32_t)items, out);
        if (!live) continue;
        T_* zo = z + t * HWo + (size_t)r0 * G.Wo + cw;
#pragma unroll
        for (int rr = 0; rr < RB; ++rr) {
            tvec o;
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = from_f32<T_>(out[rr][i]);
            __builtin_nontemporal_store(o, (tvec*)(zo + rr * G.Wo));
        }
    }
}

// Rows per thread of the stage on strips, its strips and workgroups: taller strips read fewer halo rows per output; small
// problems take shorter ones to have enough threads.
inline int strip_rows(int N, int C, const DwGeom& g, long long* items, long long* blocks)
{
    const long long w4 = g.Wo / 4;
    int rb = g.Ho % 4 == 0 ? 4 : g.Ho % 2 == 0 ? 2 : 1;
    while (rb > 1 && (long long)N * C * (g.Ho / rb) * w4 < 256 * 1024) rb /= 2;
    *items = (long long)N * C * (g.Ho / rb) * w4;
    *blocks = (*items + 255) / 256;
    if (*blocks > (1ll << 20)) *blocks = 1ll << 20;   // the kernel strides over what is left
    return rb;
}

// Stand-alone depthwise stage at stride 1 for rows of any length: a thread owns ONE column of RB consecutive output
// rows, consecutive lanes own consecutive pixels of the row-major map, so every load instruction reads consecutive
// values; the pixels left and right of a lane's column are what its neighbouring lanes loaded (lane shuffle), and
// each input row is loaded once per strip.  1 + 2/RB loads per output instead of the nine of the kernel below.
template <typename T_, int RB>
__device__ __forceinline__ void columns_body(const T_* __restrict__ x, const T_* __restrict__ kdw, T_* __restrict__ z, int C,
                                             const DwGeom& G, long long items, int flip, uint32_t bid, uint32_t blocks)
{
    const size_t HW = (size_t)G.H * G.W;
    const uint32_t W = (uint32_t)G.W, SB = (uint32_t)G.H / RB;
    const uint32_t lane = threadIdx.x & 63;
    // all lanes of a wavefront run the same number of trips (they shuffle); lanes past the end redo item 0 and store nothing
    for (uint32_t e0 = bid * 256u; e0 < (uint32_t)items; e0 += blocks * 256u) {
        const uint32_t ee = e0 + threadIdx.x;
        const bool live = ee < (uint32_t)items;
        const uint32_t e = live ? ee : 0;
        const int c = (int)(e % W);
        uint32_t t = e / W;
        const int r0 = (int)(t % SB) * RB;
        t /= SB;                          // t = n*C + a
        float k[9];
        load_taps(kdw, (int)(t % (uint32_t)C), flip != 0, k);
        const T_* xc = x + t * HW + (size_t)r0 * W + c;      // input pixel (r0, c)
        const bool left = c > 0, right = c + 1 < (int)W;
        const bool lo = lane == 0, hi = lane == 63 || ee + 1 >= (uint32_t)items;
        float out[RB];
#pragma unroll
        for (int rr = 0; rr < RB; ++rr) out[rr] = 0.f;
#pragma unroll
        for (int tr = 0; tr < RB + 2; ++tr) {
            const int r = r0 - 1 + tr;
            const bool ok = r >= 0 && r < G.H;
            const T_* row = ok ? xc + (tr - 1) * (int)W : xc;
            const float mid = to_f32(row[0]);
            float lv = __shfl_up(mid, 1, 64), rv = __shfl_down(mid, 1, 64);
            if (lo && left) lv = to_f32(row[-1]);
            if (hi && right) rv = to_f32(row[1]);
            const float v0 = (ok && left) ? lv : 0.f, v1 = ok ? mid : 0.f, v2 = (ok && right) ? rv : 0.f;
#pragma unroll
            for (int rr = 0; rr < RB; ++rr) {
                const int di = tr - rr;
                if (di < 0 || di > 2) continue;
                // the order of the strips' sums, spelled out: which product of a sum of three is contracted is the compiler's
                // choice, and was another one in another kernel
                out[rr] = __builtin_fmaf(k[di * 3], v0, out[rr]);
                out[rr] = __builtin_fmaf(k[di * 3 + 1], v1, out[rr]);
                out[rr] = __builtin_fmaf(k[di * 3 + 2], v2, out[rr]);
            }
        }
        if (!live) continue;
        T_* zo = z + t * HW + (size_t)r0 * W + c;
#pragma unroll
        for (int rr = 0; rr < RB; ++rr) __builtin_nontemporal_store(from_f32<T_>(out[rr]), zo + rr * (int)W);
    }
}

// Stand-alone depthwise stage, any stride and map size: one thread per output value, taps in row-major order.
// IDX is the type of the flat output index: 32 bits whenever the tensor allows it (64-bit divisions in every lane
// cost several times the stencil).
template <typename T_, typename IDX>
__device__ __forceinline__ void pixels_body(const T_* __restrict__ x, const T_* __restrict__ kdw, T_* __restrict__ z, int C,
                                            const DwGeom& G, long long items, int flip, uint32_t bid, uint32_t blocks)
{
    const size_t HWi = (size_t)G.H * G.W;
    for (IDX e = (IDX)bid * 256 + threadIdx.x; e < (IDX)items; e += (IDX)blocks * 256) {
        const int q = (int)(e % (IDX)G.Wo);
        IDX t = e / (IDX)G.Wo;
        const int m = (int)(t % (IDX)G.Ho);
        t /= (IDX)G.Ho;
        const int a = (int)(t % (IDX)C);
        const T_* xc = x + (size_t)t * HWi;
        float out = 0.f;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const int rr = G.s * m + i - 1;
            if (rr < 0 || rr >= G.H) continue;
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const int cc = G.s * q + j - 1;
                if (cc < 0 || cc >= G.W) continue;
                out += to_f32(kdw[a * 9 + (flip ? 8 - (i * 3 + j) : i * 3 + j)]) * to_f32(xc[(size_t)rr * G.W + cc]);
            }
        }
        z[e] = from_f32<T_>(out);
    }
}

// How the stage runs on a layer: which of the bodies above, its work items and its workgroups of 256 threads.
enum { kStrips1, kStrips2, kColumns, kPixels, kPixels64 };

struct Stage {
    int kind, rb, flip;
    uint32_t blocks;
    long long items;
};

template <typename T_>
inline Stage plan_stage(const T_* x, const T_* z, int N, int C, const DwGeom& g, bool flip)
{
    Stage s;
    s.flip = flip;
    s.rb = 1;
    long long blocks;
    const bool sized = (g.s == 1 || g.s == 2) && g.H == g.s * g.Ho && g.W == g.s * g.Wo &&
                       (long long)N * C * g.Ho * ((g.Wo + 3) / 4) < (1ll << 31);
    const bool vec = g.Wo % 4 == 0 && (((uintptr_t)x | (uintptr_t)z) & (4 * sizeof(T_) - 1)) == 0;
    if (sized && vec) {
        s.kind = g.s == 1 ? kStrips1 : kStrips2;
        s.rb = strip_rows(N, C, g, &s.items, &blocks);
    } else {
        const bool columns = g.s == 1 && (long long)N * C * g.H * g.W < (1ll << 31);   // rows of any length
        if (columns) s.rb = g.H % 4 == 0 ? 4 : g.H % 2 == 0 ? 2 : 1;
        s.items = (long long)N * C * (g.Ho / s.rb) * g.Wo;
        // the index plus one grid stride still fits 32 bits
        s.kind = columns ? kColumns : s.items + (1ll << 28) < (1ll << 32) ? kPixels : kPixels64;
        blocks = (s.items + 255) / 256;
        if (blocks > (1ll << 20)) blocks = 1ll << 20;   // the kernel strides over what is left
    }
    s.blocks = (uint32_t)blocks;
    return s;
}

// The stage as a range of a grid that other work shares: the variant is chosen when the workgroup runs (any kind but kPixels64).
template <typename T_>
__device__ __forceinline__ void stage_body(const T_* __restrict__ x, const T_* __restrict__ kdw, T_* __restrict__ z, int C,
                                           const DwGeom& G, const Stage& s, uint32_t bid)
{
    switch (s.kind * 8 + s.rb) {
        case kStrips1 * 8 + 1: return strips_body<T_, 1, 1>(x, kdw, z, C, G, s.items, s.flip, bid, s.blocks);
        case kStrips1 * 8 + 2: return strips_body<T_, 1, 2>(x, kdw, z, C, G, s.items, s.flip, bid, s.blocks);
        case kStrips1 * 8 + 4: return strips_body<T_, 1, 4>(x, kdw, z, C, G, s.items, s.flip, bid, s.blocks);
        case kStrips2 * 8 + 1: return strips_body<T_, 2, 1>(x, kdw, z, C, G, s.items, s.flip, bid, s.blocks);
        case kStrips2 * 8 + 2: return strips_body<T_, 2, 2>(x, kdw, z, C, G, s.items, s.flip, bid, s.blocks);
        case kStrips2 * 8 + 4: return strips_body<T_, 2, 4>(x, kdw, z, C, G, s.items, s.flip, bid, s.blocks);
        case kColumns * 8 + 1: return columns_body<T_, 1>(x, kdw, z, C, G, s.items, s.flip, bid, s.blocks);
        case kColumns * 8 + 2: return columns_body<T_, 2>(x, kdw, z, C, G, s.items, s.flip, bid, s.blocks);
        case kColumns * 8 + 4: return columns_body<T_, 4>(x, kdw, z, C, G, s.items, s.flip, bid, s.blocks);
        default: return pixels_body<T_, uint32_t>(x, kdw, z, C, G, s.items, s.flip, bid, s.blocks);
    }
}

}  // namespace dw

}  // namespace scc
