// Grad-weight of SCC for layers in which many 32-filter tiles read the same planes: both operands go through LDS once per
// workgroup of four filter tiles.
//
// dw[k,j] = sum_{n,p} dy[n,k,p] * x[n,(s_k+j) mod Cin,p]     (the derivative of the forward definition with respect to w)
//
// scc_mfma_bww_kernel.h gives every wavefront its own 32 filters x 32..96 positions and lets the wavefronts of a workgroup
// split the columns: every x plane is fetched once per filter tile whose windows reach it, every dy plane once per chunk
// of span positions (the channel-expanding layer moves 1 GB through L2 in a pass).  Here a workgroup owns 128
// filters in the order of their window starts times 32*PT positions of the walk that covers their windows (the channels
// from the first window's start to the last one's end), for one slice of the columns.  Per round its 256 lanes fetch 16
// bytes of 128 dy planes and 32*PT x planes each (32 columns of binary32, 64 of bf16) and park them in LDS as they are:
// 16 bytes of one plane are a lane's operand of one bf16 instruction, or of four binary32 ones; wavefront t multiplies
// filter tile t with all PT position tiles and skips those none of its windows reaches.  One LDS buffer and two barriers
// per round; the next round's loads are in flight while this one is multiplied, and three workgroups per CU overlap each
// other's phases.
//
// Products are those of the per-tile kernel: exact (bf16 tensors), binary32 through v_mfma_f32_32x32x2_f32 (fp32 tensors).
// What bounds it: binary32, the matrix pipe (channel-expanding layer: 68 of 117 us at its peak rate, the idle share of
// tiles that windows fill only in part included); bf16, fetching.  (binary32 through six bf16 products of a three-way cut
// takes 101 us there, but drops the smallest partial products and loses operands near the end of the exponent range.)
//
// A wavefront's tiles are its own, so there is no sum inside a workgroup; the slices' partial sums go to the workspace in the
// layout of dw and launch_weight_reduce adds them in slice order: no atomics, bitwise reproducible.
#pragma once
#include "scc.h"
#include "scc_band.h"
#include "scc_common.h"
#include "scc_mfma_bww_kernel.h"

namespace scc {

namespace shared_bww {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct WeightTiling {
    Band b;
    int rows;       // filters in order of their starts: P*F
    int NG;         // groups of 128 rows
    int NSC;        // chunks of 32*PT walk positions (of the longest walk)
    int KS;         // slices of the columns, 0 where the layer's partial sums would cost more than the kernel saves
    int per_slice;  // consecutive rounds a slice takes; the last slice may have fewer, none is empty
    int total;      // workgroups with work: KS * NG * NSC, slice slowest
    int chunk;      // consecutive workgroups of that order given to one XCD
    Groups q;       // column groups of 16 bytes
};

// walk of row group ng: first channel, channels (at most Cin: each channel once)
__host__ __device__ inline void weight_walk(const Problem& P, const Band& b, int rows, int ng, int& first, int& len)
{
    const int r0 = ng * 128, r1 = r0 + 127 < rows ? r0 + 127 : rows - 1;
    const int m0 = r0 / b.F, m1 = r1 / b.F;
    first = b.g * m0;
    const long long span = (long long)P.L + (long long)b.g * (m1 - m0);
    len = span < P.Cin ? (int)span : P.Cin;
}

constexpr int weight_rows(int pt) { return 128 + 32 * pt; }
// bytes of one lane group's operands: 16 of padding, so that the 16-byte stores of eight lanes (one plane, eight such blocks)
// cover the 128 bytes of all banks; with 32 they conflict two by two, without any eight by eight (dw alone, binary32:
// channel-expanding layer 130 against 138 us with 32, 120 -> 500 channels on 11x9 55 against 59; bf16 the same with 32 and 16,
// 50 against 36 us for four-way conflicts on the first layer)
constexpr int weight_half(int pt) { return weight_rows(pt) * 16 + 16; }
constexpr int weight_lds(int pt) { return 8 * weight_half(pt); }

// bid: the workgroup's index in a launch whose first workgroup is a multiple of 8 (bid % 8 names the XCD)
template <typename T_, int PT>
__device__ __forceinline__ void weight_body(const T_* __restrict__ x, const T_* __restrict__ dy, float* __restrict__ out,
                                            const Problem& P, const WeightTiling& T, const int bid, char* const lds_w)
{
    constexpr uint32_t ES = sizeof(T_);
    constexpr int CT = 16 / (int)ES;                    // columns per lane and load
    constexpr int NL = 4 + PT;                          // loads per lane and round: planes tid/8 + 32*it
    constexpr int kHalf = weight_half(PT);
    typedef T_ ldvec __attribute__((ext_vector_type(CT), aligned(sizeof(T_))));

    const int xcd = bid & 7, slot = bid >> 3;
    const int tiles = T.NG * T.NSC, logical = xcd * T.chunk + slot;
    if (slot >= T.chunk || logical >= T.total) return;  // the whole workgroup leaves
    const int ks = logical / tiles, tix = logical % tiles;
    const int ng = tix / T.NSC, sc = tix % T.NSC;
    int first, len;
    weight_walk(P, T.b, T.rows, ng, first, len);
    const int pos0 = 32 * PT * sc;
    if (pos0 >= len) return;                            // shorter walk than the longest: the whole workgroup leaves

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63, f = lane & 31, h = lane >> 5;
    const int lr = tid >> 3, lc = tid & 7;              // loading role: planes lr + 32*it, column group lc of 8

    auto filter = [&](int row) {                        // filter of a row, -1 where there is none
        if (row >= T.rows) return -1;
        const int m = row / T.b.F;
        const int k = (int)(((uint32_t)m * (uint32_t)T.b.inv) % (uint32_t)T.b.P) + T.b.P * (row - m * T.b.F);
        return k < P.Cout ? k : -1;
    };
    const uint32_t plane = (uint32_t)P.HW * ES;
    uint32_t rowoff[NL];
#pragma unroll
    for (int it = 0; it < NL; ++it) {
        if (it < 4) {
            const int k = filter(128 * ng + 32 * it + lr);
            rowoff[it] = (uint32_t)(k < 0 ? 0 : k) * plane;      // rows without a filter are fetched, never stored
        } else {
            const int pos = pos0 + 32 * (it - 4) + lr;
            int c = first + (pos < len ? pos : 0);
            c -= c >= P.Cin ? P.Cin : 0;
            rowoff[it] = (uint32_t)c * plane;
        }
    }
    // this wavefront's filters start between walk positions d0 and d0 + ..., its windows end before d1; a walk around the
    // whole circle is entered again past its end
    const int row0 = 128 * ng + 32 * wave;
    const int last = row0 + 31 < T.rows ? row0 + 31 : T.rows - 1;
    const int d0 = T.b.g * (row0 / T.b.F) - first, d1 = T.b.g * (last / T.b.F) - first + P.L;
    uint32_t active = 0;
#pragma unroll
    for (int t = 0; t < PT; ++t) {
        const int p0 = pos0 + 32 * t;
        if (row0 < T.rows && p0 < len && ((p0 < d1 && p0 + 32 > d0) || p0 < d1 - P.Cin)) active |= 1u << t;
    }
    // Binary32, which the matrix pipe bounds: of a position tile that this wavefront's windows reach one half of 16 only (one such
    // tile), that half takes v_mfma_f32_16x16x4_f32 for half the matrix time.  (Windows of 64 on 8 neighbouring starts span 71
    // positions: 80 of three tiles instead of 96; 128 x 128 -> 512 on 32x32, cg 2, co 0.33: alone 131 -> 117 us, beside grad-input, which the
    // memory bounds, 202 -> 200.)
    int half_at = -1;                                   // first position of that half in the workgroup's chunk
    if constexpr (ES == 4) {
#pragma unroll
        for (int t = 0; t < PT; ++t) {
            auto reached = [&](int p0) { return p0 < len && ((p0 < d1 && p0 + 16 > d0) || p0 < d1 - P.Cin); };
            const bool lo = reached(pos0 + 32 * t), hi = reached(pos0 + 32 * t + 16);
            if (((active >> t) & 1u) && lo != hi && half_at < 0) {
                half_at = 32 * t + (hi ? 16 : 0);
                active &= ~(1u << t);
            }
        }
    }

    // this slice's rounds (8 column groups each) from r0 on.  (Slices of an XCD that take every n-th round of its columns
    // instead, so that it sweeps them on a narrow front, are slower: channel-expanding layer, bf16 40 -> 51 us.)
    const int rounds = (int)((T.q.count + 7) / 8), count = (int)T.q.count;
    const int r0 = ks * T.per_slice;
    const int nround = (r0 + T.per_slice < rounds ? r0 + T.per_slice : rounds) - r0;   // at least one

    const uint32_t per = (uint32_t)T.q.per;
    const uint32_t sampA = (uint32_t)P.Cout * plane, sampB = (uint32_t)P.Cin * plane;
    uint32_t cp, offA, offB;                            // group inside the sample, byte offsets of the sample
    int next;
    auto seek = [&](int round) {
        next = 8 * round + lc;
        const uint32_t n = (uint32_t)next / per;
        cp = (uint32_t)next - n * per;
        offA = n * sampA;
        offB = n * sampB;
    };
    // bf16, which the memory bounds: slice ks starts ks rounds in and goes round.  Started together, slices whose length is a power of two would be on the same memory
    // channels all the way: 128 x 128 -> 512 on 32x32, cg 2, co 0.33, both gradients, 66.4 -> 62.7 us; others, and binary32,
    // the same.
    const int rot = ES == 2 ? ks % nround : 0;
    seek(r0 + rot);
    int left = nround - rot;
    const uint32_t dn = 8u / per, dp = 8u % per;
    const uint32_t dup = (uint32_t)CT * per - (uint32_t)P.HW;    // pixels the last group of a sample shares with the one before
    ldvec raw[NL];
    uint32_t in = 0;                                    // one bit per column of the loaded group that counts
    auto issue = [&]() {
        const bool gin = next < count;
        in = gin ? (((1u << CT) - 1u) & (0xffffffffu << (cp == per - 1u ? dup : 0u))) : 0u;
        const uint32_t p = ((uint32_t)CT * cp < (uint32_t)T.q.last ? (uint32_t)CT * cp : (uint32_t)T.q.last) * ES;
        const uint32_t ca = gin ? offA + p : 0u, cb = gin ? offB + p : 0u;
#pragma unroll
        for (int it = 0; it < NL; ++it)
            raw[it] = *(const ldvec*)((it < 4 ? (const char*)dy + ca : (const char*)x + cb) + rowoff[it]);
        next += 8;
        cp += dp;
        const bool wr = cp >= per;
        cp -= wr ? per : 0u;
        offA += dn * sampA + (wr ? sampA : 0u);
        offB += dn * sampB + (wr ? sampB : 0u);
        if (ES == 2 && --left == 0) seek(r0);
    };
    // operand layout: [column group lc][plane], 16 bytes each; half-wave h reads group 2*j + h in step j
    char* const dst0 = lds_w + lc * kHalf + lr * 16;
    auto commit = [&](bool full) {
#pragma unroll
        for (int it = 0; it < NL; ++it) {
            ldvec v = raw[it];
            if (!full) {
#pragma unroll
                for (int e = 0; e < CT; ++e) v[e] = (in >> e) & 1u ? v[e] : (T_)0;
            }
            *(u32x4*)(dst0 + it * 512) = __builtin_bit_cast(u32x4, v);
        }
    };

    f32x16 acc[PT];
#pragma unroll
    for (int t = 0; t < PT; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;
    f32x4 part[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};   // the half tile: rows 16q .. 16q+15 of the wavefront's
    const int f4 = lane & 15, h4 = lane >> 4;
    auto compute_half = [&]() {
#pragma unroll
        for (int j = 0; j < 2; ++j) {                   // 16 columns: quarter-wave h4 reads group 4*j + h4
            const char* base = lds_w + (4 * j + h4) * kHalf + f4 * 16;
            const u32x4 b = *(const u32x4*)(base + (128 + half_at) * 16);
            const u32x4 a0 = *(const u32x4*)(base + wave * 512), a1 = *(const u32x4*)(base + wave * 512 + 256);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                part[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a0[e]), __uint_as_float(b[e]), part[0], 0, 0, 0);
                part[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a1[e]), __uint_as_float(b[e]), part[1], 0, 0, 0);
            }
        }
    };
    auto compute = [&]() {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const char* base = lds_w + (2 * j + h) * kHalf + f * 16;
            const u32x4 a = *(const u32x4*)(base + wave * 512);
#pragma unroll
            for (int t = 0; t < PT; ++t) {
                if (!((active >> t) & 1u)) continue;
                const u32x4 b = *(const u32x4*)(base + (4 + t) * 512);
                if constexpr (ES == 2) {                // 8 columns of the half-wave's
                    const uint32_t aa[4] = {a[0], a[1], a[2], a[3]}, ba[4] = {b[0], b[1], b[2], b[3]};
                    acc[t] = mfma_bf16<8>(aa, ba, acc[t]);
                } else {                                // column e of the half-wave's 4
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a[e]), __uint_as_float(b[e]), acc[t],
                                                                      0, 0, 0);
                }
            }
        }
    };

    issue();
    for (int r = 0; r < nround; ++r) {
        __syncthreads();                                // nobody reads the previous round any more
        commit(dup == 0u && 8 * (r0 + (ES == 2 ? nround : r + 1)) <= count);
        if (r + 1 < nround) issue();
        __syncthreads();
        compute();
        if constexpr (ES == 4)
            if (half_at >= 0) compute_half();
    }

    // accumulator register v holds row 8*(v/4) + 4*h + v%4 of the wavefront's tile, walk position pos0 + 32t + f
    const int k_f = filter(row0 + f);
    const int s_f = T.b.g * ((row0 + f) / T.b.F);
    char* dst = (char*)(out + (size_t)ks * ((size_t)P.Cout * P.L));
    int kr[16], sr[16];                                 // requested together: one by one each would wait for its exchange
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int fr = 8 * (v >> 2) + 4 * h + (v & 3);
        kr[v] = __shfl(k_f, fr, 64);
        sr[v] = __shfl(s_f, fr, 64);
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) {
#pragma unroll
        for (int t = 0; t < PT; ++t) {
            const int pos = pos0 + 32 * t + f;
            int j = first + pos - sr[v];                // first <= s: j starts at first - s > -Cin
            j += j < 0 ? P.Cin : 0;
            j -= j >= P.Cin ? P.Cin : 0;
            const bool here = ES == 2 || half_at < 0 || t != half_at >> 5;
            if ((kr[v] >= 0) & (pos < len) & (j < P.L) & here) *(float*)(dst + (uint32_t)(kr[v] * P.L + j) * 4u) = acc[t][v];
        }
    }
    if constexpr (ES == 4) {
        if (half_at < 0) return;
        // register v of part[q] holds row 16q + 4*h4 + v, position half_at + f4 of the chunk (of the tile's other half no row stores)
        const int pos = pos0 + half_at + f4;
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int k = __shfl(k_f, 16 * q + 4 * h4 + v, 64);
                int j = first + pos - __shfl(s_f, 16 * q + 4 * h4 + v, 64);
                j += j < 0 ? P.Cin : 0;
                j -= j >= P.Cin ? P.Cin : 0;
                if ((k >= 0) & (pos < len) & (j < P.L)) *(float*)(dst + (uint32_t)(k * P.L + j) * 4u) = part[q][v];
            }
    }
}

// beside: for the launch that carries grad-input as well (scc_shared_merged.hip)
inline WeightTiling make_weight_tiling(const Problem& p, int es, int* PT, bool beside = false)
{
    WeightTiling t = {};
    t.b = make_band(p);
    t.rows = t.b.P * t.b.F;
    t.NG = (t.rows + 127) / 128;
    int longest = 1;
    for (int ng = 0; ng < t.NG; ++ng) {
        int first, len;
        weight_walk(p, t.b, t.rows, ng, first, len);
        longest = len > longest ? len : longest;
    }
    // position tiles per workgroup: the fewest planes fetched over all chunks, ties to the larger tile
    long long best = -1;
    for (int pt = 4; pt >= 2; --pt) {
        const long long planes = (long long)((longest + 32 * pt - 1) / (32 * pt)) * (4 + pt);
        if (best < 0 || planes < best) {
            best = planes;
            *PT = pt;
        }
    }
    t.NSC = (longest + 32 * *PT - 1) / (32 * *PT);
    t.q = column_groups(p, 16 / es);
    const long long tiles = (long long)t.NG * t.NSC;
    const int rounds = (int)((t.q.count + 7) / 8);
    // No sum is longer (by 2 %, a hundredth of the error) than the per-tile kernel's, of which each wavefront and accumulator adds
    // a share of the columns: the rounding error against binary64 is then no larger (30 x 640 -> 640 on 32x32, cg 4, co 0, bf16:
    // 2.0e-7 there, 2.6e-7 with 17 slices, 2.0e-7 with the 29 this asks for, and 50 against 53 us).
    const bww::BwwTiling o = bww::make_tiling(p, beside);
    const long long its = (long long)o.per_ks * 4 / (bww::kWaves * bww::accumulators_of(o.NPT, es, p.NQ < 256));   // columns
    const long long longest_slice = its * 51 / (50 * 8 * (16 / es));
    if (longest_slice == 0) return t;
    // Workgroups to aim at, per CU: alone three, which hides most (752 channels, bf16: 89 us against 108 with two), beside
    // grad-input one (bf16) or two (binary32): channel-expanding layer f32 219 us with one, 209 with two, bf16 64 and 70; 256 -> 256, 16x16,
    // cg 1: 78 and 82, 31 and 36; 512 -> 1024, 7x7, cg 2, co 0.33: 56 and 55, 33 and 35; 37 x 336 -> 330, 20x41, cg 1: f32 132 and 122.
    // A slice's partial sums are written and read once each: with more than a quarter of the values x and dy hold they cost
    // more than the slices hide (256 -> 256, 16x16, cg 1, f32: 78 us at a quarter, 82 at a half).
    const long long dw = (long long)p.Cout * p.L, values = (long long)(p.Cin + p.Cout) * p.NQ, quarter = values / (4 * dw);
    long long best_time = -1;
    for (int per_cu = !beside ? 3 : es == 2 ? 1 : 2; per_cu > 0; --per_cu) {
        long long ks = 256 * per_cu / tiles;
        ks = ks < quarter ? ks : quarter;
        long long len = ks > 0 ? (rounds + ks - 1) / ks : rounds;
        len = len < longest_slice ? len : longest_slice;
        const long long slices = (rounds + len - 1) / len, time = (slices * tiles + 255) / 256 * len;   // of the busiest CU
        if (best_time >= 0 && 100 * time >= 95 * best_time) continue;
        best_time = time;
        t.per_slice = (int)len;
        t.KS = (int)slices;
        if (es == 2) break;                             // not bound by the matrix pipe
    }
    // Layers with few columns and many weights (16 x 768 -> 1533 on 7x7, cg 1: f32 60 us per tile, 71 here) would mostly move
    // partial sums; alone they also have to fit the buffer of scc_backward_weight_static, which runs the same kernels.
    if (t.KS * dw > 2 * values || (!beside && t.KS * dw * 4 > (long long)SCC_STATIC_SCRATCH_BYTES)) t.KS = 0;
    t.total = (int)(t.KS * tiles);
    t.chunk = (t.total + 7) / 8;
    return t;
}

inline bool weight_eligible(const Problem& p, int es)
{
    if (!backward_weight_mfma_eligible(p) || p.HW < 16 / es) return false;
    const Band b = make_band(p);
    return 4ll * b.P * b.F <= 5ll * p.Cout && b.P * (long long)b.F <= (1 << 20);   // else too many empty rows
}

struct WeightCost {
    double there, here;   // planes fetched, columns included, by the per-tile kernel and by this one
    double matrix;        // matrix time of the busiest CU with this one over that with the per-tile kernel
};

// Both sides' matrix time counts every tile of 32 x 32 that some wavefront of a workgroup may wait for (windows that reach a part
// of a walk only leave matrix pipes idle: 227 x 400 -> 200 on 20x20, cg 2: twice the tiles, f32 203 against 146 us) and the last
// generation of workgroups (per-tile kernel on 40 x 272 -> 270, cg 1: 270 of them on 256 CUs, 114 us against 77 here).
inline WeightCost weight_cost(const Problem& p, int es, const WeightTiling& t, int pt, bool beside)
{
    const bww::BwwTiling o = bww::make_tiling(p, beside);
    const long long tiles = (long long)o.IB * o.MB * o.NSC, mine = (long long)t.NG * t.NSC;
    WeightCost c;
    c.here = (double)mine * weight_rows(pt) * p.NQ;
    c.there = (double)tiles * bww::rows_of(o.NPT) * p.NQ;
    c.matrix = (double)((t.total + 255) / 256) * t.per_slice * (8 * 16 / es) * 4 * pt /
               ((double)((tiles * o.KS + 255) / 256) * o.per_ks * 4 * o.NPT);
    return c;
}

}  // namespace shared_bww

}  // namespace scc
