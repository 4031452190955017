// Forward and grad-input of SCC as one matrix product with packed weights, for layers with enough arithmetic to pay for
// a packing pass over the (small) weight matrix first.
//
//   y[n,k,p]  = sum_j w[k,j] * x[n,(s_k+j) mod Cin,p]                       (Section 4.2, output-centric forward)
//   dx[n,c,p] = sum over filters k covering c of w[k,(c-s_k) mod Cin] * dy[n,k,p]   (Section 4.2, input-centric backward)
//
// Both are rows x columns products, out = A * B: rows are filters in the order of their window starts (forward) or
// channels (grad-input), B's rows are the planes of x or dy, columns are (sample, pixel) pairs.  A group of 128
// neighbouring rows reads the planes of one contiguous stretch of the channel circle (forward: from the first window's
// start to the last window's end) or of the circle of windows (grad-input: the filters of all windows that reach one of
// the group's channels); this stretch is the group's walk, every plane at most once.  A(row, position of the walk) is
// w[k, (c - s_k) mod Cin] for that row's and position's filter k and channel c where this index is below L, else zero.
//
// pack_weights (first launch) writes, per row group: the walk as a table of plane offsets; A in the operand layout of
// the matrix instruction (per K group of 16 positions and tile of 32 rows: 64 lanes x 8 bf16, binary32 weights already
// cut into their three bf16 pieces); and which (tile, K group) pairs hold any weight at all.
// packed_product (second launch): a workgroup of four wavefronts owns one row group and 32*CT columns and walks in rounds
// of 16*KG positions.  The 256 lanes fetch a round of B planes (a group of CT pixels per lane and plane), cut each
// value once and park the pieces in LDS in operand layout; A comes from L2 straight into registers, 1 KB per
// instruction and piece, without any vector work.  Two LDS buffers, one barrier per round; B is in flight for a round, A
// for KG-1 K groups.
//
// What bounds it: a wavefront of 32 rows x 32*CT columns takes 6*CT matrix instructions per K group (binary32; bf16: CT) for
// 3*CT 16-byte LDS reads and 3 global loads of A. With tiles of 128 columns matrix and LDS pipe (shared by four SIMDs, busy
// for 0.6 of the matrix time) and the cuts' vector work add up; tiles of 64 columns read A through L1 as often for half the
// arithmetic and are bound by that. Two tiles of 32 rows per wavefront would halve the LDS reads and the cuts per matrix
// instruction and were slower (228 registers, two workgroups per CU: channel-expanding layer, forward, f32 98 us against 88).
#pragma once
#include "scc_band.h"
#include "scc_common.h"

#include <type_traits>

namespace scc {

namespace packed {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kMaxGroups = 128;   // K groups of a walk: two 64-bit masks
constexpr int kTiles = 4;         // tiles of 32 rows in a row group, one per wavefront

struct Packed {
    Band b;
    int rows;        // filters in order of their starts, P*F of them (forward), or Cin
    int NG;          // row groups of 128: one tile of 32 rows per wavefront
    int KG;          // K groups of 16 positions per round
    int nround;      // rounds of the longest walk; shorter walks are padded with empty positions
    Deal deal;       // (column tile, row group)
    uint32_t tab_group;   // table entries per row group: nround rounds
    uint32_t act_at, a_at;   // byte offsets of the activity bytes and of A in the workspace
    size_t bytes;    // of the workspace
    Groups q;        // column groups of CT pixels
};

__host__ __device__ inline int floor_div_p(int a, int b)   // b > 0
{
    const int q = a / b;
    return (a % b != 0 && a < 0) ? q - 1 : q;
}

// the walk of row group ng: first window / channel and number of positions
template <bool FWD>
__host__ __device__ inline void walk_of(const Problem& P, const Band& b, int rows, int ng, int& first, int& len)
{
    const int r0 = ng * 128, r1 = r0 + 127 < rows ? r0 + 127 : rows - 1;
    if (FWD) {
        const int m0 = r0 / b.F, m1 = r1 / b.F;
        first = b.g * m0 % P.Cin;
        const long long span = (long long)P.L + (long long)b.g * (m1 - m0);
        len = span < P.Cin ? (int)span : P.Cin;
    } else {
        first = -floor_div_p(P.L - 1 - r0, b.g);             // windows that reach channel r0 or a later one ...
        int nwin = floor_div_p(r1, b.g) - first + 1;         // ... up to the last that starts at or before r1
        nwin = nwin < 0 ? 0 : (nwin < b.P ? nwin : b.P);
        len = nwin * b.F;
    }
}

// filter of the i-th member of window m (on the circle), or -1
__device__ __forceinline__ int filter_of(const Band& b, int m, int i, int Cout)
{
    const int k = (int)(((uint32_t)m * (uint32_t)b.inv) % (uint32_t)b.P) + b.P * i;
    return k < Cout ? k : -1;
}

// bid: the workgroup's index in a launch whose first workgroup is a multiple of 8 (bid % 8 names the XCD)
template <typename T_, int CT, bool FWD, bool RUNS = true>
__device__ __forceinline__ void packed_body(const T_* __restrict__ src, const char* __restrict__ ws, T_* __restrict__ out,
                                            const Problem& P, const Packed& T, const int bid, char* const lds_p)
{
    typedef T_ bvec __attribute__((ext_vector_type(CT), aligned(sizeof(T_))));   // CT consecutive columns of one plane
    constexpr uint32_t ES = sizeof(T_);
    constexpr int NP = ES == 2 ? 1 : 3;                 // bf16 pieces of a value
    constexpr int KG = ES == 2 ? 4 : 2;                 // K groups per round
    constexpr int KR = 16 * KG;                         // positions per round
    constexpr int NQ = KR / 32;                         // quads of 4 planes a lane fetches per round
    constexpr int kCols = 32 * CT;
    constexpr int kPiece = KG * 2 * kCols * 16;         // bytes of one piece of a round: [K group][half][column][8 positions]
    constexpr int kBuf = NP * kPiece;
    uint32_t* const tab = (uint32_t*)(lds_p + 2 * kBuf);

    int ct, ng;
    if (!dealt<RUNS>(T.deal, bid, ct, ng)) return;            // the whole workgroup leaves
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63, f = lane & 31, h = lane >> 5;
    const int nround = T.nround, nkg = nround * KG;

    {   // the walk's plane offsets
        const uint32_t* t = (const uint32_t*)ws + (size_t)ng * T.tab_group;
        for (int i = tid; i < nround * KR; i += 256) tab[i] = t[i];
    }
    // which K groups reach this wavefront's rows
    unsigned long long mask0, mask1;
    {
        const uint8_t* a = (const uint8_t*)(ws + T.act_at) + (ng * kTiles + wave) * kMaxGroups;
        mask0 = __ballot(lane < nkg && a[lane] != 0);
        mask1 = __ballot(lane + 64 < nkg && a[lane + 64] != 0);
    }
    auto active = [&](int g) { return ((g < 64 ? mask0 >> g : mask1 >> (g - 64)) & 1ull) != 0; };

    // ---- A: K group g of this wavefront's tile, 16 bytes per lane and piece -----------------------
    const char* ap = ws + T.a_at + ((size_t)ng * nkg * kTiles + wave) * (NP * 1024) + lane * 16;
    u32x4 a[KG][NP];
    auto issue_a = [&](auto SET) {                      // the next K group; runs up to KG-1 groups past the last one, inside the workspace
#pragma unroll
        for (int q = 0; q < NP; ++q) a[decltype(SET)::value][q] = *(const u32x4*)(ap + q * 1024);
        ap += kTiles * NP * 1024;
    };

    // ---- B, loading role: lane (quad lu + 8z, column group lq) fetches CT columns of 4 planes ------------------
    // (eight lanes with one quad, the next eight with the other quad of the same eight positions: the 8-byte LDS stores of
    // 16 lanes then cover 128 contiguous bytes; with 16 lanes on one quad they conflict two by two)
    const int lq = (lane & 7) | (lane >> 4) << 3, lu = 2 * wave + (lane >> 3 & 1);
    const int srows = FWD ? P.Cin : P.Cout, drows = FWD ? P.Cout : P.Cin;
    uint32_t lcol;
    {
        const uint32_t u = (uint32_t)ct * 32u + (uint32_t)lq;
        uint32_t n, p;
        column_of_group(u < (uint32_t)T.q.count ? u : 0u, T.q, n, p);   // past the end: group 0, never stored
        lcol = (n * (uint32_t)srows * (uint32_t)P.HW + p) * ES;
    }
    bvec raw[NQ][4];
    auto issue_b = [&](int r) {
#pragma unroll
        for (int z = 0; z < NQ; ++z) {
            const u32x4 o = *(const u32x4*)(tab + KR * r + 4 * (lu + 8 * z));
#pragma unroll
            for (int e = 0; e < 4; ++e) raw[z][e] = *(const bvec*)((const char*)src + (lcol + o[e]));
        }
    };
    auto commit_b = [&](int buf) {
#pragma unroll
        for (int z = 0; z < NQ; ++z) {
            const int quad = lu + 8 * z;
            char* dst = lds_p + buf * kBuf + ((quad >> 1) * kCols + lq) * 16 + 8 * (quad & 1);
#pragma unroll
            for (int j = 0; j < CT; ++j) {              // column CT*lq + j of the tile is LDS column 32j + lq
                if constexpr (ES == 2) {
                    *(u32x2*)(dst + j * 512) =
                        u32x2{(uint32_t)(T_)raw[z][0][j] | ((uint32_t)(T_)raw[z][1][j] << 16),
                              (uint32_t)(T_)raw[z][2][j] | ((uint32_t)(T_)raw[z][3][j] << 16)};
                } else {
                    uint32_t hi[2], mid[2], lo[2];
                    split3<4>([&](int e) { return raw[z][e][j]; }, hi, mid, lo);
                    *(u32x2*)(dst + j * 512) = u32x2{hi[0], hi[1]};
                    *(u32x2*)(dst + j * 512 + kPiece) = u32x2{mid[0], mid[1]};
                    *(u32x2*)(dst + j * 512 + 2 * kPiece) = u32x2{lo[0], lo[1]};
                }
            }
        }
    };

    f32x16 acc[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[c][v] = 0.f;

    auto mm = [&](const u32x4& x, const u32x4& y, f32x16& d) {
        const uint32_t xa[4] = {x[0], x[1], x[2], x[3]}, ya[4] = {y[0], y[1], y[2], y[3]};
        d = mfma_bf16<8>(xa, ya, d);
    };
    auto compute = [&](auto SET, int g, int buf) {
        constexpr int j = decltype(SET)::value;
        if (!active(g)) return;
        const char* bb = lds_p + buf * kBuf + ((j * 2 + h) * kCols + f) * 16;
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            u32x4 b[NP];
#pragma unroll
            for (int q = 0; q < NP; ++q) b[q] = *(const u32x4*)(bb + q * kPiece + c * 512);
            if constexpr (NP == 1) {
                mm(a[j][0], b[0], acc[c]);
            } else {                                    // six of the nine partial products, the smallest first
                mm(a[j][2], b[0], acc[c]);
                mm(a[j][0], b[2], acc[c]);
                mm(a[j][1], b[1], acc[c]);
                mm(a[j][1], b[0], acc[c]);
                mm(a[j][0], b[1], acc[c]);
                mm(a[j][0], b[0], acc[c]);
            }
        }
    };

    // Per round r: the raw registers hold round r+1 (in flight), LDS buffer r & 1 round r.  K group 0 is multiplied, round
    // r+1 parked in the other buffer (the barrier that ended round r-1 says nobody reads it), round r+2 requested, then
    // the other K groups.  A is requested KG-1 groups ahead, so the wait for an A that was requested after round r+2's
    // planes comes a round later.  The last two rounds are written out: no load is conditional inside the loop (a wait
    // behind a branch that may have issued loads has to assume it did not).  Requesting B two rounds and A three K groups
    // further ahead costs the registers of the third workgroup per CU and is slower (channel-expanding layer, forward, f32 94 us
    // against 86, bf16 64 against 46).
    auto body = [&](int r, auto ISSUE, auto COMMIT) {
        const int buf = r & 1;
        auto step = [&](auto J) {
            constexpr int j = decltype(J)::value;
            issue_a(std::integral_constant<int, (j + KG - 1) % KG>{});
            compute(J, r * KG + j, buf);
            if constexpr (j == 0 && decltype(COMMIT)::value) {
                commit_b(buf ^ 1);
                if constexpr (decltype(ISSUE)::value) issue_b(r + 2);
            }
        };
        step(std::integral_constant<int, 0>{});
        step(std::integral_constant<int, 1>{});
        if constexpr (KG == 4) {
            step(std::integral_constant<int, 2>{});
            step(std::integral_constant<int, 3>{});
        }
        __syncthreads();
    };
    const std::true_type yes;
    const std::false_type no;
    __syncthreads();                                    // the table is complete
    issue_b(0);
    issue_a(std::integral_constant<int, 0>{});
    if constexpr (KG == 4) {
        issue_a(std::integral_constant<int, 1>{});
        issue_a(std::integral_constant<int, 2>{});
    }
    commit_b(0);
    if (nround > 1) issue_b(1);
    __syncthreads();
    int r = 0;
    for (; r + 2 < nround; ++r) body(r, yes, yes);
    if (r + 1 < nround) body(r++, no, yes);
    body(r, no, no);

    // ---- store: accumulator register v holds tile row 8*(v/4) + 4*h + v%4, columns CT*f .. CT*f + CT-1 of the tile ----
    const uint32_t u = (uint32_t)ct * 32u + (uint32_t)f;
    const bool live = u < (uint32_t)T.q.count;
    uint32_t n, p;
    column_of_group(live ? u : 0u, T.q, n, p);
    const uint32_t step = (uint32_t)P.HW * ES, ob = (n * (uint32_t)drows * (uint32_t)P.HW + p) * ES;
    const int row0 = (ng * kTiles + wave) * 32;
    int plane = row0 + f < T.rows ? row0 + f : -1;      // output plane of tile row f
    if (FWD && plane >= 0) plane = filter_of(T.b, plane / T.b.F, plane % T.b.F, P.Cout);
    int prow[16];                                       // requested together: one by one each would wait for its exchange
#pragma unroll
    for (int v = 0; v < 16; ++v) prow[v] = __shfl(plane, 8 * (v >> 2) + 4 * h + (v & 3), 64);
    auto store_row = [&](int v) {
        bvec o;
#pragma unroll
        for (int c = 0; c < CT; ++c) o[c] = from_f32<T_>(acc[c][v]);
        __builtin_nontemporal_store(o, (bvec*)((char*)out + (ob + (uint32_t)prow[v] * step)));   // written once, never re-read here
    };
    if (__all((int)(live && plane >= 0))) {             // a whole tile: no row and no column is asked for
#pragma unroll
        for (int v = 0; v < 16; ++v) store_row(v);
    } else {
#pragma unroll
        for (int v = 0; v < 16; ++v)
            if (prow[v] >= 0 && live) store_row(v);
    }
}

constexpr int lds_bytes(int es, int ct) { return 2 * (es == 2 ? 4 * 2 * 32 * ct * 16 : 3 * 2 * 2 * 32 * ct * 16); }

template <bool FWD>
inline Packed make_packed(const Problem& p, int es, int CT)
{
    Packed t;
    t.b = make_band(p);
    t.rows = FWD ? t.b.P * t.b.F : p.Cin;
    t.NG = (t.rows + 127) / 128;
    t.KG = es == 2 ? 4 : 2;
    int longest = 1;
    for (int ng = 0; ng < t.NG; ++ng) {
        int first, len;
        walk_of<FWD>(p, t.b, t.rows, ng, first, len);
        longest = len > longest ? len : longest;
    }
    t.nround = (longest + 16 * t.KG - 1) / (16 * t.KG);
    t.q = column_groups(p, CT);
    t.deal = make_deal((t.q.count + 31) / 32, t.NG);
    t.tab_group = (uint32_t)(t.nround * 16 * t.KG);
    const long long np = es == 2 ? 1 : 3, nkg = (long long)t.nround * t.KG;
    long long at = (long long)t.NG * t.tab_group * 4;
    t.act_at = (uint32_t)at;
    at = (at + t.NG * kTiles * kMaxGroups + 1023) / 1024 * 1024;
    t.a_at = (uint32_t)at;
    at += (t.NG * nkg + t.KG) * kTiles * np * 1024;   // slack of one round: A is requested ahead of its use
    t.bytes = (size_t)at;
    return t;
}

// Plane values the kernels without a workspace fetch for a layer, NQ * (sum over their tiles of the tile's span): what
// sharing them saves.  again: over the values there are.
template <bool FWD>
inline double fetches_without_sharing(const Problem& p, const Band& b, double* again)
{
    double per_column;
    if (FWD) {
        int ti = 1;
        while (2 * ti <= b.F && 2 * ti <= 32) ti *= 2;
        const int tm = 32 / ti < b.P ? 32 / ti : b.P;
        const long long tiles = (long long)((b.F + ti - 1) / ti) * ((b.P + tm - 1) / tm);
        per_column = (double)tiles * (p.L + (double)b.g * (tm - 1));
    } else {
        per_column = (double)((p.Cin + 31) / 32) * ((p.L + 31) / b.g + 1) * b.F;
    }
    *again = per_column / (FWD ? p.Cin : p.Cout);
    return per_column * (double)p.NQ;
}

// Windows that start off multiples of 4 channels, or planes that are not a multiple of 4 pixels: where the kernels without
// sharing lose most (scalar weight loads, unaligned plane loads).
inline bool uneven(const Problem& p, const Band& b) { return b.g % 4 != 0 || p.L % 4 != 0 || p.HW % 4 != 0; }

// Pixels per lane and plane this path takes the layer with, 0 where it cannot.
template <bool FWD>
inline int tile_width(const Problem& p, int es)
{
    if (FWD ? !forward_mfma_eligible(p) : !backward_input_mfma_eligible(p)) return 0;
    if (p.HW < 4) return 0;
    const Band b = make_band(p);
    if (4ll * b.P * b.F > 5ll * p.Cout) return 0;           // few filters on many starts: too many empty rows
    const long long rows = FWD ? (long long)b.P * b.F : p.Cin;
    const long long wide = (column_groups(p, 4).count + 31) / 32 * ((rows + 127) / 128);
    // 64 instead of 128 columns where the wide tiles do not give every CU one and a half workgroups (grad-input of the
    // 7x7 layer: 100 workgroups of 128 columns 44 us, 200 of 64 30 us)
    const int ct = wide < 384 ? 2 : 4;
    const Packed t = make_packed<FWD>(p, es, ct);
    return t.nround * t.KG <= kMaxGroups && t.bytes <= (1u << 28) && (t.q.count + 31) / 32 * t.NG < (1 << 28) ? ct : 0;
}

// tile_width where the pass on its own is faster this way, else 0.
//
// The packing launch costs 4 to 5 us, so the path is for layers whose tiles fetch the same planes many times.  Measured
// against the kernels that need no workspace, forward / grad-input, us (30 drawn layers besides):
//   128 x 128 -> 512, 32x32, cg 2, co 0.33   f32 118 -> 86 / 116 -> 93     bf16 100 -> 46 / 63 -> 38
//   64 x 512 -> 1024, 7x7, cg 2, co 0.33     f32 31 -> 23 / 25 -> 30       bf16 19 -> 16 / 18 -> 19
//   128 x 256 -> 256, 16x16, cg 1            f32 31 -> 31 / 35 -> 32       bf16 20 -> 17 / 22 -> 17
//   the same, cg 2                           f32 22 -> 24 / 23 -> 25       bf16 13 -> 15 / 14 -> 15
//   225 x 320 -> 160, 28x28, cg 4, co 0      f32 88 -> 124 (every plane fetched twice only) / 88 -> 73
// The others lose most on uneven layers and, forward, where a tile's window starts differ (`banded`).
template <bool FWD>
inline int choose(const Problem& p, int es)
{
    const int ct = tile_width<FWD>(p, es);
    if (!ct) return 0;
    const Band b = make_band(p);
    // weights packed once per call: with more bytes than half of x and y hold (few columns, many weights) they are what the pass
    // moves (4 x 2048 -> 2048 on 7x7, cg 1: forward f32 36 -> 65, bf16 22 -> 43, grad-input bf16 29 -> 45; 16 x 768 -> 1533 on 7x7: 30 -> 31, 18 -> 22)
    if (2 * (long long)make_packed<FWD>(p, es, ct).bytes > (long long)(p.Cin + p.Cout) * p.NQ * es) return 0;
    double again;
    const double fetches = fetches_without_sharing<FWD>(p, b, &again);
    const bool odd = uneven(p, b), banded = FWD && b.F < 32 && b.P > 1;
    // Layers of whole groups of 4 pixels and weights and one window per tile, forward: the kernels without a workspace lose least
    // there (fp32 has forward_shared32), so it counts how much longer the row groups' walks are than their windows, and whether the
    // rows fill their groups: where they do not, the others' tiles of 32 filters have empty rows as well.  Null / packed over 7330 fp32
    // and 11415 bf16 layers from 2.5 fetches and 30e6 on, geometric mean: of those taken here 1.17 and 1.09, of those left 1.00 and 0.89.  fp32 whose
    // walks are long is left to forward_shared32 where that shares nearly all four tiles' planes (0.96: 141 x 800 -> 800 on 12x12, cg 4 62 us
    // and 75); bf16 that fills its groups is taken from 7 fetches on only (256 -> 1088 .. 3328 from 70e6 0.5 to 0.9).
    if (FWD && !odd && !banded && (es == 2 || p.L < 300)) {
        double walks = 0;
        const int rows = b.P * b.F, groups = (rows + 127) / 128;
        int longest = 0;
        for (int ng = 0; ng < groups; ++ng) {
            int first, len;
            walk_of<true>(p, b, rows, ng, first, len);
            walks += len;
            longest = len > longest ? len : longest;
        }
        const double longer = walks * 128 / ((double)rows * p.L);
        if (es == 2) {
            if (again >= 7.0 && fetches >= (longer < 1.05 ? 60e6 : 80e6)) return ct;
            const bool partial = 1000ll * rows <= 976ll * 128 * groups;
            return partial && again >= 3.0 && fetches >= 55e6 && (b.P <= 2 || p.L > 236 || fetches >= 114e6) ? ct : 0;
        }
        if (longest > 300 && forward_shared_gain(p) >= 3.4) return 0;
        return (again >= 5.0 && longer < 1.2 && fetches >= 60e6) || (again >= 7.0 && fetches >= 120e6) ? ct : 0;
    }
    if (es == 2) return again >= 3.0 && fetches >= (odd ? 20e6 : 55e6) ? ct : 0;
    if (FWD) return again >= 3.0 && fetches >= (odd || banded ? 25e6 : 60e6) ? ct : 0;
    return fetches >= (odd ? 80e6 : 110e6) && (again >= 5.0 || fetches >= 150e6) ? ct : 0;
}

}  // namespace packed

}  // namespace scc
