// Forward of a DW + SCC block in one kernel for layers with few columns (a network's later blocks, small batches):
//
//   z[n,a,m,q] = sum_{i,j<3} kdw[a,i,j] * x[n,a, s*m+i-1, s*q+j-1]      (pixels outside the H x W map count as zero)
//   y[n,k,p]   = sum_{j<L}  w[k,j] * z[n,(s_k+j) mod Cin,p]             (Section 4.2, output-centric forward)
//
// Such a layer is bound by latencies: the two stages are two launches of which each mostly waits for its first operands, and the
// kernel that computes z of ALL channels once per column tile (scc_dw_fwd.hip) has too few column tiles to fill the chip.  Here a
// workgroup owns 32*CP columns and TF tiles of 32 filters that share their windows (scc_band.h), so there are ntiles/TF times as
// many workgroups, and each computes z only for the channels those windows reach; the workgroups of a column tile recompute
// it, 36 multiply-adds per 4 values against the launch and the round trip through memory that this saves.  What bounds it then is
// the instructions of one wavefront from end to end (about 1300: a wavefront alone on a SIMD issues one in five cycles), so
// the maps are those whose stencils need no neighbouring lanes, and the windows those read in whole groups of four.
//
// The wavefronts (four, or eight: see the launcher) split the contraction: each walks its share of the span in rounds of 16*KR channels (KR*CP = 4), for
// which a lane computes 8 channels of 4 consecutive pixels (a round is exactly 64 such items), cuts them into bf16 pieces (fp32) or
// rounds them to bf16 (bf16, as the two stages do) and parks them in the wavefront's own LDS in the matrix instruction's operand
// layout; no barrier.  The partial tiles are added through LDS in wavefront order, an equal share of the rows by each.
//
// MFMA column f of column group c is slot 32*c + f of the tile, and slot i*(8*CP) + g holds pixel i of group g: phase 1's lanes then
// write 16 consecutive bytes each, and the matrix instruction's lanes read them the same way.
#include "scc_band.h"
#include "scc_common.h"
#include "scc_dw_strip.h"

#include <type_traits>

namespace scc {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct FewTiling {
    Band b;
    int lTI, TM;    // filter tile = TM window starts x 2^lTI filters per start
    int IB;         // tiles along i
    int GM;         // workgroups per column tile and window group: ceil(IB / TF)
    int FG;         // workgroups per column tile: GM * ceil(P / TM)
    int U;          // channels a tile spans: L + g * (TM - 1)
    Deal deal;      // (column tile, filter group)
};

// LDS of a wavefront: a round's pieces and taps (binary32), then its partial tiles in their place.
constexpr int few_block_bytes(int cp, int tf, int parts)
{
    const int kr = 4 / cp, round = parts * 2 * kr * 32 * cp * 16 + 16 * kr * 9 * 4, sum = tf * cp * 16 * 64 * 4;
    return round > sum ? round : sum;
}

enum { kMap2, kMap4 };   // output maps of 2 x 2, rows of 4: a lane's 4 pixels have no neighbours beside them

// WV: wavefronts of a workgroup, 4 or 8
template <typename T_, int S, int MAP, int CP, int TF, int WV>
__global__ __launch_bounds__(64 * WV, 2) void dw_scc_forward_few(const T_* __restrict__ x, const T_* __restrict__ kdw,
                                                          const T_* __restrict__ w, T_* __restrict__ y, Problem P, DwGeom G,
                                                          FewTiling T)
{
    constexpr int KR = 4 / CP;                  // groups of 16 channels per round
    constexpr int kParts = sizeof(T_) == 4 ? 3 : 1;
    constexpr int TP = 32 * CP;                 // columns
    constexpr int kPartB = 2 * KR * TP * 16;    // one piece of a round: [8 channels][slot][8 values]
    constexpr int kBlockB = few_block_bytes(CP, TF, kParts);   // a wavefront's
    extern __shared__ __attribute__((aligned(16))) char lds[];     // WV * kBlockB
    typedef T_ w4 __attribute__((ext_vector_type(4), aligned(sizeof(T_))));

    int ct, fg;
    if (!dealt<false>(T.deal, (int)blockIdx.x, ct, fg)) return;
    const int mb = fg / T.GM, ib0 = (fg - mb * T.GM) * TF;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63, f = lane & 31, h = lane >> 5;
    char* mine = lds + wave * kBlockB;
    float* taps = (float*)(mine + kParts * kPartB);

    // the span, on the unwrapped channel axis, in groups of 16; this wavefront's are [k0, k1)
    const int c0 = T.b.g * mb * T.TM, cb = c0 & ~15;
    const int KG = (c0 + T.U - cb + 15) >> 4, KGs = (KG + WV - 1) / WV;
    const int k0 = wave * KGs, k1 = k0 + KGs < KG ? k0 + KGs : KG;

    // ---- A side: this lane's filters ----
    const int mi = f >> T.lTI, m = mb * T.TM + mi;
    const int sf = T.b.g * m;
    const int r = (int)(((uint32_t)m * (uint32_t)T.b.inv) % (uint32_t)T.b.P);   // P < 65536
    int kf[TF];
#pragma unroll
    for (int t = 0; t < TF; ++t) {
        const int i = ((ib0 + t) << T.lTI) + (f & ((1 << T.lTI) - 1));
        const int k = r + T.b.P * i;
        kf[t] = (mi < T.TM && m < T.b.P && ib0 + t < T.IB && k < P.Cout) ? k : -1;
    }
    // the lane's 8 weights of group kg, zero outside the filter's window
    auto load_a = [&](int kg, T_ (&a)[TF][8], uint32_t (&in)[TF]) {
        const int j0 = cb + 16 * kg + 8 * h - sf;
#pragma unroll
        for (int t = 0; t < TF; ++t) {
            const T_* row = w + (size_t)(kf[t] >= 0 ? kf[t] : 0) * P.L;
            in[t] = 0;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int j = j0 + 4 * q;
                const bool ok = kf[t] >= 0 && j >= 0 && j < P.L;
                const w4 v = *(const w4*)(row + (ok ? j : 0));
#pragma unroll
                for (int e = 0; e < 4; ++e) a[t][4 * q + e] = v[e];
                in[t] |= ok ? 0xfu << (4 * q) : 0u;
            }
        }
    };

    // ---- B side: this lane's item of phase 1: 8 channels (group chg of the round's) of column group grp ----
    const int chg = lane / (8 * CP), grp = lane % (8 * CP);
    const uint32_t quads = (uint32_t)P.HW / 4;
    const uint32_t qa = (uint32_t)ct * (8 * CP) + (uint32_t)grp;
    const uint32_t qs = qa < (uint32_t)P.N * quads ? qa : 0u;     // groups past the end read group 0; nothing of them is stored
    const uint32_t n = qs / quads, p4 = qs - n * quads;
    const int r0 = MAP == kMap2 ? 0 : (int)p4;                    // the group's output row
    const size_t HWi = (size_t)G.H * G.W;
    const T_* xn = x + (size_t)n * P.Cin * HWi + (size_t)(S * r0) * G.W;
    const uint32_t rowmask = dw::strip_rowmask<S, 1>(r0, G.Ho);

    // Phase 1 fetches the pixels of kBatch channels, all rows of their stencils, before it computes any: left to itself the
    // compiler takes one channel after the other, a memory latency each.
    constexpr int kBatch = S == 1 ? 8 : 4;
    constexpr int kRows = MAP == kMap2 ? S : 3;       // 2 x 2 maps: S loads of 4 or 8 pixels are the whole input map
    typedef T_ row_t __attribute__((ext_vector_type(4 * S), aligned(sizeof(T_))));
    auto fetch = [&](const T_* xc, row_t (&raw)[kRows]) {
#pragma unroll
        for (int t = 0; t < kRows; ++t) {
            if constexpr (MAP == kMap2)
                raw[t] = *(const row_t*)(xc + 4 * S * t);
            else
                raw[t] = *(const row_t*)((rowmask >> t) & 1u ? xc + (t - 1) * G.W : xc);   // rows outside: any address inside
        }
    };
    // z of one channel at the lane's 4 pixels from those rows
    auto stencil = [&](const row_t (&raw)[kRows], const float* k9, float (&z)[4]) {
        float k[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) k[i] = k9[i];
#pragma unroll
        for (int o = 0; o < 4; ++o) z[o] = 0.f;
        if constexpr (MAP == kMap2) {
            float v[2 * S][2 * S];
#pragma unroll
            for (int e = 0; e < 4 * S * S; ++e) v[e / (2 * S)][e % (2 * S)] = to_f32((T_)raw[e / (4 * S)][e % (4 * S)]);
#pragma unroll
            for (int o = 0; o < 4; ++o)
#pragma unroll
                for (int i = 0; i < 3; ++i)
#pragma unroll
                    for (int j = 0; j < 3; ++j) {
                        const int rr = S * (o / 2) + i - 1, cc = S * (o % 2) + j - 1;
                        if (rr >= 0 && rr < 2 * S && cc >= 0 && cc < 2 * S) z[o] += k[3 * i + j] * v[rr][cc];
                    }
        } else {
#pragma unroll
            for (int t = 0; t < 3; ++t) {
                const bool ok = (rowmask >> t) & 1u;
                float v[4 * S + 2];
#pragma unroll
                for (int e = 0; e < 4 * S; ++e) v[1 + e] = ok ? to_f32((T_)raw[t][e]) : 0.f;
                v[0] = v[4 * S + 1] = 0.f;            // the map ends on both sides
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 3; ++j) z[i] += k[3 * t + j] * v[S * i + j];
            }
        }
    };

    // between a wavefront's writes to its own LDS and its reads of other lanes' values: no instruction, the wavefront's LDS
    // accesses are in order as they are issued; the compiler keeps them so
    auto parked = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };

    f32x16 acc[TF][CP];
#pragma unroll
    for (int t = 0; t < TF; ++t)
#pragma unroll
        for (int c = 0; c < CP; ++c)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[t][c][v] = 0.f;

    T_ a[2][TF][8];
    uint32_t in[2][TF];
    if (k0 < k1) load_a(k0, a[0], in[0]);
    for (int kr = k0; kr < k1; kr += KR) {
        const int ch0 = (cb + 16 * kr) % P.Cin;    // the round's first channel; a round wraps at most once (Cin >= 64)
        // taps of the round's channels: consecutive in memory, fetched once per wavefront (channel groups past the span's end
        // are fetched on the circle as well and their z is not read)
        constexpr int kTaps = 16 * KR * 9, kTapLoads = (kTaps + 63) / 64;
        T_ tv[kTapLoads];
#pragma unroll
        for (int i = 0; i < kTapLoads; ++i) {
            uint32_t e = (uint32_t)ch0 * 9u + (uint32_t)(64 * i + lane < kTaps ? 64 * i + lane : kTaps - 1);
            e -= e >= 9u * (uint32_t)P.Cin ? 9u * (uint32_t)P.Cin : 0u;
            tv[i] = kdw[e];
        }
        {
            int c = ch0 + 8 * chg;        // a multiple of 8, as Cin is of 16: its 8 channels do not straddle the wrap
            c -= c >= P.Cin ? P.Cin : 0;
            const T_* xc = xn + (size_t)c * HWi;
            float z[8][4];
#pragma unroll
            for (int e0 = 0; e0 < 8; e0 += kBatch) {
                row_t raw[kBatch][kRows];
#pragma unroll
                for (int e = 0; e < kBatch; ++e) fetch(xc + (size_t)(e0 + e) * HWi, raw[e]);
                __builtin_amdgcn_sched_barrier(0);
                if (e0 == 0) {
#pragma unroll
                    for (int i = 0; i < kTapLoads; ++i)
                        if (64 * i + lane < kTaps) taps[64 * i + lane] = to_f32(tv[i]);
                    parked();
                }
#pragma unroll
                for (int e = 0; e < kBatch; ++e)
                    stencil(raw[e], taps + (8 * chg + e0 + e) * 9, z[e0 + e]);
            }
            char* dst = mine + (chg * TP + grp) * 16;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if constexpr (sizeof(T_) == 4) {
                    uint32_t hi[4], mid[4], lo[4];
                    split3<8>([&](int e) { return z[e][i]; }, hi, mid, lo);
                    *(u32x4*)(dst + i * (8 * CP) * 16) = u32x4{hi[0], hi[1], hi[2], hi[3]};
                    *(u32x4*)(dst + kPartB + i * (8 * CP) * 16) = u32x4{mid[0], mid[1], mid[2], mid[3]};
                    *(u32x4*)(dst + 2 * kPartB + i * (8 * CP) * 16) = u32x4{lo[0], lo[1], lo[2], lo[3]};
                } else {
                    u32x4 q;
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        q[e] = (uint32_t)from_f32<T_>(z[2 * e][i]) | ((uint32_t)from_f32<T_>(z[2 * e + 1][i]) << 16);
                    *(u32x4*)(dst + i * (8 * CP) * 16) = q;
                }
            }
        }
        parked();
#pragma unroll
        for (int g = 0; g < KR; ++g) {
            const int kg = kr + g;
            if (kg >= k1) break;                   // uniform over the wavefront
            // the next group's weights are requested before this one's are used (past the end: read and not used)
            load_a(kg + 1, a[(g + 1) & 1], in[(g + 1) & 1]);
            uint32_t b[CP][kParts][4];
#pragma unroll
            for (int c = 0; c < CP; ++c)
#pragma unroll
                for (int q = 0; q < kParts; ++q) {
                    const u32x4 v = *(const u32x4*)(mine + q * kPartB + ((2 * g + h) * TP + 32 * c + f) * 16);
#pragma unroll
                    for (int e = 0; e < 4; ++e) b[c][q][e] = v[e];
                }
#pragma unroll
            for (int t = 0; t < TF; ++t) {
                const T_(&at)[8] = a[g & 1][t];
                const uint32_t am = in[g & 1][t];
                if constexpr (sizeof(T_) == 4) {
                    uint32_t ah[4], ai[4], al[4];
                    split3<8>([&](int e) { return (am >> e) & 1u ? at[e] : 0.f; }, ah, ai, al);
#pragma unroll
                    for (int c = 0; c < CP; ++c) {
                        acc[t][c] = mfma_bf16<8>(al, b[c][0], acc[t][c]);
                        acc[t][c] = mfma_bf16<8>(ah, b[c][2], acc[t][c]);
                        acc[t][c] = mfma_bf16<8>(ai, b[c][1], acc[t][c]);
                        acc[t][c] = mfma_bf16<8>(ai, b[c][0], acc[t][c]);
                        acc[t][c] = mfma_bf16<8>(ah, b[c][1], acc[t][c]);
                        acc[t][c] = mfma_bf16<8>(ah, b[c][0], acc[t][c]);
                    }
                } else {
                    uint32_t ap[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        ap[e] = ((am >> (2 * e)) & 1u ? (uint32_t)at[2 * e] : 0u) |
                                (((am >> (2 * e + 1)) & 1u ? (uint32_t)at[2 * e + 1] : 0u) << 16);
#pragma unroll
                    for (int c = 0; c < CP; ++c) acc[t][c] = mfma_bf16<8>(ap, b[c][0], acc[t][c]);
                }
            }
        }
        parked();
        if (KR & 1) {                              // the next round starts at the other buffer's place
#pragma unroll
            for (int t = 0; t < TF; ++t) {
                in[0][t] = in[1][t];
#pragma unroll
                for (int e = 0; e < 8; ++e) a[0][t][e] = a[1][t][e];
            }
        }
    }

    // ---- the wavefronts' partial tiles, added in wavefront order; wavefront v takes RW accumulator registers from RW*v on (tile row
    // 8*(r/4) + 4h + r%4 for register r) ----
    constexpr int RW = 16 / WV;
    float* part = (float*)mine + lane;
#pragma unroll
    for (int t = 0; t < TF; ++t)
#pragma unroll
        for (int c = 0; c < CP; ++c)
#pragma unroll
            for (int v = 0; v < 16; ++v) part[((t * CP + c) * 16 + v) * 64] = acc[t][c][v];
    __syncthreads();
    const float* sum = (const float*)lds + lane;
    constexpr int kStep = kBlockB / 4;
#pragma unroll
    for (int t = 0; t < TF; ++t) {
        float o[CP][RW];
#pragma unroll
        for (int c = 0; c < CP; ++c)
#pragma unroll
            for (int v = 0; v < RW; ++v) {
                const float* s = sum + ((t * CP + c) * 16 + RW * wave + v) * 64;
                o[c][v] = s[0];
#pragma unroll
                for (int u = 1; u < WV; ++u) o[c][v] += s[u * kStep];
            }
#pragma unroll
        for (int v = 0; v < RW; ++v) {
            const int reg = RW * wave + v;
            const int k = __shfl(kf[t], 8 * (reg >> 2) + 4 * h + (reg & 3), 64);
#pragma unroll
            for (int c = 0; c < CP; ++c) {
                const int sl = 32 * c + f, gq = sl % (8 * CP), i = sl / (8 * CP);
                const uint32_t q = (uint32_t)ct * (8 * CP) + (uint32_t)gq;
                if (k < 0 || q >= (uint32_t)P.N * quads) continue;
                const uint32_t nn = q / quads, px = (q - nn * quads) * 4 + (uint32_t)i;
                __builtin_nontemporal_store(from_f32<T_>(o[c][v]), y + ((size_t)nn * P.Cout + k) * P.HW + px);
            }
        }
    }
}

FewTiling few_tiling(const Problem& p, int cp, int tf)
{
    FewTiling t;
    t.b = make_band(p);
    t.lTI = 0;
    while (t.lTI < 5 && 2 << t.lTI <= t.b.F) ++t.lTI;
    const int TI = 1 << t.lTI;
    t.TM = 32 / TI < t.b.P ? 32 / TI : t.b.P;
    t.IB = (t.b.F + TI - 1) / TI;
    t.GM = (t.IB + tf - 1) / tf;
    t.FG = t.GM * ((t.b.P + t.TM - 1) / t.TM);
    t.U = p.L + t.b.g * (t.TM - 1);
    const long long nct = (p.NQ + 32 * cp - 1) / (32 * cp);
    t.deal = in_eighths(make_deal(nct, t.FG));
    return t;
}

// Column groups of 32 per workgroup: 1, 2 or 4, as many as leave a wavefront whole rounds of its quarter of the span.
int few_cp(const FewTiling& t)
{
    const int quarter = ((t.U + 15) / 16 + 3) / 4;
    return quarter >= 4 ? 1 : quarter >= 2 ? 2 : 4;
}

}  // namespace

// Maps of rows of 4 or of 2 x 2 pixels, read at stride 1 or 2 from maps of exactly that many times their size; windows whose
// groups of four weights are wholly inside or outside a tile's groups of 16 channels; offsets that fit 32 bits.
bool dw_forward_few_eligible(const Problem& p, const DwGeom& g)
{
    const bool sized = (g.s == 1 || g.s == 2) && g.H == g.s * g.Ho && g.W == g.s * g.Wo;
    const bool map = g.Wo == 4 || (g.Wo == 2 && g.Ho == 2);
    const long long rows = p.Cin > p.Cout ? p.Cin : p.Cout;
    return sized && map && p.Cin % 16 == 0 && p.Cin >= 64 && p.Cin < 65536 && p.L % 4 == 0 && make_band(p).g % 4 == 0 &&
           (long long)p.NQ * rows < (1ll << 30) && (long long)p.Cout * p.L < (1ll << 30);
}

// How a layer is cut.  Two filter tiles per workgroup once one would make more than 768 workgroups of one column group: 128 x 512 -> 512 on
// 4x4 15.5 -> 12.1 us, 64 of them 8.8 -> 9.1; four tiles gain nothing more (12.8).  Eight wavefronts where four would walk their quarter of
// the span in more than one round and the chip holds all workgroups at once (one per CU): 16 x 1024 -> 1024 on 2x2, cg 2, 9.6 -> 8.3 us,
// bf16 9.4 -> 7.9; 16 x 512 -> 512 on 4x4, cg 1, 9.7 -> 7.8.
struct FewPlan {
    FewTiling t;
    int units;         // tiles of 32 filters x 32 columns
    int cp, tf, wv;    // column groups, filter tiles, wavefronts of a workgroup
    int rounds;        // of channels, of one wavefront
};

static FewPlan few_plan(const Problem& p)
{
    FewPlan f;
    f.t = few_tiling(p, 1, 1);
    f.units = f.t.deal.total;
    f.cp = few_cp(f.t);
    f.tf = f.cp <= 2 && f.units > 768 ? 2 : 1;
    f.t = few_tiling(p, f.cp, f.tf);
    f.wv = f.cp == 1 && f.tf == 1 && f.t.U > 256 && f.t.deal.total <= 256 ? 8 : 4;
    // a tile starts g * TM channels behind the one before it: at any multiple of that step's common factor with 16 into a group
    int align = 16;
    while (f.t.TM < f.t.b.P && (f.t.b.g * f.t.TM) % align != 0) align /= 2;
    const int all = (f.t.U + 16 - align + 15) / 16, own = (all + f.wv - 1) / f.wv, kr = 4 / f.cp;      // groups of 16: a tile's, a wavefront's, a round's
    f.rounds = (own + kr - 1) / kr;
    return f;
}

// Against the two stages, of which the second reaches its tiled kernels from 64 columns up; below, this kernel is as fast or faster over 1338
// layers, three times as fast on average (one image of 512 -> 512 on 4x4 43 -> 6.4 us).  From 64 up its time goes with the rounds that a CU
// walks one after another: rounds of a wavefront x generations of 256 workgroups, wider workgroups somewhat longer ones (3 + column groups x
// filter tiles quarters of the narrowest's).  Left to the two stages besides, over 46814 layers of up to 1100 tiles, two stages / this kernel, geometric mean: maps
// of one row of 4, where a lane's pixels share a cache line with no neighbour's, 0.86; a second generation at stride 2 in fp32 0.91, or of two column
// groups by two filter tiles 0.96; bf16, whose second stage is cheaper, in more than one round 0.94 (from 2x2 to 2x2 1.14); fp32 from 4x4 to 2x2 on
// two column groups 1.00 (0.66 at worst).
// Those taken: stride 1, rows of 4, fp32 1.20 (one in 50 below 0.94), bf16 1.14 (0.90); 2x2 maps, fp32 1.27 (0.96), bf16 1.25 (0.89); stride 2, where every tile
// recomputes from four times the input, rows of 4, fp32 1.13 (0.89), bf16 1.13 (0.90); 2x2, fp32 1.16 (0.88), bf16 1.10 (0.85).  Without the rules 2.5 times slower at
// worst (18 x 1984 -> 5948 on 4x4, cg 1: 46 -> 118).  us at the lines: 128 x 512 -> 512 on 4x4 13.2 -> 12.1, 128 x 1024 -> 1024 on 2x2 15.5 -> 14.9, left: 128 x 512 ->
// 1024 from 4x4 14.0 (16.0 here), 128 x 256 -> 512 from 8x8 11.8 (12.5), 18 x 608 -> 1216 on 1x4, cg 1, bf16 9.0 (17.6).
// Against the kernel that computes all channels once per tile of 64 columns, which a call without workspace would take (fp32, 2507 layers):
// median 2.5 times as fast, as few columns leave that one most of the chip idle; from 4096 columns up it can lose (291 x 64 -> 96 from 8x8 9.1 to 10.8).
bool dw_forward_few_preferred(const Problem& p, const DwGeom& g, int es, bool against_fused)
{
    if (!dw_forward_few_eligible(p, g)) return false;
    if (p.NQ < 64) return true;
    const FewPlan f = few_plan(p);
    if (f.units > 1100) return false;                                           // not measured above
    if (against_fused) return p.NQ < 4096;
    const bool planes = g.Wo == 2, second = f.t.deal.total > 256;
    if (!planes && g.Ho == 1) return false;
    if (second && f.cp == 2 && f.tf == 2) return false;
    if (es == 4 && g.s == 2 && (second || f.wv == 8 || (planes && f.cp == 2))) return false;
    if (es == 2 && !(planes && g.s == 1) && f.rounds > 1) return false;
    const long long width = f.cp == 1 ? 4 : 3 + f.cp * f.tf;
    const long long walked = width * f.rounds * (f.t.deal.total < 256 ? 256 : f.t.deal.total);
    return walked <= (g.s == 2 ? (es == 4 ? 1280 : 2048) : planes && f.cp == 1 ? 4096 : 2048);
}

template <typename T_>
hipError_t launch_dw_forward_few(const T_* x, const T_* kdw, const T_* w, T_* y, const Problem& p, const DwGeom& g,
                                 hipStream_t st)
{
    const FewPlan f = few_plan(p);
    using std::integral_constant;
    hipError_t e = hipSuccess;
    auto go = [&](auto s, auto map, auto c, auto tf, auto wv) {
        constexpr int S = decltype(s)::value, MAP = decltype(map)::value, CP = decltype(c)::value, TF = decltype(tf)::value;
        constexpr int WV = decltype(wv)::value, kLds = WV * few_block_bytes(CP, TF, sizeof(T_) == 4 ? 3 : 1);
        if constexpr (kLds > 64 * 1024) {
            // more than 64 KiB of LDS per workgroup has to be allowed once
            static const hipError_t allowed = hipFuncSetAttribute((const void*)dw_scc_forward_few<T_, S, MAP, CP, TF, WV>,
                                                                  hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
            e = allowed;
            if (e != hipSuccess) return;
        }
        dw_scc_forward_few<T_, S, MAP, CP, TF, WV><<<dim3(8u * (unsigned)f.t.deal.chunk), dim3(64 * WV), kLds, st>>>(x, kdw, w, y, p, g, f.t);
        e = hipGetLastError();
    };
    const integral_constant<int, 4> four;
    auto with_tf = [&](auto s, auto map, auto c) {
        if constexpr (decltype(c)::value <= 2)
            if (f.tf == 2) return go(s, map, c, integral_constant<int, 2>{}, four);
        if constexpr (decltype(c)::value == 1)
            if (f.wv == 8) return go(s, map, c, integral_constant<int, 1>{}, integral_constant<int, 8>{});
        go(s, map, c, integral_constant<int, 1>{}, four);
    };
    auto with_cp = [&](auto s, auto map) {
        f.cp == 1 ? with_tf(s, map, integral_constant<int, 1>{})
        : f.cp == 2 ? with_tf(s, map, integral_constant<int, 2>{}) : with_tf(s, map, integral_constant<int, 4>{});
    };
    auto with_map = [&](auto s) {
        g.Wo == 2 ? with_cp(s, integral_constant<int, kMap2>{}) : with_cp(s, integral_constant<int, kMap4>{});
    };
    g.s == 1 ? with_map(integral_constant<int, 1>{}) : with_map(integral_constant<int, 2>{});
    return e;
}

template hipError_t launch_dw_forward_few<float>(const float*, const float*, const float*, float*, const Problem&, const DwGeom&,
                                                 hipStream_t);
template hipError_t launch_dw_forward_few<bf16_t>(const bf16_t*, const bf16_t*, const bf16_t*, bf16_t*, const Problem&,
                                                  const DwGeom&, hipStream_t);

}  // namespace scc
