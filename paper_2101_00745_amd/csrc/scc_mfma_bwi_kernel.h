// Grad-input of SCC on the gfx950 matrix cores (bf16 matrix instructions with fp32 sums: directly for bf16
// tensors, on an exact three-way bf16 split of each value for fp32 tensors), as a per-input-channel gather.
//
// dx[n,c,p] = sum over filters k whose window covers c of w[k,(c-s_k) mod Cin] * dy[n,k,p]
// (Section 4.2, input-centric backward: every input-gradient element PULLS from the filters
// covering its channel, so nothing is accumulated with atomics).
//
// A tile is 32 consecutive input channels c0..c0+31 times 32*CT columns.  The filters that can
// cover any of those channels are the ones whose window start s lies in (c0-L, c0+31] on the
// channel circle; starts are the multiples g*m (see scc_band.h), so the contraction runs over
// the grid (mm, i): window m = mlo+mm, i-th filter of that window, k = r(m) + P*i.  The A
// operand of a K-slot is row k of the weight matrix read at consecutive positions by
// consecutive channels (one coalesced 128-byte read per half-wave), zero where the window
// does not reach the channel; the B operand is the plane dy[n,k,:].
#pragma once
#include "scc_band.h"
#include "scc_common.h"

#include <type_traits>

namespace scc {

namespace bwi {

typedef float f32x16 __attribute__((ext_vector_type(16)));

struct BwiTiling {
    Band b;
    int CB;   // channel blocks of 32
    int FG;     // workgroups per column tile = ceil(CB / 4)
    Deal deal;     // (column tile, group of workgroups that read its planes)
    int even;   // every window start has F filters and F is a multiple of a chunk: see the walk below
    Groups q;   // column groups of CT pixels
};

__device__ __forceinline__ int floor_div(int a, int b)  // b > 0
{
    const int q = a / b;
    return (a % b != 0 && a < 0) ? q - 1 : q;
}

// T_ is the storage type of dy, w, dx (float or bf16_t); arithmetic is binary32 either way.
// S wavefronts (1, 2 or 4) share one tile, each taking a slice of the (window, filter) slots; their partial
// tiles are added through LDS in slice order (layers with few columns and many covering filters).
// WPB wavefronts per workgroup: 4, or 8 (all channel blocks of a column tile on one CU, sharing its L1) for grids
// that fill the chip exactly once: see launch_split.
// Bytes of LDS in which the wavefronts that share a tile add their partial tiles (S > 1).
template <int CT, int S, int WPB>
constexpr size_t reduce_bytes() { return S > 1 ? (size_t)(WPB / S) * (S - 1) * CT * 16 * 64 * sizeof(float) : 0; }

// `shared_red`: LDS of at least reduce_bytes<CT, S, WPB>() that the caller provides for that sum (a kernel that
// holds dynamic LDS for other workgroups of its grid lends it); null: the body declares its own.  ALONE: the whole kernel is this body.
template <typename T_, int CT, int KC, int S, int WPB, bool LENT = false, bool ALONE = false>
__device__ __forceinline__ void backward_input_body(const T_* __restrict__ dy, const T_* __restrict__ w,
                                                    T_* __restrict__ dx, const Problem& P, const BwiTiling& T,
                                                    const int bid, float* shared_red = nullptr)
{
    typedef T_ bvec __attribute__((ext_vector_type(CT), aligned(sizeof(T_))));   // CT consecutive columns of one plane
    constexpr uint32_t ES = sizeof(T_);
    // Alone and with one column per lane: few columns, one generation of workgroups at most, and a tile's time is that of its
    // loads, chunk after chunk.  The compiler does not see that: with anything changed around it, it packs the bf16 of a chunk pair
    // by pair as they come, with one load in flight, or cuts binary32 values before it asks for the next.  HELD spells the order
    // out (below), and names all arguments here, so that they are fetched together.  Grad-input, us, left to itself -> so: 2 x 208
    // -> 832 on 16x16, cg 1, co 0.25, bf16 14.6 -> 6.9; 46 x 256 -> 1024 on 2x2, cg 2, co 0.25, bf16 8.1 -> 5.3; 1 x 736 -> 1472 on
    // 16x16, cg 4, co 0.33, f32 6.9 -> 6.1.  (Binary32 tiles of one wavefront, and wider ones, have the right order by themselves.)
    constexpr bool HELD = CT == 1 && ALONE && (ES == 2 || S > 1), WIDE = HELD && ES == 2;
    if constexpr (HELD)
        asm volatile("" ::"s"(T.deal.total), "s"(T.deal.inner), "s"(T.deal.chunk), "s"(T.deal.recip), "s"(T.b.g), "s"(T.b.P), "s"(T.b.inv),
                     "s"(T.b.F), "s"(T.CB), "s"(T.even), "s"(T.q.per), "s"(T.q.last), "s"((int)T.q.count), "s"(P.L), "s"(P.HW), "s"(P.Cin),
                     "s"(P.Cout));
    // bid is the workgroup's index in a launch whose first workgroup is a multiple of 8: bid % 8 names the XCD; the
    // channel blocks of a column tile, which re-read the same dy planes, share one and its L2
    int ct, fg;
    if (!dealt<!LENT && !HELD>(T.deal, bid, ct, fg)) return;          // the whole workgroup leaves
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int cb = fg * (WPB / S) + wave / S, split = wave % S;
    const bool tvalid = cb < T.CB;
    if (S == 1 && !tvalid) return;              // with S > 1 every wavefront has to reach the barrier

    const int lane = threadIdx.x & 63;
    const int f = lane & 31, h = lane >> 5;
    const int c0 = cb * 32;
    const int c = c0 + f;                       // this lane's input channel (A row)
    const bool cvalid = tvalid && c < P.Cin;
    // unwrapped window index range: g*m in [c0-L+1, c0+31]
    const int mlo = -floor_div(P.L - 1 - c0, T.b.g);   // ceil((c0-L+1)/g)
    const int M = floor_div(c0 + 31, T.b.g) - mlo + 1;  // window starts this block can see (>= 1)
    const char* wb = (const char*)w;
    const char* gb = (const char*)dy;

    const uint32_t u = (uint32_t)ct * 32u + (uint32_t)f;       // this lane's group of CT columns
    const bool live = u < (uint32_t)T.q.count;
    uint32_t gcol, dcol;
    {
        uint32_t n, p;
        column_of_group(live ? u : 0u, T.q, n, p);
        gcol = (n * (uint32_t)P.Cout * (uint32_t)P.HW + p) * ES;
        dcol = n * (uint32_t)P.Cin * (uint32_t)P.HW + p;
    }

    const uint32_t plane = (uint32_t)P.HW * ES;

    f32x16 acc[CT];
#pragma unroll
    for (int cc = 0; cc < CT; ++cc)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[cc][v] = 0.f;

    auto mma_chunk = [&](const T_ (&as)[KC], uint32_t am, const bvec (&bs)[KC]) {
        if constexpr (ES == 2) {
            // bf16 storage: the KC slots of a chunk are the K values of ONE bf16 matrix instruction per column
            // group (which K-slot a value takes does not matter as long as A and B agree); exact products
            uint32_t ap[KC / 2];
#pragma unroll
            for (int e = 0; e < KC / 2; ++e) {
                // am holds one bit per slot; with all of them equal (chunks of one window) a pair is kept or dropped as one
                if (T.even) {
                    ap[e] = am ? (uint32_t)as[2 * e] | ((uint32_t)as[2 * e + 1] << 16) : 0u;
                } else {
                    const uint32_t lo = (am >> (2 * e)) & 1u ? (uint32_t)as[2 * e] : 0u;
                    const uint32_t hi = (am >> (2 * e + 1)) & 1u ? (uint32_t)as[2 * e + 1] : 0u;
                    ap[e] = lo | (hi << 16);
                }
            }
#pragma unroll
            for (int cc = 0; cc < CT; ++cc) {
                uint32_t bp[KC / 2];
#pragma unroll
                for (int e = 0; e < KC / 2; ++e)
                    bp[e] = (uint32_t)(T_)bs[2 * e][cc] | ((uint32_t)(T_)bs[2 * e + 1][cc] << 16);
                acc[cc] = mfma_bf16<KC>(ap, bp, acc[cc]);
            }
        } else {
            // fp32 storage: exact three-way bf16 split of every operand, six of the nine partial products
            // (the dropped ones are below 2^-21 of the product), fp32 accumulation
            uint32_t ah[KC / 2], amd[KC / 2], al[KC / 2];
            split3<KC>([&](int e) { return (T.even ? am : (am >> e) & 1u) ? as[e] : 0.f; }, ah, amd, al);
#pragma unroll
            for (int cc = 0; cc < CT; ++cc) {
                uint32_t bh[KC / 2], bm[KC / 2], bl[KC / 2];
                split3<KC>([&](int e) { return bs[e][cc]; }, bh, bm, bl);
                acc[cc] = mfma_bf16<KC>(al, bh, acc[cc]);
                acc[cc] = mfma_bf16<KC>(ah, bl, acc[cc]);
                acc[cc] = mfma_bf16<KC>(amd, bm, acc[cc]);
                acc[cc] = mfma_bf16<KC>(amd, bh, acc[cc]);
                acc[cc] = mfma_bf16<KC>(ah, bm, acc[cc]);
                acc[cc] = mfma_bf16<KC>(ah, bh, acc[cc]);
            }
        }
    };

    // Software pipelined over an even number n of chunks, which load(a, in, b) requests one after the other.  HELD: nothing of a
    // chunk moves past the next one's loads; WIDE: its bf16 stay in a register each until they are multiplied.
    typedef std::conditional_t<WIDE, uint32_t, T_> aheld;
    typedef std::conditional_t<WIDE, uint32_t, bvec> bheld;
    typedef std::conditional_t<WIDE, T_, bvec> bmem;
    auto use_chunk = [&](const aheld (&ah)[KC], uint32_t am, const bheld (&bh)[KC]) __attribute__((always_inline)) {
        if constexpr (HELD) {
            __builtin_amdgcn_sched_barrier(0);
            T_ as[KC];
            bvec bs[KC];
#pragma unroll
            for (int e = 0; e < KC; ++e) {
                if constexpr (WIDE) {
                    as[e] = (T_)ah[e];
                    bs[e][0] = (T_)bh[e];
                } else {
                    as[e] = ah[e];
                    float v = bh[e][0];
                    asm volatile("" : "+v"(as[e]), "+v"(v));
                    bs[e][0] = v;
                }
            }
            mma_chunk(as, am, bs);
        } else {
            mma_chunk(ah, am, bh);
        }
    };
    auto pipeline = [&](int n, auto&& load) __attribute__((always_inline)) {
        aheld a0[KC], a1[KC];
        bheld b0[KC], b1[KC];
        uint32_t m0, m1;
        if (n <= 0) return;
        load(a0, m0, b0);
        for (int cix = 0; cix + 2 < n; cix += 2) {
            load(a1, m1, b1);
            use_chunk(a0, m0, b0);
            load(a0, m0, b0);
            use_chunk(a1, m1, b1);
        }
        load(a1, m1, b1);
        use_chunk(a0, m0, b0);
        use_chunk(a1, m1, b1);
    };
    // K-steps: each half-wave walks Uh (window, filter) slots; an even number of chunks
    const int Uh = ((M * T.b.F + 1) / 2 + 2 * KC - 1) / (2 * KC) * (2 * KC);
    const int Us = ((Uh + S - 1) / S + 2 * KC - 1) / (2 * KC) * (2 * KC);   // K-steps of one slice
    const int t0 = split * Us < Uh ? split * Us : Uh;                         // this wavefront's K-steps [t0, t1)
    const int t1 = !tvalid ? t0 : (t0 + Us < Uh ? t0 + Us : Uh);
    // K-slot state of this half-wave: slot u = h*Uh + t  <->  (mm, i) = (u / F, u % F)
    const int u0 = h * Uh + t0;
    int mm = u0 / T.b.F, i = u0 % T.b.F;
    int mw = (mlo + mm) % T.b.P;                 // window index on the circle
    if (mw < 0) mw += T.b.P;
    int r = (int)(((uint32_t)mw * (uint32_t)T.b.inv) % (uint32_t)T.b.P);   // residue class owning window mw
    int ju = c - T.b.g * (mlo + mm);             // position of channel c inside that window (unwrapped)
    // `step` filters further in the walk
    auto advance = [&](int step) {
        i += step;
        const bool nextw = (i == T.b.F);
        i = nextw ? 0 : i;
        mm += nextw ? 1 : 0;
        ju -= nextw ? T.b.g : 0;
        int rn = r + T.b.inv;                    // r(m+1) = r(m) + inv (mod P)
        rn = (rn >= T.b.P) ? rn - T.b.P : rn;
        r = nextw ? rn : r;
    };
    if (T.even) {
        // A chunk is KC filters of ONE window, P apart: one offset per lane and operand for all of them, and scalar bases that do
        // not change from chunk to chunk.  Taking every slot for itself (below) costs 25 vector instructions per slot, most of
        // what a bf16 tile executes: 226 per chunk of 4 matrix instructions (fp32: 345 of 24), 45 (fp32: 160) here; same
        // operands in the same order.
        const uint32_t wstep = (uint32_t)T.b.P * (uint32_t)P.L * ES, gstep = (uint32_t)T.b.P * plane;
        // WIDE: these bases in scalar registers, not added up again for every chunk
        typedef const __attribute__((address_space(1))) char* gptr;
        gptr wat[KC], gat[KC];
        if constexpr (WIDE) {
#pragma unroll
            for (int s = 0; s < KC; ++s) {
                wat[s] = (gptr)(wb + (size_t)(s * wstep));
                gat[s] = (gptr)(gb + (size_t)(s * gstep));
                asm("" : "+s"(wat[s]), "+s"(gat[s]));
            }
        }
        pipeline((t1 - t0) / KC, [&](aheld(&ad)[KC], uint32_t& am, bheld(&bd)[KC]) __attribute__((always_inline)) {
            const int k = mm < M ? r + T.b.P * i : 0;
            const bool in = (mm < M) & cvalid & (ju >= 0) & (ju < P.L);
            am = in ? 0xffffffffu : 0u;
            const uint32_t wofs = (uint32_t)(k * P.L + (in ? ju : 0)) * ES, gofs = gcol + (uint32_t)k * plane;
#pragma unroll
            for (int s = 0; s < KC; ++s) {
                if constexpr (WIDE) {
                    ad[s] = *(const __attribute__((address_space(1))) T_*)(wat[s] + wofs);
                    bd[s] = *(const __attribute__((address_space(1))) T_*)(gat[s] + gofs);
                } else {
                    ad[s] = *(const T_*)(wb + (size_t)(s * wstep) + wofs);
                    bd[s] = *(const bvec*)(gb + (size_t)(s * gstep) + gofs);
                }
            }
            advance(KC);
        });
    } else {
        pipeline((t1 - t0) / KC, [&](aheld(&ad)[KC], uint32_t& am, bheld(&bd)[KC]) {
            am = 0;
#pragma unroll
            for (int s = 0; s < KC; ++s) {
                const int k = r + T.b.P * i;
                // bitwise: short-circuit forms became branches with a load behind each
                const bool kvalid = (mm < M) & (k < P.Cout);
                const bool in = kvalid & cvalid & (ju >= 0) & (ju < P.L);
                const int at = k * P.L + ju;
                ad[s] = *(const T_*)(wb + (uint32_t)(in ? at : 0) * ES);
                am |= in ? (1u << s) : 0u;
                const uint32_t rowofs = (uint32_t)(kvalid ? k : 0) * plane;
                bd[s] = *(const bmem*)(gb + (uint32_t)(gcol + rowofs));
                advance(1);                      // next filter of this window, or the first filter of the next window
            }
        });
    }

    if constexpr (S > 1) {   // add the slices of each tile, in slice order, into the wavefront that took slice 0
        float* red;
        if constexpr (LENT) {
            red = shared_red;
        } else {
            __shared__ float own[(S > 1 ? (WPB / S) * (S - 1) : 1) * CT * 16 * 64];
            red = own;
        }
        float* mine = red + ((wave / S) * (S - 1) + (split - 1)) * (CT * 16 * 64) + lane;
        if (split > 0) {
#pragma unroll
            for (int cc = 0; cc < CT; ++cc)
#pragma unroll
                for (int v = 0; v < 16; ++v) mine[(cc * 16 + v) * 64] = acc[cc][v];
        }
        __syncthreads();
        if (split > 0 || !tvalid) return;
#pragma unroll
        for (int sp = 1; sp < S; ++sp) {
            const float* other = red + ((wave / S) * (S - 1) + (sp - 1)) * (CT * 16 * 64) + lane;
#pragma unroll
            for (int cc = 0; cc < CT; ++cc)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[cc][v] += other[(cc * 16 + v) * 64];
        }
    }

    // accumulator register v holds tile row 8*(v/4) + 4*h + v%4 (= channel c0 + that), column f
    const uint32_t dofs = (dcol + (uint32_t)(c0 + 4 * h) * (uint32_t)P.HW) * ES;
    auto store_row = [&](int v) {
        bvec o;
#pragma unroll
        for (int cc = 0; cc < CT; ++cc) o[cc] = from_f32<T_>(acc[cc][v]);
        __builtin_nontemporal_store(o, (bvec*)((char*)dx + (size_t)((uint32_t)(8 * (v >> 2) + (v & 3)) * plane) + dofs));  // written once, not re-read here
    };
    if (c0 + 32 <= P.Cin && __all((int)live)) {      // a whole tile: no row and no column is asked for
#pragma unroll
        for (int v = 0; v < 16; ++v) store_row(v);
    } else {
#pragma unroll
        for (int v = 0; v < 16; ++v)
            if (c0 + 8 * (v >> 2) + 4 * h + (v & 3) < P.Cin && live) store_row(v);
    }
}


// ---- host side: which variant of the body a layer takes, and its tiling -----------------------------------

template <int CT, int S, int WPB>
inline BwiTiling make_tiling(const Problem& p, long long* blocks)
{
    BwiTiling t;
    t.b = make_band(p);
    t.CB = (p.Cin + 31) / 32;
    t.even = t.b.F % 8 == 0 && p.Cout == t.b.P * t.b.F;
    t.q = column_groups(p, CT);
    const long long nct = (t.q.count + 31) / 32;
    t.FG = (t.CB * S + WPB - 1) / WPB;
    t.deal = make_deal(nct, t.FG);
    *blocks = (long long)8 * t.deal.chunk;
    return t;
}

// Calls f(CT, S, WPB, tiling, blocks) with the first three as std::integral_constant
// values: the variant backward_input_body<T_, CT, 8, S, WPB> that the layer takes, and its launch shape
// (blocks workgroups of WPB * 64 threads).
template <typename T_, typename F>
void select_backward_input(const Problem& p, F&& f)
{
    using std::integral_constant;
    // workgroups of 8 wavefronts (0.6 us faster at the metric layer; delaying half of them, which pays in the
    // forward, does not here): only for grids that fill the chip exactly once with two wavefronts per SIMD, fp32,
    // windows that start on multiples of 32 channels, and at most 16 flop per byte, the shapes it was measured on
    auto with_wpb = [&](auto ct, auto s) {
        constexpr int CT = decltype(ct)::value, S = decltype(s)::value;
        long long blocks = 0;
        if constexpr (sizeof(T_) == 4 && CT == 4 && S == 1) {
            const Band b = make_band(p);
            const long long cbs = (p.Cin + 31) / 32, nct = (column_groups(p, CT).count + 31) / 32, waves = nct * cbs;
            const bool once = waves >= 2048 && waves < 2048 + 256;
            const bool light = (long long)p.Cout * p.L <= 32ll * (p.Cin + p.Cout);
            if (b.g % 32 == 0 && p.Cin % 32 == 0 && cbs % 8 == 0 && once && light) {
                const BwiTiling t = make_tiling<CT, S, 8>(p, &blocks);
                f(ct, s, integral_constant<int, 8>{}, t, blocks);
                return;
            }
        }
        const BwiTiling t = make_tiling<CT, S, 4>(p, &blocks);
        f(ct, s, integral_constant<int, 4>{}, t, blocks);
    };
    // share a tile between 2 or 4 wavefronts while there are fewer than two wavefronts per SIMD and each slice
    // keeps at least 32 K-steps; a block of 32 channels sees about (L+31)/g windows of F filters each
    auto with_split = [&](auto ct, long long waves) {
        constexpr int CT = decltype(ct)::value;
        const Band b = make_band(p);
        const long long slots = ((long long)(p.L + 31) / b.g + 1) * b.F;
        int split = 1;
        while (split < 4 && waves * split < 2048 && slots / (4 * split) >= 32) split *= 2;
        if (split == 1)
            with_wpb(ct, integral_constant<int, 1>{});
        else if (split == 2)
            with_wpb(ct, integral_constant<int, 2>{});
        else
            with_wpb(ct, integral_constant<int, 4>{});
    };
    // columns per wavefront: 128 when that still gives every SIMD a wavefront, else 64 or 32; a plane has to hold at
    // least one group of columns
    constexpr long long kEnoughWaves = 1024;
    const long long blocks32 = (p.Cin + 31) / 32;
    auto waves = [&](int ct) { return (column_groups(p, ct).count + 31) / 32 * blocks32; };
    // a tile's contraction can be shared by up to 4 wavefronts (with_split): wide tiles, whose loads move 16 bytes
    // per lane and instruction, are kept as long as that sharing still gives every SIMD a wavefront
    auto shared = [&](long long wv) {
        const Band b = make_band(p);
        const long long slots = ((long long)(p.L + 31) / b.g + 1) * b.F;
        int sp = 1;
        while (sp < 4 && wv * sp < 2048 && slots / (4 * sp) >= 32) sp *= 2;
        return wv * sp;
    };
    if (p.HW >= 4 && shared(waves(4)) >= kEnoughWaves)
        with_split(integral_constant<int, 4>{}, waves(4));
    else if (p.HW >= 2 && shared(waves(2)) >= kEnoughWaves)
        with_split(integral_constant<int, 2>{}, waves(2));
    else
        with_split(integral_constant<int, 1>{}, waves(1));
}

}  // namespace bwi

}  // namespace scc
