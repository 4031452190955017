// Forward of SCC in bf16 with the weights resident in registers, for layers with many columns and short windows.
//
// y[n,k,p] = sum_j w[k,j] * x[n,(s_k+j) mod Cin,p]     (Section 4.2, output-centric forward)
//
// A workgroup of four wavefronts owns a group of 128 filters in the order of their window starts (scc_band.h), a wavefront 32 of
// them, and walks over tiles of 256 columns.  The group reads the channels of one stretch of the channel circle (its walk,
// from the first window's start to the last one's end); the 256 lanes fetch a tile's planes, 16 bytes per lane and plane, and park
// them in LDS in the matrix instruction's operand layout.  A wavefront's weights, masked once when the workgroup starts, stay in
// its registers: per tile it reads B operands from LDS, multiplies and stores 512 contiguous bytes of a row per half-wave.  The planes of
// the next tile are in flight meanwhile.
//
// What bounds it: HBM where x is not on the chip, else a tile's chain of load, barrier, product and store.  The kernels with a workgroup
// per tile spend most of a tile on its first loads (weights, table, planes) and its last stores; here a CU holds one workgroup (more put
// more columns in flight and are slower: 128 x 128 -> 512 on 32x32, cg 2, co 0.33 37.5 us, 40.7 with two), the tiles' loads and
// stores are in flight together, and the chip sweeps the tensors on one front in pieces of 512 bytes (loads and stores alone, in this
// pattern: 32 us; x is read once, 33 of 32 MiB: the groups' reads meet in the L2s).  us, packed weights and their packing launch -> this,
// x cold / x in three buffers in turn: that layer 44 -> 39 / 36.7 -> 33-35; 312 x 224 -> 893 on 14x14, cg 4, co 0.33 65 -> 39 / 59 -> 32;
// 434 x 448 -> 1792 on 12x6, cg 8, co 0.25 82 -> 44 / 75 -> 35.  Binary32 layers, whose three pieces and six products per
// value leave no room for 256 columns, gained 4 % at most and stay with the other kernels.
//
// Products and sums are those of the kernels with packed weights (scc_packed_kernel.h).
#include "scc_packed_kernel.h"

namespace scc {

namespace {

using packed::filter_of;
using packed::walk_of;
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int CT = 8;   // columns per lane and plane
constexpr int KA = 6;   // K groups of 16 positions whose weights a wavefront keeps

struct Resident {
    Band b;
    int rows;      // filters in order of their starts: P*F
    int NG;        // groups of 128 rows
    int lanes;     // workgroups of an XCD that share the column tiles of a row group
    Deal deal;     // column tiles
    Groups q;      // column groups of CT pixels
    uint32_t bytes;   // of y
};

// Past the end of any y (these layers' has less than 2^31 bytes, forward_mfma_eligible), and 16 bytes from there do not wrap around 2^32.
constexpr uint32_t kDropped = 0x80000000u;

// A row without a filter is stored there and the hardware drops it: with a branch around a store the next tile's
// loads could not be waited for without the stores.
template <bool PAST>
__device__ __forceinline__ void store_row(u32x4 v, __amdgpu_buffer_rsrc_t to, uint32_t at)
{
    __builtin_amdgcn_raw_buffer_store_b128(v, to, (int)at, 0, PAST ? 2 : 0);   // 2: nontemporal
}

// NQ  quads of planes a lane fetches per tile: walks of up to 32*NQ positions
// PAST  y is written past the caches
template <int NQ, bool PAST>
__global__ __launch_bounds__(256) void forward_resident(const bf16_t* __restrict__ x, const bf16_t* __restrict__ w,
                                                        bf16_t* __restrict__ y, Problem P, Resident T)
{
    typedef bf16_t bvec __attribute__((ext_vector_type(CT), aligned(sizeof(bf16_t))));   // CT consecutive columns of one plane
    constexpr uint32_t ES = sizeof(bf16_t);
    constexpr int kCols = 32 * CT;
    constexpr int kOctets = 4 * NQ;                     // groups of 8 positions
    static_assert(2 * KA <= kOctets, "a wavefront's positions are among those staged");
    extern __shared__ __attribute__((aligned(16))) char lds_r[];   // a tile's planes: [octet][column][8 positions]
    uint32_t* const rowat = (uint32_t*)(lds_r + kOctets * kCols * 16);   // byte offset of a row's output plane in a sample, or kDropped

    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int ng = slot % T.NG;
    int i = slot / T.NG;                                // this workgroup's tiles: the XCD's i-th, i + lanes, ...
    const int mine = tiles_of(T.deal, xcd);
    if (i >= mine) return;                              // the whole workgroup leaves

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63, f = lane & 31, h = lane >> 5;
    int first, len;
    walk_of<true>(P, T.b, T.rows, ng, first, len);
    const uint32_t plane = (uint32_t)P.HW * ES;

    // ---- weights: K group g of this wavefront is the octets o0 + 2g (lanes 0-31) and o0 + 2g + 1 ----
    const int row0 = (ng * 4 + wave) * 32;
    int o0 = 0;
    {
        const int m0 = row0 / T.b.F, last = row0 + 31 < T.rows ? row0 + 31 : T.rows - 1;
        const int d0 = T.b.g * (m0 - ng * 128 / T.b.F);                  // walk position of the first window's start
        const int d1 = d0 + T.b.g * (last / T.b.F - m0) + P.L;
        if (row0 < T.rows && d1 <= len) o0 = d0 / 8 < kOctets - 2 * KA ? d0 / 8 : kOctets - 2 * KA;   // else once around the circle
        o0 = __builtin_amdgcn_readfirstlane(o0);
    }
    bf16_t wraw[KA][8];
    uint32_t in[KA];
    {
        const int row = row0 + f;
        const int k = row < T.rows ? filter_of(T.b, row / T.b.F, row % T.b.F, P.Cout) : -1;
        const int s = T.b.g * (row / T.b.F);
        if (h == 0) rowat[wave * 32 + f] = k < 0 ? kDropped : (uint32_t)k * plane;
#pragma unroll
        for (int g = 0; g < KA; ++g) {
            in[g] = 0;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int pos = 8 * (o0 + 2 * g + h) + e;
                int j = first + pos - s;
                j += j < 0 ? P.Cin : 0;
                j -= j >= P.Cin ? P.Cin : 0;
                const bool here = (k >= 0) & (pos < len) & (j < P.L);
                in[g] |= here ? 1u << e : 0u;
                wraw[g][e] = w[here ? (uint32_t)k * (uint32_t)P.L + (uint32_t)j : 0u];
            }
        }
    }

    // ---- B, loading role: lane (quad lu + 8z, column group lq) fetches CT columns of 4 planes, as in packed_body ----
    const int lq = (lane & 7) | (lane >> 4) << 3, lu = 2 * wave + (lane >> 3 & 1);
    uint32_t planeat[NQ][4];
#pragma unroll
    for (int z = 0; z < NQ; ++z)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            int pos = 4 * (lu + 8 * z) + e;
            pos = pos < len ? pos : len - 1;            // past the walk: meets zero weights
            int c = first + pos;
            c -= c >= P.Cin ? P.Cin : 0;
            planeat[z][e] = (uint32_t)c * plane;
        }
    const uint32_t count = (uint32_t)T.q.count;
    auto column = [&](int tile, uint32_t lane_group, uint32_t planes) {   // past the end: the last group once more, the same bits are stored
        const uint32_t u = (uint32_t)tile * 32u + lane_group;
        uint32_t n, p;
        column_of_group(u < count ? u : count - 1u, T.q, n, p);
        return (n * planes * (uint32_t)P.HW + p) * ES;
    };
    bvec raw[NQ][4];
    auto issue = [&](int tile) {
        const uint32_t at = column(tile, (uint32_t)lq, (uint32_t)P.Cin);
#pragma unroll
        for (int z = 0; z < NQ; ++z)
#pragma unroll
            for (int e = 0; e < 4; ++e) raw[z][e] = *(const bvec*)((const char*)x + (at + planeat[z][e]));
    };
    auto commit = [&]() {
#pragma unroll
        for (int z = 0; z < NQ; ++z) {
            const int quad = lu + 8 * z;
            char* dst = lds_r + ((quad >> 1) * kCols + lq) * 16 + 8 * (quad & 1);
#pragma unroll
            for (int j = 0; j < CT; ++j) {              // column CT*lq + j of the tile is LDS column 32j + lq
                *(u32x2*)(dst + j * 512) = u32x2{(uint32_t)(bf16_t)raw[z][0][j] | ((uint32_t)(bf16_t)raw[z][1][j] << 16),
                                                 (uint32_t)(bf16_t)raw[z][2][j] | ((uint32_t)(bf16_t)raw[z][3][j] << 16)};
            }
        }
    };

    int tile = nth_tile(T.deal, xcd, i);
    issue(tile);                                        // in flight while the weights are cut
    u32x4 a[KA];
#pragma unroll
    for (int g = 0; g < KA; ++g)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            a[g][e] = ((in[g] >> (2 * e)) & 1u ? (uint32_t)wraw[g][2 * e] : 0u) |
                      ((in[g] >> (2 * e + 1)) & 1u ? (uint32_t)wraw[g][2 * e + 1] << 16 : 0u);
    auto mm = [&](const u32x4& p, const u32x4& q, f32x16& d) {
        const uint32_t pa[4] = {p[0], p[1], p[2], p[3]}, qa[4] = {q[0], q[1], q[2], q[3]};
        d = mfma_bf16<8>(pa, qa, d);
    };
    __amdgpu_buffer_rsrc_t to = __builtin_amdgcn_make_buffer_rsrc((void*)y, 0, T.bytes, 0x00027000);
    auto product = [&]() {
        f32x16 acc[CT];
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[c][v] = 0.f;
        const char* bb = lds_r + ((o0 + h) * kCols + f) * 16;
#pragma unroll
        for (int g = 0; g < KA; ++g)
#pragma unroll
            for (int c = 0; c < CT; ++c) mm(a[g], *(const u32x4*)(bb + g * 2 * kCols * 16 + c * 512), acc[c]);
        // accumulator register v holds tile row 8*(v/4) + 4*h + v%4, columns CT*f .. CT*f + CT-1 of the tile
        const uint32_t at = column(tile, (uint32_t)f, (uint32_t)P.Cout);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const u32x4 ra = *(const u32x4*)(rowat + wave * 32 + 8 * r + 4 * h);
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                bvec o;
#pragma unroll
                for (int c = 0; c < CT; ++c) o[c] = from_f32<bf16_t>(acc[c][4 * r + s]);
                store_row<PAST>(__builtin_bit_cast(u32x4, o), to, ra[s] == kDropped ? kDropped : at + ra[s]);
            }
        }
    };

    // One LDS buffer and two barriers per tile; the last tile is written out, so that no load is conditional inside the loop.
    for (;;) {
        __syncthreads();                                // nobody reads the previous tile any more
        commit();
        i += T.lanes;
        if (i >= mine) break;
        const int next = nth_tile(T.deal, xcd, i);
        issue(next);
        __syncthreads();
        product();
        tile = next;
    }
    __syncthreads();
    product();
}

// Octets of positions that a wavefront's filters reach at most, and positions of the longest walk
void reach(const Problem& p, const Band& b, int rows, int* octets, int* longest)
{
    *octets = *longest = 1;
    for (int ng = 0; ng < (rows + 127) / 128; ++ng) {
        int first, len;
        walk_of<true>(p, b, rows, ng, first, len);
        *longest = len > *longest ? len : *longest;
        for (int row0 = ng * 128; row0 < rows && row0 < (ng + 1) * 128; row0 += 32) {
            const int last = row0 + 31 < rows ? row0 + 31 : rows - 1;
            const int d0 = b.g * (row0 / b.F - ng * 128 / b.F), d1 = d0 + b.g * (last / b.F - row0 / b.F) + p.L;
            const int n = d1 <= len ? (d1 + 7) / 8 - d0 / 8 : (len + 7) / 8;
            *octets = n > *octets ? n : *octets;
        }
    }
}

Resident make_resident(const Problem& p)
{
    Resident t;
    t.b = make_band(p);
    t.rows = t.b.P * t.b.F;
    t.NG = (t.rows + 127) / 128;
    t.q = column_groups(p, CT);
    t.deal = make_runs((t.q.count + 31) / 32, 1);
    int lanes = 32 / t.NG;                              // one workgroup per CU: 32 for each XCD
    lanes = lanes < 1 ? 1 : lanes < t.deal.chunk ? lanes : t.deal.chunk;
    const int each = (t.deal.chunk + lanes - 1) / lanes;
    t.lanes = (t.deal.chunk + each - 1) / each;
    t.bytes = (uint32_t)((long long)p.NQ * p.Cout * (long long)sizeof(bf16_t));
    return t;
}

// What the kernel takes: a workgroup's start costs 3 us, so 64 MB of x and y, and more than three tiles of 256 columns per workgroup,
// more than four where a tile's filters start together; windows whose 32 filters span at most KA K groups and, where they start
// together, 80 positions (the walks get long: from 88 on 0.74 to 0.92 of the per-tile kernel's speed); row groups filled to more than
// half; tiles of the others that fetch planes again, 1.7 times with differing starts in a tile, 2.5 times without.
bool resident_eligible(const Problem& p, const Band& b, const Resident& t, int* longest)
{
    if (t.deal.chunk <= (b.F < 32 ? 3 : 4) * t.lanes || 100ll * p.Cout < 55ll * 128 * t.NG || t.NG > 32) return false;
    double again;
    packed::fetches_without_sharing<true>(p, b, &again);
    if (b.F < 32 ? again < 1.7 : again < 2.5 || p.L > 80) return false;
    int octets;
    reach(p, b, t.rows, &octets, longest);
    return octets <= 2 * KA && *longest <= 192;
}

template <int NQ>
hipError_t launch_variant(const bf16_t* x, const bf16_t* w, bf16_t* y, const Problem& p, const Resident& t, hipStream_t st)
{
    constexpr int kLds = 4 * NQ * 32 * CT * 16 + 512;
    auto launch = [&](auto past) {
        constexpr bool PAST = decltype(past)::value;
        static const hipError_t allowed = hipFuncSetAttribute((const void*)forward_resident<NQ, PAST>,
                                                              hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
        if (allowed != hipSuccess) return allowed;
        forward_resident<NQ, PAST><<<dim3((unsigned)(8 * t.lanes * t.NG)), dim3(256), kLds, st>>>(x, w, y, p, t);
        return hipGetLastError();
    };
    // past the caches where rows are whole pieces of 64 bytes, as in the per-tile forward (512 x 128 -> 128 on 28x28, cg 2, co
    // 0.25: 51.3 us past them, 49.1 through them; 128 x 128 -> 512 on 32x32 37.4 and 38.3)
    return p.HW * sizeof(bf16_t) % 64 == 0 ? launch(std::true_type()) : launch(std::false_type());
}

}  // namespace

// Which of these gain: of 1300 drawn layers that the kernel takes, and 250 more of those chosen here, times of the packed kernel with its
// packing launch where that is preferred, else of the per-tile kernel, over this one's, mean (least), with x in three buffers in turn or
// just written by another kernel, the lower of the two | with x cold.  Cold operands alone (1.16, least 0.79, over all of them) do not
// show what is lost: this kernel waits for a tile's planes wherever they come from, the others are faster with planes that the last
// level cache still holds.
//   No packed weights: with starts or windows off multiples of four, whose weights the per-tile kernel loads one by one, at least eight
//   starts to a tile and windows of more than 8 channels 1.26 (0.95) | 1.34; shorter windows 1.11 (0.94), fewer starts 0.83 (0.74);
//   even weights 0.89 (0.67) | 1.06 (258 x 128 -> 512 on 16x16, cg 4, co 0.5 20.4 us, per tile 14.3).
//   Packed weights, planes that are no whole pieces of 64 bytes, which that kernel writes past the caches: below 600 bytes 1.33 (0.85,
//   0.97 in turn) | 1.40; larger ones with Cout >= 3 Cin 1.24 (0.95) | 1.23, others of less than 70e6 values of x and y 1.07 (0.93) | 1.23,
//   of more 0.95 (0.76) | 1.33.
//   Packed weights, whole pieces: with workgroups on 7/8 of the CUs and walks past 64 positions that end by 96, or whose groups are
//   filled to three quarters at most (the other kernel multiplies the empty rows as well), 1.06 (0.90) | 1.21; the rest 0.98 (0.71) | 1.10.
// Without a workspace even weights stay with the per-tile kernel (0.72 to 1.3 here), uneven ones gain more than with one (1.10 to 3.1).
// Stores take rows of whole words.
bool forward_resident_preferred(const Problem& p, int es, const void* y, bool workspace)
{
    if (es != 2 || p.L > 16 * KA || p.HW < CT || p.HW % 2 != 0 || ((uintptr_t)y & 3u) != 0 || !forward_mfma_eligible(p)) return false;
    if ((double)(p.Cin + p.Cout) * (double)p.NQ < 32e6) return false;
    const Band b = make_band(p);
    if (4ll * b.P * b.F > 5ll * p.Cout) return false;       // few filters on many starts: too many empty rows
    const Resident t = make_resident(p);
    int longest;
    if (!resident_eligible(p, b, t, &longest)) return false;
    const bool uneven = b.g % 4 != 0 || p.L % 4 != 0, packs = packed::choose<true>(p, es) > 0;
    if (!uneven && !(packs && workspace)) return false;
    if (!packs) return b.F < 8 && b.P >= 8 && p.L > 8;
    if (p.HW % 32 != 0) return p.HW < 300 || p.Cout >= 3 * p.Cin || (double)(p.Cin + p.Cout) * (double)p.NQ < 70e6;
    return 8 * t.lanes * t.NG >= 224 && longest > 64 && (longest <= 96 || 4 * p.Cout <= 3 * 128 * t.NG);
}

hipError_t launch_forward_resident(const bf16_t* x, const bf16_t* w, bf16_t* y, const Problem& p, hipStream_t st)
{
    const Resident t = make_resident(p);
    int octets, longest;
    reach(p, t.b, t.rows, &octets, &longest);
    return longest <= 96    ? launch_variant<3>(x, w, y, p, t, st)
           : longest <= 128 ? launch_variant<4>(x, w, y, p, t, st)
                            : launch_variant<6>(x, w, y, p, t, st);
}

}  // namespace scc
