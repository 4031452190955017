// Which workgroup of a launch takes which column tile: index arithmetic for device and host.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace scc {

// Workgroups of a launch as (outer, inner) pairs, inner fastest: outer is a column tile, inner the groups of rows that read its
// planes.  Consecutive workgroups go to consecutive XCDs, so blockIdx % 8 names the XCD, and an XCD takes runs of that order, so
// that the groups of a column tile meet in its L2.  A grid of several generations (from 1024 workgroups on) is dealt out in runs of
// 16 column tiles, so that the chip sweeps the tensors on one front.  With an eighth of the columns each, the XCDs are an eighth of
// a tensor apart, which for many sizes (powers of two) puts them on the same memory channels at the same time.  Forward, us,
// eighths -> runs of 16: 1024 x 256 -> 256 on 16x16, cg 4, f32 102 -> 101 (no more than noise), bf16 63.4 -> 53.4; 128 x 128 -> 512
// on 32x32, cg 2, co 0.33, bf16 50 -> 45; 512 x 512 -> 512 on 8x8, cg 8, bf16 17.2 -> 16.1; grad-input of 256 x 512 -> 512 on
// 14x14, cg 4, bf16 42.2 -> 38.0; of 66 drawn layers 0.98 to 1.07.  Shorter runs put tiles that share cache lines on two XCDs: 256
// x 512 -> 512 on 14x14, cg 4, bf16 41.5 in eighths, 43.7 with runs of one, 41.4 with 16. Grids of one generation are everywhere at
// once (64 x 512 -> 512 on 14x14, cg 8, bf16 11.2 in eighths, 12.7 and 11.2 with runs of one and 16), and where a tile has one
// group only, neither order is better (0.91 to 1.07).
struct Deal {
    int total;   // workgroups with work: outer * inner
    int inner;
    int chunk;   // workgroups of one XCD: ceil(total / 8)
    int even;    // of these, the first, which are dealt in runs; what then is left goes in eighths ...
    int rest;    // ... from this outer index on
    uint32_t recip;   // floor(2^32 / inner), 2^32 - 1 for 1
};
constexpr int kRun = 16;   // a constant: nothing to divide by in a workgroup's first instructions

inline Deal make_runs(long long outer, int inner)
{
    const long long total = outer * inner;
    const int runs = (int)(outer / (8 * kRun));   // of each XCD
    return {(int)total, inner, (int)((total + 7) / 8), runs * kRun * inner, 8 * runs * kRun,
            inner == 1 ? 0xffffffffu : (uint32_t)((1ull << 32) / (uint32_t)inner)};
}

// An eighth of the order for each XCD, whatever the grid: where grad-weight's workgroups, which keep to slices of the columns, run
// beside these and read the same dy through an XCD's L2 (both gradients of 128 x 256 -> 256 on 16x16, cg 4, co 0.25, bf16 19.1 us, 21.3
// with runs of one; 554 x 120 -> 60 on 16x16, cg 1, f32 102 and 104 with runs of four).
inline Deal in_eighths(Deal d)
{
    d.even = d.rest = 0;
    return d;
}

inline Deal make_deal(long long outer, int inner)
{
    const Deal d = make_runs(outer, inner);
    return d.total >= 1024 && inner > 1 ? d : in_eighths(d);
}

// The tile is a product with the reciprocal and one correction: a division is 0.1 us of every launch (forward of 1 x 32 -> 32 on
// 8x8 3.72 -> 3.61 us, 16 x 128 -> 128 on 14x14, bf16 3.49 -> 3.36).  Returns false where there is no work and the whole
// workgroup leaves.  RUNS false: the deal, whatever it is, is read as one of in_eighths.  Without a branch in here: behind one, the
// kernel's other arguments are fetched after the deal's (1 us for each generation of workgroups).
template <bool RUNS = true>
__host__ __device__ __forceinline__ bool dealt(const Deal& d, int bid, int& outer, int& inner)
{
    const int xcd = bid & 7, slot = bid >> 3;
    const bool runs = RUNS && slot < d.even;
    const int left = RUNS ? xcd * (d.chunk - d.even) + slot - d.even : xcd * d.chunk + slot;
    const int at = runs ? slot : left;
    int tile = (int)(((uint64_t)(uint32_t)at * d.recip) >> 32);   // the quotient or one less
    inner = at - tile * d.inner;
    const bool more = inner >= d.inner;
    tile += more ? 1 : 0;
    inner -= more ? d.inner : 0;
    outer = runs ? tile + (7 * (tile / kRun) + xcd) * kRun : RUNS ? tile + d.rest : tile;
    return (slot < d.chunk) & (runs | (left < (RUNS ? d.total - 8 * d.even : d.total)));
}

// For workgroups that take several tiles (inner == 1): tiles of an XCD, and the i-th of them
__host__ __device__ __forceinline__ int tiles_of(const Deal& d, int xcd)
{
    const int each = d.chunk - d.even, left = d.total - 8 * d.even - xcd * each;
    return d.even + (left < 0 ? 0 : left < each ? left : each);
}

__host__ __device__ __forceinline__ int nth_tile(const Deal& d, int xcd, int i)
{
    return i < d.even ? i + (7 * (i / kRun) + xcd) * kRun : d.rest + xcd * (d.chunk - d.even) + i - d.even;
}

}  // namespace scc
