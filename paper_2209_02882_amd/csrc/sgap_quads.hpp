// Four consecutive rows ("a quad") that go together because they share columns, as neighbouring rows of grids, meshes and
// bands do: what the kernels that take them so have in common.
#pragma once
#include "sgap_common.hpp"

namespace sgap {

constexpr int kQuad = 4;
constexpr int kQuadRow = 32;      // rows of fewer entries are listed: there is kNoColumn behind every one
constexpr int32_t kNoColumn = 0x7fffffff;
constexpr int64_t kDealBytes = 4 << 20;  // an L2

typedef float f32x4 __attribute__((ext_vector_type(4)));

// LDS is written and read by the lanes of one wavefront only, whose LDS instructions are carried out in order: what is
// needed is that the compiler keeps them in order.
__device__ __forceinline__ void wave_lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// How many of a row's columns (ascending, kNoColumn behind them) are below c
__device__ __forceinline__ int below(const int32_t* __restrict__ row, int32_t c)
{
    int lo = 0;
#pragma unroll
    for (int half = kQuadRow / 2; half > 0; half /= 2) lo += row[lo + half - 1] < c ? half : 0;
    return lo;
}

// A row of a three-dimensional grid in its natural order wants three stretches of B a plane apart, and planes that no L2 holds come from memory three times
// where a die goes through one run of rows.  There the planes are better dealt out: each die takes an eighth of every
// plane, the same one, and finds the rows of B that the plane below has brought.  How far apart the planes are is read off
// a row in the middle: half the distance of its outer columns.  It decides nothing but the order of the work.
// Returns a die's rows of a plane, or 0: three planes of rows of B (b_row_bytes each) fit an L2, or the matrix has
// fewer than eight.
__device__ __forceinline__ uint32_t plane_share(const SpmmArgs& a, uint32_t dies, uint32_t b_row_bytes)
{
    const int32_t begin = a.rowptr[a.M / 2], end = a.rowptr[a.M / 2 + 1];
    if (dies < 2 || end <= begin) return 0;
    const int32_t first = a.colidx[begin], last = a.colidx[end - 1];
    if (last <= first) return 0;
    const uint32_t reach = (uint32_t)(last - first) / 2;
    if ((int64_t)reach * 8 > a.M || (int64_t)reach * 3 * b_row_bytes <= kDealBytes) return 0;
    return reach / dies;
}

// Which block of rows a die takes in its turn: those of one contiguous run for each die, or of its share of every plane (in
// blocks).
__device__ __forceinline__ uint32_t die_block(uint32_t share, uint32_t die, uint32_t turn, uint32_t blocks, uint32_t dies)
{
    const uint32_t per_die = (blocks + dies - 1) / dies;
    if (share < 2) return die * per_die + turn;
    const uint32_t rounds = blocks / (share * dies);
    const uint32_t round = turn / share;
    if (round < rounds) return (round * dies + die) * share + turn % share;
    const uint32_t rest = blocks - rounds * share * dies;  // dealt evenly: every die has per_die turns, or one without a block
    const uint32_t each = (rest + dies - 1) / dies, at = turn - rounds * share;
    return at < each ? rounds * share * dies + die * each + at : blocks;
}

}  // namespace sgap
