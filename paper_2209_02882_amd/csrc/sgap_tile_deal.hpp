// Assignment of tiles of stored entries to persistent workgroups.  Plain
// integer arithmetic, usable on the host (tests) and on the device.
#pragma once
#include <stdint.h>

#if defined(__HIPCC__)
#define SGAP_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define SGAP_HOST_DEVICE inline
#endif

namespace sgap {

// Which tiles a persistent workgroup takes.  The 8 dies (XCDs) of the chip
// have private L2s and receive workgroups round-robin (workgroup b runs on die
// b % 8).  Tiles are therefore handed out in chunks of consecutive tiles:
// chunk c goes to die c % 8, and the workgroups of a die take the tiles of the
// die's chunks in order, round-robin.  A die then works on one or a few
// stretches of neighbouring rows at a time, so a row of the dense operand that
// neighbouring rows of A share is fetched into one L2, not into all eight,
// while every die still receives an even sample of the whole matrix (stretches
// of short or empty rows cost several times more per entry than long rows).
// With fewer than 8 workgroups, a grid that is no multiple of 8, or no more
// tiles than workgroups, plain round-robin over the workgroups is used.
struct TileDeal {
    int64_t tiles;   // tiles of the matrix
    int32_t dies;    // 8 or 1
    int32_t chunk;   // tiles per chunk
    int32_t die;     // this workgroup's die
    int32_t wg;      // this workgroup's number on its die
    int32_t wgs;     // workgroups per die
    int64_t mine;    // tiles this workgroup takes

    // block = this workgroup's number in a grid of `grid` workgroups
    SGAP_HOST_DEVICE TileDeal(int64_t tiles_, uint32_t block, uint32_t grid) : tiles(tiles_)
    {
        // (a grid with a workgroup per tile just takes tile = workgroup)
        dies = (grid >= 8 && grid % 8 == 0 && tiles > grid) ? 8 : 1;
        die = (int32_t)(block % dies);
        wg = (int32_t)(block / dies);
        wgs = (int32_t)(grid / dies);
        // about 16 chunks per die, at most one round of the die's workgroups
        int64_t c = tiles / (dies * 16);
        if (c > wgs) c = wgs;
        if (c < 1) c = 1;
        chunk = (int32_t)c;
        const int64_t full = tiles / chunk, rem = tiles % chunk;
        const int64_t die_tiles = (full / dies + (die < full % dies ? 1 : 0)) * chunk + (die == full % dies ? rem : 0);
        mine = wg < die_tiles ? (die_tiles - wg + wgs - 1) / wgs : 0;
    }
    // global number of this workgroup's j-th tile, j < mine
    SGAP_HOST_DEVICE int64_t tile(int64_t j) const
    {
        const int64_t q = wg + j * wgs;  // q-th tile of this die
        return (die + (int64_t)dies * (q / chunk)) * chunk + q % chunk;
    }
};

// A workgroup's tiles one after the other: deal.tile(0), deal.tile(1), ... without a division per tile (a 64-bit
// division is a hundred instructions, which a tile of a few hundred entries feels).
struct TileWalk {
    uint32_t chunk, blk, rem, blk_step, rem_step, die, dies;
    SGAP_HOST_DEVICE explicit TileWalk(const TileDeal& d)
        : chunk((uint32_t)d.chunk), die((uint32_t)d.die), dies((uint32_t)d.dies)
    {
        blk = (uint32_t)d.wg / chunk;
        rem = (uint32_t)d.wg % chunk;
        blk_step = (uint32_t)d.wgs / chunk;
        rem_step = (uint32_t)d.wgs % chunk;
    }
    SGAP_HOST_DEVICE uint32_t tile() const { return (die + dies * blk) * chunk + rem; }  // below 2^31 / 256
    SGAP_HOST_DEVICE void next()
    {
        blk += blk_step;
        rem += rem_step;
        if (rem >= chunk) {
            rem -= chunk;
            ++blk;
        }
    }
};

// Which rows a team of workgroups looks through for long ones.  Units of four neighbouring rows (a 16-byte piece of rowptr) are
// dealt so that neighbours, and units a power of two apart, go to workgroups far from each other: long rows often sit
// together (the first rows of an R-MAT matrix, those with few one bits in their number), and the workgroups that find
// them produce them one after the other.  Unit u has place u * g mod 2^k, g the odd number nearest to the golden section
// of 2^k, and team i takes the i-th stretch of places; step is the inverse of g.  R-MAT with 2^21 rows, row-split
// parallel, G = 16, N = 4, 16 and 32: 5.0, 6.9 and 9.6 ms with a stretch of rows for each workgroup, 1.5, 1.4 and 1.6 so.
struct FinderDeal {
    static constexpr uint32_t kUnit = 4;
    uint32_t units, mask, step;
    FinderDeal() = default;
    explicit FinderDeal(int64_t M)
    {
        units = (uint32_t)((M + kUnit - 1) / kUnit);  // below 2^29
        uint64_t places = 1;
        while (places < units) places *= 2;
        mask = (uint32_t)(places - 1);
        const uint32_t g = (uint32_t)((double)places * 0.6180339887498949) | 1u;
        step = g;  // right in three bits; every round doubles them
        for (int i = 0; i < 4; ++i) step *= 2u - g * step;
    }
    // first place of team i of n (of team n: behind the last place)
    SGAP_HOST_DEVICE uint32_t first_place(uint32_t i, uint32_t n) const
    {
        const uint64_t p = (uint64_t)(mask / n + 1) * i;
        return p <= mask ? (uint32_t)p : mask + 1;
    }
    // row number r < kUnit of the unit at a place (M or beyond: no such row)
    SGAP_HOST_DEVICE int64_t row(uint32_t place, uint32_t r) const { return (int64_t)((place * step) & mask) * kUnit + r; }
};

}  // namespace sgap
