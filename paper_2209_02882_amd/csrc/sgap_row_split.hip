// Row-split schedule: the unit of work is a row of A (the paper's second
// atomic-parallelism family, <x row, y col>, Section 3.2).  Every row is
// produced by exactly one group (parallel strategy) or one lane (serial
// strategy), so results are written with plain stores and empty rows are
// written as zeros by their owner; no atomics, no zero-fill pass.
//
// One kernel template serves both strategies:
//   parallel  {<1/g row, c col>, r}, g = r = G (Section 6.2, "1/g row"):
//             the G members of a group share a row; member m takes the row's
//             entries m, m+G, ... serially, the group tree-sums, member 0
//             stores.  A group works through `rows_per_slot` rows of its row
//             block (finite resource parallelism, Section 3.3), interleaved
//             with the other groups' rows so that neighbouring rows, which
//             tend to share columns, are in flight together.
//   serial    {<g row, c col>, 1} (Section 6.1, "g row"): the same kernel with
//             G = 1 and rows_per_slot = group_size.
// Lane layout:  thread = (slot*G + member)*LC + chunk over the workgroup.
//
// A work item is (block of consecutive rows, column tile), one workgroup per
// item (or, as a tuning option, a grid that fits the chip at once whose
// workgroups loop over items); the stored entries of a row block are contiguous in
// colidx/vals, so the workgroup copies them (coalesced, streaming) into LDS in
// chunks together with the block's slice of rowptr, and its lanes then read
// (column, value) pairs from LDS: the vector memory path carries only the
// gathered rows of B.
#include "sgap_row_split_impl.hpp"

namespace sgap {

namespace {

constexpr int kShareMin = 256;    // the shortest row that a whole workgroup takes together
constexpr int kFinderRows = 64;   // a finder looks at no fewer rows (32 cost matrices without long rows: 10,000 rows of 16
                                  // entries, N = 32, G = 8 6.3 -> 6.7 us)
constexpr int kFinderEntries = 2048;  // ... unless most rows are long, and then no more entries: 2,000 rows of 400, N = 37, G = 16 330 us by
                                      // 32 finders, 31 by 400 (4,000 rows of 400, N = 32, G = 8, none of which is long enough: 15.1 by 64, 18.9 by 800)
constexpr int kSmallShare = 512;  // where groups have four members, or several passes, ...
constexpr int kFewRows = 8192;    // ... and so few rows, the half of that in the mean is enough (20,000 rows of 200, N = 8, G = 4 29 us, by 2,048 finders 38)
// Few entries leave the chip to the rows that workgroups take together; with more the others want the wavefront per SIMD that
// those rows' registers cost, and where B is small there is little to wait for.  us, without / with: power laws, 3,000 rows, N = 64 8.7 / 7.0;
// 10,000, N = 64 16.8 / 12.7; 361,000 entries, N = 39, B of 14 MB 48 / 35; 464,000, N = 42, of 3.2 MB 26.7 / 19.2; 508,000, N = 51 38.2 / 31.7; 2.7 M, N = 19, of 3 MB
// 56.7 / 60.4; uniform, 84,000 entries, N = 56 5.8 / 6.8, 571,000, N = 56, B of 0.2 MB 13.7 / 16.3; 1.2 M, N = 14 18.0 / 20.4; 40 to a row, 316,000
// entries, B of 0.8 MB 8.2 / 8.7; 1,024 rows of 10, N = 32 3.05 / 3.12.
constexpr int64_t kDeepFewest = 30'000, kDeepMost = 600'000, kDeepBytes = 1 << 20;  // entries; of B
constexpr double kDeepMean = 22.0;
constexpr int64_t kDeepColumns = 64;
constexpr int kFindersPerCu = 8;  // as many workgroups as are resident
constexpr int kTeamRows = 256;    // a team of two looks through no more rows: a look of its workgroups' threads
constexpr int kTeamsPerCu = 4;    // no teams where there are more finders: they come in rounds then

// A group's rounds of loads on a row of len entries are about len / (g * kDepthGroups) for each pass over the columns,
// each of them a round trip to memory with a handful of loads in flight.  From a dozen rounds on, the whole workgroup
// takes the row instead; never a row that is only a few steps of the workgroup long.
int32_t share_rows_from(int g, int passes)
{
    const int len = 12 * g * kDepthGroups / passes;
    return len < kShareMin ? kShareMin : len;
}

}  // namespace

// Finders cost a look at every row pointer, so there are none where the caller's count of entries says that no row can
// be long enough.  That count may be too small: the walk then takes every row, whatever its length (share_from).
// Finders per compute unit, G = 8 (all measured before their loads were masked, and before flat_shared_rows_kernel took the
// larger of these matrices): the longest rows of a power law (4,096 entries) bind it otherwise.  65,536 rows,
// N = 37: 73 us without finders, 70.7 with one, 58.4 with two, 47.5 with four or eight; 114,150 rows, N = 34: 100.5
// without, 100.4, 90.2 and 82.8 with one, two and four, 72.5 with eight (a stretch of rows for each; FinderDeal says
// what dealing them out changed).  Where there are few finders two look through the same rows and take the long ones in
// turn, so that two of the longest seldom wait for each other.  Power laws, ten matrices each, in the mean: 9,437 rows,
// N = 45 26.6 -> 23.1 us, 20,000 rows, N = 16 13.2 -> 11.4, 50,021 rows, N = 37 43.8 -> 40.3.  Teams of four gain 3 %
// more at best and cost 60,000 rows without long ones 18.7 -> 19.1; teams where finders come in rounds lose (150,000
// rows, N = 37: 92.2 -> 98.0).
RowSplitGrid plan_row_split_grid(int g, int passes, int64_t M, int64_t items, int xcds, int compute_units,
                                 int64_t nnz_hint, int resident)
{
    RowSplitGrid p = {0x7fffffff, 0, 0, FinderDeal(M), 0, 0};
    const int64_t items_per_xcd = (items + xcds - 1) / xcds;
    int64_t wgs_per_xcd = resident > 0 ? (resident / xcds > 0 ? resident / xcds : 1) : items_per_xcd;
    if (wgs_per_xcd > items_per_xcd) wgs_per_xcd = items_per_xcd;
    if (wgs_per_xcd * xcds > 0x7ffffff0LL) wgs_per_xcd = 0x7ffffff0LL / xcds;
    const int64_t walkers = wgs_per_xcd * xcds;
    const int32_t share_from = share_rows_from(g, passes);
    if (g > 1 && (nnz_hint < 0 || nnz_hint >= share_from)) {
        const int64_t most = (int64_t)kFindersPerCu * compute_units;
        // where most rows are long (few rows, small groups: where many are), as many rows as hold kFinderEntries
        const double mean = (double)nnz_hint / (double)M;
        int64_t rows = kFinderRows;
        const bool many = mean >= (double)share_from || (share_from <= kSmallShare && M <= kFewRows && 2.0 * mean >= (double)share_from);
        if (many && kFinderEntries / mean < (double)kFinderRows) rows = (int64_t)(kFinderEntries / mean);
        if (rows < (int64_t)FinderDeal::kUnit) rows = FinderDeal::kUnit;
        int64_t finders = (M + rows - 1) / rows < most ? (M + rows - 1) / rows : most;
        if (resident > 0 && finders > walkers) finders = walkers;
        const int64_t rows_each = (M + finders - 1) / finders;
        if (2 * rows_each <= kTeamRows && finders >= 2 && finders <= (int64_t)kTeamsPerCu * compute_units) p.log2_team = 1;
        const int64_t team = 1LL << p.log2_team;
        if (resident > 0) {
            // a persistent grid is resident all at once: its own workgroups are the finders
            finders = finders / team * team;
        } else {
            const int64_t whole = team > xcds ? team : xcds;  // whole teams, whole rounds of the dies
            finders = (finders + whole - 1) / whole * whole;
            p.walk_from = (int32_t)finders;
        }
        p.share_from = share_from;
        p.finders = (int32_t)finders;
    }
    p.grid = (uint32_t)(walkers + p.walk_from);
    return p;
}

hipError_t launch_row_split(const SpmmArgs& a, int g, int lc, int vec, int rows_per_slot, bool interleave,
                            int tile_cols, int xcds, int compute_units, bool persistent, int block, int64_t nnz_hint, double mean_row,
                            hipStream_t s)
{
    row_split_detail::Launch<false> f{a, rows_per_slot, interleave ? 1 : 0, tile_cols, xcds, compute_units,
                                      offsets_fit_32(a), persistent, 0, block, s, nnz_hint, mean_row <= kShortRowMean};
    f.deep = a.N <= kDeepColumns && nnz_hint >= kDeepFewest && nnz_hint <= kDeepMost && mean_row <= kDeepMean && a.K * a.N * 4 >= kDeepBytes;
    if (!dispatch_group(g, lc, vec, f)) return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace sgap
