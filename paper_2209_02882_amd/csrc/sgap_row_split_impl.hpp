// Row-split kernel template and its launcher; included by the translation
// units that instantiate it (sgap_row_split.hip: one group per row, plain
// stores; sgap_row_split_partial.hip: sub-groups merged with atomics).
#pragma once
#include "sgap_common.hpp"
#include "sgap_flat.hpp"
#include "sgap_gather.hpp"
#include "sgap_lane_ops.hpp"

namespace sgap {

// Rows of B a lane keeps in flight, chosen with the columns' layout (DEPTH of the kernel):
//   6  one lane per row: 70 vector registers, seven wavefronts per SIMD (stencil27, N = 128: 593 us; with eight in flight
//      and five wavefronts 641, with four 619);
//   4  one lane per row and rows of a dozen entries or fewer: more wavefronts beat deeper batches that are mostly masked
//      (fibers of 1 to 16 entries, 32 columns, two rows per lane: 231 us, 234 with six, 262 with eight);
//   8  several lanes per row: rows that a workgroup takes together are done the sooner (power law, N = 37, G = 16: 77 us
//      with six, 73 with eight, before those had workgroups of their own).  For the other rows it depends: stencil27,
//      N = 16, G = 8 203 us against 233 with six, N = 128 700 against 712, but N = 4, G = 16 164 against 145, and fibers
//      of 1 to 16 entries, 32 columns, two lanes 339 against 300.
constexpr int kDepthRows = 6, kDepthShort = 4, kDepthGroups = 8;
constexpr double kShortRowMean = 12.0;
constexpr int kStageCap = 2048;  // (column, value) pairs per LDS chunk: 16 KB
constexpr int kRowCap = 1024;    // rowptr entries kept in LDS per row block (+1)
constexpr int kRowSplitMaxBlock = 512;  // threads per workgroup: 128, 256 or 512, chosen at launch

// A thread's place among those that take a row together.
struct SharedLanes {
    uint32_t lanes, members, member, chunk;  // member number `members` has no entries
    __device__ __forceinline__ SharedLanes(int64_t chunks, int block)
    {
        lanes = chunks < kWave ? (uint32_t)chunks : (uint32_t)kWave;
        // (divisions of numbers up to 512 by up to 64: exact)
        const float per_lane = __builtin_amdgcn_rcpf((float)lanes);
        members = (uint32_t)(((float)block + 0.5f) * per_lane);
        member = (uint32_t)(((float)threadIdx.x + 0.5f) * per_lane);
        chunk = threadIdx.x - member * lanes;
    }
};

// One row by the whole workgroup: as many chunk lanes as the columns take (a wavefront's at most) and block / lanes members,
// each of which takes every (block / lanes)-th stored entry with DEPTH rows of B in flight; the members' sums are added up
// through LDS in a fixed order, and the row has one plain store as ever.  For the rows whose length would keep the one group
// that owns them busy long after the rest of the chip is done (see plan_row_split_grid).  A round of loads is a round trip to
// memory whatever is in it, so lanes that hold no columns cost in proportion: with the next power of two of chunk lanes, 16
// members instead of 25 at N = 37, a row of 4,096 entries took 32 rounds instead of 21.  Power laws, four matrices each, us,
// power of two / as many as the columns take: 50,021 rows, N = 37 40.2 to 62.4 / 35.2 to 50.3; 20,396 rows, N = 37 34.9 to
// 40.6 / 29.0 to 33.9; 53,897 rows, N = 51 28.9 to 47.2 / 27.6 to 42.5; columns that fill a power of two within 2 %.
// MASKED: entries past the end are masked loads (MaskedRows) of places that exist, not branches (18,205 rows, N = 27 17.2 / 13.5;
// 10,000, N = 24 13.6 / 9.6); where registers leave six wavefronts per SIMD branches are better (R-MAT, 65,536 rows, N = 64 106 / 112).
// s_A and s_part may be the same memory.  Block-uniform; barriers inside.
template <int VEC, bool OFF32, int DEPTH, bool MASKED>
__device__ __forceinline__ void shared_row(const SpmmArgs& a, int64_t row, uint32_t p_begin, uint32_t p_end,
                                           const SharedLanes& l, StagedEntry* __restrict__ s_A, int block)
{
    constexpr int D = DEPTH;
    constexpr uint32_t PARTS = 8;  // of the members' sums, added up side by side
    const int64_t N = a.N;
    const uint32_t lanes = l.lanes, members = l.members, member = l.member, chunk = l.chunk;
    Vec<VEC>* const s_part = reinterpret_cast<Vec<VEC>*>(s_A);  // of each thread
    static_assert(kRowSplitMaxBlock * sizeof(Vec<VEC>) <= kStageCap * sizeof(StagedEntry), "s_part");
    for (int64_t k0 = 0; k0 < N; k0 += (int64_t)lanes * VEC) {
        const int64_t k = k0 + (int64_t)chunk * VEC;
        const bool k_ok = k < N && member < members;
        const int64_t first = k_ok ? lane_first_col<VEC>(k, N) : 0;
        const std::conditional_t<MASKED, MaskedRows<VEC, OFF32>, GlobalRows<VEC, OFF32>> B(a.B, N, (uint32_t)first);
        Vec<VEC> acc;
        acc.zero();
        for (uint32_t base = p_begin; base < p_end; base += kStageCap) {
            const uint32_t cnt = p_end - base < (uint32_t)kStageCap ? p_end - base : (uint32_t)kStageCap;
            __syncthreads();
            stage_entries<8>(a.colidx + base, a.vals + base, cnt, s_A, block);
            __syncthreads();
            for (uint32_t q = member; k_ok && q < cnt; q += D * members) {
                Vec<VEC> b[D];
                if constexpr (MASKED) {
#pragma unroll
                    for (int u = 0; u < D; ++u) {
                        const uint32_t at = q + u * members;
                        b[u] = B.load(s_A[at < cnt ? at : q].col, at < cnt);
                    }
                    asm volatile("" ::: "memory");  // (the values are read meanwhile: registers)
#pragma unroll
                    for (int u = 0; u < D; ++u) {
                        const uint32_t at = q + u * members;
                        const float val = s_A[at < cnt ? at : q].val;
                        acc.fma(at < cnt ? val : 0.0f, b[u]);
                    }
                } else {
                    StagedEntry e[D];
#pragma unroll
                    for (int u = 0; u < D; ++u) {
                        e[u] = {0, 0.0f};
                        if (q + u * members < cnt) e[u] = s_A[q + u * members];
                    }
#pragma unroll
                    for (int u = 0; u < D; ++u) {
                        b[u].zero();
                        if (q + u * members < cnt) b[u] = B.load(e[u].col);
                    }
#pragma unroll
                    for (int u = 0; u < D; ++u) acc.fma(e[u].val, b[u]);
                }
            }
        }
        __syncthreads();  // the last entries are consumed
        uint32_t sums = PARTS < members ? PARTS : members;  // that the first member adds up, `lanes` places apart
        if ((lanes & (lanes - 1)) == 0) {
            // whole members in every wavefront: they hand their sums down
            for (int d = kWave / 2; d >= (int)lanes; d /= 2) {
#pragma unroll
                for (int i = 0; i < VEC; ++i) acc.v[i] += __shfl_down(acc.v[i], d, kWave);
            }
            sums = (uint32_t)block / kWave;
            if (threadIdx.x % kWave < lanes) s_part[threadIdx.x / kWave * lanes + chunk] = acc;
        } else {
            // member m of the first PARTS adds up those of m, m + PARTS, ...
            s_part[threadIdx.x] = acc;
            __syncthreads();
            if (member < PARTS && member < members) {
                for (uint32_t m = member + PARTS; m < members; m += PARTS) {
                    const Vec<VEC> other = s_part[m * lanes + chunk];
#pragma unroll
                    for (int i = 0; i < VEC; ++i) acc.v[i] += other.v[i];
                }
                s_part[threadIdx.x] = acc;
            }
        }
        __syncthreads();
        if (member == 0 && k_ok) {
            for (uint32_t m = 1; m < sums; ++m) {
                const Vec<VEC> other = s_part[m * lanes + chunk];
#pragma unroll
                for (int i = 0; i < VEC; ++i) acc.v[i] += other.v[i];
            }
            store_vec_stream<VEC>(a.C + row * N + first, acc);
        }
    }
}

// A finder's share of the rows (plan_row_split_grid): those that is_shared(row, entries) says, one after the other.  s_rp and
// s_mask: places for kRowCap rows and for a mask of every wavefront.
template <int VEC, bool OFF32, int DEPTH, bool MASKED, typename SHARED>
__device__ __forceinline__ void find_rows(const SpmmArgs& a, const RowSplitGrid& plan, SHARED&& is_shared, StagedEntry* __restrict__ s_A,
                                          int32_t* __restrict__ s_rp, unsigned long long* __restrict__ s_mask, int block)
{
    const int64_t N = a.N;
    constexpr uint32_t UNIT = FinderDeal::kUnit;
    const uint32_t team = blockIdx.x >> plan.log2_team, teams = (uint32_t)plan.finders >> plan.log2_team;
    const uint32_t mine = blockIdx.x & ((1u << plan.log2_team) - 1u);  // of the rows found, this one's turns
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    const uint32_t last = plan.deal.first_place(team + 1, teams);
    const SharedLanes lanes((N + VEC - 1) / VEC, block);
    for (uint32_t first = plan.deal.first_place(team, teams); first < last; first += kRowCap / UNIT) {
        const uint32_t look = (last - first < kRowCap / UNIT ? last - first : kRowCap / UNIT) * UNIT;
        uint32_t found = 0;  // the same in all members of the team, and in the same order
        for (uint32_t q0 = 0; q0 < look; q0 += block) {
            const uint32_t q = q0 + threadIdx.x;
            const int64_t r = plan.deal.row(first + q / UNIT, q % UNIT);
            bool shared = q < look && r < a.M;
            if (shared) shared = is_shared(r, a.rowptr[r + 1] - a.rowptr[r]);
            const unsigned long long mask = __ballot(shared);
            __syncthreads();  // the last rows found, or the last masks, are done with
            if (lane == 0) s_mask[wave] = mask;
            __syncthreads();
            uint32_t rank = found + (uint32_t)__popcll(mask & ((1ull << lane) - 1ull));
            for (int w = 0; w < block / kWave; ++w) {
                const uint32_t c = (uint32_t)__popcll(s_mask[w]);
                if (w < wave) rank += c;
                found += c;
            }
            if (shared && (rank & ((1u << plan.log2_team) - 1u)) == mine) s_rp[rank >> plan.log2_team] = (int32_t)r;
        }
        __syncthreads();
        const int n = (int)((found + (1u << plan.log2_team) - 1u - mine) >> plan.log2_team);
        for (int i = 0; i < n; ++i) {
            const int32_t row = __builtin_amdgcn_readfirstlane(s_rp[i]);
            shared_row<VEC, OFF32, DEPTH, MASKED>(a, row, (uint32_t)a.rowptr[row], (uint32_t)a.rowptr[row + 1], lanes, s_A, block);
        }
    }
}

// PARTIAL: the G members of a row reduce in sub-groups of `reduce_members`
// (a power of two below G) and the first member of every sub-group adds its
// sum to C with atomics; C must hold zeros before the launch.
// SKIP: leave the rows described by `skip` alone.
// grid (plan_row_split_grid; G > 1, whole-group reductions): rows of at least share_from stored entries are left out of
// the walk; the first `finders` workgroups of the grid look for them, a team of them in each share of the rows
// (FinderDeal), and produce them in turn, one after the other with all their lanes (shared_row).  They start first, so that the longest rows are done while
// the others are walked: a workgroup that came across one during its walk ended some 40 us behind the rest.
// DEEP: the rows that a workgroup takes together have more loads in flight, with registers that leave five wavefronts per SIMD, one
// less (launch_row_split).
// The workgroup size (the paper's blockSz, Section 7.2) is the launch's: SLOTS = blockDim.x / (G*LC)
// groups work side by side on the rows of a row block.
template <int G, int LC, int VEC, bool OFF32, bool PARTIAL, bool SKIP, int DEPTH, bool DEEP>
__global__ __launch_bounds__(kRowSplitMaxBlock)
__attribute__((amdgpu_waves_per_eu(2, DEEP ? 5 : 8)))
void row_split_kernel(SpmmArgs a, TileSched ts, int rows_per_slot, int interleave, int reduce_members, RowSplitGrid plan, RowSkip skip)
{
    __shared__ StagedEntry s_A[kStageCap];
    __shared__ int32_t s_rp[kRowCap + 1];
    constexpr bool SHARE = G > 1 && !PARTIAL;
    __shared__ unsigned long long s_mask[kRowSplitMaxBlock / kWave];
    // entries per thread in flight to LDS: single lanes' row blocks have one or two for each thread, and the registers of
    // four would cost the instance a wavefront per SIMD (stencil of 1,048,576 rows, N = 128: 602 us against 593)
    constexpr int STAGED = G == 1 && DEPTH == kDepthRows ? 1 : 4;
    constexpr int SPAN = G * LC;
    const int block = blockDim.x;
    const int SLOTS = block / SPAN;

    const int slot = threadIdx.x / SPAN;
    const int member = (threadIdx.x / LC) % G;
    const int chunk = threadIdx.x % LC;
    const int64_t N = a.N;
    const int64_t rows_per_block = (int64_t)SLOTS * rows_per_slot;
    const bool rp_in_lds = rows_per_block <= kRowCap;
    bool skip_on = false;
    if constexpr (SKIP) skip_on = *skip.count <= skip.max_rows;

    if constexpr (SHARE) {
        if ((int)blockIdx.x < plan.finders) {
            const int32_t skip_from = SKIP && skip_on ? skip.min_len : 0x7fffffff;
            find_rows<VEC, OFF32, DEPTH, DEEP>(a, plan, [&](int64_t, int32_t len) { return len >= plan.share_from && len < skip_from; }, s_A, s_rp,
                                         s_mask, block);
            if ((int)blockIdx.x < plan.walk_from) return;
        }
    }

    // persistent walk over this die's run of work items
    const int64_t wg = blockIdx.x - plan.walk_from;
    const int64_t xcd = wg % ts.xcds;
    const int64_t wg_in_xcd = wg / ts.xcds;
    const int64_t wgs_per_xcd = (gridDim.x - plan.walk_from) / ts.xcds;
    for (int64_t it = wg_in_xcd; it < ts.items_per_xcd; it += wgs_per_xcd) {
        const int64_t item = xcd * ts.items_per_xcd + it;
        if (item >= ts.items) break;
        const int32_t col_tile = (int32_t)(item / ts.row_blocks);
        const int64_t row_block = item % ts.row_blocks;

        const int64_t row_first = row_block * rows_per_block;
        const int64_t row_last = row_first + rows_per_block < a.M ? row_first + rows_per_block : a.M;
        // this slot's rows, counted from row_first: my_first, my_first + row_step, ... below my_last
        // (32-bit: a row block has at most SLOTS * rows_per_slot rows)
        const int32_t block_rows = (int32_t)(row_last - row_first);
        const int32_t row_step = interleave ? SLOTS : 1;
        int32_t my_first = interleave ? slot : slot * rows_per_slot;
        int32_t my_last = interleave ? block_rows : my_first + rows_per_slot;
        if (my_first > block_rows) my_first = block_rows;
        if (my_last > block_rows) my_last = block_rows;

        __syncthreads();  // everyone is done with the previous item's LDS contents
        uint32_t nz_first, nz_last;
        if (rp_in_lds) {
            for (int i = threadIdx.x; i <= block_rows; i += block)
                s_rp[i] = a.rowptr[row_first + i];
            __syncthreads();
            nz_first = (uint32_t)__builtin_amdgcn_readfirstlane(s_rp[0]);  // the same in all lanes: scalar registers
            nz_last = (uint32_t)__builtin_amdgcn_readfirstlane(s_rp[block_rows]);
        } else {
            nz_first = (uint32_t)a.rowptr[row_first];
            nz_last = (uint32_t)a.rowptr[row_last];
        }
        const bool one_chunk = nz_last - nz_first <= (uint32_t)kStageCap;

        const int64_t k_tile_end =
            (int64_t)(col_tile + 1) * ts.tile_cols < N ? (int64_t)(col_tile + 1) * ts.tile_cols : N;
        // a tile may be wider than one pass of the LC chunk lanes
        for (int64_t k0 = (int64_t)col_tile * ts.tile_cols; k0 < k_tile_end; k0 += (int64_t)LC * VEC) {
            const int32_t k = (int32_t)k0 + chunk * VEC;  // N < 2^31
            const bool k_ok = k < k_tile_end;
            const int32_t k_lane = k_ok ? (int32_t)lane_first_col<VEC>((uint32_t)k, (uint32_t)N) : 0;  // the VEC columns this lane holds
            const GlobalRows<VEC, OFF32> Brow(a.B, N, k_lane);

            int32_t row = my_first;
            Vec<VEC> acc;
            acc.zero();
            for (uint32_t base = nz_first;; base += kStageCap) {  // runs at least once: empty rows get stored
                const uint32_t cnt = nz_last - base < (uint32_t)kStageCap ? nz_last - base : (uint32_t)kStageCap;
                const bool staged = one_chunk && k0 != (int64_t)col_tile * ts.tile_cols;  // by the pass before
                if (!staged) {
                    if (base != nz_first || k0 != (int64_t)col_tile * ts.tile_cols) __syncthreads();
                    stage_entries<STAGED>(a.colidx + base, a.vals + base, cnt, s_A, block);
                    __syncthreads();
                }
                // rows of this slot that have entries in the chunk (or are empty)
                while (row < my_last) {
                    uint32_t p_begin, p_end;
                    if (rp_in_lds) {
                        p_begin = (uint32_t)s_rp[row];
                        p_end = (uint32_t)s_rp[row + 1];
                    } else {
                        p_begin = (uint32_t)a.rowptr[row_first + row];
                        p_end = (uint32_t)a.rowptr[row_first + row + 1];
                    }
                    const uint32_t lo = p_begin > base ? p_begin : base;
                    const uint32_t hi = p_end < base + cnt ? p_end : base + cnt;
                    bool skipped = false;
                    if constexpr (SKIP) skipped = skip_on && p_end - p_begin >= (uint32_t)skip.min_len;
                    if constexpr (SHARE) skipped = skipped || p_end - p_begin >= (uint32_t)plan.share_from;
                    if (!skipped && k_ok && lo < hi) {
                        // first position >= lo that belongs to this member
                        const uint32_t first = lo + ((member - (lo - p_begin)) & (G - 1));
                        if (first < hi) gather_fma<VEC, G, DEPTH>(acc, s_A, first - base, hi - base, Brow);
                    }
                    if (p_end > base + cnt) break;  // the row continues in the next chunk
                    // members without entries contributed +0 (zero extension);
                    // the lanes of a slot reach this point together
                    if constexpr (PARTIAL) {
#pragma unroll
                        for (int i = 0; i < VEC; ++i)
                            acc.v[i] = group_partial_sum<G, LC>(acc.v[i], reduce_members * LC);
                        from_last_columns<VEC>(acc, k - k_lane);
                        // a sub-group whose first member has no entry of the row holds +0
                        const bool adds = (member & (reduce_members - 1)) == 0 && (uint32_t)member < p_end - p_begin;
                        if constexpr (LC >= VEC) {
                            // The LC chunk lanes of a member hold LC*VEC consecutive columns, VEC per
                            // lane.  An atomic instruction whose lanes are 16 bytes apart costs four
                            // times one over consecutive words (451 against 115 clocks of the memory
                            // pipeline, measured), so the sums change hands first: in round q lane c
                            // adds column q*LC + c, which lane (q*LC + c) / VEC of the member holds.
#pragma unroll
                            for (int q = 0; q < VEC; ++q) {
                                const int col = q * LC + chunk;
                                float mine = 0.0f;
#pragma unroll
                                for (int v = 0; v < VEC; ++v) {
                                    const float t = __shfl(acc.v[v], col / VEC, LC);
                                    if (col % VEC == v) mine = t;
                                }
                                if (adds && k0 + col < k_tile_end)
                                    unsafeAtomicAdd(a.C + (row_first + row) * N + k0 + col, mine);
                            }
                        } else {
                            if (adds && k_ok) {
#pragma unroll
                                for (int i = 0; i < VEC; ++i)
                                    if (k + i < k_tile_end) unsafeAtomicAdd(a.C + (row_first + row) * N + k + i, acc.v[i]);
                            }
                        }
                    } else {
#pragma unroll
                        for (int i = 0; i < VEC; ++i) acc.v[i] = group_tree_sum<G, LC>(acc.v[i]);
                        if (member == 0 && k_ok && !skipped) store_vec_stream<VEC>(a.C + (row_first + row) * N + k_lane, acc);
                    }
                    acc.zero();
                    row += row_step;
                }
                if (base + cnt >= nz_last) break;
            }
        }
    }
}

namespace row_split_detail {

template <bool PARTIAL, bool SKIP = false>
struct Launch {
    const SpmmArgs& a;
    int rows_per_slot, interleave, tile_cols, xcds, compute_units;
    bool off32, persistent;
    int reduce_members;
    int block;  // threads per workgroup: 128, 256 or 512 (at least G*LC)
    hipStream_t s;
    int64_t nnz_hint;  // stored entries, -1 = unknown
    bool short_rows;  // rows of kShortRowMean entries or fewer in the mean
    RowSkip skip = {nullptr, 0, 0};
    bool deep = false;  // the instance for rows that workgroups take together, where there is one

    // workgroups of this instance that one compute unit can hold at once
    template <typename K>
    static int resident_per_cu(K kernel, int block)
    {
        int n = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, block, 0) != hipSuccess || n < 1) n = 1;
        return n;
    }

    template <int G, int LC, int VEC>
    void operator()() const
    {
        if constexpr (G > 1 && !PARTIAL && !SKIP && VEC == 4 && LC > 2 && G * LC == kWave) {
            if (deep) go<G, LC, VEC, kDepthGroups, true>();
            else go<G, LC, VEC, kDepthGroups>();
        } else if constexpr (G > 1) go<G, LC, VEC, kDepthGroups>();
        else if constexpr (SKIP) go<G, LC, VEC, kDepthRows>();
        else if (short_rows) go<G, LC, VEC, kDepthShort>();
        else go<G, LC, VEC, kDepthRows>();
    }

    template <int G, int LC, int VEC, int DEPTH, bool DEEP = false>
    void go() const
    {
        // a persistent grid must be resident all at once (asked of the runtime only for such launches)
        int resident = 0;
        if (persistent)
            resident = compute_units * (off32 ? resident_per_cu(row_split_kernel<G, LC, VEC, true, PARTIAL, SKIP, DEPTH, DEEP>, block)
                                              : resident_per_cu(row_split_kernel<G, LC, VEC, false, PARTIAL, SKIP, DEPTH, DEEP>, block));
        const int slots = block / (G * LC);
        const int64_t rows_per_block = (int64_t)slots * rows_per_slot;
        TileSched ts;
        ts.row_blocks = (a.M + rows_per_block - 1) / rows_per_block;
        ts.tile_cols = tile_cols;
        ts.col_tiles = (int32_t)((a.N + tile_cols - 1) / tile_cols);
        ts.items = ts.row_blocks * ts.col_tiles;
        ts.xcds = xcds;
        ts.items_per_xcd = (ts.items + xcds - 1) / xcds;
        const int passes = (int)(((int64_t)tile_cols + LC * VEC - 1) / (LC * VEC));
        const RowSplitGrid plan =
            plan_row_split_grid(PARTIAL ? 1 : G, passes, a.M, ts.items, xcds, compute_units, nnz_hint, resident);
        const uint32_t grid = plan.grid;
        if (off32)
            hipLaunchKernelGGL((row_split_kernel<G, LC, VEC, true, PARTIAL, SKIP, DEPTH, DEEP>), dim3(grid), dim3(block), 0, s, a,
                               ts, rows_per_slot, interleave, reduce_members, plan, skip);
        else
            hipLaunchKernelGGL((row_split_kernel<G, LC, VEC, false, PARTIAL, SKIP, DEPTH, DEEP>), dim3(grid), dim3(block), 0, s, a,
                               ts, rows_per_slot, interleave, reduce_members, plan, skip);
    }
};

}  // namespace row_split_detail

}  // namespace sgap
