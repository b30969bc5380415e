// Row-split schedule, serial strategy, for rows that share columns with their neighbours (grids, meshes, bands): four
// consecutive rows ("a quad") go together, and a row of B that several of them want is gathered once.
//
// What bounds the plain row-split kernel on such matrices is the vector-memory path: a 27-point stencil gathers 27 rows of
// B per row of A, although four neighbouring rows want 54 distinct ones and not 108.  Here the LC lanes that hold a
// quad's columns first list those distinct rows of B in LDS, a lane per stored entry.  A record is a column and the four
// rows' values, +0 where a row has no such entry; an entry opens one unless the row above (its columns ascend) has the
// column too, and the records lie in the order of their columns, since an entry finds its record by counting what
// opens below its column in each of the four rows.  (A column that row i has, row i - 1 lacks and row i - 2 had is opened
// twice: both entries go into one record, and a place behind it stays empty.)  Then every record costs one gather and four
// v_mfma_f32_4x4x1: four rows' values times the four columns of each lane.
//
// 27-point stencil of 1,000,000 rows, N = 128: 593 -> 419 us (N = 64 288 -> 242, N = 256 1,218 -> 853; 90 x 40 x 95 points,
// N = 128 179 -> 134).  By steps: listed in the order of opening, fp32 multiply-adds 499; on the matrix cores, which halves
// the vector instructions, 493; planes dealt over the dies (die_block) 450, L2 misses 19.9 M -> 10.9 M lines; in the order
// of the columns, so that neighbouring quads ask for a line at the same time and the L1 answers one of them, 430, L1 misses
// 56.0 M -> 44.7 M.  What is left is those: a compute unit's L1 has 256 lines to wait in, and 44.7 M of them at some 0.5 us
// each take 0.36 ms.  More rows of B in flight (9, 12) or workgroups that go on to further rows with the next entries on
// their way gain nothing (430 to 530 us).
//
// +0 times a finite element of B adds nothing; an infinity or a NaN would.  A quad with a sum that is not finite is
// therefore done again row by row, as is, from the start, a quad with a row of kQuadRow entries or more, a row that
// does not ascend, or too little to share.  Nothing is assumed of the matrix.
#include "sgap_common.hpp"
#include "sgap_gather.hpp"
#include "sgap_quads.hpp"

namespace sgap {

namespace {

constexpr int kQuadRecords = 64;  // records of a quad at most (27-point stencil: 54)
constexpr int kQuadPlaces = 80;   // those, +0 up to a whole batch behind them, and in the last place what belongs to none
constexpr int kQuadChunk = 160;   // entries staged at a time where rows go one by one
constexpr int kQuadDepth = 6;     // rows of B in flight per lane
constexpr int kPlainDepth = 8;    // the same where rows go one by one
static_assert(kQuadRecords + kQuadDepth < kQuadPlaces, "a batch of +0 behind the records");

struct alignas(16) QuadLds {
    union {
        struct {
            float val[kQuadPlaces][kQuad];
            int32_t col[kQuadPlaces];
        } rec;
        StagedEntry staged[kQuadChunk];
    };
    int32_t row_col[kQuad][1 + kQuadRow];  // the rows' columns from place 1 on, kNoColumn behind them
};

__device__ __forceinline__ bool finite(float x) { return (__float_as_uint(x) & 0x7f800000u) != 0x7f800000u; }

// U records from number q on: all U rows of B are requested before the first is consumed.  acc[j][i] is row i's sum in this
// lane's column j: v_mfma_f32_4x4x1 multiplies, for every four lanes by themselves, the four rows' values (one per lane)
// with one element of B per lane.  It takes no notice of the lanes switched off, so the whole wavefront comes here.
// TAIL: records from `records` on are +0 times +0.
template <int U, bool TAIL, bool OFF32>
__device__ __forceinline__ void quad_batch(f32x4 (&acc)[4], const QuadLds& lds, int q, int records, int row,
                                           const GlobalRows<4, OFF32>& B)
{
    Vec<4> b[U];
    float v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if constexpr (TAIL) {
            b[u].zero();
            if (q + u < records) b[u] = B.load(lds.rec.col[q + u]);
        } else {
            b[u] = B.load(lds.rec.col[q + u]);
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        v[u] = 0.0f;
        if (!TAIL || q + u < records) v[u] = lds.rec.val[q + u][row];
    }
    __builtin_amdgcn_sched_barrier(0);  // or the last loads wait for the first products
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j] = __builtin_amdgcn_mfma_f32_4x4x1f32(v[u], b[u].v[j], acc[j], 0, 0, 0);
}

}  // namespace

template <int LC, bool OFF32>
__global__ __launch_bounds__(kBlock) void row_quads_kernel(SpmmArgs a, TileSched ts)
{
    constexpr int SLOTS = kBlock / LC;
    constexpr int EPL = LC < kQuadRow ? kQuadRow / LC : 1;  // entries of a row per lane
    constexpr unsigned long long SLOT_MASK = LC == 64 ? ~0ull : (1ull << LC) - 1ull;
    __shared__ QuadLds s_lds[SLOTS];

    const int slot = threadIdx.x / LC;
    const int t = threadIdx.x % LC;
    const int shift = (threadIdx.x % kWave) / LC * LC;
    QuadLds& lds = s_lds[slot];
    auto slot_ballot = [&](bool p) { return (__ballot(p) >> shift) & SLOT_MASK; };

    const uint32_t row_blocks = (uint32_t)ts.row_blocks;  // (fit 32 bits: launch_row_quads)
    const uint32_t per_die = (row_blocks + ts.xcds - 1) / ts.xcds;
    const uint32_t die = blockIdx.x % ts.xcds, turn = blockIdx.x / ts.xcds;
    const uint32_t col_tile = turn / per_die;
    const uint32_t share = (plane_share(a, ts.xcds, (uint32_t)(a.N < ts.tile_cols ? a.N : ts.tile_cols) * 4u) + SLOTS * kQuad / 2) / (SLOTS * kQuad);
    const uint32_t block = die_block(share, die, turn % per_die, row_blocks, ts.xcds);
    if (block >= row_blocks) return;  // the whole workgroup
    const int64_t row_first = ((int64_t)block * SLOTS + slot) * kQuad;

    const uint32_t k_end = (uint32_t)((int64_t)(col_tile + 1) * ts.tile_cols < a.N ? (int64_t)(col_tile + 1) * ts.tile_cols : a.N);
    const uint32_t k = col_tile * (uint32_t)ts.tile_cols + t * 4;
    const bool k_ok = k < k_end;
    // (a lane without columns reads the last ones of the tile, and nothing of it is stored)
    const uint32_t k_lane = k_ok ? lane_first_col<4>(k, (uint32_t)a.N) : k_end - 4;
    const GlobalRows<4, OFF32> B(a.B, a.N, k_lane);

    // rows past the last one have no entries and are not stored
    int32_t p[kQuad + 1];
    {
        const int64_t r = row_first + (t <= kQuad ? t : kQuad);
        const int32_t mine = a.rowptr[r < a.M ? r : a.M];
#pragma unroll
        for (int i = 0; i <= kQuad; ++i) p[i] = __shfl(mine, i, LC);
    }
    bool listed = true;
#pragma unroll
    for (int i = 0; i < kQuad; ++i) listed = listed && p[i + 1] - p[i] < kQuadRow;
    const bool staged = listed;  // in registers, and in LDS where the rows go one by one
    int records = 0;
    {
        int32_t col[kQuad][EPL];
        float val[kQuad][EPL];
#pragma unroll
        for (int i = 0; i < kQuad; ++i)
#pragma unroll
            for (int u = 0; u < EPL; ++u) {
                const int q = t + u * LC;
                col[i][u] = kNoColumn;
                val[i][u] = 0.0f;
                if (staged && q < p[i + 1] - p[i]) {
                    col[i][u] = load_stream(a.colidx + p[i] + q);
                    val[i][u] = load_stream(a.vals + p[i] + q);
                }
            }
        // Nothing below is left out by a lane on its own: every lane of the wavefront comes by every ballot and shuffle.
#pragma unroll
        for (int i = 0; i < kQuad; ++i)
#pragma unroll
            for (int u = 0; u < EPL; ++u) {
                const int q = t + u * LC;
                if (q < kQuadRow) lds.row_col[i][1 + q] = col[i][u];
                if (q == 0) lds.row_col[i][0] = -1;
            }
        wave_lds_order();
        // columns without order, told by the second row and the first, or else (where a line of the grid ends between them) by
        // the fourth and the third: nothing is listed (300,000 rows of 27 entries, N = 64: 299 us where they were, 294 so, 287
        // by the plain kernel; N = 128: 605, 587 and 593; the second look: 75 x 75 x 30 points, N = 36 56.9 -> 49.1, by the plain
        // kernel 49.6; 99 x 97 x 31, N = 56 88.9 -> 81.1, by that 88.9)
        auto shares = [&](const int32_t* __restrict__ above, const int32_t (&row)[EPL], int32_t entries) {
            int seen = 0;
#pragma unroll
            for (int u = 0; u < EPL; ++u) {
                const int lo = below(above + 1, row[u]);
                seen += __popc((uint32_t)slot_ballot(row[u] != kNoColumn && above[1 + lo] == row[u]));
            }
            return 4 * seen >= entries;
        };
        bool some_shared = shares(lds.row_col[0], col[1], p[2] - p[1]);
        if (__ballot(listed && !some_shared) != 0) {
            const bool others = shares(lds.row_col[2], col[3], p[4] - p[3]);
            some_shared = some_shared || others;
        }
        listed = listed && some_shared;
        if (__ballot(listed) != 0) {
            // (an empty place counts as a record of the quad's first column and of no row)
            int32_t some = kNoColumn;
#pragma unroll
            for (int i = kQuad - 1; i >= 0; --i) {
                const int32_t first = __shfl(col[i][0], 0, LC);
                some = first != kNoColumn ? first : some;
            }
#pragma unroll
            for (int q = t; q < kQuadPlaces; q += LC) {
                *reinterpret_cast<float4*>(lds.rec.val[q]) = float4{0.0f, 0.0f, 0.0f, 0.0f};
                lds.rec.col[q] = some;
            }
            wave_lds_order();
            int before[kQuad][EPL][kQuad];  // of row j, the columns below this one
            uint32_t opens[kQuad];          // bit q: the row's entry q opens a record
            bool descends = false;
#pragma unroll
            for (int i = 0; i < kQuad; ++i) {
                opens[i] = 0;
#pragma unroll
                for (int u = 0; u < EPL; ++u) {
                    const int q = t + u * LC;
                    const int32_t c = col[i][u];
                    const bool have = c != kNoColumn;
                    descends = descends || (have && lds.row_col[i][q < kQuadRow ? q : 0] >= c);
#pragma unroll
                    for (int j = 0; j < kQuad; ++j) {
                        const int32_t* __restrict__ row = lds.row_col[j] + 1;
                        before[i][u][j] = j == i ? q : below(row, c);
                    }
                    const bool found = i > 0 && have && lds.row_col[i > 0 ? i - 1 : 0][1 + before[i][u][i > 0 ? i - 1 : 0]] == c;
                    const uint32_t here = (uint32_t)slot_ballot(have && !found);
                    opens[i] |= here << (u * LC % kQuadRow);
                }
                records += __popc(opens[i]);
            }
#pragma unroll
            for (int i = 0; i < kQuad; ++i)
#pragma unroll
                for (int u = 0; u < EPL; ++u) {
                    int mine = 0;
#pragma unroll
                    for (int j = 0; j < kQuad; ++j) mine += __popc(opens[j] & ((1u << (before[i][u][j] & 31)) - 1u));
                    mine = col[i][u] != kNoColumn && mine < kQuadRecords ? mine : kQuadPlaces - 1;
                    lds.rec.col[mine] = col[i][u];
                    lds.rec.val[mine][i] = val[i][u];
                }
            // worth it from a quarter shared on
            listed = listed && slot_ballot(descends) == 0 && records <= kQuadRecords && 4 * records <= 3 * (p[kQuad] - p[0]);
        }
        wave_lds_order();
        if (staged && !listed) {
            // row i's entries from kQuadRow * i on
#pragma unroll
            for (int i = 0; i < kQuad; ++i)
#pragma unroll
                for (int u = 0; u < EPL; ++u)
                    if (t + u * LC < kQuadRow) lds.staged[kQuadRow * i + t + u * LC] = StagedEntry{col[i][u], val[i][u]};
        }
        wave_lds_order();
    }
    const bool in_lds = staged && !listed;

    bool done = false;
    if (__ballot(listed) != 0) {
        f32x4 acc[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        // the wavefront's quads go through their records together
        const int mine = listed ? (records + kQuadDepth - 1) / kQuadDepth * kQuadDepth : 0;
        int fewest = kQuadPlaces, most = 0;
#pragma unroll
        for (int l = 0; l < kWave; l += LC) {
            const int theirs = __builtin_amdgcn_readlane(mine, l);
            fewest = theirs < fewest ? theirs : fewest;
            most = theirs > most ? theirs : most;
        }
        int q = 0;
        for (; q + kQuadDepth <= fewest; q += kQuadDepth) quad_batch<kQuadDepth, false>(acc, lds, q, mine, t % kQuad, B);
        for (; q < most; q += kQuadDepth) quad_batch<kQuadDepth, true>(acc, lds, q, mine, t % kQuad, B);
        bool good = true;
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int i = 0; i < kQuad; ++i) good = good && finite(acc[j][i]);
        done = listed && slot_ballot(!good) == 0;
        if (done && k_ok) {
#pragma unroll
            for (int i = 0; i < kQuad; ++i) {
                Vec<4> sum;
#pragma unroll
                for (int j = 0; j < 4; ++j) sum.v[j] = acc[j][i];
                if (row_first + i < a.M) store_vec_stream<4>(a.C + (row_first + i) * a.N + k_lane, sum);
            }
        }
    }
    if (!done) {
        for (int i = 0; i < kQuad && row_first + i < a.M; ++i) {
            int32_t begin = p[0], end = p[1];
            if (i == 1) { begin = p[1]; end = p[2]; }
            if (i == 2) { begin = p[2]; end = p[3]; }
            if (i == 3) { begin = p[3]; end = p[4]; }
            Vec<4> acc;
            acc.zero();
            for (int32_t base = begin; base < end; base += kQuadChunk) {
                const int32_t cnt = end - base < kQuadChunk ? end - base : kQuadChunk;
                if (!in_lds) {
                    wave_lds_order();
                    for (int q = t; q < cnt; q += LC) {
                        StagedEntry e;
                        e.col = load_stream(a.colidx + base + q);
                        e.val = load_stream(a.vals + base + q);
                        lds.staged[q] = e;
                    }
                    wave_lds_order();
                }
                const uint32_t at = in_lds ? kQuadRow * i : 0;
                if (k_ok) gather_fma<4, 1, kPlainDepth>(acc, lds.staged, at, at + (uint32_t)cnt, B);
            }
            if (k_ok) store_vec_stream<4>(a.C + (row_first + i) * a.N + k_lane, acc);
        }
    }
}

// Rows of more than a dozen entries and of no more than kQuadRow in the mean, whose columns take 16 lanes or more: on those
// nothing is lost where the quads turn out to share nothing (in the kernel, and 100,000 rows of 31 entries, N = 128: 215 us
// by the plain kernel, 213 so).  Enough blocks of rows for the chip, since a quad's rows are one after the other then: 312
// blocks of 64 rows of 20 entries without order take 17 us and 12 by the plain kernel, 938 of 16 entries 31.1 and 30.9;
// stencils gain from 844 blocks of 32 rows on (N = 128: 17.3 -> 14.2 us) and from 938 of 64 (19.1 -> 18.2).
// A column tile has to fit one pass of its lanes: the kernel makes no second one (row_split_kernel does).
bool row_quads_apply(const SpmmArgs& a, int lc, int64_t tile_cols, double mean_row, int compute_units)
{
    if (tile_cols > (int64_t)lc * 4) return false;
    const int64_t blocks = a.M / ((int64_t)(kBlock / lc) * kQuad);
    return lc >= 16 && mean_row > 12.0 && mean_row <= (double)kQuadRow && blocks >= (int64_t)(lc >= 32 ? 3 : 5) * compute_units;
}

// lc = chunk lanes that hold a column tile in one pass (16, 32 or 64)
hipError_t launch_row_quads(const SpmmArgs& a, int lc, int tile_cols, int xcds, hipStream_t s)
{
    if (tile_cols > lc * 4) return hipErrorInvalidValue;
    const int64_t rows = (int64_t)(kBlock / lc) * kQuad;
    TileSched ts;
    ts.row_blocks = (a.M + rows - 1) / rows;
    ts.tile_cols = tile_cols;
    ts.col_tiles = (int32_t)((a.N + tile_cols - 1) / tile_cols);
    ts.items = ts.row_blocks * ts.col_tiles;
    ts.xcds = xcds;
    ts.items_per_xcd = (ts.row_blocks + xcds - 1) / xcds * ts.col_tiles;
    if (ts.items_per_xcd * xcds > 0x7fffffffLL) return hipErrorInvalidValue;
    const dim3 grid((uint32_t)(ts.items_per_xcd * xcds)), block(kBlock);
    const bool off32 = offsets_fit_32(a);
    if (lc == 16 && off32) hipLaunchKernelGGL((row_quads_kernel<16, true>), grid, block, 0, s, a, ts);
    else if (lc == 16) hipLaunchKernelGGL((row_quads_kernel<16, false>), grid, block, 0, s, a, ts);
    else if (lc == 32 && off32) hipLaunchKernelGGL((row_quads_kernel<32, true>), grid, block, 0, s, a, ts);
    else if (lc == 32) hipLaunchKernelGGL((row_quads_kernel<32, false>), grid, block, 0, s, a, ts);
    else if (lc == 64 && off32) hipLaunchKernelGGL((row_quads_kernel<64, true>), grid, block, 0, s, a, ts);
    else if (lc == 64) hipLaunchKernelGGL((row_quads_kernel<64, false>), grid, block, 0, s, a, ts);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace sgap
