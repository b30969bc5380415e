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
// 27-point stencil of 1,000,000 rows, N = 128: 589 -> 418 us (N = 64 286 -> 238, N = 256 1,217 -> 849; 212,040 rows, N = 128 112 ->
// 81).  By steps: listed in the order of opening, fp32 multiply-adds 499; on the matrix cores, which halves
// the vector instructions, 493; planes dealt over the dies (die_block) 450, L2 misses 19.9 M -> 10.9 M lines; in the order
// of the columns, so that neighbouring quads ask for a line at the same time and the L1 answers one of them, 430, L1 misses
// 56.0 M -> 44.7 M.  What is left is those: a compute unit's L1 has 256 lines to wait in, and 44.7 M of them at some 0.5 us
// each take 0.36 ms.  More rows of B in flight (9, 12) or workgroups that go on to further rows with the next entries on
// their way gain nothing (430 to 530 us).
//
// A wavefront lists its quads where all of their rows have fewer than kQuadRow entries and share columns.  The rows of the others,
// and of quads that turn out not to be worth it, are taken one by one by all the workgroup's slots, with their entries in LDS: where
// a slot took its own quad's rows it kept the others waiting, and read entry by entry.  us by row_split_kernel, that way and so: a
// mesh of three unknowns a node and 7 to 11 neighbours, 300,000 rows, a third of them of 32 entries or more, N = 64 102, 187 and
// 103, N = 128 175, 250 and 163; power law, 1,000,000 rows, N = 64 890, 1,170 and 810; rows of 27 neighbouring columns and one in
// eight of 40, 400,000 rows, N = 128 227, 280 and 194.  Five wavefronts per SIMD: with four, as the compiler has it by itself in 16
// lanes, the stencil takes 235 us at N = 40 and 245 at N = 64 (214 and 236 with five); with six (and six rows of B in flight) N = 128
// took 457 against 428.
//
// +0 times a finite element of B adds nothing; an infinity or a NaN would.  A quad with a sum that is not finite is
// therefore done again row by row.  Nothing is assumed of the matrix.
#include "sgap_common.hpp"
#include "sgap_gather.hpp"
#include "sgap_quads.hpp"

namespace sgap {

namespace {

constexpr int kQuadRecords = 64;  // records of a quad at most (27-point stencil: 54)
constexpr int kQuadPlaces = 80;   // those, +0 up to a whole batch behind them, and in the last place what belongs to none
constexpr int kQuadChunk = 160;   // entries of a quad whose rows go one by one that are in LDS together
constexpr int kQuadDepth = 6;     // rows of B in flight per lane
constexpr int kPlainDepth = 8;    // the same where rows go one by one
static_assert(kQuadRecords + kQuadDepth < kQuadPlaces, "a batch of +0 behind the records");

struct alignas(16) QuadLds {
    union {
        int32_t row_col[kQuad][1 + kQuadRow];  // the rows' columns from place 1 on, kNoColumn behind them
        struct {
            float val[kQuadPlaces][kQuad];
            int32_t col[kQuadPlaces];
        } rec;
        StagedEntry staged[kQuadChunk];  // where rows go one by one
    };
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
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(5))) void row_quads_kernel(SpmmArgs a, TileSched ts)
{
    constexpr int SLOTS = kBlock / LC;
    constexpr int EPL = LC < kQuadRow ? kQuadRow / LC : 1;  // entries of a row per lane
    constexpr int EACH = (kQuadChunk + LC - 1) / LC;         // the same of kQuadChunk
    constexpr int NEXT = EACH < 5 ? EACH : 5;                // entries per lane in flight to LDS where a row goes by itself,
    constexpr int32_t CHUNK = NEXT * LC < kQuadChunk ? NEXT * LC : kQuadChunk;  // of a slot
    constexpr unsigned long long SLOT_MASK = LC == 64 ? ~0ull : (1ull << LC) - 1ull;
    __shared__ QuadLds s_lds[SLOTS];
    __shared__ int32_t s_ptr[SLOTS][kQuad + 1];  // of the quads, for rows that go one by one
    __shared__ unsigned long long s_open[kWavesPerBlock], s_read[kWavesPerBlock];  // bit: lane, of a quad that is open; and not in LDS

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
    bool listed;
    {
        bool shorts = true;
#pragma unroll
        for (int i = 0; i < kQuad; ++i) shorts = shorts && p[i + 1] - p[i] < kQuadRow;
        listed = __ballot(!shorts) == 0;  // all quads of the wavefront, or none
    }
    const bool loaded = listed;  // into registers
    int records = 0;
    if (loaded) {
        int32_t col[kQuad][EPL];
        float val[kQuad][EPL];
#pragma unroll
        for (int i = 0; i < kQuad; ++i)
#pragma unroll
            for (int u = 0; u < EPL; ++u) {
                const int q = t + u * LC;
                col[i][u] = kNoColumn;
                val[i][u] = 0.0f;
                if (q < p[i + 1] - p[i]) {
                    col[i][u] = load_stream(a.colidx + p[i] + q);
                    val[i][u] = load_stream(a.vals + p[i] + q);
                }
            }
        // Nothing below is left out by a lane on its own: every lane of the wavefront comes by every ballot and shuffle.
        auto put_columns = [&] {
#pragma unroll
            for (int i = 0; i < kQuad; ++i)
#pragma unroll
                for (int u = 0; u < EPL; ++u) {
                    const int q = t + u * LC;
                    if (q < kQuadRow) lds.row_col[i][1 + q] = col[i][u];
                    if (q == 0) lds.row_col[i][0] = -1;
                }
            wave_lds_order();
        };
        // whether a row shares columns with the row above: half of them, at its own place or the next one above (16 lanes), or a
        // quarter, wherever
        auto shares = [&](int above) {
            const int32_t (&row)[EPL] = col[above + 1];
            int seen = 0;
#pragma unroll
            for (int u = 0; u < EPL; ++u) {
                bool found;
                if constexpr (LC == 16) {
                    const int32_t own = col[above][u];
                    found = own == row[u] || __builtin_amdgcn_update_dpp(kNoColumn, own, 0x101, 0xF, 0xF, false) == row[u];  // row_shl:1
                } else {
                    const int32_t* __restrict__ columns = lds.row_col[above] + 1;
                    found = columns[below(columns, row[u])] == row[u];
                }
                seen += __popc((uint32_t)slot_ballot(row[u] != kNoColumn && found));
            }
            if constexpr (LC == 16) return 2 * seen >= p[above + 2] - p[above + 1];
            return 4 * seen >= p[above + 2] - p[above + 1] && p[kQuad] - p[0] - (kQuad - 1) * seen <= kQuadRecords;
        };
        // columns without order, told by the second row and the first, or else (where a line of the grid ends between them) by
        // the fourth and the third: nothing is listed (without the second look: 75 x 75 x 30 points, N = 36 56.9 us, 49.1 with it,
        // 49.6 by row_split_kernel; 99 x 97 x 31, N = 56 88.9, 81.1 and 88.9)
        if constexpr (LC > 16) put_columns();
        bool some_shared = shares(0);
        if (__ballot(!some_shared) != 0) {
            const bool others = shares(2);
            some_shared = some_shared || others;
        }
        listed = __ballot(!some_shared) == 0;
        if (listed) {
            if constexpr (LC == 16) put_columns();
            uint32_t before[kQuad][EPL];  // byte j: of row j, the columns below this one
            uint32_t opens[kQuad];        // bit q: the row's entry q opens a record
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
                    before[i][u] = 0;
                    bool found = false;
#pragma unroll
                    for (int j = 0; j < kQuad; ++j) {
                        const int32_t* __restrict__ row = lds.row_col[j] + 1;
                        const int lower = j == i ? q : below(row, c);
                        before[i][u] |= (uint32_t)lower << (8 * j);
                        if (j == i - 1) found = have && row[lower] == c;
                    }
                    const uint32_t here = (uint32_t)slot_ballot(have && !found);
                    opens[i] |= here << (u * LC % kQuadRow);
                }
                records += __popc(opens[i]);
            }
            // (an empty place counts as a record of the quad's first column and of no row)
            int32_t some = kNoColumn;
#pragma unroll
            for (int i = kQuad - 1; i >= 0; --i) {
                const int32_t first = __shfl(col[i][0], 0, LC);
                some = first != kNoColumn ? first : some;
            }
            wave_lds_order();  // the rows' columns have been read
#pragma unroll
            for (int q = t; q < kQuadPlaces; q += LC) {
                *reinterpret_cast<float4*>(lds.rec.val[q]) = float4{0.0f, 0.0f, 0.0f, 0.0f};
                lds.rec.col[q] = some;
            }
            wave_lds_order();
#pragma unroll
            for (int i = 0; i < kQuad; ++i)
#pragma unroll
                for (int u = 0; u < EPL; ++u) {
                    int mine = 0;
#pragma unroll
                    for (int j = 0; j < kQuad; ++j) mine += __popc(__builtin_amdgcn_ubfe(opens[j], 0u, before[i][u] >> (8 * j) & 31u));
                    mine = col[i][u] != kNoColumn && mine < kQuadRecords ? mine : kQuadPlaces - 1;
                    lds.rec.col[mine] = col[i][u];
                    lds.rec.val[mine][i] = val[i][u];
                }
            // worth it from a quarter shared on
            listed = slot_ballot(descends) == 0 && records <= kQuadRecords && 4 * records <= 3 * (p[kQuad] - p[0]);
        }
        wave_lds_order();
        if (!listed) {
#pragma unroll
            for (int i = 0; i < kQuad; ++i)
#pragma unroll
                for (int u = 0; u < EPL; ++u)
                    if (t + u * LC < p[i + 1] - p[i]) lds.staged[p[i] - p[0] + t + u * LC] = StagedEntry{col[i][u], val[i][u]};
        }
    }
    const bool in_lds = !listed && p[kQuad] - p[0] <= kQuadChunk;  // the whole quad, one row after the other
    if (in_lds && !loaded) {
        StagedEntry e[EACH];
#pragma unroll
        for (int u = 0; u < EACH; ++u)
            if (t + u * LC < p[kQuad] - p[0]) {
                e[u].col = load_stream(a.colidx + p[0] + t + u * LC);
                e[u].val = load_stream(a.vals + p[0] + t + u * LC);
            }
#pragma unroll
        for (int u = 0; u < EACH; ++u)
            if (t + u * LC < p[kQuad] - p[0]) lds.staged[t + u * LC] = e[u];
    }

    // The workgroup's quads that go row by row, known before the gathers: where there are none nobody waits for anybody behind them
    // (27-point stencil of 1,000,000 rows, with the meeting behind the gathers and so: N = 128 425 -> 416 us, N = 256 868 -> 848).
    const int wave = threadIdx.x / kWave;
    {
        const unsigned long long open = __ballot(!listed), read = __ballot(!listed && !in_lds);
        if (threadIdx.x % kWave == 0) {
            s_open[wave] = open;
            s_read[wave] = read;
        }
        if (t <= kQuad) s_ptr[slot][t] = t == 0 ? p[0] : t == 1 ? p[1] : t == 2 ? p[2] : t == 3 ? p[3] : p[4];
    }
    __syncthreads();

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

    // Rows one by one, a row to a slot: those of quads that are open by all the workgroup's slots, whichever slot's they are, first those
    // whose entries are in LDS, then those that are read into it; in between, by its own slots, a wavefront's that were not finite.
    uint32_t here = 0, elsewhere = 0, again = 0;  // bit: slot
#pragma unroll
    for (int w = 0; w < kWavesPerBlock; ++w) {
        const unsigned long long all = s_open[w], read = s_read[w];
#pragma unroll
        for (int l = 0; l < kWave / LC; ++l) {
            here |= (uint32_t)((all & ~read) >> (l * LC) & 1) << (w * (kWave / LC) + l);
            elsewhere |= (uint32_t)(read >> (l * LC) & 1) << (w * (kWave / LC) + l);
        }
    }
    const unsigned long long redo = __ballot(listed && !done);
    if (redo == 0 && (here | elsewhere) == 0) return;
#pragma unroll
    for (int l = 0; l < kWave / LC; ++l) again |= (uint32_t)(redo >> (l * LC) & 1) << (wave * (kWave / LC) + l);
    // number n of the rows of the slots in mask
    auto row_number = [&](uint32_t mask, int n) {
        for (int i = 0; i < n / kQuad; ++i) mask &= mask - 1;
        return (__ffs(mask) - 1) * kQuad + n % kQuad;
    };
    auto store = [&](int row, const Vec<4>& sum) {
        const int64_t r = (int64_t)block * (SLOTS * kQuad) + row;
        if (k_ok && r < a.M) store_vec_stream<4>(a.C + r * a.N + k_lane, sum);
    };
    for (int n = slot; n < __popc(here) * kQuad; n += SLOTS) {
        const int row = row_number(here, n);
        const int32_t* __restrict__ ptr = s_ptr[row / kQuad];
        const uint32_t at = (uint32_t)(ptr[row % kQuad] - ptr[0]);
        Vec<4> acc;
        acc.zero();
        if (k_ok) gather_fma<4, 1, kPlainDepth>(acc, s_lds[row / kQuad].staged, at, (uint32_t)(ptr[row % kQuad + 1] - ptr[0]), B);
        store(row, acc);
    }
    if (here != 0) __syncthreads();  // the rows in LDS are done with
    for (int pass = 0; pass < 2; ++pass) {
        const uint32_t mask = pass == 0 ? again : elsewhere;
        const int first = pass == 0 ? slot % (kWave / LC) : slot, step = pass == 0 ? kWave / LC : SLOTS;
        const int rows = __popc(mask) * kQuad;
        if (rows == 0) continue;
        StagedEntry next[NEXT];  // of a row, the next ones on their way while these are gathered for
        int row = 0;
        int32_t base = 0, end = 0;
        auto fetch = [&] {
#pragma unroll
            for (int u = 0; u < NEXT; ++u)
                if (t + u * LC < CHUNK && base + t + u * LC < end) {
                    next[u].col = load_stream(a.colidx + base + t + u * LC);
                    next[u].val = load_stream(a.vals + base + t + u * LC);
                }
        };
        auto begin_row = [&](int n) {
            row = row_number(mask, n);
            base = s_ptr[row / kQuad][row % kQuad];
            end = s_ptr[row / kQuad][row % kQuad + 1];
        };
        Vec<4> acc;
        acc.zero();
        if (first < rows) {
            begin_row(first);
            fetch();
        }
        for (int n = first; n < rows;) {
            const int this_row = row;
            const int32_t cnt = end - base < CHUNK ? end - base : CHUNK;
            const bool last = end - base <= CHUNK;
            wave_lds_order();
#pragma unroll
            for (int u = 0; u < NEXT; ++u)
                if (t + u * LC < cnt) lds.staged[t + u * LC] = next[u];
            wave_lds_order();
            base += CHUNK;
            if (last) {
                n += step;
                if (n < rows) begin_row(n);
            }
            if (n < rows) fetch();
            if (k_ok) gather_fma<4, 1, kPlainDepth>(acc, lds.staged, 0, (uint32_t)cnt, B);
            if (last) {
                store(this_row, acc);
                acc.zero();
            }
        }
    }
}

// Rows of more than a dozen entries and of no more than kQuadRow in the mean, whose columns take 16 lanes or more, and enough blocks
// of them for the chip, since a quad's rows are one after the other where it is not listed.  us by row_split_kernel and so, of
// 27-point stencils, rows of 25 columns without order and the first mesh above: 27,000 rows, N = 128 17.0 / 13.7, 38.4 / 42.3 and
// 18.4 / 21.0; 54,000 rows 31.7 / 26.3, 88.0 / 88.8 and 35.3 / 40.2; 110,000 rows 59.6 / 46.1, 196 / 195 and 67.5 / 63.8; in 16 lanes,
// N = 64, 91,000 to 110,000 rows 30.0 / 31.0, 91.7 / 96.2 and 40.6 / 45.4; 140,000 rows 43.4 / 42.9, 121 / 123; 300,000 rows without order
// 182 / 184.  What still loses by more than that in 16 lanes are grid points with a random part of the 125 around each, which share a little more
// than half (268,800 rows, N = 40 81 / 85, N = 64 87 / 93; N = 128 152 / 126, and with a sixth of the rows of 32 entries or more
// 175 / 171 to 204, by where the operands lie).
// A column tile has to fit one pass of its lanes: the kernel makes no second one (row_split_kernel does).
bool row_quads_apply(int64_t M, int lc, int64_t tile_cols, double mean_row, int compute_units)
{
    if (tile_cols > (int64_t)lc * 4) return false;
    const int64_t blocks = M / ((int64_t)(kBlock / lc) * kQuad);
    return lc >= 16 && mean_row > 12.0 && mean_row <= (double)kQuadRow && blocks >= (int64_t)(lc >= 32 ? 5 : 8) * compute_units;
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
