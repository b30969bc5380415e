// Nnz-balanced schedule, serial strategy, 16 to 128 columns: {<g nnz, c col>, 1} (Section 6.1) with a tile's entries dealt out to
// teams of lanes that go through them each at its own pace (sgap_flat.hpp), whatever group_size says.
//
// A tile of stored entries comes into LDS with its rows that have entries.  A team takes consecutive entries, eight of one
// row at a time, or the last four of one and the first four of the next; a row that begins and ends among them is stored
// plainly.  What a team has of a row that began in front of it goes to LDS, where the team that has the row's beginning adds it
// up in order; the two rows that cross a tile's ends are added into C with atomics (the merge rule of sgap_nnz_common.hpp with the
// tile as its block).  No LDS atomics, no slots.
// The teams' shares are even in the turns that they take rather than in entries: a row counts kRowCost entries beside its own,
// since its last turn is seldom full (R-MAT, 2^19 rows, N = 32: 158 us with shares of entries, 115 so).
//
// With fixed shares, batches of eight whatever the rows' ends, and a flush wherever one fell (nnz_serial_kernel, which serves
// other widths), each entry cost a look at its row's end and row sums met in LDS slots by compare-and-swap.  Large R-MAT
// matrices are bound by their 128-byte reads either way (2^21 rows, 50 M entries, N = 32: 4.4 GB at 6.1 TB/s).  us, before / now:
//   power law, 65,536 rows, N = 64, G = 16 52.2 / 43.9; the same with N = 32 45.9 / 23.7; 300,000 rows, N = 64 197 / 192;
//   8,000 rows, N = 20 14.2 / 13.1; uniform, 60,000 rows of 32, N = 64, G = 8 101 / 65; R-MAT, G = 16, 2^19 rows, 8 M edges, N = 32
//   156 / 112, N = 16 124 / 95; 2^17 rows, 1.9 M edges, N = 128 137 / 108; 2^21 rows, 50 M entries, N = 32, G = 32 747 / 717
#include "sgap_common.hpp"
#include "sgap_flat.hpp"
#include "sgap_nnz_common.hpp"

namespace sgap {

namespace {

constexpr int kRowCost = kFlatRunCost;  // (with 3, 9 and 13 up to 4 % slower)
constexpr int kNfTile = 1024;  // entries of a tile at most
constexpr int kNfResident = 5;  // workgroups of a compute unit
static_assert(kNfTile <= kWindowCap, "a row of the window for every entry of a tile");

struct NnzFlatShared {
    __attribute__((aligned(16))) StagedEntry entry[kNfTile + kFlatBatch];  // (a batch reads past the last one)
    int32_t win[kWindowCap + 1];  // first positions of the tile's rows with entries
    int32_t row[kWindowCap];      // ... and their numbers
    FlatHeads<4> heads;
    float edge[2][4 * kWave];  // of the rows that cross the tile's ends: the one that comes in, the one that goes on
    int32_t edge_row[2];     // -1: none
    int32_t begin[kBlock + 1], begin_row[kBlock + 1];  // a team's first entry, and the window's row that holds it
    int32_t scan[kWavesPerBlock];
    int32_t tile_row[kTileRowBatch];
};

}  // namespace

template <bool OFF32>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(kNfResident)))
void nnz_flat_kernel(SpmmArgs a, int lanes, int teams, int tile)
{
    __shared__ NnzFlatShared s;
    const int32_t M = (int32_t)a.M;
    const int32_t nnz = a.rowptr[a.M];
    const TileDeal deal(((int64_t)nnz + tile - 1) / tile, blockIdx.x, gridDim.x);
    if (deal.mine == 0) return;
    TileWalk at(deal);
    if (threadIdx.x < 2) s.edge_row[threadIdx.x] = -1;

    const uint32_t N = (uint32_t)a.N;  // at most a wavefront's columns

    const int mine = (int)deal.mine;
    for (int j0 = 0; j0 < mine; j0 += kTileRowBatch) {
        find_tile_rows(a, deal, j0, tile, s.tile_row);
        const int j1 = j0 + kTileRowBatch < mine ? j0 + kTileRowBatch : mine;
        for (int j = j0; j < j1; ++j) {
            const int32_t tile_start = (int32_t)(at.tile() * tile);
            at.next();
            const int32_t cnt = nnz - tile_start < tile ? nnz - tile_start : tile;
            const int32_t row_lb = s.tile_row[j - j0];
            {
                const FlatPlace p(lanes);
                constexpr int WPT = kWindowCap / kBlock + 1;
                int32_t win[WPT];
#pragma unroll
                for (int i = 0; i < WPT; ++i) {
                    const int w = p.tid + i * kBlock;
                    const int64_t r = (int64_t)row_lb + w;
                    win[i] = w <= kWindowCap ? a.rowptr[r <= M ? r : M] : 0;
                }
                flat_stage<kNfTile>(s.entry, a.colidx, a.vals, tile_start, cnt, p.tid);
#pragma unroll
                for (int i = 0; i < WPT; ++i)
                    if (p.tid + i * kBlock <= kWindowCap) s.win[p.tid + i * kBlock] = win[i];
            }
            __syncthreads();
            int32_t n;
            if (s.win[kWindowCap] >= tile_start + cnt) {
                n = compact_window(s.win, s.row, row_lb, tile_start + cnt, s.scan);
            } else {
                __syncthreads();  // everyone has read the plain window
                n = load_compact_window(a, row_lb, tile_start + cnt, s.win, s.row, s.scan);
            }
            n = __builtin_amdgcn_readfirstlane(n);
            // Where the teams begin: even shares of the turns that a team will take.  A row counts as kRowCost entries beside its own.
            {
                const FlatPlace p(lanes);
                if (p.tid <= teams) {
                    const int32_t x = (int32_t)((float)((cnt + kRowCost * n) * p.tid) * __builtin_amdgcn_rcpf((float)teams));
                    int32_t lo = 0, hi = n - 1;
                    auto first_of = [&](int32_t i) {
                        const int32_t at = s.win[i] - tile_start;
                        return at > 0 ? at : 0;
                    };
                    while (lo < hi) {
                        const int32_t mid = (lo + hi + 1) / 2;
                        if (first_of(mid) + kRowCost * mid <= x) lo = mid; else hi = mid - 1;
                    }
                    const int32_t first = first_of(lo), last = s.win[lo + 1] - tile_start < cnt ? s.win[lo + 1] - tile_start : cnt;
                    int32_t q = x - kRowCost * (lo + 1);
                    q = p.tid == 0 ? 0 : p.tid == teams ? cnt : q < first ? first : q;
                    if (q >= last) {
                        q = last;
                        ++lo;
                    }
                    s.begin[p.tid] = q;
                    s.begin_row[p.tid] = lo;
                }
            }
            __syncthreads();

            {
                const FlatPlace p(lanes);
                const uint32_t k = p.chunk * 4, first_col = lane_first_col<4>(k, N);
                int32_t q = p.team < teams ? s.begin[p.team] : 0;
                const int32_t end = p.team < teams ? s.begin[p.team + 1] : 0;  // of this team's entries
                auto store = [&](int32_t row, const Vec<4>& sum) {
                    store_vec_stream<4>(a.C + ((uint64_t)(uint32_t)row * N + first_col), sum);
                };
                Vec<4> sum;
                sum.zero();
                int wi = 0;
                bool goes_on = false, head_ends = false;
                if (q < end) {
                    const MaskedRows<4, OFF32> B(a.B, a.N, first_col);
                    wi = s.begin_row[p.team];
                    bool whole = s.win[wi] - tile_start == q;  // the row begins with this team's entries
                    int32_t row_end = s.win[wi + 1] - tile_start;
                    auto end_of = [&](int row) { return s.win[row + 1 <= n ? row + 1 : n] - tile_start; };
#pragma unroll 1
                    do {
                        constexpr int D = kFlatBatch, H = D / 2;
                        StagedEntry e[D];
                        Vec<4> b[D];
                        const int32_t stop = row_end < end ? row_end : end;
                        const int32_t left = stop - q;
                        const bool ends = left <= D, row_done = ends && row_end <= end;
                        // Half a batch is enough for the row's last entries: the other half is the next row's.  (Rows of one to four entries
                        // are a turn for two of them: power law of 40,000 rows, longest first, N = 64 40.2 us with a turn each, 33.2 so; 65,536 in
                        // no order 43.8 / 44.8; 500,000 of 1 to 9 101.8 / 94.7; R-MAT, 2^15 rows 23 / 21.5.)
                        const bool two = left <= H && row_end < end;
                        const int32_t next_end = end_of(wi + 1), after_end = end_of(wi + 2);
                        const int32_t at = two ? row_end : q + H;
                        const int32_t left_there = (two ? (next_end < end ? next_end : end) : stop) - at;
#pragma unroll
                        for (int u = 0; u < H; ++u) {
                            e[u] = s.entry[q + u];
                            e[H + u] = s.entry[at + u];
                        }
#pragma unroll
                        for (int u = 0; u < H; ++u) {
                            b[u] = B.load(e[u].col, u < left);
                            if (u >= left) e[u].val = 0.0f;
                        }
#pragma unroll
                        for (int u = 0; u < H; ++u) {
                            b[H + u] = B.load(e[H + u].col, u < left_there);
                            if (u >= left_there) e[H + u].val = 0.0f;
                        }
                        const int now = wi;
                        const bool both_done = two && left_there <= H && next_end <= end;  // the next row too
                        q = two ? at + (left_there < H ? left_there : H) : ends ? stop : q + D;
                        if (row_done) {
                            wi += both_done ? 2 : 1;
                            row_end = both_done ? after_end : next_end;
                        }
                        const Vec<4> low = flat_dot_half<4>(e, b);
                        Vec<4> high = flat_dot_half<4>(e + H, b + H);
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            sum.v[i] += low.v[i] + (two ? 0.0f : high.v[i]);
                            high.v[i] = two ? high.v[i] : 0.0f;
                        }
                        if (row_done) {
                            if (whole) {
                                store(s.row[now], sum);
                            } else {
                                s.heads.head[p.tid] = sum;
                                head_ends = true;
                            }
                            sum = high;
                            whole = true;
                            if (both_done) {
                                store(s.row[now + 1], sum);
                                sum.zero();
                            }
                        }
                        if (q >= end && !(two ? both_done : row_done)) {
                            if (whole) goes_on = true;
                            else s.heads.head[p.tid] = sum;
                        }
                    } while (q < end);
                } else {
                    s.heads.head[p.tid] = sum;
                }
                if (p.team < teams && p.chunk == 0) s.heads.ended[p.team] = head_ends ? 1 : 0;
                if (p.tid < 2) s.edge_row[p.tid] = -1;
                __syncthreads();
                // a row that goes on is added up, in order, by the team that has its beginning; what came in from the tile in
                // front by the first team
#pragma unroll 1
                for (int round = 0; round < 2; ++round) {
                    if (round == 1) {
                        goes_on = p.team == 0 && s.win[0] < tile_start;
                        sum.zero();
                        wi = 0;
                    }
                    if (!goes_on) continue;
                    const bool ended = add_heads<4, false>(sum, s.heads, round == 1 ? 0 : p.team + 1, teams, lanes, p.chunk);
                    if (round == 0 && ended) {
                        store(s.row[wi], sum);
                    } else {
                        if (p.chunk == 0) s.edge_row[1 - round] = s.row[wi];
                        from_last_columns<4>(sum, (int)(k - first_col));
#pragma unroll
                        for (int i = 0; i < 4; ++i) s.edge[1 - round][p.chunk * 4 + i] = sum.v[i];
                    }
                }
                __syncthreads();
                // (an atomic instruction over consecutive words costs a quarter of one whose lanes are 16 bytes apart)
                for (uint32_t i = p.tid; i < 2 * N; i += kBlock) {
                    const uint32_t which = i >= N ? 1 : 0, col = i - which * N;
                    const int32_t row = s.edge_row[which];
                    if (row >= 0) unsafeAtomicAdd(a.C + ((uint64_t)(uint32_t)row * N + col), s.edge[which][col]);
                }
            }
            // (the next tile's entries and window are put down behind what the walk and the sums have read; the edges' places are
            // written again two barriers from here)
        }
    }
}

// The tile for a matrix, 0 where this is not the kernel (us, by shares of entries / here).  Fewer columns leave a team with a lane or
// two (65,536 rows of a power law, N = 8: 19.9 / 24.0; 8,000, N = 16 11.9 / 13.9, N = 17 14.3 / 13.2; 16,000, N = 16 13.7 / 14.9, 38,000 23.1 / 18.9; uniform rows gain there too, 18,000, N = 16 15.1 / 11.0), with more a tile has too few teams
// (100,000 rows, N = 200 220 / 219; R-MAT, 2^17 rows, N = 256 276 / 282).  Where rows are long and the caller asks for shares of 64
// entries nothing is left for this kernel to gain (5,000 rows of 4,000, N = 16 179 / 199; 10,000 of 200, N = 64 63.8 / 65.8; shares of 16,
// 40,000 of 300, N = 16 145 / 122).
// A team has some 16 to 32 entries of a tile; 33 to 64 columns take the larger tile where all of them fit the chip at once
// (power law, 65,536 rows, N = 64: 43.4 us with 1,030 tiles of 1,024 entries, 45.7 with 512; 300,000 rows 200 and 192).  A small matrix
// has smaller tiles (10,000 rows, N = 44 16.6 us with 512 entries and 17.3 with 1,024).
// Power laws whose rows come in order of their lengths, the longest first, end in tiles of a row to an entry: 40,000 rows, G = 16, N = 32 31.3 /
// 21.1, N = 64 34.1 / 33.2, N = 128 55 / 58; 150,000, N = 32 61 / 60, N = 48 93 / 103, N = 64 98 / 107, N = 128 188 / 189.
int nnz_flat_tile(int64_t N, int group, double mean_row, int64_t nnz_hint, int compute_units)
{
    if (N < 16 || N > 128 || (N <= 64 && group > 32 && mean_row >= 200.0)) return 0;
    int tile = N <= 32 ? kNfTile : N <= 64 ? kNfTile / 2 : kNfTile / 4;
    if (nnz_hint < 0) return tile;
    if (N < 17 && nnz_hint < 250'000) return 0;
    if (N > 32 && N <= 64 && nnz_hint > kNfTile * 3 * (int64_t)compute_units && nnz_hint <= kNfTile * kNfResident * (int64_t)compute_units)
        tile = kNfTile;
    const int least = N <= 32 ? kNfTile / 2 : kNfTile / 4;
    while (tile > least && 2 * (nnz_hint / tile) < 5 * (int64_t)compute_units) tile /= 2;
    return tile;
}

hipError_t launch_nnz_flat(const SpmmArgs& a, int tile, int compute_units, int64_t nnz_hint, hipStream_t s)
{
    const int lanes = (int)((a.N + 3) / 4);
    auto go = [&](auto kernel, int& per_cu) {
        if (per_cu == 0) per_cu = resident_per_cu(kernel, 0);
        hipLaunchKernelGGL(kernel, dim3(persistent_grid(per_cu, compute_units, nnz_hint, tile)), dim3(kBlock), 0, s, a, lanes, kBlock / lanes, tile);
    };
    static int per_cu[2];  // resident workgroups of a compute unit, 0 = not asked yet
    if (offsets_fit_32(a)) go(nnz_flat_kernel<true>, per_cu[0]);
    else go(nnz_flat_kernel<false>, per_cu[1]);
    return hipGetLastError();
}

}  // namespace sgap
