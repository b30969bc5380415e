// Row-split schedule, serial strategy, short rows: teams of lanes go through consecutive rows each at its own pace
// (sgap_flat.hpp).  A workgroup owns a block of consecutive rows and takes them in pieces (one, as a rule); every row has one
// owner and one plain store.
//
// Bound by the gathers from beyond the L2s where B is large (2,000,000 rows of 1 to 16 entries, N = 32, a B of 8.4 MB: 1.6 GB
// at 7.5 TB/s), else by the address units.  us, a lane group per row that meets the others of its wavefront after each
// (row_split_kernel) / this: 2,000,000 rows of 1 to 15 entries, B of 65,536 rows, N = 32 228 / 200, N = 64 513 / 414; 250,000, N = 32
// 32.9 / 31.1, N = 48 62.5 / 58.4, B of 20,000 rows 29.6 / 24.7 and 50.8 / 35.6; 700,000 of 1 to 11, N = 32, in order of their
// lengths 83 / 64 (86 with a die's blocks in one run); 64,000, N = 16, four rows to a lane 17.4 / 8.3; 200,000 of 10 in the mean, N = 8, four
// rows to a lane 45.7 / 22.3.
#include "sgap_common.hpp"
#include "sgap_flat.hpp"
#include "sgap_nnz_common.hpp"

namespace sgap {

constexpr int kFrEntries = 2560;   // entries of a piece at most: four workgroups' LDS, as many as the registers leave
constexpr int kFrRows = 1024;      // rows of a piece at most
constexpr int kFrResident = 4;     // workgroups of a compute unit
constexpr int kFrMean = 1900;      // entries of a block in the mean at most
constexpr int kFrPieces = 8;      // runs of blocks of a die, where the columns are not cut into tiles
constexpr int kFrTile = 32;        // columns of a tile: a cache line of each row of B

template <int VEC, bool OFF32>
__global__ __launch_bounds__(kBlock) void flat_rows_kernel(SpmmArgs a, int lanes, int block_rows, int64_t blocks, FlatBlocks items,
                                                           int tile_cols)
{
    __shared__ FlatShared<kFrEntries, kFrRows> s;
    __shared__ Vec<VEC> s_part[kBlock];
    const int teams = kBlock / lanes;
    int64_t block = items.at(blockIdx.x);  // tile by tile
    if (block >= items.blocks) return;     // the whole workgroup
    const int64_t tile_first = block / blocks * tile_cols;  // (a tile has no more columns than the lanes hold)
    block %= blocks;
    const int64_t row_first = block * block_rows;
    const int64_t row_last = row_first + block_rows < a.M ? row_first + block_rows : a.M;

    struct Columns {
        bool ok;
        uint32_t first;  // of the VEC columns this lane holds
        __device__ __forceinline__ Columns(const FlatPlace& p, int64_t tile_first, int64_t N, int teams)
        {
            const uint32_t k = (uint32_t)tile_first + p.chunk * VEC;  // N < 2^31
            ok = k < (uint32_t)N && p.team < teams;
            first = ok ? lane_first_col<VEC>(k, (uint32_t)N) : 0;
        }
    };
    for (int64_t r0 = row_first; r0 < row_last;) {
        int n = row_last - r0 < kFrRows ? (int)(row_last - r0) : kFrRows;
        __syncthreads();  // the piece before is done with
        {
            const FlatPlace p(lanes);
            for (int i = p.tid; i <= n; i += kBlock) s.ptr[i] = a.rowptr[r0 + i];
        }
        __syncthreads();
        const int32_t e0 = __builtin_amdgcn_readfirstlane(s.ptr[0]);
        if (s.ptr[n] - e0 > kFrEntries) {
            const FlatPlace p(lanes);
            int fit = 0;
            for (int i = 0; i < n; i += kBlock) fit += __syncthreads_count(i + p.tid < n && s.ptr[i + p.tid + 1] - e0 <= kFrEntries);
            n = fit;
        }
        n = __builtin_amdgcn_readfirstlane(n);
        if (n == 0) {
            // a row of more entries than there is room for: all teams together
            const FlatPlace p(lanes);
            const Columns c(p, tile_first, a.N, teams);
            const MaskedRows<VEC, OFF32> B(a.B, a.N, c.first);
            const int32_t e1 = __builtin_amdgcn_readfirstlane(s.ptr[1]);
            Vec<VEC> t;
            t.zero();
            for (int32_t base = e0; base < e1; base += kFrEntries) {
                const int32_t cnt = e1 - base < kFrEntries ? e1 - base : kFrEntries;
                __syncthreads();
                flat_stage<kFrEntries>(s.entry, a.colidx, a.vals, base, cnt, p.tid);
                __syncthreads();
#pragma unroll 1
                for (int q = p.team; c.ok && q < cnt; q += teams) t.fma(s.entry[q].val, B.load(s.entry[q].col, true));
            }
            s_part[p.tid] = t;
            __syncthreads();
            if (p.team == 0 && c.ok) {
#pragma unroll 1
                for (int m = 1; m < teams; ++m) {
                    const Vec<VEC> other = s_part[m * lanes + p.chunk];
#pragma unroll
                    for (int i = 0; i < VEC; ++i) t.v[i] += other.v[i];
                }
                store_vec_stream<VEC>(a.C + r0 * a.N + c.first, t);
            }
            ++r0;
            continue;
        }
        const int32_t cnt = __builtin_amdgcn_readfirstlane(s.ptr[n]) - e0;
        {
            const FlatPlace p(lanes);
            flat_stage<kFrEntries>(s.entry, a.colidx, a.vals, e0, cnt, p.tid);
            flat_deal<false>(s, e0, cnt, n, teams, p.tid);
        }
        __syncthreads();
        {
            const FlatPlace p(lanes);
            const Columns c(p, tile_first, a.N, teams);
            float* const C = a.C + r0 * a.N + c.first;
            const uint32_t N = (uint32_t)a.N;
            auto store = [&](int row, const Vec<VEC>& sum) { store_vec_stream<VEC>(C + (uint64_t)(uint32_t)row * N, sum); };
            const int first = c.ok ? s.start[p.team] : 0, last = c.ok ? s.start[p.team + 1] : 0;
            if (first < last) {
                const MaskedRows<VEC, OFF32> B(a.B, a.N, c.first);
                const Vec<VEC> sum = flat_walk<VEC, OFF32, FlatChain<VEC>>(s, first, last, s.ptr[first] - e0, 0x7fffffff, e0, B, true,
                                                              [](int, bool, bool) {}, store);
                store(last - 1, sum);
            }
        }
        r0 += n;
    }
}

namespace {

// Column tiles: where B is larger than a die's L2 and a tile of it is not much larger, dies with a tile each gather more out of
// their L2s (items go tile by tile over the dies).  Not where rows of B begin amid cache lines.  us for the whole B / tiles of
// 32 columns, 2,000,000 rows of 1 to 16 entries, N = 64, B of 5 MB 292 / 324, 6.4 MB 324 / 324, 8.4 MB 391 / 337, 16.8 MB
// 545 / 441, 33.6 MB 632 / 610, 51 MB 663 / 671; 760,000 rows, N = 128, 10 MB 327 / 260, 33.6 MB 480 / 348; N = 96, 15 MB
// 295 / 200.
int64_t flat_tile(int64_t K, int64_t N)
{
    const bool tiles = N % kFrTile == 0 && N > kFrTile && K * N * 4 > (6 << 20) && K * kFrTile * 4 <= (14 << 20);
    return tiles ? kFrTile : N;
}

}  // namespace

// Where a lane group per row is the better one (us, that / this): few entries, one row to a lane (331,000 and 16 to a row, N = 64 12.5 / 15.5;
// 353,000, N = 20 7.5 / 7.4; 593,000 of 7 in the mean, N = 32 15.4 / 11.8); up to eleven columns, which leave a team a lane or few, one row to a
// lane and not many entries (672,000, N = 2 6.7 / 10.6; 1.3 M, 3 to a row, N = 6 12.1 / 17.0; 5.5 M, N = 1 28.6 / 21.7, 1.9 M, N = 8 16.0 / 14.1; two
// rows to a lane, 588,000, N = 4 7.5 / 8.3); wide rows of a B larger than an L2 that no tiles cut.  Rows that all fill a batch of eight and a
// little of the next are the shape that teams take longer for (1.3 M rows of 9, N = 28 137 / 154, 727,000, N = 64, four rows to a lane 105 / 116;
// 58,000, N = 24 8.3 / 9.2), and so are some matrices in order of their rows' lengths, of which blocks of equal numbers of rows have uneven shares
// (121,000 rows of 9 in the mean, N = 32 23.5 / 38.7; but 624,000 entries, 10 to a row, N = 6 8.2 / 6.4).  Where rows have mixed
// lengths the gain is larger, and the host cannot tell them apart (2.0 M entries, 10 to a row, N = 30 31.3 / 27.6; 665,000, N = 24 13.1 / 10.8; 521,000,
// 3 to a row, N = 64 28.2 / 17.9; 679,000, 8 to a row, N = 40 19.5 / 15.0).
bool flat_rows_apply(int64_t K, int64_t N, int group, double mean_row, int64_t nnz_hint)
{
    constexpr int64_t kFlatMinEntries = 500'000, kFlatFewColumns = 1'400'000;
    constexpr double kFlatMean = 12.0;
    if (nnz_hint < kFlatMinEntries || mean_row > kFlatMean || (group < 2 && N < 12 && nnz_hint < kFlatFewColumns)) return false;
    return N <= 48 || flat_tile(K, N) < N || (N <= 64 && K * N * 4 <= (6 << 20));
}

hipError_t launch_flat_rows(const SpmmArgs& a, int vec, int xcds, int compute_units, int64_t nnz_hint, hipStream_t s)
{
    const int64_t tile_cols = flat_tile(a.K, a.N);
    const int64_t chunks = (tile_cols + vec - 1) / vec, tiles = (a.N + tile_cols - 1) / tile_cols;
    if (chunks > kWave) return hipErrorInvalidValue;
    const int lanes = (int)chunks;
    // blocks of even numbers of rows, as many as make whole rounds of the resident workgroups
    const int64_t resident = (int64_t)kFrResident * compute_units;
    const int64_t rounds = nnz_hint / (resident * kFrMean) + 1;
    int64_t rows = (a.M + resident * rounds - 1) / (resident * rounds);
    if (rows > kFrRows) rows = kFrRows;
    const int64_t blocks = (a.M + rows - 1) / rows;
    const FlatBlocks items(blocks * tiles, xcds, tiles > 1 ? 1 : kFrPieces);
    if (items.grid() > 0x7ffffff0LL) return hipErrorInvalidValue;
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)items.grid()), dim3(kBlock), 0, s, a, lanes, (int)rows, blocks, items, (int)tile_cols);
    };
    const bool off32 = offsets_fit_32(a);
    if (vec == 4) { if (off32) go(flat_rows_kernel<4, true>); else go(flat_rows_kernel<4, false>); }
    else if (vec == 2) { if (off32) go(flat_rows_kernel<2, true>); else go(flat_rows_kernel<2, false>); }
    else { if (off32) go(flat_rows_kernel<1, true>); else go(flat_rows_kernel<1, false>); }
    return hipGetLastError();
}

}  // namespace sgap
