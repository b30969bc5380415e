// Row-split schedule, parallel strategy: a workgroup owns a block of consecutive rows, and teams of lanes share what it has
// evenly (sgap_flat.hpp): whole rows a team each, a row of more than kFlatCut entries by several, whose sums are added up in a
// fixed order.  One plain store per row, no atomics.  A row that goes on in the next piece of a block is carried over in LDS; rows that
// are too long for that (768 entries) are left to the workgroups in front of the grid that look for them (find_rows), and the other
// rows of the piece close up.  Where long rows lie together a block of equal numbers of rows has many times the others' entries:
// there the workgroups in front take rows of kFsHeavyRow entries and more too, and a die's blocks are spread over the matrix.
//
// Bound by the gathers from beyond the L2s where B is large, else by the chain of loads that a block is; power laws by their
// longest rows, which a workgroup takes 20 us for (4,096 entries, N = 37).  With a group of lanes per row (row_split_kernel)
// the groups of a wavefront meet at every row, and members without entries wait for those with most.  us, group per row
// / this: uniform, 60,000 rows of 16, N = 13, G = 16 18.3 / 11.4, N = 32 21.7 / 14.1, N = 48 27.9 / 25.8; 40,000 of 8, N = 32
// 15.4 / 8.9; 60,000 of 12, N = 64 29.7 / 24.8.  Power laws, mean 16: 50,000 rows, N = 24 30.3 / 27.8, N = 32 30.2 / 25.2, N = 37
// 37.0 / 35.1, N = 48 37.1 / 34.1; 120,000, N = 32 50.5 / 46.8; 200,000, N = 32 77 / 68.  50,000 rows in order of their lengths,
// N = 32 95 / 42 (254 with every row below 768 entries in its block); R-MAT, 65,536 rows, N = 16, G = 32 76 / 33 (164), N = 48 102 / 59
// (164), 131,072, N = 32 124 / 84 (181).
#include "sgap_common.hpp"
#include "sgap_flat.hpp"
#include "sgap_nnz_common.hpp"
#include "sgap_row_split_impl.hpp"

namespace sgap {

constexpr int kFsEntries = 2048;  // entries of a piece at most
constexpr int kFsRows = 1024;     // rows of a block at most
constexpr int kFsResident = 5;    // workgroups of a compute unit
constexpr int kFsMean = 1200;     // entries of a block in the mean at most (800 and 1,800: up to 6 % slower)
constexpr int kFsPieces = 8;      // runs of blocks of a die
constexpr int kFsDepth = 12;      // rows of B in flight of a row that a workgroup takes together
constexpr int kFsGroup = 8;       // plan_row_split_grid as for groups of so many: rows of 768 entries and more are looked for
constexpr int kFsHeavy = 3072;    // entries of a block from which on ...
constexpr int kFsHeavyRow = 96;   // ... rows of so many are looked for too

namespace {

struct FsShared {
    FlatShared<kFsEntries, kFsRows> flat;
    FlatHeads<4> heads;      // of rows
    Vec<4> carry[2][kWave];  // of the row that goes on in the next piece
    unsigned long long mask[kWavesPerBlock];
    unsigned long long left_out[kFsRows / kWave];  // rows of the piece that are a finder's
    int32_t scan[kWavesPerBlock], gaps;
};
static_assert(kFsEntries >= kStageCap && kFsRows >= kRowCap, "find_rows has the same places");

// Rows of so many entries and more are a finder's in a block of that many entries.
__device__ __forceinline__ int32_t flat_shared_left_out(int32_t share_from, int32_t block_entries)
{
    return block_entries > kFsHeavy && kFsHeavyRow < share_from ? kFsHeavyRow : share_from;
}

// The pointers of a piece's n rows as if those that are left out had no entries and the first row began at e0; from 0 on.
template <typename OUT>
__device__ __forceinline__ void close_up(FsShared& sh, int n, int32_t e0, OUT&& is_left_out)
{
    constexpr int EACH = kFsRows / kBlock;  // consecutive rows to a thread
    int32_t* const ptr = sh.flat.ptr;
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave, first = threadIdx.x * EACH;
    int32_t len[EACH], sum = 0;
#pragma unroll
    for (int j = 0; j < EACH; ++j) {
        const int i = first + j;
        const int32_t from = i == 0 || i >= n ? e0 : ptr[i];
        len[j] = i < n && !is_left_out(i) ? ptr[i + 1] - from : 0;
        sum += len[j];
    }
    int32_t before = sum;
    for (int d = 1; d < kWave; d *= 2) {
        const int32_t other = __shfl_up(before, d, kWave);
        if (lane >= d) before += other;
    }
    if (lane == kWave - 1) sh.scan[wave] = before;
    __syncthreads();  // everyone has read the pointers, too
    before -= sum;
    for (int w = 0; w < wave; ++w) before += sh.scan[w];
#pragma unroll
    for (int j = 0; j < EACH; ++j) {
        if (first + j <= n) ptr[first + j] = before;
        before += len[j];
        if (first + j == n - 1) ptr[n] = before;
    }
    __syncthreads();
}

}  // namespace

// N <= kWave * 4
template <bool OFF32>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(kFsResident)))
void flat_shared_rows_kernel(SpmmArgs a, int lanes, int block_rows, FlatBlocks blocks, RowSplitGrid plan)
{
    __shared__ FsShared sh;
    auto& s = sh.flat;
    if (__builtin_expect((int)blockIdx.x < plan.walk_from, 1)) {  // (said to come first: a register less is held meanwhile by the others)
        auto is_shared = [&](int64_t row, int32_t len) {
            if (len < kFsHeavyRow || len >= plan.share_from) return len >= plan.share_from;
            const int64_t first = (int64_t)((uint32_t)row / (uint32_t)block_rows) * block_rows;
            const int64_t last = a.M - first < block_rows ? a.M : first + block_rows;
            return len >= flat_shared_left_out(plan.share_from, a.rowptr[last] - a.rowptr[first]);
        };
        if ((int)blockIdx.x < plan.finders) find_rows<4, OFF32, kFsDepth, true>(a, plan, is_shared, s.entry, s.ptr, sh.mask, kBlock);
        return;
    }
    const int teams = kBlock / lanes;
    const int64_t block = blocks.at(blockIdx.x - plan.walk_from);
    if (block >= blocks.blocks) return;  // the whole workgroup
    const int32_t row_first = (int32_t)(block * block_rows);  // M < 2^31
    const int rows = (int32_t)a.M - row_first < block_rows ? (int32_t)a.M - row_first : block_rows;

    struct Columns {
        bool ok;
        uint32_t first;  // of the four columns this lane holds
        __device__ __forceinline__ Columns(const FlatPlace& p, uint32_t N, int teams)
        {
            const uint32_t k = p.chunk * 4;
            ok = k < N && p.team < teams;
            first = ok ? lane_first_col<4>(k, N) : 0;
        }
    };
    int32_t left_out_from = 0;
    bool comes_in = false;  // row r0 began in the piece before
    int32_t e0 = 0;         // where the piece begins (comes_in)
    for (int r0 = 0, turn = 0; r0 < rows; turn ^= 1) {
        int n = rows - r0 < kFsRows ? rows - r0 : kFsRows;
        __syncthreads();  // the piece before is done with
        {
            const FlatPlace p(lanes);
            for (int i = p.tid; i <= n; i += kBlock) s.ptr[i] = a.rowptr[row_first + r0 + i];
            if (p.tid == 0) sh.gaps = 0;
            __syncthreads();
            if (r0 == 0 && !comes_in) left_out_from = flat_shared_left_out(plan.share_from, __builtin_amdgcn_readfirstlane(s.ptr[n] - s.ptr[0]));  // the whole block
            for (int i = p.tid; i - p.tid < n; i += kBlock) {
                const bool out = i < n && s.ptr[i + 1] - s.ptr[i] >= left_out_from;
                const unsigned long long mask = __ballot(out);
                if (p.tid % kWave == 0) sh.left_out[i / kWave] = mask;
                if (out) sh.gaps = 1;
            }
        }
        __syncthreads();
        const bool gaps = __builtin_amdgcn_readfirstlane(sh.gaps) != 0;  // rows of the piece are a finder's: the others close up in LDS
        if (!comes_in) e0 = __builtin_amdgcn_readfirstlane(s.ptr[0]);
        auto is_left_out = [&](int row) { return (sh.left_out[row / kWave] >> (row % kWave) & 1) != 0; };
        const int32_t came_from = e0;
        if (gaps) {
            close_up(sh, n, e0, is_left_out);
            e0 = 0;
        }
        bool cut = false;  // the last row goes on in the next piece
        int32_t end = __builtin_amdgcn_readfirstlane(s.ptr[n]);
        if (end - e0 > kFsEntries) {
            const FlatPlace p(lanes);
            int fit = 0;
            for (int i = 0; i < n; i += kBlock) fit += __syncthreads_count(i + p.tid < n && s.ptr[i + p.tid] - e0 < kFsEntries);
            n = __builtin_amdgcn_readfirstlane(fit);
            end = __builtin_amdgcn_readfirstlane(s.ptr[n]);
            cut = end - e0 > kFsEntries;
            if (cut) end = e0 + kFsEntries;
        }
        if ((comes_in && !gaps) || cut) {
            __syncthreads();
            if (threadIdx.x == 0) {
                if (comes_in) s.ptr[0] = e0;
                if (cut) s.ptr[n] = end;
            }
            __syncthreads();
        }
        const int32_t cnt = end - e0;
        {
            const FlatPlace p(lanes);
            if (!gaps) {
                flat_stage<kFsEntries>(s.entry, a.colidx, a.vals, e0, cnt, p.tid);
            } else {
                // entry by entry from where its row is
                constexpr int U = 4;
#pragma unroll 1
                for (int q0 = p.tid; q0 < cnt; q0 += U * kBlock) {
                    int32_t at[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int q = q0 + u * kBlock;
                        const int row = last_row_at_or_before(s.ptr, 0, n - 1, q < cnt ? q : cnt - 1);
                        at[u] = (row == 0 && comes_in ? came_from : a.rowptr[row_first + r0 + row]) + q - s.ptr[row];
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u)
                        if (q0 + u * kBlock < cnt) s.entry[q0 + u * kBlock] = {load_stream(a.colidx + at[u]), load_stream(a.vals + at[u])};
                }
            }
            flat_deal<true>(s, e0, cnt, n, teams, p.tid);
        }
        __syncthreads();

        const FlatPlace p(lanes);
        const Columns c(p, (uint32_t)a.N, teams);
        float* const C = a.C + (int64_t)(row_first + r0) * a.N + c.first;
        auto store = [&](uint32_t row, const Vec<4>& sum) {
            if (c.ok) store_vec_stream<4>(C + (uint64_t)row * (uint32_t)a.N, sum);
        };
        Vec<4> sum;         // of the last row that this team has entries of
        int open_row = -1;  // that row, where it begins among them and goes on behind them
        if (p.team < teams) {
            const uint32_t from = s.start[p.team], to = s.start[p.team + 1];
            const int first = from & 0xffff, finished = to & 0xffff;  // rows before `finished` end here
            const bool goes_on = (int)(to >> 16) > s.ptr[finished] - e0;
            const int last = finished + (goes_on ? 1 : 0);
            bool ended = false;
            if (first < last) {
                const MaskedRows<4, OFF32> B(a.B, a.N, c.first);
                bool whole = (int)(from >> 16) == s.ptr[first] - e0 && !(first == 0 && comes_in);
                const int ends = cut && finished == n ? n - 1 : finished;
                auto done = [&](int row, const Vec<4>& of_row) {
                    const bool is_end = row < ends;
                    if (whole && is_end) {
                        if (!gaps || !is_left_out(row)) store((uint32_t)row, of_row);
                    } else if (whole) {
                        open_row = row;
                    } else {
                        sh.heads.head[p.tid] = of_row;
                        ended = is_end;
                    }
                    whole = true;
                };
                sum = flat_walk<4, OFF32, FlatChains<4>>(s, first, last, from >> 16, to >> 16, e0, B, true, [](int, bool, bool) {}, done);
                done(last - 1, sum);
            } else {
                float none = 0.0f;
                asm volatile("" : "+v"(none));  // (four zeros would be held, or kept in memory, from the kernel's beginning on)
                sh.heads.head[p.tid] = {{none, none, none, none}};
            }
            sh.heads.ended[p.team] = ended ? 1 : 0;
        }
        if (__syncthreads_or(open_row >= 0 || comes_in)) {
            batch_heads(sh.heads, teams, lanes, p);
            __syncthreads();
            // what goes on is added up by the team that has its beginning, what came in from the piece before by the first team
#pragma unroll 1
            for (int round = 0; round < 2; ++round) {
                if (round == 1) {
                    if (!comes_in || p.team != 0) continue;
                    sum = sh.carry[turn][p.chunk];
                    open_row = 0;
                }
                if (open_row < 0) continue;
                if (add_heads_in_chains<4, true>(sum, sh.heads, round == 1 ? 0 : p.team + 1, teams, lanes, p.chunk)) store((uint32_t)open_row, sum);
                else sh.carry[turn ^ 1][p.chunk] = sum;
            }
        }
        if (gaps && cut) {  // where the last row goes on: what it has here behind where it was
            const int32_t begin = n == 1 && comes_in ? came_from : a.rowptr[row_first + r0 + n - 1];
            end += __builtin_amdgcn_readfirstlane(begin - s.ptr[n - 1]);
        }
        r0 += n - (cut ? 1 : 0);
        e0 = end;
        comes_in = cut;
    }
}

// Where groups of lanes are the better ones (us, group per row / this): few entries (ragged rows, 346,000 entries, 24 to a row, N = 37
// 9.0 / 11.4; power laws, 159,000, N = 17 11.4 / 18.5, 590,000, N = 27 17.6 / 20.1, but 849,000, N = 31 37.6 / 34.5, 2.9 M, N = 23 60 / 47, N = 17
// 73 / 59), fewer where rows are short, which leave most members idle (302,000 entries, 4 to a row, N = 60 26 / 21; 458,000, 12 to a row, N = 41
// 13.9 / 10.9; groups of four have fewer idle ones: 604,000, 15 to a row, N = 31 13.8 / 15.3, 907,000, 13 to a row, N = 25 17.9 / 15.5); few columns
// (50,000 rows, N = 8 17.5 / 24.3; 46,000, N = 13, G = 8 17.5 / 21.8; groups of 16: 2.1 M entries, N = 14 42.2 / 39.2); long rows (650,000 entries,
// 37 to a row, N = 31 17.3 / 20.6, 1.8 M, 39 to a row, N = 55 58.0 / 59.7; 3.3 M, 34 to a row, N = 25, G = 4 36.9 / 36.8); wide rows of a B from
// beyond the L2s (500,000 rows of 16, N = 64 292 / 309).
bool flat_shared_rows_apply(int64_t K, int64_t N, int members, double mean_row, int64_t nnz_hint)
{
    constexpr double kRowMean = 35.0, kShortRowMean = 12.0;
    if (N < 12 || N > 64 || mean_row > kRowMean || (N < 17 && members < 16) || (N > 40 && K * N * 4 > (32 << 20))) return false;
    if (mean_row <= kShortRowMean && N >= 20 && (N > 32 || members >= 8) && nnz_hint >= 300'000) return true;
    return nnz_hint >= (N < 24 ? 700'000 : 600'000);
}

hipError_t launch_flat_shared_rows(const SpmmArgs& a, int xcds, int compute_units, int64_t nnz_hint, hipStream_t s)
{
    if (a.N > kWave * 4 || nnz_hint < 1) return hipErrorInvalidValue;
    const int lanes = (int)((a.N + 3) / 4);
    // Blocks of even numbers of rows, as many as make whole rounds of the resident workgroups, but not of fewer entries than
    // about 800, with more than 8 lanes to a team 512 (power law, 50,000 rows, N = 32: 625 entries 25.6 us, 800 22.5; N = 37: 625
    // 34.7, 800 35.5).
    const int64_t resident = (int64_t)kFsResident * compute_units;
    const int64_t rounds = nnz_hint / (resident * kFsMean) + 1;
    int64_t rows = (a.M + resident * rounds - 1) / (resident * rounds);
    const int64_t least = (int64_t)((lanes <= 8 ? 800.0 : 512.0) * (double)a.M / (double)nnz_hint);
    if (rows < least) rows = least;
    if (rows > kFsRows) rows = kFsRows;
    const FlatBlocks blocks((a.M + rows - 1) / rows, xcds, kFsPieces);
    const RowSplitGrid plan = plan_row_split_grid(kFsGroup, 1, a.M, blocks.grid(), xcds, compute_units, nnz_hint, 0);
    if (plan.finders == 0) return hipErrorInvalidValue;  // (rows are left out for them)
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(plan.grid), dim3(kBlock), 0, s, a, lanes, (int)rows, blocks, plan);
    };
    if (offsets_fit_32(a)) go(flat_shared_rows_kernel<true>); else go(flat_shared_rows_kernel<false>);
    return hipGetLastError();
}

}  // namespace sgap
