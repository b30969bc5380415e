// Row-split schedule, parallel strategy: a workgroup owns a block of consecutive rows, and teams of lanes share what it has
// evenly (sgap_flat.hpp): whole rows a team each, a row of more than kFlatCut entries by several, whose sums are added up in
// order.  One plain store per row, no atomics.  A row that goes on in the next piece of a block is carried over in LDS; rows
// that are too long for that (768 entries) are left to the workgroups in front of the grid that look for them (find_rows), and
// a piece goes on behind such a row.
//
// Bound by the gathers from beyond the L2s where B is large, else by the chain of loads that a block is; power laws by their
// longest rows, which a workgroup takes 20 us for (4,096 entries, N = 37).  With a group of lanes per row (row_split_kernel)
// the groups of a wavefront meet at every row, and members without entries wait for those with most.  us, group per row
// / this: uniform, 60,000 rows of 16, N = 16 19.2 / 10.3; 50,000 of 16, N = 32 19.9 / 12.3, N = 37 24.3 / 20.3; 60,000 of 8,
// N = 32 20.7 / 10.6; of 12, N = 64 30.9 / 25.8; 500,000 of 16, N = 32, a B of 6.4 MB 131 / 75.  Power laws, mean 16, three
// matrices each, in the mean: 50,000 rows, N = 16 22.6 / 20.9, N = 32 30.8 / 22.5; 120,000, N = 32 51 / 37, N = 64 71 / 65.
#include "sgap_common.hpp"
#include "sgap_flat.hpp"
#include "sgap_row_split_impl.hpp"

namespace sgap {

constexpr int kFsEntries = 2048;  // entries of a piece at most
constexpr int kFsRows = 1024;     // rows of a block at most
constexpr int kFsResident = 5;    // workgroups of a compute unit
constexpr int kFsMean = 1200;     // entries of a block in the mean at most (800 and 1,800: up to 6 % slower)
constexpr int kFsDepth = 12;      // rows of B in flight of a row that a workgroup takes together
constexpr int kFsGroup = 8;       // plan_row_split_grid as for groups of so many: rows of 768 entries and more are looked for

namespace {

struct FsShared {
    FlatShared<kFsEntries, kFsRows> flat;
    FlatHeads<4> heads;      // of rows
    Vec<4> carry[2][kWave];  // of the row that goes on in the next piece
    unsigned long long mask[kWavesPerBlock];
    int first_long, next_long;
};
static_assert(kFsEntries >= kStageCap && kFsRows >= kRowCap, "find_rows has the same places");

}  // namespace

// N <= kWave * 4
template <bool OFF32>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(kFsResident)))
void flat_shared_rows_kernel(SpmmArgs a, int lanes, int block_rows, int64_t blocks, int64_t blocks_per_xcd, int xcds, RowSplitGrid plan)
{
    __shared__ FsShared sh;
    auto& s = sh.flat;
    if (__builtin_expect((int)blockIdx.x < plan.walk_from, 1)) {  // (said to come first: a register less is held meanwhile by the others)
        auto is_shared = [&](int64_t, int32_t len) { return len >= plan.share_from; };
        if ((int)blockIdx.x < plan.finders) find_rows<4, OFF32, kFsDepth, true>(a, plan, is_shared, s.entry, s.ptr, sh.mask, kBlock);
        return;
    }
    const uint32_t wg = blockIdx.x - plan.walk_from;
    const int teams = kBlock / lanes;
    // workgroup b runs on die b % xcds: every die gets one contiguous run of blocks
    const int64_t block = (int64_t)(wg % xcds) * blocks_per_xcd + wg / xcds;
    if (block >= blocks) return;  // the whole workgroup
    const int64_t row_first = block * block_rows;
    const int rows = (int)(a.M - row_first < block_rows ? a.M - row_first : block_rows);

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
    bool comes_in = false;  // row r0 began in the piece before
    int32_t e0 = 0;         // where the piece begins (comes_in)
    for (int r0 = 0, turn = 0; r0 < rows; turn ^= 1) {
        int n = rows - r0 < kFsRows ? rows - r0 : kFsRows;
        __syncthreads();  // the piece before is done with
        {
            const FlatPlace p(lanes);
            for (int i = p.tid; i <= n; i += kBlock) s.ptr[i] = a.rowptr[row_first + r0 + i];
            if (p.tid == 0) sh.first_long = n;
        }
        __syncthreads();
        {
            const FlatPlace p(lanes);
            for (int i = p.tid; i < n; i += kBlock)
                if (s.ptr[i + 1] - s.ptr[i] >= plan.share_from) atomicMin(&sh.first_long, i);
        }
        __syncthreads();
        int hole_row = __builtin_amdgcn_readfirstlane(sh.first_long);  // a finder's; the piece ends in front of another one
        int32_t hole = 0, hole_at = 0;                                 // its entries, and where they were
        if (hole_row < n) {
            hole_at = __builtin_amdgcn_readfirstlane(s.ptr[hole_row]);
            hole = __builtin_amdgcn_readfirstlane(s.ptr[hole_row + 1]) - hole_at;
            if (threadIdx.x == 0) sh.next_long = n;
            __syncthreads();
            const FlatPlace p(lanes);
            for (int i = p.tid; i < n; i += kBlock)
                if (i > hole_row && s.ptr[i + 1] - s.ptr[i] >= plan.share_from) atomicMin(&sh.next_long, i);
            __syncthreads();
            n = __builtin_amdgcn_readfirstlane(sh.next_long);
            for (int i = p.tid; i <= n; i += kBlock)
                if (i > hole_row) s.ptr[i] -= hole;
            __syncthreads();
        }
        if (!comes_in) e0 = __builtin_amdgcn_readfirstlane(s.ptr[0]);
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
        if (comes_in || cut) {
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
            const int32_t front = hole > 0 && hole_at < end ? hole_at - e0 : cnt;
            flat_stage<kFsEntries>(s.entry, a.colidx, a.vals, e0, front, p.tid);
            if (front < cnt) flat_stage<kFsEntries>(s.entry + front, a.colidx, a.vals, e0 + front + hole, cnt - front, p.tid);
            flat_deal<true>(s, e0, cnt, n, teams, p.tid);
        }
        __syncthreads();

        const FlatPlace p(lanes);
        const Columns c(p, (uint32_t)a.N, teams);
        float* const C = a.C + (row_first + r0) * a.N + c.first;
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
                        if (row != hole_row) store((uint32_t)row, of_row);
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
        r0 += n - (cut ? 1 : 0);
        e0 = end + (hole_at < end ? hole : 0);
        comes_in = cut;
    }
}

// Where groups of lanes are the better ones: few entries (us, group per row / this: power laws of 10,000 rows, N = 16 8.8 /
// 11.2, N = 24 11.3 / 12 to 18; 25,000 rows, N = 16 14.0 / 17.3, N = 48 24.7 / 24.7; uniform, 5,000 rows of 16, N = 32 5.3 / 6.1,
// 20,000 9.0 / 7.2), few columns (50,000 rows, N = 8 17.5 / 24.3, N = 4 16.2 / 32), and where wide rows come from beyond
// the L2s (500,000 rows of 16, N = 64 292 / 309; 200,000, N = 41, a B of 33 MB 129 / 128).  Long rows leave no members idle
// (200,000 rows of 64, N = 32 118 / 107; 20,000 of 400 66 / 75).
// Groups of 8 and fewer have few idle members, and up to 16 columns that is enough (power law of 46,000 rows, N = 13, G = 8 17.5 /
// 21.8, of 16 23 / 23; 130,000 32.6 / 36.6 and 53 / 50).
bool flat_shared_rows_apply(int64_t K, int64_t N, int members, double mean_row, int64_t nnz_hint)
{
    constexpr double kFsLongMean = 128.0;
    if (N < 12 || N > 64 || mean_row > kFsLongMean || (N > 40 && K * N * 4 > (32 << 20))) return false;
    if (N <= 16 && members <= 8) return false;
    return nnz_hint >= (N < 24 ? 700'000 : 300'000);
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
    const int64_t blocks = (a.M + rows - 1) / rows;
    const int64_t blocks_per_xcd = (blocks + xcds - 1) / xcds;
    const RowSplitGrid plan = plan_row_split_grid(kFsGroup, 1, a.M, blocks, xcds, compute_units, nnz_hint, 0);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(plan.grid), dim3(kBlock), 0, s, a, lanes, (int)rows, blocks, blocks_per_xcd, xcds, plan);
    };
    if (offsets_fit_32(a)) go(flat_shared_rows_kernel<true>); else go(flat_shared_rows_kernel<false>);
    return hipGetLastError();
}

}  // namespace sgap
