// Sampled dense-dense matrix product on the pattern of a CSR matrix
// (Section 2.1, the SDDMM form under Eq. 1):
//     out[p] = vals[p] * sum_{j<J} X1[row(p), j] * X2T[colidx[p], j]
// The paper's point in naming this operator next to SpMM is that the
// reduction is the same kind of object in both (Section 2.1: here it runs
// along the dense dimension j), so the same segment-group primitives serve:
//   parallel  G lanes share one stored entry, each takes every G-th chunk of
//             c columns of the two dense rows, the group tree-sums
//             (group_tree_sum, the library's atomicAddGroup) and its first
//             lane writes the entry: {<1 nnz, 1/g col>, g} in the notation of
//             Section 3.3 with the dense dimension split instead of a row.
//   serial    r = 1: a lane walks group_size consecutive stored entries by
//             itself, whole dot products in its own register.
// Every output has exactly one writer: no atomics, no zeroing.
//
// The unit of work is a stored entry, so the schedule is nnz-balanced by
// construction: tiles of 256 to 1,024 entries are dealt to persistent workgroups
// (chunks of neighbouring tiles per die, see TileDeal), the rows of a tile's entries come from a bisection of rowptr
// for the tile's first entry and an LDS window of rowptr for the rest (the
// same pieces as the nnz-balanced SpMM kernels).  sddmm_tile_kernel has the
// parallel strategy wherever four steps of its lanes cover a dense row,
// sddmm_kernel has the rest.  Matrices whose neighbouring rows share columns go by four rows together, in the same launch.
#include <type_traits>

#include "sgap_common.hpp"
#include "sgap_lane_ops.hpp"
#include "sgap_nnz_common.hpp"
#include "sgap_sddmm_quads.hpp"

namespace sgap {

constexpr int kSddmmTile = 1024;   // stored entries per tile
constexpr int kSddmmDepth = 4;     // entries (parallel) or column chunks (serial) in flight per lane

struct SddmmArgs {
    SpmmArgs a;       // M, K, N = J, rowptr, colidx, vals; B = X2T; C unused
    const float* __restrict__ X1;
    float* __restrict__ out;
    RowSkip skip;     // entries of these rows are left alone (kernels instantiated with SKIP only),
    int32_t from_len; // and of rows shorter than this, while the list of those rows holds
};

template <int VEC>
__device__ __forceinline__ float dot_vec(const Vec<VEC>& x, const Vec<VEC>& y, float acc)
{
#pragma unroll
    for (int i = 0; i < VEC; ++i) acc = __builtin_fmaf(x.v[i], y.v[i], acc);
    return acc;
}

// The VEC columns from lane_first_col(c, J) on with those in front of c set to zero: they are the lane's in front.
template <int VEC, bool RAGGED>
__device__ __forceinline__ Vec<VEC> load_own(const float* __restrict__ row, int64_t c, int64_t J)
{
    const int64_t first = lane_first_col<VEC, RAGGED>(c, J);
    Vec<VEC> x = load_vec<VEC>(row + first);
    if constexpr (VEC > 1 && RAGGED) {
#pragma unroll
        for (int i = 0; i < VEC - 1; ++i)
            if (first + i < c) x.v[i] = 0.0f;
    }
    return x;
}

// Copy the tile's columns and values into LDS and look up the row of every
// entry through the rowptr window (cut at row boundaries where long runs of
// empty rows overflow it).  row_lb = a row at or before the tile's first
// entry.  Block-uniform; the LDS arrays are ready on return.
// skip_len > 0: entries of rows of at least skip_len or fewer than from_len stored
// entries get the one's complement of their row (a negative number) instead.
__device__ __forceinline__ void stage_tile(const SpmmArgs& a, int32_t tile_start, int32_t tile_end, int32_t row_lb,
                                           int32_t* __restrict__ s_col, float* __restrict__ s_val,
                                           int32_t* __restrict__ s_row, int32_t* __restrict__ s_win,
                                           int32_t skip_len = 0, int32_t from_len = 0)
{
    const int tid = threadIdx.x;
    const int cnt = tile_end - tile_start;
    __syncthreads();  // the previous tile is consumed
    for (int i = tid; i < cnt; i += kBlock) {
        s_col[i] = load_stream(a.colidx + tile_start + i);
        s_val[i] = load_stream(a.vals + tile_start + i);
    }
    for (int32_t base = tile_start; base < tile_end;) {
        __syncthreads();
        const RowWindow w = load_row_window(a, row_lb, base, tile_end - base, s_win);
        for (int i = tid; i < w.cnt; i += kBlock) {
            const int32_t wi = last_row_at_or_before(s_win, w.n_first, w.n_last, base + i);
            const int32_t len = s_win[wi + 1] - s_win[wi];
            const bool skipped = skip_len > 0 && (len >= skip_len || len < from_len);
            s_row[base - tile_start + i] = skipped ? ~(row_lb + wi) : row_lb + wi;
        }
        row_lb += w.n_last;
        base += w.cnt;
    }
    __syncthreads();
}

// per_lane = 0: parallel strategy, G lanes per entry.  per_lane > 0 (G = 1):
// serial strategy, per_lane consecutive entries per lane.
// SKIP: leave the entries of the rows described by s.skip alone.
template <int G, int VEC, bool RAGGED, bool SKIP = false>
__global__ __launch_bounds__(kBlock) void sddmm_kernel(SddmmArgs s, int per_lane)
{
    __shared__ int32_t s_col[kSddmmTile];
    __shared__ float s_val[kSddmmTile];
    __shared__ int32_t s_row[kSddmmTile];
    __shared__ int32_t s_win[kWindowCap + 1];
    __shared__ int32_t s_tile_row[kTileRowBatch];
    constexpr int SLOTS = kBlock / G;

    const SpmmArgs& a = s.a;
    const int tid = threadIdx.x;
    const int slot = tid / G;
    const int member = tid % G;
    const int64_t J = a.N;
    const float* __restrict__ X2T = a.B;
    const int32_t nnz = a.rowptr[a.M];
    const int64_t tiles = ((int64_t)nnz + kSddmmTile - 1) / kSddmmTile;
    const TileDeal deal(tiles, blockIdx.x, gridDim.x);
    const int64_t my_tiles = deal.mine;
    if (my_tiles == 0) return;
    int32_t skip_len = 0;
    if constexpr (SKIP) {
        skip_len = *s.skip.count <= s.skip.max_rows ? s.skip.min_len : 0;
        if (skip_len > 0 && s.from_len >= skip_len) return;  // other kernels have every row
    }

    for (int64_t j0 = 0; j0 < my_tiles; j0 += kTileRowBatch) {
        find_tile_rows(a, deal, j0, kSddmmTile, s_tile_row);
        const int64_t j1 = j0 + kTileRowBatch < my_tiles ? j0 + kTileRowBatch : my_tiles;
        for (int64_t j = j0; j < j1; ++j) {
            const int64_t t = deal.tile(j);
            const int32_t tile_start = (int32_t)(t * kSddmmTile);
            const int32_t tile_end = nnz - tile_start < kSddmmTile ? nnz : tile_start + kSddmmTile;
            const int cnt = tile_end - tile_start;
            const int32_t row_lb = s_tile_row[j - j0];

            if constexpr (SKIP) {
                // a tile that lies inside one skipped row is not even staged (row_lb is the row of the tile's
                // first entry; the same two words for every lane, so the workgroup stays together)
                if (skip_len > 0 && a.rowptr[row_lb + 1] >= tile_end &&
                    a.rowptr[row_lb + 1] - a.rowptr[row_lb] >= skip_len)
                    continue;
            }
            stage_tile(a, tile_start, tile_end, row_lb, s_col, s_val, s_row, s_win, skip_len, s.from_len);

            if (per_lane == 0) {
                // U entries per group at a time, so that 2*U rows are in flight
                constexpr int U = kSddmmDepth;
                for (int e0 = 0; e0 < cnt; e0 += U * SLOTS) {  // same trip count in every lane
                    float acc[U];
                    const float* x1p[U];
                    const float* x2p[U];
                    bool ok[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int e = e0 + u * SLOTS + slot;
                        ok[u] = e < cnt;
                        if constexpr (SKIP) ok[u] = ok[u] && s_row[e] >= 0;
                        const int32_t row = ok[u] ? s_row[e] : 0;
                        const int32_t col = ok[u] ? s_col[e] : 0;
                        x1p[u] = s.X1 + (int64_t)row * J;
                        x2p[u] = X2T + (int64_t)col * J;
                        acc[u] = 0.0f;
                    }
                    for (int64_t c = (int64_t)member * VEC; c < J; c += (int64_t)G * VEC) {
                        Vec<VEC> x1[U], x2[U];
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            x1[u].zero();
                            x2[u].zero();
                            if (ok[u]) {
                                x1[u] = load_own<VEC, RAGGED>(x1p[u], c, J);
                                x2[u] = load_own<VEC, RAGGED>(x2p[u], c, J);
                            }
                        }
#pragma unroll
                        for (int u = 0; u < U; ++u) acc[u] = dot_vec<VEC>(x1[u], x2[u], acc[u]);
                    }
                    // members past the end of the dense rows contributed +0 (zero extension)
#pragma unroll
                    for (int u = 0; u < U; ++u) acc[u] = group_tree_sum<G, 1>(acc[u]);
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int e = e0 + u * SLOTS + slot;
                        if (member == 0 && ok[u]) s.out[tile_start + e] = s_val[e] * acc[u];
                    }
                }
            } else if constexpr (G == 1) {
                constexpr int U = kSddmmDepth;
                for (int i = 0; i < per_lane; ++i) {
                    for (int e = (tid * per_lane + i); e < cnt; e += kBlock * per_lane) {
                        if constexpr (SKIP) {
                            if (s_row[e] < 0) continue;
                        }
                        const float* __restrict__ x1p = s.X1 + (int64_t)s_row[e] * J;
                        const float* __restrict__ x2p = X2T + (int64_t)s_col[e] * J;
                        float acc = 0.0f;
                        int64_t c = 0;
                        for (; c + U * VEC <= J; c += U * VEC) {
                            Vec<VEC> x1[U], x2[U];
#pragma unroll
                            for (int u = 0; u < U; ++u) {
                                x1[u] = load_vec<VEC>(x1p + c + u * VEC);
                                x2[u] = load_vec<VEC>(x2p + c + u * VEC);
                            }
#pragma unroll
                            for (int u = 0; u < U; ++u) acc = dot_vec<VEC>(x1[u], x2[u], acc);
                        }
                        for (; c < J; c += VEC) acc = dot_vec<VEC>(load_own<VEC, RAGGED>(x1p, c, J), load_own<VEC, RAGGED>(x2p, c, J), acc);
                        s.out[tile_start + e] = s_val[e] * acc;
                    }
                }
            }
        }
    }
}

// Parallel strategy when the G lanes of a group cover a dense row in S <= 4 steps of 4 columns each (J <= S*G*4).
// Every wavefront walks a quarter of the tile, (64/G)*U consecutive entries at a time, U consecutive ones per group.
// What bounds the kernel is the vector memory path that brings in one row of X2T per entry, so everything else is kept
// off it and off the vector units:
//   - the rows of X1 that the tile touches are copied to LDS once (x1_rows of them fit; a tile of short rows, whose
//     rows change with nearly every entry, reads them from memory), and read from there when a group's row changes;
//   - the row of an entry comes from the window of rows with entries (compact_window): a thread bisects it for the
//     first of its EPT entries and steps along for the others;
//   - one multiply-add forms the address of a row of X2T, its S steps differ by a constant offset;
//   - the next tile's entries and row pointers are requested before this one is multiplied out.
// stencil27, J = 128, G = 8: 1,031 us with tiles of 1,024 entries, rows of X1 read from memory per batch and a
// bisection per entry; 831 us with the above, at 2.3 instead of 4.7 GB moved (the tile: see try_tile).
// IN_STEP: what was left then was the L1: a workgroup that takes the rows one after the other finds only consecutive
// columns there, and asks the L2 for twice the lines that SpMM's row-split kernel does with eight rows in step.  So a
// tile's entries change their order: the first ones of all its rows, then the second ones, and so on, the wavefronts
// through it together.  No lane waits for a longer row (a kernel that gave every row its lanes took two to three times as
// long on R-MAT, whose heavy rows sit together).  Four instead of eight loads in flight per lane, six wavefronts per SIMD
// instead of four: 831 -> 675 us (stencil of 60 x 57 x 62: 160 -> 132; in step with eight loads in flight: 790).  Columns
// without order: uniform, 5 entries a row 97 -> 94, R-MAT of 2^18 rows 186 -> 184; uniform, 30 a row 99 -> 102, power law
// 123 -> 128.
// EDGE: J is not S*G*4 (lanes without columns, or a ragged last chunk).  Those instances with S = 4 and 512 entries keep
// two registers in memory; computed anew per tile, what they hold costs more (R-MAT of 2^19 rows, J = 35, G = 4: 165.9
// us against 164.8).
// In step: J above 64 that is one, two or four times G * 4, so that no lane is to spare (at the groups of 8 and 16 that is 128
// alone, and 256 with 16).  Tiles of 512 entries, J up to 64, keep a wavefront's entries together, and so do the EDGE
// instances: in step they measured 182 -> 171 us (stencil of 60 x 57 x 62, G = 8, J = 120), 176 -> 171 (100), 161 -> 165 (96),
// 161 -> 162 (72), R-MAT of 2^18 rows 234 -> 221 (100), 184 -> 174 (96).
__host__ __device__ constexpr bool in_step(bool edge, int ept) { return !edge && ept == 1; }
constexpr int kX1LdsBytes = 10 * 1024;  // rows of X1 in LDS per 256 entries of a tile: 20 of 512 bytes
__host__ __device__ constexpr int x1_pitch(int columns, bool edge, int ept)
{
    return in_step(edge, ept) && columns % 64 == 0 ? columns + 32 : columns;
}

// QUADS: where rows turn out to share columns, the matrix is taken by four rows together (sgap_sddmm_quads.hpp), by all
// workgroups of the grid; else by the first `workers` of them, tile by tile, as above.  resident: workgroups of a die at a time.
// QUADS with IN_STEP: seven wavefronts per SIMD, as without QUADS, which takes 72 vector registers and 96 scalar ones.  The occupancy
// that sizes the grid goes by the vector registers; of scalar ones a SIMD has 800, handed out in sixteens, and the trap handler
// takes sixteen of each wavefront: with 100 six wavefronts were resident, and the persistent grid's last seventh ran in a second
// round (tile by tile, J = 128, G = 16: 4.8 M entries without order 366 -> 385 us, 366 so; 6.5 M that share half of their columns with
// the row above 161 -> 231, 162 so).  With six, and 76 vector registers, the stencil below takes 546 us by four rows together instead
// of 553, but tile by tile everything takes 1 to 8 % more.
// From 68 columns on, and 132 where an entry has twice the lanes or steps (of 64, a 60 x 57 x 62 stencil takes 86 us tile by tile and
// 94 so); with one step from 72 and 136 on: just above 64 a lane has four columns tile by tile, or twice that, and sums them no
// less exactly than CHAINS do here.  Relative error against 64 bits, tile by tile and so, and time on that stencil: G = 8, J = 65
// 7.63e-8 / 7.69e-8 and 157 / 127 us, J = 68 7.75e-8 / 7.66e-8 and 158 / 129; G = 16, J = 67 7.30e-8 / 7.32e-8, J = 68 7.34e-8 / 7.32e-8,
// 163 / 129 us; G = 32, one step, J = 68 7.29e-8 / 7.32e-8, J = 72 7.35e-8 / 7.35e-8; G = 64, J = 132 7.76e-8 / 7.78e-8.
__host__ __device__ constexpr bool has_quads(int g, int s, int ept) { return ept == 1 && (s * g == 32 || s * g == 64); }  // up to 256 columns
// Stored entries from which on a matrix is looked at for such rows: the look takes 2 us where it finds none.  40 x 41 x 42
// points, 1.8 M entries: J = 100 59.9 -> 49.7 us, J = 72 55.2 -> 49.0, J = 256 141 -> 82, but J = 128, which the tiles have in
// step, 55.0 -> 51.4 in groups of 8 and 59.4 -> 62.6 of 16; 60 x 57 x 62, 5.5 M, J = 128: 123 -> 118 and 128 -> 115; 31 x 30 x 33
// points, 0.8 M: J = 100 35.6 -> 32.6, J = 128 27.2 -> 28.6.
constexpr int64_t quads_from(bool step128) { return step128 ? 3000000 : 1500000; }
// Whether a call is launched so that it looks (chunks: of four columns, that the lanes and steps of an entry hold)
constexpr bool looks_for_quads(int64_t M, int64_t K, int64_t J, int steps, int chunks, int64_t nnz_hint)
{
    return J >= chunks * 2 + (steps > 1 ? 4 : 8) && K * J * 4 <= 0xffffffffLL && nnz_hint >= quads_from(J == 128 && chunks == 32) &&
           nnz_hint > kQuadMeanRow * M && nnz_hint < kQuadRow * M;
}
static_assert(1500000 / kQuadRow >= kLookRun, "so many entries come with enough rows to look at");
// Chains that four lanes' sixteen columns are summed in by four rows together: none longer than a lane has tile by tile, which
// takes S steps of four columns, with EDGE more than half of them.
__host__ __device__ constexpr int quad_chains(int s, bool edge) { return edge ? (s == 4 ? 2 : 4) : 4 / s; }

template <int G, int S, bool EDGE, int EPT, bool QUADS>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(QUADS && in_step(EDGE, EPT) ? 7 : 4))) void sddmm_tile_kernel(SddmmArgs s, int x1_rows, uint32_t workers, uint32_t resident)
{
    constexpr int VEC = 4;
    constexpr bool IN_STEP = in_step(EDGE, EPT);
    constexpr int GROUPS = kWave / G;
    constexpr int TILE = EPT * kBlock;
    constexpr int WAVE_RUN = TILE / kWavesPerBlock;
    constexpr int U0 = (IN_STEP ? 4 : 8) / S;  // entries per group and batch: 4 or 8 loads in flight per lane
    constexpr int U = U0 * GROUPS > WAVE_RUN ? WAVE_RUN / GROUPS : U0;
    // floats of one row of X1 in LDS, zeros behind column J; IN_STEP: groups read neighbouring rows at the same columns
    // together, so neighbours begin in different halves of the banks
    constexpr int PITCH = x1_pitch(S * G * VEC, EDGE, EPT);
    constexpr int ROW_CHUNKS = S * G;
    constexpr int WPT = EPT + 1;  // row pointers per thread: a window of TILE rows
    extern __shared__ __align__(16) float s_x1[];
    __shared__ __align__(16) int32_t s_col[TILE];
    __shared__ __align__(16) float s_val[TILE];
    __shared__ __align__(16) uint16_t s_idx[TILE];  // window index of the entry's row
    // IN_STEP: where an entry comes from in the tile, and the results in the tile's order
    __shared__ uint16_t s_from[IN_STEP ? TILE : 1];
    __shared__ float s_out[IN_STEP ? TILE : 1];
    __shared__ int32_t s_win[TILE + 1];
    __shared__ int32_t s_row[TILE];
    __shared__ int32_t s_scan[kWavesPerBlock];
    __shared__ int32_t s_tile_row[kTileRowBatch];

    const SpmmArgs& a = s.a;
    const int tid = threadIdx.x;
    const int lane = tid % kWave;
    const int wave = tid / kWave;
    const int grp = lane / G;
    const int member = lane % G;
    const int32_t J = (int32_t)a.N;
    const uint32_t row_bytes = (uint32_t)J * 4u;
    const int32_t M = (int32_t)a.M;
    const int32_t nnz = a.rowptr[a.M];
    bool by_quads = false;
    if constexpr (QUADS) {
        by_quads = rows_share_columns(a, nnz, S * G > 32, s_tile_row);
        if (by_quads)
            sddmm_quads(a, s.X1, s.out, DotColumns<S * G / 4, quad_chains(S, EDGE), EDGE>(J), reinterpret_cast<QuadDots*>(s_x1)[__builtin_amdgcn_readfirstlane(wave)], TILE, resident);
    }
    if (blockIdx.x >= workers) return;
    const int64_t tiles = ((int64_t)nnz + TILE - 1) / TILE;
    const TileDeal deal(tiles, blockIdx.x, workers);
    const int64_t my_tiles = deal.mine;
    if constexpr (QUADS) {
        if (by_quads) {
            for (int64_t j0 = 0; j0 < my_tiles; j0 += kTileRowBatch) {
                find_tile_rows(a, deal, j0, TILE, s_tile_row);
                const bool have = j0 + tid < my_tiles;
                const int32_t tile_start = have ? (int32_t)(deal.tile(j0 + tid) * TILE) : 0;
                tiles_of_long_quads(a, s.X1, s.out, DotColumns<S * G / 4, quad_chains(S, EDGE), EDGE>(J), have, have ? s_tile_row[tid] : 0, tile_start, TILE);
            }
            return;
        }
    }
    if (my_tiles == 0) return;
    TileWalk ahead(deal);  // the tile that is fetched next

    // this lane's columns in step st: (st*G + member)*4 ..; c_first = the first column it loads
    bool c_ok[S];
    int32_t c_first[S];
#pragma unroll
    for (int st = 0; st < S; ++st) {
        const int32_t c = (st * G + member) * VEC;
        c_ok[st] = !EDGE || c < J;
        c_first[st] = EDGE ? (c_ok[st] ? (int32_t)lane_first_col<VEC>((uint32_t)c, (uint32_t)J) : 0) : c;
    }
    // the lane's chunk of a row of X1 or X2T (the columns it shares with the lane in front of it as zeros)
    auto load_chunk = [&](const float* base, int32_t row, int st) {
        const char* p = reinterpret_cast<const char*>(base + (EDGE ? c_first[st] : member * VEC)) + (uint64_t)(uint32_t)row * row_bytes;
        Vec<VEC> x;
        if constexpr (EDGE) {
            x.zero();
            if (c_ok[st]) x = load_vec<VEC>(reinterpret_cast<const float*>(p));
#pragma unroll
            for (int i = 0; i < VEC - 1; ++i)
                if (c_first[st] + i < (st * G + member) * VEC) x.v[i] = 0.0f;
        } else {
            x = load_vec<VEC>(reinterpret_cast<const float*>(p) + st * G * VEC);
        }
        return x;
    };

    int32_t nx_col[EPT];
    float nx_val[EPT];
    int32_t nx_win[WPT];
    auto fetch_tile = [&](int32_t row_lb) {  // the tile `ahead` stands at
        const int32_t start = (int32_t)(ahead.tile() * TILE);
#pragma unroll
        for (int i = 0; i < EPT; ++i) {
            const int32_t p = start + tid + i * kBlock;
            nx_col[i] = 0;  // (positions past the end gather row 0 of X2T, and nothing of them is written)
            nx_val[i] = 0.0f;
            if (p < nnz) {
                nx_col[i] = load_stream(a.colidx + p);
                nx_val[i] = load_stream(a.vals + p);
            }
        }
#pragma unroll
        for (int i = 0; i < WPT; ++i) {
            const int w = tid + i * kBlock;
            const int64_t r = (int64_t)row_lb + w;
            nx_win[i] = w <= TILE ? a.rowptr[r <= M ? r : M] : 0;
        }
    };

    for (int64_t j0 = 0; j0 < my_tiles; j0 += kTileRowBatch) {
        find_tile_rows(a, deal, j0, TILE, s_tile_row);
        const int64_t j1 = j0 + kTileRowBatch < my_tiles ? j0 + kTileRowBatch : my_tiles;
        fetch_tile(s_tile_row[0]);
        for (int64_t j = j0; j < j1; ++j) {
            const int32_t tile_start = (int32_t)(ahead.tile() * TILE);
            ahead.next();
            const int32_t tile_end = nnz - tile_start < TILE ? nnz : tile_start + TILE;
            const int cnt = tile_end - tile_start;
            const int32_t row_lb = s_tile_row[j - j0];
            // install the tile that was fetched ahead (the barrier at the end of the loop: the last one is consumed)
            const int32_t my_col = nx_col[0];
            const float my_val = nx_val[0];
            if constexpr (!IN_STEP) {
#pragma unroll
                for (int i = 0; i < EPT; ++i) {
                    s_col[tid + i * kBlock] = nx_col[i];
                    s_val[tid + i * kBlock] = nx_val[i];
                }
            }
#pragma unroll
            for (int i = 0; i < WPT; ++i)
                if (tid + i * kBlock <= TILE) s_win[tid + i * kBlock] = nx_win[i];
            __syncthreads();
            if (j + 1 < j1) fetch_tile(s_tile_row[j + 1 - j0]);
            int32_t n;  // rows with entries in the tile: first positions in s_win, numbers in s_row
            if (s_win[TILE] >= tile_end) {
                n = compact_window<TILE>(s_win, s_row, row_lb, tile_end, s_scan);
            } else {
                __syncthreads();  // everyone has read the plain window
                n = load_compact_window(a, row_lb, tile_end, s_win, s_row, s_scan);
            }
            const bool x1_in_lds = n <= x1_rows;
            if (x1_in_lds) {
                for (int i = tid; i < n * ROW_CHUNKS; i += kBlock) {
                    const int r = i / ROW_CHUNKS;
                    const int32_t c = i % ROW_CHUNKS * VEC;
                    Vec<VEC> x;
                    if constexpr (EDGE) {
                        x.zero();
                        if (c < J) {
                            const int32_t first = (int32_t)lane_first_col<VEC>((uint32_t)c, (uint32_t)J);
                            x = load_vec<VEC>(s.X1 + (int64_t)s_row[r] * J + first);
#pragma unroll
                            for (int v = 0; v < VEC - 1; ++v)
                                if (first + v < c) x.v[v] = 0.0f;
                        }
                    } else {
                        x = load_vec<VEC>(s.X1 + (int64_t)s_row[r] * J + c);
                    }
                    *reinterpret_cast<float4*>(s_x1 + r * PITCH + c) = make_float4(x.v[0], x.v[1], x.v[2], x.v[3]);
                }
            }
            if constexpr (IN_STEP) {
                // Entry number i of its row in the tile comes behind the entries number 0 .. i - 1 of every row and those
                // number i of the rows in front: where rows have entries alike, neighbouring rows' come together.
                const int32_t p = tile_start + tid;
                const int32_t wi = last_row_at_or_before(s_win, 0, n - 1, p);
                int32_t place = tid;
                if (x1_in_lds && tid < cnt) {
                    const int32_t number = p - (s_win[wi] > tile_start ? s_win[wi] : tile_start);
                    int32_t begin = tile_start;  // of a row, in the tile
                    place = 0;
                    for (int32_t r = 0; r < n; ++r) {
                        const int32_t end = s_win[r + 1] < tile_end ? s_win[r + 1] : tile_end;
                        const int32_t limit = number + (r < wi ? 1 : 0);
                        place += end - begin < limit ? end - begin : limit;
                        begin = end;
                    }
                }
                s_col[place] = my_col;
                s_val[place] = my_val;
                s_idx[place] = (uint16_t)wi;
                s_from[place] = (uint16_t)tid;
            } else {
                int32_t wi = last_row_at_or_before(s_win, 0, n - 1, tile_start + tid * EPT);
#pragma unroll
                for (int i = 0; i < EPT; ++i) {
                    // (every row of the window has entries: at most one step per position; the last row's end is the window's)
                    if (wi + 1 < n && s_win[wi + 1] <= tile_start + tid * EPT + i) ++wi;
                    s_idx[tid * EPT + i] = (uint16_t)wi;
                }
            }
            __syncthreads();

            // One batch of B entries per group from slot b on; LDS_X1: the rows of X1 come from LDS, where a group reads
            // one when its row changes (cur); else every entry's row is requested along with its row of X2T.
            int32_t cur = -1;
            Vec<VEC> x1c[S];  // the chunk of X1's row `cur` this lane owns
#pragma unroll
            for (int st = 0; st < S; ++st) x1c[st].zero();
            auto batch = [&](int b, auto b_const, auto lds_const) {
                constexpr int B = decltype(b_const)::value;
                constexpr bool LDS_X1 = decltype(lds_const)::value;
                // (IN_STEP: neighbouring groups on neighbouring entries; else a group's entries, and so its results, together)
                const int e = IN_STEP ? b + grp : b + grp * B;
                constexpr int NEXT = IN_STEP ? GROUPS : 1;
                float acc[B];
                Vec<VEC> x2[B][S];
#pragma unroll
                for (int u = 0; u < B; ++u) {
                    acc[u] = 0.0f;
#pragma unroll
                    for (int st = 0; st < S; ++st) x2[u][st] = load_chunk(a.B, s_col[e + u * NEXT], st);
                }
                if constexpr (LDS_X1) {
#pragma unroll
                    for (int u = 0; u < B; ++u) {
                        const int32_t idx = s_idx[e + u * NEXT];
                        if (idx != cur) {
#pragma unroll
                            for (int st = 0; st < S; ++st) {
                                const float4 t = *reinterpret_cast<const float4*>(s_x1 + idx * PITCH + (st * G + member) * VEC);
                                x1c[st].v[0] = t.x; x1c[st].v[1] = t.y; x1c[st].v[2] = t.z; x1c[st].v[3] = t.w;
                            }
                            cur = idx;
                        }
#pragma unroll
                        for (int st = 0; st < S; ++st) acc[u] = dot_vec<VEC>(x1c[st], x2[u][st], acc[u]);
                    }
                } else {
                    Vec<VEC> x1[B][S];
#pragma unroll
                    for (int u = 0; u < B; ++u) {
                        const int32_t row = s_row[s_idx[e + u * NEXT]];
#pragma unroll
                        for (int st = 0; st < S; ++st) x1[u][st] = load_chunk(s.X1, row, st);
                    }
#pragma unroll
                    for (int u = 0; u < B; ++u) {
#pragma unroll
                        for (int st = 0; st < S; ++st) acc[u] = dot_vec<VEC>(x1[u][st], x2[u][st], acc[u]);
                    }
                }
#pragma unroll
                for (int u = 0; u < B; ++u) acc[u] = group_tree_sum<G, 1>(acc[u]);
                if constexpr (IN_STEP) {
                    if (member == 0) {
#pragma unroll
                        for (int u = 0; u < B; ++u) s_out[s_from[e + u * NEXT]] = acc[u] * s_val[e + u * NEXT];
                    }
                } else if (member == 0) {
                    // the group's outputs are consecutive, and so are the groups'
#pragma unroll
                    for (int u = 0; u < B; ++u) acc[u] *= s_val[e + u];
                    if (B % VEC == 0 && e + B <= cnt) {
#pragma unroll
                        for (int u = 0; u + VEC <= B; u += VEC) {
                            const Vec<VEC> o = {acc[u], acc[u + 1], acc[u + 2], acc[u + 3]};
                            store_vec_stream<VEC>(s.out + tile_start + e + u, o);
                        }
                    } else {
#pragma unroll
                        for (int u = 0; u < B; ++u)
                            if (e + u < cnt) s.out[tile_start + e + u] = acc[u];
                    }
                }
            };
            const int run_end = (wave + 1) * WAVE_RUN < cnt ? (wave + 1) * WAVE_RUN : cnt;
            if (x1_in_lds) {
                if constexpr (IN_STEP) {
                    for (int b = wave * GROUPS * U; b < cnt; b += kWavesPerBlock * GROUPS * U)
                        batch(b, std::integral_constant<int, U>{}, std::true_type{});
                } else {
                    for (int b = wave * WAVE_RUN; b < run_end; b += GROUPS * U)
                        batch(b, std::integral_constant<int, U>{}, std::true_type{});
                }
            } else {
                constexpr int H = U < 2 ? 1 : U / 2;
                for (int b = wave * WAVE_RUN; b < run_end; b += GROUPS * H)
                    batch(b, std::integral_constant<int, H>{}, std::false_type{});
            }
            __syncthreads();  // the tile is consumed
            if constexpr (IN_STEP) {
                // (nobody writes here before the barriers of the next tile)
                if (tid < cnt) __builtin_nontemporal_store(s_out[tid], s.out + tile_start + tid);
            }
        }
    }
}

namespace {

template <int G, int S, bool EDGE, int EPT>
void launch_tile(const SddmmArgs& s, int compute_units, int64_t nnz_hint, hipStream_t stream)
{
    constexpr int x1_rows = EPT * kX1LdsBytes / (S * G * 16);
    constexpr int x1_bytes = x1_rows * x1_pitch(S * G * 4, EDGE, EPT) * 4;
    if constexpr (has_quads(G, S, EPT)) {
        if (looks_for_quads(s.a.M, s.a.K, s.a.N, S, S * G, nnz_hint)) {
            static_assert(x1_bytes >= (int)sizeof(QuadDots) * kWavesPerBlock, "either is in the same place");
            static const int per_cu = resident_per_cu(sddmm_tile_kernel<G, S, EDGE, EPT, true>, x1_bytes);
            const uint32_t workers = (uint32_t)persistent_grid(per_cu, compute_units, nnz_hint, EPT * kBlock);
            const uint32_t all = (uint32_t)(per_cu * compute_units), resident = all >= kQuadDies ? all / kQuadDies : 1;
            const uint32_t grid = quad_workgroups(s.a.M, resident) > workers ? quad_workgroups(s.a.M, resident) : workers;
            hipLaunchKernelGGL((sddmm_tile_kernel<G, S, EDGE, EPT, true>), dim3(grid), dim3(kBlock), x1_bytes, stream, s, x1_rows, workers, resident);
            return;
        }
    }
    static const int per_cu = resident_per_cu(sddmm_tile_kernel<G, S, EDGE, EPT, false>, x1_bytes);
    const uint32_t grid = (uint32_t)persistent_grid(per_cu, compute_units, nnz_hint, EPT * kBlock);
    hipLaunchKernelGGL((sddmm_tile_kernel<G, S, EDGE, EPT, false>), dim3(grid), dim3(kBlock), x1_bytes, stream, s, x1_rows, grid, 0u);
}

// Steps of G*4 columns that cover J: 1, 2 or 4 pick sddmm_tile_kernel, 0 = more than 4.
constexpr int tile_steps(int64_t J, int g)
{
    const int64_t steps = (J + g * 4 - 1) / (g * 4);
    return steps <= 2 ? (steps <= 1 ? 1 : 2) : steps <= 4 ? 4 : 0;
}

// Tile: the entries that all resident workgroups work on at a time decide whether neighbouring rows find each other's
// rows of X2T in the die's L2: 256 entries for wide rows (stencil27, J = 128: 825 us, 512 entries 958, 1,024 entries
// 1,038), twice that for rows of up to 64 columns, where the work per tile weighs more (57 x 60 x 62 stencil, J = 34:
// 92 us against 107; R-MAT alike).
template <int G>
bool try_tile(const SddmmArgs& s, int64_t J, int compute_units, int64_t nnz_hint, hipStream_t stream)
{
    auto pick = [&](auto s_const) {
        constexpr int S = decltype(s_const)::value;
        const bool edge = J != S * G * 4;
        if (S * G <= 16 || J <= 64) {
            if (edge) launch_tile<G, S, true, 2>(s, compute_units, nnz_hint, stream);
            else launch_tile<G, S, false, 2>(s, compute_units, nnz_hint, stream);
        } else if constexpr (S * G > 16) {
            if (edge) launch_tile<G, S, true, 1>(s, compute_units, nnz_hint, stream);
            else launch_tile<G, S, false, 1>(s, compute_units, nnz_hint, stream);
        }
    };
    switch (tile_steps(J, G)) {
        case 1: pick(std::integral_constant<int, 1>{}); return true;
        case 2: pick(std::integral_constant<int, 2>{}); return true;
        case 4: pick(std::integral_constant<int, 4>{}); return true;
        default: return false;
    }
}

template <int G, int VEC, bool RAGGED>
void launch_one(const SddmmArgs& s, int per_lane, int compute_units, int64_t nnz_hint, hipStream_t stream)
{
    static const int per_cu = resident_per_cu(sddmm_kernel<G, VEC, RAGGED>, 0);
    const int grid = persistent_grid(per_cu, compute_units, nnz_hint, kSddmmTile);
    hipLaunchKernelGGL((sddmm_kernel<G, VEC, RAGGED>), dim3(grid), dim3(kBlock), 0, stream, s, per_lane);
}

template <int G>
void launch_skip(const SddmmArgs& s, int per_lane, int compute_units, int64_t nnz_hint, hipStream_t stream)
{
    static const int per_cu = resident_per_cu(sddmm_kernel<G, 4, false, true>, 0);
    const int grid = persistent_grid(per_cu, compute_units, nnz_hint, kSddmmTile);
    hipLaunchKernelGGL((sddmm_kernel<G, 4, false, true>), dim3(grid), dim3(kBlock), 0, stream, s, per_lane);
}

template <int G>
bool launch_vec(const SddmmArgs& s, int vec, int per_lane, int compute_units, int64_t nnz_hint, hipStream_t stream)
{
    switch (vec) {
        case 4:
            if (s.a.N % 4 != 0) launch_one<G, 4, true>(s, per_lane, compute_units, nnz_hint, stream);
            else launch_one<G, 4, false>(s, per_lane, compute_units, nnz_hint, stream);
            return true;
        case 2: launch_one<G, 2, true>(s, per_lane, compute_units, nnz_hint, stream); return true;
        case 1: launch_one<G, 1, false>(s, per_lane, compute_units, nnz_hint, stream); return true;
        default: return false;
    }
}

}  // namespace

// a: M, K, N = J, rowptr, colidx, vals, B = X2T (C unused).  g = lanes per
// stored entry (parallel strategy, per_lane = 0) or 1 with per_lane = entries
// per lane (serial strategy).  vec = columns per lane and load (lane_columns(J)).
// row_cache: let the parallel strategy keep the rows of X1 that a tile touches
// in LDS where the shape allows it.
hipError_t launch_sddmm(const SpmmArgs& a, const float* X1, float* out, int g, int per_lane, int vec, bool row_cache,
                        int compute_units, int64_t nnz_hint, hipStream_t stream)
{
    SddmmArgs s;
    s.a = a;
    s.X1 = X1;
    s.out = out;
    s.skip = RowSkip{nullptr, 0, 0};
    s.from_len = 0;
    bool ok = false;
    if (per_lane > 0) {
        ok = launch_vec<1>(s, vec, per_lane, compute_units, nnz_hint, stream);
    } else if (vec == 4 && row_cache && a.N > 0) {
        switch (g) {
            case 1: ok = try_tile<1>(s, a.N, compute_units, nnz_hint, stream); break;
            case 2: ok = try_tile<2>(s, a.N, compute_units, nnz_hint, stream); break;
            case 4: ok = try_tile<4>(s, a.N, compute_units, nnz_hint, stream); break;
            case 8: ok = try_tile<8>(s, a.N, compute_units, nnz_hint, stream); break;
            case 16: ok = try_tile<16>(s, a.N, compute_units, nnz_hint, stream); break;
            case 32: ok = try_tile<32>(s, a.N, compute_units, nnz_hint, stream); break;
            case 64: ok = try_tile<64>(s, a.N, compute_units, nnz_hint, stream); break;
            default: break;
        }
        if (!ok) return launch_sddmm(a, X1, out, g, per_lane, vec, false, compute_units, nnz_hint, stream);
    } else {
        switch (g) {
            case 1: ok = launch_vec<1>(s, vec, 0, compute_units, nnz_hint, stream); break;
            case 2: ok = launch_vec<2>(s, vec, 0, compute_units, nnz_hint, stream); break;
            case 4: ok = launch_vec<4>(s, vec, 0, compute_units, nnz_hint, stream); break;
            case 8: ok = launch_vec<8>(s, vec, 0, compute_units, nnz_hint, stream); break;
            case 16: ok = launch_vec<16>(s, vec, 0, compute_units, nnz_hint, stream); break;
            case 32: ok = launch_vec<32>(s, vec, 0, compute_units, nnz_hint, stream); break;
            case 64: ok = launch_vec<64>(s, vec, 0, compute_units, nnz_hint, stream); break;
            default: break;
        }
    }
    if (!ok) return hipErrorInvalidValue;
    return hipGetLastError();
}

// What the parallel strategy with g lanes per entry does with a matrix in host memory: rows_share_columns by a single thread.
bool sddmm_by_quads(int64_t M, int64_t K, int64_t J, int g, int64_t nnz_hint, const int32_t* rowptr, const int32_t* colidx)
{
    const int steps = tile_steps(J, g), chunks = steps * g;
    if (J <= 64 || !(chunks == 32 || chunks == 64) || !looks_for_quads(M, K, J, steps, chunks, nnz_hint)) return false;
    int long_rows = 0, shared = 0, total = 0;
    for (int i = 0; i < kLookRuns; ++i) {
        const int32_t* p = rowptr + look_run((uint32_t)i, M);
        for (int r = 0; r < kLookRun; ++r) long_rows += p[r + 1] - p[r] >= kQuadRow;
        for (int n = 0; n < kLookPairs; ++n) {
            const int32_t* row = p + look_at(n / 2, n % 2);
            int32_t above[kQuadRow];
            for (int q = 0; q < kQuadRow; ++q) above[q] = row[0] + q < row[1] ? colidx[row[0] + q] : kNoColumn;
            for (int q = 0; q < kQuadRow && row[1] + q < row[2]; ++q) {
                const int32_t c = colidx[row[1] + q];
                int lo = 0;
                for (int half = kQuadRow / 2; half > 0; half /= 2) lo += above[lo + half - 1] < c ? half : 0;
                shared += above[lo] == c;
                ++total;
            }
        }
    }
    return lengths_for_quads(M, rowptr[M], long_rows, chunks > 32) && columns_for_quads(shared, total, chunks > 32);
}

// The plain kernel (16-byte loads: J % 4 == 0, aligned operands) on the rows of at least from_len entries
// that are not described by `skip`; on every row if that list is too long to hold.
hipError_t launch_sddmm_rest(const SpmmArgs& a, const float* X1, float* out, int g, int per_lane, int compute_units,
                             int64_t nnz_hint, const RowSkip& skip, int32_t from_len, hipStream_t stream)
{
    SddmmArgs s;
    s.a = a;
    s.X1 = X1;
    s.out = out;
    s.skip = skip;
    s.from_len = from_len;
    switch (per_lane > 0 ? 1 : g) {
        case 1: launch_skip<1>(s, per_lane, compute_units, nnz_hint, stream); break;
        case 2: launch_skip<2>(s, per_lane, compute_units, nnz_hint, stream); break;
        case 4: launch_skip<4>(s, per_lane, compute_units, nnz_hint, stream); break;
        case 8: launch_skip<8>(s, per_lane, compute_units, nnz_hint, stream); break;
        case 16: launch_skip<16>(s, per_lane, compute_units, nnz_hint, stream); break;
        case 32: launch_skip<32>(s, per_lane, compute_units, nnz_hint, stream); break;
        case 64: launch_skip<64>(s, per_lane, compute_units, nnz_hint, stream); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace sgap
