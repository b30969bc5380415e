// Nnz-balanced schedule, parallel strategy, for rows of B that a few lanes hold (N <= kNarrowColumns): the
// segmented reduction with several consecutive stored entries per lane.
//
// With one entry per lane (sgap_nnz_parallel_impl.hpp) a 16-byte row of B costs a 16-byte LDS record that has to be built
// first, behind the row window, and a shuffle step per entry and column.  Here a lane holds E consecutive entries, which
// come with 16-byte loads straight into registers, so that
//   - the rows of B are asked for before anything is known about the rows of A, which are looked up meanwhile;
//   - a lane adds up its own entries, and a run of entries of one row that spans lanes costs one segmented scan per E
//     entries (inside 16 lanes by DPP, then two steps across them), whatever `group_size` says;
//   - no record is built: the rows of the tile mark the place of their last entry in LDS, and a lane reads the E places
//     of its entries with one or two 16-byte reads.
// Runs that span wavefronts go on through LDS, in order and without atomics; rows that cross a tile's boundary are
// merged with global atomics under the merge rule (tile mode), 32 tiles' of them together: among the tiles, where they
// share the wavefronts' one counter of outstanding accesses and its order with the gathers, the few of them cost as much
// as all other writes (R-MAT of 2^21 rows, N = 1: 341 us with them in their places, 295 without them, 300 so).
//   thread = entry_lane * LC + chunk ; tile = kBlock / LC * E positions
// Bound by the gathers: 50 M of them, each of a line of its own, take 243 us (4 bytes) and 282 us (16 bytes) with R-MAT's
// columns and nothing else to do (the L2s deliver some 220 G lines a second, 63 G where they come from beyond), to which
// come 200 MB of values and the zeroing pass.  us, R-MAT with 2^21 rows and 50 M entries, one entry per lane / E:
//   N = 1 418 / 285   N = 2 359 / 315   N = 4 396 / 340   N = 8 646 / 455   N = 16 1,112 / 614;
//   2^16 rows and 0.9 M entries: 18.5 / 11.0, 19.0 / 11.7, 20.0 / 12.7, 26.5 / 15.1, 34.5 / 18.2
// Rows of one entry each lose, since every entry is then a store by itself, and neighbouring lanes' are E rows apart: 2,000,000 of
// them, N = 1 37.1 / 41.5 (G = 64), N = 8 63.8 / 66.8 and N = 16 76.7 / 84.9 (G = 8); rows of three gain again.
// E = 4 where one lane holds the columns (with eight N = 4 takes 357 us, N = 2 320, N = 1 286), 8 elsewhere (N = 8 with
// four 440 us, but 16.1 on the small matrix).
#include "sgap_common.hpp"
#include "sgap_lane_ops.hpp"
#include "sgap_nnz_common.hpp"

namespace sgap {

namespace {

typedef int32_t native_i4 __attribute__((ext_vector_type(4), aligned(4)));
typedef int32_t lds_i4 __attribute__((ext_vector_type(4)));

// Place of a row's last entry in the tile: the row, kOutside with it where the row also has entries in other tiles;
// kNoEnd where no row ends.  (M <= 2^31 - 1, so that no row's number with kOutside is kNoEnd.)
constexpr int32_t kNoEnd = -1;
constexpr int32_t kOutside = (int32_t)0x80000000;

// DPP move of a float: lane i receives the lane that CTRL names, 0 where there is none.
template <int CTRL>
__device__ __forceinline__ float dpp_from(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
constexpr int kRowShr = 0x110, kWaveShr1 = 0x138, kRowBcast15 = 0x142, kRowBcast31 = 0x143;

// Value of the last entry lane of the 16 lanes in front of mine (of lane 31's 16 lanes where HALF), same chunk.  Valid
// in the odd rows of 16 lanes (HALF: in the upper 32 lanes).
template <int LC, bool HALF>
__device__ __forceinline__ float from_row_in_front(float v)
{
    if constexpr (LC == 1) {
        return dpp_from<HALF ? kRowBcast31 : kRowBcast15>(v);
    } else {
        const int lane = lane_id();
        const int src = (HALF ? 32 : (lane & ~15)) - LC + lane % LC;
        return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute((src & 63) << 2, __builtin_bit_cast(int, v)));
    }
}

// Value of the entry lane in front of mine, same chunk; 0 in the first one.
template <int LC>
__device__ __forceinline__ float from_lane_in_front(float v)
{
    if constexpr (LC == 1) {
        return dpp_from<kWaveShr1>(v);
    } else {
        const int lane = lane_id();
        const float t = __builtin_bit_cast(
            float, __builtin_amdgcn_ds_bpermute(((lane - LC) & 63) << 2, __builtin_bit_cast(int, v)));
        return lane < LC ? 0.0f : t;
    }
}

template <int D, int LC, int VEC>
__device__ __forceinline__ void scan_rows_of_16(Vec<VEC>& v, int dist)
{
    if constexpr (D * LC < 16) {
        Vec<VEC> t;
#pragma unroll
        for (int i = 0; i < VEC; ++i) t.v[i] = v.v[i] + dpp_from<kRowShr + D * LC>(v.v[i]);
        if (D <= dist) v = t;
        scan_rows_of_16<D * 2, LC, VEC>(v, dist);
    }
}

// Segmented sum along a wavefront's entry lanes: v of mine and of the lanes in front of it down to number `from` (-1:
// all), which is the nearest one, at or in front of mine, whose sum starts afresh.  All 64 lanes call together.
template <int LC, int VEC>
__device__ __forceinline__ void scan_from(Vec<VEC>& v, int from)
{
    const int lane = lane_id();
    scan_rows_of_16<1, LC, VEC>(v, lane / LC - from);
    Vec<VEC> t;
#pragma unroll
    for (int i = 0; i < VEC; ++i) t.v[i] = v.v[i] + from_row_in_front<LC, false>(v.v[i]);
    if ((lane & 16) && from * LC < (lane & ~15)) v = t;
#pragma unroll
    for (int i = 0; i < VEC; ++i) t.v[i] = v.v[i] + from_row_in_front<LC, true>(v.v[i]);
    if (lane >= 32 && from * LC < 32) v = t;
}

// Rows that cross a tile's boundary: two of a tile at most, the one that comes in and the one that goes on.  Their sums
// are collected for kEdgeTiles tiles and then added into C together.
constexpr int kEdgeTiles = 32;
template <int WIDTH>
struct Edges {
    int32_t row[kEdgeTiles * 2];  // -1: none
    float sum[kEdgeTiles * 2][WIDTH];
};

// The sum of a run leaves the registers.  place: of the tile's edges, the row that comes in is row_lb.
template <int VEC, bool RAGGED, int WIDTH>
__device__ __forceinline__ void write_run(const SpmmArgs& a, Edges<WIDTH>& edges, int place, int32_t row_lb, int32_t end,
                                          uint32_t k, uint32_t k_lane, Vec<VEC> x)
{
    if (end >= 0) {
        store_vec<VEC>(a.C + (int64_t)end * a.N + k_lane, x);
    } else {
        const int32_t row = end & ~kOutside;
        if (row != row_lb) ++place;
        from_last_columns<VEC, RAGGED>(x, (int)(k - k_lane));
        edges.row[place] = row;
#pragma unroll
        for (int i = 0; i < VEC; ++i) edges.sum[place][k + i] = x.v[i];
    }
}

// Block-uniform, behind a barrier.
template <int WIDTH>
__device__ __forceinline__ void add_edges(const SpmmArgs& a, Edges<WIDTH>& edges, int n)
{
    for (int i = threadIdx.x; i < n * WIDTH; i += kBlock) {
        const int32_t row = edges.row[i / WIDTH];
        if (row >= 0 && i % WIDTH < a.N) unsafeAtomicAdd(a.C + (int64_t)row * a.N + i % WIDTH, edges.sum[i / WIDTH][i % WIDTH]);
    }
}

template <int E>
__device__ __forceinline__ void arrived(int32_t (&col)[E], float (&val)[E], int32_t& lo, int32_t& hi)
{
#pragma unroll
    for (int u = 0; u < E; ++u) asm volatile("" : "+v"(col[u]), "+v"(val[u]));
    asm volatile("" : "+v"(lo), "+v"(hi));
}

}  // namespace

template <int LC, int VEC, int E, bool OFF32, bool RAGGED>
__global__ __launch_bounds__(kBlock) void nnz_narrow_kernel(SpmmArgs a)
{
    constexpr int TILE = kBlock / LC * E;
    static_assert(E % 4 == 0, "a lane's entries come with 16-byte loads");
    __shared__ __align__(16) int32_t s_end[TILE];
    __shared__ float s_tail[kWavesPerBlock][LC * VEC];  // what a wavefront's last run has so far
    __shared__ int32_t s_any[kWavesPerBlock];           // whether a row ends in the wavefront's entries
    __shared__ int32_t s_last[2];
    __shared__ Edges<LC * VEC> s_edges;
    __shared__ int32_t s_tile_row[kTileRowBatch];

    const int32_t M = (int32_t)a.M;
    const int32_t nnz = a.rowptr[a.M];
    const TileDeal deal(((int64_t)nnz + TILE - 1) / TILE, blockIdx.x, gridDim.x);
    const int64_t my_tiles = deal.mine;
    if (my_tiles == 0) return;
    TileWalk ahead(deal);  // the tile that is fetched next

    const int tid = threadIdx.x;
    const int lane = tid % kWave, wave = tid / kWave;
    const int chunk = tid % LC;
    const int q0 = tid / LC * E;  // my first place in a tile
    const uint32_t k = chunk * VEC;
    const bool k_ok = k < (uint32_t)a.N;
    const uint32_t k_lane = k_ok ? lane_first_col<VEC, RAGGED>(k, (uint32_t)a.N) : 0;  // the VEC columns this lane holds
    const BRow<OFF32> Brow(a.B, a.N, k_lane);

    // (every lane clears the places that it reads, here and in every tile)
#pragma unroll
    for (int u = 0; u < E; u += 4) *reinterpret_cast<lds_i4*>(s_end + q0 + u) = lds_i4{kNoEnd, kNoEnd, kNoEnd, kNoEnd};

    if (tid < kEdgeTiles * 2) s_edges.row[tid] = -1;

    // registers that carry a tile in: a lane's entries and the bounds of one row
    int32_t nx_col[E], nx_lo, nx_hi;
    float nx_val[E];
    auto fetch_row = [&](int64_t r, int32_t& lo, int32_t& hi) {
        lo = a.rowptr[r < M ? r : M];
        hi = a.rowptr[r < M ? r + 1 : M];
    };
    auto fetch_tile = [&](int32_t row_lb) {  // the tile `ahead` stands at
        const int32_t start = (int32_t)(ahead.tile() * TILE) + q0;
#pragma unroll
        for (int u = 0; u < E; u += 4) {
            if (start + u + 4 <= nnz) {
                const native_i4 c = __builtin_nontemporal_load(reinterpret_cast<const native_i4*>(a.colidx + start + u));
                const native_f4 v = __builtin_nontemporal_load(reinterpret_cast<const native_f4*>(a.vals + start + u));
                nx_col[u] = c.x; nx_col[u + 1] = c.y; nx_col[u + 2] = c.z; nx_col[u + 3] = c.w;
                nx_val[u] = v.x; nx_val[u + 1] = v.y; nx_val[u + 2] = v.z; nx_val[u + 3] = v.w;
            } else {
#pragma unroll
                for (int i = u; i < u + 4; ++i) {
                    nx_col[i] = 0;
                    nx_val[i] = 0.0f;
                    if (start + i < nnz) {
                        nx_col[i] = load_stream(a.colidx + start + i);
                        nx_val[i] = load_stream(a.vals + start + i);
                    }
                }
            }
        }
        fetch_row((int64_t)row_lb + tid, nx_lo, nx_hi);
    };

    for (int64_t j0 = 0; j0 < my_tiles; j0 += kTileRowBatch) {
        find_tile_rows(a, deal, j0, TILE, s_tile_row);
        const int64_t j1 = j0 + kTileRowBatch < my_tiles ? j0 + kTileRowBatch : my_tiles;
        fetch_tile(s_tile_row[0]);

        for (int64_t j = j0; j < j1; ++j) {
            const int32_t tile_start = (int32_t)(ahead.tile() * TILE);
            ahead.next();
            const int32_t tile_end = nnz - tile_start < TILE ? nnz : tile_start + TILE;
            const int32_t row_lb = s_tile_row[j - j0];
            const int edge = (int)(j - j0) % kEdgeTiles * 2;

            // the rows of B (lanes without columns or behind the last entry read what exists; no sum of theirs is written)
            Vec<VEC> x[E];
            float val[E];
#pragma unroll
            for (int u = 0; u < E; ++u) {
                val[u] = nx_val[u];
                x[u] = load_vec<VEC>(Brow.at(nx_col[u]));
            }
            int32_t lo = nx_lo, hi = nx_hi;
            if (j + 1 < j1) fetch_tile(s_tile_row[j + 1 - j0]);

            // where the tile's rows end: a row per thread, and where that is not enough (long runs of rows without entries)
            // four per thread and round; every thread leaves in the same round
            auto mark = [&](int64_t r, int32_t lo, int32_t hi) {
                if (hi > lo && lo < tile_end) {
                    const bool outside = lo < tile_start || hi > tile_end;
                    s_end[(hi < tile_end ? hi : tile_end) - 1 - tile_start] = (int32_t)r | (outside ? kOutside : 0);
                }
            };
            mark((int64_t)row_lb + tid, lo, hi);
            if (tid == kBlock - 1) s_last[0] = hi;
            __syncthreads();
            if (s_last[0] < tile_end) {
                int64_t r = (int64_t)row_lb + kBlock + tid * 4;
                for (int round = 1;; ++round, r += kBlock * 4) {
                    int32_t p[5];
#pragma unroll
                    for (int i = 0; i < 5; ++i) p[i] = a.rowptr[r + i < M ? r + i : M];
#pragma unroll
                    for (int i = 0; i < 4; ++i) mark(r + i, p[i], p[i + 1]);
                    if (tid == kBlock - 1) s_last[round & 1] = p[4];
                    __syncthreads();
                    if (s_last[round & 1] >= tile_end) break;
                }
            }
            int32_t end[E];
#pragma unroll
            for (int u = 0; u < E; u += 4) {
                lds_i4* __restrict__ mine = reinterpret_cast<lds_i4*>(s_end + q0 + u);
                const lds_i4 t = *mine;
                end[u] = t.x; end[u + 1] = t.y; end[u + 2] = t.z; end[u + 3] = t.w;
                *mine = lds_i4{kNoEnd, kNoEnd, kNoEnd, kNoEnd};  // for the next tile
            }

            // Everything asked for is here before the first store: the next tile's rows of B are then asked for without a wait
            // for the stores of this one, which share the loads' counter (vmcnt).
            arrived(nx_col, nx_val, nx_lo, nx_hi);

            // my own entries: the run that ends first may have begun in a lane in front of mine, the runs behind it are
            // whole (unless their row goes on in another tile), and what is left goes on in the lanes behind
            Vec<VEC> run, first;
            int32_t first_end = kNoEnd;
            run.zero();
            first.zero();
#pragma unroll
            for (int u = 0; u < E; ++u) {
                run.fma(val[u], x[u]);
                if (end[u] != kNoEnd) {
                    if (first_end == kNoEnd) {
                        first_end = end[u];
                        first = run;
                    } else if (k_ok) {
                        write_run<VEC, RAGGED>(a, s_edges, edge, row_lb, end[u], k, k_lane, run);
                    }
                    run.zero();
                }
            }
            const unsigned long long ends = __ballot(first_end != kNoEnd);  // the LC lanes of an entry lane alike
            const unsigned long long upto = ends & (~0ull >> (kWave - 1 - lane));
            scan_from<LC, VEC>(run, upto ? (kWave - 1 - __builtin_clzll(upto)) / LC : -1);
#pragma unroll
            for (int i = 0; i < VEC; ++i) first.v[i] += from_lane_in_front<LC>(run.v[i]);
            // the wavefront's first run may have begun in the wavefronts in front
            const bool waits = first_end != kNoEnd && (ends & ((1ull << (lane - chunk)) - 1ull)) == 0;
            if (first_end != kNoEnd && !waits && k_ok) write_run<VEC, RAGGED>(a, s_edges, edge, row_lb, first_end, k, k_lane, first);
            if (lane >= kWave - LC) {
#pragma unroll
                for (int i = 0; i < VEC; ++i) s_tail[wave][chunk * VEC + i] = run.v[i];
                s_any[wave] = ends != 0;
            }
            __syncthreads();
            if (waits) {
                for (int w = wave - 1; w >= 0; --w) {
#pragma unroll
                    for (int i = 0; i < VEC; ++i) first.v[i] += s_tail[w][chunk * VEC + i];
                    if (s_any[w]) break;
                }
                if (k_ok) write_run<VEC, RAGGED>(a, s_edges, edge, row_lb, first_end, k, k_lane, first);
            }
            if (edge == kEdgeTiles * 2 - 2 || j + 1 == j1) {
                __syncthreads();
                add_edges(a, s_edges, edge + 2);
                __syncthreads();
                if (tid < kEdgeTiles * 2) s_edges.row[tid] = -1;
            }
        }
    }
}

namespace {

template <void (*KERNEL)(SpmmArgs)>
struct Instance {
    static int per_cu()
    {
        static const int n = resident_per_cu(KERNEL, 0);
        return n;
    }
    static void launch(int grid, const SpmmArgs& a, hipStream_t s)
    {
        hipLaunchKernelGGL(KERNEL, dim3(grid), dim3(kBlock), 0, s, a);
    }
};

// Calls f with the instance for a problem: f(instance, positions per tile).
template <int LC, int VEC, int E, bool RAGGED, typename F>
auto with_form(const SpmmArgs& a, F&& f)
{
    constexpr int TILE = kBlock / LC * E;
    return offsets_fit_32(a) ? f(Instance<nnz_narrow_kernel<LC, VEC, E, true, RAGGED>>{}, TILE)
                             : f(Instance<nnz_narrow_kernel<LC, VEC, E, false, RAGGED>>{}, TILE);
}

template <typename F>
auto with_kernel(const SpmmArgs& a, F&& f)
{
    switch (a.N) {
        case 1: return with_form<1, 1, 4, false>(a, f);
        case 2: return with_form<1, 2, 4, false>(a, f);
        case 3: return with_form<2, 2, 8, true>(a, f);
        case 4: return with_form<1, 4, 4, false>(a, f);
        case 8: return with_form<2, 4, 8, false>(a, f);
        case 5: case 6: case 7: return with_form<2, 4, 8, true>(a, f);
        case 12: case 16: return with_form<4, 4, 8, false>(a, f);
        default: return with_form<4, 4, 8, true>(a, f);
    }
}

}  // namespace

NnzPlan plan_nnz_narrow(const SpmmArgs& a)
{
    return with_kernel(a, [&](auto, int tile) {
        NnzPlan p;
        p.tile = tile;
        p.merge = true;
        p.merge_log2 = __builtin_ctz(tile);
        p.lc = 0;
        p.share = a.group;
        return p;
    });
}

hipError_t launch_nnz_narrow(const SpmmArgs& a, int compute_units, int64_t nnz_hint, hipStream_t s)
{
    if (a.N < 1 || a.N > kNarrowColumns) return hipErrorInvalidValue;
    return with_kernel(a, [&](auto instance, int tile) {
        instance.launch(persistent_grid(instance.per_cu(), compute_units, nnz_hint, tile), a, s);
        return hipGetLastError();
    });
}

}  // namespace sgap
