// Shared declarations of the SpMM kernels: argument block, per-lane column
// vectors (the paper's coarsening factor c = VEC dense columns per lane) and
// the host-side launch entry points of each kernel family.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sgap_tile_deal.hpp"

namespace sgap {

constexpr int kWave = 64;          // wavefront size on gfx950
constexpr int kBlock = 256;        // threads per workgroup (4 waves)
constexpr int kWavesPerBlock = kBlock / kWave;
// Up to so many columns the nnz-balanced schedule's parallel strategy is sgap_nnz_narrow.hip.  Beyond, where a row of B takes
// more than four lanes, the entries of a lane have not been measured.  R-MAT with 2^21 rows, N = 16, G = 16: 1,112 us with an
// entry per lane, 614 with eight.
constexpr int kNarrowColumns = 16;

struct SpmmArgs {
    int64_t M, K, N;
    const int32_t* __restrict__ rowptr;
    const int32_t* __restrict__ colidx;
    const float* __restrict__ vals;
    const float* __restrict__ B;
    float* __restrict__ C;
    int log2_group;   // log2(group_size)
    int group;        // group_size
};

// A third-order tensor as compressed sparse fibers (first index dense) and the dense operands of MTTKRP.
struct MttkrpArgs {
    int64_t I, K, L, J;
    const int32_t* __restrict__ fptr;
    const int32_t* __restrict__ fidx;
    const int32_t* __restrict__ eptr;
    const int32_t* __restrict__ eidx;
    const float* __restrict__ vals;
    const float* __restrict__ X1;
    const float* __restrict__ X2;
    float* __restrict__ Y;
};

// Rows another kernel produces: when *count <= max_rows, rows of at least
// min_len stored entries are neither computed nor written by the kernel that
// is handed this.  count = nullptr: no row is left out.
struct RowSkip {
    const uint32_t* __restrict__ count;
    uint32_t max_rows;
    int32_t min_len;
};

// How the (row block x column tile) work items of a row-split launch are
// laid over the grid.  The 8 accelerator dies (XCDs) of the chip each have a
// private L2 and receive workgroups round-robin (workgroup b runs on XCD
// b % 8), so item = (b % 8) * items_per_xcd + b / 8 hands every XCD one
// contiguous run of the column-tile-major item order: one column tile and a
// contiguous range of rows at a time, which keeps the rows of B it gathers
// resident in its own L2.
struct TileSched {
    int64_t row_blocks;     // number of row blocks
    int64_t items;          // row_blocks * col_tiles
    int64_t items_per_xcd;  // ceil(items / xcds)
    int32_t col_tiles;      // number of column tiles
    int32_t tile_cols;      // columns per tile (multiple of VEC)
    int32_t xcds;           // 8, or 1 to switch the remapping off
};

// The workgroups of a row-split launch.  The first `finders` look for the rows of at least share_from stored entries and
// produce them with all their lanes; those from number walk_from on walk the work items and pass over such rows.
struct RowSplitGrid {
    int32_t share_from;  // 0x7fffffff, which no row reaches, exactly where nobody looks for such rows
    int32_t finders;
    int32_t log2_team;   // 2^log2_team of them look through the same rows and take the long ones in turn
    FinderDeal deal;     // which rows a team looks through
    int32_t walk_from;   // = finders; 0 on a persistent grid, whose workgroups look for rows first and then walk
    uint32_t grid;
};

template <int VEC>
struct Vec {
    float v[VEC];
    __device__ __forceinline__ void zero()
    {
#pragma unroll
        for (int i = 0; i < VEC; ++i) v[i] = 0.0f;
    }
    __device__ __forceinline__ void fma(float a, const Vec& b)
    {
#pragma unroll
        for (int i = 0; i < VEC; ++i) v[i] = __builtin_fmaf(a, b.v[i], v[i]);
    }
};

// Two and four floats as one access that asks for no more than 4-byte alignment: the vector memory path of this
// chip takes such addresses, so that the columns per lane need not divide the row length (N = 37: ten 16-byte loads
// per row of B instead of thirty-seven 4-byte ones).
typedef float native_f4 __attribute__((ext_vector_type(4), aligned(4)));
typedef float native_f2 __attribute__((ext_vector_type(2), aligned(4)));

// VEC consecutive floats (any 4-byte aligned address).
template <int VEC>
__device__ __forceinline__ Vec<VEC> load_vec(const float* __restrict__ p)
{
    Vec<VEC> r;
    if constexpr (VEC == 4) {
        const native_f4 t = *reinterpret_cast<const native_f4*>(p);
        r.v[0] = t.x; r.v[1] = t.y; r.v[2] = t.z; r.v[3] = t.w;
    } else if constexpr (VEC == 2) {
        const native_f2 t = *reinterpret_cast<const native_f2*>(p);
        r.v[0] = t.x; r.v[1] = t.y;
    } else {
        r.v[0] = *p;
    }
    return r;
}

template <int VEC>
__device__ __forceinline__ void store_vec(float* __restrict__ p, const Vec<VEC>& r)
{
    if constexpr (VEC == 4) {
        native_f4 t = {r.v[0], r.v[1], r.v[2], r.v[3]};
        *reinterpret_cast<native_f4*>(p) = t;
    } else if constexpr (VEC == 2) {
        native_f2 t = {r.v[0], r.v[1]};
        *reinterpret_cast<native_f2*>(p) = t;
    } else {
        *p = r.v[0];
    }
}

// Streaming accesses: data touched once (A going in, C going out) should not
// displace the rows of B that the L2 keeps for reuse.
template <typename T>
__device__ __forceinline__ T load_stream(const T* __restrict__ p)
{
    return __builtin_nontemporal_load(p);
}

template <int VEC>
__device__ __forceinline__ void store_vec_stream(float* __restrict__ p, const Vec<VEC>& r)
{
    if constexpr (VEC == 4) {
        native_f4 t = {r.v[0], r.v[1], r.v[2], r.v[3]};
        __builtin_nontemporal_store(t, reinterpret_cast<native_f4*>(p));
    } else if constexpr (VEC == 2) {
        native_f2 t = {r.v[0], r.v[1]};
        __builtin_nontemporal_store(t, reinterpret_cast<native_f2*>(p));
    } else {
        __builtin_nontemporal_store(r.v[0], p);
    }
}

// The columns of a lane whose chunk starts at column k < N: k .. k + VEC, or, where fewer than VEC columns are left,
// the last VEC columns of the row (N >= VEC): no lane reads past a row, and the columns it shares with the lane in
// front of it come out the same in both, so that a plain store of all VEC of them is right whichever lands last.
// Where sums are ADDED somewhere the lane first brings its own columns to the front (from_last_columns).
// RAGGED = false: N is known to be a multiple of VEC (kernels whose registers are all spoken for come in both forms).
template <int VEC, bool RAGGED = true>
__device__ __forceinline__ int64_t lane_first_col(int64_t k, int64_t N)
{
    if constexpr (VEC == 1 || !RAGGED) return k;
    else return k + VEC <= N ? k : N - VEC;
}
template <int VEC, bool RAGGED = true>
__device__ __forceinline__ uint32_t lane_first_col(uint32_t k, uint32_t N)
{
    if constexpr (VEC == 1 || !RAGGED) return k;
    else return k + VEC <= N ? k : N - VEC;
}

// Columns of this lane's chunk that the lane in front of it holds as well: k - lane_first_col(k, N), 0 .. VEC-1.
// Afterwards v[i] belongs to column k + i; what lies past the end of the row is zero.
template <int VEC, bool RAGGED = true>
__device__ __forceinline__ void from_last_columns(Vec<VEC>& x, int shared)
{
    if constexpr (VEC > 1 && RAGGED) {
        if (shared <= 0) return;
        Vec<VEC> y;
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
            y.v[i] = 0.0f;
#pragma unroll
            for (int j = i + 1; j < VEC; ++j)
                if (j - i == shared) y.v[i] = x.v[j];
        }
        x = y;
    }
}

// Address of B[col, k..): with OFF32 every byte offset into B fits 32 bits and
// col, N*4 fit 24 bits, so one 24-bit multiply-add forms the offset and the
// load uses the uniform base pointer plus a 32-bit lane offset.
template <bool OFF32>
struct BRow {
    const char* __restrict__ base;  // B as bytes
    uint32_t row_bytes;             // N * 4          (OFF32)
    uint32_t k_bytes;               // k * 4          (OFF32)
    int64_t N;                      // row stride     (!OFF32)
    int64_t k;
    __device__ __forceinline__ BRow(const float* B, int64_t n, int64_t k_)
        : base(reinterpret_cast<const char*>(B)), row_bytes((uint32_t)(n * 4)), k_bytes((uint32_t)(k_ * 4)), N(n), k(k_)
    {
    }
    __device__ __forceinline__ const float* at(int32_t col) const
    {
        if constexpr (OFF32) {
            const uint32_t off = __umul24((uint32_t)col, row_bytes) + k_bytes;
            return reinterpret_cast<const float*>(base + off);
        } else {
            return reinterpret_cast<const float*>(base) + ((int64_t)col * N + k);
        }
    }
};

// Where the operands end whose rows are found by byte offsets of 32 bits.  The 32 bytes behind it are room for a load at
// an offset that lies past every operand (MaskedRows).
constexpr int64_t kOffsets32End = 0xffffffe0LL;

// Both factors of a row's offset have 24 bits then.
inline bool offsets_fit_32(int64_t rows, int64_t columns)
{
    return rows <= (1 << 24) && columns * 4 < (1 << 24) && rows * columns * 4 <= kOffsets32End;
}

inline bool offsets_fit_32(const SpmmArgs& a) { return offsets_fit_32(a.K, a.N); }

// How an nnz-balanced kernel cuts the stored entries: tile = positions per LDS
// tile, merge = tile mode of the merge rule, merge_log2 = log2 of the merge
// block the zeroing pass must assume (tile in tile mode, group otherwise),
// lc = chunk lanes per stored entry the kernel is to run with (the plan may
// narrow the layout it was asked about so that the accumulators fit the LDS).
// share = consecutive entries a lane walks (the serial strategy: the group size, or less where the tile has no more for
// a lane).
struct NnzPlan {
    int tile;
    bool merge;
    int merge_log2;
    int lc;
    int share;
};
NnzPlan plan_nnz_serial(int group, int lc, int vec, int64_t nnz_hint, int compute_units, int forced_tile);
NnzPlan plan_nnz_parallel(int group, int lc, int vec);
NnzPlan plan_nnz_narrow(const SpmmArgs& a);  // parallel, N <= kNarrowColumns
// g = lanes per row of a whole-group reduction (1: no rows are shared), passes = passes of a group over its columns,
// resident = workgroups that fit the chip at once for a persistent launch (0: a workgroup per item).
RowSplitGrid plan_row_split_grid(int g, int passes, int64_t M, int64_t items, int xcds, int compute_units,
                                 int64_t nnz_hint, int resident);
// ---- host-side launchers, one per kernel family (defined in the .hip files)
// lc = chunk lanes per row (power of two), vec = columns per lane (1, 2, 4).
// g = lanes per row (1 for the serial strategy), rows_per_slot = rows a group
// works through per work item (consecutive rows, or every slots-th row of the
// block when `interleave` is set), tile_cols = columns per work item, xcds = 8
// or 1, compute_units = CUs of the device; persistent = launch only as many
// workgroups as fit the chip and let each walk several items (else one
// workgroup per item); block = threads per workgroup (128, 256 or 512).
// mean_row: stored entries per row as far as the host knows.
hipError_t launch_row_split(const SpmmArgs& a, int g, int lc, int vec, int rows_per_slot, bool interleave,
                            int tile_cols, int xcds, int compute_units, bool persistent, int block, int64_t nnz_hint,
                            double mean_row,
                            hipStream_t s);
// serial strategy, four consecutive rows together (sgap_row_quads.hip); vec must be 4.  row_quads_apply: whether that is
// the kernel for so many rows of mean_row stored entries and lc lanes per column tile
bool row_quads_apply(int64_t M, int lc, int64_t tile_cols, double mean_row, int compute_units);
hipError_t launch_row_quads(const SpmmArgs& a, int lc, int tile_cols, int xcds, hipStream_t s);
// whether the parallel strategy of SDDMM takes a matrix in host memory by four rows together (g lanes per entry)
bool sddmm_by_quads(int64_t M, int64_t K, int64_t J, int g, int64_t nnz_hint, const int32_t* rowptr, const int32_t* colidx);
// parallel strategy, blocks of rows shared by teams of lanes (sgap_flat_shared.hip), where groups would have so many members;
// never without a count of the entries
bool flat_shared_rows_apply(int64_t K, int64_t N, int members, double mean_row, int64_t nnz_hint);
hipError_t launch_flat_shared_rows(const SpmmArgs& a, int xcds, int compute_units, int64_t nnz_hint, hipStream_t s);
// serial strategy, short rows (sgap_flat_rows.hip).  flat_rows_apply: whether that is the kernel for so many rows of
// mean_row stored entries, `group` to a lane; never without a count of them
bool flat_rows_apply(int64_t K, int64_t N, int group, double mean_row, int64_t nnz_hint);
hipError_t launch_flat_rows(const SpmmArgs& a, int vec, int xcds, int compute_units, int64_t nnz_hint, hipStream_t s);
// the same with g lanes per row reducing in sub-groups of r < g lanes whose sums
// are merged with atomics; C must have been zeroed (launch_nnz_zero_rows, -1)
hipError_t launch_row_split_partial(const SpmmArgs& a, int g, int r, int lc, int vec, int rows_per_slot,
                                    int tile_cols, int xcds, int compute_units, bool persistent, int block,
                                    hipStream_t s);
// the row-split launch with rows of at least min_len stored entries taken out and
// produced window by window of about window_bytes of B (sgap_panels.hip; window_asked: the caller names that size); vec must be 4;
// wave_vec > 0: the other rows by launch_wave_rows with that many columns per lane and rows_per_slot rows per wavefront;
// workspace = device memory of spmm_panels_workspace_bytes(K, N, window_bytes, cap) bytes
// for a list of up to cap long rows (more long rows than that: the row-split kernel takes every row)
hipError_t launch_row_split_panels(const SpmmArgs& a, int g, int lc, int vec, int rows_per_slot, bool interleave,
                                   int tile_cols, int xcds, int compute_units, bool persistent, int block,
                                   int wave_vec, int32_t min_len, int64_t window_bytes, bool window_asked,
                                   void* workspace, int64_t cap, hipStream_t s);
int64_t spmm_panels_workspace_bytes(int64_t K, int64_t N, int64_t window_bytes, int64_t cap);
int64_t sddmm_panels_workspace_bytes(int64_t K, int64_t J, int64_t window_bytes, int64_t cap);
// row-split, serial strategy, one wavefront per rows_per_wave consecutive rows and 64 * vec columns
// (sgap_wave_rows.hip); skip = rows another kernel produces, or nullptr
hipError_t launch_wave_rows(const SpmmArgs& a, int vec, int rows_per_wave, int xcds, const RowSkip* skip,
                            hipStream_t s);
// zero the rows of C that receive atomic adds under a merge block of
// 2^merge_log2 positions, and the rows without entries; merge_log2 = -1: all rows
hipError_t launch_nnz_zero_rows(const SpmmArgs& a, int vec, int merge_log2, hipStream_t s);
// compute_units sizes the persistent grid; nnz_hint (-1 = unknown) caps it.
hipError_t launch_nnz_parallel(const SpmmArgs& a, int lc, int vec, const NnzPlan& plan, int compute_units,
                               int64_t nnz_hint, hipStream_t s);
// the same for N <= kNarrowColumns (sgap_nnz_narrow.hip)
hipError_t launch_nnz_narrow(const SpmmArgs& a, int compute_units, int64_t nnz_hint, hipStream_t s);
// the serial strategy by teams of lanes that go each at its own pace (sgap_nnz_flat.hip); nnz_flat_tile: the tile, 0 where
// that is not the kernel
int nnz_flat_tile(int64_t N, int group, double mean_row, int64_t nnz_hint, int compute_units);
hipError_t launch_nnz_flat(const SpmmArgs& a, int tile, int compute_units, int64_t nnz_hint, hipStream_t s);
hipError_t launch_nnz_serial(const SpmmArgs& a, int lc, int vec, const NnzPlan& plan, int compute_units,
                             int64_t nnz_hint, hipStream_t s);
// r = members per reducing sub-group (r = g: the whole group)
hipError_t launch_debug_group_reduce(const float* in, float* out, int g, int r, int lc, hipStream_t s);
// Sampled dense-dense product on A's pattern: a carries M, K, N = J, rowptr,
// colidx, vals and B = X2T (K x J); X1 is M x J; out has one value per stored
// entry.  g lanes per entry (per_lane = 0) or one lane per per_lane entries.
// row_cache lets the parallel strategy keep rows of X1 in LDS where the shape allows.
hipError_t launch_sddmm(const SpmmArgs& a, const float* X1, float* out, int g, int per_lane, int vec, bool row_cache,
                        int compute_units, int64_t nnz_hint, hipStream_t stream);
// the same with the stored entries of rows of at least min_len entries produced
// window by window of X2T (sgap_panels.hip) and all others by the plain kernel;
// vec must be 4 and 32 <= J <= 256
hipError_t launch_sddmm_panels(const SpmmArgs& a, const float* X1, float* out, int g, int per_lane, int xcds,
                               int compute_units, int64_t nnz_hint, int32_t min_len, int64_t window_bytes, bool window_asked,
                               void* workspace, int64_t cap, hipStream_t stream);
// the plain SDDMM kernel on the rows of at least from_len entries that are not described by `skip` (on every row if
// there are more of those than skip.max_rows)
hipError_t launch_sddmm_rest(const SpmmArgs& a, const float* X1, float* out, int g, int per_lane, int compute_units,
                             int64_t nnz_hint, const RowSkip& skip, int32_t from_len, hipStream_t stream);
// MTTKRP on compressed sparse fibers with slices as the unit of work: g lanes per slice (1 for the serial strategy),
// rows_per_slot slices per group (consecutive, or interleaved with the other groups' slices), lc chunk lanes of vec columns each.
hipError_t launch_mttkrp(const MttkrpArgs& a, int g, int rows_per_slot, bool interleave, int lc, int vec, int xcds, hipStream_t s);
// The parallel strategy by blocks of slices that teams of lanes share (sgap_mttkrp_fibers.hip), and whether that is the
// kernel (nnz_hint: -1 where there is no count).
bool mttkrp_fibers_apply(int64_t I, int64_t J, int group, int64_t nnz_hint);
hipError_t launch_mttkrp_fibers(const MttkrpArgs& a, int vec, int xcds, int compute_units, int64_t nnz_hint, hipStream_t s);
hipError_t launch_debug_group_seg_reduce(const float* in, const int32_t* span, float* out, int g, int lc,
                                         hipStream_t s);
// MTTKRP with the stored entries as the unit of work (sgap_mttkrp_nnz.hip): g = lanes per segment group
// (parallel) or entries per lane (serial); Y must hold zeros.
hipError_t launch_mttkrp_nnz(const MttkrpArgs& a, int g, bool parallel, int lc, int vec, int compute_units,
                             int64_t nnz_hint, hipStream_t s);
// its serial strategy: by teams of lanes at their own pace (sgap_mttkrp_fibers.hip), or, few entries of few columns
// (sgap_mttkrp_serial.hip), by lanes with an even share each
hipError_t launch_mttkrp_tiles(const MttkrpArgs& a, int vec, int compute_units, int64_t nnz_hint, hipStream_t s);
bool mttkrp_serial_applies(int64_t J, int64_t nnz_hint);
hipError_t launch_mttkrp_serial(const MttkrpArgs& a, int lc, int vec, int compute_units, int64_t nnz_hint, hipStream_t s);
// Rows grouped by a coarse key (sgap_reorder.hip): the permutation and the permuted copy of the matrix.
int64_t reorder_workspace_bytes(int64_t M);
hipError_t launch_reorder_rows(int64_t M, int64_t K, const int32_t* rowptr, const int32_t* colidx, const float* vals,
                               bool by_length, int32_t* perm, int32_t* rowptr_out, int32_t* colidx_out,
                               float* vals_out, void* workspace, int compute_units, hipStream_t s);

// Columns per lane for rows of N dense columns: four wherever a row has four, since a 16-byte access costs the
// vector memory path as much as a 4-byte one and needs no more than 4-byte alignment.
inline int lane_columns(int64_t N) { return N >= 4 ? 4 : N >= 2 ? 2 : 1; }

// Generic (g, lc, vec) -> template instance dispatch.  F is a functor with
//   template <int G, int LC, int VEC> void operator()() const
// Rows of one column take one lane, rows of two or three at most two (lane_columns), so the narrow instances exist
// for those lane counts only.
template <int G, int LC, typename F>
inline bool dispatch_vec(int vec, F&& f)
{
    switch (vec) {
        case 4: f.template operator()<G, LC, 4>(); return true;
        case 2: if constexpr (LC <= 2) { f.template operator()<G, LC, 2>(); return true; } break;
        case 1: if constexpr (LC == 1) { f.template operator()<G, LC, 1>(); return true; } break;
        default: break;
    }
    return false;
}

template <int G, typename F>
inline bool dispatch_lc(int lc, int vec, F&& f)
{
    switch (lc) {
        case 1: if constexpr (G * 1 <= 64) return dispatch_vec<G, 1>(vec, f); break;
        case 2: if constexpr (G * 2 <= 64) return dispatch_vec<G, 2>(vec, f); break;
        case 4: if constexpr (G * 4 <= 64) return dispatch_vec<G, 4>(vec, f); break;
        case 8: if constexpr (G * 8 <= 64) return dispatch_vec<G, 8>(vec, f); break;
        case 16: if constexpr (G * 16 <= 64) return dispatch_vec<G, 16>(vec, f); break;
        case 32: if constexpr (G * 32 <= 64) return dispatch_vec<G, 32>(vec, f); break;
        case 64: if constexpr (G * 64 <= 64) return dispatch_vec<G, 64>(vec, f); break;
        default: break;
    }
    return false;
}

template <typename F>
inline bool dispatch_group(int g, int lc, int vec, F&& f)
{
    switch (g) {
        case 1: return dispatch_lc<1>(lc, vec, f);
        case 2: return dispatch_lc<2>(lc, vec, f);
        case 4: return dispatch_lc<4>(lc, vec, f);
        case 8: return dispatch_lc<8>(lc, vec, f);
        case 16: return dispatch_lc<16>(lc, vec, f);
        case 32: return dispatch_lc<32>(lc, vec, f);
        case 64: return dispatch_lc<64>(lc, vec, f);
        default: return false;
    }
}

}  // namespace sgap
