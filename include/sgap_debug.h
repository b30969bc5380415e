/*
 * sgap_debug.h - test and measurement scaffolding of the MI355X CSR SpMM
 * library: exported by the same shared library as sgap.h's calls, but not
 * part of the interface an application programs against.  Used by the parity
 * tests (device self-checks of the cross-lane primitives, host-side pieces of
 * the schedules) and by the benchmark (event timing of the library's own
 * launches, a streaming copy that the hardware counters are calibrated on).
 * Conventions as in sgap.h.
 */
#ifndef SGAP_DEBUG_H
#define SGAP_DEBUG_H

#include <stdint.h>

#include "sgap.h"

#ifdef __cplusplus
extern "C" {
#endif

/*
 * Timing hooks for benchmarks.  While enabled, every compute call (SpMM,
 * SDDMM, TTM, MTTKRP) brackets ALL the kernels it enqueues (the row-zeroing
 * pass and the preparation of the window path included) with a pair of HIP
 * events on the call's stream.  sgap_profile_collect waits for those events,
 * adds their elapsed times in milliseconds into *total_ms, their number into
 * *count, and forgets them.  Not thread-safe; host pointers.
 */
int sgap_profile_enable(int on);
int sgap_profile_collect(double* total_ms, int* count);

/*
 * Device self-checks of the two cross-lane primitives behind the strategies
 * (the paper's macro instructions atomicAddGroup<T,G> and
 * segReduceGroup<T,G>, Section 5.3), one wavefront each.  `lanes_per_row`
 * (1..64/group_size, power of two) is the lane stride between neighbouring
 * members of a group.
 *   sgap_debug_group_reduce: in fp32[64] device -> out fp32[64] device; the
 *     first lane of every group receives the sum of its group's inputs, other
 *     lanes receive 0.
 *   sgap_debug_group_seg_reduce: in fp32[64], span int32[64] device (span[l] =
 *     how many following members of lane l's group continue lane l's run,
 *     0..group_size-1) -> out[l] = in[l] + the next span[l] members' inputs.
 *   sgap_debug_group_partial_reduce: the same for sub-groups of reduce_size
 *     members (power of two <= group_size): the first lane of every sub-group
 *     receives the sub-group's sum, other lanes 0.
 */
int sgap_debug_group_reduce(const float* in, float* out, int group_size,
                            int lanes_per_row, void* stream);
int sgap_debug_group_partial_reduce(const float* in, float* out, int group_size,
                                    int reduce_size, int lanes_per_row, void* stream);
int sgap_debug_group_seg_reduce(const float* in, const int32_t* span, float* out,
                                int group_size, int lanes_per_row, void* stream);

/*
 * Host-side pieces of the schedules, exported for tests; no GPU
 * is touched.
 *   sgap_debug_tile_deal: which tiles of stored entries workgroup `block` of a
 *     persistent grid of `grid` workgroups takes when the matrix has `tiles`
 *     tiles (chunks of neighbouring tiles per die).  Writes up to `capacity`
 *     tile numbers, ascending, into out_tiles (host) and returns how many
 *     tiles the workgroup takes, or -1 on bad arguments.
 *   sgap_debug_plan_nnz_serial: tile size (stored entries), whether a
 *     tile's partial sums are merged on chip, and the chunk lanes per stored
 *     entry the kernel runs with (lanes_per_row, or fewer where the on-chip
 *     accumulators of a small group would not fit otherwise), for the serial
 *     strategy with lanes_per_row chunk lanes of cols_per_lane columns each on
 *     a chip of compute_units; forced_tile as sgap_config.nnz_tile.  Host
 *     pointers; lanes_used may be null.
 *   sgap_debug_plan_row_split: the grid of a row-split launch with
 *     lanes_per_row lanes per row and `passes` passes over its columns, for M
 *     rows in `items` work items: the first `finders` of `grid` workgroups
 *     look for the rows of at least share_from stored entries and produce them
 *     whole, `team` of them looking through the same rows; the workgroups from
 *     walk_from on walk the items and leave such rows out.  resident: workgroups that the chip holds at once, for a
 *     persistent grid (0: a workgroup per item).  Host pointers.
 *   sgap_debug_finder_rows: the rows of M that team number `team` of `teams`
 *     looks through.  Writes up to `capacity` of them into out_rows
 *     (host) and returns how many there are, or -1 on bad arguments.
 *   sgap_debug_plan_windows: the form that long rows by column windows take
 *     (SpMM, or SDDMM with N for J) for a list of `rows` rows that hold
 *     `entries` of nnz stored entries, the longest `longest`; apart of them,
 *     at most worst of one row, are what windows in LDS would not serve.
 *     window_kb and max_long_rows as in sgap_config.  *in_lds 1: windows in LDS
 *     of `window` columns, the rows in `groups` groups, `shares` shares of the
 *     columns per die; 0: gathers (then those are 0).  The clocks that the
 *     library expects of both (0: the one in LDS does not come into question).
 *     The device decides by the same functions; 32-bit word 19 of the
 *     workspace says what it decided.
 *   sgap_debug_row_quads: 1 if the row-split schedule takes M rows of nnz_hint
 *     stored entries by four neighbouring rows together, 0 if not, -1 on bad
 *     arguments (config: a host sgap_config; long_row_min and wave_rows come
 *     first where they apply).
 *   sgap_debug_spmm_teams, sgap_debug_mttkrp_teams: 1 if teams of lanes that go
 *     each at its own pace take such a call, 0 if another kernel does, -1 on
 *     bad arguments (config: a host sgap_config; long_row_min, wave_rows and,
 *     for MTTKRP, SGAP_TUNE_ROWS_PER_GROUP come first where they apply).
 *   sgap_debug_sddmm_quads: 1 if sgap_sddmm_csr with the parallel strategy
 *     takes the matrix by four neighbouring rows together, 0 if entry by
 *     entry, -1 on bad arguments (rowptr and colidx in host memory; the device
 *     looks at the same rows of its own).
 */
int64_t sgap_debug_tile_deal(int64_t tiles, int grid, int block, int64_t* out_tiles, int64_t capacity);
int sgap_debug_plan_nnz_serial(int group_size, int lanes_per_row, int cols_per_lane, int64_t nnz_hint,
                               int compute_units, int forced_tile, int* tile, int* merge_on_chip,
                               int* lanes_used);
int sgap_debug_plan_row_split(int lanes_per_row, int passes, int64_t M, int64_t items, int dies, int compute_units,
                              int64_t nnz_hint, int resident, int64_t* share_from, int64_t* finders,
                              int64_t* team, int64_t* walk_from, int64_t* grid);
int64_t sgap_debug_finder_rows(int64_t M, int teams, int team, int64_t* out_rows, int64_t capacity);
int sgap_debug_plan_windows(int sddmm, int64_t K, int64_t N, int64_t rows, int64_t entries, int64_t longest,
                            int64_t nnz, int64_t apart, int64_t worst, int window_kb, int max_long_rows,
                            int compute_units, int* in_lds, int* groups, int* shares, int* window,
                            double* lds_clocks, double* gather_clocks);
int sgap_debug_row_quads(int64_t M, int64_t N, int64_t nnz_hint, const sgap_config* config, int compute_units);
int sgap_debug_spmm_teams(int64_t M, int64_t K, int64_t N, int64_t nnz_hint, const sgap_config* config, int compute_units);
int sgap_debug_mttkrp_teams(int64_t I, int64_t J, int group_size, int strategy, int schedule, int64_t nnz_hint);
int sgap_debug_sddmm_quads(int64_t M, int64_t K, int64_t J, int group_size, int64_t nnz_hint, const int32_t* rowptr,
                           const int32_t* colidx);

/*
 * Streaming kernels over n fp32 elements (16-byte aligned device buffers):
 * what the memory system delivers to a kernel that does nothing but stream,
 * reported next to the roofline fractions, and what the hardware traffic
 * counters are calibrated on.
 *   mode 0  copy src -> dst (sgap_copy_f32 is this)
 *   mode 1  read src only; dst points to one float that is (in practice
 *           never) written, so that the reads cannot be optimised away
 *   mode 2  write dst only (the value 1.0f); src is ignored
 */
int sgap_stream_f32(const float* src, float* dst, int64_t n, int mode, void* stream);
int sgap_copy_f32(const float* src, float* dst, int64_t n, void* stream);

#ifdef __cplusplus
}
#endif
#endif /* SGAP_DEBUG_H */
