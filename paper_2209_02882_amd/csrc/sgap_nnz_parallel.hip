// Nnz-balanced schedule: the row-zeroing pass, the plan (tile size, merge mode)
// of the parallel strategy and the dispatch of its launch to the translation
// units that hold the kernel instances.
#include "sgap_common.hpp"
#include "sgap_nnz_common.hpp"

namespace sgap {

// Rows that will receive global atomic adds (their positions straddle an
// aligned merge block of 2^merge_log2 positions) and rows without stored
// entries are set to +0; merge_log2 < 0: every row is.
// A lane looks at one row (the row pointers are read once, in order), and the wavefront then clears the rows that
// want it, lcz lanes to a row.  A wavefront has rows_per_wave rows: 64, or eight where that leaves the chip idle.  Bound by
// the writes: R-MAT with 2^21 rows of which 922,500 have no entries, N = 32: 33 us
// with eight lanes looking at every row.
template <int VEC>
__global__ __launch_bounds__(kBlock) void zero_rows_kernel(SpmmArgs a, int log2_lcz, int merge_log2, int rows_per_wave)
{
    __shared__ uint8_t s_list[kWavesPerBlock][kWave];
    const int lane = threadIdx.x % kWave;
    uint8_t* list = s_list[threadIdx.x / kWave];
    const int64_t row0 = ((int64_t)blockIdx.x * kWavesPerBlock + threadIdx.x / kWave) * rows_per_wave;
    const int64_t row = row0 + lane;
    bool wanted = lane < rows_per_wave && row < a.M;
    if (wanted && merge_log2 >= 0) {
        const int32_t p_begin = a.rowptr[row];
        const int32_t p_end = a.rowptr[row + 1];
        wanted = !(p_end > p_begin && (p_begin >> merge_log2) == ((p_end - 1) >> merge_log2));
    }
    const unsigned long long mask = __ballot(wanted);
    if (mask == 0) return;
    if (wanted) list[__popcll(mask & ((1ull << lane) - 1ull))] = (uint8_t)lane;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const int n = __popcll(mask);
    const int chunk = lane & ((1 << log2_lcz) - 1);
    Vec<VEC> z;
    z.zero();
    for (int i = lane >> log2_lcz; i < n; i += kWave >> log2_lcz) {
        float* __restrict__ dst = a.C + (row0 + list[i]) * a.N;
        for (int64_t k = (int64_t)chunk * VEC; k < a.N; k += (int64_t)VEC << log2_lcz)
            store_vec<VEC>(dst + lane_first_col<VEC>(k, a.N), z);
    }
}

NnzPlan plan_nnz_parallel(int group, int lc, int vec)
{
    NnzPlan p;
    // one step covers 4*64/lc positions, kParDepth steps are issued together:
    // at most 1024 positions, so one tile size serves every layout
    p.tile = kParTile;
    const int nslots = p.tile / group + 1;
    p.merge = nslots * (lc * vec * 4 + 8) <= kMergeLdsBudget;
    p.lc = lc;
    p.share = group;
    // Most of the LDS, and if need be narrower passes: for G = 1 (else a global atomic add per stored entry:
    // stencil27 32 ms against 20 ms, rmat 43 against 10) and for narrow passes (rmat, N = 32, G = 2 and 4:
    // 23 and 10 ms against 6.0 and 3.4).  Wider passes of G >= 2 do better with their few global atomics per
    // row than with one or two resident workgroups per compute unit (stencil27, N = 128, G = 2 and 4: 6.4 and
    // 4.1 ms against 12.1 and 9.3; skewed, N = 256, G = 4: 30 against 39).
    if (!p.merge && (group == 1 || lc * vec <= 32)) {
        int lanes = lc;
        while (nslots * (lanes * vec * 4 + 8) > kMergeLdsLimit && lanes > 1) lanes /= 2;
        if (nslots * (lanes * vec * 4 + 8) <= kMergeLdsLimit) {
            p.lc = lanes;
            p.merge = true;
        }
    }
    int lg = 0;
    while ((1 << lg) < (p.merge ? p.tile : group)) ++lg;
    p.merge_log2 = lg;
    return p;
}

// per-group-size launchers, defined in sgap_nnz_parallel_g*.hip
hipError_t launch_nnz_parallel_g1(const SpmmArgs&, int, int, int, int64_t, bool, hipStream_t);
hipError_t launch_nnz_parallel_g2(const SpmmArgs&, int, int, int, int64_t, bool, hipStream_t);
hipError_t launch_nnz_parallel_g4_16(const SpmmArgs&, int, int, int, int64_t, bool, hipStream_t);
hipError_t launch_nnz_parallel_g8_32_64(const SpmmArgs&, int, int, int, int64_t, bool, hipStream_t);

hipError_t launch_nnz_parallel(const SpmmArgs& a, int lc, int vec, const NnzPlan& plan, int compute_units,
                               int64_t nnz_hint, hipStream_t s)
{
    lc = plan.lc;
    switch (a.group) {
        case 1: return launch_nnz_parallel_g1(a, lc, vec, compute_units, nnz_hint, plan.merge, s);
        case 2: return launch_nnz_parallel_g2(a, lc, vec, compute_units, nnz_hint, plan.merge, s);
        case 4: case 16: return launch_nnz_parallel_g4_16(a, lc, vec, compute_units, nnz_hint, plan.merge, s);
        case 8: case 32: case 64: return launch_nnz_parallel_g8_32_64(a, lc, vec, compute_units, nnz_hint, plan.merge, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_nnz_zero_rows(const SpmmArgs& a, int vec, int merge_log2, hipStream_t s)
{
    const int64_t chunks = (a.N + vec - 1) / vec;
    int log2_lcz = 0;
    while (log2_lcz < 6 && (1 << log2_lcz) < chunks) ++log2_lcz;
    const int rows_per_wave = a.M < (1 << 17) && log2_lcz >= 2 ? 8 : kWave;  // (2^17 rows: two workgroups per compute unit)
    const int64_t rows_per_block = (int64_t)kWavesPerBlock * rows_per_wave;
    const dim3 grid((unsigned)((a.M + rows_per_block - 1) / rows_per_block)), block(kBlock);
    switch (vec) {
        case 4: hipLaunchKernelGGL((zero_rows_kernel<4>), grid, block, 0, s, a, log2_lcz, merge_log2, rows_per_wave); break;
        case 2: hipLaunchKernelGGL((zero_rows_kernel<2>), grid, block, 0, s, a, log2_lcz, merge_log2, rows_per_wave); break;
        case 1: hipLaunchKernelGGL((zero_rows_kernel<1>), grid, block, 0, s, a, log2_lcz, merge_log2, rows_per_wave); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace sgap
