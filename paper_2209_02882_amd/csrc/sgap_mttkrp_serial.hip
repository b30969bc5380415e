// MTTKRP on compressed sparse fibers with the stored entries as the unit of work, serial strategy: {<g nnz, c col>, 1}, few
// entries and few columns (where that ends: mttkrp_serial_applies; the rest is mttkrp_tiles_kernel's).
//     t[f,:]  = sum over the entries (l, v) of fiber f of  v * X2[l,:]
//     Y[i,:]  = sum over the fibers f of slice i of        X1[fidx[f],:] * t[f,:]
// A lane walks g consecutive entries (g = the tile's entries over the workgroup's entry lanes, so that a tile is one walk
// of every lane: smaller shares flush more often and need more accumulators, larger ones leave lanes idle; group_size
// does not enter) and passes the slice's sum on where a slice (or its share) ends: the conditional
// flush.  The merge rule is the one of the SpMM kernels (sgap_nnz_common.hpp): a slice inside one lane's share is stored
// plainly, the others are combined per tile in LDS, and only slices that reach beyond the tile use global atomics.
//
// What bounds it is the gathers of rows of X2 (a factor that does not fit a die's L2 comes from the Infinity Cache); what
// kept it from that was its own control flow: a fiber holds a handful of entries, and the eight entry lanes of a wavefront
// close a fiber at two of three steps.  So a step does little beside its gather and multiply-add:
//   - a tile's fibers (a thread each) find their slice and bring their row of X1 into LDS, once per tile, from where
//     t[f,:] is scaled when the fiber ends;
//   - where a fiber and where a slice ends is marked in the entry's fiber number;
//   - the next tile's entries, fiber pointers and slice pointers are requested before this tile is multiplied out.
// A tile with more fibers than LDS has rows for is cut into pieces of that many fibers, each merged by itself.
// 262,144 slices, one in a thousand with 2,000 to 20,000 fibers, J = 32, G = 32: 873 us with a 16-byte record per entry
// (two bisections and three loads each) and two searches per tile, 540 with this (and 455 by mttkrp_tiles_kernel, whose it is).  (v * X1[k,:]) * X2[l,:] added up entry by
// entry, with nothing to do where a fiber ends, takes as long; it rounds once more per entry and adds in one long chain
// (mean error 1.82e-8 of the sum of absolute values against 1.56e-8), and v * X1[k,:] may leave the range of the numbers
// where no t[f,:] does.
#include "sgap_gather.hpp"
#include "sgap_nnz_common.hpp"

namespace sgap {

constexpr int kMsColumns = 8;
constexpr int kMsEpt = 4;
constexpr int kMsTile = kMsEpt * kBlock;
constexpr int kMsBatch = 64;             // tiles whose first fibers and slices are looked up at once
constexpr int kMsFibers = kBlock - 1;    // fibers of a piece at most: a thread each, and a pointer more
constexpr int kMsSlices = kBlock - 1;    // slices whose pointers a tile keeps (a fiber beyond them bisects the pointers)
constexpr uint16_t kMsEnds = 1 << 15;       // the slice ends with this entry
constexpr uint16_t kMsFiberEnds = 1 << 14;  // the fiber does
constexpr int kMsFiberMask = kMsFiberEnds - 1;

// LDS place of a tile's entry: the entry lanes of a wavefront read at strides of g entries, which without the padding
// all fall on the same banks.
__device__ __forceinline__ int ms_place(int q) { return q + (q >> 5); }

template <int LC, int VEC, bool OFF32, bool RAGGED>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4))) void mttkrp_serial_kernel(MttkrpArgs a)
{
    constexpr int x1_rows = kMsFibers;  // rows of X1 in LDS
    constexpr int ENTRY_LANES = kBlock / LC;
    constexpr int GROUP = kMsTile / ENTRY_LANES;  // entries of a lane's share
    constexpr int D = 4;  // gathered rows of X2 in flight per lane
    constexpr int PITCH = LC * VEC;
    extern __shared__ __align__(16) unsigned char s_raw[];
    __shared__ StagedEntry s_A[kMsTile + (kMsTile >> 5)];
    __shared__ __align__(16) uint16_t s_fiber[kMsTile];  // an entry's fiber, counted from the piece's first, and the two marks
    __shared__ int32_t s_fwin[kMsFibers + 1];  // first positions of the piece's fibers
    __shared__ int32_t s_k[kMsFibers];         // their rows of X1
    __shared__ int32_t s_i[kMsFibers];         // their slices
    __shared__ int32_t s_begin[kMsFibers];     // where their slices begin (-1: before the piece)
    __shared__ int32_t s_end[kMsFibers];       // ... and end (kNever: after it, or not known)
    __shared__ int32_t s_swin[kMsSlices + 1];  // slice pointers
    __shared__ int32_t s_tile_fiber[kMsBatch], s_tile_slice[kMsBatch];
    constexpr int32_t kNever = 0x7fffffff;
    const int32_t I = (int32_t)a.I;
    const int32_t F = a.fptr[a.I];
    const int32_t E = F > 0 ? a.eptr[F] : 0;
    const int64_t tiles = ((int64_t)E + kMsTile - 1) / kMsTile;
    const TileDeal deal(tiles, blockIdx.x, gridDim.x);
    const int64_t my_tiles = deal.mine;
    if (my_tiles == 0) return;
    TileWalk ahead(deal);  // the tile that is fetched next
    SpmmArgs out;          // what the write-back needs
    out.N = a.J;
    out.C = a.Y;
    float* s_x1 = reinterpret_cast<float*>(s_raw);
    MergeBuf mb;
    mb.nslots = ENTRY_LANES + 1;
    mb.width = PITCH;
    mb.accum = s_x1 + x1_rows * PITCH;
    mb.slot_row = reinterpret_cast<int32_t*>(mb.accum + mb.nslots * mb.width);
    mb.slot_atomic = mb.slot_row + mb.nslots;
    merge_reset(mb);  // made visible by the barriers below

    int32_t nx_idx[kMsEpt];
    float nx_val[kMsEpt];
    int32_t nx_fwin, nx_swin, nx_k;
    auto fetch_tile = [&](int32_t f_lb, int32_t i_lb) {  // the tile `ahead` stands at
        const int32_t start = (int32_t)(ahead.tile() * kMsTile);
#pragma unroll
        for (int i = 0; i < kMsEpt; ++i) {
            const int32_t p = start + threadIdx.x + i * kBlock;
            nx_idx[i] = 0;
            nx_val[i] = 0.0f;
            if (p < E) {
                nx_idx[i] = load_stream(a.eidx + p);
                nx_val[i] = load_stream(a.vals + p);
            }
        }
        const int tid = threadIdx.x;
        nx_fwin = a.eptr[(int64_t)f_lb + tid <= F ? f_lb + tid : F];
        nx_swin = a.fptr[(int64_t)i_lb + tid <= I ? i_lb + tid : I];
        nx_k = (int64_t)f_lb + tid < F ? a.fidx[f_lb + tid] : 0;
    };

    for (int64_t j0 = 0; j0 < my_tiles; j0 += kMsBatch) {
        // the fibers of the tiles' first entries, and those fibers' slices
        const int batch = (int)(my_tiles - j0 < kMsBatch ? my_tiles - j0 : kMsBatch);
        __syncthreads();  // the previous batch's are no longer needed
        find_positions(a.eptr, F - 1, batch, [&](int j) { return (int32_t)(deal.tile(j0 + j) * kMsTile); }, s_tile_fiber);
        __syncthreads();
        find_positions(a.fptr, I - 1, batch, [&](int j) { return s_tile_fiber[j]; }, s_tile_slice);
        __syncthreads();
        fetch_tile(s_tile_fiber[0], s_tile_slice[0]);

        for (int j = 0; j < batch; ++j) {
            // (the thread's number through an opaque copy: what is computed from it in front of the walk would otherwise
            // be hoisted out of the loop over tiles and hold registers throughout the walk)
            int tid = threadIdx.x;
            asm volatile("" : "+v"(tid));
            const int entry_lane = tid / LC;
            const int chunk = tid % LC;
            const int32_t tile_start = (int32_t)(ahead.tile() * kMsTile);
            ahead.next();
            const int32_t tile_end = E - tile_start < kMsTile ? E : tile_start + kMsTile;
            int32_t f_lb = s_tile_fiber[j];
            const int32_t i_lb = s_tile_slice[j];
            // install the tile that was fetched ahead
#pragma unroll
            for (int i = 0; i < kMsEpt; ++i) {
                StagedEntry e;
                e.col = nx_idx[i];
                e.val = nx_val[i];
                s_A[ms_place(tid + i * kBlock)] = e;
            }
            s_fwin[tid] = nx_fwin;
            s_swin[tid] = nx_swin;
            if (tid < kMsFibers) s_k[tid] = nx_k;
            __syncthreads();
            if (j + 1 < batch) fetch_tile(s_tile_fiber[j + 1], s_tile_slice[j + 1]);

            for (int32_t base = tile_start; base < tile_end;) {
                // the piece [base, end): as many fibers from f_lb on as there are rows in LDS
                if (s_fwin[x1_rows] <= base) {
                    // nothing but fibers without entries: on to the one that holds base
                    __syncthreads();
                    f_lb = last_row_at_or_before(a.eptr, f_lb + x1_rows, F - 1, base);
                    s_fwin[tid] = a.eptr[(int64_t)f_lb + tid <= F ? f_lb + tid : F];
                    if (tid < kMsFibers) s_k[tid] = (int64_t)f_lb + tid < F ? a.fidx[f_lb + tid] : 0;
                    __syncthreads();
                    continue;
                }
                const int32_t top = s_fwin[x1_rows];
                const int32_t end = top < tile_end ? top : tile_end;
                // the rows of X1 (in the lanes' own layout)
                for (int q = tid; q < x1_rows * LC; q += kBlock) {
                    const int r = q / LC;
                    const uint32_t k = q % LC * VEC;
                    if (s_fwin[r] >= end || k >= (uint32_t)a.J) continue;
                    const Vec<VEC> x = load_vec<VEC>(a.X1 + (int64_t)s_k[r] * a.J + lane_first_col<VEC, RAGGED>(k, (uint32_t)a.J));
#pragma unroll
                    for (int v = 0; v < VEC; ++v) s_x1[q * VEC + v] = x.v[v];
                }
                // a thread per fiber: its slice, where its slice begins and ends
                if (tid < x1_rows && s_fwin[tid] < end && s_fwin[tid + 1] > s_fwin[tid]) {
                    const int32_t f = f_lb + tid;
                    int32_t i, first, next;  // the slice, its first fiber and the next slice's
                    if (s_swin[kMsSlices] > f) {
                        const int w = first_above(s_swin, kMsSlices + 1, f) - 1;
                        i = i_lb + w;
                        first = s_swin[w];
                        next = s_swin[w + 1];
                    } else {
                        i = last_row_at_or_before(a.fptr, i_lb + kMsSlices, I - 1, f);
                        first = a.fptr[i];
                        next = a.fptr[i + 1];
                    }
                    s_i[tid] = i;
                    s_begin[tid] = first >= f_lb && s_fwin[first - f_lb] >= base ? s_fwin[first - f_lb] : -1;
                    s_end[tid] = next - f_lb <= x1_rows ? s_fwin[next - f_lb] : kNever;
                }
                __syncthreads();
                {
                    const int32_t p = tile_start + tid * kMsEpt;
                    int32_t w = last_row_at_or_before(s_fwin, 0, x1_rows - 1, p);
#pragma unroll
                    for (int i = 0; i < kMsEpt; ++i) {
                        if (p + i < base || p + i >= end) continue;
                        while (s_fwin[w + 1] <= p + i) ++w;  // ends: some fiber of the piece holds the entry
                        s_fiber[tid * kMsEpt + i] = (uint16_t)(
                            w | (s_fwin[w + 1] == p + i + 1 ? kMsFiberEnds : 0) | (s_end[w] == p + i + 1 ? kMsEnds : 0));
                    }
                }
                __syncthreads();

                {
                    const uint32_t k = chunk * VEC;
                    const bool k_ok = k < (uint32_t)a.J;
                    const uint32_t k_lane = k_ok ? lane_first_col<VEC, RAGGED>(k, (uint32_t)a.J) : 0;
                    const BRow<OFF32> X2row(a.X2, a.J, k_lane);
                    const float* __restrict__ my_x1 = s_x1 + chunk * VEC;
                    // this lane's share, clipped to the piece
                    const int32_t blk = tile_start + entry_lane * GROUP;
                    const int32_t blk_begin = blk > base ? blk : base;
                    const int32_t blk_end = blk + GROUP < end ? blk + GROUP : end;
                    if (k_ok && blk_begin < blk_end) {
                        int32_t run_begin = blk_begin;  // where the slice's run in this share begins
                        Vec<VEC> sum, t;  // of the slice's fibers, of the fiber's entries
                        sum.zero();
                        t.zero();
                        // the run that ends with entry p leaves the registers
                        auto flush = [&](int32_t p, int fiber) {
                            const int w = fiber & kMsFiberMask;
                            const bool ends = (fiber & kMsEnds) != 0;
                            const int32_t row = s_i[w], begin = s_begin[w];
                            if (ends && begin == run_begin) {
                                store_vec_stream<VEC>(a.Y + (int64_t)row * a.J + k_lane, sum);
                            } else {
                                from_last_columns<VEC, RAGGED>(sum, (int)(k - k_lane));
                                merge_add<VEC, (LC >= 8)>(mb, begin < 0 ? mb.nslots - 1 : (begin - tile_start) / GROUP,
                                                          chunk * VEC, sum, chunk == 0 && run_begin == (begin < 0 ? base : begin),
                                                          row, begin < 0 || s_end[w] > end);
                            }
                            sum.zero();
                            run_begin = p + 1;
                        };
                        for (int32_t p0 = tile_start + ((blk_begin - tile_start) & ~(D - 1)); p0 < blk_end; p0 += D) {
                            StagedEntry e[D];
                            int fiber[D];
                            Vec<VEC> b[D];
                            const bool full = p0 >= blk_begin && p0 + D <= blk_end;
                            const StagedEntry* __restrict__ here = s_A + ms_place(p0 - tile_start);
                            auto mine = [&](int u) { return p0 + u >= blk_begin && p0 + u < blk_end; };
                            if (full) {
#pragma unroll
                                for (int u = 0; u < D; ++u) e[u] = here[u];
#pragma unroll
                                for (int u = 0; u < D; ++u) b[u] = load_vec<VEC>(X2row.at(e[u].col));
#pragma unroll
                                for (int u = 0; u < D; u += 4) {
                                    const uint2 f4 = *reinterpret_cast<const uint2*>(s_fiber + (p0 + u - tile_start));
                                    fiber[u] = f4.x & 0xffff; fiber[u + 1] = f4.x >> 16;
                                    fiber[u + 2] = f4.y & 0xffff; fiber[u + 3] = f4.y >> 16;
                                }
                            } else {
#pragma unroll
                                for (int u = 0; u < D; ++u) {
                                    e[u].col = 0;
                                    e[u].val = 0.0f;
                                    if (mine(u)) e[u] = here[u];
                                }
#pragma unroll
                                for (int u = 0; u < D; ++u) {
                                    b[u].zero();
                                    if (mine(u)) b[u] = load_vec<VEC>(X2row.at(e[u].col));
                                }
#pragma unroll
                                for (int u = 0; u < D; ++u) fiber[u] = mine(u) ? s_fiber[p0 + u - tile_start] : 0;
                            }
#pragma unroll
                            for (int u = 0; u < D; ++u) {
                                if (!full && !mine(u)) continue;
                                t.fma(e[u].val, b[u]);
                                const bool last = p0 + u + 1 == blk_end;
                                if ((fiber[u] & kMsFiberEnds) || last) {
                                    const float* x = my_x1 + (fiber[u] & kMsFiberMask) * PITCH;
                                    if constexpr (VEC == 4) {
                                        const float4 f = *reinterpret_cast<const float4*>(x);
                                        sum.v[0] = __builtin_fmaf(f.x, t.v[0], sum.v[0]);
                                        sum.v[1] = __builtin_fmaf(f.y, t.v[1], sum.v[1]);
                                        sum.v[2] = __builtin_fmaf(f.z, t.v[2], sum.v[2]);
                                        sum.v[3] = __builtin_fmaf(f.w, t.v[3], sum.v[3]);
                                    } else {
#pragma unroll
                                        for (int v = 0; v < VEC; ++v) sum.v[v] = __builtin_fmaf(x[v], t.v[v], sum.v[v]);
                                    }
                                    t.zero();
                                    if ((fiber[u] & kMsEnds) || last) flush(p0 + u, fiber[u]);
                                }
                            }
                        }
                    }
                    __syncthreads();  // all sums are in LDS
                    merge_write_out<LC, VEC, RAGGED>(out, mb, k, k_ok);
                }
                __syncthreads();  // slots are clear again, the piece is consumed
                base = end;
                if (base < tile_end) {  // the fibers that follow
                    f_lb += x1_rows;
                    s_fwin[tid] = a.eptr[(int64_t)f_lb + tid <= F ? f_lb + tid : F];
                    if (tid < kMsFibers) s_k[tid] = (int64_t)f_lb + tid < F ? a.fidx[f_lb + tid] : 0;
                    __syncthreads();
                }
            }
        }
    }
}

namespace {

struct LaunchSerial {
    const MttkrpArgs& a;
    int compute_units;
    int64_t nnz_hint;
    bool off32;
    hipStream_t s;

    template <int LC, int VEC, bool OFF32, bool RAGGED>
    void go() const
    {
        auto kernel = mttkrp_serial_kernel<LC, VEC, OFF32, RAGGED>;
        constexpr int smem = kMsFibers * LC * VEC * 4 + (kBlock / LC + 1) * (LC * VEC * 4 + 8);
        static const int per_cu = resident_per_cu(kernel, smem);
        const int grid = persistent_grid(per_cu, compute_units, nnz_hint, kMsTile);
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(kBlock), smem, s, a);
    }
    template <int G, int LC, int VEC>
    void operator()() const
    {
        constexpr bool WIDE = VEC > 1;  // rows whose columns the lanes need not divide
        if constexpr (LC * VEC > kMsColumns) return;  // (launch_mttkrp_serial asks for none)
        else if (!off32) go<LC, VEC, false, WIDE>();
        else if (WIDE && a.J % VEC != 0) go<LC, VEC, true, WIDE>();
        else go<LC, VEC, true, false>();
    }
};

}  // namespace

// A tile here is one step through the loads less, and there is no more of it.  us, this / teams of lanes at their own pace
// (slices of 4 fibers of 4.5 entries): J = 4, 1,000 slices 13.0 / 17.0, 10,000 16.3 / 18.1, 30,000 22.8 / 24, 60,000
// 36.7 / 29.3; J = 8, 1,000 14.2 / 16.5, 10,000 17.2 / 18.0, 30,000 23.3 / 23.4; J = 16, 1,000 15.7 / 16, 10,000 20.1 / 20.1;
// one slice in a thousand with 2,000 to 20,000 fibers: J = 4, 5,000 slices 20.8 / 21.5, 20,000 42.7 / 37.6; J = 1, 5,000
// 14.6 / 17.4, 100,000 95 / 96.
bool mttkrp_serial_applies(int64_t J, int64_t nnz_hint)
{
    return J <= kMsColumns && nnz_hint > 0 && nnz_hint < (J < 4 ? 2000000 / J : J < 8 ? 700000 : 500000);
}

hipError_t launch_mttkrp_serial(const MttkrpArgs& a, int lc, int vec, int compute_units, int64_t nnz_hint,
                                hipStream_t s)
{
    if (a.J > kMsColumns || lc * vec > kMsColumns) return hipErrorInvalidValue;
    if (!dispatch_lc<1>(lc, vec, LaunchSerial{a, compute_units, nnz_hint, offsets_fit_32(a.K, a.J) && offsets_fit_32(a.L, a.J), s}))
        return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace sgap
