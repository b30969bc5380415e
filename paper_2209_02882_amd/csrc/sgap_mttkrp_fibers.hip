// MTTKRP on compressed sparse fibers with the slices as the unit of work, parallel strategy:
//     t[f,:]  = sum over the entries (l, v) of fiber f of  v * X2[l,:]
//     Y[i,:]  = sum over the fibers f of slice i of        X1[fidx[f],:] * t[f,:]
// A workgroup owns a block of consecutive slices and works through their fibers in pieces (one piece, as a rule) whose
// fibers and entries it brings into LDS with coalesced loads.  A team of lanes, four columns each, takes consecutive
// fibers of a piece, cut where the entries are about even, and goes through them at its own pace (sgap_flat.hpp) with the
// slice's sum in registers; it stores what begins and ends among them.  What a team has of a slice that began in front of it goes to LDS, where the team that has the
// slice's beginning adds it up in order: one plain store per slice, no atomics, the same result every time.  A slice that
// goes on in the next piece is carried over in LDS, and a fiber that a piece has no room for is the whole workgroup's.
//
// Bound by the gathers: of two factors of 8.4 MB 1.7 GB come from beyond the L2s, at 7.1 TB/s; small tensors by the chain
// of loads that a block is (pointers, fibers, entries, then a team's rows of X2).  With a group of lanes per slice, members
// m, m + G, ... of which took the slice's fibers (the form before), a third of the members had no fiber, each waited for the
// longest of its wavefront's, and every slice ended in a tree sum.  us, group per slice / this, J = 32 unless said, slices x
// fibers of a slice: 262,144 x 8 268 / 240, with factors of 256 KB 235 / 164; 227,077 x 4, J = 16 104 / 78; 133,470 x 6
// 123 / 95; 43,825 x 7 62 to 76 / 41; 21,755 x 8 39 to 49 / 25; 15,510 x 6, J = 16 23 to 27 / 15; 100,000 x 8, J = 64
// 254 / 230.
#include "sgap_common.hpp"
#include "sgap_flat.hpp"
#include "sgap_nnz_common.hpp"

namespace sgap {

constexpr int kMfSlices = 256;    // slices of a block at most
constexpr int kMfFibers = 512;    // fibers of a piece at most
constexpr int kMfEntries = 3328;  // entries of a piece at most: four workgroups' LDS, as many as the registers leave
constexpr int kMfResident = 4;    // workgroups of a compute unit
constexpr int kMfMean = 2600;     // entries of a block in the mean at most; 2,000 from kMfRounds rounds of blocks on
constexpr int kMfRounds = 5;
constexpr int kMfBlock = 16;      // slices of a block where the caller does not say how many entries there are

template <int VEC, bool OFF32>
__global__ __launch_bounds__(kBlock) void mttkrp_fibers_kernel(MttkrpArgs a, int lanes, int block_slices,
                                                               int64_t blocks, int64_t blocks_per_xcd, int xcds)
{
    const int teams = kBlock / lanes;
    __shared__ FlatShared<kMfEntries, kMfFibers> s;  // its runs are fibers
    __shared__ int32_t s_fk[kMfFibers];
    __shared__ int32_t s_fp[kMfSlices + 1];
    __shared__ Vec<VEC> s_head[kBlock];    // what a team has of a slice that began in front of its fibers
    __shared__ uint8_t s_ended[kBlock];    // whether that slice ends there
    __shared__ Vec<VEC> s_carry[2][kWave];  // of the slice that goes on in the next piece
    struct Columns {
        bool ok;
        uint32_t first;  // of the VEC columns this lane holds
        __device__ __forceinline__ Columns(const FlatPlace& p, int64_t k0, int64_t J, int teams)
        {
            const uint32_t k = (uint32_t)k0 + p.chunk * VEC;  // J < 2^31
            ok = k < (uint32_t)J && p.team < teams;
            first = ok ? lane_first_col<VEC>(k, (uint32_t)J) : 0;
        }
    };

    // workgroup b runs on die b % xcds: every die gets one contiguous run of blocks
    const int64_t block = (int64_t)(blockIdx.x % xcds) * blocks_per_xcd + blockIdx.x / xcds;
    if (block >= blocks) return;  // the whole workgroup
    const int64_t first_slice = block * block_slices;
    const int slices = (int)(a.I - first_slice < block_slices ? a.I - first_slice : block_slices);
    for (int i = threadIdx.x; i <= slices; i += kBlock) s_fp[i] = a.fptr[first_slice + i];
    __syncthreads();
    const int32_t f_begin = __builtin_amdgcn_readfirstlane(s_fp[0]);
    const int32_t f_end = __builtin_amdgcn_readfirstlane(s_fp[slices]);

    for (int64_t k0 = 0; k0 < a.J; k0 += (int64_t)lanes * VEC) {
        auto store = [&](int slice, const Columns& c, const Vec<VEC>& sum) {
            if (c.ok) store_vec_stream<VEC>(a.Y + (first_slice + slice) * a.J + c.first, sum);
        };
        {
            const FlatPlace p(lanes);
            const Columns c(p, k0, a.J, teams);
            Vec<VEC> none;
            none.zero();
            for (int r = p.team; r < slices; r += teams)
                if (s_fp[r] == s_fp[r + 1]) store(r, c, none);
        }

        int turn = 0;  // which of s_carry the piece takes over
        for (int32_t f0 = f_begin; f0 < f_end; turn ^= 1) {
            int32_t n = f_end - f0 < kMfFibers ? f_end - f0 : kMfFibers;  // fibers of the piece
            __syncthreads();  // the piece before is done with
            {
                const FlatPlace p(lanes);
#pragma unroll 2
                for (int i = p.tid; i <= n; i += kBlock) {
                    s.ptr[i] = a.eptr[f0 + i];
                    if (i < n) s_fk[i] = a.fidx[f0 + i];
                }
            }
            __syncthreads();
            const int32_t e0 = __builtin_amdgcn_readfirstlane(s.ptr[0]);
            if (s.ptr[n] - e0 > kMfEntries) {
                const FlatPlace p(lanes);
                int fit = 0;
                for (int i = 0; i < n; i += kBlock) fit += __syncthreads_count(i + p.tid < n && s.ptr[i + p.tid + 1] - e0 <= kMfEntries);
                n = fit;
            }
            n = __builtin_amdgcn_readfirstlane(n);
            if (n == 0) {
                // a fiber of more entries than there is room for: all teams together
                const FlatPlace p(lanes);
                const Columns c(p, k0, a.J, teams);
                const MaskedRows<VEC, OFF32> x1(a.X1, a.K, a.J, c.first), x2(a.X2, a.L, a.J, c.first);
                const int32_t e1 = __builtin_amdgcn_readfirstlane(s.ptr[1]);
                Vec<VEC> t;
                t.zero();
                for (int32_t base = e0; base < e1; base += kMfEntries) {
                    const int32_t cnt = e1 - base < kMfEntries ? e1 - base : kMfEntries;
                    __syncthreads();
                    flat_stage<kMfEntries>(s, a.eidx, a.vals, base, cnt, p.tid);
                    __syncthreads();
#pragma unroll 1
                    for (int q = p.team; c.ok && q < cnt; q += teams) t.fma(s.entry[q].val, x2.load(s.entry[q].col, true));
                }
                s_head[p.tid] = t;
                __syncthreads();
                if (p.team == 0) {
#pragma unroll 1
                    for (int m = 1; m < teams; ++m) {
                        const Vec<VEC> other = s_head[m * lanes + p.chunk];
#pragma unroll
                        for (int i = 0; i < VEC; ++i) t.v[i] += other.v[i];
                    }
                    const int slice = last_row_at_or_before(s_fp, 0, slices - 1, f0);
                    const Vec<VEC> x = x1.load(s_fk[0], c.ok);
                    Vec<VEC> sum;
                    sum.zero();
                    if (s_fp[slice] < f0) sum = s_carry[turn][p.chunk];
#pragma unroll
                    for (int i = 0; i < VEC; ++i) sum.v[i] = __builtin_fmaf(x.v[i], t.v[i], sum.v[i]);
                    if (s_fp[slice + 1] == f0 + 1) store(slice, c, sum);
                    else s_carry[turn ^ 1][p.chunk] = sum;
                }
                ++f0;
                continue;
            }

            // the piece's entries, and meanwhile where the teams begin
            const int32_t cnt = __builtin_amdgcn_readfirstlane(s.ptr[n]) - e0;
            {
                const FlatPlace p(lanes);
                flat_stage<kMfEntries>(s, a.eidx, a.vals, e0, cnt, p.tid);
                flat_deal(s, e0, cnt, n, teams, p.tid);
            }
            __syncthreads();

            const FlatPlace p(lanes);
            const Columns c(p, k0, a.J, teams);
            Vec<VEC> sum;
            sum.zero();
            int slice = 0;
            bool goes_on = false;  // the slice that begins in this team's fibers goes on behind them
            {
                const int first = p.team < teams ? s.start[p.team] : 0, last = p.team < teams ? s.start[p.team + 1] : 0;
                bool head_ends = false;
                if (first < last) {
                    const MaskedRows<VEC, OFF32> x1(a.X1, a.K, a.J, c.first), x2(a.X2, a.L, a.J, c.first);
                    slice = last_row_at_or_before(s_fp, 0, slices - 1, f0 + first);
                    bool whole = s_fp[slice] == f0 + first;
                    int32_t slice_end = s_fp[slice + 1] - f0;
                    Vec<VEC> x;
                    flat_walk<VEC, OFF32>(
                        s, first, last, e0, x2, c.ok, [&](int f, bool ends) { x = x1.load(s_fk[f], ends && c.ok); },
                        [&](int f, const Vec<VEC>& t) {
#pragma unroll
                            for (int i = 0; i < VEC; ++i) sum.v[i] = __builtin_fmaf(x.v[i], t.v[i], sum.v[i]);
                            if (f + 1 != slice_end) return;
                            if (whole) {
                                store(slice, c, sum);
                            } else {
                                s_head[p.tid] = sum;
                                head_ends = true;
                            }
                            sum.zero();
                            whole = true;
                            if (f + 1 < last) {
                                do slice_end = s_fp[++slice + 1] - f0;
                                while (slice_end == f + 1);
                            }
                        });
                    goes_on = last != slice_end && whole;
                    if (last != slice_end && !whole) s_head[p.tid] = sum;
                } else {
                    s_head[p.tid] = sum;
                }
                if (p.team < teams) s_ended[p.team] = head_ends ? 1 : 0;
            }
            __syncthreads();
            // what goes on is added up by the team that has its beginning, what came in from the piece before by the first team
            const int32_t came_in = f0 > f_begin ? last_row_at_or_before(s_fp, 0, slices - 1, f0) : 0;
            const bool comes_in = f0 > f_begin && s_fp[came_in] < f0;
#pragma unroll 1
            for (int round = 0; round < 2; ++round) {
                if (round == 1) {
                    goes_on = comes_in && p.team == 0;
                    if (goes_on) sum = s_carry[turn][p.chunk];
                    slice = came_in;
                }
                if (!goes_on) continue;
                const bool ended = add_heads<VEC>(sum, s_head, s_ended, round == 1 ? 0 : p.team + 1, teams, lanes, p.chunk);
                if (ended) store(slice, c, sum);
                else s_carry[turn ^ 1][p.chunk] = sum;
            }
            f0 += n;
        }
    }
}

// Blocks of even numbers of slices, as many as make whole rounds of the chip's resident workgroups: a tensor of 45,373 slices of
// 5 fibers, J = 24, takes 34.8 us in one round of 964 blocks and 43.1 in 1,286.  The larger a block the better, up to what
// leaves few blocks in more than one piece; with many rounds those count more than the rounds (2,600 entries a block / 2,000:
// 76,491 slices of 4 fibers, J = 32, two rounds 42.0 us / 46.2, 262,144 of 8, seven rounds or nine, 264 to 272 / 263).
int mttkrp_block_slices(int64_t I, int64_t nnz_hint, int compute_units)
{
    if (nnz_hint <= 0) return kMfBlock;
    const int64_t resident = (int64_t)kMfResident * compute_units;
    int64_t rounds = nnz_hint / (resident * kMfMean) + 1;
    if (rounds >= kMfRounds) rounds = nnz_hint / (resident * 2000) + 1;
    const int64_t slices = (I + resident * rounds - 1) / (resident * rounds);
    return slices < kMfSlices ? (int)slices : kMfSlices;
}

hipError_t launch_mttkrp_fibers(const MttkrpArgs& a, int block_slices, int vec, int xcds, hipStream_t s)
{
    if (block_slices > kMfSlices) block_slices = kMfSlices;
    const int64_t blocks = (a.I + block_slices - 1) / block_slices;
    if (blocks + xcds > 0x7ffffff0LL) return hipErrorInvalidValue;
    const int64_t blocks_per_xcd = (blocks + xcds - 1) / xcds;
    const int64_t chunks = (a.J + vec - 1) / vec;
    const int lanes = chunks < kWave ? (int)chunks : kWave;
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)(blocks_per_xcd * xcds)), dim3(kBlock), 0, s, a, lanes, block_slices, blocks, blocks_per_xcd, xcds);
    };
    // every byte offset into X1 and X2 fits 32 bits and both factors of it fit 24 bits
    auto fits = [&](int64_t rows) { return rows <= (1 << 24) && a.J * 4 < (1 << 24) && rows * a.J * 4 <= 0xffffffffLL; };
    const bool off32 = fits(a.K) && fits(a.L);
    if (vec == 4) { if (off32) go(mttkrp_fibers_kernel<4, true>); else go(mttkrp_fibers_kernel<4, false>); }
    else if (vec == 2) { if (off32) go(mttkrp_fibers_kernel<2, true>); else go(mttkrp_fibers_kernel<2, false>); }
    else { if (off32) go(mttkrp_fibers_kernel<1, true>); else go(mttkrp_fibers_kernel<1, false>); }
    return hipGetLastError();
}

}  // namespace sgap
