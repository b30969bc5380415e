// MTTKRP on compressed sparse fibers with the slices as the unit of work, parallel strategy:
//     t[f,:]  = sum over the entries (l, v) of fiber f of  v * X2[l,:]
//     Y[i,:]  = sum over the fibers f of slice i of        X1[fidx[f],:] * t[f,:]
// A workgroup owns a block of consecutive slices and works through their fibers in pieces (one piece, as a rule) whose
// fibers and entries it brings into LDS with coalesced loads.  A team of LC lanes, four columns each, takes consecutive
// fibers of a piece, cut where the entries are about even; it walks them with the slice's sum in registers and stores what
// begins and ends among them.  What a team has of a slice that began in front of it goes to LDS, where the team that has the
// slice's beginning adds it up in order: one plain store per slice, no atomics, the same result every time.  A slice that
// goes on in the next piece is carried over in LDS, and a fiber that a piece has no room for is the whole workgroup's.
//
// Bound by the gathers: of two factors of 8.4 MB 1.7 GB come from beyond the L2s, at 6.6 TB/s; small tensors by the chain
// of loads that a block is (pointers, fibers, entries, then a team's rows of X2).  With a group of lanes per slice, members
// m, m + G, ... of which took the slice's fibers (the form before), a third of the members had no fiber, each waited for the
// longest of its wavefront's, and every slice ended in a tree sum.  us, group per slice / this, J = 32 unless said, slices x
// fibers of a slice: 262,144 x 8 268 / 263; 227,077 x 4, J = 16 104 / 85; 133,470 x 6 123 / 104; 43,825 x 7 62 to 76 / 47;
// 21,755 x 8 39 to 49 / 30; 15,510 x 6, J = 16 23 to 27 / 16; 100,000 x 8, J = 2 219 / 55, J = 128 549 / 501; one slice in a
// thousand with 2,000 to 20,000 25,200 / 2,340.
#include "sgap_common.hpp"
#include "sgap_gather.hpp"
#include "sgap_nnz_common.hpp"

namespace sgap {

constexpr int kMfDepth = 8;       // gathered rows of X2 in flight per lane (16 MB of factors, us: 262 with 8, 292 with 6)
constexpr int kMfSlices = 256;    // slices of a block at most
constexpr int kMfFibers = 512;    // fibers of a piece at most
constexpr int kMfEntries = 3584;  // entries of a piece at most: four workgroups' LDS, as many as the registers leave
constexpr int kMfResident = 4;    // workgroups of a compute unit
constexpr int kMfMean = 2600;     // entries of a block in the mean at most; 2,000 from kMfRounds rounds of blocks on
constexpr int kMfRounds = 5;
constexpr int kMfBlock = 16;      // slices of a block where the caller does not say how many entries there are

// Rows of a dense operand by number; `ok` = false reads as zeros, without a branch where byte offsets have 32 bits (an offset
// past the end of a buffer descriptor is not fetched).
template <int VEC, bool OFF32>
struct MaskedRows {
    __amdgpu_buffer_rsrc_t rows;
    uint32_t row_bytes, k_bytes;
    const float* base;
    int64_t J;
    __device__ __forceinline__ MaskedRows(const float* X, int64_t count, int64_t j, uint32_t k)
        : rows(__builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(X), 0, (int)(uint32_t)(OFF32 ? count * j * 4 : 0), 0x00020000)),
          row_bytes((uint32_t)(j * 4)), k_bytes(k * 4), base(X + k), J(j)
    {
    }
    __device__ __forceinline__ Vec<VEC> load(int32_t row, bool ok) const
    {
        Vec<VEC> r;
        if constexpr (OFF32) {
            const uint32_t off = ok ? __umul24((uint32_t)row, row_bytes) + k_bytes : 0xfffffffcu;
            if constexpr (VEC == 4) {
                typedef uint32_t raw_u4 __attribute__((ext_vector_type(4)));
                const raw_u4 t = __builtin_amdgcn_raw_buffer_load_b128(rows, (int)off, 0, 0);
                r.v[0] = __uint_as_float(t.x); r.v[1] = __uint_as_float(t.y); r.v[2] = __uint_as_float(t.z); r.v[3] = __uint_as_float(t.w);
            } else if constexpr (VEC == 2) {
                typedef uint32_t raw_u2 __attribute__((ext_vector_type(2)));
                const raw_u2 t = __builtin_amdgcn_raw_buffer_load_b64(rows, (int)off, 0, 0);
                r.v[0] = __uint_as_float(t.x); r.v[1] = __uint_as_float(t.y);
            } else {
                r.v[0] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rows, (int)off, 0, 0));
            }
        } else {
            r.zero();
            if (ok) r = load_vec<VEC>(base + (int64_t)row * J);
        }
        return r;
    }
};

// acc += the entries q, q + STRIDE, ... < q1 of s_A (which is read up to D * STRIDE places further), D rows in flight.
template <int VEC, int STRIDE, int D, bool OFF32>
__device__ __forceinline__ void masked_fma(Vec<VEC>& acc, const StagedEntry* __restrict__ s_A, uint32_t q, uint32_t q1,
                                           const MaskedRows<VEC, OFF32>& X)
{
#pragma unroll 1
    for (; q < q1; q += D * STRIDE) {
        StagedEntry e[D];
        Vec<VEC> b[D];
#pragma unroll
        for (int u = 0; u < D; ++u) e[u] = s_A[q + u * STRIDE];
#pragma unroll
        for (int u = 0; u < D; ++u) b[u] = X.load(e[u].col, q + u * STRIDE < q1);
#pragma unroll
        for (int u = 0; u < D; ++u) acc.fma(q + u * STRIDE < q1 ? e[u].val : 0.0f, b[u]);
    }
}

template <int LC, int VEC, bool OFF32>
__global__ __launch_bounds__(kBlock) void mttkrp_fibers_kernel(MttkrpArgs a, int block_slices, int64_t blocks,
                                                               int64_t blocks_per_xcd, int xcds)
{
    constexpr int TEAMS = kBlock / LC;
    __shared__ StagedEntry s_A[kMfEntries + kMfDepth];  // (read beyond the last entry, not used)
    __shared__ int32_t s_fk[kMfFibers];
    __shared__ int32_t s_ep[kMfFibers + 1];
    __shared__ int32_t s_fp[kMfSlices + 1];
    __shared__ int32_t s_start[TEAMS + 1];  // a team's first fiber, counted from the piece's
    __shared__ Vec<VEC> s_head[kBlock];     // what a team has of a slice that began in front of its fibers
    __shared__ int32_t s_ended[TEAMS];      // whether that slice ends there
    __shared__ Vec<VEC> s_carry[2][LC];     // of the slice that goes on in the next piece
    // (Phases of a piece compute what they need from the thread's number anew, through an opaque copy: the compiler would
    // hoist it all out of the loops over columns and pieces and hold half of the registers for it throughout the walk.)
    struct Place {
        int tid, team, chunk;
        __device__ __forceinline__ Place()
        {
            tid = threadIdx.x;
            asm volatile("" : "+v"(tid));
            team = tid / LC;
            chunk = tid % LC;
        }
    };
    struct Columns {
        bool ok;
        uint32_t first;  // of the VEC columns this lane holds
        __device__ __forceinline__ Columns(const Place& p, int64_t k0, int64_t J)
        {
            const uint32_t k = (uint32_t)k0 + p.chunk * VEC;  // J < 2^31
            ok = k < (uint32_t)J;
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

    for (int64_t k0 = 0; k0 < a.J; k0 += (int64_t)LC * VEC) {
        auto store = [&](int slice, const Columns& c, const Vec<VEC>& sum) {
            if (c.ok) store_vec_stream<VEC>(a.Y + (first_slice + slice) * a.J + c.first, sum);
        };
        {
            const Place p;
            const Columns c(p, k0, a.J);
            Vec<VEC> none;
            none.zero();
            for (int r = p.team; r < slices; r += TEAMS)
                if (s_fp[r] == s_fp[r + 1]) store(r, c, none);
        }

        int turn = 0;  // which of s_carry the piece takes over
        for (int32_t f0 = f_begin; f0 < f_end; turn ^= 1) {
            int32_t n = f_end - f0 < kMfFibers ? f_end - f0 : kMfFibers;  // fibers of the piece
            __syncthreads();  // the piece before is done with
            {
                const Place p;
#pragma unroll 2
                for (int i = p.tid; i <= n; i += kBlock) {
                    s_ep[i] = a.eptr[f0 + i];
                    if (i < n) s_fk[i] = a.fidx[f0 + i];
                }
            }
            __syncthreads();
            const int32_t e0 = __builtin_amdgcn_readfirstlane(s_ep[0]);
            if (s_ep[n] - e0 > kMfEntries) {
                const Place p;
                int fit = 0;
                for (int i = 0; i < n; i += kBlock) fit += __syncthreads_count(i + p.tid < n && s_ep[i + p.tid + 1] - e0 <= kMfEntries);
                n = fit;
            }
            n = __builtin_amdgcn_readfirstlane(n);
            if (n == 0) {
                // a fiber of more entries than there is room for: all teams together
                const Place p;
                const Columns c(p, k0, a.J);
                const MaskedRows<VEC, OFF32> x1(a.X1, a.K, a.J, c.first), x2(a.X2, a.L, a.J, c.first);
                const int32_t e1 = __builtin_amdgcn_readfirstlane(s_ep[1]);
                Vec<VEC> t;
                t.zero();
                for (int32_t base = e0; base < e1; base += kMfEntries) {
                    const int32_t cnt = e1 - base < kMfEntries ? e1 - base : kMfEntries;
                    __syncthreads();
                    stage_entries<4>(a.eidx + base, a.vals + base, (uint32_t)cnt, s_A);
                    __syncthreads();
                    masked_fma<VEC, TEAMS, 1>(t, s_A, (uint32_t)p.team, c.ok ? (uint32_t)cnt : 0u, x2);
                }
                s_head[p.tid] = t;
                __syncthreads();
                if (p.team == 0) {
#pragma unroll 1
                    for (int m = 1; m < TEAMS; ++m) {
                        const Vec<VEC> other = s_head[m * LC + p.chunk];
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
            const int32_t cnt = __builtin_amdgcn_readfirstlane(s_ep[n]) - e0;
            {
                const Place p;
                constexpr int U = 4;
                for (int q0 = p.tid; q0 < cnt; q0 += U * kBlock) {
                    StagedEntry e[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int q = q0 + u * kBlock;
                        if (q < cnt) {
                            e[u].col = load_stream(a.eidx + (e0 + q));
                            e[u].val = load_stream(a.vals + (e0 + q));
                        }
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u)
                        if (q0 + u * kBlock < cnt) s_A[q0 + u * kBlock] = e[u];
                }
                const int share = cnt > TEAMS ? (cnt + TEAMS - 1) / TEAMS : 1;
                const float per_share = __builtin_amdgcn_rcpf((float)share);
                auto team_of = [&](int32_t fiber) {  // (a division of numbers up to 2,048: exact)
                    const int t = (int)(((float)(s_ep[fiber] - e0) + 0.5f) * per_share);
                    return t < TEAMS ? t : TEAMS - 1;
                };
#pragma unroll 1
                for (int i = p.tid; i < n; i += kBlock) {
                    const int mine = team_of(i);
#pragma unroll 1
                    for (int t = i == 0 ? 0 : team_of(i - 1) + 1; t <= mine; ++t) s_start[t] = i;
                    if (i == n - 1)
#pragma unroll 1
                        for (int t = mine + 1; t <= TEAMS; ++t) s_start[t] = n;
                }
            }
            __syncthreads();

            const Place p;
            const Columns c(p, k0, a.J);
            Vec<VEC> sum;
            sum.zero();
            int slice = 0;
            bool goes_on = false;  // the slice that begins in this team's fibers goes on behind them
            {
                const int32_t mine_end = s_start[p.team + 1];
                int32_t f = s_start[p.team];
                bool head_ends = false;
                if (f < mine_end) {
                    const MaskedRows<VEC, OFF32> x1(a.X1, a.K, a.J, c.first), x2(a.X2, a.L, a.J, c.first);
                    slice = last_row_at_or_before(s_fp, 0, slices - 1, f0 + f);
                    bool whole = s_fp[slice] == f0 + f;
                    int32_t slice_end = s_fp[slice + 1] - f0;
                    do {
                        // the fiber's row of X1 is in flight while its entries are multiplied out
                        const Vec<VEC> x = x1.load(s_fk[f], c.ok);
                        Vec<VEC> t;
                        t.zero();
                        const uint32_t q0 = (uint32_t)(s_ep[f] - e0), q1 = (uint32_t)(s_ep[f + 1] - e0);
                        masked_fma<VEC, 1, kMfDepth>(t, s_A, q0, c.ok ? q1 : q0, x2);
#pragma unroll
                        for (int i = 0; i < VEC; ++i) sum.v[i] = __builtin_fmaf(x.v[i], t.v[i], sum.v[i]);
                        ++f;
                        if (f != slice_end) continue;
                        if (whole) {
                            store(slice, c, sum);
                        } else {
                            s_head[p.tid] = sum;
                            head_ends = true;
                        }
                        sum.zero();
                        whole = true;
                        if (f < mine_end) {
                            do slice_end = s_fp[++slice + 1] - f0;
                            while (slice_end == f);
                        }
                    } while (f < mine_end);
                    goes_on = f != slice_end && whole;
                    if (f != slice_end && !whole) s_head[p.tid] = sum;
                } else {
                    s_head[p.tid] = sum;
                }
                s_ended[p.team] = head_ends ? 1 : 0;
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
                bool ended = false;
#pragma unroll 1
                for (int t = round == 1 ? 0 : p.team + 1; t < TEAMS && !ended; ++t) {
                    const Vec<VEC> other = s_head[t * LC + p.chunk];
#pragma unroll
                    for (int i = 0; i < VEC; ++i) sum.v[i] += other.v[i];
                    ended = s_ended[t] != 0;
                }
                if (ended) store(slice, c, sum);
                else s_carry[turn ^ 1][p.chunk] = sum;
            }
            f0 += n;
        }
    }
}

namespace {

struct LaunchFibers {
    const MttkrpArgs& a;
    int block_slices, xcds;
    hipStream_t s;
    template <int G, int LC, int VEC>
    void operator()() const
    {
        const int64_t blocks = (a.I + block_slices - 1) / block_slices;
        const int64_t blocks_per_xcd = (blocks + xcds - 1) / xcds;
        const unsigned grid = (unsigned)(blocks_per_xcd * xcds);
        // every byte offset into X1 and X2 fits 32 bits and both factors of it fit 24 bits
        auto fits = [&](int64_t rows) { return rows <= (1 << 24) && a.J * 4 < (1 << 24) && rows * a.J * 4 <= 0xffffffffLL; };
        const bool off32 = fits(a.K) && fits(a.L);
        if (off32)
            hipLaunchKernelGGL((mttkrp_fibers_kernel<LC, VEC, true>), dim3(grid), dim3(kBlock), 0, s, a, block_slices, blocks,
                               blocks_per_xcd, xcds);
        else
            hipLaunchKernelGGL((mttkrp_fibers_kernel<LC, VEC, false>), dim3(grid), dim3(kBlock), 0, s, a, block_slices, blocks,
                               blocks_per_xcd, xcds);
    }
};

}  // namespace

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

hipError_t launch_mttkrp_fibers(const MttkrpArgs& a, int block_slices, int lc, int vec, int xcds, hipStream_t s)
{
    if (block_slices > kMfSlices) block_slices = kMfSlices;
    if ((a.I + block_slices - 1) / block_slices + xcds > 0x7ffffff0LL) return hipErrorInvalidValue;
    if (!dispatch_lc<1>(lc, vec, LaunchFibers{a, block_slices, xcds, s})) return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace sgap
