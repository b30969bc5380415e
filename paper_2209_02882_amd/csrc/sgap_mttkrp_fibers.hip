// MTTKRP on compressed sparse fibers with the slices as the unit of work, parallel strategy:
//     t[f,:]  = sum over the entries (l, v) of fiber f of  v * X2[l,:]
//     Y[i,:]  = sum over the fibers f of slice i of        X1[fidx[f],:] * t[f,:]
// A workgroup owns a block of consecutive slices and works through their fibers in pieces (one piece, as a rule) whose
// fibers and entries it brings into LDS with coalesced loads.  A team of lanes, four columns each, takes consecutive
// fibers of a piece, cut where the entries are about even, and goes through them at its own pace (sgap_flat.hpp) with the
// slice's sum in registers; it stores what begins and ends among them.  What a team has of a slice that began in front of
// it goes to LDS, where the team that has the slice's beginning adds it up in order: one plain store per slice, no atomics,
// the same result every time.  A slice that goes on in the next piece is carried over in LDS, and a fiber that a piece has
// no room for is the whole workgroup's.
//
// Bound by the gathers: of two factors of 8.4 MB 1.7 GB come from beyond the L2s, at 7.2 TB/s; small tensors by the chain
// of loads that a block is (pointers, fibers, entries, then a team's rows of X2).  With a group of lanes per slice, members
// m, m + G, ... of which take the slice's fibers (mttkrp_kernel), a third of the members have no fiber, each waits for the
// longest of its wavefront's, and every slice ends in a tree sum.  us, group per slice (G = 8) / this, slices x fibers of a slice x
// entries of a fiber in the mean: 262,144 x 8 x 8 J = 32 262 / 234, J = 16 196 / 160; 100,000 x 4 x 4 55.1 / 44.1, J = 64 98 / 80; 10,000 x 8 x 8 36.3 /
// 19.5; 100,000 x 2 x 2 31.9 / 18.8; 20,000 x 20 x 4 70.6 / 45.6; 3,000 x 60 x 8 292 / 52.
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
constexpr int kMfBatch = 64;      // tiles whose first fibers and slices are looked up at once
constexpr int kMfBlock = 16;      // slices of a block where the caller does not say how many entries there are

namespace {

template <int VEC>
struct MfShared {
    FlatShared<kMfEntries, kMfFibers> flat;  // its runs are fibers
    int32_t fk[kMfFibers];
    int32_t fp[kMfSlices + 1];  // first fibers of the slices at hand
    FlatHeads<VEC> heads;       // of slices
    Vec<VEC> carry[2][kWave];   // of the slice that goes on in the next piece
    int32_t cut;                // whether several teams have a part of one fiber
};

// The fibers [f_begin, f_end), slice number first_slice holding the first of them.
// SHARED_SLICES: of them the entries [e_begin, e_end), kMfEntries at most; a slice may have some outside, its sum is added into
// Y (which holds zeros), and slices without entries are left alone; cut_first, cut_last: the first fiber begins in front of
// them, the last one goes on behind them.  Else the block's slices are whole, `slices` of them, their
// pointers in fp, and every one is stored.
template <int VEC, bool OFF32, bool SHARED_SLICES>
__device__ __forceinline__ void mttkrp_block(const MttkrpArgs& a, MfShared<VEC>& sh, int lanes, int teams, int64_t first_slice,
                                             int slices, int32_t f_begin, int32_t f_end, int32_t e_begin, int32_t e_end,
                                             bool cut_first, bool cut_last)
{
    auto& s = sh.flat;
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

    for (int64_t k0 = 0; k0 < a.J; k0 += (int64_t)lanes * VEC) {
        int64_t base = first_slice;  // number of the slice that fp begins with
        auto store = [&](int slice, const Columns& c, const Vec<VEC>& sum) {
            if (c.ok) store_vec_stream<VEC>(a.Y + (base + slice) * a.J + c.first, sum);
        };
        // a sum that a slice outside has a part in
        auto add = [&](int slice, const FlatPlace& p, const Columns& c, Vec<VEC> sum) {
            const int64_t k = k0 + (int64_t)p.chunk * VEC;
            from_last_columns<VEC>(sum, (int)(k - c.first));
#pragma unroll
            for (int i = 0; i < VEC; ++i)
                if (c.ok && k + i < a.J) unsafeAtomicAdd(a.Y + (base + slice) * a.J + k + i, sum.v[i]);
        };
        if constexpr (!SHARED_SLICES) {
            const FlatPlace p(lanes);
            const Columns c(p, k0, a.J, teams);
            Vec<VEC> none;
            none.zero();
            for (int r = p.team; r < slices; r += teams)
                if (sh.fp[r] == sh.fp[r + 1]) store(r, c, none);
        }

        int turn = 0;  // which of s_carry the piece takes over
        for (int32_t f0 = f_begin; f0 < f_end; turn ^= 1) {
            auto next_piece = [&](int fibers) {
                f0 += fibers;
                if constexpr (SHARED_SLICES) {
                    if (f0 >= f_end) return;
                    base = sh.fp[slices] > f0 ? base + last_row_at_or_before(sh.fp, 0, slices - 1, f0)
                                             : last_row_at_or_before(a.fptr, (int32_t)(base + slices), (int32_t)a.I - 1, f0);
                }
            };
            int32_t n = f_end - f0 < kMfFibers ? f_end - f0 : kMfFibers;  // fibers of the piece
            __syncthreads();  // the piece before is done with
            {
                const FlatPlace p(lanes);
                if (p.tid == 0) sh.cut = 0;
#pragma unroll 2
                for (int i = p.tid; i <= n; i += kBlock) {
                    int32_t e = a.eptr[f0 + i];
                    if (SHARED_SLICES && e < e_begin) e = e_begin;
                    if (SHARED_SLICES && e > e_end) e = e_end;
                    s.ptr[i] = e;
                    if (i < n) sh.fk[i] = a.fidx[f0 + i];
                }
                if constexpr (SHARED_SLICES) {
                    slices = a.I - base < kMfSlices ? (int)(a.I - base) : kMfSlices;
                    // (a slice that begins or ends with a fiber that is not all here does so outside)
                    for (int i = p.tid; i <= slices; i += kBlock) {
                        const int32_t f = a.fptr[base + i];
                        sh.fp[i] = f + (cut_last && f == f_end ? 1 : 0) - (cut_first && f == f_begin ? 1 : 0);
                    }
                }
            }
            __syncthreads();
            if constexpr (SHARED_SLICES) {
                // the fibers of the slices at hand
                if (sh.fp[slices] - f0 < n) n = sh.fp[slices] - f0;
            }
            const int32_t e0 = __builtin_amdgcn_readfirstlane(s.ptr[0]);
            if (!SHARED_SLICES && s.ptr[n] - e0 > kMfEntries) {
                const FlatPlace p(lanes);
                int fit = 0;
                for (int i = 0; i < n; i += kBlock) fit += __syncthreads_count(i + p.tid < n && s.ptr[i + p.tid + 1] - e0 <= kMfEntries);
                n = fit;
            }
            n = __builtin_amdgcn_readfirstlane(n);
            if (!SHARED_SLICES && n == 0) {
                // a fiber of more entries than there is room for: all teams together
                const FlatPlace p(lanes);
                const Columns c(p, k0, a.J, teams);
                const MaskedRows<VEC, OFF32> x1(a.X1, a.J, c.first), x2(a.X2, a.J, c.first);
                const int32_t e1 = __builtin_amdgcn_readfirstlane(s.ptr[1]);
                Vec<VEC> t;
                t.zero();
                for (int32_t base = e0; base < e1; base += kMfEntries) {
                    const int32_t cnt = e1 - base < kMfEntries ? e1 - base : kMfEntries;
                    __syncthreads();
                    flat_stage<kMfEntries>(s.entry, a.eidx, a.vals, base, cnt, p.tid);
                    __syncthreads();
#pragma unroll 1
                    for (int q = p.team; c.ok && q < cnt; q += teams) t.fma(s.entry[q].val, x2.load(s.entry[q].col, true));
                }
                sh.heads.head[p.tid] = t;
                __syncthreads();
                if (p.team == 0) {
#pragma unroll 1
                    for (int m = 1; m < teams; ++m) {
                        const Vec<VEC> other = sh.heads.head[m * lanes + p.chunk];
#pragma unroll
                        for (int i = 0; i < VEC; ++i) t.v[i] += other.v[i];
                    }
                    const int slice = last_row_at_or_before(sh.fp, 0, slices - 1, f0);
                    const Vec<VEC> x = x1.load(sh.fk[0], c.ok);
                    Vec<VEC> sum;
                    sum.zero();
                    if (sh.fp[slice] < f0 && f0 > f_begin) sum = sh.carry[turn][p.chunk];
#pragma unroll
                    for (int i = 0; i < VEC; ++i) sum.v[i] = __builtin_fmaf(x.v[i], t.v[i], sum.v[i]);
                    if (sh.fp[slice + 1] == f0 + 1) store(slice, c, sum);
                    else sh.carry[turn ^ 1][p.chunk] = sum;
                }
                next_piece(1);
                continue;
            }

            // the piece's entries, and meanwhile where the teams begin
            const int32_t cnt = __builtin_amdgcn_readfirstlane(s.ptr[n]) - e0;
            {
                const FlatPlace p(lanes);
                flat_stage<kMfEntries>(s.entry, a.eidx, a.vals, e0, cnt, p.tid);
                if (flat_deal<true>(s, e0, cnt, n, teams, p.tid)) sh.cut = 1;
            }
            __syncthreads();

            // What a team has of the piece's fibers.  (Looked up again behind the walk, which has no registers left for it.)
            struct Share {
                int first, begun, finished, last;  // fibers from `begun` on begin here, those before `finished` end here
                int32_t from, to;                  // entries
                __device__ __forceinline__ Share(const FlatShared<kMfEntries, kMfFibers>& s, const FlatPlace& p, int teams, int32_t e0)
                {
                    first = begun = finished = last = from = to = 0;
                    if (p.team >= teams) return;
                    const uint32_t at = s.start[p.team], end = s.start[p.team + 1];
                    begun = first = at & 0xffff;
                    finished = last = end & 0xffff;
                    from = at >> 16, to = end >> 16;
                    begun += from > s.ptr[first] - e0 ? 1 : 0;
                    last += to > s.ptr[finished] - e0 ? 1 : 0;
                }
                __device__ __forceinline__ bool open() const { return last > finished && finished >= begun; }  // the last one begins here and goes on behind
            };
            Vec<VEC> sum, head, t, x;  // of the slice at hand; of one that began in front; of the fiber; X1's row
            std::conditional_t<SHARED_SLICES, FlatChain<VEC>, FlatFours<VEC>> fibers;  // of the slice at hand, while it is walked through
            fibers.zero();
            head.zero();
            int slice = 0;
            int32_t slice_end = 0;
            bool whole = false, head_ends = false;  // the slice at hand begins here; what is in head ends here
            {
                const FlatPlace p(lanes);
                const Columns c(p, k0, a.J, teams);
                const Share m(s, p, teams, e0);
                if (m.first < m.last) {
                    const MaskedRows<VEC, OFF32> x1(a.X1, a.J, c.first), x2(a.X2, a.J, c.first);
                    slice = last_row_at_or_before(sh.fp, 0, slices - 1, f0 + m.first);
                    whole = sh.fp[slice] == f0 + m.first && m.begun == m.first;
                    slice_end = sh.fp[slice + 1] - f0;
                    auto done = [&](int f, const Vec<VEC>& of_fiber) {
                        if (!SHARED_SLICES && f < m.begun) {
                            sh.heads.head[p.tid] = of_fiber;  // of a fiber that began in front
                            sh.heads.ended[p.team] = f < m.finished ? 1 : 0;
                        } else if (SHARED_SLICES || f < m.finished) {
                            fibers.add_product(x, of_fiber);
                        }
                        if (f + 1 != slice_end || f == m.finished) return;
                        sum = fibers.total();
                        if (whole) {
                            store(slice, c, sum);
                        } else if (SHARED_SLICES || f >= m.begun) {  // (else the team that has the fiber's beginning closes the slice)
                            head = sum;
                            head_ends = true;
                        }
                        fibers.zero();
                        whole = true;
                        if (f + 1 < m.last) {
                            do slice_end = sh.fp[++slice + 1] - f0;
                            while (slice_end == f + 1);
                        }
                    };
                    // (a stored fiber without entries has no part in a tile, as with every other kernel whose unit of work is the
                    // entry: whether the tile takes it up depends on where others end, and X1 may be infinite there)
                    auto ahead = [&](int f, bool ends, bool any) { x = x1.load(sh.fk[f], ends && c.ok && (any || !SHARED_SLICES)); };
                    t = flat_walk<VEC, OFF32, FlatChain<VEC>>(s, m.first, m.last, m.from, m.to, e0, x2, c.ok, ahead, done);
                    done(m.last - 1, t);
                }
            }
            sum = fibers.total();
            const FlatPlace p(lanes);
            const Columns c(p, k0, a.J, teams);
            bool goes_on = false;  // the slice that begins in this team's fibers goes on behind them
            const Share m(s, p, teams, e0);
            const bool begins_late = !SHARED_SLICES && m.begun > m.first, open = !SHARED_SLICES && m.open();
            // what the team has of the slice at hand, with all of its fibers in it
            auto rest = [&](bool ends) {
                if (!ends) {
                    goes_on = whole;
                    if (!whole) head = sum;
                } else if (whole) {
                    store(slice, c, sum);
                } else {
                    head = sum;
                    head_ends = true;
                }
            };
            if (!open && m.first < m.last && (m.last != slice_end || m.last > m.finished)) rest(false);
            auto put_head = [&] {
                sh.heads.head[p.tid] = head;
                if (p.team < teams) sh.heads.ended[p.team] = head_ends ? 1 : 0;
            };
            if (!begins_late && !open) put_head();
            __syncthreads();
            // A fiber that several teams share: its sum comes together before it is multiplied with its row of X1, as that of any
            // other does (parts of it may be zero, cancel or leave the range where the sum does not, and an infinity in X1 is to
            // meet the sum).  Not in a tile, which cuts fibers itself.
            if (!SHARED_SLICES && sh.cut != 0) {
                batch_heads(sh.heads, teams, lanes, p);
                __syncthreads();
                if (open) {
                    add_heads_in_chains<VEC, true>(t, sh.heads, p.team + 1, teams, lanes, p.chunk);
#pragma unroll
                    for (int i = 0; i < VEC; ++i) sum.v[i] = __builtin_fmaf(x.v[i], t.v[i], sum.v[i]);
                    rest(m.last == slice_end);
                }
                __syncthreads();
                if (begins_late || open) put_head();
                __syncthreads();
            }
            if constexpr (SHARED_SLICES) {
                batch_heads(sh.heads, teams, lanes, p);
                __syncthreads();
            }
            // what goes on is added up by the team that has its beginning, what came in from the piece before by the first team
            const bool look = SHARED_SLICES || f0 > f_begin;
            const int32_t came_in = look ? last_row_at_or_before(sh.fp, 0, slices - 1, f0) : 0;
            const bool comes_in = look && sh.fp[came_in] < f0;
#pragma unroll 1
            for (int round = 0; round < 2; ++round) {
                if (round == 1) {
                    goes_on = comes_in && p.team == 0;
                    sum.zero();
                    if (goes_on && f0 > f_begin) sum = sh.carry[turn][p.chunk];
                    slice = came_in;
                }
                if (!goes_on) continue;
                const int from = round == 1 ? 0 : p.team + 1;
                bool ended;
                if constexpr (SHARED_SLICES) ended = add_heads<VEC, true>(sum, sh.heads, from, teams, lanes, p.chunk);
                else ended = add_heads_in_chains<VEC, false>(sum, sh.heads, from, teams, lanes, p.chunk);
                if (SHARED_SLICES && (ended ? sh.fp[slice] < f_begin : f0 + n == f_end)) add(slice, p, c, sum);
                else if (ended) store(slice, c, sum);
                else sh.carry[turn ^ 1][p.chunk] = sum;
            }
            next_piece(n);
        }
    }
}

}  // namespace

template <int VEC, bool OFF32>
__global__ __launch_bounds__(kBlock) void mttkrp_fibers_kernel(MttkrpArgs a, int lanes, int block_slices,
                                                               int64_t blocks, int64_t blocks_per_xcd, int xcds)
{
    __shared__ MfShared<VEC> s;
    // workgroup b runs on die b % xcds: every die gets one contiguous run of blocks
    const int64_t block = (int64_t)(blockIdx.x % xcds) * blocks_per_xcd + blockIdx.x / xcds;
    if (block >= blocks) return;  // the whole workgroup
    const int64_t first_slice = block * block_slices;
    const int slices = (int)(a.I - first_slice < block_slices ? a.I - first_slice : block_slices);
    for (int i = threadIdx.x; i <= slices; i += kBlock) s.fp[i] = a.fptr[first_slice + i];
    __syncthreads();
    const int32_t f_begin = __builtin_amdgcn_readfirstlane(s.fp[0]);
    const int32_t f_end = __builtin_amdgcn_readfirstlane(s.fp[slices]);
    mttkrp_block<VEC, OFF32, false>(a, s, lanes, kBlock / lanes, first_slice, slices, f_begin, f_end, 0, 0, false, false);
}

// Stored entries as the unit of work, serial strategy: {<g nnz, c col>, 1}, whatever group_size says.  A workgroup takes tiles of
// entries, whose first and last fibers may go on outside, and works through them as through a block of slices; slices that go
// on outside are merged with atomics.
// Bound by the gathers too, where the factors do not fit an L2 (two of 8.4 MB, 262,144 slices and 34.8 M entries: 3.5 GB come from
// beyond the L2s in 0.50 ms, 6.9 TB/s).  With a lane to an even share of the entries (sgap_mttkrp_serial.hip, the form before) the lanes of a wavefront met at every ending of a fiber, two steps of three.
// us, even shares / this, one slice in a thousand of 2,000 to 20,000 fibers, the others of 4, J = 32 unless said: 262,144
// slices 542 / 455; 76,491 173 / 133; 20,000 63 / 57; 5,000 34 / 29; 15,510, J = 16 41.5 / 29.5; 100,000, J = 64 1,283 / 1,020
// and J = 256 2,490 / 1,775, J = 8 158 / 116, J = 4 161 / 116, J = 2 111 / 106, J = 1 95 / 96.  1,000 slices of two fibers of
// 1,000 entries each 41.7 / 34.1.
template <int VEC, bool OFF32>
__global__ __launch_bounds__(kBlock) void mttkrp_tiles_kernel(MttkrpArgs a, int lanes, int tile)
{
    __shared__ MfShared<VEC> s;
    __shared__ int32_t s_fiber[2 * kMfBatch], s_slice[kMfBatch];  // a tile's first and last fiber, the slice of the first
    __shared__ uint8_t s_cut[2 * kMfBatch];
    const int32_t F = a.fptr[a.I];
    const int32_t E = F > 0 ? a.eptr[F] : 0;
    const TileDeal deal(((int64_t)E + tile - 1) / tile, blockIdx.x, gridDim.x);
    const int mine = (int)deal.mine;
    for (int j0 = 0; j0 < mine; j0 += kMfBatch) {
        const int batch = mine - j0 < kMfBatch ? mine - j0 : kMfBatch;
        __syncthreads();  // the last ones are done with
        // the fibers of the tiles' first and last entries
        find_positions(a.eptr, F - 1, 2 * batch, [&](int j) {
            const int64_t at = (deal.tile(j0 + j / 2) + j % 2) * tile;
            return (int32_t)(at > E ? E : at) - j % 2;
        }, s_fiber);
        __syncthreads();
        // (whether those are cut, on the way)
        bool cut = false;
        if ((int)threadIdx.x < 2 * batch) {
            const int64_t at = (deal.tile(j0 + threadIdx.x / 2) + threadIdx.x % 2) * tile;
            const int32_t e = a.eptr[s_fiber[threadIdx.x] + threadIdx.x % 2];
            cut = threadIdx.x % 2 ? e > at : e < at;
        }
        find_positions(a.fptr, (int32_t)a.I - 1, batch, [&](int j) { return s_fiber[2 * j]; }, s_slice);
        if ((int)threadIdx.x < 2 * batch) s_cut[threadIdx.x] = cut;
        __syncthreads();
        for (int j = 0; j < batch; ++j) {
            const int32_t f_begin = __builtin_amdgcn_readfirstlane(s_fiber[2 * j]);
            const int32_t f_end = __builtin_amdgcn_readfirstlane(s_fiber[2 * j + 1]) + 1;
            const int32_t slice = __builtin_amdgcn_readfirstlane(s_slice[j]);
            const int64_t at = deal.tile(j0 + j) * tile;
            mttkrp_block<VEC, OFF32, true>(a, s, lanes, kBlock / lanes, slice, 0, f_begin, f_end, (int32_t)at,
                                           (int32_t)(at + tile < E ? at + tile : E), s_cut[2 * j], s_cut[2 * j + 1]);
        }
    }
}

// Blocks of even numbers of slices, as many as make whole rounds of the chip's resident workgroups: a tensor of 45,373 slices of
// 5 fibers, J = 24, takes 34.8 us in one round of 964 blocks and 43.1 in 1,286.  The larger a block the better, up to what
// leaves few blocks in more than one piece; with many rounds those count more than the rounds (2,600 entries a block / 2,000:
// 76,491 slices of 4 fibers, J = 32, two rounds 42.0 us / 46.2, 262,144 of 8, seven rounds or nine, 264 to 272 / 263).
static int mttkrp_block_slices(int64_t I, int64_t nnz_hint, int compute_units)
{
    if (nnz_hint <= 0) return kMfBlock;
    const int64_t resident = (int64_t)kMfResident * compute_units;
    int64_t rounds = nnz_hint / (resident * kMfMean) + 1;
    if (rounds >= kMfRounds) rounds = nnz_hint / (resident * 2000) + 1;
    const int64_t slices = (I + resident * rounds - 1) / (resident * rounds);
    return slices < kMfSlices ? (int)slices : kMfSlices;
}

// Where this is the kernel.  Teams of a lane or two share a slice that a group of lanes has by itself, and small tensors are over
// when a block has been dealt out; without a count of the entries blocks are small.  The fewer columns, the longer the slices
// have to be for the groups' idle and waiting members to cost more than that.  us, group per slice / this, G = 8 unless said,
// slices x fibers of a slice x entries of a fiber in the mean:
//   J = 100  100,000 x 1.2 x 8, G = 2 77 / 81, J = 64 44 / 42
//   J = 64   100,000 x 2 x 2 52.2 / 31.1, no count 52.3 / 56.6; 1,000 x 4 x 4 18.6 / 8.8
//   J = 32   30,000 x 2 x 2, G = 2 9.9 / 10.2; 1,000 x 4 x 4 10.5 / 10.2, J = 24 10.6 / 11.3; 10,000 x 4 x 4 13.4 / 11.1; no count, 100,000 x 2 x 2
//            32.0 / 45.8
//   J = 16   10,000 x 4 x 4 9.5 / 9.6; 100,000 x 2 x 2 22.0 / 14.3; 30,000 x 2 x 2, G = 2 7.2 / 8.9
//   J = 8    100,000 x 4 x 4 28.9 / 29.4, G = 2 30.3 / 32.1; 20,000 x 20 x 4 62 / 40, G = 32 35.2 / 36.0; 10,000 x 8 x 8, G = 32 13.0 / 14.4
//   J = 4    100,000 x 4 x 4 18.5 / 31.1; 20,000 x 20 x 4 59 / 51, G = 32 25 / 43; 3,000 x 60 x 8 284 / 64; 10,000 x 8 x 8, G = 32 9.6 / 19.0
bool mttkrp_fibers_apply(int64_t I, int64_t J, int group, int64_t nnz_hint)
{
    if (nnz_hint <= 0) return J >= 80;
    if (J >= 48) return group > 2 || nnz_hint >= 12 * I;
    if (J >= 20) return nnz_hint >= 150'000 || (J >= 32 && nnz_hint >= 12 * I);
    if (J >= 12) return nnz_hint >= 300'000;
    return nnz_hint >= 400'000 && nnz_hint / I >= 10 * group;
}

hipError_t launch_mttkrp_fibers(const MttkrpArgs& a, int vec, int xcds, int compute_units, int64_t nnz_hint, hipStream_t s)
{
    const int block_slices = mttkrp_block_slices(a.I, nnz_hint, compute_units);
    const int64_t blocks = (a.I + block_slices - 1) / block_slices;
    if (blocks + xcds > 0x7ffffff0LL) return hipErrorInvalidValue;
    const int64_t blocks_per_xcd = (blocks + xcds - 1) / xcds;
    const int64_t chunks = (a.J + vec - 1) / vec;
    const int lanes = chunks < kWave ? (int)chunks : kWave;
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)(blocks_per_xcd * xcds)), dim3(kBlock), 0, s, a, lanes, block_slices, blocks, blocks_per_xcd, xcds);
    };
    const bool off32 = offsets_fit_32(a.K, a.J) && offsets_fit_32(a.L, a.J);
    if (vec == 4) { if (off32) go(mttkrp_fibers_kernel<4, true>); else go(mttkrp_fibers_kernel<4, false>); }
    else if (vec == 2) { if (off32) go(mttkrp_fibers_kernel<2, true>); else go(mttkrp_fibers_kernel<2, false>); }
    else { if (off32) go(mttkrp_fibers_kernel<1, true>); else go(mttkrp_fibers_kernel<1, false>); }
    return hipGetLastError();
}

hipError_t launch_mttkrp_tiles(const MttkrpArgs& a, int vec, int compute_units, int64_t nnz_hint, hipStream_t s)
{
    const int64_t chunks = (a.J + vec - 1) / vec, resident = (int64_t)kMfResident * compute_units;
    const int lanes = chunks < kWave ? (int)chunks : kWave;
    // Tiles that make whole rounds of the resident workgroups, 2,000 entries at most.  At least 1,024, although few entries
    // would make more workgroups: each adds to the same few rows where slices are long (5,000 slices as above, J = 32: tiles
    // of 512 34.6 us, of 1,024 29; 10,000 slices of 4 fibers 21.1 and 22.6).  1,536 with four lanes to a team or fewer (20,000
    // slices as above, J = 4 44 and 37.6, J = 8 41.7 and 38; 5,000, J = 16 25 and 23).
    int64_t tile = 2000;
    if (nnz_hint > 0) {
        const int64_t rounds = nnz_hint / (resident * 2000) + 1;
        tile = (nnz_hint + resident * rounds - 1) / (resident * rounds);
        const int least = lanes <= 4 ? 1536 : 1024;
        if (tile < least) tile = least;
    }
    const int grid = persistent_grid(kMfResident, compute_units, nnz_hint, (int)tile);
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(grid), dim3(kBlock), 0, s, a, lanes, (int)tile); };
    const bool off32 = offsets_fit_32(a.K, a.J) && offsets_fit_32(a.L, a.J);
    if (vec == 4) { if (off32) go(mttkrp_tiles_kernel<4, true>); else go(mttkrp_tiles_kernel<4, false>); }
    else if (vec == 2) { if (off32) go(mttkrp_tiles_kernel<2, true>); else go(mttkrp_tiles_kernel<2, false>); }
    else { if (off32) go(mttkrp_tiles_kernel<1, true>); else go(mttkrp_tiles_kernel<1, false>); }
    return hipGetLastError();
}

}  // namespace sgap
