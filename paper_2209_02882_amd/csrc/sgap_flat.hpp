// Short runs of stored entries (rows of A, fibers of a tensor) by teams of lanes that go each at its own pace.
//
// A workgroup copies consecutive runs into LDS; a team takes consecutive runs, cut where the entries are about even, up to
// eight entries of one run at a time.  The next eight are the same run's or the next one's, whatever the other teams of the
// wavefront are at: where they all take a run each and meet before the next (a loop over a run's entries inside one over
// runs), they wait for the longest of eight at every turn.  The figures are beside the
// kernels (sgap_flat_rows.hip, sgap_mttkrp_fibers.hip, sgap_nnz_flat.hip).
//   lanes of a team   as many as the columns take, four each: nothing is handed from lane to lane, so that a team may lie
//                     anywhere in a workgroup
#pragma once
#include "sgap_common.hpp"
#include "sgap_gather.hpp"

#include <type_traits>

namespace sgap {

// Rows of a dense operand by number; `ok` = false reads as zeros, without a branch where byte offsets have 32 bits (an offset
// past the end of a buffer descriptor is not fetched).  The masked offset is the descriptor's end, with room for a load of 16
// bytes behind it: none of its words has an offset that wraps round to the operand's first ones.
template <int VEC, bool OFF32>
struct MaskedRows {
    __amdgpu_buffer_rsrc_t rows;
    uint32_t row_bytes, k_bytes;
    const float* base;
    int64_t J;
    // (The descriptor reaches as far as byte offsets of 32 bits may (kOffsets32End), not to the end of X: the number of X's rows
    // would have to be held for it, and row_split_kernel, with no scalar registers left, lost a wavefront per SIMD to that.)
    __device__ __forceinline__ MaskedRows(const float* X, int64_t j, uint32_t k)
        : rows(__builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(X), 0, (int)kOffsets32End, 0x00020000)), row_bytes((uint32_t)(j * 4)),
          k_bytes(k * 4), base(X + k), J(j)
    {
    }
    __device__ __forceinline__ Vec<VEC> load(int32_t row, bool ok) const
    {
        Vec<VEC> r;
        if constexpr (OFF32) {
            const uint32_t off = ok ? __umul24((uint32_t)row, row_bytes) + k_bytes : (uint32_t)kOffsets32End;
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

// Where a thread stands: computed anew in every phase through an opaque copy of its number, because the compiler would
// hoist what follows from it out of the loops over columns and pieces and hold it in registers throughout the walk.
struct FlatPlace {
    int tid, team, chunk;
    __device__ __forceinline__ explicit FlatPlace(int lanes)
    {
        tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        team = (int)(((float)tid + 0.5f) * __builtin_amdgcn_rcpf((float)lanes));  // (below 256 by up to 64: exact)
        chunk = tid - team * lanes;
    }
};

constexpr int kFlatBatch = 8;

// Which block of rows a workgroup takes: workgroup b runs on die b % xcds, and a die gets `pieces` contiguous runs of blocks, spread
// over the matrix (where long rows lie together, they are not all one die's).
struct FlatBlocks {
    int64_t blocks;
    int32_t xcds, run;  // blocks of a run
    FlatBlocks() = default;
    FlatBlocks(int64_t blocks_, int xcds_, int pieces) : blocks(blocks_), xcds(xcds_), run((int32_t)((blocks_ + (int64_t)xcds_ * pieces - 1) / ((int64_t)xcds_ * pieces))) {}
    int64_t grid() const
    {
        const int64_t round = (int64_t)xcds * run;
        return (blocks + round - 1) / round * round;
    }
    __device__ __forceinline__ int64_t at(uint32_t wg) const  // `blocks` or more: none
    {
        const uint32_t turn = wg / (uint32_t)xcds;
        return ((int64_t)(turn / (uint32_t)run) * xcds + wg % (uint32_t)xcds) * run + turn % (uint32_t)run;
    }
};

// ENTRIES and RUNS: the most of a piece.
template <int ENTRIES, int RUNS>
struct FlatShared {
    __attribute__((aligned(16))) StagedEntry entry[ENTRIES + kFlatBatch];  // (a batch reads past the last one)
    int32_t ptr[RUNS + 1];      // first entries of the piece's runs
    int32_t start[kBlock + 1];  // a team's first run
};

// The piece's entries [e0, e0 + cnt) on their way into LDS, four neighbours to a thread, all of them requested before the
// first is put down.  The caller synchronises.
template <int ENTRIES>
__device__ __forceinline__ void flat_stage(StagedEntry* __restrict__ entry, const int32_t* __restrict__ idx, const float* __restrict__ vals, int32_t e0,
                                           int32_t cnt, int tid)
{
    typedef int32_t native_i4 __attribute__((ext_vector_type(4), aligned(4)));
    constexpr int U = (ENTRIES + kBlock * 4 - 1) / (kBlock * 4);
    idx += e0;
    vals += e0;
    native_i4 c[U];
    native_f4 v[U];
    int32_t last_c = 0;
    float last_v = 0.0f;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int q = (u * kBlock + tid) * 4;
        if (q + 4 <= cnt) {
            c[u] = __builtin_nontemporal_load(reinterpret_cast<const native_i4*>(idx + q));
            v[u] = __builtin_nontemporal_load(reinterpret_cast<const native_f4*>(vals + q));
        }
    }
    const int rest = (cnt & ~3) + tid;  // the last one to three
    if (rest < cnt) {
        last_c = load_stream(idx + rest);
        last_v = load_stream(vals + rest);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int q = (u * kBlock + tid) * 4;
        if (q + 4 <= cnt) {
            entry[q] = {c[u].x, v[u].x};
            entry[q + 1] = {c[u].y, v[u].y};
            entry[q + 2] = {c[u].z, v[u].z};
            entry[q + 3] = {c[u].w, v[u].w};
        }
    }
    if (rest < cnt) entry[rest] = {last_c, last_v};
}

// Where the teams begin: with whole runs, at the first one that starts at or behind an even share of the work; CUT: inside a run
// where that is one of more than kFlatCut entries, and s.start is made of flat_at().  The caller synchronises.  Whether this
// thread cut a run.
// Work: a run costs a turn and what it does at its end, whatever it has, and kFlatRunCost entries more are about that.  us, even
// shares of the entries / of this: TTM, 21,755 fibers of 1 to 16, N = 64 18.2 / 17.3, 76,491 slices of four, N = 48 62.0 / 59.7;
// MTTKRP, 262,144 slices 241.0 / 238.4, 21,755 25.3 / 24.3; 100,000, J = 4, one in a thousand of 2,000 to 20,000 fibers 116 /
// 109; 100,000 with one fiber in a hundred of 500 entries 84.8 / 73.9.  (3 entries: between the two.)
// (A team may meet a run of any length: 20,000 slices of two fibers of 100 entries each, J = 32, 271 us by a lane group per
// slice, 49 by teams that share the fibers.  Shorter ones stay whole: a cut costs a turn, and a head to add up.)
constexpr int32_t kFlatCut = 32;
constexpr int32_t kFlatRunCost = 6;
__device__ __forceinline__ int32_t flat_at(int run, int32_t pos) { return run | pos << 16; }

template <bool CUT, typename SH>
__device__ __forceinline__ bool flat_deal(SH& s, int32_t e0, int32_t cnt, int n, int teams, int tid)
{
    const int32_t all = cnt + kFlatRunCost * n;
    const int32_t share = all > teams ? (all + teams - 1) / teams : 1;
    const float per_share = __builtin_amdgcn_rcpf((float)share);
    auto weight = [&](int run) { return s.ptr[run] - e0 + kFlatRunCost * run; };  // in front of it
    auto team_of = [&](int run) {  // (a division of numbers up to 2^14, up to 256 times as large: exact)
        const int t = (int)(((float)weight(run) + 0.5f) * per_share);
        return t < teams ? t : teams - 1;
    };
    bool cut = false;
    // the teams behind `from` up to `to`, whose share begins behind the beginning of run i - 1, at the latest with run i
    auto set = [&](int from, int to, int i) {
        int32_t pos = 0, before = 0, front = 0;
        if constexpr (CUT) {
            pos = s.ptr[i] - e0;
            before = i > 0 ? s.ptr[i - 1] - e0 : 0;
            front = before + kFlatRunCost * i;  // weight in front of the first entry of run i - 1
        }
#pragma unroll 1
        for (int t = from + 1; t <= to; ++t) {
            if constexpr (!CUT) {
                s.start[t] = i;
            } else {
                const int32_t at = t * share > front ? t * share - front : 0;  // of run i - 1's entries
                const bool inside = pos - before > kFlatCut && before + at < pos;
                s.start[t] = inside ? flat_at(i - 1, before + at) : flat_at(i, pos);
                cut = cut || (inside && at > 0);
            }
        }
    };
#pragma unroll 1
    for (int i = tid; i < n; i += kBlock) {
        const int mine = team_of(i);
        set(i == 0 ? -1 : team_of(i - 1), mine, i);
        if (i == n - 1) set(mine, teams, n);
    }
    return cut;
}

// The sum of a batch's products, four and four: one chain of additions as long as a team's share of a row had up to 1.7 times the
// error of the groups' trees and of their members' and lanes' short chains.
template <int VEC>
__device__ __forceinline__ Vec<VEC> flat_dot_half(const StagedEntry* e, const Vec<VEC>* b)
{
    Vec<VEC> sum;
#pragma unroll
    for (int i = 0; i < VEC; ++i) {
        float t = e[0].val * b[0].v[i];
#pragma unroll
        for (int u = 1; u < kFlatBatch / 2; ++u) t = __builtin_fmaf(e[u].val, b[u].v[i], t);
        sum.v[i] = t;
    }
    return sum;
}

template <int VEC>
__device__ __forceinline__ Vec<VEC> flat_dot(const StagedEntry (&e)[kFlatBatch], const Vec<VEC> (&b)[kFlatBatch])
{
    Vec<VEC> sum = flat_dot_half<VEC>(e, b);
    const Vec<VEC> high = flat_dot_half<VEC>(e + kFlatBatch / 2, b + kFlatBatch / 2);
#pragma unroll
    for (int i = 0; i < VEC; ++i) sum.v[i] += high.v[i];
    return sum;
}

// A sum in two chains that take turns: its error grows with the number of terms as that of two sums half as long.
template <int VEC>
struct FlatChains {
    Vec<VEC> turn, other;
    __device__ __forceinline__ void zero() { turn.zero(), other.zero(); }
    __device__ __forceinline__ void add(const Vec<VEC>& term)
    {
        const Vec<VEC> last = turn;
        turn = other;
#pragma unroll
        for (int i = 0; i < VEC; ++i) other.v[i] = last.v[i] + term.v[i];
    }
    __device__ __forceinline__ Vec<VEC> total() const
    {
        Vec<VEC> sum;
#pragma unroll
        for (int i = 0; i < VEC; ++i) sum.v[i] = turn.v[i] + other.v[i];
        return sum;
    }
};

template <int VEC>
struct FlatChain {
    Vec<VEC> sum;
    __device__ __forceinline__ void zero() { sum.zero(); }
    __device__ __forceinline__ void add(const Vec<VEC>& term)
    {
#pragma unroll
        for (int i = 0; i < VEC; ++i) sum.v[i] += term.v[i];
    }
    __device__ __forceinline__ void add_product(const Vec<VEC>& x, const Vec<VEC>& t)
    {
#pragma unroll
        for (int i = 0; i < VEC; ++i) sum.v[i] = __builtin_fmaf(x.v[i], t.v[i], sum.v[i]);
    }
    __device__ __forceinline__ Vec<VEC> total() const { return sum; }
};

// A sum of products in chains of four, whose sums are a chain.
template <int VEC>
struct FlatFours {
    Vec<VEC> four, before;
    int terms;
    __device__ __forceinline__ void zero() { four.zero(), before.zero(), terms = 0; }
    __device__ __forceinline__ void add_product(const Vec<VEC>& x, const Vec<VEC>& t)
    {
        const bool full = (++terms & 3) == 0;
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
            const float sum = __builtin_fmaf(x.v[i], t.v[i], four.v[i]);
            before.v[i] += full ? sum : 0.0f;
            four.v[i] = full ? 0.0f : sum;
        }
    }
    __device__ __forceinline__ Vec<VEC> total() const
    {
        Vec<VEC> sum;
#pragma unroll
        for (int i = 0; i < VEC; ++i) sum.v[i] = before.v[i] + four.v[i];
        return sum;
    }
};

// The runs [run, last), run < last, from entry q (of run `run`) on up to entry `stop`.  ahead(run, ok, any) is called before the last
// entries of a run are multiplied (ok; else before others; any: there are such), done(run, sum) when they are and another
// run follows; the last one's sum is returned (what a caller keeps of it then needs no registers meanwhile).
// SUM: how the batches of a run are added up.
template <int VEC, bool OFF32, typename SUM, typename SH, typename AHEAD, typename DONE>
__device__ __forceinline__ Vec<VEC> flat_walk(const SH& s, int run, int last, int32_t q, int32_t stop, int32_t e0,
                                              const MaskedRows<VEC, OFF32>& X, bool k_ok, AHEAD&& ahead, DONE&& done)
{
    constexpr int D = kFlatBatch;
    SUM all;
    all.zero();
    auto end_of = [&](int r) {
        const int32_t e = s.ptr[r + 1 <= last ? r + 1 : last] - e0;
        return e < stop ? e : stop;
    };
    int32_t end = end_of(run);
#pragma unroll 1
    do {
        StagedEntry e[D];
        Vec<VEC> b[D];
        const int32_t left = k_ok ? end - q : 0;
#pragma unroll
        for (int u = 0; u < D; ++u) e[u] = s.entry[q + u];
#pragma unroll
        for (int u = 0; u < D; ++u) {
            b[u] = X.load(e[u].col, u < left);
            if (u >= left) e[u].val = 0.0f;
        }
        const bool ends = end - q <= D;
        ahead(run, ends, left > 0);
        const int now = run;
        if (ends) {
            ++run;
            q = end;
            end = end_of(run);
        } else {
            q += D;
        }
        all.add(flat_dot<VEC>(e, b));
        if (ends && run < last) {
            done(now, all.total());
            all.zero();
        }
    } while (run < last);
    return all.total();
}

// What teams have of runs that began in front of them.
template <int VEC>
struct FlatHeads {
    static constexpr int kTeams = 8;  // to a batch
    Vec<VEC> head[kBlock];
    uint8_t ended[kBlock];            // whether the run ends there
    // Batches of teams, summed by a team each: where all teams of a tile are at one run, the first of them otherwise waits for
    // one LDS read after the other.  MTTKRP by tiles, 100,000 slices, one in a thousand of 2,000 to 20,000 fibers, us without /
    // with: J = 4 185 / 115, J = 1 117 / 96; 15,510 slices, J = 16 31.5 / 29.
    Vec<VEC> batch[kBlock / kTeams];
    uint8_t batch_ended[kBlock / kTeams];
};

// The caller synchronises in front of it and behind it.
template <int VEC>
__device__ __forceinline__ void batch_heads(FlatHeads<VEC>& s, int teams, int lanes, const FlatPlace& p)
{
    constexpr int T = FlatHeads<VEC>::kTeams;
    if (p.team < teams / T) {
        Vec<VEC> sum;
        sum.zero();
        int any = 0;
#pragma unroll
        for (int j = 0; j < T; ++j) {
            const int t = p.team * T + j;
            any |= s.ended[t];
            const Vec<VEC> other = s.head[t * lanes + p.chunk];
#pragma unroll
            for (int i = 0; i < VEC; ++i) sum.v[i] += other.v[i];
        }
        s.batch[p.team * lanes + p.chunk] = sum;
        s.batch_ended[p.team] = any;
    }
}

// What the teams from number `from` on have of a run that began in front of them, added to sum in order, up to the one where it
// ends; whether it does.
template <int VEC, bool BATCHES>
__device__ __forceinline__ bool add_heads(Vec<VEC>& sum, const FlatHeads<VEC>& s, int from, int teams, int lanes, int chunk)
{
    constexpr int T = FlatHeads<VEC>::kTeams;
    int t = from;
    bool done = false;
    auto single = [&](int until) {
#pragma unroll 1
        for (; t < until && !done; ++t) {
            const Vec<VEC> other = s.head[t * lanes + chunk];
#pragma unroll
            for (int i = 0; i < VEC; ++i) sum.v[i] += other.v[i];
            done = s.ended[t] != 0;
        }
    };
    if constexpr (BATCHES) {
        const int next = (from + T - 1) & ~(T - 1);
        single(next < teams ? next : teams);
#pragma unroll 1
        for (bool all = !done; all && t + T <= teams;) {
            const Vec<VEC> other = s.batch[t / T * lanes + chunk];
            all = s.batch_ended[t / T] == 0;
#pragma unroll
            for (int i = 0; i < VEC; ++i) sum.v[i] += all ? other.v[i] : 0.0f;
            t += all ? T : 0;
        }
    }
    single(teams);
    return done;
}

// The same with two chains that take turns, for what was a tree.
template <int VEC, bool BATCHES>
__device__ __forceinline__ bool add_heads_in_chains(Vec<VEC>& sum, const FlatHeads<VEC>& s, int from, int teams, int lanes, int chunk)
{
    constexpr int T = FlatHeads<VEC>::kTeams;
    FlatChains<VEC> all;
    all.zero();
    all.add(sum);
    int t = from;
    bool done = false;
#pragma unroll 1
    while (t < teams && !done) {
        const bool eight = BATCHES && t % T == 0 && t + T <= teams && s.batch_ended[t / T] == 0;
        const Vec<VEC> other = eight ? s.batch[t / T * lanes + chunk] : s.head[t * lanes + chunk];
        done = !eight && s.ended[t] != 0;
        all.add(other);
        t += eight ? T : 1;
    }
    sum = all.total();
    return done;
}

}  // namespace sgap
