// SDDMM on long rows whose windows of X2T lie in LDS: the teams, slots, windows and shares of sgap_panels_lds.hpp, with the
// sum over the columns inside.  A window's 64-column tiles come into LDS one after the other, and what a slot has in the
// window (up to 32 entries of each team) is multiplied with the row of X1 tile by tile; the entries' sums so far stay in
// two registers per slot, and leave as they get the last tile's part: one writer per entry, no atomics.
//   entries  lane i of a team looks after the entries i and 16 + i at the slot's position
//   dots     a team has 16 partial sums of four columns for every entry; four entries are folded to a quarter of the team
//            each in 6 vector instructions, and the quarters of sixteen are added up in 10 (dots_fold, dots_pair)
//   X1       16 bytes per lane and slot, requested two slots ahead like the entries
// The first tile's pass looks up what belongs to the window (dots_find); the others know how many entries there are and let
// the rest of their lanes add up what nobody asks for, in front of rows that exist.
//
// Bound by the vector instructions: on the skewed matrix (500,000 rows, 5,000 long ones with 55 M entries, J = 256) 717 M of
// them, 2.8 M clocks of a SIMD of 3.3 M (1.6 to 1.7 ms; the owner wavefronts that gather through the L2 took 2.28 ms, the call
// 2.73 ms and now 1.98 ms).  A third are the products that the entries ask for, as many what four rows differ by in a
// window and the adding up over lanes, a sixth the addresses, the rest what a slot costs.  7.7 GB come from beyond the L2s:
// a row of X1 is read again in every window.  Looking entries up in every
// tile and eight-entry sums of 18 instructions were 833 M (1.84 ms); the next window's first tile on its way while the
// entries leave gave nothing.
#pragma once
#include "sgap_panels_lds.hpp"

namespace sgap {

struct DotsShared {
    __attribute__((aligned(16))) float b[(kDotsWindow + 1) * kLdsCols];
    uint32_t end[kLdsWaves * kLdsTeams * kLdsSlots];  // of the slots' shares, as byte offsets of entries
    int32_t row[kLdsWaves * kLdsTeams * kLdsSlots];   // of the slots
};
static_assert(sizeof(DotsShared) <= 160 * 1024, "of a compute unit");

// What a lane wants next of a slot: its two entries' columns and its four columns of the row of X1.
struct DotsAhead {
    int32_t col[2];
    Vec<4> x1;
};

// The four sums v over a team's sixteen lanes, half way: lane 4 q + m gets the m-th quarter of the sum of v[q].  (The no-ops:
// wait states between a write and its DPP read, which the compiler does not see inside this text; v may just have been written.)
__device__ __forceinline__ float dots_fold(float (&v)[4])
{
    asm volatile("s_nop 1\n\t"
                 "v_add_f32_dpp %0, %0, %0 row_shl:8 row_mask:0xf bank_mask:0x3\n\t"
                 "v_add_f32_dpp %0, %2, %2 row_shr:8 row_mask:0xf bank_mask:0xc\n\t"
                 "v_add_f32_dpp %1, %1, %1 row_shl:8 row_mask:0xf bank_mask:0x3\n\t"
                 "v_add_f32_dpp %1, %3, %3 row_shr:8 row_mask:0xf bank_mask:0xc\n\t"
                 "v_add_f32_dpp %0, %0, %0 row_shl:4 row_mask:0xf bank_mask:0x5\n\t"
                 "s_nop 0\n\t"
                 "v_add_f32_dpp %0, %1, %1 row_shr:4 row_mask:0xf bank_mask:0xa\n\t"
                 "s_nop 1"
                 : "+&v"(v[0]), "+&v"(v[1])
                 : "v"(v[2]), "v"(v[3]));
    return v[0];
}

// Lanes with bit S of their number clear: a of this lane and of its neighbour at distance S (1 or 2), else b of the two.
template <int S>
__device__ __forceinline__ float dots_pair(float a, float b)
{
    constexpr unsigned long long kSet = S == 2 ? 0xCCCCCCCCCCCCCCCCull : 0xAAAAAAAAAAAAAAAAull;
    const bool set = __builtin_amdgcn_inverse_ballot_w64(kSet);
    const float keep = set ? b : a;
    const float give = set ? a : b;
    const int came = __builtin_amdgcn_update_dpp(0, __float_as_int(give), S == 2 ? 0x4E : 0xB1, 0xF, 0xF, true);
    return keep + __int_as_float(came);
}

// What a lane gets in the end: lane 4 q + m has the entry 4 m + q of sixteen.
__device__ __forceinline__ int dots_entry(int member) { return member % 4 * 4 + member / 4; }

// val * (sum + last) with one rounding fewer, of the two largest: adding up the tiles one after the other costs one more than
// the tree over all columns that the gathering kernels have.
__device__ __forceinline__ float dots_result(float val, float sum, float last)
{
    const float result = __builtin_fmaf(val, last, val * sum);
    return __builtin_isfinite(result) ? result : val * (sum + last);
}

// A slot's entries in the window that a window's first tile looks up for the others.
struct DotsFound {
    unsigned long long taken[2];  // lanes whose entry i is one of the window's
    uint32_t most;                // entries of the team with the most
    bool full;                    // a team has taken all 32 and may have more
    unsigned long long odd;       // lanes that show that a team's are not the first ones (columns that are not sorted)
};

// over as for lds_slot.
__device__ __forceinline__ DotsFound dots_find(const uint32_t (&at)[2], int32_t over, const LdsWindow& w, const LdsLanes& l)
{
    constexpr unsigned long long kFirst = 0x0001000100010001ull;
    DotsFound f;
#pragma unroll
    for (int i = 0; i < 2; ++i)
        f.taken[i] = __ballot(at[i] < w.bytes) & __ballot(over < -(int32_t)(l.member8 / 2) - 4 * kLdsTeam * i);
    const unsigned long long gaps = ((f.taken[0] & ~(f.taken[0] << 1)) | (f.taken[1] & ~(f.taken[1] << 1))) & ~kFirst;
    const unsigned long long late = f.taken[1] & kFirst & ~(f.taken[0] >> (kLdsTeam - 1));
    f.odd = gaps | late;
    f.full = (f.taken[1] >> (kLdsTeam - 1) & kFirst) != 0;
    f.most = 0;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const uint32_t both = (uint32_t)f.taken[i] | (uint32_t)(f.taken[i] >> 32);
        f.most += (uint32_t)__popc((both | both >> 16) & 0xFFFFu);
    }
    return f;
}

// Four entries' products with the lane's four columns, entry Q and on of the sixteen that off has the places in LDS of.
struct DotsRows {
    lds_f4 t[4];
};
template <int Q>
__device__ __forceinline__ DotsRows dots_read(lds_bytes mine, int32_t off)
{
    DotsRows rows;
    lds_each<4>([&](auto J) {
        constexpr int j = decltype(J)::value;
        rows.t[j] = *(const __attribute__((address_space(3))) lds_f4*)(mine + team_bcast<Q + j>(off));
    });
    return rows;
}
__device__ __forceinline__ float dots_four(const DotsRows& rows, const Vec<4>& x1, bool edge, bool own)
{
    float v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        v[j] = x1.v[0] * rows.t[j].x;
        v[j] = __builtin_fmaf(x1.v[1], rows.t[j].y, v[j]);
        v[j] = __builtin_fmaf(x1.v[2], rows.t[j].z, v[j]);
        v[j] = __builtin_fmaf(x1.v[3], rows.t[j].w, v[j]);
    }
    if (edge) {  // lanes without columns
        asm volatile("" : "+v"(v[0]));  // (a branch: this is most often left out)
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = own ? v[j] : 0.0f;
    }
    return dots_fold(v);
}

// One tile's part of the dot products of sixteen entries, of which the first `most` are looked at (what the lanes of others
// get is nothing, and not used).
__device__ __forceinline__ float dots_sixteen(lds_bytes mine, const Vec<4>& x1, int32_t off, int32_t most, bool edge, bool own)
{
    float quarter[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) asm volatile("" : "=v"(quarter[j]));
    lds_each<2>([&](auto H) {
        constexpr int h = decltype(H)::value * 2;
        if (most > h * 4) {
            const DotsRows rows = dots_read<h * 4>(mine, off);
            if (most > h * 4 + 4) quarter[h + 1] = dots_four(dots_read<h * 4 + 4>(mine, off), x1, edge, own);
            quarter[h] = dots_four(rows, x1, edge, own);
        }
    });
    return dots_pair<1>(dots_pair<2>(quarter[0], quarter[2]), dots_pair<2>(quarter[1], quarter[3]));
}

// The rest of a slot in front of column c1 and from memory: up to sixteen entries of every team at a time,
// the rows of X2T for four of each on their way together (one at a time, each entry waited for its column, its row and its
// sum in turn: 500,000 rows, the 55 M entries of the 5,000 long ones without order, J = 256: 165 ms; 50).
__device__ __forceinline__ uint32_t dots_rest(const LdsMatrix& matrix, const float* __restrict__ X1_row,
                                              const float* __restrict__ X2T, float* __restrict__ out, int64_t J, uint32_t p,
                                              uint32_t end, int32_t c1, const LdsLanes& l)
{
    const int member = LdsThread().member;
    for (;;) {
        const uint32_t at = p + l.member8 / 2;
        const int32_t col = (int32_t)__builtin_amdgcn_raw_buffer_load_b32(matrix.cols, (int)at, 0, 0);
        const int32_t val = (int32_t)__builtin_amdgcn_raw_buffer_load_b32(matrix.vals, (int)at, 0, 0);
        // (the bits past a field's sixteenth are zero)
        const int taken = __ffs((int)~team_field(__ballot(at < end && col < c1), l)) - 1;
#pragma unroll 1
        for (int j = 0; __any(j < taken); j += 4) {
            int32_t c[4];
            float sum[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                c[u] = __shfl(col, (j + u) % kLdsTeam, kLdsTeam);
                sum[u] = 0.0f;
            }
            if (j < taken) {
#pragma unroll 1
                for (int32_t k = member * 4; k < (int32_t)J; k += kLdsCols) {
                    const Vec<4> a = load_vec<4>(X1_row + k);
                    Vec<4> b[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        b[u].zero();
                        if (j + u < taken) b[u] = load_vec<4>(X2T + (int64_t)c[u] * J + k);
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u)
#pragma unroll
                        for (int i = 0; i < 4; ++i) sum[u] = __builtin_fmaf(a.v[i], b[u].v[i], sum[u]);
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
#pragma unroll
                for (int m = 1; m < kLdsTeam; m *= 2) sum[u] += __shfl_xor(sum[u], m, kLdsTeam);
                if (member == (j + u) % kLdsTeam && j + u < taken) out[at / 4] = __int_as_float(val) * sum[u];
            }
        }
        p += (uint32_t)taken * 4;
        if (!__any(taken == kLdsTeam)) return p;
    }
}

// A workgroup of kLdsBlock threads that has its compute unit to itself.
__device__ __forceinline__ void panel_lds_dots(const int32_t* __restrict__ colidx, const float* __restrict__ vals,
                                               const float* __restrict__ X1, const float* __restrict__ X2T,
                                               float* __restrict__ out, const PanelView& scr, int64_t K, int64_t J,
                                               const LdsArgs& args, uint32_t wave, DotsShared& shared)
{
    constexpr int R = kLdsSlots;
    const uint32_t n = scr.head->count;
    const LdsPlan plan = scr.head->lds;
    const LdsMatrix matrix(colidx, vals, scr.head->nnz);
    const __amdgpu_buffer_rsrc_t results = __builtin_amdgcn_make_buffer_rsrc(out, 0, (int)(scr.head->nnz * 4), 0x00020000);
    const uint32_t die = blockIdx.x % args.dies;
    LdsLanes l;
    lds_bytes mine;
    uint32_t* end_of;
    int32_t* row_of;
    {
        const LdsThread t;
        l.member8 = (uint32_t)t.member * 8;
        l.shift = t.team % 2 * kLdsTeam;
        l.high = t.team >= 2;
        mine = (lds_bytes)shared.b + t.member * 16;
        end_of = shared.end + (wave * kLdsTeams + t.team) * R;
        row_of = shared.row + (wave * kLdsTeams + t.team) * R;
        if (wave == 0) shared.b[kDotsWindow * kLdsCols + t.lane] = 0.0f;
    }
    const uint32_t member4 = l.member8 / 2;
    const int32_t entry = dots_entry((int)(l.member8 / 8));
    const uint32_t row_bytes = (uint32_t)J * 4;
    const uint32_t jobs = plan.groups * plan.per_die;
    const uint32_t shares = plan.per_die * args.dies;
    for (uint32_t job = blockIdx.x / args.dies; job < jobs; job += args.workgroups) {
        const uint32_t share = die * plan.per_die + job / plan.groups;
        const uint32_t group = job % plan.groups;
        const int64_t share_begin = (int64_t)share * plan.share_cols;
        if (share_begin >= K) continue;
        const int32_t share_end = (int32_t)(K - share_begin < plan.share_cols ? K : share_begin + plan.share_cols);
        int32_t pos[2] = {0, 0};  // lane i of a team: where slots i and 16 + i stand, as byte offsets
        {
            const LdsThread t;
            const uint32_t units = kLdsWaves * plan.groups;
            const uint32_t me = group * kLdsWaves + wave;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint32_t slot = (uint32_t)(h * kLdsTeam + t.member);
                const uint32_t q = (slot * units + (slot & 1 ? units - 1 - me : me)) * kLdsTeams + (uint32_t)t.team;
                uint32_t end = 0;
                int32_t row = 0;
                if (slot < plan.slots && q < n) {
                    const int32_t i = scr.order[q];
                    const int64_t at = (int64_t)i * (shares + 1) + share;
                    pos[h] = scr.ptr[at] * 4;
                    end = (uint32_t)scr.ptr[at + 1] * 4;
                    row = scr.rows[i];
                }
                if (slot < R) {  // (read by this wavefront alone)
                    end_of[slot] = end;
                    row_of[slot] = row;
                }
            }
        }
        const int32_t count = (share_end - (int32_t)share_begin + plan.window - 1) / plan.window;  // windows
        const int32_t width = (share_end - (int32_t)share_begin + count - 1) / count;
        for (int32_t w = 0; w < count; ++w) {
            const int32_t c0 = (int32_t)share_begin + w * width;
            const int32_t cols = share_end - c0 < width ? share_end - c0 : width;
            LdsWindow window{0u - (uint32_t)c0 * kLdsRowBytes, (uint32_t)cols * kLdsRowBytes};
            asm volatile("" : "+s"(window.minus_first));
            float sum[R][2];
#pragma unroll
            for (int r = 0; r < R; ++r) sum[r][0] = sum[r][1] = 0.0f;
            int32_t taken[2] = {0, 0};  // as pos: entries that the slot has taken in this window
            int32_t most = 0;           // lane r: the most that a team has taken for slot r
            uint32_t open = 0;          // slots for dots_rest
            auto pass = [&](uint32_t tile, auto Last) {
                constexpr bool last = decltype(Last)::value;
                const int32_t tile_k = (int32_t)(tile * plan.tile_cols);
                const LdsThread t;
                const int64_t k = lds_columns(tile_k, t, J);
                const bool own = tile_k + t.member * 4 < J && t.member * 4 < (int)plan.tile_cols;
                const bool edge = plan.tile_cols < kLdsCols || tile_k + kLdsCols > J;
                const char* const X1_k = (const char*)(X1 + k);
                auto ask = [&](auto I) {
                    constexpr int r = decltype(I)::value;
                    DotsAhead a;
                    const uint32_t at = (uint32_t)team_bcast<r % kLdsTeam>(pos[r / kLdsTeam]) + member4;
                    a.col[0] = (int32_t)__builtin_amdgcn_raw_buffer_load_b32(matrix.cols, (int)at, 0, 0);
                    a.col[1] = (int32_t)__builtin_amdgcn_raw_buffer_load_b32(matrix.cols, (int)at, 4 * kLdsTeam, 0);
                    a.x1 = load_vec<4>((const float*)(X1_k + (uint64_t)(uint32_t)row_of[r] * row_bytes));
                    return a;
                };
                DotsAhead held[2] = {ask(std::integral_constant<int, 0>{}), ask(std::integral_constant<int, 1>{})};
                uint32_t next_end = end_of[0];
                __syncthreads();  // everyone is done with the tile before
                for (int32_t i = (int32_t)wave * kLdsTeams; i < cols; i += kLdsWaves * kLdsTeams) {
                    const int32_t row = i + t.team < cols ? i + t.team : cols - 1;
                    const float* from = X2T + (int64_t)(c0 + row) * J + k;
                    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)from,
                                                     (__attribute__((address_space(3))) void*)(shared.b + i * kLdsCols), 16, 0, 0);
                }
                __builtin_amdgcn_s_waitcnt(kLdsNoLoads);
                __syncthreads();
                const bool first = tile == 0;
                lds_each<R>([&](auto I) {
                    constexpr int r = decltype(I)::value, ahead = (r + 2) % R;
                    if constexpr (r % (R / 4) == 0) __builtin_amdgcn_s_setprio(3 - r / (R / 4));  // (see panel_lds_rows)
                    DotsAhead e = held[0];
                    held[0] = held[1];
                    const uint32_t end = next_end;
                    next_end = end_of[(r + 1) % R];
                    const int p = team_bcast<r % kLdsTeam>(pos[r / kLdsTeam]) + entry * 4;
                    float val[2] = {0.0f, 0.0f};
                    if constexpr (last)
#pragma unroll
                        for (int i = 0; i < 2; ++i)
                            val[i] = __int_as_float((int)__builtin_amdgcn_raw_buffer_load_b32(matrix.vals, p, i * 4 * kLdsTeam, 0));
                    if constexpr (ahead > 1) held[1] = ask(std::integral_constant<int, ahead>{});
                    asm volatile("" : "+v"(e.col[0]), "+v"(e.col[1]));  // (waits for them here, not in front of the loads above)
                    const uint32_t at[2] = {((uint32_t)e.col[0] << 8) + window.minus_first,
                                            ((uint32_t)e.col[1] << 8) + window.minus_first};
                    if (first) {
                        // (this way round: see panel_lds_rows)
                        const int32_t over = team_bcast<r % kLdsTeam>(pos[r / kLdsTeam]) - (int32_t)end;
                        const DotsFound f = dots_find(at, over, window, l);
                        most = __builtin_amdgcn_inverse_ballot_w64(1ull << r) ? (int32_t)f.most : most;
                        int32_t here = __popc(team_field(f.taken[0], l)) + __popc(team_field(f.taken[1], l));
                        // (such a team takes none, and the others what they have: how a row's sums are made does not depend on
                        // the rows beside it)
                        if (f.odd && team_field(f.odd, l)) here = 0;
                        taken[r / kLdsTeam] = __builtin_amdgcn_inverse_ballot_w64(0x0001000100010001ull << (r % kLdsTeam)) ? here : taken[r / kLdsTeam];
                        if (f.full || f.odd != 0) open |= 1u << r;
                        open = (uint32_t)__builtin_amdgcn_readfirstlane((int)open);
                        asm volatile("" : "+s"(open));
                    }
                    // what lies outside the window, or belongs to another row, is in front of some row of it or of the zeros:
                    // those sums are not used
                    constexpr uint32_t kPast = kDotsWindow * kLdsRowBytes;
                    const int32_t off[2] = {(int32_t)(at[0] < kPast ? at[0] : kPast), (int32_t)(at[1] < kPast ? at[1] : kPast)};
                    const int32_t many = __builtin_amdgcn_readlane(most, r);
                    float part[2];
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        asm volatile("" : "=v"(part[i]));
                        if (many > kLdsTeam * i) part[i] = dots_sixteen(mine, e.x1, off[i], many - kLdsTeam * i, edge, own);
                    }
                    if constexpr (last) {
                        const int32_t here = team_bcast<r % kLdsTeam>(taken[r / kLdsTeam]);
#pragma unroll
                        for (int i = 0; i < 2; ++i) {
                            const int to = entry + i * kLdsTeam < here ? p : (int)0x80000000;  // (past the end: not stored)
                            __builtin_amdgcn_raw_buffer_store_b32((uint32_t)__float_as_int(dots_result(val[i], sum[r][i], part[i])),
                                                                  results, to, i * 4 * kLdsTeam, 0);
                        }
                    } else {
                        sum[r][0] += part[0];
                        sum[r][1] += part[1];
                    }
                    asm volatile("" : "+v"(sum[r][0]), "+v"(sum[r][1]));  // (now: not all slots' together at the end)
                });
            };
            // (A pass of its own: were this a branch in the slot, every wait for the loads under way would reckon with both ways.
            // Neither pass stays in the instruction cache, one is as good as the other.)
            for (uint32_t tile = 0; tile + 1 < plan.tiles; ++tile) pass(tile, std::false_type{});
            pass(plan.tiles - 1, std::true_type{});
            const LdsThread t;
            pos[0] += taken[0] * 4;
            pos[1] += taken[1] * 4;
            const bool final = w + 1 == count;  // of the share: takes all that is left (of rows that are not sorted)
            if (final) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int slot = h * kLdsTeam + t.member;
                    const unsigned long long some = __ballot(slot < R && (uint32_t)pos[h] < end_of[slot < R ? slot : 0]);
                    open |= (uint32_t)((some | some >> 16 | some >> 32 | some >> 48) & 0xFFFFu) << (h * kLdsTeam);
                }
            }
            while (open) {
                const uint32_t r = (uint32_t)__ffs((int)open) - 1u;
                open &= open - 1u;
                const bool upper = r >= kLdsTeam;
                const uint32_t p = (uint32_t)__shfl(upper ? pos[1] : pos[0], (int)(r % kLdsTeam), kLdsTeam);
                // The teams that have more to do here, each by its own row (else which entries come out of LDS, and with that
                // the rounding, would depend on the rows beside it): those that took all 32, and those that took none of
                // the window's.
                const int32_t took = __shfl(upper ? taken[1] : taken[0], (int)(r % kLdsTeam), kLdsTeam);
                bool more = final || took == 2 * kLdsTeam;
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const uint32_t at = p + member4 + 4 * kLdsTeam * i;
                    const uint32_t col = __builtin_amdgcn_raw_buffer_load_b32(matrix.cols, (int)at, 0, 0);
                    const bool here = at < end_of[r] && (col << 8) + window.minus_first < window.bytes;
                    more |= team_field(__ballot(here && took == 0), l) != 0;
                }
                const uint32_t after = dots_rest(matrix, X1 + (int64_t)row_of[r] * J, X2T, out, J, p, more ? end_of[r] : p,
                                                 final ? 0x7fffffff : c0 + cols, l);
                if (t.member == (int)(r % kLdsTeam)) (upper ? pos[1] : pos[0]) = (int32_t)after;
            }
        }
    }
}

}  // namespace sgap
