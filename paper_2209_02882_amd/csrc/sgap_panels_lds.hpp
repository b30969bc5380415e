// Long rows by column windows that a compute unit holds in LDS (the preparation, and the forms that gather through the
// L2 instead, are in sgap_panels.hip).
//
// A form that gathers a row of B per stored entry is bound by the vector memory path, 64 bytes per clock and compute
// unit (skewed matrix, 500,000 rows, N = 256: 57.6 GB in 2.2 ms, 26 TB/s).  LDS has four times that (a 16-byte read of a
// wavefront takes 4.6 clocks), and long rows that hold a fair share of all columns have a few entries in any run of some
// hundred of them: so a workgroup that owns a whole compute unit brings 64 columns of a run of rows of B (a window) into
// LDS, multiplies out what its long rows have there, and goes on to the next window, the sums of its rows in registers.
//   team   16 lanes x 4 columns hold one long row's 64 columns; a wavefront is four teams, side by side on four rows of
//          about the same length (neighbours in the list sorted by length)
//   slot   a team owns up to kLdsSlots rows, one after the other in every window: 16 wavefronts x 4 teams x 20 slots =
//          1,280 rows per workgroup, 80 registers of sums per lane
//   job    (share of the columns, 64 columns of B, 1,280 long rows); a die's workgroups work on the same few
//          shares together (3.8 GB fetched beyond the L2s, A once per 64 columns of B; the gathers fetched 1.2 GB there and
//          57.6 GB out of the L2s)
// Four entries of four rows cost a wavefront one addition (the address), one 16-byte LDS read and four multiply-adds; a
// pair is handed round its team by DPP (row_newbcast), at no cost.  That makes the vector instructions the bound: 568 M on
// the skewed matrix, 2.2 M clocks of a SIMD of 2.8 M in all (1.2 to 1.3 ms; the whole call 2.54 ms before, 1.62 now).  Half of
// them are multiply-adds that A asks for; a sixth is what the four rows of a wavefront differ by in a window (the more
// entries a row has there, the less: hence windows as large as LDS allows), a quarter what a slot costs by itself, and
// the rest fills up pairs.  The remaining clocks are the windows' way into LDS (10 %) and waiting for the slowest
// wavefront (8 %).  Windows in two halves by turns would hide the former at the price of half the entries per slot.
//
// Nothing relies on sorted columns or columns without repetition: where what a row has in a window is not one run of its
// entries, or more than a slot takes at once, the rest is gathered from memory; where that would be much, the kernels that
// gather all of it run (lds_apart, lds_layout).
#pragma once
#include <type_traits>

#include "sgap_common.hpp"
#include "sgap_panel_view.hpp"

namespace sgap {

constexpr int kLdsBlock = 1024;
constexpr int kLdsWaves = kLdsBlock / kWave;
constexpr int kLdsTeam = 16;                       // lanes of a team, 4 columns each
constexpr int kLdsTeams = kWave / kLdsTeam;        // teams of a wavefront
constexpr int kLdsCols = kLdsTeam * 4;             // columns of a job
constexpr int kLdsSlots = 20;                      // rows a team owns
constexpr int kLdsWindow = 616;                    // rows of B in LDS (and one of zeros): 157,952 of 163,840 bytes
constexpr int kDotsWindow = 596;                   // of X2T, for SDDMM: the rows' numbers lie in LDS too
constexpr int kLdsRowBytes = kLdsCols * 4;
constexpr uint32_t kLdsMaxNnz = 1u << 29;          // byte offsets of entries have 31 bits
constexpr int64_t kLdsMaxCols = 1 << 24;           // byte offsets of rows of 64 columns have 32 bits
constexpr uint32_t kLdsMinRows = 256;
constexpr int kLdsMinCols = 64;                    // columns of B from which on the kernel runs
constexpr int kLdsNoLoads = 0x0F70;                // s_waitcnt vmcnt(0)
static_assert(kLdsSlots <= 2 * kLdsTeam, "positions of the slots lie in two registers of a team");

// Entries of a long row that windows in LDS would not serve, estimated from sixteen places of it: those that the window of
// a slot has no room for, and all where the columns have no order.  The kernels gather them from memory, a few at a time.
// (A window as the row by itself would have it: 16 entries wide in the mean.)  worst: raised to the row's, in entries
// without order: crowded ones wait a sixteenth as long, and one place alone is crowded now and then where columns are random.
__device__ __forceinline__ uint32_t lds_apart(const int32_t* __restrict__ cols, int32_t len, int64_t K, uint32_t& worst)
{
    constexpr int kPlaces = 16, kRoom = 2 * kLdsTeam;
    const int32_t width = (int32_t)fminf((float)kLdsWindow, 16.0f * (float)K / (float)len);
    int32_t here[kPlaces], there[kPlaces];
#pragma unroll
    for (int j = 0; j < kPlaces; ++j) {
        const int32_t at = len / kPlaces * j;
        here[j] = cols[at];
        there[j] = cols[at + kRoom < len ? at + kRoom : len - 1];
    }
    uint32_t crowded = 0;
    bool order = true;
#pragma unroll
    for (int j = 0; j < kPlaces; ++j) {
        order = order && there[j] >= here[j] && (j == 0 || here[j] >= here[j - 1]);
        crowded += len / kPlaces * j + kRoom < len && there[j] - here[j] < width ? 1u : 0u;
    }
    const uint32_t apart = order ? (uint32_t)((unsigned long long)len * crowded / kPlaces) : (uint32_t)len;
    const uint32_t alone = order ? (crowded > 1 ? apart / 16 : 0u) : apart;
    worst = worst < alone ? alone : worst;
    return apart;
}

// What the host knows of it.
struct LdsArgs {
    uint32_t min_rows;    // the kernel runs for lists of at least so many rows
    uint32_t dies;
    uint32_t workgroups;  // of a die
    int64_t ptr_room;     // pointers there is room for
    uint32_t gather_windows;  // that the kernels which gather would have
    int32_t window;       // columns of a window at most, as the caller asks for them (the kernel runs then); 0: he does not
    bool dots;            // SDDMM: a job has all columns of its rows
};

// a / b of clocks, on the device by the reciprocal instruction (every workgroup works out the plan before it begins: 10.2 us
// for panel_pointers_kernel on 300 rows with divisions and four layouts a lane, 7.8 with these and two).
__host__ __device__ inline float lds_ratio(float a, float b)
{
#ifdef __HIP_DEVICE_COMPILE__
    return a * __builtin_amdgcn_rcpf(b);
#else
    return a / b;
#endif
}

// What all layouts of a list have in common.
struct LdsShape {
    uint32_t tiles, quads, least;  // column tiles; teams' rows by fours; groups of rows at least
    int32_t window;                // columns of a window
    float per_col;                 // entries of a long row per column
};

__host__ __device__ inline LdsShape lds_shape(const LdsList& list, const LdsArgs& args, int64_t K, int64_t N)
{
    LdsShape s;
    s.tiles = ((uint32_t)N + kLdsCols - 1) / kLdsCols;
    s.quads = (list.count + kLdsTeams - 1) / kLdsTeams;
    s.least = (s.quads + kLdsWaves * kLdsSlots - 1) / (kLdsWaves * kLdsSlots);
    s.per_col = (float)list.entries / ((float)list.count * (float)K);
    // of the longest row about two thirds of the 32 entries that a slot takes at once, and of a row in the mean 4 at least
    const int32_t room = args.dots ? kDotsWindow : kLdsWindow;
    float window = 16.0f / s.per_col;
    if (window > (float)room) window = (float)room;
    const float longest = 20.0f * (float)K / (float)list.longest;
    window = longest > 0.25f * window ? longest : 0.25f * window;
    s.window = args.window > 0 ? args.window : window < 1.0f ? 1 : window > (float)room ? room : (int32_t)window;
    return s;
}

// The choice between the windows in LDS and the kernels that gather through the L2 is made by the clocks that both are
// expected to take: the three functions below, whose constants are fitted to the kernels' own times over 350 lists (9 % off in
// the mean, 28 % in the case of most).  A layout that the workspace has no room for takes for ever.
// Measured, us for the whole call, LDS against gathers; one row in a hundred is long, columns at random:
//   SpMM
//       rows    mean  N = 64         N = 128        N = 160        N = 256        N = 384        N = 1,024
//    500,000  11,000    773 / 1,054  1,020 / 1,733  1,699 / 2,421  1,622 / 2,528  2,566 / 4,645  6,573 / 10,272
//    500,000   5,500    583 /   622    777 / 1,038  1,262 / 1,413  1,249 / 1,542  2,113 / 2,787  5,064 /  6,330
//    500,000   2,750    499 /   432    670 /   732  1,087 /   918  1,103 / 1,042  1,907 / 1,872  4,511 /  4,375
//    250,000   4,400    288 /   324    361 /   474    524 /   634    537 /   682    888 / 1,233  1,822 /  2,667
//    120,000   8,250    230 /   304    301 /   447    418 /   514    398 /   541    561 / 1,010  1,170 /  2,315
//    120,000   3,300    166 /   174    212 /   245    270 /   273    324 /   333    410 /   541    774 /  1,160
//    120,000   1,320    123 /   110    161 /   158    218 /   176    240 /   198    356 /   351    644 /    732
//     88,000   6,050    176 /   270    219 /   307    301 /   288    274 /   292    394 /   533    795 /  1,106
//     60,000   4,125    153 /   256    178 /   208    237 /   229    277 /   292    337 /   464    538 /  1,033
//     60,000   1,650     96 /   135    123 /   121    149 /   130    176 /   160    229 /   256    358 /    551
//     30,000   2,062     89 /   208     99 /   195    126 /   130    136 /   146    162 /   219    266 /    448
//   SDDMM           J = 64         J = 96         J = 128        J = 160        J = 256
//    500,000  11,000    750 / 1,033  1,167 / 1,504  1,204 / 1,732  1,602 / 2,218  2,036 / 2,737
//    500,000   5,500    594 /   636    901 /   935    942 / 1,099  1,225 / 1,329  1,581 / 1,675
//    500,000   2,750    518 /   458    791 /   662    842 /   811  1,078 /   881  1,386 / 1,152
//    250,000   4,400    232 /   298    318 /   409    354 /   467    453 /   573    590 /   713
//    120,000   8,250    184 /   290    281 /   375    248 /   417    289 /   460    386 /   562
//    120,000   3,300    183 /   228    222 /   263    225 /   291    258 /   302    314 /   349
//    120,000   1,320     95 /   112    134 /   144    131 /   165    156 /   162    203 /   211
//     88,000   6,050    138 /   182    165 /   238    172 /   278    215 /   253    274 /   309
//     60,000   4,125    172 /   279    200 /   275    205 /   285    227 /   263    257 /   298
//     60,000   1,650    103 /   148    116 /   150    119 /   154    138 /   145    154 /   159
//     30,000   2,062    104 /   218    109 /   238    113 /   208    121 /   144    133 /   155
// The rule takes the slower one where the two are within a few per cent; one row eight times as long as the others costs it
// up to 28 % (120,000 rows, N = 128).
__host__ __device__ inline float lds_cost(const LdsShape& s, const LdsList& list, const LdsArgs& args, int64_t K, int64_t N,
                                          uint32_t groups, uint32_t per_die)
{
    const uint32_t slots = (s.quads + kLdsWaves * groups - 1) / (kLdsWaves * groups);
    const uint32_t shares = per_die * args.dies;
    if ((int64_t)(shares + 1) * list.count > args.ptr_room) return __builtin_inff();
    const uint32_t share_cols = ((uint32_t)K + shares - 1) / shares;
    const uint32_t windows = (share_cols + (uint32_t)s.window - 1) / (uint32_t)s.window;
    const float in_window = lds_ratio(s.per_col * (float)share_cols, (float)windows);  // entries of a row
    const uint32_t rounds = ((args.dots ? 1 : s.tiles) * groups * per_die + args.workgroups - 1) / args.workgroups;
    const float tiles = (float)s.tiles, rows = (float)slots;
    // Of a job: its windows on their way into LDS (faster where B is small enough to meet in the L2s), a wavefront's passes
    // over its slots, the sums added into C at the end.  SDDMM passes once for every tile, and looking up and writing the
    // entries is about half a pass more.
    const float tile = args.dots ? (tiles + 0.45f) * (14500.0f + 531.0f * rows) : 0.0f;
    const float cols = lds_ratio((float)share_cols, (float)windows);  // of a window
    float far = (float)K * (float)N * (1.0f / (8 << 20));             // B in 32 MiB, 1 at most
    if (far > 1.0f) far = 1.0f;
    const float job = args.dots ? (float)windows * (tile + tiles * (17.7f * cols + 97.5f * rows * in_window))
                                : ((float)windows * (10700.0f + 4460.0f * far + rows * (124.0f + 359.0f * far + 74.5f * in_window)) +
                                   9700.0f * rows) *
                                      (N % kLdsCols == 0 ? 0.97f : 1.22f);  // (a tile's rows of B begin amid cache lines: 5 to 25 %)
    // what the longest row has in a window beyond the 32 entries that a slot takes at once, where its window is as narrow as
    // it gets: the fewer the rounds, the longer the others wait for it
    const float share = lds_ratio((float)list.longest * (float)s.window, (float)K);
    const float over = share > 32.0f && args.window == 0 ? lds_ratio((float)list.longest * (1.0f - lds_ratio(32.0f, share)) * 32.0f, tiles) : 0.0f;
    const float pointers = (args.dots ? 0.17f : 0.4f) * (float)list.count * (float)shares;
    return (args.dots ? 23500.0f : 60000.0f) + (float)rounds * job + over + pointers;
}

// Clocks of what the windows would not serve.  A few rows of it cost four times what their share of all entries would (the
// other teams and wavefronts wait), and all wait for the team whose row has the most.  500,000 rows, 5,000 of them long, us, LDS
// against gathers:
//   without order, share of the long rows   0.02 %        0.1 %           1 %             all
//     SpMM  N = 64                          765 / 1,050   3,260 / 1,224   6,843 / 1,392   19,578 /  2,730
//           N = 256                       1,642 / 2,536   4,181 / 3,176   8,234 / 3,764   48,440 / 16,519
//     SDDMM J = 64                          709 / 1,030   2,763 / 1,251   6,096 / 1,476   17,415 /  2,768
//           J = 256                       1,922 / 2,729   7,369 / 3,498  16,017 / 4,239   49,890 / 16,758
//   a quarter full over a run of columns    0.1 %         1 %             all
//     SpMM  N = 64                          981 / 1,052   1,238 / 1,079   5,620 / 1,119
//           N = 256                       2,666 / 3,156   3,566 / 3,499  16,398 / 5,562
//     SDDMM J = 64                          951 / 1,041   1,190 / 1,083   4,448 / 1,253
//           J = 256                       2,586 / 3,526   3,287 / 3,923  10,879 / 6,013
__host__ __device__ inline float lds_apart_cost(const LdsShape& s, const LdsList& list, const LdsArgs& args)
{
    const float all = lds_ratio((float)list.apart, (float)(args.dies * args.workgroups)) *
                      (args.dots ? 280.0f + 460.0f * (float)s.tiles : 440.0f + 410.0f * (float)s.tiles);
    const float one = (float)list.worst * (args.dots ? 200.0f + 200.0f * (float)s.tiles : 600.0f);
    return all > one ? all : one;
}

// Clocks of the kernels that gather every entry's row of B through the L2.
__host__ __device__ inline float gather_cost(const LdsList& list, const LdsArgs& args, int64_t N)
{
    const float n = (float)list.count, entries = (float)list.entries, windows = (float)args.gather_windows;
    const float die_windows = (float)((args.gather_windows + args.dies - 1) / args.dies);  // of the die with the most
    if (N > 128) {
        // owner wavefronts: every die walks its windows once per 256 columns, as long as a wavefront needs for all its rows
        // or for the longest
        const float tiles = (float)((N + 255) / 256);
        const uint32_t owners = args.workgroups * kLdsWaves;
        const float rounds = (float)((list.count + owners - 1) / owners);
        const float rows = lds_ratio(rounds * entries, n);
        const float most = rows > (float)list.longest ? rows : (float)list.longest;
        const float row = 270.0f + lds_ratio(0.28f * (float)N, tiles);  // of B
        return tiles * (23000.0f + lds_ratio(row * most * die_windows, windows) + lds_ratio(1800.0f * rounds * windows, (float)args.dies));
    }
    // wavefronts that claim pieces, sixteen to a workgroup: what the chip moves (columns filled up to 64 or 128), and what a
    // workgroup's pieces take one after the other
    const float columns = N <= 64 ? 64.0f : 128.0f;
    const float bytes = lds_ratio(entries * columns * 4.0f * die_windows, (float)args.workgroups * windows);
    const float claims = lds_ratio(n * die_windows, 112.0f * (float)args.workgroups);
    const float piece = lds_ratio(4.0f * entries, n * windows) * (claims > 1.0f ? claims : 1.0f);
    const float pointers = (args.dots ? 0.17f : 0.4f) * n * windows;
    return args.dots ? 96000.0f + 0.0194f * bytes + piece * (70.0f + 60.6f * columns / 64.0f) + pointers
                     : 84000.0f + 0.0222f * bytes + piece * (38.5f + 52.3f * columns / 64.0f) + pointers;
}

constexpr uint32_t kLdsMore = 4, kLdsShares = 32;  // layouts tried: the fewest groups of rows and up to three more, shares per die

__host__ __device__ inline LdsPlan lds_layout(const LdsShape& s, const LdsList& list, const LdsArgs& args, int64_t K, int64_t N,
                                              uint32_t groups, uint32_t per_die, float cost)
{
    LdsPlan p;
    const bool faster = args.window > 0 || cost + lds_apart_cost(s, list, args) < gather_cost(list, args, N);
    p.on = cost < __builtin_inff() && faster && list.nnz < kLdsMaxNnz && N < (1 << 30);
    p.tiles = s.tiles;
    p.tile_cols = ((uint32_t)N / 4 + s.tiles - 1) / s.tiles * 4;
    p.groups = groups;
    p.slots = (s.quads + kLdsWaves * groups - 1) / (kLdsWaves * groups);
    p.per_die = per_die;
    p.share_cols = (int32_t)(((uint32_t)K + per_die * args.dies - 1) / (per_die * args.dies));
    p.window = s.window;
    return p;
}

// How the list's rows are laid over the workgroups.  Their number is not known on the host: the workgroups of
// panel_pointers_kernel each work it out (all lanes of a wavefront together, two layouts each), one leaves it in the header.
__device__ __forceinline__ LdsPlan lds_plan(const LdsList& list, const LdsArgs& args, int64_t K, int64_t N)
{
    LdsPlan p;
    p.on = 0;
    if (list.count < args.min_rows) return p;
    const LdsShape s = lds_shape(list, args, K, N);
    const uint32_t lane = threadIdx.x % kWave, shares = lane % kLdsShares;
    unsigned long long best = ~0ull;
#pragma unroll
    for (uint32_t half = 0; half < kLdsMore; half += kWave / kLdsShares) {
        const uint32_t more = half + lane / kLdsShares;
        const float cost = lds_cost(s, list, args, K, N, s.least + more, shares + 1);
        const unsigned long long key = (unsigned long long)__float_as_uint(cost) << 32 | more << 8 | shares;
        if (key < best) best = key;
    }
#pragma unroll
    for (int m = 1; m < kWave; m *= 2) {
        const unsigned long long other = __shfl_xor(best, m, kWave);
        if (other < best) best = other;
    }
    const uint32_t chosen = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)best);
    const float cost = __int_as_float(__builtin_amdgcn_readfirstlane((int)(uint32_t)(best >> 32)));
    return lds_layout(s, list, args, K, N, s.least + (chosen >> 8), (chosen & 255) + 1, cost);
}

// The value that lane J of a lane's team holds.
template <int J>
__device__ __forceinline__ int32_t team_bcast(int32_t v)
{
    return __builtin_amdgcn_update_dpp(0, v, 0x150 + J, 0xF, 0xF, true);
}
// The value that the lane D above holds (zero past the end of the team).
template <int D>
__device__ __forceinline__ int32_t team_shift(int32_t v)
{
    return __builtin_amdgcn_update_dpp(0, v, 0x100 + D, 0xF, 0xF, true);
}

// Two neighbouring stored entries.
struct LdsEntries {
    int32_t col[2], val[2];  // the bits of the values
};

// The stored entries by their byte offsets in colidx and vals: 32 bits, and what lies past the last entry reads as zero.
struct LdsMatrix {
    __amdgpu_buffer_rsrc_t cols, vals;
    __device__ __forceinline__ LdsMatrix(const int32_t* colidx, const float* values, uint32_t nnz)
        : cols(__builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(colidx), 0, (int)(nnz * 4), 0x00020000)),
          vals(__builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(values), 0, (int)(nnz * 4), 0x00020000))
    {
    }
    __device__ __forceinline__ LdsEntries load(uint32_t at) const
    {
        typedef uint32_t raw_u2 __attribute__((ext_vector_type(2)));
        const raw_u2 c = __builtin_amdgcn_raw_buffer_load_b64(cols, (int)at, 0, 0);
        const raw_u2 v = __builtin_amdgcn_raw_buffer_load_b64(vals, (int)at, 0, 0);
        return {{(int32_t)c.x, (int32_t)c.y}, {(int32_t)v.x, (int32_t)v.y}};
    }
};

// f(0), f(1), ... f(R - 1), each with its number as a type.
template <int R, int I = 0, typename F>
__device__ __forceinline__ void lds_each(F&& f)
{
    if constexpr (I < R) {
        f(std::integral_constant<int, I>{});
        lds_each<R, I + 1>(f);
    }
}

// acc += (lane J of the team's val[0]) * b[0] + (its val[1]) * b[1], two fused multiply-adds per column; FIRST: acc = that.
// The compiler does not fold the DPP move into a fused multiply-add by itself.  (The no-op is the two wait states between
// a write of val and its DPP read, which the compiler does not see inside this text.)
template <int J, bool FIRST>
__device__ __forceinline__ void team_fma(Vec<4>& acc, const int32_t (&val)[2], const Vec<4> (&b)[2])
{
    if constexpr (FIRST) {
        asm volatile("s_nop 1\n\t"
                     "v_mul_f32_dpp %0, %4, %6 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
                     "v_mul_f32_dpp %1, %4, %7 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
                     "v_mul_f32_dpp %2, %4, %8 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
                     "v_mul_f32_dpp %3, %4, %9 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
                     "v_fmac_f32_dpp %0, %5, %10 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
                     "v_fmac_f32_dpp %1, %5, %11 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
                     "v_fmac_f32_dpp %2, %5, %12 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
                     "v_fmac_f32_dpp %3, %5, %13 row_newbcast:%14 row_mask:0xf bank_mask:0xf"
                     : "=&v"(acc.v[0]), "=&v"(acc.v[1]), "=&v"(acc.v[2]), "=&v"(acc.v[3])
                     : "v"(val[0]), "v"(val[1]), "v"(b[0].v[0]), "v"(b[0].v[1]), "v"(b[0].v[2]), "v"(b[0].v[3]),
                       "v"(b[1].v[0]), "v"(b[1].v[1]), "v"(b[1].v[2]), "v"(b[1].v[3]), "n"(J));
    } else {
        asm volatile("s_nop 1\n\t"
                     "v_fmac_f32_dpp %0, %4, %6 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
                     "v_fmac_f32_dpp %1, %4, %7 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
                     "v_fmac_f32_dpp %2, %4, %8 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
                     "v_fmac_f32_dpp %3, %4, %9 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
                     "v_fmac_f32_dpp %0, %5, %10 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
                     "v_fmac_f32_dpp %1, %5, %11 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
                     "v_fmac_f32_dpp %2, %5, %12 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
                     "v_fmac_f32_dpp %3, %5, %13 row_newbcast:%14 row_mask:0xf bank_mask:0xf"
                     : "+&v"(acc.v[0]), "+&v"(acc.v[1]), "+&v"(acc.v[2]), "+&v"(acc.v[3])
                     : "v"(val[0]), "v"(val[1]), "v"(b[0].v[0]), "v"(b[0].v[1]), "v"(b[0].v[2]), "v"(b[0].v[3]),
                       "v"(b[1].v[0]), "v"(b[1].v[1]), "v"(b[1].v[2]), "v"(b[1].v[3]), "n"(J));
    }
}

typedef float lds_f4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(3))) char* lds_bytes;

// Two rows of the window for each of the four teams: those whose byte offsets in LDS lane J of the team has.
template <int J>
__device__ __forceinline__ void lds_read(Vec<4> (&b)[2], lds_bytes mine, const int32_t (&off)[2])
{
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const lds_f4 t = *(const __attribute__((address_space(3))) lds_f4*)(mine + team_bcast<J>(off[i]));
        b[i].v[0] = t.x; b[i].v[1] = t.y; b[i].v[2] = t.z; b[i].v[3] = t.w;
    }
}

// This thread's place, worked out anew where it is asked for: what the phases between the windows make of it would
// otherwise be kept in registers throughout, of which there are none to spare.
struct LdsThread {
    int lane, team, member;
    __device__ __forceinline__ LdsThread()
    {
        uint32_t all = ~0u;
        asm volatile("" : "+s"(all));
        lane = (int)__builtin_amdgcn_mbcnt_hi(all, __builtin_amdgcn_mbcnt_lo(all, 0));
        team = lane / kLdsTeam;
        member = lane % kLdsTeam;
    }
};

// First column of this lane in the tile that begins at tile_k; a lane past the last column gets columns that exist (its
// sums are thrown away).
__device__ __forceinline__ int64_t lds_columns(int32_t tile_k, const LdsThread& t, int64_t N)
{
    return tile_k + t.member * 4 + 4 <= N ? tile_k + t.member * 4 : N - 4;
}

struct LdsLanes {
    uint32_t member8;  // eight times the lane's number in its team: byte offset of its two entries
    int shift;         // first lane of the team in its half of the wavefront
    bool high;         // the upper half
};

__device__ __forceinline__ uint32_t team_field(unsigned long long mask, const LdsLanes& l)
{
    const uint32_t half = l.high ? (uint32_t)(mask >> 32) : (uint32_t)mask;
    return __builtin_amdgcn_ubfe(half, l.shift, kLdsTeam);
}

// The window a workgroup is at: columns [first, first + cols), as byte offsets of rows in LDS (of less than 2^24 columns).
struct LdsWindow {
    uint32_t minus_first;  // -first * kLdsRowBytes
    uint32_t bytes;        // cols * kLdsRowBytes
};

// What one slot has in the window, into acc; returns the bytes of entries taken.  over: minus the bytes of entries to the end
// of the slot's share.  Of the sixteen times two entries at the slot's position the first ones that lie in the window are taken.
// `open` is set where that may not be all of them: where a team has more than 32, and where one in the window lies behind
// one that does not (columns that are not sorted; nothing is taken then).
__device__ __forceinline__ uint32_t lds_slot(lds_bytes mine, Vec<4>& acc, const LdsEntries& e, int32_t over, const LdsWindow& w,
                                             const LdsLanes& l, bool& open)
{
    constexpr unsigned long long kNotFirst = 0xFFFEFFFEFFFEFFFEull, kLast = 0x8000800080008000ull;
    static_assert(kLdsRowBytes == 256, "the shift");
    int32_t off[2], val[2];
    unsigned long long taken[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const uint32_t at = ((uint32_t)e.col[i] << 8) + w.minus_first;
        const bool there = over < -(int32_t)l.member8 - 4 * i;
        taken[i] = __ballot(at < w.bytes) & __ballot(there);
        const bool in = at < w.bytes && there;
        off[i] = in ? (int32_t)at : kLdsWindow * kLdsRowBytes;
        val[i] = in ? e.val[i] : 0;
    }
    const unsigned long long gaps = (taken[1] & ~taken[0]) | (taken[0] & ~(taken[1] << 1) & kNotFirst);
    open = gaps != 0 || (taken[1] & kLast) != 0;
    if (gaps != 0) return 0;
    const uint32_t both = (uint32_t)taken[0] | (uint32_t)(taken[0] >> 32);
    uint32_t pairs = (uint32_t)__popc((both | both >> 16) & 0xFFFFu);  // of the team with the most
    // sixteen entries at a time, by twos, the next two rows read before these are multiplied.  The window's sums are made
    // by themselves and then added to the row's: a row of n entries, m of them in a window, has rounding errors as of
    // m + n / m additions in a row instead of n (one long sum was less exact than the gathering forms' many short ones).
    Vec<4> sum;
    for (;;) {
        Vec<4> b[2][2];
        lds_read<0>(b[0], mine, off);
        lds_each<kLdsTeam / 2>([&](auto Q) {
            constexpr int q = decltype(Q)::value;
            if (q == 0 || pairs > q) {
                if constexpr (q + 1 < kLdsTeam / 2) lds_read<q + 1>(b[(q + 1) % 2], mine, off);
                team_fma<q, q == 0>(sum, val, b[q % 2]);
            }
        });
#pragma unroll
        for (int i = 0; i < 4; ++i) acc.v[i] += sum.v[i];
        if (pairs <= kLdsTeam / 2) break;
        pairs -= kLdsTeam / 2;
        asm volatile("" : "+s"(pairs));  // (one copy of the sixteen: two for each of twenty slots do not fit the instruction cache)
        off[0] = team_shift<kLdsTeam / 2>(off[0]);
        off[1] = team_shift<kLdsTeam / 2>(off[1]);
        val[0] = team_shift<kLdsTeam / 2>(val[0]);
        val[1] = team_shift<kLdsTeam / 2>(val[1]);
    }
    return ((uint32_t)__popc(team_field(taken[0], l)) + (uint32_t)__popc(team_field(taken[1], l))) * 4;
}

// The rest of a slot: the entries in front of column c1 up to the first that is not, in any order of the columns, rows of
// B from memory (B points to the lane's columns).  The sums are added to `row` (nullptr: the team has no row, or the lane
// no columns).
__device__ __forceinline__ uint32_t lds_rest(const LdsMatrix& matrix, const float* __restrict__ B, int64_t N,
                                             float* __restrict__ row, uint32_t p, uint32_t end, int32_t c1, const LdsLanes& l)
{
    Vec<4> acc;
    acc.zero();
    for (;;) {
        const LdsEntries e = matrix.load(p + l.member8);
        const uint32_t rest = end - p;
        // (the bits past a field's sixteenth are zero)
        const uint32_t even = (uint32_t)__ffs((int)~team_field(__ballot(e.col[0] < c1 && l.member8 < rest), l)) - 1u;
        const uint32_t odd = (uint32_t)__ffs((int)~team_field(__ballot(e.col[1] < c1 && l.member8 + 4 < rest), l)) - 1u;
        const uint32_t taken = even <= odd ? 2 * even : 2 * odd + 1;
#pragma unroll 1
        for (uint32_t j = 0; __any(2 * j < taken); ++j) {
            Vec<4> b[2];
            float val[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int32_t col = __shfl(e.col[i], (int)j, kLdsTeam);
                val[i] = __int_as_float(__shfl(e.val[i], (int)j, kLdsTeam));
                b[i].zero();
                if (2 * j + i < taken) b[i] = load_vec<4>(B + (int64_t)col * N);
                else val[i] = 0.0f;
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) acc.fma(val[i], b[i]);
        }
        p += taken * 4;
        if (!__any(taken == 2 * kLdsTeam)) break;
    }
    if (row)
        for (int i = 0; i < 4; ++i) unsafeAtomicAdd(row + i, acc.v[i]);
    return p;
}

// The kernel's shared memory.
struct LdsShared {
    __attribute__((aligned(16))) float b[(kLdsWindow + 1) * kLdsCols];
    uint32_t end[kLdsWaves * kLdsTeams * kLdsSlots];
};
static_assert(sizeof(LdsShared) <= 160 * 1024, "of a compute unit");

// A workgroup of kLdsBlock threads that has its compute unit to itself.
__device__ __forceinline__ void panel_lds_rows(const int32_t* __restrict__ colidx, const float* __restrict__ vals,
                                               const float* __restrict__ B, float* __restrict__ C, const PanelView& scr,
                                               int64_t K, int64_t N, const LdsArgs& args, uint32_t wave, LdsShared& shared)
{
    constexpr int R = kLdsSlots;
    float* const s_b = shared.b;
    uint32_t* const s_end = shared.end;
    const uint32_t n = scr.head->count;
    const LdsPlan plan = scr.head->lds;
    const LdsMatrix matrix(colidx, vals, scr.head->nnz);
    const uint32_t die = blockIdx.x % args.dies;
    LdsLanes l;
    lds_bytes mine;    // LDS address of this lane's columns in the window's first row
    uint32_t* end_of;  // where the share of a slot's row ends, of the team's slots
    {
        const LdsThread t;
        l.member8 = (uint32_t)t.member * 8;
        l.shift = t.team % 2 * kLdsTeam;
        l.high = t.team >= 2;
        mine = (lds_bytes)s_b + t.member * 16;
        end_of = s_end + (wave * kLdsTeams + t.team) * R;
    }
    static_assert(kLdsCols == kWave, "the row of zeros");
    if (wave == 0) s_b[kLdsWindow * kLdsCols + LdsThread().lane] = 0.0f;

    const uint32_t per_share = plan.tiles * plan.groups;
    const uint32_t jobs = per_share * plan.per_die;
    const uint32_t shares = plan.per_die * args.dies;
    for (uint32_t job = blockIdx.x / args.dies; job < jobs; job += args.workgroups) {
        const uint32_t share = die * plan.per_die + job / per_share;
        const uint32_t tile = job % per_share % plan.tiles;
        const uint32_t group = job % per_share / plan.tiles;
        const int64_t share_begin = (int64_t)share * plan.share_cols;
        if (share_begin >= K) continue;
        const int32_t share_end = (int32_t)(K - share_begin < plan.share_cols ? K : share_begin + plan.share_cols);
        const int32_t tile_k = (int32_t)(tile * plan.tile_cols);  // first column

        auto list_place = [&](uint32_t slot, int team) {  // place of the team's row in the ranked list
            const uint32_t units = kLdsWaves * plan.groups;
            const uint32_t me = group * kLdsWaves + wave;
            return (slot * units + (slot & 1 ? units - 1 - me : me)) * kLdsTeams + (uint32_t)team;
        };
        int32_t pos[2] = {0, 0};  // lane i of a team: where slots i and 16 + i stand, as byte offsets
        {
            const LdsThread t;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint32_t slot = (uint32_t)(h * kLdsTeam + t.member);
                const uint32_t q = list_place(slot, t.team);
                uint32_t end = 0;
                if (slot < plan.slots && q < n) {
                    const int64_t at = (int64_t)scr.order[q] * (shares + 1) + share;
                    pos[h] = scr.ptr[at] * 4;
                    end = (uint32_t)scr.ptr[at + 1] * 4;
                }
                if (slot < R) end_of[slot] = end;  // (read by this wavefront alone)
            }
        }
        Vec<4> acc[R];
#pragma unroll
        for (int r = 0; r < R; ++r) acc[r].zero();

        const int32_t count = (share_end - (int32_t)share_begin + plan.window - 1) / plan.window;  // windows
        const int32_t width = (share_end - (int32_t)share_begin + count - 1) / count;
        LdsEntries held[2];           // of the next two slots
        uint32_t next_end = end_of[0];  // of the next slot
        lds_each<2>([&](auto I) {
            constexpr int i = decltype(I)::value;
            held[i] = matrix.load((uint32_t)team_bcast<i>(pos[0]) + l.member8);
        });
        for (int32_t w = 0; w < count; ++w) {
            const int32_t c0 = (int32_t)share_begin + w * width;
            const int32_t cols = share_end - c0 < width ? share_end - c0 : width;
            __syncthreads();  // everyone is done with the window before
            const LdsThread t;
            const int64_t k = lds_columns(tile_k, t, N);
            for (int32_t i = (int32_t)wave * kLdsTeams; i < cols; i += kLdsWaves * kLdsTeams) {
                const int32_t row = i + t.team < cols ? i + t.team : cols - 1;
                const float* from = B + (int64_t)(c0 + row) * N + k;
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)from,
                                                 (__attribute__((address_space(3))) void*)(s_b + i * kLdsCols), 16, 0, 0);
            }
            __builtin_amdgcn_s_waitcnt(kLdsNoLoads);
            __syncthreads();
            LdsWindow window{0u - (uint32_t)c0 * kLdsRowBytes, (uint32_t)cols * kLdsRowBytes};
            asm volatile("" : "+s"(window.minus_first));  // (else a subtraction and a shift, where one instruction does both)
            uint32_t open = 0;  // slots with more to do
            lds_each<R>([&](auto I) {
                constexpr int r = decltype(I)::value, ahead = (r + 2) % R;
                // A compute unit issues its oldest wavefronts first: with nothing said the youngest take twice as long and
                // the others wait for them at the end of the window.  So a wavefront steps back as it gets on.
                if constexpr (r % (R / 4) == 0) __builtin_amdgcn_s_setprio(3 - r / (R / 4));
                const LdsEntries e = held[0];
                held[0] = held[1];
                const uint32_t end = next_end;
                next_end = end_of[(r + 1) % R];
                // (this way round: v_subrev with row_newbcast, which end - pos becomes, hands round the wrong operand)
                const int32_t over = team_bcast<r % kLdsTeam>(pos[r / kLdsTeam]) - (int32_t)end;
                bool slot_open;
                const uint32_t taken = lds_slot(mine, acc[r], e, over, window, l, slot_open);
                if (slot_open) open |= 1u << r;
                open = (uint32_t)__builtin_amdgcn_readfirstlane((int)open);
                asm volatile("" : "+s"(open));  // (now: the compiler would keep every slot's masks until the last)
                pos[r / kLdsTeam] += __builtin_amdgcn_inverse_ballot_w64(0x0001000100010001ull << (r % kLdsTeam)) ? (int32_t)taken : 0;
                held[1] = matrix.load((uint32_t)team_bcast<ahead % kLdsTeam>(pos[ahead / kLdsTeam]) + l.member8);
            });
            const bool final = w + 1 == count;  // of the share: takes all that is left (of rows that are not sorted)
            if (final) {
                const LdsThread t;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int slot = h * kLdsTeam + t.member;
                    const unsigned long long some = __ballot(slot < R && (uint32_t)pos[h] < end_of[slot < R ? slot : 0]);
                    open |= (uint32_t)((some | some >> 16 | some >> 32 | some >> 48) & 0xFFFFu) << (h * kLdsTeam);
                }
            }
            if (open) {
                const LdsThread t;
                const int64_t k = lds_columns(tile_k, t, N);
                const bool own = tile_k + t.member * 4 < N && t.member * 4 < (int)plan.tile_cols;
                do {
                    const uint32_t r = (uint32_t)__ffs((int)open) - 1u;
                    open &= open - 1u;
                    const bool upper = r >= kLdsTeam;
                    const uint32_t p = (uint32_t)__shfl(upper ? pos[1] : pos[0], (int)(r % kLdsTeam), kLdsTeam);
                    const uint32_t q = list_place(r, t.team);
                    float* row = own && q < n ? C + (int64_t)scr.rows[scr.order[q]] * N + k : nullptr;
                    const uint32_t after = lds_rest(matrix, B + k, N, row, p, end_of[r], final ? 0x7fffffff : c0 + cols, l);
                    if (t.member == (int)(r % kLdsTeam)) (upper ? pos[1] : pos[0]) = (int32_t)after;
                } while (open);
                // (the first two slots may have been among them)
                lds_each<2>([&](auto I) {
                    constexpr int i = decltype(I)::value;
                    held[i] = matrix.load((uint32_t)team_bcast<i>(pos[0]) + l.member8);
                });
            }
        }
        __syncthreads();  // everyone is done with the last window: its place serves the sums on their way out
        // (a wavefront's sums change lanes, so that an atomic instruction covers consecutive words: lanes that are 16
        // bytes apart keep the memory pipeline busy four times longer)
        const LdsThread t;
        float* out = s_b + wave * (kWave * 4);
        lds_each<R>([&](auto I) {
            constexpr int r = decltype(I)::value;
            const uint32_t q = list_place(r, t.team);
            *reinterpret_cast<float4*>(out + t.lane * 4) = make_float4(acc[r].v[0], acc[r].v[1], acc[r].v[2], acc[r].v[3]);
            __builtin_amdgcn_wave_barrier();
            if (q < n) {
                float* row = C + (int64_t)scr.rows[scr.order[q]] * N + tile_k;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int col = i * kLdsTeam + t.member;
                    const float sum = out[t.team * kLdsCols + col];
                    if (col < (int)plan.tile_cols && tile_k + col < N) unsafeAtomicAdd(row + col, sum);
                }
            }
            __builtin_amdgcn_wave_barrier();
        });
    }
}

}  // namespace sgap
