// SDDMM on matrices whose neighbouring rows share columns: four consecutive rows ("a quad") together, a wavefront each, and
// a row of X2T that several of them want is gathered once.
//
// sddmm_tile_kernel gathers a row of X2T for every stored entry; on a 27-point stencil half of them a second time for the
// same four rows.  Here a wavefront lists the distinct columns of its quad in LDS, in their order (a column opens a record
// unless the row above has it too, and an entry finds its record by counting what opens below its column in each of the
// four rows), and multiplies them with the four rows of X1, which its lanes hold.  v_mfma_f32_4x4x1 sums row times record over
// 16 columns for every four lanes by themselves; what is left is a sum over 4 to 16 places.  Of the sixteen products of four
// records those are kept that the pattern has.
// No value of a row gets into another's products: infinities and NaN stay where they are.
//
// 27-point stencils, tile by tile and so (groups of 8; of 16 from J = 200 on): 1,000,000 rows, J = 128 692 -> 553 us, J = 100 889 -> 581,
// J = 256 2,272 -> 999; 212,040 rows, J = 128 123 -> 118, J = 100 170 -> 125, J = 72 152 -> 123, J = 200 402 -> 206, J = 256 436 -> 213.  Half of the gathers
// are gone (L1 accesses 142 M at J = 128), and the time is no longer theirs alone: without any gather from beyond the L1 it is
// 472 of 554 us, without products 185.  Vector instructions keep their units busy for 0.7 of the time (690 a quad beside 109
// MFMA, of which 260 change places between lanes), X1 and the stored entries come from memory once.  What the steps gave:
// rows of X2T in neighbouring lanes 889 -> 645; workgroups dispatched in order instead of persistent ones that drift apart 621;
// the look at the matrix shared by the wavefronts 590; rows that are the first one shifted listed without a search 554; a
// workgroup's quads a round of the resident workgroups apart, so that those at work are on neighbouring rows, 529 to 546.  More quads
// per workgroup (8: 544, 16: 563) or fewer (2: 533), barriers between quads, more registers or wavefronts gain nothing.
//
// Columns that do not ascend in some row open a record each.  A quad with a row of kQuadRow entries or more goes entry by
// entry, and from a whole tile of entries on it is dealt out by tiles, so that no wavefront has more than a tile to itself.
#pragma once
#include "sgap_nnz_common.hpp"
#include "sgap_quads.hpp"

namespace sgap {

constexpr int kDotBatch = 16;                   // records that are multiplied together at most
constexpr int kDotRecords = kQuad * kQuadRow;   // records of a quad at most
constexpr uint32_t kNoPlace = 0xff;
constexpr int kQuadMeanRow = 12;

struct alignas(16) QuadDots {  // of a wavefront
    uint32_t offset[kDotRecords + kDotBatch];  // of the record's row of X2T, in bytes
    uint32_t place[kDotRecords + kDotBatch];  // byte i: which of row i's entries the record is, kNoPlace: none
    float out[kQuad][kQuadRow];
    int32_t row_col[kQuad][1 + kQuadRow];     // the rows' columns from place 1 on, kNoColumn behind them
};

// Whether a matrix is taken by four rows together is told by kLookRuns runs of kLookRun rows, spread over it (by multiples of the
// golden section): by the lengths of all of them and, of kLookPairs rows of each run, whether the row above has their columns.  It
// decides nothing but which way the products are formed.
constexpr int kLookRuns = kWavesPerBlock, kLookRun = kWave - 1, kLookPairs = 4;  // (a lane for each row pointer of a run)
__host__ __device__ constexpr int64_t look_run(uint32_t number, int64_t M)  // its first row; M >= kLookRun
{
    return (int64_t)(((uint64_t)((number + 1u) * 0x9e3779b9u) * (uint32_t)(M - kLookRun + 1)) >> 32);
}
// More than a dozen entries and less than kQuadRow in the mean, and few rows of kQuadRow or more: such a row leaves its whole
// quad to quad_entries.  400,000 rows of 27 neighbouring columns, one in 64, 32, 16 or 8 of 40, tile by tile and by four rows
// together: J = 128, G = 8 253 / 216, 253 / 258, 261 / 317, 262 / 435 us; J = 72, G = 8 286 / 258, 290 / 313, 295 / 400, 302 / 534;
// J = 200, G = 16 (wide) 689 / 437, 676 / 542, 673 / 704, 642 / 955.
__host__ __device__ constexpr bool lengths_for_quads(int64_t M, int64_t nnz, int long_rows, bool wide)
{
    return nnz > kQuadMeanRow * M && nnz < kQuadRow * M && long_rows * (wide ? 20 : 42) <= kLookRuns * kLookRun;
}
// Of the rows' columns the row above has nine in sixteen, or half (wide).  268,800 rows that share 54 %, tile by tile and by four rows
// together: J = 72 179 / 203 us, J = 128 161 / 172 (G = 8), 168 / 171 (G = 16), J = 200 524 / 335, J = 256 657 / 322; a 27-point
// stencil shares two thirds but at the ends of its lines.
__host__ __device__ constexpr bool columns_for_quads(int shared, int total, bool wide) { return wide ? 2 * shared >= total : 16 * shared >= 9 * total; }
// The rows of a run whose columns are looked at, behind the first: no two pairs of them as far apart
__host__ __device__ constexpr int look_at(int half, int i) { return half ? 29 + 23 * i : 11 * i; }

// Called by whole workgroups (counts: an integer for each wavefront, in LDS); the same result everywhere.  A matrix that does not
// pass costs the look one way to memory beside that of its last row pointer, or two where the lengths pass.
__device__ __forceinline__ bool rows_share_columns(const SpmmArgs& a, int32_t nnz, bool wide, int32_t* __restrict__ counts)
{
    constexpr int MINE = kLookPairs / 2;  // rows whose columns half a wavefront looks at, of its first run
    const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave)), q = lane % kQuadRow;
    int32_t p[kLookRuns];
#pragma unroll
    for (int i = 0; i < kLookRuns; ++i) p[i] = a.rowptr[look_run((uint32_t)(wave + i) % kLookRuns, a.M) + lane];
    int long_rows = 0;
#pragma unroll
    for (int i = 0; i < kLookRuns; ++i) {
        const int32_t next = __builtin_amdgcn_update_dpp(p[i], p[i], 0x130, 0xF, 0xF, false);  // wave_shl:1; the last lane keeps its own
        long_rows += (int)__popcll(__ballot(next - p[i] >= kQuadRow));
    }
    if (!lengths_for_quads(a.M, nnz, long_rows, wide)) return false;
    int32_t above[MINE], col[MINE];
#pragma unroll
    for (int i = 0; i < MINE; ++i) {
        const int at = look_at(lane / kQuadRow, i);
        const int32_t begin = __shfl(p[0], at), mid = __shfl(p[0], at + 1), end = __shfl(p[0], at + 2);
        above[i] = begin + q < mid ? a.colidx[begin + q] : kNoColumn;
        col[i] = mid + q < end ? a.colidx[mid + q] : kNoColumn;
    }
    int shared = 0, total = 0;
#pragma unroll
    for (int i = 0; i < MINE; ++i) {
        int lo = 0;
#pragma unroll
        for (int half = kQuadRow / 2; half > 0; half /= 2) lo += __shfl(above[i], lo + half - 1, kQuadRow) < col[i] ? half : 0;
        const bool found = __shfl(above[i], lo, kQuadRow) == col[i];
        shared += (int)__popcll(__ballot(found && col[i] != kNoColumn));
        total += (int)__popcll(__ballot(col[i] != kNoColumn));
    }
    if (lane == 0) counts[wave] = shared << 16 | total;
    __syncthreads();
    int sum = 0;
#pragma unroll
    for (int w = 0; w < kWavesPerBlock; ++w) sum += counts[w];
    return columns_for_quads(sum >> 16, sum & 0xffff, wide);
}

// Sum of v over the lanes 4, 8 and 12 further in each row of 16 lanes
__device__ __forceinline__ float sum_every_fourth(float v)
{
    const int four = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x124, 0xF, 0xF, true);  // row_ror:4
    v += __builtin_bit_cast(float, four);
    const int eight = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x128, 0xF, 0xF, true);  // row_ror:8
    return v + __builtin_bit_cast(float, eight);
}

// (x.lower + x.upper, y.lower + y.upper) in the halves of 32 lanes
__device__ __forceinline__ float fold_halves(float x, float y)
{
    auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, y), false, false);
    const unsigned a = r[0], b = r[1];
    return __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b);
}

// The same in the rows of 16 lanes of each half
__device__ __forceinline__ float fold_rows(float x, float y)
{
    auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, y), false, false);
    const unsigned a = r[0], b = r[1];
    return __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b);
}

// Four registers of four neighbouring lanes change places: afterwards x[t].v of lane j is what x[j].v of lane t was (lanes
// counted within four).  Two rounds that swap a bit of the register's number with one of the lane's.
// (v_cndmask with DPP, which the compiler does not form: it takes two instructions.  A register may be read through DPP two
// instructions after it was written, and by an MFMA two after as well.)
__device__ __forceinline__ void transpose_fours(Vec<4> (&x)[4])
{
    Vec<4> p, q;
    asm("s_mov_b64 vcc, %[even]\n\t"
        "s_nop 1\n\t"
        "v_cndmask_b32_dpp %[p0], %[b0], %[a0], vcc quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_cndmask_b32_dpp %[p1], %[b1], %[a1], vcc quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_cndmask_b32_dpp %[p2], %[b2], %[a2], vcc quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_cndmask_b32_dpp %[p3], %[b3], %[a3], vcc quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_cndmask_b32_dpp %[q0], %[d0], %[c0], vcc quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_cndmask_b32_dpp %[q1], %[d1], %[c1], vcc quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_cndmask_b32_dpp %[q2], %[d2], %[c2], vcc quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_cndmask_b32_dpp %[q3], %[d3], %[c3], vcc quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "s_not_b64 vcc, vcc\n\t"
        "v_cndmask_b32_dpp %[b0], %[a0], %[b0], vcc quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_cndmask_b32_dpp %[b1], %[a1], %[b1], vcc quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_cndmask_b32_dpp %[b2], %[a2], %[b2], vcc quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_cndmask_b32_dpp %[b3], %[a3], %[b3], vcc quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_cndmask_b32_dpp %[d0], %[c0], %[d0], vcc quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_cndmask_b32_dpp %[d1], %[c1], %[d1], vcc quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_cndmask_b32_dpp %[d2], %[c2], %[d2], vcc quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_cndmask_b32_dpp %[d3], %[c3], %[d3], vcc quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "s_mov_b64 vcc, %[low]\n\t"
        "v_cndmask_b32_dpp %[a0], %[q0], %[p0], vcc quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_cndmask_b32_dpp %[a1], %[q1], %[p1], vcc quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_cndmask_b32_dpp %[a2], %[q2], %[p2], vcc quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_cndmask_b32_dpp %[a3], %[q3], %[p3], vcc quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_cndmask_b32_dpp %[c0], %[d0], %[b0], vcc quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_cndmask_b32_dpp %[c1], %[d1], %[b1], vcc quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_cndmask_b32_dpp %[c2], %[d2], %[b2], vcc quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_cndmask_b32_dpp %[c3], %[d3], %[b3], vcc quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "s_not_b64 vcc, vcc\n\t"
        "v_cndmask_b32_dpp %[q0], %[p0], %[q0], vcc quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_cndmask_b32_dpp %[q1], %[p1], %[q1], vcc quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_cndmask_b32_dpp %[q2], %[p2], %[q2], vcc quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_cndmask_b32_dpp %[q3], %[p3], %[q3], vcc quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_cndmask_b32_dpp %[d0], %[b0], %[d0], vcc quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_cndmask_b32_dpp %[d1], %[b1], %[d1], vcc quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_cndmask_b32_dpp %[d2], %[b2], %[d2], vcc quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_cndmask_b32_dpp %[d3], %[b3], %[d3], vcc quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1"
        : [a0] "+v"(x[0].v[0]), [a1] "+v"(x[0].v[1]), [a2] "+v"(x[0].v[2]), [a3] "+v"(x[0].v[3]), [b0] "+v"(x[1].v[0]), [b1] "+v"(x[1].v[1]), [b2] "+v"(x[1].v[2]), [b3] "+v"(x[1].v[3]), [c0] "+v"(x[2].v[0]), [c1] "+v"(x[2].v[1]), [c2] "+v"(x[2].v[2]), [c3] "+v"(x[2].v[3]), [d0] "+v"(x[3].v[0]), [d1] "+v"(x[3].v[1]), [d2] "+v"(x[3].v[2]), [d3] "+v"(x[3].v[3]),
          [p0] "=&v"(p.v[0]), [p1] "=&v"(p.v[1]), [p2] "=&v"(p.v[2]), [p3] "=&v"(p.v[3]), [q0] "=&v"(q.v[0]), [q1] "=&v"(q.v[1]), [q2] "=&v"(q.v[2]), [q3] "=&v"(q.v[3])
        : [even] "s"(0x5555555555555555ull), [low] "s"(0x3333333333333333ull)
        : "vcc", "scc");
    x[1] = x[2];
    x[2] = q;
}

// A lane's part of the rows of X1 and X2T.  A row takes 4 * BL lanes (BL: 8 or 16), four columns each, so that a load covers
// 16 / BL rows from end to end (lanes in the rows' order, which is what a load is quick with: with four rows in every four
// lanes, as the products want them, every 16 bytes are a cache access of their own, 475 M of them and 889 us on the stencil
// below).  Four loads make a batch of 64 / BL rows: lane group number p has rows 4 * p .. + 4 of it.
// CHAINS: the sixteen columns of every four lanes are summed in so many chains (1, 2 or 4), none longer than what a lane of
// sddmm_tile_kernel sums by itself, so that the error is no larger.  Relative error (2-norm) against 64 bits, uniform values,
// J = 128: tile by tile 9.1e-8, 8.1e-8 and 7.7e-8 with groups of 8, 16 and 32, with one chain 9.1e-8 for all, so 9.1e-8, 8.1e-8 and
// 7.7e-8; J = 72 7.9e-8, 7.4e-8 and 7.3e-8, 8.7e-8 for all, 7.7e-8, 7.3e-8 and 7.3e-8.  (Shorter chains of MFMA are quicker too:
// stencil of 1,000,000 rows, J = 72 573 -> 559 us, J = 200 1,000 -> 970.)
// EDGE: J is not BL * 16.  The last lane with columns begins where it ends with the row at the latest; what of a lane's four
// columns is another lane's, or none, is zero.
template <int BL, int CHAINS, bool EDGE>
struct DotColumns {
    static constexpr int ROWS = 64 / BL;  // of X2T, in a batch
    uint32_t row_bytes;
    int32_t first;
    bool keep[4];
    __device__ __forceinline__ explicit DotColumns(int32_t J) : row_bytes((uint32_t)J * 4u)
    {
        const int32_t c = (int32_t)(threadIdx.x % (4 * BL)) * 4;
        first = EDGE && c + 4 > J ? J - 4 : c;
#pragma unroll
        for (int v = 0; v < 4; ++v) keep[v] = !EDGE || (c < J && first + v >= c);
    }
    // offset: of the row, in bytes
    __device__ __forceinline__ Vec<4> load_row(const float* __restrict__ base, uint32_t offset) const
    {
        return load_vec<4>(reinterpret_cast<const float*>(reinterpret_cast<const char*>(base) + (offset + (uint32_t)first * 4u)));
    }
    __device__ __forceinline__ void own(Vec<4> (&x)[4]) const
    {
        if constexpr (EDGE) {
#pragma unroll
            for (int m = 0; m < 4; ++m)
#pragma unroll
                for (int v = 0; v < 4; ++v) x[m].v[v] = keep[v] ? x[m].v[v] : 0.0f;
        }
    }
    // the quad's rows of X1 (past the last row of the matrix: that one), read once and never again
    __device__ __forceinline__ void load_quad(Vec<4> (&x)[4], const float* __restrict__ X1, int32_t row_first, int32_t M) const
    {
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const int32_t row = row_first + m < M ? row_first + m : M - 1;
            const native_f4 t = __builtin_nontemporal_load(reinterpret_cast<const native_f4*>(X1 + (int64_t)row * (row_bytes / 4) + first));
            x[m].v[0] = t.x; x[m].v[1] = t.y; x[m].v[2] = t.z; x[m].v[3] = t.w;
        }
    }
    __device__ __forceinline__ void turn_quad(Vec<4> (&x)[4]) const
    {
        own(x);
        transpose_fours(x);
    }
};

// Products of the quad's rows with a batch of rows of X2T, of which offset[m] is number 4 * p + m's: a lane gets row dot_row's times
// number dot_number's, where dot_here.
template <int BL>
__device__ __forceinline__ int dot_row(int lane)
{
    return BL == 16 ? lane / 16 % 2 * 2 + lane / 32 : lane / 4 % 2 * 2 + lane / 16 % 2;
}
template <int BL>
__device__ __forceinline__ int dot_number(int lane) { return lane / (4 * BL) * 4 + lane % 4; }
template <int BL>
__device__ __forceinline__ bool dot_here(int lane) { return lane % 16 < (BL == 16 ? 4 : 8); }

template <int BL, int CHAINS, bool EDGE>
__device__ __forceinline__ float quad_dots(const Vec<4> (&x1)[4], const uint32_t (&offset)[4], const float* __restrict__ X2T,
                                           const DotColumns<BL, CHAINS, EDGE>& columns)
{
    Vec<4> x2[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) x2[m] = columns.load_row(X2T, offset[m]);
    columns.own(x2);
    transpose_fours(x2);
    constexpr int EACH = 4 / CHAINS;
    f32x4 part[CHAINS];
#pragma unroll
    for (int n = 0; n < CHAINS; ++n) {
        part[n] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int t = n * EACH; t < (n + 1) * EACH; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) part[n] = __builtin_amdgcn_mfma_f32_4x4x1f32(x1[t].v[v], x2[t].v[v], part[n], 0, 0, 0);
        if (n % 2 == 1) part[n - 1] += part[n];
    }
    f32x4 acc = part[0];
    if constexpr (CHAINS == 4) acc += part[2];
    if constexpr (BL == 16) return sum_every_fourth(fold_rows(fold_halves(acc[0], acc[1]), fold_halves(acc[2], acc[3])));
    const float x = sum_every_fourth(fold_rows(acc[0], acc[1])), y = sum_every_fourth(fold_rows(acc[2], acc[3]));
    return threadIdx.x / 4 % 2 ? y : x;
}

// Stored entries [begin, end) of the quad's rows one by one
template <int BL, int CHAINS, bool EDGE>
__device__ __forceinline__ void quad_entries(const SpmmArgs& a, const float* __restrict__ X1, float* __restrict__ out,
                                             const DotColumns<BL, CHAINS, EDGE>& columns, int32_t row_first, int32_t begin, int32_t end)
{
    constexpr int ROWS = DotColumns<BL, CHAINS, EDGE>::ROWS;
    const int lane = threadIdx.x % kWave;
    const int32_t M = (int32_t)a.M;
    Vec<4> x1[4];
    columns.load_quad(x1, X1, row_first, M);
    columns.turn_quad(x1);
    for (int i = 0; i < kQuad && row_first + i < M; ++i) {
        const int32_t row_begin = a.rowptr[row_first + i], row_end = a.rowptr[row_first + i + 1];
        const int32_t from = row_begin > begin ? row_begin : begin, to = row_end < end ? row_end : end;
        for (int32_t e = from; e < to; e += ROWS) {
            uint32_t offset[4];
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const int32_t at = e + lane / (4 * BL) * 4 + m;
                offset[m] = (uint32_t)load_stream(a.colidx + (at < to ? at : to - 1)) * columns.row_bytes;
            }
            const float dot = quad_dots<BL, CHAINS, EDGE>(x1, offset, a.B, columns);
            const int32_t at = e + dot_number<BL>(lane);
            if (dot_row<BL>(lane) == i && dot_here<BL>(lane) && at < to)
                __builtin_nontemporal_store(load_stream(a.vals + at) * dot, out + at);
        }
    }
}

// A tile's part of a quad of `tile` or more entries: the quad that the tile begins in (row: of the tile's first entry),
// with what the tile in front has of it where it begins there.  Thread t brings tile number t of up to kTileRowBatch.
template <int BL, int CHAINS, bool EDGE>
__device__ __forceinline__ void tiles_of_long_quads(const SpmmArgs& a, const float* __restrict__ X1, float* __restrict__ out,
                                                    const DotColumns<BL, CHAINS, EDGE>& columns, bool have, int32_t row,
                                                    int32_t tile_start, int32_t tile)
{
    const int32_t M = (int32_t)a.M;
    const int32_t row_first = row / kQuad * kQuad;
    int32_t begin = 0, end = 0;
    if (have) {
        const int32_t quad_begin = a.rowptr[row_first], quad_end = a.rowptr[row_first + kQuad < M ? row_first + kQuad : M];
        if (quad_end - quad_begin >= tile) {
            begin = quad_begin > tile_start - tile ? quad_begin : tile_start;
            end = quad_end - tile_start < tile ? quad_end : tile_start + tile;
        }
    }
    for (unsigned long long left = __ballot(end > begin); left != 0; left &= left - 1) {
        const int l = __ffsll((unsigned long long)left) - 1;
        quad_entries<BL, CHAINS, EDGE>(a, X1, out, columns, __builtin_amdgcn_readlane(row_first, l),
                               __builtin_amdgcn_readlane(begin, l), __builtin_amdgcn_readlane(end, l));
    }
}

// Turns of a workgroup: blocks of kWavesPerBlock quads one after the other, each with the next one's entries on their way.
constexpr uint32_t kQuadTurns = 4;
constexpr uint32_t kQuadDies = 8;
constexpr int kQuadBlock = kWavesPerBlock * kQuad;  // rows
__host__ __device__ constexpr uint32_t quad_blocks(int64_t M) { return (uint32_t)((M + kQuadBlock - 1) / kQuadBlock); }
__host__ __device__ constexpr uint32_t quad_turns(int64_t M) { return (quad_blocks(M) + kQuadDies - 1) / kQuadDies; }  // of a die
__host__ __device__ constexpr uint32_t quad_workgroups(int64_t M, uint32_t resident)  // resident: of a die
{
    const uint32_t round = resident * kQuadTurns;
    return ((quad_turns(M) + round - 1) / round) * resident * kQuadDies;
}

// Records of a quad in the order of their columns: how many (with places that stay empty), and which each of a lane's entries
// goes into.  Columns that do not ascend in some row: as many as entries, in the entries' order.  Lane: entries number q of the
// rows half and 2 + half.
__device__ __forceinline__ int list_quad(QuadDots& lds, const int32_t (&col)[2], int (&place_of)[2], int total, int half, int q)
{
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        lds.row_col[2 * u + half][1 + q] = col[u];
        if (q == 0) lds.row_col[2 * u + half][0] = -1;
    }
    wave_lds_order();
    int before[2][kQuad];   // of row (i + k) % 4, the columns below this one of row i
    uint32_t opens[kQuad];  // bit q: the row's entry q opens a record
    bool ascends = true;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int i = 2 * u + half;
        const bool have = col[u] != kNoColumn;
        ascends = ascends && (!have || lds.row_col[i][q] < col[u]);
        before[u][0] = q;
#pragma unroll
        for (int k = 1; k < kQuad; ++k) before[u][k] = below(lds.row_col[(i + k) % kQuad] + 1, col[u]);
        const bool found = i > 0 && lds.row_col[(i + 3) % kQuad][1 + before[u][3]] == col[u];
        const unsigned long long here = __ballot(have && !found);
        opens[2 * u] = (uint32_t)here;
        opens[2 * u + 1] = (uint32_t)(here >> 32);
    }
    if (__ballot(!ascends) != 0) {
        const unsigned long long in0 = __ballot(col[0] != kNoColumn), in1 = __ballot(col[1] != kNoColumn);
        const int len0 = __popc((uint32_t)in0), len1 = __popcll(in0) - len0, len2 = __popc((uint32_t)in1);
        place_of[0] = (half ? len0 : 0) + q;
        place_of[1] = len0 + len1 + (half ? len2 : 0) + q;
        return total;
    }
    int records = 0;
#pragma unroll
    for (int i = 0; i < kQuad; ++i) records += __popc(opens[i]);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        place_of[u] = 0;
#pragma unroll
        for (int k = 0; k < kQuad; ++k) {
            const uint32_t theirs = half ? opens[(2 * u + 1 + k) % kQuad] : opens[(2 * u + k) % kQuad];
            place_of[u] += __popc(__builtin_amdgcn_ubfe(theirs, 0u, (uint32_t)before[u][k]));
        }
    }
    return records;
}

// This workgroup's quads of less than `tile` entries
template <int BL, int CHAINS, bool EDGE>
__device__ __forceinline__ void sddmm_quads(const SpmmArgs& a, const float* __restrict__ X1, float* __restrict__ out,
                                            const DotColumns<BL, CHAINS, EDGE>& columns, QuadDots& lds, int32_t tile, uint32_t resident)
{
    constexpr int PER_LANE = 2;  // entries of the quad per lane: number q of the rows half and 2 + half
    int lane = threadIdx.x % kWave;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const int32_t M = (int32_t)a.M;
    const uint32_t die = blockIdx.x % kQuadDies, blocks = quad_blocks(a.M), per_die = quad_turns(a.M);
    // (27-point stencils, G = 16, in one run of rows for each die and so: 1,000,000 rows, J = 256 1,022 and 991 us; 200 x 200 x 12
    // points, J = 128 250 and 245, J = 256 569 and 484; 212,040 rows, J = 72 122.9 and 123.3, J = 256 204 and 201)
    uint32_t share = 0;
    if (a.M * columns.row_bytes > kQuadDies * kDealBytes)  // (else a die's run of rows of X2T fits its L2)
        share = (plane_share(a, kQuadDies, columns.row_bytes) + kQuadBlock / 2) / kQuadBlock;

    // first row of this wavefront's quad in a turn (M: none), and its row pointers, number l in lane l
    auto quad_of = [&](uint32_t turn) {
        if (turn >= per_die) return M;
        const uint32_t block = die_block(share, die, turn, blocks, kQuadDies);
        const int64_t r = (int64_t)block * kQuadBlock + wave * kQuad;
        return block < blocks && r < M ? (int32_t)r : M;
    };
    auto pointers_of = [&](int32_t row_first) {
        const int64_t r = (int64_t)row_first + (lane < kQuad ? lane : kQuad);
        return a.rowptr[r < M ? r : M];
    };
    struct Entries {
        int32_t begin[PER_LANE], len[PER_LANE];  // of this lane's rows
        int32_t total, len_first;                // of the quad, of its first row
        bool small;                              // every row has fewer than kQuadRow
    };
    auto entries_of = [&](int32_t pointers) {
        const int half = lane / kQuadRow;
        int32_t p[kQuad + 1];
#pragma unroll
        for (int i = 0; i <= kQuad; ++i) p[i] = __builtin_amdgcn_readlane(pointers, i);
        Entries e;
        e.small = true;
#pragma unroll
        for (int i = 0; i < kQuad; ++i) e.small = e.small && p[i + 1] - p[i] < kQuadRow;
#pragma unroll
        for (int u = 0; u < PER_LANE; ++u) {
            e.begin[u] = half ? p[2 * u + 1] : p[2 * u];
            e.len[u] = half ? p[2 * u + 2] - p[2 * u + 1] : p[2 * u + 1] - p[2 * u];
        }
        e.total = p[kQuad] - p[0];
        e.len_first = p[1] - p[0];
        return e;
    };
    int32_t next_col[PER_LANE];
    float next_val[PER_LANE];
    auto fetch = [&](const Entries& e) {
        const int q = lane % kQuadRow;
#pragma unroll
        for (int u = 0; u < PER_LANE; ++u) {
            next_col[u] = kNoColumn;
            next_val[u] = 0.0f;
            if (e.small && q < e.len[u]) {
                next_col[u] = load_stream(a.colidx + e.begin[u] + q);
                next_val[u] = load_stream(a.vals + e.begin[u] + q);
            }
        }
    };

    // the next quad's entries are on their way while this one is multiplied out, and the row pointers of the one behind it
    const uint32_t wg = blockIdx.x / kQuadDies;
    uint32_t turn = wg / resident * (resident * kQuadTurns) + wg % resident;
    const uint32_t turn_end = turn + kQuadTurns * resident;
    int32_t next_row = quad_of(turn), after_row = quad_of(turn + resident);
    int32_t next_pointers = pointers_of(next_row), after_pointers = pointers_of(after_row);
    fetch(entries_of(next_pointers));
    for (; turn < turn_end; turn += resident) {
        asm volatile("" : "+v"(lane));  // (what follows from it is formed anew for every quad: it takes a score of registers)
        const int half = lane / kQuadRow, q = lane % kQuadRow;
        const int32_t row_first = next_row;
        int32_t col[PER_LANE];
        float val[PER_LANE];
#pragma unroll
        for (int u = 0; u < PER_LANE; ++u) {
            col[u] = next_col[u];
            val[u] = next_val[u];
        }
        int32_t pointers = next_pointers;
        next_row = after_row;
        next_pointers = after_pointers;
        fetch(entries_of(next_pointers));
        after_row = turn + 2 * resident < turn_end ? quad_of(turn + 2 * resident) : M;
        after_pointers = pointers_of(after_row);
        const Entries e = entries_of(pointers);
        if (e.total == 0) continue;
        if (!e.small) {
            const int32_t begin = __builtin_amdgcn_readlane(pointers, 0);
            if (e.total < tile) quad_entries<BL, CHAINS, EDGE>(a, X1, out, columns, row_first, begin, begin + e.total);
            continue;
        }
        Vec<4> x1[4];
        columns.load_quad(x1, X1, row_first, M);
        wave_lds_order();  // the last quad's results have been read
        const int32_t first_col = __shfl(col[0], q), next_of_first = __shfl(col[0], q + 1);  // of the quad's first row
        const int gap = next_of_first - first_col;
        bool alike = first_col == kNoColumn || gap > 0;
#pragma unroll
        for (int u = 0; u < PER_LANE; ++u)
            alike = alike && col[u] == (first_col == kNoColumn ? kNoColumn : first_col + 2 * u + half);
        const bool shifted = __ballot(!alike) == 0;
        int records, place_of[PER_LANE];  // where this lane's entries go
        if (shifted) {
            // Every row is the first one shifted: an entry of that opens four records, or as many as there are columns to the
            // next one, and entry q of row i has the i-th record from there on, or beyond.
            const int less = first_col != kNoColumn && gap < kQuad ? kQuad - gap : 0;
            const uint32_t ones = (uint32_t)__ballot(less & 1), twos = (uint32_t)__ballot(less & 2);
            records = kQuad * e.len_first - __popc(ones) - 2 * __popc(twos);
            const int before = kQuad * q - __popc(__builtin_amdgcn_ubfe(ones, 0u, (uint32_t)q)) -
                               2 * __popc(__builtin_amdgcn_ubfe(twos, 0u, (uint32_t)q));
#pragma unroll
            for (int u = 0; u < PER_LANE; ++u) place_of[u] = before + 2 * u + half;
        } else {
            records = list_quad(lds, col, place_of, e.total, half, q);
        }
        {
            // (places of no record gather some column of the quad)
            const unsigned long long in0 = __ballot(col[0] != kNoColumn), in1 = __ballot(col[1] != kNoColumn);
            const int32_t some = in0 ? __builtin_amdgcn_readlane(col[0], __ffsll(in0) - 1) : __builtin_amdgcn_readlane(col[1], __ffsll(in1) - 1);
#pragma unroll
            for (int u = 0; u <= (kDotRecords + kDotBatch - 1) / kWave; ++u) {
                const int at = lane + u * kWave;
                if (at < kDotRecords + kDotBatch && u * kWave < records + kDotBatch) {
                    lds.offset[at] = (uint32_t)some * columns.row_bytes;
                    lds.place[at] = ~0u;
                }
            }
        }
        wave_lds_order();
#pragma unroll
        for (int u = 0; u < PER_LANE; ++u)
            if (col[u] != kNoColumn) {
                lds.offset[place_of[u]] = (uint32_t)col[u] * columns.row_bytes;
                reinterpret_cast<uint8_t*>(lds.place)[place_of[u] * 4 + 2 * u + half] = (uint8_t)q;
            }
        wave_lds_order();

        columns.turn_quad(x1);
        const int row_mine = dot_row<BL>(lane), number_mine = dot_number<BL>(lane);
        for (int at = 0; at < records; at += DotColumns<BL, CHAINS, EDGE>::ROWS) {
            const uint4 of = *reinterpret_cast<const uint4*>(&lds.offset[at + lane / (4 * BL) * 4]);
            const uint32_t offset[4] = {of.x, of.y, of.z, of.w};
            const uint32_t place = lds.place[at + number_mine] >> (8 * row_mine) & 0xffu;
            const float dot = quad_dots<BL, CHAINS, EDGE>(x1, offset, a.B, columns);
            if (dot_here<BL>(lane) && place != kNoPlace) lds.out[row_mine][place] = dot;
        }
        wave_lds_order();
        asm volatile("" : "+v"(pointers));  // (formed anew: kept over the products, they cost four registers)
        const Entries again = entries_of(pointers);
#pragma unroll
        for (int u = 0; u < PER_LANE; ++u)
            if (q < again.len[u]) __builtin_nontemporal_store(val[u] * lds.out[2 * u + half][q], out + again.begin[u] + q);
    }
}

}  // namespace sgap
