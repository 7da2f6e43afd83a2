// Block-scaled MXFP4 GEMM  C = A * B^T  with the Macro Block Scaling correction, for gfx950: argument checks and
// the choice of kernel.  The kernels are the main template (mx_gemm_ring.h: fast form in mx_gemm_wide.hip and
// mx_gemm_mbs.hip, general form in mx_gemm_general.hip and mx_gemm_wide.hip) and the few-row kernel
// (mx_gemm_skinny.h; mx_gemm_skinny.hip, mx_gemm_skinny_rows.hip, mx_gemm_skinny_fused.hip, mx_gemm_skinny_grouped.hip).
#include "mx_gemm_shared.h"
#include "mx_internal.h"

#include <stdio.h>

#include <algorithm>

namespace mx {
namespace {

// force_shape (mx_internal_gemm only; the public entry points pass -1 = automatic): 2 / 6 / 7 = fast form without
// MBS on 256x256 / 256x128 / 128x128 tiles, 3 / 4 = fast form with MBS on 256x128 / 128x128 tiles, 5 = few-row
// kernel, 8 / 9 = general form (row pieces through registers) on 256x128 / 128x128 tiles, 11 / 12 = fast form with MBS on both operands / general form with MBS on 64x128 tiles, 17 / 18 / 19 = few-row
// kernel on tiles of 64 rows and 16 / 32 / 64 columns.
// Grouped problems with words: what the kernels take, in us, from rows, groups and the number of macro blocks; the launch cannot know the
// routing, so a group is taken to end half a tile-row short and every group to have rows.  Fitted to Zipf and equal routings over 8, 32
// and 64 groups of 768, 1536 and 2880 squared with 4 to 4096 rows per group.
struct GroupedPrices {
    double big, small, few;  // 256 x 128 tiles, 64 x 128 tiles, the few-row kernel
};
GroupedPrices grouped_prices(int64_t M, int64_t N, int64_t K, int64_t num_groups) {
    const double busy = (double)std::min(num_groups, M), st = (double)((K + kMacro - 1) / kMacro), cols = (double)((N + 127) / 128);
    const double weights_mb = busy * N * K * 0.54e-6;
    const double x256 = (M / 256.0 + 0.5 * busy) * cols / 256.0, x64 = (M / 64.0 + 0.5 * busy) * cols / 256.0;
    GroupedPrices p;
    p.big = std::max(1.0, x256) * (4.7 + 0.82 * st);
    p.small = 2.5 + std::max(std::max(x64, 1.2) * (1.2 + 0.29 * st), weights_mb / 3.4);  // (two workgroups share a compute unit)
    p.few = std::max(2.0 + 0.3 * st + (M / 32.0 + 0.5 * busy) * ((N + 31) / 32) * std::max(0.005, 0.36e-3 * st), weights_mb / 4.2);
    return p;
}
// 64 x 128 tiles for a grouped problem with words: up to 128 rows per group they leave less empty than 256 x 128 tiles, and two of
// their workgroups fit a compute unit; above, where they are cheaper by more than the prices are wrong.  GEMM alone, Zipf routing,
// 256 x 128 (or 128 x 128, where those were taken) and 64 x 128: 64 groups of 1536 x 1536, 4096 rows 55.6 and 32.3 us, 8192 rows 57.9 and
// 45.8; 64 of 2880 x 2880, 4096 rows 157 and 111; 8 of 768 x 768, 1024 rows 7.4 and 6.4; past the line 32 of 1536 x 1536, 16384 rows
// 55 and 63, 8 of 2880 x 2880, 2048 rows 24 and 32.
bool grouped_small_tile(int64_t M, int64_t N, int64_t K, int64_t num_groups) {
    // (their grid, two workgroups of 256 for one of 512, has to stay below 2^32 work-items: 3.3 million groups of 300 rows do not)
    if ((M / 64 + num_groups) * ((N + 127) / 128) >= (int64_t)1 << 24) return false;
    const GroupedPrices p = grouped_prices(M, N, K, num_groups);
    return M <= 128 * num_groups || p.small < 0.85 * p.big;
}

// Which kernel form and tile shape (the codes above) takes a problem with K > 0.  Tiles run in rounds of one per compute
// unit: rounds x tile area / efficiency (the small tile reaches about 0.8 of the large tile's rate per output
// with MBS, 0.85 / 0.72 without; measured) picks the tile.  With words on both operands, ungrouped, 64 x 128 tiles
// take what they cover in one round: twice the compute units have work, and a tile of few rows is bound by a stage's serial chain
// and not by its arithmetic.  GEMM alone, 64 x 128 against 128 x 128: 333 x 4096 x 4096 14.0 and 17.6 us, 512 x 4096 x 4096 14.1
// and 17.8, 333 x 4000 x 2880 11.1 and 13.7; past one round 800 x 4096 x 4096 20.4 and 19.1, 1024 x 4096 x 2880 17.7 and 15.9.
//
// The general form fetches a row's pieces through registers, which any K % 32 == 0 at any address can use: it costs what the fast form
// does, where single bytes (K % 64 = 32 once took them) keep the texture-address unit busy three times as long as the codes and leave
// LDS for 128 x 128 tiles only.  With the quantizer: 305 x 1205 x 1632 21.8 -> 13.3 us, 5680 x 1130 x 6880 110 -> 75.
int choose_shape(int64_t M, int64_t N, int64_t K, int64_t num_groups, bool use_mbs, bool ring_ok, bool skinny_ok, int row_tile_cols,
                 bool tile64_ok, bool c_lines) {
    const int64_t t256x128 = ((M + 255) / 256) * ((N + 127) / 128), t128 = ((M + 127) / 128) * ((N + 127) / 128);
    const double big = 2.0 * ((t256x128 + 255) / 256) / (use_mbs ? 1.0 : 0.85),
                 small = ((t128 + 255) / 256) / (use_mbs ? 0.8 : 0.72);
    if (skinny_ok) return 5;
    if (row_tile_cols > 0) return row_tile_cols == 16 ? 17 : row_tile_cols == 32 ? 18 : 19;
    if (num_groups > 0 && use_mbs) return grouped_small_tile(M, N, K, num_groups) ? 12 : 8;
    if (tile64_ok && ((M + 63) / 64) * ((N + 127) / 128) <= 256) return ring_ok ? 11 : 12;
    // Past one round, with words on both operands or in the general form: by the kernels' prices (mx_gemm_shared.h)
    // (256 x 128, 128 x 128 and 64 x 128 tiles, us: 2316 x 3815 x 5120 65, 69, 60; 5676 x 1854 x 512 18.2, 19.0, 16.8;
    // 1579 x 2784 x 1024 11.2, 14.6, 12.5; 1367 x 3890 x 7296 50, 73, 61)
    // The prices were fitted to rows of C on any element.  Rows on whole 128-byte lines (c_lines) cost the larger tile's epilogue less, and near a tie
    // the price picks the smaller: one round of 256 x 128 against more than one of 64 x 128 (two on a compute unit), K = 512, in bf16 1.00 and 1.11 of the fastest
    // tile's time in the mean of 103 problems (784 x 6272 x 512 7.9 and 9.1 us), longer K more; in the general form one round of 128 x 128 against 64 x 128,
    // K < 640, to 1024, to 1536, to 2560 1.00 and 1.05, 1.03, 1.03, 1.01 (from 2560 on even, then 64 x 128 gains).
    if (c_lines && tile64_ok && t256x128 <= 256 && ((M + 63) / 64) * ((N + 127) / 128) > 512) return ring_ok ? 3 : 8;
    if (c_lines && tile64_ok && !ring_ok && t128 <= 256 && K < 2048) return 9;
    if (more_than_a_round_of_64x128(M, N) && (tile64_ok || (!use_mbs && !ring_ok))) {
        static const TilePrice kFast[3] = {{256, 128, 256, 0.7, 3.40, 0.003, 4.91, 0.726}, {128, 128, 256, 0.8, 2.72, 0.018, 3.26, 0.480}, {64, 128, 512, 0.4, 3.83, 0.098, 2.29, 0.453}};
        static const TilePrice kGeneral[3] = {{256, 128, 256, 0.7, 2.82, 0.030, 5.48, 0.815}, {128, 128, 256, 0.8, 2.64, 0.021, 3.25, 0.592}, {64, 128, 512, 0.6, 3.27, 0.100, 2.81, 0.523}};
        static const TilePrice kPlain[2] = {{256, 128, 256, 0.8, 3.27, -0.051, 4.71, 0.651}, {128, 128, 256, 0.4, 3.00, 0.146, 1.93, 0.313}};
        if (!use_mbs) return kPlain[0].of(M, N, K) <= kPlain[1].of(M, N, K) ? 8 : 9;
        const TilePrice* t = ring_ok ? kFast : kGeneral;
        const double a = t[0].of(M, N, K), b = t[1].of(M, N, K), c = t[2].of(M, N, K);
        if (a <= b && a <= c) return ring_ok ? 3 : 8;
        if (b <= c) return ring_ok ? 4 : 9;
        return ring_ok ? 11 : 12;
    }
    if (ring_ok) return use_mbs ? (big <= small ? 3 : 4) : 2;  // (without MBS the launcher also has 256 x 256 tiles)
    return big <= small ? 8 : 9;
}

// The few-row kernel's tile for M <= 64: the smallest fm that covers the rows; fn so that the launch has about one
// workgroup per compute unit (one workgroup's wavefronts hold all of its weights in flight, so a second round costs a
// second round trip to memory, and every workgroup reads - or, fused, quantizes - all of A).  Measured, M = 16 / K = 4096,
// fn = 1, 2, 4: N = 4096 5.1, 5.6, 7.0 us; N = 14336 11.0, 10.5, 9.1 us (fused 17.5, 15.1, 11.3).
struct SkinnyPlan {
    int fm, fn, form;
};
SkinnyPlan plan_skinny(int64_t M, int64_t N, int64_t K, bool ring_ok, bool pairs_ok) {
    SkinnyPlan p;
    p.fm = M <= 16 ? 1 : M <= 32 ? 2 : 4;
    // (K % 512 == 0: shares of whole chunks where a wavefront's share comes out as a multiple of four macro blocks)
    p.form = ring_ok ? (((K / kMacro + 7) / 8) % 4 == 0 ? 0 : 1) : pairs_ok ? 2 : 3;
    const int64_t frags = (N + 15) / 16;
    p.fn = frags > 2 * 256 ? 4 : frags > 256 ? 2 : 1;
    // (what the forms with one LDS dword per piece have room for)
    if (p.form == 2 && p.fn > 2) p.fn = 2;
    if (p.form == 3) p.fn = 1;
    return p;
}
// Grouped problems take the few-row kernel up to this many rows per group on average: it streams the weights once per
// 32 rows.  Zipf routing, 8, 16 and 32 rows per group, few-row kernel and 64 x 128 tiles: 32 groups of 2880 x 2880 34.9, 43.4, 54.2 and 43.1,
// 46.2, 48.8 us; 64 of 1536 x 1536 22.0, 25.8, 33.0 and 22.3, 24.4, 25.5; 64 of 768 x 768 9.0, 11.7, 14.7 and 8.3, 8.4, 8.5.  All rows
// in one group, 8, 16 and 32 per group on average: 32 of 2880 x 2880 13, 22, 35 against 16, 17, 19; 64 of 1024 x 1024 7, 11, 17
// against 9, 9, 9.  The launch cannot know the routing: it goes by what routers produce and loses up to half there.
//
// Where the tiles are faster they are not always as exact: with words, their sum over K is one chain of macro blocks, the few-row kernel's is
// split over four wavefronts.  Error against 64 bits, tiles over few rows: K = 512 0.92, 640 0.97, 672 to 768 1.003 to 1.02, 800 to 896
// 0.99 to 1.0, 1024 1.02, 1536 1.11, 2880 1.24, 8192 1.46.  So tiles take up to five macro blocks, and seven, where their price
// is lower by more than the microsecond that prices of small launches are off (few rows and tiles, K = 512: 64 groups, 91 rows in all, N = 4687 47.3 and
// 27.3 us; 128, 211 rows, N = 2582 54.2 and 32.0; within the microsecond 16, 92 rows, N = 2026 5.2 and 7.0; 32, 143 rows, N = 963 5.2 and 6.2).
constexpr int64_t kFewRowsPerGroup = 32;

// Whether the few-row kernel takes a problem that is not grouped and has at most 64 rows.  With K % 512 == 0 and aligned
// arrays (forms 0 and 1): always.  In the forms 2 and 3 a workgroup has LDS for 32 and 16 columns only, so many columns
// are many rounds, and each costs a round trip to memory, while the main kernel's 64 x 128 (without words on both sides
// 128 x 128) tiles cover 32768 columns in one round.  More than one round is therefore priced against the main kernel, in
// us, by what both take on the device with weights from memory.  Few-row and main kernel at M = 1, 32, 64, words on both sides:
//   K = 2880   N =  8192  5.8, 7.2, 9.6      and 15.9, 17.1, 17.9;   N = 28672  18.1, 23.8, 32.2   and 17.9, 19.1, 20.0
//   K = 1088   N =  8192  4.4, 5.3, 6.7      and 7.2, 7.4, 7.7;      N = 28672  12.8, 15.8, 20.8   and 9.1, 9.4, 9.8
//   K = 4128   N =  4096  5.8, 8.0, 11.5      and 18.1, 20.5, 19.8;   N = 28672  23.4, 41.1, 67.1   and 26.5, 27.3, 28.9
// Over K of 64 to 8160, N of 1024 to 57344 and 1 to 64 rows the few-row kernel is chosen where it is at most 4 % slower, the
// main kernel where it is at most a third slower: the prices lean to the kernel that had all of these problems before.
bool few_rows_pay(int64_t M, int64_t N, int64_t K, const SkinnyPlan& p, int sides) {
    const bool use_mbs = sides > 0;
    if (p.form <= 1) return true;
    const bool bytes = p.form == 3;
    const int64_t rounds = ((N + 15) / 16 + p.fn * 256 - 1) / (p.fn * 256), tile_rounds = ((N + 127) / 128 + 255) / 256;
    if (rounds == 1) return true;
    const int at = p.fm == 1 ? 0 : p.fm == 2 ? 1 : 2;
    static const double kRound[2][3] = {{1.6, 2.2, 2.8}, {0.8, 1.1, 1.4}}, kRoundPerK[2][3] = {{0.92e-3, 1.14e-3, 1.6e-3}, {0.6e-3, 1.15e-3, 2.0e-3}};
    const double few = 1.7 + rounds * (kRound[bytes][at] + kRoundPerK[bytes][at] * K);
    // Single bytes, K > 1024: tiles only far behind the line of their time.  Their one chain over K is less exact with words than the few-row
    // kernel's eight shares (error against 64 bits, tiles over few rows: K = 992 0.93, 1056 1.01, 2080 1.15, 4128 1.36).
    if (bytes && K > 1024) return few <= (use_mbs ? 4.5 + 6.2e-3 * K : 3.5 + 5.2e-3 * K) * tile_rounds;
    const double tile = use_mbs ? std::max(4.3, 1.5 + 5.5e-3 * K) : std::max(4.0, 1.4 + 4.7e-3 * K);
    // (a further round of the tiles starts while the one before ends, where two workgroups fit a compute unit)
    // (single bytes: the few-row prices are a quarter too high for one row; words on one side only and none take 128 x 128 tiles, for which the
    // tile price is too low.  Few rows and tiles: 45 x 5264 x 352 with words on A 5.9 and 6.8 us, 20 x 8415 x 224 6.1 and 6.5; without words
    // 25 x 6218 x 512 4.9 and 5.7; on the tiles' side of the line 9 x 14974 x 640 with words on B 7.8 and 7.6)
    return few <= tile * (bytes ? (sides == 2 ? 1.25 : sides == 1 ? 1.5 : 1.3) : 1.0) * (0.5 + 0.5 * tile_rounds);
}
// Whether the few-row kernel takes a problem (num_groups: 0 = not grouped; sides: how many operands have words).
bool takes_few_rows(int64_t M, int64_t N, int64_t K, int64_t num_groups, bool ring_ok, bool pairs_ok, int sides) {
    if (num_groups > 0) {
        if (M > kFewRowsPerGroup * num_groups || few_rows_blocks(M, N, num_groups, !pairs_ok) > kFewRowsMaxBlocks) return false;
        const int64_t st = (K + kMacro - 1) / kMacro;
        if (K < 512 || sides == 0 || (st > 5 && st != 7)) return true;
        const GroupedPrices p = grouped_prices(M, N, K, num_groups);
        return p.few <= 1.02 * p.small + 1.0;
    }
    return M <= 64 && K <= 8192 && few_rows_pay(M, N, K, plan_skinny(M, N, K, ring_ok, pairs_ok), sides);
}

// More than 64 rows on the few-row kernel: the columns of its tiles of 64 rows (0: the main kernel).  Its eight wavefronts share K and
// meet no barrier, so a small output with a long K, which leaves most compute units idle on the main kernel's tiles and runs one
// stage of K after the other there, takes a fraction of the time, as long as one round of workgroups covers it.  The wider the tile, the
// longer K has to be.  Main kernel (64 x 128 tiles) and this one, words on both sides, us, K = 512, 2048, 4096, 8192:
//   512 x 512    4.6, 8.1, 14.3, 26.1   16 columns 4.5, 6.0, 7.2, 11.9
//   512 x 1024   4.8, 8.8, 15.4, 26.3   16 columns (two rounds) 5.4, 8.0, 10.2, 18.9   32 columns 5.0, 7.1, 8.9, 13.9
//   1024 x 1024  4.9, 9.5, 15.9, 27.1   32 columns (two rounds) 8.1, 12.0, 15.8, 25.0  64 columns 6.7, 9.7, 12.7, 20.3
// without words 512 x 1024 4.6, 6.7, 13.0, 22.2 and 32 columns 4.6, 6.2, 7.6, 11.8; K = 1056 (single bytes, 16 columns) 512 x 512 7.2 and 5.7.
// From nine macro blocks on: below, a wavefront has one at most, its product is rounded before the sum instead of in the main kernel's one
// multiply-add, and with words the error against 64-bit arithmetic is 7 to 9 % larger (K = 1024 8.1e-8 of the result's norm against 7.5e-8;
// K = 1056 7.7e-8 against 7.8e-8, K = 4096 8.5e-8 against 1.14e-7, K = 8192 9.2e-8 against 1.53e-7; without words the same sums).
int row_tile_columns(int64_t M, int64_t N, int64_t K, int64_t num_groups, bool ring_ok, bool pairs_ok) {
    if (num_groups > 0 || M <= 64 || K <= 1024 || K > 8192) return 0;
    const int64_t rows = (M + 63) / 64, frags = (N + 15) / 16;
    if (rows * frags <= 256) return 16;
    if (rows * ((frags + 1) / 2) <= 256 && (ring_ok || pairs_ok)) return 32;
    if (rows * ((frags + 3) / 4) <= 256 && ring_ok && K >= 3072) return 64;
    return 0;
}

// K = 0, an empty sum: the rows of C become zero, of a grouped problem those that belong to a group.
template <typename T>
__global__ __launch_bounds__(256) void gemm_zero_kernel(GemmArgs g) {
    constexpr int per = 16 / sizeof(T);
    const int64_t rows = g.num_groups > 0 ? min(g.row_offsets[g.num_groups], g.M) : g.M, pieces = (g.N + per - 1) / per;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < rows * pieces; i += (int64_t)gridDim.x * 256) {
        const int64_t n = i % pieces * per;
        T* o = static_cast<T*>(g.C) + i / pieces * g.ldc + n;
        if (n + per <= g.N) {
            *reinterpret_cast<v4i_any*>(o) = v4i{0, 0, 0, 0};
        } else {
            for (int e = 0; n + e < g.N; ++e) o[e] = 0;
        }
    }
}
int launch_gemm_zero(const GemmArgs& g, hipStream_t s) {
    const int64_t pieces = g.c_bf16 ? (g.N + 7) / 8 : (g.N + 3) / 4;
    const unsigned blocks = (unsigned)std::min<int64_t>((g.M * pieces + 255) / 256, 8192);
    if (g.c_bf16) gemm_zero_kernel<uint16_t><<<dim3(blocks), dim3(256), 0, s>>>(g);
    else gemm_zero_kernel<uint32_t><<<dim3(blocks), dim3(256), 0, s>>>(g);
    return launch_status();
}

int launch_gemm(const uint8_t* a_codes, const uint8_t* a_scales, const uint8_t* a_mbs, const uint8_t* b_codes,
                const uint8_t* b_scales, const uint8_t* b_mbs, int num_groups, const int64_t* row_offsets,
                bool grouped, int64_t M, int64_t N, int64_t K, int c_dtype, void* C, int64_t ldc, bool mbs_entry,
                void* stream, int force_shape = -1) {
    if (M < 0 || N < 0 || K < 0 || (K % kBlock) != 0 || ldc < N) return MX_EINVAL;
    if (c_dtype != MX_OUT_F32 && c_dtype != MX_OUT_BF16) return MX_EINVAL;
    if (grouped && num_groups < 0) return MX_EINVAL;
    // (a tile's rows times the bytes of a row must fit the 32-bit offsets of the buffer loads)
    if (K > (int64_t)1 << 22 || M > (int64_t)1 << 30 || N > (int64_t)1 << 30 ||
        (grouped && (int64_t)num_groups * N > (int64_t)1 << 40))
        return MX_EINVAL;
    if (M == 0 || N == 0 || (grouped && num_groups == 0)) return MX_OK;
    if (!C || (grouped && !row_offsets)) return MX_ENULL;
    if (K > 0 && (!a_codes || !a_scales || !b_codes || !b_scales)) return MX_ENULL;
    const size_t esz = c_dtype == MX_OUT_F32 ? 4 : 2;
    if (!aligned(C, esz) || (K > 0 && (!aligned(a_codes, 16) || !aligned(b_codes, 16)))) return MX_EALIGN;
    if (int st = check_device()) return st;

    GemmArgs g;
    g.a_codes = a_codes; g.a_scales = a_scales; g.a_mbs = a_mbs;
    g.b_codes = b_codes; g.b_scales = b_scales; g.b_mbs = b_mbs;
    g.C = C; g.row_offsets = row_offsets;
    g.M = M; g.N = N; g.K = K; g.ldc = ldc;
    g.num_groups = grouped ? num_groups : 0;
    g.tiles_m = g.tiles_n = 0;
    g.c_bf16 = c_dtype == MX_OUT_BF16;
    g.vec_store16 = aligned(C, 16) && (ldc * esz) % 16 == 0;

    hipStream_t s = static_cast<hipStream_t>(stream);
    if (K == 0) return force_shape < 0 ? launch_gemm_zero(g, s) : MX_EINVAL;
    const bool use_mbs = mbs_entry && (a_mbs || b_mbs);
    // Fast form: K in whole groups of four macro blocks and aligned per-row arrays.
    const bool ring_ok = !grouped && (K % 512) == 0 && aligned(a_scales, 16) && aligned(b_scales, 16) &&
                         (!use_mbs || ((!a_mbs || aligned(a_mbs, 4)) && (!b_mbs || aligned(b_mbs, 4))));
    // (few-row kernel: pairs of E8M0 bytes; else single ones)
    const bool pairs_ok = (K % 64) == 0 && aligned(a_scales, 2) && aligned(b_scales, 2);
    const bool skinny_ok = takes_few_rows(M, N, K, g.num_groups, ring_ok, pairs_ok, use_mbs ? (a_mbs != nullptr) + (b_mbs != nullptr) : 0);
    const bool tile64_ok = !grouped && a_mbs && b_mbs && mbs_entry;
    int shape = choose_shape(M, N, K, g.num_groups, use_mbs, ring_ok, skinny_ok, row_tile_columns(M, N, K, g.num_groups, ring_ok, pairs_ok), tile64_ok,
                             aligned(C, 128) && (ldc * esz) % 128 == 0);
    if (force_shape >= 0) shape = force_shape;
    // (the checks below only matter for forced shapes)
    if (shape == 5) {
        if (!grouped && (M > 64 || K > 8192)) return MX_EINVAL;
        if (grouped) return launch_gemm_skinny_grouped(g, use_mbs, !pairs_ok, s);
        const SkinnyPlan p = plan_skinny(M, N, K, ring_ok, pairs_ok);
        return launch_gemm_skinny_tile(g, use_mbs, p.fm, p.fn, p.form, s);
    }
    if (shape >= 17 && shape <= 19) {
        if (grouped || K > 8192) return MX_EINVAL;
        return launch_gemm_skinny_rows(g, use_mbs, shape == 17 ? 1 : shape == 18 ? 2 : 4, plan_skinny(64, N, K, ring_ok, pairs_ok).form, s);
    }
    if (shape == 11 || shape == 12) {
        if (!use_mbs || (shape == 11 && (!ring_ok || !a_mbs || !b_mbs))) return MX_EINVAL;
        return shape == 11 ? launch_gemm_mbs_ring(g, 2, s) : launch_gemm_mbs_general(g, 2, s);
    }
    if (shape == 8 || shape == 9) return use_mbs ? launch_gemm_mbs_general(g, shape - 8, s) : launch_gemm_wide_general(g, shape - 8, s);
    const bool plain_shape = shape == 2 || shape == 6 || shape == 7;
    if (shape < 2 || shape > 7 || !ring_ok || plain_shape == use_mbs) return MX_EINVAL;
    if (plain_shape) return launch_gemm_wide(g, force_shape < 0 ? 0 : shape == 2 ? 1 : shape == 6 ? 2 : 3, s);
    return launch_gemm_mbs_ring(g, shape == 4, s);
}

// Few-row GEMM with A given as bf16 and quantized inside the kernel (mx_gemm_skinny_fused.hip).
int launch_gemm_quantize_a(const void* a_bf16, int64_t lda, int rule, int a_use_mbs, const uint8_t* b_codes,
                           const uint8_t* b_scales, const uint8_t* b_mbs, int64_t M, int64_t N, int64_t K, int c_dtype,
                           void* C, int64_t ldc, void* stream) {
    if (M < 0 || N < 0 || K < 0 || (K % kBlock) != 0 || ldc < N || lda < K) return MX_EINVAL;
    if (c_dtype != MX_OUT_F32 && c_dtype != MX_OUT_BF16) return MX_EINVAL;
    if (rule != MX_RULE_OCP && rule != MX_RULE_FLOOR && rule != MX_RULE_OAS) return MX_EINVAL;
    if (N > (int64_t)1 << 30) return MX_EINVAL;
    if (M == 0 || N == 0) return MX_OK;
    if (!C || !a_bf16 || !b_codes || !b_scales) return MX_ENULL;
    const size_t esz = c_dtype == MX_OUT_F32 ? 4 : 2;
    if (!aligned(C, esz) || !aligned(a_bf16, 16) || (lda % 8) != 0 || !aligned(b_codes, 16)) return MX_EALIGN;
    // what the few-row kernel covers; larger problems take mx_quantize_mbs + mx_gemm_mbs
    if (M > 64 || K == 0 || (K % 512) != 0 || K > 8192 || !aligned(b_scales, 16) || (b_mbs && !aligned(b_mbs, 4)) ||
        ((M - 1) * lda + K) * 2 >= (int64_t)1 << 31)
        return MX_EUNSUPPORTED;
    if (int st = check_device()) return st;
    GemmArgs g = {};
    g.b_codes = b_codes; g.b_scales = b_scales; g.b_mbs = b_mbs;
    g.C = C;
    g.M = M; g.N = N; g.K = K; g.ldc = ldc;
    g.c_bf16 = c_dtype == MX_OUT_BF16;
    const SkinnyPlan p = plan_skinny(M, N, K, true, true);
    return launch_gemm_skinny_fused_tile(g, a_bf16, lda, rule, a_use_mbs != 0, p.fm, p.fn, p.form, static_cast<hipStream_t>(stream));
}

}  // namespace
}  // namespace mx

extern "C" {

int mx_gemm_mbs_quantize_a(const void* a_bf16, int64_t lda, mx_rule_t rule, int a_use_mbs, const uint8_t* b_codes,
                           const uint8_t* b_scales, const uint8_t* b_mbs_or_null, int64_t M, int64_t N, int64_t K,
                           mx_dtype_t c_dtype, void* C, int64_t ldc, void* stream) {
    return mx::launch_gemm_quantize_a(a_bf16, lda, (int)rule, a_use_mbs, b_codes, b_scales, b_mbs_or_null, M, N, K,
                                      (int)c_dtype, C, ldc, stream);
}

int mx_gemm(const uint8_t* a_codes, const uint8_t* a_scales, const uint8_t* b_codes, const uint8_t* b_scales,
            int64_t M, int64_t N, int64_t K, mx_dtype_t c_dtype, void* C, int64_t ldc, void* stream) {
    return mx::launch_gemm(a_codes, a_scales, nullptr, b_codes, b_scales, nullptr, 0, nullptr, false, M, N, K,
                           (int)c_dtype, C, ldc, false, stream);
}

int mx_gemm_mbs(const uint8_t* a_codes, const uint8_t* a_scales, const uint8_t* a_mbs_or_null,
                const uint8_t* b_codes, const uint8_t* b_scales, const uint8_t* b_mbs_or_null, int64_t M, int64_t N,
                int64_t K, mx_dtype_t c_dtype, void* C, int64_t ldc, void* stream) {
    return mx::launch_gemm(a_codes, a_scales, a_mbs_or_null, b_codes, b_scales, b_mbs_or_null, 0, nullptr, false, M,
                           N, K, (int)c_dtype, C, ldc, true, stream);
}

int mx_gemm_mbs_grouped(const uint8_t* a_codes, const uint8_t* a_scales, const uint8_t* a_mbs_or_null,
                        const uint8_t* b_codes, const uint8_t* b_scales, const uint8_t* b_mbs_or_null,
                        int32_t num_groups, const int64_t* row_offsets, int64_t M_total, int64_t N, int64_t K,
                        mx_dtype_t c_dtype, void* C, int64_t ldc, void* stream) {
    return mx::launch_gemm(a_codes, a_scales, a_mbs_or_null, b_codes, b_scales, b_mbs_or_null, num_groups,
                           row_offsets, true, M_total, N, K, (int)c_dtype, C, ldc, true, stream);
}

int mx_internal_gemm_plan(int64_t M, int64_t N, int64_t K, int a_has_mbs, int b_has_mbs, int num_groups, char* out, int cap) {
    if (!out || cap <= 0 || M < 0 || N < 0 || K < 0 || (K % mx::kBlock) != 0 || num_groups < 0) return MX_EINVAL;
    const bool use_mbs = a_has_mbs || b_has_mbs, grouped = num_groups > 0;
    if (K == 0) return snprintf(out, (size_t)cap, "gemm_zero_kernel"), MX_OK;
    const bool ring_ok = !grouped && (K % 512) == 0, pairs_ok = (K % 64) == 0;
    const int shape = mx::choose_shape(M, N, K, num_groups, use_mbs, ring_ok, mx::takes_few_rows(M, N, K, num_groups, ring_ok, pairs_ok, (a_has_mbs != 0) + (b_has_mbs != 0)),
                                       mx::row_tile_columns(M, N, K, num_groups, ring_ok, pairs_ok),
                                       !grouped && a_has_mbs && b_has_mbs, N % 64 == 0);  // (C in bf16 and whole)
    const char* sides = a_has_mbs && b_has_mbs ? "MBS words on A and B" : a_has_mbs ? "MBS words on A" : b_has_mbs ? "MBS words on B" : "no MBS";
    const char* what;
    switch (shape) {
        case 2: what = mx::describe_gemm_wide(M, N, K); break;
        case 3: what = a_has_mbs && b_has_mbs ? "gemm_ring_kernel, fast form, 256x128 tile, 8 wavefronts of 64x64"
                                              : "gemm_ring_kernel, fast form, 256x128 tile, 8 wavefronts of 128x32"; break;
        case 4: what = "gemm_ring_kernel, fast form, 128x128 tile, 8 wavefronts of 64x32"; break;
        case 5: what = grouped ? "gemm_skinny_grouped_kernel (few rows per group)" : "gemm_skinny_kernel (few rows)"; break;
        case 17: what = "gemm_skinny_kernel, tiles of 64 rows and 16 columns"; break;
        case 18: what = "gemm_skinny_kernel, tiles of 64 rows and 32 columns"; break;
        case 19: what = "gemm_skinny_kernel, tiles of 64 rows and 64 columns"; break;
        case 11: what = "gemm_ring_kernel, fast form, 64x128 tile, 4 wavefronts of 64x32"; break;
        case 12: what = "gemm_ring_kernel, general form (row pieces through registers), 64x128 tile, 4 wavefronts of 64x32"; break;
        case 8: what = use_mbs ? "gemm_ring_kernel, general form (row pieces through registers), 256x128 tile, 8 wavefronts" : "gemm_ring_kernel, general form (row pieces through registers), 256x128 tile, 4 wavefronts"; break;
        default: what = "gemm_ring_kernel, general form (row pieces through registers), 128x128 tile"; break;
    }
    // (how the few-row kernel fetches E8M0 bytes where a row's pieces are not aligned)
    const bool few = shape == 5 || shape >= 17;
    const char* pieces = !few || ring_ok ? "" : pairs_ok ? ", pairs of scale bytes" : ", single scale bytes";
    snprintf(out, (size_t)cap, "%s%s; %s", what, pieces, sides);
    return MX_OK;
}

int mx_internal_gemm(const uint8_t* a_codes, const uint8_t* a_scales, const uint8_t* a_mbs_or_null,
                     const uint8_t* b_codes, const uint8_t* b_scales, const uint8_t* b_mbs_or_null, int grouped,
                     int32_t num_groups, const int64_t* row_offsets, int64_t M, int64_t N, int64_t K, mx_dtype_t c_dtype,
                     void* C, int64_t ldc, int mbs_entry, int force_shape, void* stream) {
    return mx::launch_gemm(a_codes, a_scales, a_mbs_or_null, b_codes, b_scales, b_mbs_or_null, num_groups, row_offsets,
                           grouped != 0, M, N, K, (int)c_dtype, C, ldc, mbs_entry != 0, stream, force_shape);
}

}  // extern "C"
