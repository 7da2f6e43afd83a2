// GEMM on operands in the 8-bit and 6-bit element formats: argument checks, the choice of kernel, and the main kernel
// (mx_gemm_f8.h) for the 8-bit formats.  Those for the 6-bit formats are in mx_gemm_f6.hip: the template takes minutes to compile.
#include "mx_gemm_f8.h"

namespace mx {
namespace {

// force: 0 = automatic, 1 = the main kernel's general form, 2 = the main kernel in the form the problem allows, 3 = the
// few-row kernel, 16 / 17 / 18 = the main kernel on 256 x 128 / 128 x 128 / 64 x 128 tiles
int launch_gemm_elem(int a_elem, const uint8_t* a_codes, const uint8_t* a_scales, const uint8_t* a_mbs, int b_elem,
                     const uint8_t* b_codes, const uint8_t* b_scales, const uint8_t* b_mbs, int num_groups,
                     const int64_t* row_offsets, bool grouped, int64_t M, int64_t N, int64_t K, int c_dtype, void* C,
                     int64_t ldc, void* stream, int force = 0) {
    if (a_elem <= MX_ELEM_E2M1 || a_elem > MX_ELEM_E3M2 || b_elem <= MX_ELEM_E2M1 || b_elem > MX_ELEM_E3M2) return MX_EINVAL;
    if (M < 0 || N < 0 || K < 0 || (K % kBlock) != 0 || ldc < N) return MX_EINVAL;
    if (c_dtype != MX_OUT_F32 && c_dtype != MX_OUT_BF16) return MX_EINVAL;
    if (grouped && num_groups < 0) return MX_EINVAL;
    // (a tile's rows times the bytes of a row must fit the 32-bit offsets of the buffer loads)
    if (K > (int64_t)1 << 22 || M > (int64_t)1 << 30 || N > (int64_t)1 << 30 ||
        (grouped && (int64_t)num_groups * N > (int64_t)1 << 40))
        return MX_EINVAL;
    if (M == 0 || N == 0 || (grouped && num_groups == 0)) return MX_OK;
    if (!C || (grouped && !row_offsets) || (K > 0 && (!a_codes || !a_scales || !b_codes || !b_scales))) return MX_ENULL;
    const size_t esz = c_dtype == MX_OUT_F32 ? 4 : 2;
    if (!aligned(C, esz)) return MX_EALIGN;
    const bool a8 = a_elem == MX_ELEM_E4M3 || a_elem == MX_ELEM_E5M2, b8 = b_elem == MX_ELEM_E4M3 || b_elem == MX_ELEM_E5M2;
    // K in whole macro blocks, or ending with half of one (rows of E8M0 bytes then start on even
    // addresses only)
    const bool half_tail = (K % kMacro) != 0;
    if (a8 != b8 || K == 0 || (K % (kMacro / 2)) != 0 || K < kMacro || !aligned(a_codes, 16) || !aligned(b_codes, 16) ||
        !aligned(a_scales, half_tail ? 2 : 4) || !aligned(b_scales, half_tail ? 2 : 4))
        return MX_EUNSUPPORTED;
    if (int st = check_device()) return st;
    GemmArgs g = {};
    g.a_codes = a_codes; g.a_scales = a_scales; g.a_mbs = a_mbs;
    g.b_codes = b_codes; g.b_scales = b_scales; g.b_mbs = b_mbs;
    g.C = C; g.row_offsets = row_offsets;
    g.M = M; g.N = N; g.K = K; g.ldc = ldc;
    g.num_groups = grouped ? num_groups : 0;
    g.c_bf16 = c_dtype == MX_OUT_BF16;
    g.vec_store16 = aligned(C, 16) && (ldc * esz) % 16 == 0;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const bool use_mbs = a_mbs || b_mbs;
    const bool force_general = force == 1;
    // few activation rows: the weights are streamed once, nothing is staged (mx_gemm_skinny_f8.hip)
    // Taken where its rows and its rounds of 4096 columns are few, against one round of 64 x 128 tiles of the main kernel.  With the
    // quantizer in front and words, few-row kernel and tiles, us, K = 512, 1536, 2560, 5120: E4M3, 8 rows, N = 8192 8.0, 10.5, 12.3,
    // 16.5 and 8.8, 13.1, 16.8, 25.6, N = 8800 9.7, 13.7, 16.7, 23.4 and 8.8, 13.3, 16.7, 25.8; 26 rows, N = 4945 10.2, 13.1, 16.9, 23.7 and 9.2,
    // 12.9, 16.7, 25.7, N = 8800 12.0, 17.3, 21.5, 31.6 and 9.1, 13.2, 17.0, 25.9; 64 rows, N = 4096 10.3, 13.0, 16.1, 24.0 and 9.2, 13.1, 16.7, 26.1,
    // N = 4160 15.2, 20.2, 25.8, 38.7 and 9.3, 13.1, 16.9, 26.2.  E3M2: 8 rows, N = 10548 8.6, 12.2, 15.2, 22.1 and 9.0, 13.3, 16.9, 25.6; 26
    // rows, N = 4945 8.9, 11.6, 14.8, 22.5 and 9.4, 12.9, 16.6, 25.6; 64 rows, N = 4096 10.2, 12.8, 15.6, 23.7 and 9.5, 13.1, 16.7, 26.0.  More than
    // 32 rows in one round are 64 to this kernel's tile and fewer to its loads.  Tiles over few rows, words, GEMM alone, 14000 problems of N = 128 to 4096, rows 33
    // to 40, to 48, to 56, to 64: K = 512 0.98, 0.97, 0.94, 0.92 in E4M3 and 1.01, 1.00, 0.98, 0.96 in E3M2; 1024 1.10, 1.07, 1.03, 1.00 (0.97 in bf16) and
    // 1.13, 1.11, 1.07, 1.04; 1536 1.19, 1.16, 1.10, 1.08 and 1.22, 1.19, 1.14, 1.10; without words K = 2048 0.99, 0.96, 0.94, 0.88 at 33,
    // 40, 48 and 64, 3072 1.05, 1.0, 0.98, 0.91.
    // Without words the tiles gain more, and from K = 5120 on, with 8-bit weights that no cache holds, the few rows again: 8 rows, N = 8800 19.1
    // and 23.1 in E4M3 (the other formats and row counts within 14 % either way).  In six bits short K leaves tiles little to gain: tiles over few rows, three
    // and four rounds, to 8 and to 16 rows: K = 512 1.11, 1.06, 1024 1.05, 0.99, 1536 1.00, 0.95 (8 bits 0.88, 0.86; 0.86, 0.82; 0.86, 0.81).
    const int64_t few_work = (M <= 16 ? 1 : M <= 32 ? 2 : 4) * ((N + 4095) / 4096);
    const bool short_six = !use_mbs && !a8 && M <= 16 && K <= (M <= 8 ? 1024 : 512);
    const int64_t few_from = !use_mbs ? (short_six ? 0 : M > 32 && M <= 40 ? 3072 : 5120) : M > 56 && a8 ? 1536 : M > 32 ? 1024 : a8 ? 2560 : 0;
    // E2M3's products fit the matrix unit's sum without a cut, so the order of the sum over K shows: error against 64 bits, tiles over
    // few rows, with words, E2M3 on either side: K = 512 1.0, 1024 1.06, 2048 1.19, 4096 1.36, 8192 1.69.  Past K = 512 it stays with this
    // kernel's split sum.  Without words both are exact on such data, and the other formats' cut hides the order (1.0000 at every K).
    const bool exact_products = a_elem == MX_ELEM_E2M3 || b_elem == MX_ELEM_E2M3;
    const bool few_pays = few_work <= 2 || (few_work <= 4 && K >= few_from) || (exact_products && use_mbs && K > 512);
    const bool skinny_ok = !grouped && M <= 64 && (K % 512) == 0 && K <= 8192 && aligned(a_scales, 16) && aligned(b_scales, 16) &&
                           (!a_mbs || aligned(a_mbs, 4)) && (!b_mbs || aligned(b_mbs, 4));
    if (force == 3 && !skinny_ok) return MX_EINVAL;
    if (skinny_ok && ((force == 0 && few_pays) || force == 3)) return launch_gemm_skinny_elem(g, a_elem, b_elem, s);
    if (force > 18 || (force > 16 && K < 512)) return MX_EINVAL;
    const int tile = force >= 16 ? force - 16 : force_general ? 0 : f8_tile(g, use_mbs);
    if (!a8) {
        if (tile == 2) return launch_gemm_six_tiny(g, a_elem == MX_ELEM_E3M2, b_elem == MX_ELEM_E3M2, use_mbs, s);
        if (tile == 1) return launch_gemm_six_small(g, a_elem == MX_ELEM_E3M2, b_elem == MX_ELEM_E3M2, use_mbs, s);
        return launch_gemm_six(g, a_elem == MX_ELEM_E3M2, b_elem == MX_ELEM_E3M2, use_mbs, force_general, s);
    }
    const bool a5 = a_elem == MX_ELEM_E5M2, b5 = b_elem == MX_ELEM_E5M2;
    if (tile == 2) return launch_gemm_eight_tiny(g, a5, b5, use_mbs, s);
    if (tile == 1) return launch_gemm_eight_small(g, a5, b5, use_mbs, s);
    if (!a5 && !b5) return launch_f8<0, 0>(g, use_mbs, force_general, s);
    if (!a5 && b5) return launch_f8<0, 1>(g, use_mbs, force_general, s);
    if (a5 && !b5) return launch_f8<1, 0>(g, use_mbs, force_general, s);
    return launch_f8<1, 1>(g, use_mbs, force_general, s);
}

}  // namespace
}  // namespace mx

extern "C" int mx_gemm_mbs_elem(mx_elem_t a_elem, const uint8_t* a_codes, const uint8_t* a_scales,
                                const uint8_t* a_mbs_or_null, mx_elem_t b_elem, const uint8_t* b_codes,
                                const uint8_t* b_scales, const uint8_t* b_mbs_or_null, int64_t M, int64_t N, int64_t K,
                                mx_dtype_t c_dtype, void* C, int64_t ldc, void* stream) {
    return mx::launch_gemm_elem((int)a_elem, a_codes, a_scales, a_mbs_or_null, (int)b_elem, b_codes, b_scales,
                                b_mbs_or_null, 0, nullptr, false, M, N, K, (int)c_dtype, C, ldc, stream);
}

extern "C" int mx_gemm_mbs_elem_grouped(mx_elem_t a_elem, const uint8_t* a_codes, const uint8_t* a_scales,
                                        const uint8_t* a_mbs_or_null, mx_elem_t b_elem, const uint8_t* b_codes,
                                        const uint8_t* b_scales, const uint8_t* b_mbs_or_null, int32_t num_groups,
                                        const int64_t* row_offsets, int64_t M_total, int64_t N, int64_t K,
                                        mx_dtype_t c_dtype, void* C, int64_t ldc, void* stream) {
    return mx::launch_gemm_elem((int)a_elem, a_codes, a_scales, a_mbs_or_null, (int)b_elem, b_codes, b_scales,
                                b_mbs_or_null, num_groups, row_offsets, true, M_total, N, K, (int)c_dtype, C, ldc, stream);
}

extern "C" int mx_internal_gemm_elem(mx_elem_t a_elem, const uint8_t* a_codes, const uint8_t* a_scales,
                                     const uint8_t* a_mbs_or_null, mx_elem_t b_elem, const uint8_t* b_codes,
                                     const uint8_t* b_scales, const uint8_t* b_mbs_or_null, int64_t M, int64_t N,
                                     int64_t K, mx_dtype_t c_dtype, void* C, int64_t ldc, int force, void* stream) {
    return mx::launch_gemm_elem((int)a_elem, a_codes, a_scales, a_mbs_or_null, (int)b_elem, b_codes, b_scales,
                                b_mbs_or_null, 0, nullptr, false, M, N, K, (int)c_dtype, C, ldc, stream, force);
}
