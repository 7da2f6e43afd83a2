// GEMM on operands in the 8-bit and 6-bit element formats: argument checks, the choice of kernel, and the main kernel
// (mx_gemm_f8.h) for the 8-bit formats.  Those for the 6-bit formats are in mx_gemm_f6.hip: the template takes minutes to compile.
#include "mx_gemm_f8.h"

namespace mx {
namespace {

// force: 0 = automatic, 1 = the main kernel's general form, 2 = the main kernel in the form the problem allows, 3 = the
// few-row kernel
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
    const bool skinny_ok = !grouped && M <= 64 && (K % 512) == 0 && K <= 8192 && aligned(a_scales, 16) && aligned(b_scales, 16) &&
                           (!a_mbs || aligned(a_mbs, 4)) && (!b_mbs || aligned(b_mbs, 4));
    if (force == 3 && !skinny_ok) return MX_EINVAL;
    if (skinny_ok && (force == 0 || force == 3)) return launch_gemm_skinny_elem(g, a_elem, b_elem, s);
    const bool small_tile = !force_general && f8_small_tile(g, use_mbs);
    if (!a8) {
        if (small_tile) return launch_gemm_six_small(g, a_elem == MX_ELEM_E3M2, b_elem == MX_ELEM_E3M2, use_mbs, s);
        return launch_gemm_six(g, a_elem == MX_ELEM_E3M2, b_elem == MX_ELEM_E3M2, use_mbs, force_general, s);
    }
    const bool a5 = a_elem == MX_ELEM_E5M2, b5 = b_elem == MX_ELEM_E5M2;
    if (small_tile) return launch_gemm_eight_small(g, a5, b5, use_mbs, s);
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
