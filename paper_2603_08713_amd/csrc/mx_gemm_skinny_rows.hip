// The few-row MXFP4 GEMM (mx_gemm_skinny.h) on more than 64 rows: tiles of 64 rows.
#include "mx_gemm_skinny.h"

namespace mx {
namespace {

template <int FN>
int launch_form(const SkinnyArgs& a, int form, hipStream_t s) {
    if (form == 0) return launch_skinny_variant<8, 4, FN, false, 0, true>(a, s);
    if (form == 1) return launch_skinny_variant<8, 4, FN, false, 1, true>(a, s);
    if constexpr (FN <= 2) {
        if (form == 2) return launch_skinny_variant<8, 4, FN, false, 2, true>(a, s);
    }
    if constexpr (FN == 1) {
        if (form == 3) return launch_skinny_variant<8, 4, FN, false, 3, true>(a, s);
    }
    return MX_EINVAL;
}

}  // namespace

// fn fragments of 16 rows of B per workgroup; form as in mx_gemm_skinny.h
int launch_gemm_skinny_rows(const GemmArgs& g, bool use_mbs, int fn, int form, hipStream_t s) {
    SkinnyArgs a = {};
    a.g = g;
    if (!use_mbs) a.g.a_mbs = a.g.b_mbs = nullptr;
    return fn == 1 ? launch_form<1>(a, form, s) : fn == 2 ? launch_form<2>(a, form, s) : fn == 4 ? launch_form<4>(a, form, s) : MX_EINVAL;
}

}  // namespace mx
