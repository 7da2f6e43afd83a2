// Few-row MXFP4 GEMM on quantized activations (kernel: mx_gemm_skinny.h).
#include "mx_gemm_skinny.h"

namespace mx {
namespace {

template <int FM, int FN>
int launch_form(const SkinnyArgs& a, int form, hipStream_t s) {
    if (form == 0) return launch_skinny_variant<8, FM, FN, false, 0>(a, s);
    if (form == 1) return launch_skinny_variant<8, FM, FN, false, 1>(a, s);
    if constexpr (FN <= 2) {
        if (form == 2) return launch_skinny_variant<8, FM, FN, false, 2>(a, s);
    }
    if constexpr (FN == 1) {
        if (form == 3) return launch_skinny_variant<8, FM, FN, false, 3>(a, s);
    }
    return MX_EINVAL;
}

}  // namespace

// M <= 16 fm rows: fm, fn fragments of 16 rows of A and of B per workgroup; form as in mx_gemm_skinny.h
int launch_gemm_skinny_tile(const GemmArgs& g, bool use_mbs, int fm, int fn, int form, hipStream_t s) {
    SkinnyArgs a = {};
    a.g = g;
    if (!use_mbs) a.g.a_mbs = a.g.b_mbs = nullptr;
    switch (fm * 8 + fn) {
        case 8 + 1: return launch_form<1, 1>(a, form, s);
        case 8 + 2: return launch_form<1, 2>(a, form, s);
        case 8 + 4: return launch_form<1, 4>(a, form, s);
        case 16 + 1: return launch_form<2, 1>(a, form, s);
        case 16 + 2: return launch_form<2, 2>(a, form, s);
        case 16 + 4: return launch_form<2, 4>(a, form, s);
        case 32 + 1: return launch_form<4, 1>(a, form, s);
        case 32 + 2: return launch_form<4, 2>(a, form, s);
        case 32 + 4: return launch_form<4, 4>(a, form, s);
        default: return MX_EINVAL;
    }
}

}  // namespace mx
