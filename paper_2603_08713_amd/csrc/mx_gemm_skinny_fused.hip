// Few-row MXFP4 GEMM with the activations quantized inside the kernel (kernel: mx_gemm_skinny.h).
#include "mx_gemm_skinny.h"

namespace mx {
namespace {

template <int FM, int FN>
int launch_form(const SkinnyArgs& a, int form, hipStream_t s) {
    if (form == 0) return launch_skinny_variant<8, FM, FN, true, 0>(a, s);
    if (form == 1) return launch_skinny_variant<8, FM, FN, true, 1>(a, s);
    return MX_EINVAL;
}

}  // namespace

int launch_gemm_skinny_fused_tile(const GemmArgs& g, const void* x, int64_t ldx, int rule, bool a_mbs, int fm, int fn, int form, hipStream_t s) {
    SkinnyArgs a = {};
    a.g = g;
    a.g.a_codes = a.g.a_scales = a.g.a_mbs = nullptr;
    a.x = static_cast<const uint16_t*>(x);
    a.ldx = ldx;
    a.carry = rule_carry(rule);
    a.a_mbs = a_mbs ? 1 : 0;
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
