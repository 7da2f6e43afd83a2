// The main kernel of mx_gemm_f8.h for the 6-bit formats (E2M3, E3M2).
#include "mx_gemm_f8.h"

namespace mx {

// a32, b32: the operand is E3M2, else E2M3
int launch_gemm_six(const GemmArgs& g, bool a32, bool b32, bool use_mbs, bool force_general, hipStream_t s) {
    if (!a32 && !b32) return launch_f8<2, 2>(g, use_mbs, force_general, s);
    if (!a32 && b32) return launch_f8<2, 3>(g, use_mbs, force_general, s);
    if (a32 && !b32) return launch_f8<3, 2>(g, use_mbs, force_general, s);
    return launch_f8<3, 3>(g, use_mbs, force_general, s);
}

}  // namespace mx
