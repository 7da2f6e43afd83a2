// The main kernel of mx_gemm_f8.h on 128 x 128 tiles, 8-bit formats.
#include "mx_gemm_f8.h"

namespace mx {

// a5, b5: the operand is E5M2, else E4M3
int launch_gemm_eight_small(const GemmArgs& g, bool a5, bool b5, bool use_mbs, hipStream_t s) {
    if (!a5 && !b5) return launch_f8_small<0, 0, 1>(g, use_mbs, s);
    if (!a5 && b5) return launch_f8_small<0, 1, 1>(g, use_mbs, s);
    if (a5 && !b5) return launch_f8_small<1, 0, 1>(g, use_mbs, s);
    return launch_f8_small<1, 1, 1>(g, use_mbs, s);
}

}  // namespace mx
