// The main kernel of mx_gemm_f8.h on 64 x 128 tiles, 6-bit formats.
#include "mx_gemm_f8.h"

namespace mx {

// a32, b32: the operand is E3M2, else E2M3
int launch_gemm_six_tiny(const GemmArgs& g, bool a32, bool b32, bool use_mbs, hipStream_t s) {
    if (!a32 && !b32) return launch_f8_small<2, 2, 2>(g, use_mbs, s);
    if (!a32 && b32) return launch_f8_small<2, 3, 2>(g, use_mbs, s);
    if (a32 && !b32) return launch_f8_small<3, 2, 2>(g, use_mbs, s);
    return launch_f8_small<3, 3, 2>(g, use_mbs, s);
}

}  // namespace mx
