// The main GEMM kernel template in its general form: any K, rows of E8M0 bytes and MBS words at any address,
// and grouped problems (mixture of experts).  A row's E8M0 bytes and MBS words travel in the fast form's pieces, but
// through registers;
// the fast form, whose loads need no registers, keeps every problem it can take.  This file holds the kernels with MBS (compiled with the
// VGPR form of the matrix instructions, as in mx_gemm_mbs.hip); those without are in mx_gemm_wide.hip.
#include "mx_gemm_ring.h"

namespace mx {

// K > 0; the caller has checked this.  A null MBS array reads as
// words of zero (sigma = 1, which multiplies exactly), so one instantiation serves one-sided MBS as well.
// tile: 0 = 256 x 128, 1 = 128 x 128, 2 = 64 x 128.
int launch_gemm_mbs_general(const GemmArgs& g, int tile, hipStream_t s) {
    if (tile == 0) return launch_ring<RingShape<4, 2, 2, 2, 3, 1>>(g, s);
    if (tile == 2) return launch_ring<RingShape<1, 4, 2, 1, 3, 1>>(g, s);
    return launch_ring<RingShape<2, 4, 2, 1, 3, 1>>(g, s);
}

}  // namespace mx
