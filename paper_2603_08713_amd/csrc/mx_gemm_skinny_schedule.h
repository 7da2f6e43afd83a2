// Loads of the few-row GEMM kernel (mx_gemm_skinny.h): how many a wavefront issues for a chunk of four macro blocks and how
// many of the youngest may still be in flight when it reads the chunk's weights.  Plain constexpr C++ with no device
// code, so that a host program can replay every form and check it (tests/schedule_check.cpp).
//
// A wavefront's loads complete in the order it issued them, and it shares nothing with the others before its end: no
// barrier, the wait alone makes its weights readable.  The weights (direct to LDS: E8M0 bytes and MBS words, then codes
// fragment by fragment) are requested behind the activations of the chunk (into registers, whose users the compiler makes wait).
// Quantized activations: those of the next chunk are requested at the end of a chunk, so the weights are the youngest loads
// and everything has to land.  Fused form: the bf16 activations travel in units, two macro blocks of one fragment of
// A; while the first fragment's two units are quantized the second fragment's are requested, behind the weights.
// How many loads those are depends on the macro blocks that the chunk has: a unit does not fetch what lies past the
// wavefront's share of K.  A wait that counted loads which were not issued would let as many loads of the weights fly.
#pragma once

#include "mx_constants.h"

namespace mx {

constexpr int kSkinnyMacs = 4;  // macro blocks per chunk

template <int FM, int FN, int kForm>
struct SkinnySchedule {
    // E8M0 bytes and MBS words of a chunk, codes of one fragment of B
    static constexpr int kScaleLoads = kForm == 0 ? 1 : kForm == 1 ? FN : kForm == 2 ? 2 * FN : 4 * FN;
    static constexpr int kWordLoads = kForm == 0 ? 1 : kForm == 1 ? (FN + 1) / 2 : FN;
    static constexpr int kCodeLoads = 4;
    // fused: loads of one macro block of a fragment of A, one per block
    static constexpr int kRawLoads = 4;

    // Macro blocks that unit `half` of a chunk holds, `left` of them left to the wavefront from the chunk's first on
    // (form 0: the shares are whole chunks).
    static constexpr int unit_macs(int left, int half) {
        const int n = left - 2 * half;
        return kForm == 0 || n > 2 ? 2 : n < 0 ? 0 : n;
    }
    // Fused: loads younger than the weights when the first fragment of A has been quantized, i.e. what its wait may leave in flight.
    // (One fragment: the youngest are the next chunk's, if there is one, and everything has to land.)
    static constexpr int weights_wait(int left) {
        return FM == 1 ? 0 : kRawLoads * (unit_macs(left, 0) + unit_macs(left, 1));
    }
};

}  // namespace mx
