// Few-row MXFP4 GEMM for grouped problems (mixture of experts) with few rows per group (tile: mx_gemm_skinny.h).
#include "mx_gemm_skinny.h"

namespace mx {
namespace {

// A workgroup owns 16 FN columns of one group's C and walks over the group's rows, at most 16 kMaxFM at a time; g.tiles_m
// workgroups share the rows of a group and a column tile.  (No workgroup looks its tile-row up in a prefix sum over the
// groups, as the main kernel does: that is a round trip to memory and a scan in front of a tile that takes a few us.)
template <int NW, int kMaxFM, int FN, int kForm, bool kSingle>
__global__ __launch_bounds__(NW * kWave) void gemm_skinny_grouped_kernel(SkinnyArgs args) {
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const GemmArgs& g = args.g;
    // column tiles innermost: a group's tiles spread over all XCDs, whatever its share of the rows
    const int tn = (int)(blockIdx.x % (unsigned)g.tiles_n), rest = (int)(blockIdx.x / (unsigned)g.tiles_n);
    const int part = rest % g.tiles_m, e = rest / g.tiles_m;
    const int64_t lo = g.row_offsets[e], hi = g.row_offsets[e + 1];
    const int64_t b0 = (int64_t)e * g.N + (int64_t)tn * (16 * FN), b_end = (int64_t)(e + 1) * g.N;
    for (int64_t m0 = lo + part * (16 * kMaxFM); m0 < hi;) {
        const int64_t m_end = min(hi, m0 + 16 * kMaxFM);
        if (kMaxFM == 1 || m_end - m0 <= 16) {
            skinny_tile<NW, 1, FN, false, kForm, kSingle>(args, smem, m0, m_end, b0, b_end, (int64_t)tn * (16 * FN));
        } else if constexpr (kMaxFM == 2) {
            skinny_tile<NW, 2, FN, false, kForm, kSingle>(args, smem, m0, m_end, b0, b_end, (int64_t)tn * (16 * FN));
        } else if constexpr (kMaxFM == 4) {
            skinny_tile<NW, 4, FN, false, kForm, kSingle>(args, smem, m0, m_end, b0, b_end, (int64_t)tn * (16 * FN));
        }
        m0 += g.tiles_m * (16 * kMaxFM);
        if (m0 < hi) __syncthreads();  // the partial results have been read before the next weights land on them
    }
}

// Workgroups that share a group's rows: enough for groups with a few times the average (measured, average 32 rows, 1, 2, 4
// parts: 8 groups of 2048 x 2048 14.0, 11.2, 9.0 us, 64 of 1024 x 1024 39.9, 23.5, 24.9), but workgroups without rows
// cost their launch (average 1 row, 32 groups of 2880 x 2880: 21.3, 21.4, 22.6).
int64_t parts_of(int64_t rows, int64_t groups) { return rows > 16 * groups ? 4 : rows > 8 * groups ? 2 : 1; }

template <int NW, int kMaxFM, int FN, int kForm>
int launch(SkinnyArgs a, hipStream_t s) {
    GemmArgs& g = a.g;
    const int64_t tiles_n = (g.N + 16 * FN - 1) / (16 * FN), parts = parts_of(g.M, g.num_groups);
    const int64_t blocks = tiles_n * g.num_groups * parts;
    if (blocks > (int64_t)1 << 30) return MX_EINVAL;
    g.tiles_m = (int)parts;
    g.tiles_n = (int)tiles_n;
    using S = SkinnyShape<NW, kMaxFM, FN, false, kForm>;
    auto launch = [&](auto single_) {
        auto* fn = gemm_skinny_grouped_kernel<NW, kMaxFM, FN, kForm, decltype(single_)::value>;
        static LdsOptIn opt_in;  // one per kernel instantiation
        if (int st = opt_in.ensure(reinterpret_cast<const void*>(fn), S::kLdsBytes)) return st;
        hipLaunchKernelGGL(fn, dim3((unsigned)blocks), dim3(S::NT), S::kLdsBytes, s, a);
        return launch_status();
    };
    if (g.K <= kSingleChunkK(NW)) return launch(std::integral_constant<bool, true>{});
    return launch(std::integral_constant<bool, false>{});
}

}  // namespace

// K > 0; scale arrays 2-byte aligned and K % 64 == 0, or `bytes`.  Few wavefronts per workgroup, so that several workgroups
// are resident per compute unit and one streams while another starts or adds up (8 wavefronts: 52 us at the case below);
// 32 columns and up to 32 rows each.  Measured, 32 groups of 2880 x 2880 with 256 rows (Zipf): 35 us = 4.0 TB/s of weight
// bytes with 3 wavefronts, 36 with 4; 64 groups of 1024 x 1024 with 512 rows 15.5 with 3, 15.9 with 4, and 8 of 2048 x 2048
// with 64 rows 9.1 and 7.2: the fewer K elements, the more wavefronts to share them.
int launch_gemm_skinny_grouped(const GemmArgs& g, bool use_mbs, bool bytes, hipStream_t s) {
    SkinnyArgs a = {};
    a.g = g;
    if (!use_mbs) a.g.a_mbs = a.g.b_mbs = nullptr;
    if (bytes) return launch<4, 1, 1, 3>(a, s);
    return g.K > 2048 ? launch<3, 2, 2, 2>(a, s) : launch<4, 2, 2, 2>(a, s);
}

}  // namespace mx
