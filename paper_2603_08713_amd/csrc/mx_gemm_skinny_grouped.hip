// Few-row MXFP4 GEMM for grouped problems (mixture of experts) with few rows per group (tile: mx_gemm_skinny.h).
#include "mx_gemm_skinny.h"

namespace mx {
namespace {

// A workgroup owns up to 16 kMaxFM rows of one group and 16 FN columns of its C; every wavefront finds the group of its
// tile-row as the main kernel does (grouped_find).  The launch takes an upper bound of the tile-rows, the surplus exits.
// The lookup is a scan in front of a tile that takes a few us, but it spreads a group's rows over as many workgroups as
// they need.  A fixed number of workgroups for every group (four for an average of 32 rows) was up to 0.4 us faster where none has
// more than its workgroups take, and far slower where one group has all rows: 64 groups of 1024 x 1024, 1024 rows 46.3 us instead
// of 10.7, 32 of 2880 x 2880, 1024 rows 56.6 instead of 34.6 (Zipf routing: 18.9 and 19.1, 58.0 and 54.4).  Workgroups without a lookup for each group's first rows and the rest behind them: up to 18 %
// slower than this, because the largest group's rows start last.
template <int NW, int kMaxFM, int FN, int kForm, bool kSingle>
__global__ __launch_bounds__(NW * kWave) void gemm_skinny_grouped_kernel(SkinnyArgs args) {
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const GemmArgs& g = args.g;
    // column tiles innermost: a group's tiles spread over all XCDs, whatever its share of the rows
    const int tn = (int)(blockIdx.x % (unsigned)g.tiles_n), tm = (int)(blockIdx.x / (unsigned)g.tiles_n);
    const int lane = (int)(threadIdx.x & 63);
    GroupOfTileRow gr;
    const GroupLane first = group_lane(g.row_offsets, g.num_groups, 16 * kMaxFM, lane, 0);
    if (!grouped_find(g.row_offsets, g.num_groups, 16 * kMaxFM, lane, tm, first, gr)) return;
    const int64_t m0 = gr.lo + (int64_t)(tm - gr.first) * (16 * kMaxFM), m_end = min(gr.hi, m0 + 16 * kMaxFM);
    const int64_t c_n0 = (int64_t)tn * (16 * FN), b0 = (int64_t)gr.group * g.N + c_n0, b_end = (int64_t)(gr.group + 1) * g.N;
    if (kMaxFM == 1 || m_end - m0 <= 16) {
        skinny_tile<NW, 1, FN, false, kForm, kSingle>(args, smem, m0, m_end, b0, b_end, c_n0);
    } else if constexpr (kMaxFM == 2) {
        skinny_tile<NW, 2, FN, false, kForm, kSingle>(args, smem, m0, m_end, b0, b_end, c_n0);
    }
}

template <int NW, int kMaxFM, int FN, int kForm>
int launch(SkinnyArgs a, hipStream_t s) {
    GemmArgs& g = a.g;
    static_assert(NW <= 4 && kMaxFM * 16 == few_rows_tile(kForm == 3) && FN * 16 == few_rows_tile(kForm == 3), "as few_rows_blocks counts");
    const int64_t blocks = few_rows_blocks(g.M, g.N, g.num_groups, kForm == 3);
    if (blocks > kFewRowsMaxBlocks) return MX_EINVAL;
    g.tiles_n = (int)((g.N + 16 * FN - 1) / (16 * FN));
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
// are resident per compute unit and one streams while another starts or adds up; 32 columns and up to 32 rows each.  32 groups
// of 2880 x 2880 with 256 rows (Zipf) take 38 us, 3.7 TB/s of weight bytes.  Measured with a fixed number of workgroups per group:
// the same 35 us with 3 wavefronts, 36 with 4, 52 with 8; 64 groups of 1024 x 1024 with 512 rows 15.5 with 3, 15.9 with 4, and 8 of 2048 x 2048
// with 64 rows 9.1 and 7.2: the fewer K elements, the more wavefronts to share them.
int launch_gemm_skinny_grouped(const GemmArgs& g, bool use_mbs, bool bytes, hipStream_t s) {
    SkinnyArgs a = {};
    a.g = g;
    if (!use_mbs) a.g.a_mbs = a.g.b_mbs = nullptr;
    if (bytes) return launch<4, 1, 1, 3>(a, s);
    return g.K > 2048 ? launch<3, 2, 2, 2>(a, s) : launch<4, 2, 2, 2>(a, s);
}

}  // namespace mx
