// MXFP4 GEMM  C = A * B^T  for a handful of activation rows: bound by streaming the weights once (private;
// instantiated by mx_gemm_skinny.hip, mx_gemm_skinny_fused.hip and mx_gemm_skinny_grouped.hip).
//
// A workgroup owns 16 FN columns of C (16 FN rows of B) and 16 FM rows of A; its NW wavefronts split K between
// them, each taking consecutive macro blocks in chunks of four, and add their partial results through LDS at the
// end.  Until then the wavefronts share nothing: no barrier, and each streams its own weights through its own piece
// of LDS with direct-to-LDS loads.
//
// Why through LDS, although no byte of B is used twice: the texture-address unit takes one clock per group of four
// consecutive lanes and memory line.  Loaded straight into the operand registers of v_mfma_scale_f32_16x16x128
// (lane = 16 q + r holds row r, k-block q), four consecutive lanes are four rows, so 1 KiB of codes costs 64 clocks;
// as a direct-to-LDS load of 4 rows x 256 contiguous bytes it costs 16, and the data in flight occupies no
// registers.  The LDS image of a fragment's chunk is [row][256 B] with the 16-byte piece c of row r at position
// c ^ r, so that the 16 rows of a fragment read cover all banks.
//
// v_mfma_scale_f32_16x16x128_f8f6f4 is one macro block deep.  The activations feed srcA and the weights srcB, so
// D[4 q + i][r] leaves a lane with C[m = 4 q + i][n = r]: sigma_B of the lane's own weight row is a per-lane scalar,
// and the four sigma_A values come from a small LDS table per wavefront.
//
// How the E8M0 bytes and MBS words of a chunk travel depends on the alignment of a row's bytes (kForm):
//   0  every wavefront's share of K is whole chunks (eight wavefronts: K of 3584, 4096, 7680 and 8192), scale rows 16-byte
//      and word rows 4-byte aligned: a row's 16 E8M0 bytes as one piece, its four words as one dword (one load of each
//      kind per chunk)
//   1  K % 512 == 0, the same alignment of the arrays: a macro block's four E8M0 bytes as one dword, words as the two
//      aligned dwords that hold the chunk's four
//   2  K % 64 == 0, scale arrays on even addresses: E8M0 bytes in pairs, words one by one, each piece in an LDS dword of
//      its own
//   3  any K % 32 == 0, any address: single bytes
//
// Fused form (activations quantized inside this kernel, Sec. 4.3 / 5.3): each wavefront quantizes exactly the K range
// it multiplies, while its weights are on their way.  Four consecutive lanes fetch one block of one row (the
// texture-address unit again), so block and macro-block absmax are DPP maxima and every lane of the four works out the
// figures of one of the macro block's four blocks; codes and E8M0 bytes go through a small piece of LDS into the
// matrix instruction's layout.  MBS word, scale byte and codes follow the quantizer's arithmetic to the bit.
//
// Grouped form (mixture of experts with few rows per expert): a workgroup has up to 32 rows of one group.
#pragma once

#include "mx_gemm_shared.h"
#include "mx_gemm_skinny_schedule.h"
#include "mx_quantize_math.h"

namespace mx {

struct SkinnyArgs {
    GemmArgs g;
    // fused form only: bf16 activations [M, ldx], the scale rule's carry and whether MBS-Static words are formed
    const uint16_t* x;
    int64_t ldx;
    uint32_t carry;
    int a_mbs;
};

namespace {

// what a wavefront keeps in LDS
template <int NW, int FM, int FN, bool kFused, int kForm>
struct SkinnyShape {
    static constexpr int NT = NW * kWave;
    static constexpr int kRows = 16 * FN;
    static constexpr int kCodes = FN * 4096;  // [fragment][16 rows][256 B]; at the end its partial results
    static constexpr int kPiece = kForm == 2 ? 2 : 1;  // bytes of an E8M0 piece in the forms 2 and 3
    // E8M0 bytes and MBS words of a chunk: loads, bytes of LDS
    using Sched = SkinnySchedule<FM, FN, kForm>;
    static constexpr int kScaleLoads = Sched::kScaleLoads;
    static constexpr int kScaleBytes = kForm == 0 ? 1024 : kScaleLoads * 256;
    static constexpr int kWordLoads = Sched::kWordLoads;
    static constexpr int kSigma = FM * 256;                   // sigma_A [macro block of the chunk][FM * 16]
    // A's way from the layout it is fetched (or quantized) in into the operand's: codes of a macro block [block][row][16 B]
    // (the blocks 320 bytes apart: bank conflicts) and its E8M0 bytes, [block][row] or (not fused) [macro block][row][4]
    static constexpr int kExchangeScales = 4 * 320, kExchange = kExchangeScales + 256;
    static constexpr int kScaleBase = kCodes, kWordBase = kScaleBase + kScaleBytes, kSigmaBase = kWordBase + kWordLoads * 256;
    static constexpr int kExchangeBase = kSigmaBase + kSigma;
    static constexpr int kBytes = kExchangeBase + kExchange;
    static constexpr int kLdsBytes = NW * kBytes;
    static_assert(FM * FN * 1024 <= kCodes, "the partial results fit the code region");
    static_assert(kLdsBytes <= 160 * 1024, "LDS capacity of a gfx950 compute unit");
};

// Quantizes one macro block of 16 rows: raw[b] is the 16-byte piece l % 4 of block b of row l / 4.
struct MacroQuant {
    uint32_t codes[4];  // the lane's eight codes of block b
    uint32_t E;         // E8M0 byte of block l % 4
    uint32_t m8;        // MBS word of the row
};
__device__ __forceinline__ uint32_t quad_max(uint32_t v) {
    v = max(v, dpp_quad_xor1(v));
    return max(v, dpp_quad_xor2(v));
}
__device__ __forceinline__ uint32_t pick4(uint32_t v0, uint32_t v1, uint32_t v2, uint32_t v3, int p) {
    const uint32_t lo = (p & 1) ? v1 : v0, hi = (p & 1) ? v3 : v2;
    return (p & 2) ? hi : lo;
}
// The products with F * 2^(127-E) are exact in fp32 for every bf16 value (17 significant bits, denormals kept), so only
// the block's own figures need care outside the comfortable range: there the absmax is moved by 2^64 before its
// exponent and mantissa are read, and the multiplier is formed by ldexp (it may be denormal).
__device__ __forceinline__ MacroQuant quantize_macro(const v4i (&raw)[4], uint32_t carry, int use_mbs, int l) {
    uint32_t amax[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        uint32_t m = (uint32_t)raw[b][0] & 0x7FFF7FFFu;
#pragma unroll
        for (int i = 1; i < 4; ++i) m = pk_max_u16(m, (uint32_t)raw[b][i] & 0x7FFF7FFFu);
        amax[b] = quad_max(max(m & 0xFFFFu, m >> 16));
    }
    // every lane of four works out the figures of its own block
    uint32_t own = pick4(amax[0], amax[1], amax[2], amax[3], l);
    // exponent field outside [24, 249] (or Inf/NaN): the careful figures, wave-uniformly
    const bool odd = (own >= (250u << 7)) || (own != 0 && own < (24u << 7));
    const bool careful = __builtin_amdgcn_ballot_w64(odd) != 0;
    MacroQuant out;
    float mult;
    if (careful) {
        const bool finite = own < 0x7F80u;
#pragma unroll
        for (int b = 0; b < 4; ++b) {  // non-finite elements do not count for the macro block's absmax
            uint32_t m = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t lo = (uint32_t)raw[b][i] & 0x7FFFu, hi = ((uint32_t)raw[b][i] >> 16) & 0x7FFFu;
                m = max(m, max(lo < 0x7F80u ? lo : 0u, hi < 0x7F80u ? hi : 0u));
            }
            amax[b] = quad_max(m);
        }
        own = pick4(amax[0], amax[1], amax[2], amax[3], l);
        uint32_t m8 = 0;
        if (use_mbs) {
            const uint32_t mmax = max(max(amax[0], amax[1]), max(amax[2], amax[3]));
            const float f = __builtin_ldexpf(__uint_as_float(mmax << 16), 64);  // (a normal number if mmax was subnormal)
            const uint32_t word = mbs_word_of_mantissa_fast((mmax < 0x80u ? __float_as_uint(f) >> 16 : mmax) & 0x7Fu);
            m8 = mmax ? word : 0u;
        }
        const float F = __uint_as_float(0x3F800000u | (m8 << 15));
        const int move = own < (64u << 7) ? 64 : -64;
        const float scaled_max = __builtin_ldexpf(__uint_as_float(own << 16), move) * F;
        const int E = (int)((__float_as_uint(scaled_max) + carry) >> 23) - 2 - move;
        out.E = !finite ? 255u : own == 0 ? 127u : (uint32_t)min(max(E, 0), 254);
        out.m8 = m8;
        mult = __builtin_ldexpf(F, 127 - (int)out.E);
    } else {
        uint32_t m8 = 0;
        if (use_mbs) {
            const uint32_t mmax = max(max(amax[0], amax[1]), max(amax[2], amax[3]));
            const uint32_t word = mbs_word_of_mantissa_fast(mmax & 0x7Fu);
            m8 = mmax ? word : 0u;
        }
        // absmax * F is exact in fp32; exponent field + carry gives the stored byte; multiplier F * 2^(127-E)
        const float scaled_max = __uint_as_float(own << 16) * __uint_as_float(0x3F800000u | (m8 << 15));
        const uint32_t E = ((__float_as_uint(scaled_max) + carry) >> 23) - 2u;
        out.E = own ? E : 127u;
        out.m8 = m8;
        mult = __uint_as_float(((254u - out.E) << 23) | (m8 << 15));
    }
    const uint32_t mult_bits = __float_as_uint(mult);
    // the multiplier of block b from lane b of the four
    const float mults[4] = {__uint_as_float(__builtin_amdgcn_update_dpp(0u, mult_bits, 0x00, 0xF, 0xF, true)),
                            __uint_as_float(__builtin_amdgcn_update_dpp(0u, mult_bits, 0x55, 0xF, 0xF, true)),
                            __uint_as_float(__builtin_amdgcn_update_dpp(0u, mult_bits, 0xAA, 0xF, 0xF, true)),
                            __uint_as_float(__builtin_amdgcn_update_dpp(0u, mult_bits, 0xFF, 0xF, 0xF, true))};
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        uint32_t c = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t w = (uint32_t)raw[b][j];
            const float t0 = __uint_as_float(w << 16) * mults[b], t1 = __uint_as_float(w & 0xFFFF0000u) * mults[b];
            if (j == 0) c = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(c, t0, t1, 1.0f, 0);
            if (j == 1) c = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(c, t0, t1, 1.0f, 1);
            if (j == 2) c = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(c, t0, t1, 1.0f, 2);
            if (j == 3) c = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(c, t0, t1, 1.0f, 3);
        }
        out.codes[b] = c;
    }
    if (careful) {  // a block holding Inf/NaN stores zero codes
        const uint32_t e0 = __builtin_amdgcn_update_dpp(0u, out.E, 0x00, 0xF, 0xF, true), e1 = __builtin_amdgcn_update_dpp(0u, out.E, 0x55, 0xF, 0xF, true);
        const uint32_t e2 = __builtin_amdgcn_update_dpp(0u, out.E, 0xAA, 0xF, 0xF, true), e3 = __builtin_amdgcn_update_dpp(0u, out.E, 0xFF, 0xF, 0xF, true);
        out.codes[0] = e0 == 255u ? 0u : out.codes[0];
        out.codes[1] = e1 == 255u ? 0u : out.codes[1];
        out.codes[2] = e2 == 255u ? 0u : out.codes[2];
        out.codes[3] = e3 == 255u ? 0u : out.codes[3];
    }
    return out;
}

// LDS stores as bare instructions: in front of a store to LDS the compiler waits for every outstanding direct-to-LDS
// load, which may write the same place for all it knows.  (A wavefront's LDS operations run in order, so its own
// later reads see the stored values.)
__device__ __forceinline__ uint32_t lds_address(const void* p) {
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)p;
}
__device__ __forceinline__ void lds_store32(void* p, uint32_t v) {
    asm volatile("ds_write_b32 %0, %1" ::"v"(lds_address(p)), "v"(v) : "memory");
}
__device__ __forceinline__ void lds_store128(void* p, v4i v) {
    asm volatile("ds_write_b128 %0, %1" ::"v"(lds_address(p)), "v"(v) : "memory");
}
__device__ __forceinline__ void lds_store8(void* p, uint32_t v) {
    asm volatile("ds_write_b8 %0, %1" ::"v"(lds_address(p)), "v"(v) : "memory");
}
// every load of this wavefront has landed
__device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
// at most n loads of this wavefront are outstanding
template <int n>
__device__ __forceinline__ void wait_loads_but() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(n) : "memory"); }
// every LDS read of this wavefront has returned
__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// K up to which no wavefront has more than one chunk (kSingle: the kernel without the loop over chunks, in which the
// compiler also counts outstanding loads exactly instead of for the worst of two iterations)
constexpr int kSingleChunkK(int waves) { return waves * kSkinnyMacs * kMacro; }

// Rows m0 .. m_end - 1 (at most 16 FM of them) of A against weight rows n0 .. n_end - 1 (at most 16 FN) of B; C starts
// at row m0 and column c_n0.  smem: the workgroup's LDS.
// kWords: false = no MBS words on either side: nothing is fetched, kept or multiplied for them.  (A choice at compile time: a
// branch between a matrix instruction and the use of its result got no wait for that result from the compiler.)
template <int NW, int FM, int FN, bool kFused, int kForm, bool kSingle, bool kWords = true>
__device__ __forceinline__ void skinny_tile(const SkinnyArgs& args, uint8_t* smem, int64_t m0, int64_t m_end, int64_t n0,
                                            int64_t n_end, int64_t c_n0) {
    using S = SkinnyShape<NW, FM, FN, kFused, kForm>;
    using Sched = typename S::Sched;
    const GemmArgs& g = args.g;
    const int K = (int)g.K, nmac = (K + kMacro - 1) / kMacro;
    const int row_bytes = K >> 1, scale_bytes = K >> 5;
    const int tid = threadIdx.x, l = tid & 63, r = l & 15, q = l >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint8_t* mine = smem + w * S::kBytes;
    float* sig_a = reinterpret_cast<float*>(mine + S::kSigmaBase);
    uint8_t* exchange = mine + S::kExchangeBase;

    const Operand opa = make_operand(kFused ? g.b_codes : g.a_codes, g.a_scales, g.a_mbs, kFused ? 0 : m0, kFused ? 0 : m_end,
                                     FM * 16, g.K);  // (fused: empty, not used)
    // fused: the bf16 rows as one buffer ending with the last row's K elements; rows past M read zero
    const __amdgpu_buffer_rsrc_t opx = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t*>(args.x), 0, kFused ? (int)(((g.M - 1) * args.ldx + g.K) * 2) : 0, 0x00020000);
    const Operand opb = make_operand(g.b_codes, g.b_scales, g.b_mbs, n0, n_end, FN * 16, g.K);

    // this wavefront's macro blocks
    const int per_wave = (nmac + NW - 1) / NW;
    const int first = w * per_wave, last = min(first + per_wave, nmac);
    // (code bytes of a row past this wavefront's share, or past K, are fetched out of range: they read zero)
    const int code_end = min(last * 64, row_bytes);

    // ---- loads of the weights of a chunk that starts with macro block `mac` ----
    const int lane_row_off = (l >> 4) * row_bytes;
    const int piece0 = (l & 15) ^ (l >> 4);  // load i of a fragment: row 4 i + l / 16, piece (l % 16) ^ row
    // (the row strides are made opaque so that the addresses are formed where they are used, one addition each, and
    // not kept in registers over the loop)
    auto opaque = [](int v) {
        asm volatile("" : "+s"(v));
        return v;
    };
    auto issue_codes = [&](int mac, auto j_) {
        constexpr int j = decltype(j_)::value;
        const int stride = opaque(row_bytes);
        static_for<Sched::kCodeLoads>([&](auto i_) {
            constexpr int i = decltype(i_)::value;
            const int piece = piece0 ^ (4 * i);
            int voff = lane_row_off + (j * 16 + 4 * i) * stride + piece * 16;
            if constexpr (kForm != 0) voff = mac * 64 + piece * 16 < code_end ? voff : kOob;
            uint8_t* dst = mine + j * 4096 + i * 1024;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(opb.codes, (lds_ptr_t)dst, 16, voff, mac * 64, 0, 0);
        });
    };
    auto issue_small = [&](int mac) {
        uint8_t* sdst = mine + S::kScaleBase;
        uint8_t* wdst = mine + S::kWordBase;
        if constexpr (kForm == 0) {
            __builtin_amdgcn_raw_ptr_buffer_load_lds(opb.scales, (lds_ptr_t)sdst, 16, l < S::kRows ? l * scale_bytes : kOob, mac * 4, 0, 0);
            if constexpr (kWords) __builtin_amdgcn_raw_ptr_buffer_load_lds(opb.mbs, (lds_ptr_t)wdst, 4, l < S::kRows ? l * nmac : kOob, mac, 0, 0);
        } else if constexpr (kForm == 1) {
            static_for<S::kScaleLoads>([&](auto i_) {  // 16 rows x 4 macro blocks
                constexpr int i = decltype(i_)::value;
                const int voff = mac + (l & 3) < last ? (i * 16 + (l >> 2)) * scale_bytes + (l & 3) * 4 : kOob;
                uint8_t* dst = sdst + i * 256;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(opb.scales, (lds_ptr_t)dst, 4, voff, mac * 4, 0, 0);
            });
            if constexpr (kWords) static_for<S::kWordLoads>([&](auto i_) {  // 32 rows x 2 dwords
                constexpr int i = decltype(i_)::value;
                const int from = mac & ~3, row = i * 32 + (l >> 1);
                const int voff = row < S::kRows && from + (l & 1) * 4 < nmac ? row * nmac + (l & 1) * 4 : kOob;
                uint8_t* dst = wdst + i * 256;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(opb.mbs, (lds_ptr_t)dst, 4, voff, from, 0, 0);
            });
        } else {
            static_for<S::kScaleLoads>([&](auto i_) {  // 8 rows x 8 pairs, or 4 rows x 16 bytes
                constexpr int i = decltype(i_)::value;
                const int col = kForm == 2 ? (l & 7) * 2 : l & 15, row = kForm == 2 ? i * 8 + (l >> 3) : i * 4 + (l >> 4);
                const int voff = mac * 4 + col < scale_bytes ? row * scale_bytes + col : kOob;
                uint8_t* dst = sdst + i * 256;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(opb.scales, (lds_ptr_t)dst, S::kPiece, voff, mac * 4, 0, 0);
            });
            if constexpr (kWords) static_for<S::kWordLoads>([&](auto i_) {  // 16 rows x 4 words
                constexpr int i = decltype(i_)::value;
                const int voff = mac + (l & 3) < nmac ? (i * 16 + (l >> 2)) * nmac + (l & 3) : kOob;
                uint8_t* dst = wdst + i * 256;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(opb.mbs, (lds_ptr_t)dst, 1, voff, mac, 0, 0);
            });
        }
    };

    // ---- activations of a chunk: lane l fetches piece l % 4 of macro block t of row l / 4 (four consecutive lanes one
    // 64-byte piece of a row), the E8M0 bytes and the MBS word of macro block l % 4 of that row; they go through LDS
    // into the operand's layout, lane 16 q + r = block q of row r: ac, and in `as` the lane's byte of each macro block ----
    v4i ac[FM][kSkinnyMacs];
    uint32_t as[FM], a_scale[FM], a_word[FM];
    const int a_row = l >> 2, a_piece = l & 3;
    auto load_a = [&](int mac) {
        const int stride = opaque(row_bytes);
        static_for<FM>([&](auto f_) {
            constexpr int f = decltype(f_)::value;
            static_for<kSkinnyMacs>([&](auto t_) {
                constexpr int t = decltype(t_)::value;
                if (kForm != 0 && mac + t >= last) return;  // (even out of range a load costs the texture-address unit its turn)
                int voff = a_row * row_bytes + a_piece * 16 + f * 16 * stride;
                if constexpr (kForm != 0) voff = (mac + t) * 64 + a_piece * 16 < code_end ? voff : kOob;
                ac[f][t] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(opa.codes, voff, (mac + t) * 64, 0));
            });
            const int at = (f * 16 + a_row) * scale_bytes + a_piece * 4, k = mac * 4 + a_piece * 4;
            if constexpr (kForm <= 1) {
                a_scale[f] = __builtin_amdgcn_raw_buffer_load_b32(opa.scales, kForm == 0 || mac + a_piece < last ? at : kOob, mac * 4, 0);
            } else if constexpr (kForm == 2) {
                const uint32_t lo = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(opa.scales, k < scale_bytes ? at : kOob, mac * 4, 0);
                const uint32_t hi = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(opa.scales, k + 2 < scale_bytes ? at + 2 : kOob, mac * 4, 0);
                a_scale[f] = lo | (hi << 16);
            } else {
                a_scale[f] = 0;
                static_for<4>([&](auto b_) {
                    constexpr int b = decltype(b_)::value;
                    a_scale[f] |= (uint32_t)(uint8_t)__builtin_amdgcn_raw_buffer_load_b8(opa.scales, k + b < scale_bytes ? at + b : kOob, mac * 4, 0) << (8 * b);
                });
            }
            a_word[f] = 0;
            if constexpr (kWords) a_word[f] = (uint8_t)__builtin_amdgcn_raw_buffer_load_b8(opa.mbs, mac + a_piece < nmac ? (f * 16 + a_row) * nmac + a_piece : kOob, mac, 0);
        });
    };
    auto place_a = [&](int count) {
        static_for<FM>([&](auto f_) {
            constexpr int f = decltype(f_)::value;
            static_for<kSkinnyMacs>([&](auto t_) {
                constexpr int t = decltype(t_)::value;
                if (kForm != 0 && t >= count) return;
                lds_store128(exchange + a_piece * 320 + a_row * 16, ac[f][t]);
                ac[f][t] = *reinterpret_cast<const v4i*>(exchange + q * 320 + r * 16);
            });
            lds_store32(exchange + S::kExchangeScales + a_piece * 64 + a_row * 4, a_scale[f]);
            if constexpr (kWords) lds_store32(sig_a + a_piece * (FM * 16) + f * 16 + a_row, __float_as_uint(__builtin_amdgcn_rcpf(1.0f + (float)a_word[f] * (1.0f / 256.0f))));
            as[f] = 0;
            static_for<kSkinnyMacs>([&](auto t_) {
                constexpr int t = decltype(t_)::value;
                as[f] |= (uint32_t)exchange[S::kExchangeScales + t * 64 + r * 4 + q] << (8 * t);
            });
        });
    };
    // fused: unit u = two macro blocks of fragment u / 2; load b of a macro block: lane l fetches piece l % 4 of block b of
    // row l / 4.  (The wait for the weights counts these loads: both go by unit_macs.)
    typedef v4i RawUnit[2][Sched::kRawLoads];
    const int x_off = (l >> 2) * (int)args.ldx * 2 + (l & 3) * 16;
    auto load_raw = [&](RawUnit& raw, int mac, auto u_) {
        constexpr int f = decltype(u_)::value / 2, h = decltype(u_)::value % 2, t0 = h * 2;
        const int stride = opaque((int)args.ldx * 2);
        static_for<2>([&](auto t_) {
            constexpr int t = decltype(t_)::value;
            const int voff = x_off + f * 16 * stride;
            if (t < Sched::unit_macs(last - mac, h)) static_for<Sched::kRawLoads>([&](auto b_) {
                constexpr int b = decltype(b_)::value;
                raw[t][b] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(opx, voff, (mac + t0 + t) * 256 + b * 64, 0));
            });
        });
    };
    auto quantize_raw = [&](RawUnit& raw, v4i (&codes)[kSkinnyMacs], uint32_t& scales, int count, auto f_, auto h_) {
        constexpr int f = decltype(f_)::value, h = decltype(h_)::value, t0 = h * 2;
        static_for<2>([&](auto t_) {
            constexpr int t = decltype(t_)::value;
            if (t >= Sched::unit_macs(count, h)) return;
            const MacroQuant m = quantize_macro(raw[t], args.carry, args.a_mbs, l);
            // through LDS into the operand's layout (the wavefront's LDS operations run in order: no wait between them)
            static_for<4>([&](auto b_) {
                constexpr int b = decltype(b_)::value;
                lds_store32(exchange + b * 320 + l * 4, m.codes[b]);
            });
            lds_store8(exchange + S::kExchangeScales + (l & 3) * 16 + (l >> 2), m.E);
            // (the same value from all four lanes of a row)
            lds_store32(sig_a + (t0 + t) * (FM * 16) + f * 16 + (l >> 2), __float_as_uint(__builtin_amdgcn_rcpf(1.0f + (float)m.m8 * (1.0f / 256.0f))));
            codes[t0 + t] = *reinterpret_cast<const v4i*>(exchange + q * 320 + r * 16);
            scales |= (uint32_t)exchange[S::kExchangeScales + l] << (8 * (t0 + t));
        });
    };

    v4f acc[FM][FN];
#pragma unroll
    for (int f = 0; f < FM; ++f)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[f][j] = v4f{0.f, 0.f, 0.f, 0.f};

    // weights of fragment j of the chunk, out of LDS
    struct Weights {
        v4i codes[kSkinnyMacs];
        uint32_t scale[kSkinnyMacs], word[kSkinnyMacs];
    };
    auto read_weights = [&](Weights& d, [[maybe_unused]] int mac, auto j_) {
        constexpr int j = decltype(j_)::value;
        const uint8_t* scales = mine + S::kScaleBase;
        const uint8_t* words = mine + S::kWordBase;
        static_for<kSkinnyMacs>([&](auto t_) {
            constexpr int t = decltype(t_)::value;
            d.codes[t] = *reinterpret_cast<const v4i*>(mine + j * 4096 + r * 256 + (((q ^ r) ^ (4 * t)) * 16));
        });
        if constexpr (kForm <= 1) {
            const v4i s4 = *reinterpret_cast<const v4i*>(scales + (j * 16 + r) * 16);
            uint32_t m4;
            if constexpr (kForm == 0) {
                m4 = *reinterpret_cast<const uint32_t*>(words + (j * 16 + r) * 4);
            } else {
                typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
                const u32x2 two = *reinterpret_cast<const u32x2*>(words + (j * 16 + r) * 8);
                m4 = __builtin_amdgcn_alignbit(two.y, two.x, 8 * (mac & 3));  // the word of macro block mac in byte 0
            }
            static_for<kSkinnyMacs>([&](auto t_) {
                constexpr int t = decltype(t_)::value;
                d.scale[t] = (uint32_t)s4[t] >> (8 * q);  // the instruction reads byte 0
                d.word[t] = (m4 >> (8 * t)) & 0xFFu;
            });
        } else {
            static_for<kSkinnyMacs>([&](auto t_) {
                constexpr int t = decltype(t_)::value;
                if constexpr (kForm == 2) d.scale[t] = scales[(j * 16 + r) * 32 + (2 * t + (q >> 1)) * 4 + (q & 1)];
                else d.scale[t] = scales[(j * 16 + r) * 64 + (4 * t + q) * 4];
                d.word[t] = words[(j * 16 + r) * 16 + t * 4];
            });
        }
        wait_lds();
    };
    // behind the last read of fragment j: its codes of the next chunk, and behind the last fragment the small arrays
    auto request = [&](int mac, auto j_) {
        issue_codes(mac, j_);
        if constexpr (decltype(j_)::value == FN - 1) issue_small(mac);
    };
    // macro block t of the chunk, fragment pair (f, j): the lane's codes and E8M0 byte (low byte of a_scale) of A
    auto multiply = [&](const Weights& d, auto f_, auto j_, auto t_, v4i a_codes, uint32_t a_scale) {
        constexpr int f = decltype(f_)::value, j = decltype(j_)::value, t = decltype(t_)::value;
        const v4f zero = {0.f, 0.f, 0.f, 0.f};
        const v4f p = mfma_fp4(a_codes, d.codes[t], zero, a_scale, d.scale[t]);  // D[4 q + i][r]: m = 4 q + i, n = r
        // F = 1 + m8/256 is exact, the reciprocal within an ulp; m8 = 0 (also: no words) gives exactly 1
        if constexpr (kWords) {
            const float sn = __builtin_amdgcn_rcpf(1.0f + (float)d.word[t] * (1.0f / 256.0f));
            const v4f sm = *reinterpret_cast<const v4f*>(sig_a + t * (FM * 16) + f * 16 + q * 4);
            acc[f][j] += p * (sm * sn);
        } else {
            acc[f][j] += p;
        }
        asm volatile("" : "+v"(acc[f][j]));  // (keeps the compiler from moving the sums behind the next branch, products alive)
    };

    // fused: the weights of a chunk of `count` macro blocks have landed
    auto wait_weights = [&](int count) {
        if constexpr (Sched::weights_wait(1) == Sched::weights_wait(kSkinnyMacs)) {
            wait_loads_but<Sched::weights_wait(kSkinnyMacs)>();
        } else {  // (uniform over the wavefront)
            if (count >= 4) wait_loads_but<Sched::weights_wait(4)>();
            else if (count == 3) wait_loads_but<Sched::weights_wait(3)>();
            else if (count == 2) wait_loads_but<Sched::weights_wait(2)>();
            else wait_loads_but<Sched::weights_wait(1)>();
        }
    };

    // Everything is requested before anything waits, the activations first: loads return in order, and bringing the
    // activations into the operand's layout (fused: quantizing them) is to run while the weights are on their way.
    if constexpr (kFused) {
        if (first < last) {
            RawUnit raw[2];
            load_raw(raw[0], first, std::integral_constant<int, 0>{});
            load_raw(raw[1], first, std::integral_constant<int, 1>{});
            __builtin_amdgcn_sched_barrier(0);
            issue_small(first);
            static_for<FN>([&](auto j_) { issue_codes(first, j_); });
            __builtin_amdgcn_sched_barrier(0);
            auto chunk = [&](int mac, auto more) __attribute__((always_inline)) {
                const int count = min(last - mac, kSkinnyMacs);
                // fragment by fragment of A: quantize its four macro blocks, request the next activations, multiply
                static_for<FM>([&](auto f_) {
                    constexpr int f = decltype(f_)::value;
                    v4i codes[kSkinnyMacs];
                    uint32_t scales = 0;
                    static_for<2>([&](auto h_) {
                        constexpr int h = decltype(h_)::value;
                        quantize_raw(raw[h], codes, scales, count, f_, h_);
                        __builtin_amdgcn_sched_barrier(0);
                        if constexpr (f + 1 < FM) load_raw(raw[h], mac, std::integral_constant<int, 2 * f + 2 + h>{});
                        else if (more) load_raw(raw[h], mac + kSkinnyMacs, h_);
                        __builtin_amdgcn_sched_barrier(0);
                    });
                    if constexpr (f == 0) wait_weights(count);
                    static_for<FN>([&](auto j_) {
                        Weights d;
                        read_weights(d, mac, j_);
                        if constexpr (f + 1 == FM) {
                            if (more) request(mac + kSkinnyMacs, j_);
                        }
                        static_for<kSkinnyMacs>([&](auto t_) {
                            constexpr int t = decltype(t_)::value;
                            if (kForm == 0 || t < count) multiply(d, f_, j_, t_, codes[t], scales >> (8 * t));
                        });
                        __builtin_amdgcn_sched_barrier(0);
                    });
                });
            };
            using Yes = std::integral_constant<bool, true>;
            using No = std::integral_constant<bool, false>;
            // K <= 8192 is one chunk or two.  Up to 32 rows they are written out: where a loop's two ends meet the compiler's own waits
            // for activations count as if nothing else were in flight, and the weights land before anything is quantized (1 x
            // 4096 x 8192 12.7 -> 12.0 us, 16 x 14336 x 6144 18.3 -> 17.4, 32 x 28672 x 5120 44.3 -> 42.2).  With 64 rows the weights'
            // share of the time is small and the loop's smaller code is faster (64 x 14336 x 8192 48.9 -> 47.1).
            if (kSingle || (FM <= 2 && first + kSkinnyMacs >= last)) {
                chunk(first, No{});
            } else if constexpr (FM <= 2) {
                chunk(first, Yes{});
                chunk(first + kSkinnyMacs, No{});
            } else {
                for (int mac = first; mac < last; mac += kSkinnyMacs) chunk(mac, mac + kSkinnyMacs < last);
            }
        }
    } else {
        if (first < last) {
            load_a(first);
            __builtin_amdgcn_sched_barrier(0);
            issue_small(first);
            static_for<FN>([&](auto j_) { issue_codes(first, j_); });
            __builtin_amdgcn_sched_barrier(0);
            for (int mac = first; mac < last; mac += kSkinnyMacs) {
                const bool more = !kSingle && mac + kSkinnyMacs < last;
                const int count = min(last - mac, kSkinnyMacs);
                place_a(count);
                wait_loads();
                static_for<FN>([&](auto j_) {
                    Weights d;
                    read_weights(d, mac, j_);
                    if (more) request(mac + kSkinnyMacs, j_);
                    static_for<kSkinnyMacs>([&](auto t_) {
                        constexpr int t = decltype(t_)::value;
                        if (kForm == 0 || t < count) {
                            static_for<FM>([&](auto f_) {
                                constexpr int f = decltype(f_)::value;
                                multiply(d, f_, j_, t_, ac[f][t], as[f] >> (8 * t));
                            });
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    });
                    __builtin_amdgcn_sched_barrier(0);
                });
                if (kSingle) break;
                if (more) load_a(mac + kSkinnyMacs);
            }
        }
    }

    // ---- add the partial results, store --------------------------------------------------------
    v4f* red = reinterpret_cast<v4f*>(mine);
#pragma unroll
    for (int f = 0; f < FM; ++f)
#pragma unroll
        for (int j = 0; j < FN; ++j) red[(f * FN + j) * kWave + l] = acc[f][j];
    __syncthreads();
    for (int x = w; x < FM * FN; x += NW) {
        const int f = x / FN, j = x % FN;
        v4f sum = *reinterpret_cast<const v4f*>(smem + (x * kWave + l) * 16);
#pragma unroll
        for (int o = 1; o < NW; ++o) sum += *reinterpret_cast<const v4f*>(smem + o * S::kBytes + (x * kWave + l) * 16);
        const int64_t n = c_n0 + j * 16 + r;
        if (n >= g.N) continue;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int64_t m = m0 + f * 16 + q * 4 + i;
            if (m >= m_end) continue;
            if (g.c_bf16) static_cast<uint16_t*>(g.C)[m * g.ldc + n] = (uint16_t)f32_to_bf16_bits(sum[i]);
            else static_cast<float*>(g.C)[m * g.ldc + n] = sum[i];
        }
    }
}

// A workgroup per 16 FN columns; M <= 16 FM rows or, kTall, as many tiles of 16 FM rows as M has (compiled apart: the second grid dimension
// costs the calls of a few microseconds, which have one, 0.04 to 0.08 us, 1 % of 16 x 4096 x 512).
template <int NW, int FM, int FN, bool kFused, int kForm, bool kSingle, bool kWords, bool kTall>
__global__ __launch_bounds__(NW * kWave) void gemm_skinny_kernel(SkinnyArgs args) {
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const int64_t n0 = (int64_t)blockIdx.x * (16 * FN);
    const int64_t m0 = kTall ? (int64_t)blockIdx.y * (16 * FM) : 0;
    skinny_tile<NW, FM, FN, kFused, kForm, kSingle, kWords>(args, smem, m0, kTall ? min(args.g.M, m0 + 16 * FM) : args.g.M, n0, args.g.N, n0);
}

template <int NW, int FM, int FN, bool kFused, int kForm, bool kTall = false>
int launch_skinny_variant(const SkinnyArgs& a, hipStream_t s) {
    const GemmArgs& g = a.g;
    const int64_t blocks = (g.N + 16 * FN - 1) / (16 * FN), row_tiles = (g.M + 16 * FM - 1) / (16 * FM);
    if (row_tiles > (kTall ? 65535 : 1) || blocks > (int64_t)1 << 30) return MX_EINVAL;
    using S = SkinnyShape<NW, FM, FN, kFused, kForm>;
    auto launch = [&](auto single_, auto words_) {
        auto* fn = gemm_skinny_kernel<NW, FM, FN, kFused, kForm, decltype(single_)::value, decltype(words_)::value, kTall>;
        static LdsOptIn opt_in;  // one per kernel instantiation
        if (int st = opt_in.ensure(reinterpret_cast<const void*>(fn), S::kLdsBytes)) return st;
        hipLaunchKernelGGL(fn, dim3((unsigned)blocks, (unsigned)row_tiles), dim3(S::NT), S::kLdsBytes, s, a);
        return launch_status();
    };
    if (kFused && g.K > 2 * kSingleChunkK(NW)) return MX_EUNSUPPORTED;  // (the kernel takes two chunks at most)
    using Yes = std::integral_constant<bool, true>;
    using No = std::integral_constant<bool, false>;
    const bool single = g.K <= kSingleChunkK(NW);
    if constexpr (!kFused) {
        if (!g.a_mbs && !g.b_mbs) return single ? launch(Yes{}, No{}) : launch(No{}, No{});
    }
    return single ? launch(Yes{}, Yes{}) : launch(No{}, Yes{});
}

}  // namespace
}  // namespace mx
