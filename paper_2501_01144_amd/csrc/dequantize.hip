// DialectFP4 / MXFP4 dequantizer for gfx950 (paper Section 3.3, Figure 6):
// 3-bit index -> 4-bit unsigned integer u through the dialect's table,
// value = (-1)^sign * u * 2^(e-1).  One lane expands one dword of codes
// (8 elements); the dialect's 8 table bytes sit in two registers and
// v_perm_b32 does four lookups per instruction.  Both output types hold the
// values exactly (u has 4 significant bits).
#include <type_traits>

#include "common.h"
#include "formatbook.h"

namespace dfp4 {

static_assert(kBook[7][6] == kE2M1[6] && kBook[7][7] == kE2M1[7] && kBook[7][5] == kE2M1[5],
              "MXFP4 dequantization reuses dialect 7 (FP4 E2M1)");

// book rows packed as two little-endian dwords each
struct BookWords { uint32_t w[kDialects][2]; };
constexpr BookWords make_book_words() {
    BookWords b{};
    for (int d = 0; d < kDialects; ++d)
        for (int j = 0; j < 8; ++j) b.w[d][j / 4] |= (uint32_t)kBook[d][j] << (8 * (j % 4));
    return b;
}
__device__ const BookWords g_book_words = make_book_words();

namespace {

constexpr int kThreads = 256;

typedef uint32_t v4u __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t as_u(float f) { return __builtin_bit_cast(uint32_t, f); }

// The dword of codes c (8 elements) with its dialect and exponent byte.  bf16: all 8, one 16-byte store; fp32: the
// elements 4 half .. 4 half + 3, one 16-byte store.
template <bool BF16>
__device__ __forceinline__ void expand_store(uint32_t c, uint32_t half, uint32_t d, int byte, void* __restrict__ y, int64_t off) {
    constexpr int kElems = BF16 ? 8 : 4;
    const int e = byte - 128;                              // 0.5 u 2^(byte-127) = u 2^(byte-128)
    if constexpr (!BF16) c >>= 16u * half;
    const uint32_t lo = g_book_words.w[d][0], hi = g_book_words.w[d][1];
    const uint32_t mag_even = __builtin_amdgcn_perm(hi, lo, c & 0x07070707u);
    const uint32_t mag_odd = __builtin_amdgcn_perm(hi, lo, (c >> 4) & 0x07070707u);
    uint32_t v[kElems];
#pragma unroll
    for (int j = 0; j < kElems / 2; ++j) {
        const uint32_t ue = (mag_even >> (8 * j)) & 0xffu, uo = (mag_odd >> (8 * j)) & 0xffu;
        v[2 * j] = as_u(ldexpf((float)ue, e)) | ((c << (28 - 8 * j)) & 0x80000000u);
        v[2 * j + 1] = as_u(ldexpf((float)uo, e)) | ((c << (24 - 8 * j)) & 0x80000000u);
    }
    if constexpr (BF16) {
        const v4u o = {(v[0] >> 16) | (v[1] & 0xffff0000u), (v[2] >> 16) | (v[3] & 0xffff0000u),
                       (v[4] >> 16) | (v[5] & 0xffff0000u), (v[6] >> 16) | (v[7] & 0xffff0000u)};
        __builtin_nontemporal_store(o, reinterpret_cast<v4u*>(static_cast<uint16_t*>(y) + off));
    } else {
        const v4u o = {v[0], v[1], v[2], v[3]};
        __builtin_nontemporal_store(o, reinterpret_cast<v4u*>(static_cast<float*>(y) + off));
    }
}

// A wave takes PASSES times 16 blocks (bf16, a dword of codes per lane) or 8 (fp32, half a dword), the loads of all passes
// first; a lane stores 16 bytes and a pass whole lines, past the caches (nobody reads the results soon).  Bound by memory:
// 4096 x 14336 to bf16, operands from HBM, 23.1 us = 6.5 TB/s; 8192 x 4096 to fp32, operands and results in turn from six
// sets, 23.5 us = 6.5 TB/s.  Four passes suit large bf16 tensors (4096 x 14336 in rows with gaps 23.5 us, one pass 27.1),
// one pass everything else: small tensors are latency and want waves (1024 blocks to fp32 2.2 us, with eight passes 3.5;
// to bf16 2.1, with four 2.7), and fp32 has twice the waves (8192 x 4096 again and again 20.8 us, with eight passes 24.6).
// Before: one load, table look-up and store at a time in 4096 persistent workgroups (2.2, 2.1, 38.8 and 43.9 us); a whole
// dword per lane for fp32 stores half a line twice, 56.7 us past the caches and 44.3 through them (whole lines through
// them: 42.4).  `narrow`: one exponent byte and dialect id per 16 elements.
template <bool MX, bool BF16, bool CONTIG, uint32_t PASSES>
__global__ __launch_bounds__(kThreads) void dequantize_kernel(
    const uint32_t* __restrict__ codes, const uint8_t* __restrict__ dialect,
    const uint8_t* __restrict__ exponent, void* __restrict__ y, int64_t ld, uint32_t blocks_per_row,
    uint32_t nblocks, uint32_t narrow) {
    constexpr uint32_t kLanes = BF16 ? 4 : 8, kBlocksPerPass = 64 / kLanes, kPasses = PASSES, kPerWave = kPasses * kBlocksPerPass, kElems = kBlock / kLanes;
    const uint32_t lane = threadIdx.x & 63u, part = lane % kLanes, sub = part * 4u / kLanes;     // dword of the block
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t nsuper = (nblocks + kPerWave - 1u) / kPerWave, stride = gridDim.x * (kThreads / 64);
    for (uint32_t sc = blockIdx.x * (kThreads / 64) + wave; sc < nsuper; sc += stride) {
        uint32_t c[kPasses], e[kPasses], d[kPasses];
#pragma unroll
        for (uint32_t p = 0; p < kPasses; ++p) {
            const uint32_t b = min(sc * kPerWave + p * kBlocksPerPass + lane / kLanes, nblocks - 1u);
            const size_t mb = narrow ? (size_t)b * 2u + (sub >> 1) : (size_t)b;
            c[p] = codes[(size_t)b * 4u + sub];
            e[p] = exponent[mb];
            d[p] = MX ? 7u : ((uint32_t)dialect[mb] & 15u);
        }
#pragma unroll
        for (uint32_t p = 0; p < kPasses; ++p) {
            const uint32_t b = sc * kPerWave + p * kBlocksPerPass + lane / kLanes;
            if (b >= nblocks) break;
            int64_t off;
            if constexpr (CONTIG) {
                off = (int64_t)b * kBlock + part * kElems;
            } else {
                const uint32_t row = b / blocks_per_row;
                off = (int64_t)row * ld + (int64_t)(b - row * blocks_per_row) * kBlock + part * kElems;
            }
            expand_store<BF16>(c[p], part & 1u, d[p], (int)e[p], y, off);
        }
    }
}

}  // namespace

int launch_dequantize(bool mx, dfp4_tensor in, void* y, int y_dtype, int64_t ld, hipStream_t stream, bool narrow) {
    const int64_t nblocks64 = in.rows * (in.K / kBlock);
    if (nblocks64 == 0) return DFP4_OK;
    if (nblocks64 >= (int64_t)1 << 31) return DFP4_ERR_SHAPE;
    const uint32_t nblocks = (uint32_t)nblocks64;
    const bool contig = (ld == in.K), bf16 = y_dtype == DFP4_BF16;
    const uint32_t kb = (uint32_t)(in.K / kBlock);
    const uint32_t* cp = reinterpret_cast<const uint32_t*>(in.codes);
    auto launch = [&](auto mx_c, auto bf16_c, auto contig_c, auto passes_c) {
        constexpr bool kBf16 = decltype(bf16_c)::value;
        constexpr uint32_t kPasses = decltype(passes_c)::value, kPerGroup = (kBf16 ? 16 : 8) * kPasses * (kThreads / 64);
        const uint32_t want = (nblocks + kPerGroup - 1) / kPerGroup, grid = want < (1u << 23) ? want : 1u << 23;   // at most 2^31 threads
        hipLaunchKernelGGL((dequantize_kernel<decltype(mx_c)::value, kBf16, decltype(contig_c)::value, kPasses>), dim3(grid), dim3(kThreads), 0,
                           stream, cp, in.dialect, in.exponent, y, ld, kb, nblocks, narrow ? 1u : 0u);
    };
    auto pick = [](bool v, auto&& f) { if (v) f(std::true_type{}); else f(std::false_type{}); };
    using One = std::integral_constant<uint32_t, 1>;
    using Four = std::integral_constant<uint32_t, 4>;
    pick(mx, [&](auto m) {
        pick(contig, [&](auto c) {
            if (!bf16) launch(m, std::false_type{}, c, One{});
            else if (nblocks < (1u << 20)) launch(m, std::true_type{}, c, One{});
            else launch(m, std::true_type{}, c, Four{});
        });
    });
    return check_launch();
}

}  // namespace dfp4
