// DialectFP4 values in the FP6 E2M3 operand format of the block-scaled matrix instruction,
// and the layout of a packed operand (see gemm_native.hip).  Shared by the packing kernel and
// by the quantizer that writes the packed form directly.
#pragma once
#include "common.h"
#include "formatbook.h"

namespace dfp4 {
namespace {

// E2M3 bit pattern of the magnitude 0.5 u, u = 0..15 (all exact: step 1/8 below 1, 1/4 below 4, 1/2 below 8)
constexpr uint8_t e2m3_of_half_units(int u) {
    return u < 2 ? (uint8_t)(4 * u) : u < 4 ? (uint8_t)(8 + 4 * (u - 2)) : u < 8 ? (uint8_t)(16 + 2 * (u - 4))
                                                                                 : (uint8_t)(24 + (u - 8));
}
struct Fp6Book { uint32_t w[kDialects][2]; };   // [dialect] -> 8 six-bit magnitudes, one per byte
constexpr Fp6Book make_fp6_book() {
    Fp6Book b{};
    for (int d = 0; d < kDialects; ++d)
        for (int j = 0; j < 8; ++j) b.w[d][j / 4] |= (uint32_t)e2m3_of_half_units(kBook[d][j]) << (8 * (j % 4));
    return b;
}
static __device__ const Fp6Book g_fp6_book = make_fp6_book();

// 32 codes -> the 192 bits of a lane's registers: 32 six-bit values, element j in bits [6 j, 6 j + 6).  Twelve-bit pairs in the
// 16-bit halves of a dword first, 24 bits of four elements from those, no 64-bit shifts.
struct Fp6Lane { uint32_t w[6]; };
__device__ __forceinline__ void pack6_quarter(uint32_t c, uint32_t tlo, uint32_t thi, uint32_t& lo24, uint32_t& hi24) {
    const uint32_t e = __builtin_amdgcn_perm(thi, tlo, c & 0x07070707u) | ((c << 2) & 0x20202020u);           // elements 0, 2, 4, 6
    const uint32_t o = __builtin_amdgcn_perm(thi, tlo, (c >> 4) & 0x07070707u) | ((c >> 2) & 0x20202020u);    // elements 1, 3, 5, 7
    const uint32_t p = (e & 0x003f003fu) | ((o & 0x003f003fu) << 6);                                         // 0 1 | 4 5
    const uint32_t q = ((e >> 8) & 0x003f003fu) | (((o >> 8) & 0x003f003fu) << 6);                           // 2 3 | 6 7
    lo24 = (p & 0xffffu) | ((q & 0xffffu) << 12);
    hi24 = (p >> 16) | ((q >> 16) << 12);
}
__device__ __forceinline__ Fp6Lane pack6_lane(uint4 c, uint32_t tlo, uint32_t thi) {
    uint32_t l0, h0, l1, h1, l2, h2, l3, h3;
    pack6_quarter(c.x, tlo, thi, l0, h0);
    pack6_quarter(c.y, tlo, thi, l1, h1);
    pack6_quarter(c.z, tlo, thi, l2, h2);
    pack6_quarter(c.w, tlo, thi, l3, h3);
    return Fp6Lane{{l0 | (h0 << 24), (h0 >> 8) | (l1 << 16), (l1 >> 16) | (h1 << 8),
                    l2 | (h2 << 24), (h2 >> 8) | (l3 << 16), (l3 >> 16) | (h3 << 8)}};
}

// Packed FP6 operand: per (pair of 32-row tiles, step) 3072 bytes = 64 lanes x 16 bytes (registers 0..3) of the even
// tile, the same of the odd tile, then 64 x 8 bytes (registers 4, 5) of the even and of the odd tile;
// lane = 32 * (block % 2) + row % 32.  The 8-byte parts lie in the order [half of the tile's rows][block % 2][row % 16]
// (fp6_hi_lane): the multiply loop reads both blocks of 16 rows at once, which would meet on the same LDS banks otherwise
// (the scales' dwords do, see gen_native_loop.py).  Every KiB is one direct load of a wave into LDS, and both parts are
// read back at their own width.
constexpr int kFp6PairBytes = 3072;
// behind the bits and behind the scales: the multiply loop takes two steps at a time and reads one behind an odd number
constexpr int kSlackSteps = 8;
__host__ __device__ inline size_t fp6_lo(size_t tile, size_t step, size_t S) {
    return ((tile >> 1) * S + step) * kFp6PairBytes + (tile & 1) * 1024;
}
__host__ __device__ inline size_t fp6_hi(size_t tile, size_t step, size_t S) {
    return ((tile >> 1) * S + step) * kFp6PairBytes + 2048 + (tile & 1) * 512;
}

__host__ __device__ inline uint32_t fp6_hi_lane(uint32_t lane) { return (lane & 15u) | (lane & 16u) << 1 | (lane & 32u) >> 1; }

}  // namespace
}  // namespace dfp4
