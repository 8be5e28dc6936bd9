// Block-scaled GEMM on the CDNA4 scaled matrix instructions
// (v_mfma_scale_f32_16x16x128_f8f6f4, few rows v_mfma_scale_f32_32x32x64_f8f6f4): out = A * W^T with
// one power-of-two scale per 32 elements along K applied by the hardware, fp32 accumulation.
//
// Two operand formats:
//   FP4 (E2M1)  MXFP4 tensors are multiplied as they are: the 4-bit code (sign, 3-bit
//               index into {0, .5, 1, 1.5, 2, 3, 4, 6}) is the E2M1 bit pattern and the
//               exponent byte e + 127 is the E8M0 scale.
//   FP6 (E2M3)  every DialectFP4 value 0.5 u (u <= 15) is an E2M3 number, so the codes of
//               both operands are repacked to 6 bits through the dialect tables and the
//               same kernel multiplies them; the exponent byte is again the scale.
// (Section 3.3 of the paper builds its MAC from integer products because its values are
// not a standard format; on this GPU a standard format covers them.)
//
// Operand layout of the instructions (checked on the hardware): lane l supplies row or
// column l % 32 (l % 16) and the 32 consecutive K elements of block l / 32 of the pair (l / 16 of
// the four), element j in bits [w j, w j + w) of its operand registers (w = 4 or 6); the scale is
// the byte of the scale register that op_sel names, 2^(byte - 127).  Output as the other
// MFMAs: register x of lane (h, c) is row 8 (x / 4) + 4 h + x % 4, column c, of lane (q, c) row 4 q + x.
//
// Kernels.  native_pack_kernel rewrites an operand in the order the matrix instruction
// wants it (per 32-row tile and step, 64 lanes x 16 bytes, for FP6 another 64 lanes x 8
// bytes (fp6_pack.h), plus one dword of four scale bytes per lane and group of four
// tiles), so that the multiply kernel's loads are whole lines; weights are packed once,
// offline, and quantize_native_kernel (quantize.hip) writes an activation in this form
// directly.  gemm_native_kernel: 256 x 256 outputs per workgroup, four waves as 2 x 2, each
// 128 x 128 (64 accumulator tiles = 256 registers, one wave per SIMD), or 128 x 256 per
// workgroup when there are few tiles; operands go global -> LDS by direct loads two or three
// iterations of K = 128 ahead, LDS -> registers one ahead, one barrier per iteration; the
// main loop is generated assembly (gen_native_loop.py).  With very few tiles K is split
// between workgroups and native_reduce_kernel adds their fp32 partial tiles in a fixed order.
//
// Exact products (dfp4_gemm and its prepared, batched and requantizing forms; gemm.hip).  Their sums are defined as
// exact, rounded once, and the same kernel gives that where it can be shown that no partial sum rounds.  A row's unit is
// 2^(smallest exponent of its nonzero blocks - 1): every element is a whole number of units, every product a whole
// number of (unit of A's row x unit of W's row), and as long as the absolute products of an output add up to no more
// than 2^24 of these every partial sum, in any order, is a whole number that fp32 holds.  The matrix instructions add
// such terms exactly, but for one exception (2.4e9 outputs of single instructions, 16 x 16 x 128 and 32 x 32 x 64, with
// sums of absolute terms below 2^24 units, block offsets up to 24 binades an operand and addends up to 2^23.9 checked:
// none off but of the exception).  0.5 is a subnormal number of FP6 and FP4, and the instruction aligns a product of two of them as
// if it were four times as large: with blocks 23 binades up, where such a product is 2^23 units, the last bit of the
// sum is lost (FP8, where 0.5 is normal: none).  A dialect's largest magnitude is 8 units or more, so that the product of
// two blocks' largest is 2^29 or more there, and a tile where it is counts as not proven; blocks that a quantizer has
// made hold a magnitude of 8 at least and have no proof then anyway.
// exact_prep_kernel therefore computes, beside the packed form, norms of the rows in units (ExactStat), and a workgroup
// compares three bounds of sum |a||w| with 2^24 after its main loop.  A tile that passes none is computed again in
// int32 from the 4-bit operands by the same workgroup (gemm_int8_tile.h).  On activations with 0.5 % outlier channels
// x 50 and Gaussian weights the bound is 2^20.3 at K = 4096 and 2^22.1 at K = 14336.
#include <type_traits>
#include "common.h"
#include "formatbook.h"
#include "exact_norms.h"
#include "fp6_pack.h"
#include "quant_pass.h"
#include "gemm_int8_tile.h"
#include "gemm_native_asm.inc"

namespace dfp4 {
namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int kFmtFp6 = 2, kFmtFp4 = 4;      // format codes of the instruction (E2M3, E2M1)

// Packed operands (written by native_pack_kernel): rows padded to a multiple of 256,
// S = ceil(KB / 2) steps, a missing second block is all zeros.
//   bits [row tile of 32][step][64 lanes x 16 bytes]                    FP4: registers 0..3 of the lane
//        [pair of row tiles][step][3 KiB]                              FP6: see fp6_pack.h
//   sc   [group of 4 row tiles][step][lane] dword: byte t = scale byte of row tile 4 g + t
// Both arrays end with eight steps of slack: the loop takes two steps at a time and reads one behind an odd number of them.
struct PackedOperand {
    uint8_t* bits;
    uint32_t* sc;
};

struct NativeParams {
    PackedOperand a, w;
    void* out;
    int M, N, S;
    int64_t ldc;
    int rect_w, rects_x, rect_h;      // one XCD's workgroups compute a rectangle of tiles: binary logarithms of its width and of the rectangles
                                      // side by side, and its height (0: rows of tiles one after the other)
    int ksplit;              // workgroups sharing a tile (each a range of steps); partial tiles go to `part`
    float* part;             // [ksplit][M][N] fp32
};

struct PackParams {
    const uint8_t *codes, *dial, *expo;
    PackedOperand dst;
    int rows, KB, S;
};

// One wave per (row tile, step); lane (kh, c) takes row 32 tile + c, block 2 step + kh.
template <int FMT>
__global__ __launch_bounds__(256) void native_pack_kernel(PackParams p) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int kh = lane >> 5, c = lane & 31;
    const int tile = blockIdx.y, s = blockIdx.x * 4 + wave;
    if (s >= p.S) return;
    const int row = tile * 32 + c, kb = 2 * s + kh;
    const bool on = row < p.rows && kb < p.KB;
    uint4 codes = make_uint4(0, 0, 0, 0);
    uint32_t eb = 0, dl = 7;
    if (on) {
        const int64_t blk = (int64_t)row * p.KB + kb;
        codes = *reinterpret_cast<const uint4*>(p.codes + blk * 16);
        eb = p.expo[blk];
        if constexpr (FMT == kFmtFp6) dl = p.dial ? ((uint32_t)p.dial[blk] & 15u) : 7u;
    }
    if constexpr (FMT == kFmtFp4) {
        reinterpret_cast<uint4*>(p.dst.bits)[((int64_t)tile * p.S + s) * 64 + lane] = codes;     // the MXFP4 code is the E2M1 bit pattern
    } else {
        const uint32_t tlo = g_fp6_book.w[dl][0], thi = g_fp6_book.w[dl][1];
        const Fp6Lane v = pack6_lane(codes, tlo, thi);
        *reinterpret_cast<uint4*>(p.dst.bits + fp6_lo(tile, s, p.S) + lane * 16) = make_uint4(v.w[0], v.w[1], v.w[2], v.w[3]);
        *reinterpret_cast<uint2*>(p.dst.bits + fp6_hi(tile, s, p.S) + fp6_hi_lane(lane) * 8) = make_uint2(v.w[4], v.w[5]);
    }
    reinterpret_cast<uint8_t*>(p.dst.sc)[(((int64_t)(tile >> 2) * p.S + s) * 64 + lane) * 4 + (tile & 3)] = (uint8_t)eb;
}

// ---- exact products: the norms of packed rows (ExactStat)
constexpr int kStatChunks = 32;                       // chunks of a row, at most: [row tile][32]
constexpr int kMaxChunkBlocks = 64;

struct ExactOperand {
    const uint8_t *codes, *dial, *expo;
    int64_t src_rows;                 // rows between two problems of a batch
    uint8_t* dst;                     // packed operand, then scales, then norms (ExactLayout)
    int64_t off_sc, off_stat, stride; // bytes
    uint8_t *ref, *mask;              // of gemm_f8_kernel on prepared operands (may be null): [row] and [128 rows][block]
    int rows, groups;                 // groups of 128 rows, an even number
};

struct ExactPrepParams {
    ExactOperand a, w;
    uint32_t* count;                  // cleared: arrival counters of tiles whose K is split, and the count of declined tiles
    int64_t count_stride;             // dwords between two problems; 0 dwords: none
    int counters;
    int KB, S, chunks, chunk_blocks, wgs_a;
};

// the value DPP control CTRL brings to a lane
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float lane_value(float v, int lane) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}
// the largest value of 64 lanes; of every eighth lane's (no LDS: a chain of cross-lane reads there costs a workgroup a microsecond)
__device__ __forceinline__ float rows_max(float v) {
    v = fmaxf(v, dpp<0x128>(v));                      // 8 lanes on, within 16
    return fmaxf(fmaxf(lane_value(v, 0), lane_value(v, 16)), fmaxf(lane_value(v, 32), lane_value(v, 48)));
}
__device__ __forceinline__ float wave_max(float v) {
    v = fmaxf(v, dpp<0xB1>(v));
    v = fmaxf(v, dpp<0x4E>(v));
    v = fmaxf(v, dpp<0x141>(v));
    v = fmaxf(v, dpp<0x140>(v));
    return fmaxf(fmaxf(lane_value(v, 0), lane_value(v, 16)), fmaxf(lane_value(v, 32), lane_value(v, 48)));
}

__device__ __forceinline__ float quad_pair_sum(float v) {     // over 8 neighbouring lanes, in all of them
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0xB1, 0xf, 0xf, true));
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x4E, 0xf, 0xf, true));
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x141, 0xf, 0xf, true));
    return v;
}

// Tables of a dialect: magnitudes u of its 8 indices, and their E2M3 bit patterns
struct ExactBook { uint32_t w[kDialects][4]; };
constexpr ExactBook make_exact_book() {
    ExactBook b{};
    for (int d = 0; d < kDialects; ++d)
        for (int j = 0; j < 8; ++j) {
            b.w[d][j / 4] |= (uint32_t)kBook[d][j] << (8 * (j % 4));
            b.w[d][2 + j / 4] |= (uint32_t)e2m3_of_half_units(kBook[d][j]) << (8 * (j % 4));
        }
    return b;
}
__device__ const ExactBook g_exact_book = make_exact_book();

// Packs operands and computes the norms of their rows.  A workgroup = 128 rows x `chunk_blocks` (8 or 16) blocks of K; wave
// (q, tile) takes rows 8 q .. of row tile `tile` of the four, a lane one block at a time.  Bound by latency: exponents of
// the whole rows (which every chunk reads again, 1/16 of the codes' bytes each time), then codes, tables, stores; so there are 16
// waves to a workgroup, 8 threads look through a row's exponents, and the codes are on their way meanwhile (with 4 waves of 4
// blocks per lane: 2048 x 4096 10.0 us, 2048 x 14336 21.7; so 8.3 and 15.5, one set of buffers, in the caches).  Maxima over
// lanes by DPP and lane reads instead of chains through LDS (2800 of 17000 clocks), and rows of up to 32 groups of 16
// exponents read in as many rounds of eight groups as they have (the last group again to fill a round): 2048 x 4096
// 9.0 -> 7.3 us, 4096 x 4096 14.1 -> 11.4, 2048 x 14336 17.9 -> 17.2 (over eight sets of buffers).  8 lanes read the 128 bytes
// of 8 blocks of a row, so that loads are whole lines, and the 8 rows of a wave are 128 contiguous bytes of a step's
// 16-byte parts.
template <int FMT>
__global__ __launch_bounds__(1024, 8) void exact_prep_kernel(ExactPrepParams p) {
    __shared__ __attribute__((aligned(16))) uint32_t s_book[kDialects][4];
    __shared__ uint8_t s_ref[128], s_low[128];                         // smallest exponent of the nonzero blocks; of all blocks
    __shared__ uint32_t s_mask[kMaxChunkBlocks];
    __shared__ __attribute__((aligned(4))) uint8_t s_sc[8][32][4];     // scale bytes: [block][row][tile of the group]
    __shared__ ExactStat s_stat[4][4];
    // packed lanes, [tile of the group][block][row]; a block's rows are followed by a gap, so that the 8 blocks of a row that
    // neighbouring lanes write fall on different banks
    constexpr int kLoPitch = 32 * 16 + 16, kHiPitch = 32 * 8 + 8;
    __shared__ __attribute__((aligned(16))) uint8_t s_lo[32 * kLoPitch], s_hi[FMT == kFmtFp6 ? 32 * kHiPitch : 16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool is_w = (int)blockIdx.x >= p.wgs_a;
    const ExactOperand o = is_w ? p.w : p.a;
    const int wg = (int)blockIdx.x - (is_w ? p.wgs_a : 0), group = wg / p.chunks, chunk = wg % p.chunks;
    const int64_t bz = blockIdx.z;
    const int KB = p.KB;
    const int64_t src0 = bz * o.src_rows;
    uint8_t* dst = o.dst + bz * o.stride;
    const int k8 = lane & 7, t4 = wave & 3, r = (wave >> 2) * 8 + (lane >> 3);
    const int tile = group * 4 + t4, row = tile * 32 + r;
    // (no branch around a load: a block outside the operand reads the last and is cleared where it is used)
    struct Block { uint4 c; uint32_t e, d; };
    const uint32_t blk_row = (uint32_t)min(row, o.rows - 1) * (uint32_t)KB;
    const uint8_t *codes = o.codes + src0 * KB * 16, *expo = o.expo + src0 * KB, *dial = FMT == kFmtFp6 ? o.dial + src0 * KB : nullptr;
    auto load = [&](int sub) {
        Block b;
        const uint32_t blk = blk_row + (uint32_t)min(chunk * p.chunk_blocks + sub + k8, KB - 1);
        b.c = *reinterpret_cast<const uint4*>(codes + (uint64_t)blk * 16);
        b.e = expo[blk];
        b.d = FMT == kFmtFp6 ? dial[blk] : 7;
        return b;
    };
    Block cur = load(0);
    if (tid < kDialects * 4) (&s_book[0][0])[tid] = (&g_exact_book.w[0][0])[tid];
    if (tid < kMaxChunkBlocks) s_mask[tid] = 0;
    if (blockIdx.x == 0)
        for (int i = tid; i < p.counters; i += 1024) p.count[bz * p.count_stride + i] = 0;
    {
        // references: 8 threads per row
        const int srow = group * 128 + (tid >> 3), part = tid & 7;
        // pairs of bytes minus 1 as 16-bit numbers: a zero byte (an all-zero block) becomes 0xffff and is passed over
        typedef uint16_t v2u __attribute__((ext_vector_type(2)));
        v2u mn2 = {0xffff, 0xffff}, any2 = {0, 0};
        auto scan = [&](uint32_t w) {
            const v2u one = {1, 1}, lo = __builtin_bit_cast(v2u, w & 0x00ff00ffu) - one, hi = __builtin_bit_cast(v2u, (w >> 8) & 0x00ff00ffu) - one;
            mn2 = __builtin_elementwise_min(mn2, __builtin_elementwise_min(lo, hi));
            any2 |= lo | hi;
        };
        if (srow < o.rows) {
            const uint8_t* e = o.expo + (src0 + srow) * KB;
            const int n16 = KB >> 4;
            for (int i0 = part; i0 < n16; i0 += 32) {
                uint4 v[4];
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (8 * q < n16) __builtin_memcpy(&v[q], e + 16 * min(i0 + 8 * q, n16 - 1), 16);          // no alignment assumed
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (8 * q < n16) { scan(v[q].x); scan(v[q].y); scan(v[q].z); scan(v[q].w); }
            }
            for (int i = n16 * 16 + part; i < KB; i += 8) scan(e[i] * 0x01010101u);
        }
        int mn = min((int)mn2.x, (int)mn2.y);
        mn = mn == 0xffff ? 255 : mn;
        int all = ((uint32_t)(any2.x | any2.y) & 0x8000u) ? 0 : mn + 1;
#pragma unroll
        for (int x = 1; x < 8; x <<= 1) {
            mn = min(mn, __shfl_xor(mn, x));
            all = min(all, __shfl_xor(all, x));
        }
        all = min(all, 255);
        if (part == 0) {
            s_ref[tid >> 3] = (uint8_t)(mn + 1);                       // 0: no nonzero block
            s_low[tid >> 3] = (uint8_t)all;
            if (o.ref && chunk == 0 && srow < o.rows) o.ref[srow] = (uint8_t)all;
        }
    }
    __syncthreads();
    const int ref = s_ref[t4 * 32 + r], lowest = s_low[t4 * 32 + r];
    ExactStat m{0, 0, 0, 0};                          // of this lane's blocks
    for (int sub = 0; sub < p.chunk_blocks; sub += 8) {
        const bool on = row < o.rows && chunk * p.chunk_blocks + sub + k8 < KB;
        const uint4 c = on ? cur.c : make_uint4(0, 0, 0, 0);
        const uint32_t e = on ? cur.e : 0;
        const uint4 tab = *reinterpret_cast<const uint4*>(&s_book[cur.d & 15u][0]);
        if (sub + 8 < p.chunk_blocks) cur = load(sub + 8);
        const uint32_t c4[4] = {c.x, c.y, c.z, c.w};
        uint32_t s1 = 0, s2 = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t ue = __builtin_amdgcn_perm(tab.y, tab.x, c4[k] & 0x07070707u);
            const uint32_t uo = __builtin_amdgcn_perm(tab.y, tab.x, (c4[k] >> 4) & 0x07070707u);
            s2 = __builtin_amdgcn_udot4(ue, ue, __builtin_amdgcn_udot4(uo, uo, s2, false), false);
            s1 = __builtin_amdgcn_udot4(ue, 0x01010101u, __builtin_amdgcn_udot4(uo, 0x01010101u, s1, false), false);
        }
        const int delta = (int)e - ref;
        // not for the fp32 path: a reference out of range, a nonzero block with byte 0 (passed over above), byte 255 (no scale)
        const bool off = e == 255 || (s1 != 0 && (e == 0 || ref < kMinRef || ref > kMaxRef));
        if (s1 != 0 || off) {
            const float inf = __builtin_inff(), v2 = off ? inf : ldexpf((float)s2, 2 * delta);
            m.sq += v2;
            if (off || delta < 4) m.sq_low += v2;
            if (off || delta >= 4) m.sum_high += off ? inf : ldexpf((float)s1, delta);
            m.top = off ? inf : fmaxf(m.top, ldexpf((float)(tab.y >> 24), delta));
        }
        s_sc[k8][r][t4] = (uint8_t)e;
        if constexpr (FMT == kFmtFp4) {
            *reinterpret_cast<uint4*>(s_lo + (t4 * 8 + k8) * kLoPitch + r * 16) = c;
        } else {
            const Fp6Lane v = pack6_lane(c, tab.z, tab.w);
            *reinterpret_cast<uint4*>(s_lo + (t4 * 8 + k8) * kLoPitch + r * 16) = make_uint4(v.w[0], v.w[1], v.w[2], v.w[3]);
            *reinterpret_cast<uint2*>(s_hi + (t4 * 8 + k8) * kHiPitch + r * 8) = make_uint2(v.w[4], v.w[5]);
        }
        if (o.mask) {
            uint32_t cls = on ? 1u << min(((int)e - lowest) >> 2, kMaxClass + 1) : 0u;
            cls |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)cls, 0x128, 0xf, 0xf, true);      // 8 lanes on: another row of the same blocks
            if ((lane & 8) == 0) atomicOr(&s_mask[sub + k8], cls);
        }
        __syncthreads();
        {
            // wave (q, tile) writes step q of the tile: whole lines
            const int q = wave >> 2, half = t4 * 8 + 2 * q + (lane >> 5), st = (chunk * p.chunk_blocks + sub) / 2 + q;
            if (st < p.S) {
                const uint4 lo = *reinterpret_cast<const uint4*>(s_lo + half * kLoPitch + (lane & 31) * 16);
                if constexpr (FMT == kFmtFp4) {
                    reinterpret_cast<uint4*>(dst)[((int64_t)tile * p.S + st) * 64 + lane] = lo;
                } else {
                    *reinterpret_cast<uint4*>(dst + fp6_lo(tile, st, p.S) + lane * 16) = lo;
                    *reinterpret_cast<uint2*>(dst + fp6_hi(tile, st, p.S) + fp6_hi_lane(lane) * 8) =
                        *reinterpret_cast<const uint2*>(s_hi + half * kHiPitch + (lane & 31) * 8);
                }
            }
        }
        if (tid < 256) {
            // scale dwords of the group's four tiles: 8 blocks x 32 rows
            const int blk = tid >> 5, sr = tid & 31, kbs = chunk * p.chunk_blocks + sub + blk;
            if ((kbs >> 1) < p.S)
                reinterpret_cast<uint32_t*>(dst + o.off_sc)[((int64_t)group * p.S + (kbs >> 1)) * 64 + 32 * (kbs & 1) + sr] =
                    *reinterpret_cast<const uint32_t*>(&s_sc[blk][sr][0]);
        }
        if (sub + 8 < p.chunk_blocks) __syncthreads();
    }
    if (o.mask && tid < p.chunk_blocks && chunk * p.chunk_blocks + tid < KB)
        o.mask[(int64_t)group * KB + chunk * p.chunk_blocks + tid] = (uint8_t)s_mask[tid];
    // over the 8 lanes of a row, then the largest of the wave's 8 rows, of the tile's 32
    m.sq = quad_pair_sum(m.sq);
    m.sq_low = quad_pair_sum(m.sq_low);
    m.sum_high = quad_pair_sum(m.sum_high);
    m.top = wave_max(m.top);
    m.sq = rows_max(m.sq);
    m.sq_low = rows_max(m.sq_low);
    m.sum_high = rows_max(m.sum_high);
    if (lane == 0) s_stat[wave >> 2][t4] = m;
    __syncthreads();
    if (wave < 4) {
        ExactStat* stat = reinterpret_cast<ExactStat*>(dst + o.off_stat) + (int64_t)(group * 4 + wave) * kStatChunks;
        if (lane == 0) {
            ExactStat t = s_stat[0][wave];
#pragma unroll
            for (int q = 1; q < 4; ++q) {
                const ExactStat v = s_stat[q][wave];
                t.sq = fmaxf(t.sq, v.sq);
                t.sq_low = fmaxf(t.sq_low, v.sq_low);
                t.sum_high = fmaxf(t.sum_high, v.sum_high);
                t.top = fmaxf(t.top, v.top);
            }
            stat[chunk] = t;
        }
        if (chunk == 0 && lane >= p.chunks && lane < kStatChunks) stat[lane] = ExactStat{0, 0, 0, 0};
    }
}

struct ExactParams : NativeParams {
    GemmParams g;                     // the operands in their 4-bit form, results, requantized results
    const ExactStat *a_stat, *w_stat;
    int64_t a_stride, w_stride;       // bytes between the prepared operands of two problems
    uint32_t* cnt;                    // arrival counters (split K), one per tile
    int64_t cnt_stride;               // dwords
};

// the larger of the sums over lanes 0..31 and 32..63
__device__ __forceinline__ float half_sum_max(float v) {
    v = quad_pair_sum(v);
    v += dpp<0x140>(v);                               // mirrored within 16 lanes
    return fmaxf(lane_value(v, 0) + lane_value(v, 16), lane_value(v, 32) + lane_value(v, 48));
}
// The largest norms of a wave's rows (lane: chunk lane % 32 of tile lane / 32 of each pair of tiles), in all lanes
template <int N>
__device__ __forceinline__ ExactStat reduce_stat(ExactStat (&v)[N]) {
    ExactStat m{0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < N; ++i) {
        m.sq = fmaxf(m.sq, half_sum_max(v[i].sq));
        m.sq_low = fmaxf(m.sq_low, half_sum_max(v[i].sq_low));
        m.sum_high = fmaxf(m.sum_high, half_sum_max(v[i].sum_high));
        m.top = fmaxf(m.top, v[i].top);
    }
    m.top = wave_max(m.top);
    return m;
}

constexpr float kSubnormalUnits = 536870912.0f;      // 2^29, see the file header
// two results in bf16 (round to nearest even), the first in the low half
__device__ __forceinline__ uint32_t bf16_pair(int a, int b) {
    typedef float v2f __attribute__((ext_vector_type(2)));
    typedef __bf16 v2b __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v2f{__builtin_bit_cast(float, a), __builtin_bit_cast(float, b)}, v2b));
}

constexpr int kRqPitch = 136;         // bf16 per staged output row (128 + 8: rows stay 16-byte aligned)
// requantizing epilogue: quantizer tables and, per wave, 64 rows x 128 columns of bf16 results, where the operands were
struct RequantLds {
    __attribute__((aligned(16))) uint8_t q[kDialects * 1024], s[kPairs * 1024];
    __attribute__((aligned(16))) uint16_t st[4 * 64 * kRqPitch];
};

// the quantizer's tables, by a workgroup of 256 threads
template <bool MX>
__device__ __forceinline__ void load_requant_tables(RequantLds& l) {
    if constexpr (MX) {
        if (threadIdx.x < 64) l.q[threadIdx.x] = g_quant_tables.mx[threadIdx.x];
    } else {
        const uint4* gq = reinterpret_cast<const uint4*>(g_quant_tables.q);
        const uint4* gs = reinterpret_cast<const uint4*>(g_quant_tables.s);
        for (int i = threadIdx.x; i < 1024; i += 256) reinterpret_cast<uint4*>(l.q)[i] = gq[i];
        for (int i = threadIdx.x; i < 512; i += 256) reinterpret_cast<uint4*>(l.s)[i] = gs[i];
    }
}

// Requantizing GEMM, tiles that went through the per-block flush: quantize the 128 x 128 bf16
// results the workgroup has just written to the temporary `p.out` (16 rows x 4 blocks per sweep,
// 4 lanes per block).  lds_s / lds_q: the quantizer's tables.
template <bool MX>
__device__ __forceinline__ void quantize_flushed_piece(const GemmParams& p, int64_t bz, int by, int bx,
                                                       const uint8_t* lds_s, const uint8_t* lds_q) {
    __threadfence_block();
    __syncthreads();
    const int tid = threadIdx.x;
    const int nb_row = p.N / kBlock;
    const uint16_t* src = static_cast<const uint16_t*>(p.out) + bz * p.strideC;
    for (int sweep = 0; sweep < 8; ++sweep) {
        const int q = tid >> 2, sub = tid & 3;
        const int m = by * 128 + sweep * 16 + (q >> 2), nb = bx * 4 + (q & 3);
        const bool valid = m < p.M && nb < nb_row;      // the same for the 4 lanes of a block
        uint4 wv = make_uint4(0, 0, 0, 0);
        if (valid) wv = *reinterpret_cast<const uint4*>(src + (int64_t)m * p.ldc + nb * kBlock + sub * 8);
        uint32_t code, eb, dl = 0;
        if constexpr (MX) mxfp4_pass(wv, lds_q, code, eb);
        else dfp4_pass(wv, lds_s, lds_q, code, eb, dl);
        if (valid) {
            const size_t blk = (size_t)(bz * p.M + m) * nb_row + nb;
            p.q_codes[blk * 4 + sub] = code;
            if (sub == 0) {
                p.q_exp[blk] = (uint8_t)eb;
                if constexpr (!MX) p.q_dial[blk] = (uint8_t)dl;
            }
        }
    }
    __syncthreads();
}

// TA = 32-row tiles per wave: 4 (256 x 256 per workgroup) or 2 (128 x 256, for products with few tiles)
// MODE: what is made of the sums.  kPlain: dfp4_gemm_native.  kExact: the exact products.  kRequant: those, quantized.
constexpr int kPlain = 0, kExact = 1, kRequant = 2;
template <int FMT, bool BF16, int TA, int MODE>
__global__ __launch_bounds__(256, 1) void gemm_native_kernel(std::conditional_t<MODE == kPlain, NativeParams, ExactParams> p) {
    constexpr bool kFp6 = FMT == kFmtFp6;
    using PieceShape = DirectShape<2, 2, 2, 2, 1>;           // 128 x 128 by 256 threads
    constexpr int kTileLds = kFp6 ? 1536 : 1024, kStage = (2 * TA + 8) * kTileLds + 1024;
    constexpr int kStages = kFp6 && TA == 4 ? 6 : 8;
    constexpr int kRowsWg = 64 * TA, kRowsWave = 32 * TA;
    constexpr int kGStride = kFp6 ? kFp6PairBytes : 1024;    // global bytes per (pair of tiles, step) / (tile, step)
    __shared__ __attribute__((aligned(16))) uint8_t s_stage[kStages * kStage];
    constexpr int kPieceAt = MODE == kRequant ? offsetof(RequantLds, st) : 0;      // behind the quantizer's tables
    static_assert(MODE == kPlain || (kPieceAt + sizeof(TileLds<PieceShape>) <= sizeof(s_stage) && kPieceAt % 16 == 0));
    static_assert(MODE != kRequant || sizeof(RequantLds) <= sizeof(s_stage));
    __shared__ int s_ctl[5];                                 // exact: per wave, whether its sums are exact; arrivals (split K)
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = (int)wave >> 1, wn = (int)wave & 1;
    // this workgroup's tile
    int bx = (int)blockIdx.x, by = (int)blockIdx.y;
    if (p.rect_h) {
        const int id = by * (int)gridDim.x + bx, rect = id & 7, in = id >> 3;
        bx = ((rect & ((1 << p.rects_x) - 1)) << p.rect_w) + (in & ((1 << p.rect_w) - 1));
        by = (rect >> p.rects_x) * p.rect_h + (in >> p.rect_w);
    }
    // this workgroup's range of steps (split K: blockIdx.z, in exact products below the problem of a batch)
    const int per = (p.S + p.ksplit - 1) / p.ksplit;
    const int sidx = MODE == kPlain ? (int)blockIdx.z : (int)(blockIdx.z % (unsigned)p.ksplit);
    const int64_t bz = MODE == kPlain ? 0 : blockIdx.z / (unsigned)p.ksplit;
    const int s_lo = sidx * per, S = min(p.S, s_lo + per) - s_lo;
    // norms of the wave's rows of A and of W: used after the main loop, on their way during it
    ExactStat stat_a[TA / 2], stat_w[2];
    if constexpr (MODE != kPlain) {
        p.a.bits += bz * p.a_stride;
        p.w.bits += bz * p.w_stride;
        p.a.sc += bz * (p.a_stride / 4);
        p.w.sc += bz * (p.w_stride / 4);
        const uint8_t* sa = reinterpret_cast<const uint8_t*>(p.a_stat + ((int64_t)by * (2 * TA) + wm * TA) * kStatChunks) + bz * p.a_stride;
        const uint8_t* sw = reinterpret_cast<const uint8_t*>(p.w_stat + ((int64_t)bx * 8 + wn * 4) * kStatChunks) + bz * p.w_stride;
#pragma unroll
        for (int i = 0; i < TA / 2; ++i) stat_a[i] = reinterpret_cast<const ExactStat*>(sa)[i * 64 + (threadIdx.x & 63)];
#pragma unroll
        for (int i = 0; i < 2; ++i) stat_w[i] = reinterpret_cast<const ExactStat*>(sw)[i * 64 + (threadIdx.x & 63)];
    }
    {
        const uint32_t lds = (uint32_t)__builtin_amdgcn_readfirstlane(
            (int)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)&s_stage[0]);
        const uint32_t tstride = (uint32_t)p.S * (uint32_t)kGStride;      // bytes per tile (FP4) / pair of tiles
        // this wave fetches A tiles 2w, 2w+1 (128-row form: tile w) and B tiles 2w, 2w+1 of the workgroup's 8 + 8,
        // and scale chunk w
        const uint64_t a_tile = (uint64_t)by * (2 * TA) + (TA == 4 ? 2 * wave : wave);
        const uint64_t b_tile = (uint64_t)bx * 8 + 2 * wave;
        const uint64_t ab = reinterpret_cast<uint64_t>(p.a.bits) + (kFp6 ? fp6_lo(a_tile, 0, p.S) : a_tile * tstride);
        const uint64_t bb = reinterpret_cast<uint64_t>(p.w.bits) + (kFp6 ? fp6_lo(b_tile, 0, p.S) : b_tile * tstride);
        const uint64_t sb = wave < 2
            ? reinterpret_cast<uint64_t>(p.a.sc) + (TA == 4 ? (uint64_t)by * 2 + wave : (uint64_t)by) * (uint64_t)p.S * 256
            : reinterpret_cast<uint64_t>(p.w.sc) + ((uint64_t)bx * 2 + (wave - 2)) * (uint64_t)p.S * 256;
        uint32_t lane = threadIdx.x & 63u;
        asm volatile("" : "+v"(lane));                       // nothing of it is kept through the loop for what follows, registers are short
        const uint32_t l16 = lane * 16u, l4 = lane * 4u;
        // LDS offsets of lane (q, c): stage q / 2 of a slot, block q % 2 of row c
        const uint32_t q = lane >> 4, c = lane & 15u, q_at = (q >> 1) * kStage, q_blk = (q & 1u) * 32u + c;
        const uint32_t r16 = q_at + q_blk * 16u, r8 = q_at + ((q & 1u) * 16u + c) * 8u, r4 = q_at + q_blk * 4u;
        const uint32_t g16 = l16 + (uint32_t)s_lo * kGStride, g4 = l4 + (uint32_t)s_lo * 256u;
        const uint32_t iters = (uint32_t)(S + 1) / 2u;
#define DFP4_NATIVE_RUN(LOOP)                                                                                     \
        asm volatile(LOOP                                                                                           \
                     :                                                                                              \
                     : [alo] "s"((uint32_t)ab), [ahi] "s"((uint32_t)(ab >> 32)), [blo] "s"((uint32_t)bb),        \
                       [bhi] "s"((uint32_t)(bb >> 32)), [slo] "s"((uint32_t)sb), [shi] "s"((uint32_t)(sb >> 32)), \
                       [tstride] "s"(tstride), [wv] "s"(wave), [lds] "s"(lds),                                      \
                       [iters] "s"(iters),                                                                           \
                       [half] "s"((S & 1) ? iters - 1u : 0xffffffffu),                                              \
                       [g16] "v"(g16), [g4] "v"(g4), [r16] "v"(r16), [r8] "v"(r8), [r4] "v"(r4)                   \
                     : DFP4_NATIVE_VGPR_CLOBBERS, DFP4_NATIVE_ACC_CLOBBERS, DFP4_NATIVE_SGPR_CLOBBERS, "m0", "scc", \
                       "memory")
        if constexpr (kFp6 && TA == 4) DFP4_NATIVE_RUN(DFP4_NATIVE_LOOP_FP6);
        else if constexpr (kFp6) DFP4_NATIVE_RUN(DFP4_NATIVE_LOOP_FP6_H);
        else if constexpr (TA == 4) DFP4_NATIVE_RUN(DFP4_NATIVE_LOOP_FP4);
        else DFP4_NATIVE_RUN(DFP4_NATIVE_LOOP_FP4_H);
#undef DFP4_NATIVE_RUN
    }

    // epilogue: fp32 (or bf16, round to nearest even) [M, N].  Accumulator registers come in groups of 16: group G is row tile
    // G / 2 (of 16 rows), columns 64 (G % 2) + ..; register 4 j + x of lane (q, c) is row c, column 16 j + 4 q + x of it.
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));                            // (anew, see above)
    const int lane = tid & 63, q = lane >> 4, c = lane & 15;
    const int m0 = by * kRowsWg + wm * kRowsWave, n0 = bx * 256 + wn * 128;
#define DFP4_NATIVE_READ(G, V)                                                                      \
    asm volatile(DFP4_NATIVE_ACC_READ_##G                                                           \
                 : "=v"(V[0]), "=v"(V[1]), "=v"(V[2]), "=v"(V[3]), "=v"(V[4]), "=v"(V[5]),          \
                   "=v"(V[6]), "=v"(V[7]), "=v"(V[8]), "=v"(V[9]), "=v"(V[10]), "=v"(V[11]),        \
                   "=v"(V[12]), "=v"(V[13]), "=v"(V[14]), "=v"(V[15]))
#define DFP4_NATIVE_TILES(F)                                                                        \
    F(0) F(1) F(2) F(3) F(4) F(5) F(6) F(7)                                                         \
    if constexpr (TA == 4) { F(8) F(9) F(10) F(11) F(12) F(13) F(14) F(15) }
    // exact products, split K: the tile's partial sums, [range][(16 tile + x) * 256 + thread]
    constexpr int kPartTile = TA * 4 * 16 * 256;
    const float* parts = nullptr;
    if constexpr (MODE != kPlain) {
        // (nothing of this before the loop: the norms are still on their way there)
#pragma unroll
        for (int i = 0; i < TA / 2; ++i) asm volatile("" : "+v"(stat_a[i].sq), "+v"(stat_a[i].sq_low), "+v"(stat_a[i].sum_high), "+v"(stat_a[i].top));
#pragma unroll
        for (int i = 0; i < 2; ++i) asm volatile("" : "+v"(stat_w[i].sq), "+v"(stat_w[i].sq_low), "+v"(stat_w[i].sum_high), "+v"(stat_w[i].top));
        const ExactStat top_a = reduce_stat(stat_a), top_w = reduce_stat(stat_w);
        const bool exact = sums_exactly(top_a, top_w) && top_a.top * top_w.top < kSubnormalUnits;
        if (lane == 0) s_ctl[wave] = exact ? 1 : 0;
        __syncthreads();                                     // and the operands in LDS are done with
        if (__builtin_amdgcn_readfirstlane(s_ctl[0] & s_ctl[1] & s_ctl[2] & s_ctl[3]) == 0) {
            asm volatile("; accumulators are dead from here");
            if (sidx != 0) return;                           // all that share the tile find the same
            TileLds<PieceShape>& lds = *reinterpret_cast<TileLds<PieceShape>*>(s_stage + kPieceAt);
            if constexpr (MODE == kRequant) load_requant_tables<!kFp6>(*reinterpret_cast<RequantLds*>(s_stage));
#pragma unroll 1
            for (int i = 0; i < TA; ++i) {
                int piece = i;
                asm volatile("" : "+s"(piece));              // nothing of a piece is kept in registers for the next
                const int py = by * (TA / 2) + (piece >> 1), px = bx * 2 + (piece & 1);
                if (py * 128 >= p.M || px * 128 >= p.N) continue;
                int8_tile<!kFp6, BF16, PieceShape>(p.g, lds, bz, py, px);
                __syncthreads();
                if constexpr (MODE == kRequant) {
                    const RequantLds& rq = *reinterpret_cast<const RequantLds*>(s_stage);
                    quantize_flushed_piece<!kFp6>(p.g, bz, py, px, rq.s, rq.q);
                }
            }
            return;
        }
        if (p.ksplit > 1) {
            // Every range's workgroup publishes its partial sums and counts itself in; the last adds the others' to its own (exact,
            // so in any order) and finishes the tile.  The sums travel as device-scope relaxed atomics: they pass the per-XCD L2,
            // which a fence would write back as a whole.  "All my stores have completed" is the wait before the barrier.
            const int tile_id = (int)(by * (int)gridDim.x + bx);
            const int64_t tiles = (int64_t)gridDim.x * gridDim.y;
            float* range0 = p.part + ((bz * tiles + tile_id) * p.ksplit) * (int64_t)kPartTile;
            parts = range0;
            if (m0 < p.M && n0 < p.N) {
                float* mine = range0 + (int64_t)sidx * kPartTile;
#define DFP4_NATIVE_PUBLISH(G)                                                                      \
                {                                                                                   \
                    int v[16];                                                                      \
                    DFP4_NATIVE_READ(G, v);                                                         \
                    _Pragma("unroll") for (int x = 0; x < 16; ++x)                                  \
                        __hip_atomic_store(reinterpret_cast<int*>(mine) + (G * 16 + x) * 256 + tid, v[x], __ATOMIC_RELAXED, \
                                           __HIP_MEMORY_SCOPE_AGENT);                               \
                }
                DFP4_NATIVE_TILES(DFP4_NATIVE_PUBLISH)
#undef DFP4_NATIVE_PUBLISH
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            if (tid == 0) {
                uint32_t* cnt = p.cnt + bz * p.cnt_stride + tile_id;
                const uint32_t arrived = atomicAdd(cnt, 1u);
                if (arrived == (uint32_t)p.ksplit - 1u) atomicExch(cnt, 0u);      // ready for the next product
                s_ctl[4] = (int)arrived;
            }
            __syncthreads();
            if (s_ctl[4] != p.ksplit - 1) return;
        }
        if constexpr (MODE == kRequant) {
            load_requant_tables<!kFp6>(*reinterpret_cast<RequantLds*>(s_stage));
            __syncthreads();
        }
    }
    if constexpr (MODE == kPlain) __syncthreads();               // the operands in LDS are done with
    if (m0 >= p.M || n0 >= p.N) return;
    // accumulator group G, with the other ranges' partial sums in exact products
    auto finish = [&](auto g_c, int (&v)[16]) {
        if constexpr (MODE != kPlain) {
            if (p.ksplit > 1) {
                for (int r = 0; r < p.ksplit; ++r) {
                    if (r == sidx) continue;
                    const float* other = parts + (int64_t)r * kPartTile;
#pragma unroll
                    for (int x = 0; x < 16; ++x)
                        v[x] = __builtin_bit_cast(int, __builtin_bit_cast(float, v[x]) +
                                  __builtin_bit_cast(float, __hip_atomic_load(reinterpret_cast<const int*>(other) + (decltype(g_c)::value * 16 + x) * 256 + tid,
                                                                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)));
                }
            }
        }
    };
    // Results pass between the lanes of a wave through its part of LDS.  A wave's LDS operations execute in order; this keeps the compiler to it
    auto in_order = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    if constexpr (MODE == kRequant) {
        // Section 3.3: results are quantized again for the next multiplication.  Each value is rounded to bf16 as the bf16 output
        // would be; the wave stages 64 rows x 128 columns in LDS and re-reads them in the quantizer's layout (4 lanes per
        // block of 32 consecutive columns).
        RequantLds& rq = *reinterpret_cast<RequantLds*>(s_stage);
        uint16_t* st = &rq.st[wave * 64 * kRqPitch];
        const int nb_row = p.N / kBlock;
#pragma unroll
        for (int half = 0; half < TA / 2; ++half) {
#define DFP4_NATIVE_STAGE(G)                                                                        \
            if ((G >> 3) == half) {                                                                 \
                int v[16];                                                                          \
                DFP4_NATIVE_READ(G, v);                                                             \
                finish(std::integral_constant<int, G>{}, v);                                        \
                _Pragma("unroll") for (int j = 0; j < 4; ++j)                                       \
                    *reinterpret_cast<uint2*>(&st[(((G >> 1) & 3) * 16 + c) * kRqPitch + (G & 1) * 64 + 16 * j + 4 * q]) = \
                        make_uint2(bf16_pair(v[4 * j], v[4 * j + 1]), bf16_pair(v[4 * j + 2], v[4 * j + 3])); \
            }
            DFP4_NATIVE_TILES(DFP4_NATIVE_STAGE)
#undef DFP4_NATIVE_STAGE
            in_order();
            for (int pass = 0; pass < 16; ++pass) {
                const int b = pass * 16 + (lane >> 2), row = b >> 2, cb = b & 3, sub = lane & 3;
                const uint4 wv = *reinterpret_cast<const uint4*>(&st[row * kRqPitch + cb * 32 + sub * 8]);
                uint32_t code, eb, dl = 0;
                if constexpr (!kFp6) mxfp4_pass(wv, rq.q, code, eb);
                else dfp4_pass(wv, rq.s, rq.q, code, eb, dl);
                const int m = m0 + half * 64 + row, nb = (n0 >> 5) + cb;
                if (m < p.M && nb < nb_row) {
                    const size_t blk = (size_t)(bz * p.M + m) * nb_row + nb;
                    p.g.q_codes[blk * 4 + sub] = code;
                    if (sub == 0) {
                        p.g.q_exp[blk] = (uint8_t)eb;
                        if constexpr (kFp6) p.g.q_dial[blk] = (uint8_t)dl;
                    }
                }
            }
            in_order();
        }
        return;
    }
    constexpr int kEsz = BF16 ? 2 : 4;
    // native products, split K: the fp32 partial tile of this range goes to part[blockIdx.z] (the kernel is then the fp32 one)
    const bool partial = MODE == kPlain && p.ksplit > 1;
    const int64_t ld = partial ? p.N : p.ldc;
    uint8_t* base = partial ? reinterpret_cast<uint8_t*>(p.part + (int64_t)blockIdx.z * p.M * p.N)
                            : static_cast<uint8_t*>(p.out);
    if constexpr (MODE != kPlain) base += bz * p.g.strideC * kEsz;
    uint8_t* wave_out = base + ((int64_t)m0 * ld + n0) * kEsz;                                 // uniform
    const int64_t row_bytes = ld * kEsz;                                                       // uniform
    const bool full = m0 + kRowsWave <= p.M && n0 + 128 <= p.N;                                // uniform
    // Results go through the wave's part of LDS, a group (16 rows x 64 columns) at a time, so that neighbouring lanes store neighbouring
    // columns.  (As the lanes hold them, 16 bytes of 16 rows to 16 neighbouring lanes, each lane's bytes were a write of their own: 7.5 us of fp32
    // and 3.8 of bf16 per tile of 256 x 256 instead of 5.6 and 2.4.  All compute units together store at the rate of their L2 caches, 11 TB/s;
    // bf16 before, by integer arithmetic and two columns a lane, 4.5.)
    typedef uint32_t v16u __attribute__((ext_vector_type(16)));
    constexpr int kPitch = BF16 ? 36 : 68;                                                         // dwords of a row in LDS
    uint32_t* st = reinterpret_cast<uint32_t*>(s_stage) + wave * (16 * kPitch);
    auto stage_group = [&](int (&v)[16]) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if constexpr (BF16)
                *reinterpret_cast<uint2*>(st + c * kPitch + 8 * j + 2 * q) = make_uint2(bf16_pair(v[4 * j], v[4 * j + 1]), bf16_pair(v[4 * j + 2], v[4 * j + 3]));
            else
                *reinterpret_cast<int4*>(st + c * kPitch + 16 * j + 4 * q) = make_int4(v[4 * j], v[4 * j + 1], v[4 * j + 2], v[4 * j + 3]);
        }
        in_order();
    };
    // A lane reads and stores 16 bytes of each of kRows rows, every row by kLanes lanes.  Rows may begin anywhere, memory takes 16
    // bytes at any address (with one element a lane where rows were no multiple of 16 bytes 4992 x 4864 x 32 in bf16 into rows
    // of 4867 took 23.1 us, so 16.6).  A group is stored while the next is on its way through LDS (two and four groups at once: 1 and
    // 3 % slower in fp32).
    constexpr int kElems = 16 / kEsz, kLanes = 64 / kElems, kBy = 64 / kLanes, kRows = 16 / kBy;
    auto store_all = [&](auto full_c, auto cut_c) {
        constexpr bool kFull = decltype(full_c)::value;      // no edge
        constexpr bool kCut = decltype(cut_c)::value;        // the last column lies inside a lane's 16 bytes
        const int lr = lane / kLanes, lc = lane % kLanes * kElems;
        const int64_t lane_off = lr * row_bytes + lc * kEsz;
        auto read_lines = [&] {
            v16u x = {};
#pragma unroll
            for (int k = 0; k < kRows; ++k) {
                const uint4 y = *reinterpret_cast<const uint4*>(reinterpret_cast<const uint8_t*>(st + (k * kBy + lr) * kPitch) + lc * kEsz);
                x[4 * k] = y.x;
                x[4 * k + 1] = y.y;
                x[4 * k + 2] = y.z;
                x[4 * k + 3] = y.w;
            }
            in_order();
            return x;
        };
        auto store_lines = [&](int g, v16u x) {
            const int m = m0 + (g >> 1) * 16, left = p.N - (n0 + (g & 1) * 64 + lc);              // columns from the lane's first on
            uint8_t* out = wave_out + (int64_t)((g >> 1) * 16) * row_bytes + (g & 1) * 64 * kEsz;
            if (!kFull && left <= 0) return;
            auto store_rows = [&](auto all_c) {
                auto put = [&](int64_t at, auto bytes_c) {   // so many bytes of every row
#pragma unroll
                    for (int k = 0; k < kRows; ++k) {
                        if (!decltype(all_c)::value && m + k * kBy + lr >= p.M) continue;
                        const uint32_t v[4] = {x[4 * k], x[4 * k + 1], x[4 * k + 2], x[4 * k + 3]};
                        __builtin_memcpy(out + (int64_t)(k * kBy) * row_bytes + at, v, decltype(bytes_c)::value);
                    }
                };
                if (!kCut || left >= kElems) {
                    put(lane_off, std::integral_constant<int, 16>{});
                    return;
                }
                const int bytes = left * kEsz;               // the last columns: 8 bytes, 4, 2 (by scalar branches on N no faster; 4 bytes a lane for all slower)
                int64_t at = lane_off;
                if (bytes & 8) {
                    put(at, std::integral_constant<int, 8>{});
                    at += 8;
#pragma unroll
                    for (int k = 0; k < kRows; ++k) x[4 * k] = x[4 * k + 2], x[4 * k + 1] = x[4 * k + 3];
                }
                if (bytes & 4) {
                    put(at, std::integral_constant<int, 4>{});
                    at += 4;
#pragma unroll
                    for (int k = 0; k < kRows; ++k) x[4 * k] = x[4 * k + 1];
                }
                if (bytes & 2) put(at, std::integral_constant<int, 2>{});
            };
            if (kFull || m + 16 <= p.M) store_rows(std::true_type{});        // (a branch before every store: 3 us of fp32 a tile)
            else store_rows(std::false_type{});
        };
        v16u line = {};
#define DFP4_NATIVE_STORE(G)                                                                        \
        {                                                                                           \
            int v[16];                                                                              \
            DFP4_NATIVE_READ(G, v);                                                                 \
            finish(std::integral_constant<int, G>{}, v);                                            \
            stage_group(v);                                                                         \
            const v16u next = read_lines();                                                         \
            if constexpr (G > 0) store_lines(G - 1, line);                                          \
            line = next;                                                                            \
        }
        DFP4_NATIVE_TILES(DFP4_NATIVE_STORE)
#undef DFP4_NATIVE_STORE
        store_lines(4 * TA - 1, line);
    };
    if (full) store_all(std::true_type{}, std::false_type{});
    else if (n0 + 128 <= p.N || p.N % kElems == 0) store_all(std::false_type{}, std::false_type{});
    else store_all(std::false_type{}, std::true_type{});
#undef DFP4_NATIVE_TILES
#undef DFP4_NATIVE_READ
}

// Few rows of A (decode shapes, M <= 64, MT tiles of 32): 32 W rows per workgroup, its 16 waves share K (wave w
// takes a contiguous range of steps), one or two MFMAs per step; the 16 partial tiles are added in
// a fixed order through LDS.  No vector-ALU work: both operands arrive packed.
// Bound by the latency of the packed weights' stream.  STEPS: steps whose loads are on their way at once, 2 for FP6 operands where a wave
// has four or more (K > 3072), with registers for two workgroups per compute unit where MT is 1.  Microseconds over rotating
// weights, with one step at a time in registers for two tiles of A whatever M / so:
//   FP6  16 x 14336 x 4096  15.3 / 12.4    64 x 14336 x 4096  19.0 / 17.0    FP4  16 x 14336 x 4096  10.7 / 10.1
//        16 x  4096 x 4096   7.9 /  7.0     8 x 4096 x 14336  19.1 / 17.9         16 x  4096 x 4096   6.0 /  5.4
// Three and four steps at once: 15.3 and 13.8 us for the first (one workgroup per compute unit).  Two steps of FP4: 64 x 14336 x 4096
// 12.8 instead of 11.9; of FP6 with three steps to a wave, 48 x 1024 x 2080, 5.2 instead of 4.6.
template <int FMT, bool BF16, int MT, int STEPS>
__global__ __launch_bounds__(1024, MT == 1 ? 8 : 4) void gemm_native_small_kernel(NativeParams p) {
    constexpr bool kFp6 = FMT == kFmtFp6;
    __shared__ float s_red[8][MT][16][64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kh = lane >> 5, c = lane & 31;
    const int S = p.S, t = blockIdx.x;
    const int per = (S + 15) / 16, s_lo = wave * per, s_hi = min(S, s_lo + per);
    struct Operand { uint4 lo; uint2 hi; uint32_t sc; };
    auto load = [&](const PackedOperand& src, int tile, int s) {
        Operand o;
        o.lo = *reinterpret_cast<const uint4*>(src.bits + (kFp6 ? fp6_lo(tile, s, S) : ((size_t)tile * S + s) * 1024) + lane * 16);
        if constexpr (kFp6) o.hi = *reinterpret_cast<const uint2*>(src.bits + fp6_hi(tile, s, S) + fp6_hi_lane(lane) * 8);
        o.sc = src.sc[((int64_t)(tile >> 2) * S + s) * 64 + lane];
        return o;
    };
    auto bits = [&](const Operand& o) {
        v8i v = {(int)o.lo.x, (int)o.lo.y, (int)o.lo.z, (int)o.lo.w, 0, 0, 0, 0};
        if constexpr (kFp6) {
            v[4] = (int)o.hi.x;
            v[5] = (int)o.hi.y;
        }
        return v;
    };
    v16f acc[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int x = 0; x < 16; ++x) acc[i][x] = 0.0f;
    for (int s = s_lo; s < s_hi; s += STEPS) {
        Operand w[STEPS], a[STEPS][MT];
#pragma unroll
        for (int q = 0; q < STEPS; ++q) {
            const int sq = min(s + q, s_hi - 1);                       // (no branch around a load)
            w[q] = load(p.w, t, sq);
#pragma unroll
            for (int i = 0; i < MT; ++i) a[q][i] = load(p.a, i, sq);
        }
        __builtin_amdgcn_sched_barrier(0);                             // all loads before the first wait
#pragma unroll
        for (int q = 0; q < STEPS; ++q) {
            if (s + q >= s_hi) break;
#pragma unroll
            for (int i = 0; i < MT; ++i)
                acc[i] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(bits(a[q][i]), bits(w[q]), acc[i], FMT, FMT, 0, (int)(a[q][i].sc >> (8 * i)),
                                                                         0, (int)(w[q].sc >> (8 * (t & 3))));
        }
    }
    // the 16 partial tiles, added in a fixed order: waves 8..15 hand theirs to waves 0..7
    if (wave >= 8) {
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int x = 0; x < 16; ++x) s_red[wave - 8][i][x][lane] = acc[i][x];
    }
    __syncthreads();
    if (wave < 8) {
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int x = 0; x < 16; ++x) s_red[wave][i][x][lane] += acc[i][x];
    }
    __syncthreads();
    const int n = t * 32 + c;
    #pragma unroll
    for (int i = 0; i < MT; ++i) {
        const int x = wave;                                    // thread (x, lane) finishes one output per row tile
        float sum = 0.0f;
#pragma unroll
        for (int w8 = 0; w8 < 8; ++w8) sum += s_red[w8][i][x][lane];
        const int m = i * 32 + 8 * (x >> 2) + 4 * kh + (x & 3);
        if (m < p.M && n < p.N) {
            const int64_t o = (int64_t)m * p.ldc + n;
            if constexpr (BF16) static_cast<uint16_t*>(p.out)[o] = f32_to_bf16_rne(sum);
            else static_cast<float*>(p.out)[o] = sum;
        }
    }
}

// Split K: out = sum of the ranges' fp32 partial tiles, added in range order, converted once.
template <bool BF16>
__global__ __launch_bounds__(256) void native_reduce_kernel(const float* __restrict__ part, void* out, int M, int N,
                                                            int64_t ldc, int ksplit) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x, total = (int64_t)M * N;
    if (i >= total) return;
    float s = part[i];
    for (int z = 1; z < ksplit; ++z) s += part[(int64_t)z * total + i];
    const int64_t m = i / N, o = m * ldc + (i - m * N);
    if constexpr (BF16) static_cast<uint16_t*>(out)[o] = f32_to_bf16_rne(s);
    else static_cast<float*>(out)[o] = s;
}

inline int64_t up256(int64_t x) { return (x + 255) & ~(int64_t)255; }
// Workgroups per output tile.  With at most a quarter as many tiles as compute units K can be split in 2 or 4 ranges of at
// least 8 steps; it is where the steps saved cost more than the partial tiles and the kernel that adds them, which depends
// on the format (FP6 has the longer steps) and on the type of the results (a whole product's fp32 results take longer to
// leave).  Where N is a multiple of 2048, eight columns of tiles, that kernel's workgroups run on the XCD whose cache holds
// their partial tiles, until these are too large for the caches.  The constants (us a step, us, us per MB) choose best over
// 950 drawn sizes, both formats and types, each measured whole and in every number of ranges: 0.23 % slower than the best
// choice in the mean, one in fifty by more than 5 % (up to 17); with one 0.15 us a step for both, 3 us and 0.45 us per MB
// 0.51 %, one in 23.  Whole / 2 / 4 ranges (fp32):
//   FP6  256 x 1024 x 4096  15.8 / 13.0 / 11.6     1024 x 1216 x 6176  25.4 / 22.2 / 23.5   65 x 4096 x 2560  11.9 / 11.1 / 10.0
//        512 x 4096 x 4096  17.4 / 20.4 / 22.8     512 x 4096 x 14336  46.7 / 36.1 / 33.9
//   FP4  256 x 1024 x 4096  13.3 / 11.5 / 10.5     5920 x 117 x 4736   15.4 / 16.5 / 17.3     195 x 15369 x 13568  38.6 / 46.6
//        512 x 4096 x 4096  14.6 / 17.8 / 22.0     512 x 4096 x 14336  37.6 / 31.5 / 30.2
inline int native_ksplit(int64_t M, int64_t N, int64_t KB, bool fp6, bool bf16, int64_t cu) {
    const int64_t tiles = ((M + 255) / 256) * ((N + 255) / 256), S = (KB + 1) / 2;
    const float steps = (fp6 ? 0.18f : 0.14f) * (float)S;
    int best = 1;
    float least = steps + (bf16 ? 0.0f : 0.5f);
    for (int s = 2; s <= 4 && tiles * s * 2 <= cu && S / s >= 8; s *= 2) {
        const float mb = 4e-6f * (float)s * (float)M * (float)N, per_mb = N % 2048 == 0 ? fminf(0.44f, 0.15f + 0.016f * mb) : 0.5f;
        const float us = steps / (float)s + 3.5f + per_mb * mb;
        if (us < least) least = us, best = s;
    }
    return best;
}
inline int64_t native_part_bytes(int64_t M, int64_t N, int ksplit) { return ksplit > 1 ? up256((int64_t)ksplit * M * N * 4) : 0; }
// Workgroups go to the 8 XCDs in turn, and each XCD has a cache of its own.  Where all tiles run at once the tiles of an XCD
// form a rectangle rather than every eighth column: of those that divide the grid in eight, the one that reads the fewest
// rows.  2048 x 4096 x 14336 (FP6, 128-row tiles) reads 200 MB from beyond the XCDs' caches instead of 246: 60.7 -> 60.4 us
// with operands in the last cache, 77.5 -> 75.4 with weights from memory; 2048 x 4096 x 4096 27.3 -> 26.9 (FP4 21.4 -> 19.6),
// 4096 x 4096 x 4096 34.9 -> 33.6 and 37.4 -> 36.5.  Only for a power of two of columns, which makes the mapping shifts and masks
// (other factors have not been tried), and for one round of tiles: in more an XCD's share of a round is no rectangle.
// Not for native products with K split, whose partial tiles cost more where their column does not name their XCD
// (native_ksplit; rectangles / columns: 128 x 4096 x 4096 FP6 in 4 ranges 14.8 / 11.8, 256 x 4096 x 4096 FP4 in 4 19.4 / 13.4,
// 512 x 4096 x 14336 the same); exact ones, which keep a tile's sums together, gain (2048 x 2048 x 8192 33.3 / 34.2,
// 1024 x 2048 x 14336 40.4 / 41.4) or do not care.
inline void choose_rect(NativeParams& p, dim3 grid, int tile_rows) {
    const int64_t gx = grid.x, gy = grid.y;
    p.rect_w = p.rects_x = p.rect_h = 0;
    if (gx * gy % 8 != 0 || gx * gy * grid.z > device_cu_count()) return;
    int64_t least = 0;
    for (int x = 0; x <= 3; ++x)                             // 2^x rectangles side by side, 8 / 2^x one above the other
        for (int w = 0; w < 8; ++w) {
            if (gx != (int64_t)1 << (w + x) || gy % (8 >> x) != 0) continue;
            const int64_t h = gy / (8 >> x), rows = ((int64_t)256 << w) + h * tile_rows;
            if (p.rect_h && rows >= least) continue;
            p.rect_w = w;
            p.rects_x = x;
            p.rect_h = (int)h;
            least = rows;
        }
}
// One packed operand: [bits | scales], rows padded to 256, eight steps of slack behind each array.
struct OperandLayout { int64_t sc, total; };
inline OperandLayout operand_layout(int64_t rows, int64_t KB, bool fp6) {
    const int64_t S = (KB + 1) / 2, tiles = (rows + 255) / 256 * 8;
    OperandLayout l{};
    l.sc = up256(fp6 ? (tiles / 2 * S + kSlackSteps) * kFp6PairBytes : (tiles * S + kSlackSteps) * 1024);
    l.total = up256(l.sc + ((tiles / 4) * S + kSlackSteps) * 256);
    return l;
}

}  // namespace

size_t native_packed_bytes(int64_t rows, int64_t K, bool fp6) {
    if (rows == 0 || K == 0) return 0;
    return (size_t)operand_layout(rows, K / kBlock, fp6).total;
}

size_t native_scale_offset(int64_t rows, int64_t K, bool fp6) {
    return (size_t)operand_layout(rows, K / kBlock, fp6).sc;
}

// enough for either format and type of the results
size_t native_splitk_bytes(int64_t M, int64_t N, int64_t K) {
    if (M == 0 || N == 0) return 0;
    const int64_t cu = device_cu_count();
    int most = 1;
    for (int form = 0; form < 4; ++form) {
        const int s = native_ksplit(M, N, K / kBlock, (form & 1) != 0, (form & 2) != 0, cu);
        if (s > most) most = s;
    }
    return (size_t)native_part_bytes(M, N, most);
}

size_t gemm_native_workspace_bytes(int64_t M, int64_t N, int64_t K, bool fp6) {
    return native_packed_bytes(M, K, fp6) + native_packed_bytes(N, K, fp6) + native_splitk_bytes(M, N, K);
}

// Rewrite a quantized tensor in the matrix instruction's register order (see the file header).
int launch_native_pack(bool fp6, dfp4_tensor T, void* packed, size_t bytes, hipStream_t stream) {
    const int64_t KB = T.K / kBlock;
    if (T.rows == 0 || KB == 0) return DFP4_OK;
    if (T.rows >= (1 << 30) || KB >= (1 << 20)) return DFP4_ERR_SHAPE;
    const OperandLayout lay = operand_layout(T.rows, KB, fp6);
    if ((size_t)lay.total > bytes) return DFP4_ERR_WORKSPACE;
    const int S = (int)((KB + 1) / 2);
    PackParams q{};
    q.codes = T.codes; q.dial = T.dialect; q.expo = T.exponent;
    q.dst = PackedOperand{static_cast<uint8_t*>(packed), reinterpret_cast<uint32_t*>(static_cast<uint8_t*>(packed) + lay.sc)};
    q.rows = (int)T.rows; q.KB = (int)KB; q.S = S;
    dim3 gp((unsigned)((S + 3) / 4), (unsigned)((T.rows + 255) / 256 * 8));
    if (gp.y > 65535) return DFP4_ERR_SHAPE;
    if (fp6) hipLaunchKernelGGL((native_pack_kernel<kFmtFp6>), gp, dim3(256), 0, stream, q);
    else hipLaunchKernelGGL((native_pack_kernel<kFmtFp4>), gp, dim3(256), 0, stream, q);
    return check_launch();
}

// out = A * W^T from two packed operands ([M, K] and [N, K] before packing)
// `splitk` (may be null): native_splitk_bytes(M, N, K) bytes; without it K is never split
int launch_gemm_native_packed(bool fp6, const void* a_packed, const void* w_packed, int64_t M, int64_t N, int64_t K,
                              void* out, int out_dtype, int64_t ldc, void* splitk, size_t splitk_bytes,
                              hipStream_t stream) {
    const int64_t KB = K / kBlock;
    if (M == 0 || N == 0) return DFP4_OK;
    if (M >= (1 << 30) || N >= (1 << 30) || KB >= (1 << 20) || KB == 0 || ldc >= (1 << 27)) return DFP4_ERR_SHAPE;
    NativeParams p{};
    uint8_t* ap = static_cast<uint8_t*>(const_cast<void*>(a_packed));
    uint8_t* wp = static_cast<uint8_t*>(const_cast<void*>(w_packed));
    p.a = PackedOperand{ap, reinterpret_cast<uint32_t*>(ap + operand_layout(M, KB, fp6).sc)};
    p.w = PackedOperand{wp, reinterpret_cast<uint32_t*>(wp + operand_layout(N, KB, fp6).sc)};
    p.out = out; p.M = (int)M; p.N = (int)N; p.S = (int)((KB + 1) / 2); p.ldc = ldc;
    if (M <= 64) {
        // decode shapes: one workgroup per 32 W rows (A occupies the first one or two row tiles of its layout)
        p.ksplit = 1;
        dim3 gs((unsigned)((N + 31) / 32));
        dispatch_mx_bf16(!fp6, out_dtype == DFP4_BF16, [&](auto mxc, auto bc) {
            constexpr int kFmt = decltype(mxc)::value ? kFmtFp4 : kFmtFp6, kSteps = decltype(mxc)::value ? 1 : 2;
            constexpr bool kBf16 = decltype(bc)::value;
            const bool few = p.S <= 48;                                // at most three steps to a wave
            if (M <= 32 && few) hipLaunchKernelGGL((gemm_native_small_kernel<kFmt, kBf16, 1, 1>), gs, dim3(1024), 0, stream, p);
            else if (M <= 32) hipLaunchKernelGGL((gemm_native_small_kernel<kFmt, kBf16, 1, kSteps>), gs, dim3(1024), 0, stream, p);
            else if (few) hipLaunchKernelGGL((gemm_native_small_kernel<kFmt, kBf16, 2, 1>), gs, dim3(1024), 0, stream, p);
            else hipLaunchKernelGGL((gemm_native_small_kernel<kFmt, kBf16, 2, kSteps>), gs, dim3(1024), 0, stream, p);
        });
        return check_launch();
    }
    const int64_t cu = device_cu_count();
    p.ksplit = native_ksplit(M, N, KB, fp6, out_dtype == DFP4_BF16, cu);
    if (p.ksplit > 1 && (!splitk || (int64_t)splitk_bytes < native_part_bytes(M, N, p.ksplit))) p.ksplit = 1;
    p.part = static_cast<float*>(splitk);
    // 256-row workgroups unless they would leave half of the compute units idle, or there are no more than 128 rows (128 x 4096 x 2048
    // 13.2 us with 256-row workgroups, 9.8 so)
    const int64_t tiles256 = ((M + 255) / 256) * ((N + 255) / 256);
    const bool half = tiles256 * p.ksplit * 2 <= cu || M <= 128;
    dim3 grid((unsigned)((N + 255) / 256), (unsigned)((M + (half ? 127 : 255)) / (half ? 128 : 256)), (unsigned)p.ksplit);
    if (grid.y > 65535) return DFP4_ERR_SHAPE;
    if (p.ksplit == 1) choose_rect(p, grid, half ? 128 : 256);
    const bool bf16 = out_dtype == DFP4_BF16 && p.ksplit == 1;     // partial tiles are fp32
#define DFP4_NATIVE_LAUNCH(F, B)                                                                         \
    do {                                                                                                 \
        if (half) hipLaunchKernelGGL((gemm_native_kernel<F, B, 2, kPlain>), grid, dim3(256), 0, stream, p);      \
        else hipLaunchKernelGGL((gemm_native_kernel<F, B, 4, kPlain>), grid, dim3(256), 0, stream, p);           \
    } while (0)
    if (fp6) {
        if (bf16) DFP4_NATIVE_LAUNCH(kFmtFp6, true); else DFP4_NATIVE_LAUNCH(kFmtFp6, false);
    } else {
        if (bf16) DFP4_NATIVE_LAUNCH(kFmtFp4, true); else DFP4_NATIVE_LAUNCH(kFmtFp4, false);
    }
#undef DFP4_NATIVE_LAUNCH
    if (p.ksplit > 1) {
        const unsigned gr = (unsigned)((M * N + 255) / 256);
        if (out_dtype == DFP4_BF16)
            hipLaunchKernelGGL((native_reduce_kernel<true>), dim3(gr), dim3(256), 0, stream, p.part, out, p.M, p.N, ldc, p.ksplit);
        else
            hipLaunchKernelGGL((native_reduce_kernel<false>), dim3(gr), dim3(256), 0, stream, p.part, out, p.M, p.N, ldc, p.ksplit);
    }
    return check_launch();
}

// ---- exact products
namespace {

// A prepared operand: [counters (A only) | bits | scales | norms | references | class masks]; rows padded to 256
struct ExactLayout { int64_t bits, sc, stat, ref, mask, total; };
inline ExactLayout exact_layout(int64_t rows, int64_t KB, bool fp6, bool counters) {
    const OperandLayout o = operand_layout(rows, KB, fp6);
    ExactLayout l{};
    l.bits = counters ? up256((kExactCounters) * 4) : 0;
    l.sc = l.bits + o.sc;
    l.stat = l.bits + o.total;
    l.ref = l.stat + (rows + 255) / 256 * 8 * kStatChunks * (int64_t)sizeof(ExactStat);
    l.mask = l.ref + up256(rows);
    l.total = up256(l.mask + (rows + 255) / 256 * 2 * KB);
    return l;
}

// Tile height (128 or 256 rows by 256 columns) and the workgroups that share a tile's K
struct ExactShape { bool half; int ksplit; };
inline ExactShape exact_shape(int64_t M, int64_t N, int64_t KB, int64_t batch, int64_t cu) {
    const int64_t S = (KB + 1) / 2, cols = (N + 255) / 256 * batch;
    const bool half = (M + 255) / 256 * cols * 2 <= cu && M > 128;
    const int64_t tiles = (M + (half ? 127 : 255)) / (half ? 128 : 256) * cols;
    int s = 1;
    while (s < 8 && tiles * s * 2 <= cu && S / (2 * s) >= 8) s *= 2;
    return {half, tiles <= kExactSplitTiles ? s : 1};
}
inline int64_t exact_part_bytes(int64_t M, int64_t N, ExactShape x, int64_t batch) {
    if (x.ksplit == 1) return 0;
    return (M + (x.half ? 127 : 255)) / (x.half ? 128 : 256) * ((N + 255) / 256) * batch * x.ksplit * (x.half ? 128 : 256) * 256 * 4;
}

}  // namespace

int64_t exact_operand_bytes(int64_t rows, int64_t KB, bool fp6, bool counters) { return exact_layout(rows, KB, fp6, counters).total; }

void set_prepared_classes(bool mx, GemmParams& p, const uint8_t* a_prep, const uint8_t* w_prep) {
    const ExactLayout la = exact_layout(p.M, p.KB, !mx, true), lw = exact_layout(p.N, p.KB, !mx, false);
    p.ref_a = a_prep + la.ref; p.mask_a = a_prep + la.mask;
    p.ref_w = w_prep + lw.ref; p.mask_w = w_prep + lw.mask;
}

int64_t exact_split_bytes(int64_t M, int64_t N, int64_t KB, int64_t batch) {
    return exact_part_bytes(M, N, exact_shape(M, N, KB, batch, device_cu_count()), batch);
}

// Packs A (p.a_prep, unless null) and W (p.w_prep, unless null) of `batch` problems; `classes` (batch 1): with what
// gemm_f8_kernel reads of prepared operands
int launch_exact_prep(bool mx, const GemmParams& p, int64_t batch, bool classes, hipStream_t stream) {
    const int64_t KB = p.KB, S = (KB + 1) / 2;
    ExactPrepParams q{};
    q.KB = p.KB;
    q.S = (int)S;
    // 8 blocks at a time: as many times as leave two workgroups for every compute unit (they read the exponents of whole rows:
    // fewer and longer chunks read less; 14336 x 4096 with 8 blocks each 36 us, so 28), at most 32 chunks
    const int64_t groups = ((p.a_prep ? (p.M + 255) / 256 * 2 : 0) + (p.w_prep ? (p.N + 255) / 256 * 2 : 0)) * batch, eights = (KB + 7) / 8;
    int64_t times = groups * eights / (2 * device_cu_count());
    if (times > kMaxChunkBlocks / 8) times = kMaxChunkBlocks / 8;
    if (times < (eights + kStatChunks - 1) / kStatChunks) times = (eights + kStatChunks - 1) / kStatChunks;
    q.chunk_blocks = (int)(8 * times);
    q.chunks = (int)((eights + times - 1) / times);
    if (q.chunks > kStatChunks) return DFP4_ERR_SHAPE;
    int64_t wgs = 0;
    if (p.a_prep) {
        const ExactLayout l = exact_layout(p.M, KB, !mx, true);
        q.a = ExactOperand{p.a_codes, mx ? nullptr : p.a_dial, p.a_exp, p.strideA_rows, p.a_prep + l.bits, l.sc - l.bits, l.stat - l.bits,
                           p.a_prep_stride, classes ? p.a_prep + l.ref : nullptr, classes ? p.a_prep + l.mask : nullptr, p.M, (p.M + 255) / 256 * 2};
        q.count = reinterpret_cast<uint32_t*>(p.a_prep);
        q.count_stride = p.a_prep_stride / 4;
        q.counters = kExactCounters;
        wgs = (int64_t)q.a.groups * q.chunks;
        q.wgs_a = (int)wgs;
    }
    if (p.w_prep) {
        const ExactLayout l = exact_layout(p.N, KB, !mx, false);
        q.w = ExactOperand{p.w_codes, mx ? nullptr : p.w_dial, p.w_exp, p.strideW_rows, p.w_prep, l.sc, l.stat,
                           p.w_prep_stride, classes ? p.w_prep + l.ref : nullptr, classes ? p.w_prep + l.mask : nullptr, p.N, (p.N + 255) / 256 * 2};
        wgs += (int64_t)q.w.groups * q.chunks;
    }
    if (wgs == 0) return DFP4_OK;
    if (wgs > 0x7fffffff || batch > 65535) return DFP4_ERR_SHAPE;
    dim3 g((unsigned)wgs, 1, (unsigned)batch);
    if (mx) hipLaunchKernelGGL((exact_prep_kernel<kFmtFp4>), g, dim3(1024), 0, stream, q);
    else hipLaunchKernelGGL((exact_prep_kernel<kFmtFp6>), g, dim3(1024), 0, stream, q);
    return check_launch();
}

// The product of prepared operands (p.a_prep, p.w_prep); `part`: room for the partial tiles where K is split
int launch_exact(bool mx, bool bf16, const GemmParams& g, int64_t batch, float* part, size_t part_bytes, bool rq, hipStream_t stream) {
    const int64_t KB = g.KB;
    ExactShape x = exact_shape(g.M, g.N, KB, batch, device_cu_count());
    if (x.ksplit > 1 && (!part || (size_t)exact_part_bytes(g.M, g.N, x, batch) > part_bytes)) x.ksplit = 1;      // no room: no split
    const ExactLayout la = exact_layout(g.M, KB, !mx, true), lw = exact_layout(g.N, KB, !mx, false);
    ExactParams p{};
    p.a = PackedOperand{g.a_prep + la.bits, reinterpret_cast<uint32_t*>(g.a_prep + la.sc)};
    p.w = PackedOperand{g.w_prep, reinterpret_cast<uint32_t*>(g.w_prep + lw.sc)};
    p.out = g.out; p.M = g.M; p.N = g.N; p.S = (int)((KB + 1) / 2); p.ldc = g.ldc;
    p.ksplit = x.ksplit;
    p.part = part;
    p.g = g;
    p.a_stat = reinterpret_cast<const ExactStat*>(g.a_prep + la.stat);
    p.w_stat = reinterpret_cast<const ExactStat*>(g.w_prep + lw.stat);
    p.a_stride = g.a_prep_stride; p.w_stride = g.w_prep_stride;
    p.cnt = reinterpret_cast<uint32_t*>(g.a_prep);
    p.cnt_stride = g.a_prep_stride / 4;
    dim3 grid((unsigned)((g.N + 255) / 256), (unsigned)((g.M + (x.half ? 127 : 255)) / (x.half ? 128 : 256)), (unsigned)(batch * x.ksplit));
    if (grid.y > 65535 || batch * x.ksplit > 65535) return DFP4_ERR_SHAPE;
    choose_rect(p, grid, x.half ? 128 : 256);
    dispatch_mx_bf16(mx, bf16, [&](auto mxc, auto bc) {
        constexpr int kFmt = decltype(mxc)::value ? kFmtFp4 : kFmtFp6;
        constexpr bool kBf16 = decltype(bc)::value;
        auto run = [&](auto ta_c, auto mode_c) {
            hipLaunchKernelGGL((gemm_native_kernel<kFmt, kBf16, decltype(ta_c)::value, decltype(mode_c)::value>), grid, dim3(256), 0, stream, p);
        };
        using Ta2 = std::integral_constant<int, 2>;
        using Ta4 = std::integral_constant<int, 4>;
        if constexpr (kBf16) {
            if (rq) {
                if (x.half) run(Ta2{}, std::integral_constant<int, kRequant>{});
                else run(Ta4{}, std::integral_constant<int, kRequant>{});
                return;
            }
        }
        if (x.half) run(Ta2{}, std::integral_constant<int, kExact>{});
        else run(Ta4{}, std::integral_constant<int, kExact>{});
    });
    return check_launch();
}

}  // namespace dfp4
