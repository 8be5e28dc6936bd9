// Block-scaled integer GEMM on DialectFP4 / MXFP4 operands for gfx950
// (paper Section 3.3): out = A * W^T with
//   out[m,n] = sum_kb 2^(ea[m,kb]+ew[n,kb]-2) * sum_{k in kb} (+-ua)(+-uw).
//
// The paper accumulates the products of one block pair as integers and
// applies the exponent sum once per block pair.  On gfx950 the per-block
// floating-point step would dominate (one convert + scale + add per output
// and block on the vector ALU against 32 int8 MACs per output and block on
// the matrix core), so this kernel moves the exponents into the operands:
//
//   * every row of A and of W gets a reference exponent ref = its smallest
//     block exponent; block (row, kb) has offset delta = e - ref >= 0;
//   * delta = 4 c + d.  The shift d in 0..3 is folded into the int8 operand
//     (|u| <= 15, so |u << d| <= 120); the "class" c selects a pass;
//   * passes run from the highest class down, and between classes the int32
//     accumulators are shifted left by 4 (Horner's scheme), so that all of K
//     is summed exactly in ONE int32 accumulator per output and the only
//     rounding is the final int32 -> fp32 conversion, scaled by
//     2^(refA[m] + refW[n] - 2).
//   Both operands have classes.  A block is visited once for every pair (class
//   present among the tile's 512 rows of A, class present among its 128 rows of
//   W) -- rows of other classes contribute zeros -- and the pair's class sum is
//   the number of shifts the product still receives; sums above 2 cannot be
//   taken.  With activations that have outlier channels, that is a second visit
//   for the few outlier blocks.
//
// Kernels:
//   gemm_prep_kernel     the per-operand part, once per call (dfp4_gemm) or once per
//                        tensor (dfp4_gemm_prepare).  A: per-row reference exponents,
//                        per-(512 rows, block) class masks, and A expanded to
//                        pre-shifted int8 in MFMA fragment order (A is the small
//                        operand; W stays 4-bit in HBM).  W: per-row reference
//                        exponents, per-(128 rows, block) class masks, and per class
//                        and block one dword naming the block's (dialect, shift)
//                        table, or the all-zero table for blocks of another class;
//   gemm_fast_kernel     512 x 128 outputs per workgroup, 4 waves, each wave
//                        128 x 128 with 256 accumulator registers (one wave per
//                        SIMD).  A fragments are private to a wave and come by
//                        global loads straight into registers, two steps ahead;
//                        each wave expands its own 32 rows of W from 4-bit codes
//                        (v_perm_b32 lookups) and shares the int8 result through
//                        LDS.  A lone wave issues one instruction per 4 cycles or
//                        so; the whole main loop is generated assembly that places
//                        the few non-MFMA instructions per MFMA in its shadow.
//                        With few output tiles K is split between workgroups; the
//                        last of a tile's workgroups to finish adds the others'
//                        exact int32 sums.  A tile whose exponents spread too far
//                        (or whose int32 sum could overflow) is computed by the same
//                        workgroup with one fp32 scale-and-add per block;
//   gemm_direct_kernel   (gemm_direct.hip) the same exact scheme with both operands expanded inside the
//                        kernel, in tiles from 32 x 32 to 256 x 128: few rows, few tiles, long K, batches
//                        whose expanded A would be read only once;
//   gemm_block16_kernel  operands quantized in blocks of 16: per-block fp32 flush.
//
// The order of the elements inside an MFMA operand does not matter as long
// as A and W use the same order; both sides go through unpack8() below.
#include <type_traits>
#include "common.h"
#include "formatbook.h"
#include "quant_pass.h"
#include "gemm_common.h"
#include "gemm_step_asm.inc"

namespace dfp4 {

namespace {

constexpr int kTileM = 512, kTileN = 128;   // fast kernel: outputs per workgroup
constexpr int kGroups = kTileM / 32;        // 32-row groups per tile
constexpr int kMaxKB = 512;           // fast path: K <= 16384
constexpr int kBBufBytes = 8 * 1024;  // int8 W operands of one step: 4 column tiles x 2 x 1 KiB
constexpr int kRqPitch = 136;         // bf16 per staged output row (128 + 8: rows stay 16-byte aligned)
constexpr int kVisitPad = 12;         // padding visits after the last one (the loop looks 5 steps ahead)
constexpr int kClassPairs = (kMaxClass + 1) * (kMaxClass + 2) / 2;   // (class of A, class of W) with sum <= kMaxClass
constexpr int kVisitCap = kClassPairs * kMaxKB + 2 * (kMaxClass + 1) + kVisitPad + 4;
constexpr int kMaxSplitTiles = 2048;  // arrival counters per prepared A: K is split only below this many tiles

__host__ __device__ inline int64_t align256(int64_t x) { return (x + 255) & ~(int64_t)255; }

// Prepared A [M, K] (see gemm_prep_kernel): per-row reference exponents (rows padded to 512), one
// class mask per (512-row tile, block), arrival counters of the tiles whose K is split, and the
// operand expanded to pre-shifted int8 in MFMA fragment order:
// [class][tile][32-row group][block 0..KB][1 KiB]; block KB of class 0 is all zeros.
struct PrepALayout { int64_t off_refa, off_mask, off_cnt, off_a8, total; };
inline PrepALayout prep_a_layout(int64_t M, int64_t KB) {
    const int64_t tm = (M + kTileM - 1) / kTileM;
    PrepALayout l{};
    l.off_refa = 0;
    l.off_mask = align256(tm * kTileM);
    l.off_cnt = align256(l.off_mask + tm * KB);
    l.off_a8 = align256(l.off_cnt + (int64_t)(kMaxSplitTiles + 1) * 4);    // + the count of declined tiles
    l.total = align256(l.off_a8 + (kMaxClass + 1) * tm * kGroups * (KB + 1) * 1024);
    return l;
}
// Prepared W [N, K]: per-row reference exponents (rows padded to 128), one class mask per
// (128-row tile, block), per class and block one dword naming the block's (dialect, shift)
// table -- or the all-zero table where the block is of another class -- and a copy of the 4-bit
// codes.  Table dwords and codes are laid out by 32-row group and block, [group][block][row]
// (codes: 16 bytes per row and block; dwords: [class][group][block][row]), so that what a wave
// loads for one block of its 32 rows is one contiguous run of 512 (128) bytes: four (one) cache
// lines instead of 32.  Rows of the last group beyond N carry the all-zero table.
struct PrepWLayout { int64_t off_refw, off_wmask, off_wmeta, off_wcodes, total; };
inline PrepWLayout prep_w_layout(int64_t N, int64_t KB) {
    const int64_t tn = (N + kTileN - 1) / kTileN, rows = tn * kTileN;
    PrepWLayout l{};
    l.off_refw = 0;
    l.off_wmask = align256(rows);
    l.off_wmeta = align256(l.off_wmask + tn * KB);
    l.off_wcodes = align256(l.off_wmeta + (kMaxClass + 1) * rows * KB * 4);
    l.total = align256(l.off_wcodes + rows * KB * 16);
    return l;
}
// Workgroups per output tile: when there are fewer tiles than compute units, K is split
// between 2, 4 or 8 workgroups; the last of them to finish adds the others' exact int32 sums.
inline int choose_ksplit(int64_t tiles, int64_t KB, int64_t cu) {
    int s = 1;
    while (s < 8 && tiles * s * 2 <= cu && KB / (2 * s) >= 16) s *= 2;
    return tiles <= kMaxSplitTiles ? s : 1;
}
inline int64_t partial_bytes(int64_t M, int64_t N, int64_t KB, int64_t cu) {
    const int64_t tiles = ((M + kTileM - 1) / kTileM) * ((N + kTileN - 1) / kTileN);
    const int s = choose_ksplit(tiles, KB, cu);
    return s > 1 ? align256((int64_t)s * tiles * kTileM * kTileN * 4) : 0;
}
// Which kernel.  gemm_fast_kernel multiplies expanded operands; gemm_direct_kernel (gemm_direct.hip) expands in the
// kernel and takes everything gemm_fast_kernel cannot (few rows, K beyond its visit list), and the products it is
// estimated to finish sooner: those with few output tiles, where the large kernel's one wave per SIMD leaves most
// of the chip idle or the exchange of partial sums takes longer than the product (M x N x K = 1024 x 1024 x 4096: 108 us
// with the prepass, 20 direct; 512 x 4096 x 4096: 112 and 34; 2048 x 4096 x 4096: 75 and 67; 4096 x 4096 x 4096: 90 and
// 144; 2048 x 4096 x 14336: 171 and 262; 1024 x 14336 x 4096: 84 and 127), and batches whose expanded A would
// be read only once or twice (P V of attention).  K of one iteration of the direct kernel (Q K^T) goes there unless
// it is prepared already: an expanded A of 4 blocks costs more to fetch than to expand, and the large kernel's prologue and epilogue have
// nothing to hide behind (128 heads of 2048 x 2048 x 128: 504 and 400 us; 1 x 4096 x 4096 x 128: 31 and 22).
// Against both kernels timed on 940 products not among those fitted (M 65..4096, N 64..14336, K 160..16384) the kernel and
// shape taken are 2.7 % slower than the best on average, 10 % in 5 % of them, 14 % in 1 %; prepared (630) 1.2, 6 and 13 %.
// An A operand of fewer rows than kPreparedMinRows is not expanded ahead: direct is faster by up to 3.5 times (65 x 1024 x
// 16384), but for 200 to 256 rows and N x K of 2^26 or more, where it is up to 13 % slower (256 x 14336 x 14336).
constexpr int kPreparedMinRows = 257;
inline bool fast_kernel_can(int64_t M, int64_t KB) { return M > 64 && KB > 0 && KB <= kMaxKB; }
// Estimated microseconds of gemm_fast_kernel, fitted like those of the direct shapes: per round of workgroups a fixed
// part, and per block of a workgroup's share of K more where the chip is full, growing beyond 128 blocks; the results; the exchange of partial tiles between s workgroups; the prepass unless the operands are prepared
inline float fast_cost(int64_t M, int64_t N, int64_t KB, int64_t batch, bool prepared, int64_t cu) {
    const int64_t tiles = ((M + kTileM - 1) / kTileM) * ((N + kTileN - 1) / kTileN) * batch;
    const int s = choose_ksplit(tiles, KB, cu);
    const int64_t rounds = tiles * s / cu, rest = tiles * s - rounds * cu;
    const float steps = (float)KB / (float)s, grow = 1.0f + 0.151f * (float)(KB > 128 ? KB - 128 : 0) / 384.0f;
    float t = (float)rounds * (12.8f + steps * 0.36f * grow) + (float)M * (float)N * (float)batch * 4e-6f * (N % 16 != 0 ? 0.406f : 0.012f);
    if (rest > 0) t += 12.8f + steps * (0.284f + 0.0755f * (float)rest / (float)cu) * grow;
    if (s > 1) t += 4.5f + 10.4f * (float)(s - 1);
    if (!prepared) t += 7.7f + (0.601f * (float)M + 0.332f * (float)N) * (float)(KB * kBlock * batch) * 1e-6f;
    return t;
}
// the shape of gemm_direct_kernel that is taken, -1: gemm_fast_kernel
inline int direct_shape(int64_t M, int64_t N, int64_t KB, int64_t batch, bool prepared, int64_t cu) {
    const DirectChoice d = choose_direct(M, N, KB, batch, cu);
    const bool direct = !fast_kernel_can(M, KB) || (prepared ? M < kPreparedMinRows : KB <= kDirectOnceBlocks) ||
                        d.us <= fast_cost(M, N, KB, batch, prepared, cu);
    return direct ? d.shape : -1;
}

// ---------------------------------------------------------------------------
// Prepass (one launch, 1024 threads per workgroup).  Workgroups [0, n_a) expand A,
// the others compute the per-row statistics of W.
//
// A workgroup = (512-row tile, chunk of 8 blocks); wave w owns the tile's 32-row
// group w.  Each wave first finds its rows' reference exponents (smallest block
// exponent of the whole row; the chunk-0 workgroup publishes them), then the
// classes present in each block of the chunk among all 512 rows (one 32-bit word
// in LDS: bit 4*block + class), then writes, for every class present, the 1 KiB
// fragment of its group: rows of other classes contribute zeros.  The 4-bit codes
// are read as whole 128-byte lines (8 lanes per row) and redistributed through LDS
// to the fragment order (lane = (t, row): elements 16t .. 16t+15 of the block).
//
// W rows: reference exponent, per class and block one table offset (dword), and the classes
// present in each block among the 128 rows of a tile.
// ---------------------------------------------------------------------------
// up to 8 bytes starting at q (the first n are read), little-endian in a 64-bit word
__device__ __forceinline__ uint64_t load_bytes8(const uint8_t* q, int n) {
    if (n == 8) {
        uint64_t v;
        __builtin_memcpy(&v, q, 8);                   // no alignment assumed: the compiler picks the access
        return v;
    }
    uint64_t v = 0;
    for (int i = 0; i < n; ++i) v |= (uint64_t)q[i] << (8 * i);
    return v;
}

template <bool MX>
__global__ __launch_bounds__(1024) void gemm_prep_kernel(GemmParams p, int n_a, int chunks_a) {
    constexpr int kPitch = 144;                       // LDS bytes per row of staged codes (8 blocks = 128 + pad)
    __shared__ __attribute__((aligned(16))) uint8_t s_codes[16][32 * kPitch];
    __shared__ __attribute__((aligned(16))) uint32_t s_tab[kDialects * 16];
    __shared__ uint32_t s_present;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t bz = blockIdx.z;
    uint8_t* ap = p.a_prep + bz * p.a_prep_stride;    // only touched by the A workgroups
    uint8_t* wp = p.w_prep + bz * p.w_prep_stride;    // only touched by the W workgroups
    const int KB = p.KB;

    if ((int)blockIdx.x >= n_a) {
        // ---- W: a workgroup = (128-row tile, chunk of 64 blocks), 8 lanes per row (lane s takes blocks
        // s, s + 8, ...).  Every workgroup finds the rows' reference exponents from all of K.
        __shared__ uint32_t s_wmask[64];
        const int chunks_w = (KB + 63) / 64;
        const int tile = ((int)blockIdx.x - n_a) / chunks_w, chunk = ((int)blockIdx.x - n_a) % chunks_w;
        const int kc = chunk * 64, ke = min(KB, kc + 64);
        const int row = tile * kTileN + (tid >> 3), seg = tid & 7;
        const bool valid = row < p.N;
        const int64_t base = (bz * p.strideW_rows + min(row, p.N - 1)) * KB;
        const uint8_t* we = p.w_exp + base;
        const uint8_t* wd = MX ? nullptr : p.w_dial + base;
        if (tid < 64) s_wmask[tid] = 0;
        int mn = 255;
        for (int kb = seg; kb < KB; kb += 8) mn = min(mn, (int)we[kb]);
        mn = min(mn, __shfl_xor(mn, 1));
        mn = min(mn, __shfl_xor(mn, 2));
        mn = min(mn, __shfl_xor(mn, 4));
        __syncthreads();
        {
            if (valid && seg == 0 && chunk == 0) wp[p.off_refw + row] = (uint8_t)mn;
            // [group of 32 rows][block][row]: this row's slot within block 0 of its group
            const int64_t slot = (int64_t)(row >> 5) * KB * 32 + (row & 31);
            uint32_t* wmeta = reinterpret_cast<uint32_t*>(wp + p.off_wmeta) + slot;
            uint4* wct = reinterpret_cast<uint4*>(wp + p.off_wcodes) + slot;
            const uint4* wcs = reinterpret_cast<const uint4*>(p.w_codes) + base;
            const int64_t cls_stride = (int64_t)p.tiles_n * kTileN * KB;     // dwords
            for (int kb = kc + seg; kb < ke; kb += 8) {
                uint32_t cls = kMaxClass + 2, tab = kZeroTab;               // rows beyond N: the all-zero table
                if (valid) {
                    const uint32_t delta = (uint32_t)we[kb] - (uint32_t)mn;
                    const uint32_t dd = MX ? 7u : ((uint32_t)wd[kb] & 15u);
                    cls = min(delta >> 2, (uint32_t)kMaxClass + 1u);
                    tab = (dd * 4u + (delta & 3u)) * 16u;
                    wct[(int64_t)kb * 32] = wcs[kb];
                    atomicOr(&s_wmask[kb - kc], 1u << cls);
                }
#pragma unroll
                for (uint32_t c = 0; c <= (uint32_t)kMaxClass; ++c)
                    wmeta[c * cls_stride + (int64_t)kb * 32] = cls == c ? tab : kZeroTab;
            }
        }
        __syncthreads();
        if (tid < ke - kc) wp[p.off_wmask + (int64_t)tile * KB + kc + tid] = (uint8_t)s_wmask[tid];
        return;
    }

    // ---- A: tile, chunk of 8 blocks
    const int tile = (int)blockIdx.x / chunks_a, chunk = (int)blockIdx.x % chunks_a;
    const int kc = chunk * 8, nk = min(8, KB - kc);
    for (int i = tid; i < kDialects * 16; i += 1024) s_tab[i] = (&g_shifted_book.w[0][0][0])[i];
    if (tid == 0) s_present = 0;
    if (blockIdx.x == 0) {
        // arrival counters of output tiles whose K is split between workgroups: zero here; the
        // workgroup that arrives last at a tile puts its counter back to zero
        uint32_t* cnt = reinterpret_cast<uint32_t*>(ap + p.off_cnt);
        for (int i = tid; i <= kMaxSplitTiles; i += 1024) cnt[i] = 0;     // the last one counts declined tiles
    }
    __syncthreads();

    const int r = lane & 31, t = lane >> 5;
    const int row0 = tile * kTileM + wave * 32;
    const bool group_valid = row0 < p.M;              // wave-uniform
    int cls[8], sh[8];
    uint64_t d8 = 0x0707070707070707ull;
    if (group_valid) {
        // codes: lane (row q*8 + lane/8, block lane%8) reads one block; 8 lanes cover a 128-byte line
        uint4 craw[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int k8 = lane & 7;
            const int64_t rq = bz * p.strideA_rows + min(row0 + q * 8 + (lane >> 3), p.M - 1);
            craw[q] = k8 < nk ? *reinterpret_cast<const uint4*>(p.a_codes + (rq * KB + kc + k8) * 16)
                              : make_uint4(0, 0, 0, 0);
        }
        const int64_t arow = bz * p.strideA_rows + min(row0 + r, p.M - 1);
        const uint64_t e8 = load_bytes8(p.a_exp + arow * KB + kc, nk);
        if (!MX) d8 = load_bytes8(p.a_dial + arow * KB + kc, nk);
        // reference exponent of the row: lane (t, r) scans every other 16-byte piece
        int mn = 255;
        const uint8_t* erow = p.a_exp + arow * KB;
        const int n16 = KB >> 4;
        for (int i0 = 0; i0 < n16; i0 += 8) {
            uint4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                __builtin_memcpy(&v[u], erow + 16 * min(i0 + 2 * u + t, n16 - 1), 16);   // no alignment assumed
#pragma unroll
            for (int u = 0; u < 4; ++u)
                mn = min(mn, min(min(min_bytes(v[u].x), min_bytes(v[u].y)), min(min_bytes(v[u].z), min_bytes(v[u].w))));
        }
        for (int i = n16 * 16 + t; i < KB; i += 2) mn = min(mn, (int)erow[i]);
        mn = min(mn, __shfl_xor(mn, 32));
        const bool row_valid = row0 + r < p.M;
        if (chunk == 0 && t == 0) ap[p.off_refa + row0 + r] = row_valid ? (uint8_t)mn : (uint8_t)0;
        uint32_t word = 0;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int delta = (int)((e8 >> (8 * k)) & 0xffu) - mn;
            const bool on = k < nk && row_valid;
            cls[k] = on ? min(delta >> 2, kMaxClass + 1) : -1;
            sh[k] = on ? (delta & 3) : 0;
            if (on) word |= 1u << (4 * k + cls[k]);
        }
#pragma unroll
        for (int s = 1; s < 64; s <<= 1) word |= (uint32_t)__shfl_xor((int)word, s);
        if (lane == 0) atomicOr(&s_present, word);
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *reinterpret_cast<uint4*>(&s_codes[wave][(q * 8 + (lane >> 3)) * kPitch + (lane & 7) * 16]) = craw[q];
    } else if (chunk == 0 && t == 0) {
        ap[p.off_refa + row0 + r] = 0;                // padding rows of the last tile
    }
    __syncthreads();
    const uint32_t present = s_present;
    if (wave == 0 && lane < nk) ap[p.off_mask + (int64_t)tile * KB + kc + lane] = (uint8_t)((present >> (4 * lane)) & 15u);
    const int64_t grp = (int64_t)tile * kGroups + wave;
    if (chunk == 0)                                   // the all-zero block (index KB) of this group, class 0
        *reinterpret_cast<uint4*>(ap + p.off_a8 + (grp * (KB + 1) + KB) * 1024 + lane * 16) = make_uint4(0, 0, 0, 0);
    if (!group_valid) return;
    const int64_t cls_stride = (int64_t)p.tiles_m * kGroups * (KB + 1) * 1024;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        if (k >= nk) break;
        const uint2 c = *reinterpret_cast<const uint2*>(&s_codes[wave][r * kPitch + k * 16 + t * 8]);
        const uint32_t dial = (uint32_t)(d8 >> (8 * k)) & 15u;
        const uint4 tab = *reinterpret_cast<const uint4*>(&s_tab[(dial * 4 + sh[k]) * 4]);
        const v4i data = unpack16(c.x, c.y, tab);
        uint8_t* dst = ap + p.off_a8 + (grp * (KB + 1) + kc + k) * 1024 + t * 512 + r * 16;
#pragma unroll
        for (int cc = 0; cc <= kMaxClass; ++cc)
            if ((present >> (4 * k + cc)) & 1u)
                *reinterpret_cast<v4i*>(dst + cc * cls_stride) = cls[k] == cc ? data : v4i{0, 0, 0, 0};
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

// ---------------------------------------------------------------------------
// Operands quantized in blocks of 16 (Section 4.2, Table 3: smaller blocks for the sublayers most
// sensitive to quantization, possibly mixed with blocks of 32 on the other operand): the paper's
// MAC with one exponent pair per pair of 16-element blocks.  A 32 x 32 x 32 matrix instruction adds
// up both halves of a 32-element stretch, so each stretch takes two of them, one per half with the
// other half's lanes zeroed, each followed by its own fp32 scale-and-add.  128 x 128 outputs per
// workgroup, operands straight from global memory one stretch ahead.  a16 / w16: that operand's
// dialect and exponent arrays hold one entry per 16 elements (otherwise per 32).
// ---------------------------------------------------------------------------
template <bool BF16>
__global__ __launch_bounds__(256) void gemm_block16_kernel(GemmParams p, int a16, int w16) {
    __shared__ uint8_t s_exp[2][512];                  // [buffer][A rows x 2 halves | W rows x 2 halves]
    const int KB = p.KB;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int m0 = blockIdx.y * 128, n0 = blockIdx.x * 128;
    const int half = lane >> 5, l32 = lane & 31;
    int64_t a_row[2], w_row[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        a_row[i] = min(m0 + wm * 64 + i * 32 + l32, p.M - 1);
        w_row[i] = min(n0 + wn * 64 + i * 32 + l32, p.N - 1);
    }
    // metadata index of (row, stretch kb, half h): per 16 elements (row * KB + kb) * 2 + h, per 32 row * KB + kb
    auto meta_a = [&](int64_t row, int kb, int h) { return a16 ? (row * KB + kb) * 2 + h : row * KB + kb; };
    auto meta_w = [&](int64_t row, int kb, int h) { return w16 ? (row * KB + kb) * 2 + h : row * KB + kb; };
    const int t = threadIdx.x;
    const bool t_is_a = t < 128;
    const int64_t e_row = t_is_a ? min(m0 + t, p.M - 1) : min(n0 + t - 128, p.N - 1);

    float acc[2][2][16];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int x = 0; x < 16; ++x) acc[i][j][x] = 0.0f;

    struct Stretch { uint2 ca[2], cw[2]; uint32_t da[2], dw[2], e0, e1; };
    auto load_stretch = [&](int kb) {
        Stretch o;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            o.ca[i] = *reinterpret_cast<const uint2*>(p.a_codes + (a_row[i] * KB + kb) * 16 + half * 8);
            o.cw[i] = *reinterpret_cast<const uint2*>(p.w_codes + (w_row[i] * KB + kb) * 16 + half * 8);
            o.da[i] = (uint32_t)p.a_dial[meta_a(a_row[i], kb, half)] & 15u;
            o.dw[i] = (uint32_t)p.w_dial[meta_w(w_row[i], kb, half)] & 15u;
        }
        o.e0 = t_is_a ? p.a_exp[meta_a(e_row, kb, 0)] : p.w_exp[meta_w(e_row, kb, 0)];
        o.e1 = t_is_a ? p.a_exp[meta_a(e_row, kb, 1)] : p.w_exp[meta_w(e_row, kb, 1)];
        return o;
    };
    Stretch nxt{};
    if (KB > 0) nxt = load_stretch(0);
    for (int kb = 0; kb < KB; ++kb) {
        const Stretch cur = nxt;
        if (kb + 1 < KB) nxt = load_stretch(kb + 1);
        uint8_t* se = s_exp[kb & 1];
        se[2 * t] = (uint8_t)cur.e0;
        se[2 * t + 1] = (uint8_t)cur.e1;
        v4i a[2], b[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            a[i] = unpack16(cur.ca[i].x, cur.ca[i].y, *reinterpret_cast<const uint4*>(g_shifted_book.w[cur.da[i]][0]));
            b[i] = unpack16(cur.cw[i].x, cur.cw[i].y, *reinterpret_cast<const uint4*>(g_shifted_book.w[cur.dw[i]][0]));
        }
        __syncthreads();
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                // this half's 16 elements only: the lanes that hold the other half multiply zeros
                const v4i ah = half == hh ? a[i] : v4i{0, 0, 0, 0};
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    v16i pr = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
                    pr = __builtin_amdgcn_mfma_i32_32x32x32_i8(ah, b[j], pr, 0, 0, 0);
                    const int ew = se[2 * (128 + wn * 64 + j * 32 + l32) + hh];
#pragma unroll
                    for (int x = 0; x < 16; ++x) {
                        const int row = 8 * (x >> 2) + 4 * half + (x & 3);
                        const int ea = se[2 * (wm * 64 + i * 32 + row) + hh];
                        acc[i][j][x] += ldexpf((float)pr[x], ea + ew - 256);
                    }
                }
            }
        }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int n = n0 + wn * 64 + j * 32 + l32;
#pragma unroll
            for (int x = 0; x < 16; ++x) {
                const int m = m0 + wm * 64 + i * 32 + 8 * (x >> 2) + 4 * half + (x & 3);
                if (m < p.M && n < p.N) {
                    const int64_t o = (int64_t)m * p.ldc + n;
                    if constexpr (BF16)
                        static_cast<uint16_t*>(p.out)[o] = f32_to_bf16_rne(acc[i][j][x]);
                    else
                        static_cast<float*>(p.out)[o] = acc[i][j][x];
                }
            }
        }
}

// ---------------------------------------------------------------------------
// Fast kernel: 512 x 128 outputs per workgroup, one int32 accumulator per output.
// Wave w owns rows 128w .. 128w+127 and all 128 columns (16 accumulator tiles of
// 32 x 32: tile i = 4 * gi + n is rows 32 gi .., columns 32 n ..).
// ---------------------------------------------------------------------------
template <bool MX, bool BF16, bool RQ>
__global__ __launch_bounds__(256, 1) void gemm_fast_kernel(GemmParams p) {
    // int8 W operands of a pair of blocks: [column tile n][t][lane][16 bytes]; three buffers in rotation
    __shared__ __attribute__((aligned(16))) uint8_t s_b[3][kBBufBytes];
    // requantizing epilogue only: quantizer tables and, per wave, 64 rows x 128 columns of bf16 results
    __shared__ __attribute__((aligned(16))) uint8_t s_rq_q[RQ ? (MX ? 64 : kDialects * 1024) : 16];
    __shared__ __attribute__((aligned(16))) uint8_t s_rq_s[RQ ? (MX ? 16 : kPairs * 1024) : 16];
    __shared__ __attribute__((aligned(16))) uint16_t s_rq[RQ ? 4 * 64 * kRqPitch : 8];
    __shared__ __attribute__((aligned(16))) uint32_t s_tab[kDialects * 4 * 4 + 4];   // + the all-zero table
    // visits: block | class of A << 10 | class of W << 12, from the highest class sum to the lowest
    __shared__ uint16_t s_vl[kVisitCap];
    __shared__ __attribute__((aligned(4))) uint8_t s_refa[kTileM];
    __shared__ uint8_t s_refw[kTileN];
    __shared__ int s_ctl[8];                 // segment ends (entries), feasibility

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
#ifdef DFP4_TIMING_STAMPS   // timing experiments only: 100 MHz timestamps of the kernel's phases, into the workspace
#ifndef DFP4_STAMP_ROW      // which row of tiles (blockIdx.y) writes them
#define DFP4_STAMP_ROW 0
#endif
#define DFP4_STAMP(I)                                                                                   \
    if (tid == 0 && p.ksplit == 1 && p.part && blockIdx.y == (DFP4_STAMP_ROW) && blockIdx.z == 0 && blockIdx.x < 64)   \
        reinterpret_cast<unsigned long long*>(p.part)[blockIdx.x * 8 + (I)] = wall_clock64();
#else
#define DFP4_STAMP(I)
#endif
    DFP4_STAMP(0)
    const int KB = p.KB;
    // Which output tile: the plain order (columns first).  Measured and found no faster: the workgroups of
    // one XCD (each has its own L2) walking the row tiles of a column tile before the next (W then fetched
    // once: 3 % slower), and one row tile of A per XCD (the same).
    const int tx = blockIdx.x, ty = blockIdx.y;
    const int m0 = ty * kTileM, n0 = tx * kTileN;
    const int S = p.ksplit, sidx = (int)(blockIdx.z % (unsigned)S);
    const int64_t bz = blockIdx.z / (unsigned)S;
    const uint8_t* ap = p.a_prep + bz * p.a_prep_stride;
    const uint8_t* wp = p.w_prep + bz * p.w_prep_stride;
    const int tile_id = ty * p.tiles_n + tx;
    // this workgroup's range of blocks
    const int kb_per = (KB + S - 1) / S;
    const int kb_lo = sidx * kb_per, kb_hi = min(KB, kb_lo + kb_per);

    // ---- prologue: tables, references, list of (block, class of A, class of W) visits
    // every global load of the prologue is issued before the first value is used: one memory round trip, not four
    const uint8_t* mask_a = ap + p.off_mask + (int64_t)ty * KB;
    const uint8_t* mask_w = wp + p.off_wmask + (int64_t)tx * KB;
    uint32_t ma[kMaxKB / 64], mw[kMaxKB / 64];
    if (wave == 0) {
#pragma unroll
        for (int j = 0; j < kMaxKB / 64; ++j) {
            const int kb = j * 64 + lane;
            ma[j] = kb < KB ? mask_a[kb] : 0u;
            mw[j] = kb < KB ? mask_w[kb] : 0u;
        }
    }
    static_assert(kDialects * 16 == 256 && kTileM == 512, "one table word and two reference bytes per thread");
    const uint32_t tab_word = (&g_shifted_book.w[0][0][0])[tid];
    const uint8_t refa0 = ap[p.off_refa + m0 + tid], refa1 = ap[p.off_refa + m0 + 256 + tid];   // rows padded to 512
    const uint8_t refw0 = tid < kTileN && n0 + tid < p.N ? wp[p.off_refw + n0 + tid] : (uint8_t)0;
    s_tab[tid] = tab_word;
    if (tid < 4) s_tab[kDialects * 16 + tid] = 0u;
    s_refa[tid] = refa0;
    s_refa[256 + tid] = refa1;
    if (tid < kTileN) s_refw[tid] = refw0;
    if (tid < 8) s_ctl[tid] = 0;
    if (wave == 0) {
        // A block is visited once for every pair (class present among the tile's 512 rows of A, class
        // present among its 128 rows of W); rows of other classes contribute zeros.  Visits are
        // ordered by the class sum, which is the number of 4-bit shifts the accumulators still
        // receive.  The list holds the visits of this workgroup's range of blocks; whether the tile
        // can be taken at all is decided from ALL blocks, so that every workgroup sharing the tile
        // decides the same.
        bool bad = false;
#pragma unroll
        for (int j = 0; j < kMaxKB / 64; ++j) {
            // highest classes present: their sum must not exceed the classes kept
            const int ha = 31 - __builtin_clz(ma[j] | 1u), hw = 31 - __builtin_clz(mw[j] | 1u);
            bad |= ha + hw > kMaxClass;
        }
        int pos = 0, weight = 0;                                      // weight: sum of 16^(class sum) over all of K
        for (int ct = kMaxClass; ct >= 0; --ct) {
            for (int ca = 0; ca <= ct; ++ca) {
                const int cw = ct - ca;
#pragma unroll
                for (int j = 0; j < kMaxKB / 64; ++j) {
                    if (j * 64 >= KB) break;                          // uniform
                    const int kb = j * 64 + lane;
                    const bool f = ((ma[j] >> ca) & 1u) && ((mw[j] >> cw) & 1u);
                    weight += __popcll(__ballot(f)) << (4 * ct);
                    const bool mine = f && kb >= kb_lo && kb < kb_hi;
                    const unsigned long long bal = __ballot(mine);
                    if (mine) s_vl[pos + __popcll(bal & ((1ull << lane) - 1ull))] = (uint16_t)(kb | (ca << 10) | (cw << 12));
                    pos += __popcll(bal);
                }
            }
            if (pos & 1) {                                            // a step takes two visits
                if (lane == 0) s_vl[pos] = (uint16_t)KB;              // padding: the all-zero block of class 0
                pos += 1;
            }
            if (lane == 0) s_ctl[kMaxClass - ct] = pos;               // s_ctl[0..2]: end of class sum 2, 1, 0
        }
        if (lane < kVisitPad) s_vl[pos + lane] = (uint16_t)KB;        // the loop looks five steps ahead
        // exponent offsets beyond the classes kept, or an int32 accumulator that could overflow
        if (__ballot(bad) != 0ull || weight > kIntBound) {
            if (lane == 0) s_ctl[4] = 1;
        }
    }
    __syncthreads();
    DFP4_STAMP(1)
    // segment ends in steps (uniform: they go to the loop in scalar registers)
    const int end2 = __builtin_amdgcn_readfirstlane(s_ctl[0] / 2), end1 = __builtin_amdgcn_readfirstlane(s_ctl[1] / 2),
              total = __builtin_amdgcn_readfirstlane(s_ctl[2] / 2);
    if (s_ctl[4] != 0) {
        // The tile cannot be taken (every workgroup sharing it sees the same): the first of them
        // computes it with one fp32 scale-and-add per block, 128 rows at a time; the others leave.
        if (sidx != 0) return;
        if (tid == 0)
            atomicAdd(reinterpret_cast<uint32_t*>(const_cast<uint8_t*>(ap) + p.off_cnt) + kMaxSplitTiles, 1u);
        if constexpr (RQ) {
            if constexpr (MX) {
                if (tid < 64) s_rq_q[tid] = g_quant_tables.mx[tid];
            } else {
                const uint4* gq = reinterpret_cast<const uint4*>(g_quant_tables.q);
                const uint4* gs = reinterpret_cast<const uint4*>(g_quant_tables.s);
                for (int i = tid; i < 1024; i += 256) reinterpret_cast<uint4*>(s_rq_q)[i] = gq[i];
                for (int i = tid; i < 512; i += 256) reinterpret_cast<uint4*>(s_rq_s)[i] = gs[i];
            }
        }
        uint8_t (&s_exp)[2][256] = *reinterpret_cast<uint8_t (*)[2][256]>(&s_b[0][0]);
        for (int piece = 0; piece < 4; ++piece) {
            const int by = ty * 4 + piece;
            if (by * 128 >= p.M) break;
            __syncthreads();
            block_flush_tile<MX, BF16>(p, bz, by, tx, s_exp);
            if constexpr (RQ) quantize_flushed_piece<MX>(p, bz, by, tx, s_rq_s, s_rq_q);
        }
        return;
    }

    const int h = lane >> 5, r = lane & 31;            // MFMA operand: lanes 32.. hold the pair's second block
    const uint32_t wave_u = (uint32_t)__builtin_amdgcn_readfirstlane(wave);
    const uint32_t lds_tab = (uint32_t)__builtin_amdgcn_readfirstlane(
        (int)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)&s_tab[0]);
    const uint32_t lds_vl = (uint32_t)__builtin_amdgcn_readfirstlane(
        (int)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)&s_vl[0]);
    const uint32_t lds_b = (uint32_t)__builtin_amdgcn_readfirstlane(
        (int)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)&s_b[0][0]);
    const uint32_t grp_stride = (uint32_t)(KB + 1) * 1024u;
    const uint32_t cls_stride = (uint32_t)p.tiles_m * kGroups * grp_stride;
    const uint32_t tile_off = (uint32_t)ty * kGroups * grp_stride;
#ifdef DFP4_TIMING_SAME_A   // timing experiments only: every wave reads the fragments of wave 0 (wrong results)
    const uint8_t* a8w = ap + p.off_a8;
#else
    const uint8_t* a8w = ap + p.off_a8 + (uint64_t)wave_u * 4u * grp_stride;   // uniform per wave
#endif
    const uint8_t* wcodes = wp + p.off_wcodes;                                // uniform; [group][block][row]
    const uint8_t* wmeta = wp + p.off_wmeta;                                  // uniform; [class][group][block][row]
    const int ncol = n0 + wave * 32 + r;                // this lane's W row (rows beyond N exist: all-zero tables)
    // this lane's row of W: slot (row % 32) of block 0 of its 32-row group; a block further is 32 slots further
    const uint32_t w_slot = (uint32_t)(ncol >> 5) * (uint32_t)KB * 32u + (uint32_t)(ncol & 31);
    const uint32_t w_row_codes = w_slot * 16u, w_row_meta = w_slot * 4u;

    // W operands of the first two steps (the loop expands those of step s + 2 during step s)
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const uint32_t entry = s_vl[2 * s + h];
        const uint32_t kb = min(entry & 1023u, (uint32_t)KB - 1u);
        const uint4 c = *reinterpret_cast<const uint4*>(wcodes + w_row_codes + kb * 512u);
        const uint32_t meta = *reinterpret_cast<const uint32_t*>(wmeta + ((entry >> 12) & 3u) * p.wmeta_cls_stride +
                                                                 w_row_meta + kb * 128u);
        const uint4 tab = *reinterpret_cast<const uint4*>(reinterpret_cast<const uint8_t*>(s_tab) + meta);
        *reinterpret_cast<v4i*>(&s_b[s][(wave * 2 + 0) * 1024 + lane * 16]) = unpack16(c.x, c.y, tab);
        *reinterpret_cast<v4i*>(&s_b[s][(wave * 2 + 1) * 1024 + lane * 16]) = unpack16(c.z, c.w, tab);
    }
    __syncthreads();
    DFP4_STAMP(2)

    // ---- main loop (gemm_step_asm.inc): accumulators in a[0:255]
    {
        const uint64_t a8u = reinterpret_cast<uint64_t>(a8w), wcu = reinterpret_cast<uint64_t>(wcodes),
                       wmu = reinterpret_cast<uint64_t>(wmeta);
        const uint32_t a_lane = (uint32_t)r * 16u, l16 = (uint32_t)lane * 16u, h2 = (uint32_t)h * 2u;
        const uint32_t sign_sel = 0x090b080au, kbm = (uint32_t)KB - 1u;
        asm volatile(DFP4_MAINLOOP_ASM
                     :
                     : [a8lo] "s"((uint32_t)a8u), [a8hi] "s"((uint32_t)(a8u >> 32)), [gstr] "s"(grp_stride),
                       [wclo] "s"((uint32_t)wcu), [wchi] "s"((uint32_t)(wcu >> 32)),
                       [wmlo] "s"((uint32_t)wmu), [wmhi] "s"((uint32_t)(wmu >> 32)),
                       [cstr] "s"(cls_stride), [toff] "s"(tile_off), [kbm] "s"(kbm), [tabb] "s"(lds_tab),
                       [vlb] "s"(lds_vl), [bb] "s"(lds_b), [sel] "s"(sign_sel),
                       [e2] "s"((uint32_t)end2), [e1] "s"((uint32_t)end1), [e0] "s"((uint32_t)total),
                       [wcs] "s"(p.wmeta_cls_stride),
                       [wv] "s"(wave_u), [alane] "v"(a_lane), [l16] "v"(l16), [wrc] "v"(w_row_codes),
                       [wrm] "v"(w_row_meta), [h2] "v"(h2)
                     : DFP4_LOOP_VGPR_CLOBBERS, DFP4_ACC_CLOBBERS, DFP4_LOOP_SGPR_CLOBBERS, "scc", "memory");
    }

    DFP4_STAMP(3)
    // ---- epilogue (nothing to store or publish for a wave whose 128 rows lie beyond M)
    if constexpr (RQ) {
        if constexpr (MX) {
            if (tid < 64) s_rq_q[tid] = g_quant_tables.mx[tid];
        } else {
            const uint4* gq = reinterpret_cast<const uint4*>(g_quant_tables.q);
            const uint4* gs = reinterpret_cast<const uint4*>(g_quant_tables.s);
            for (int i = tid; i < 1024; i += 256) reinterpret_cast<uint4*>(s_rq_q)[i] = gq[i];
            for (int i = tid; i < 512; i += 256) reinterpret_cast<uint4*>(s_rq_s)[i] = gs[i];
        }
        __syncthreads();
    }
    const bool active = m0 + (int)wave_u * 128 < p.M;      // wave-uniform
#define DFP4_READ_ACC(G, V)                                                                         \
    asm volatile(DFP4_ACC_READ_ASM_##G                                                              \
                 : "=v"(V[0]), "=v"(V[1]), "=v"(V[2]), "=v"(V[3]), "=v"(V[4]), "=v"(V[5]),          \
                   "=v"(V[6]), "=v"(V[7]), "=v"(V[8]), "=v"(V[9]), "=v"(V[10]), "=v"(V[11]),        \
                   "=v"(V[12]), "=v"(V[13]), "=v"(V[14]), "=v"(V[15]))
#define DFP4_FOR_TILES(F)                                                                           \
    F(0) F(1) F(2) F(3) F(4) F(5) F(6) F(7) F(8) F(9) F(10) F(11) F(12) F(13) F(14) F(15)
    // partial tiles of the workgroups that share this output tile: [range][(16 tile + x) * 256 + thread]
    const int* part = S > 1 ? p.part + bz * p.part_stride + (int64_t)tile_id * S * (kTileM * kTileN) : nullptr;
    if (S > 1) {
        // K is shared with other workgroups.  Every one publishes its exact int32 sums and then
        // counts itself in; the one that arrives last adds the others' sums to its own (the total
        // is exact and does not depend on the order) and goes on to the conversion and the stores.
        // The sums travel as device-scope relaxed atomic stores and loads (they pass the per-XCD
        // L2 instead of being written back and invalidated wholesale by a fence); "all my stores
        // have completed" is the wait on the memory counter before the barrier.
        if (active) {
            int* mine = const_cast<int*>(part) + (int64_t)sidx * (kTileM * kTileN);
#define DFP4_PUBLISH(G)                                                                             \
            {                                                                                       \
                int v[16];                                                                          \
                DFP4_READ_ACC(G, v);                                                                \
                _Pragma("unroll") for (int x = 0; x < 16; ++x)                                      \
                    __hip_atomic_store(&mine[(G * 16 + x) * 256 + tid], v[x], __ATOMIC_RELAXED,     \
                                       __HIP_MEMORY_SCOPE_AGENT);                                   \
            }
            DFP4_FOR_TILES(DFP4_PUBLISH)
#undef DFP4_PUBLISH
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0) {
            uint32_t* cnt = reinterpret_cast<uint32_t*>(const_cast<uint8_t*>(ap) + p.off_cnt) + tile_id;
            const uint32_t arrived = atomicAdd(cnt, 1u);
            if (arrived == (uint32_t)S - 1u) atomicExch(cnt, 0u);       // ready for the next product
            s_ctl[5] = (int)arrived;
        }
        __syncthreads();
        if (s_ctl[5] != S - 1) return;
    }
    if (!active) return;                                   // nothing to store for rows beyond M
#define DFP4_READ_TILE(G, V)                                                                        \
    DFP4_READ_ACC(G, V);                                                                            \
    if (S > 1) {                                                                                    \
        for (int s_ = 0; s_ < S; ++s_) {                                                            \
            if (s_ == sidx) continue;                                                               \
            const int* other_ = part + (int64_t)s_ * (kTileM * kTileN);                             \
            _Pragma("unroll") for (int x = 0; x < 16; ++x)                                          \
                V[x] += __hip_atomic_load(&other_[(G * 16 + x) * 256 + tid], __ATOMIC_RELAXED,      \
                                          __HIP_MEMORY_SCOPE_AGENT);                                \
        }                                                                                           \
    }
    if constexpr (RQ) {
        // Requantizing epilogue (Section 3.3: results are quantized again for the next
        // multiplication).  Each value is converted and rounded to bf16 exactly as the bf16
        // output would be; the wave stages 64 rows x 128 columns in LDS and re-reads them in
        // the quantizer's layout (4 lanes per block of 32 consecutive columns), then stores
        // codes, dialect ids and exponent bytes of the [M, N] result blocked along N.
        const int row0 = m0 + (int)wave_u * 128;
        uint16_t* st = &s_rq[wave * 64 * kRqPitch];
        const int nb_row = p.N / kBlock;
        int ew[4];
#pragma unroll
        for (int n = 0; n < 4; ++n) ew[n] = (int)s_refw[n * 32 + r] - 256;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
#define DFP4_STAGE(G)                                                                               \
            if ((G >> 3) == half) {                                                                 \
                int v[16];                                                                          \
                DFP4_READ_TILE(G, v);                                                               \
                const int gi = G >> 2, n = G & 3;                                                   \
                _Pragma("unroll") for (int q = 0; q < 4; ++q) {                                     \
                    const uint32_t e4 = *reinterpret_cast<const uint32_t*>(                         \
                        &s_refa[wave * 128 + gi * 32 + 8 * q + 4 * h]);                             \
                    _Pragma("unroll") for (int j = 0; j < 4; ++j) {                                 \
                        const float f = ldexpf((float)v[4 * q + j], (int)((e4 >> (8 * j)) & 0xffu) + ew[n]); \
                        st[((gi & 1) * 32 + 8 * q + 4 * h + j) * kRqPitch + n * 32 + r] = f32_to_bf16_rne(f); \
                    }                                                                               \
                }                                                                                   \
            }
            DFP4_FOR_TILES(DFP4_STAGE)
#undef DFP4_STAGE
            for (int pass = 0; pass < 16; ++pass) {
                const int b = pass * 16 + (lane >> 2), row = b >> 2, cb = b & 3, sub = lane & 3;
                const uint4 wv = *reinterpret_cast<const uint4*>(&st[row * kRqPitch + cb * 32 + sub * 8]);
                uint32_t code, eb, dl = 0;
                if constexpr (MX) mxfp4_pass(wv, s_rq_q, code, eb);
                else dfp4_pass(wv, s_rq_s, s_rq_q, code, eb, dl);
                const int m = row0 + half * 64 + row, nb = (n0 >> 5) + cb;
                if (m < p.M && nb < nb_row) {
                    const size_t blk = (size_t)(bz * p.M + m) * nb_row + nb;
                    p.q_codes[blk * 4 + sub] = code;
                    if (sub == 0) {
                        p.q_exp[blk] = (uint8_t)eb;
                        if constexpr (!MX) p.q_dial[blk] = (uint8_t)dl;
                    }
                }
            }
        }
        return;
    }
    {
        // The one rounding of the whole product: int32 -> fp32, scaled by 2^(refA + refW - 2).
        // Accumulator x of lane (h, r) of tile (gi, n) is output row 128*wave + 32*gi +
        // 8*(x>>2) + 4*h + (x&3), column 32*n + r.  Row addresses are wave-uniform (scalar
        // registers); the lane adds a constant byte offset, so a store costs a handful of
        // instructions.
        constexpr int kEsz = BF16 ? 2 : 4;
        const int row0 = m0 + (int)wave_u * 128;
        uint8_t* wave_out = static_cast<uint8_t*>(p.out) +
                            (bz * p.strideC + (int64_t)row0 * p.ldc + n0) * kEsz;            // uniform
        const int64_t row_bytes = p.ldc * kEsz;                                              // uniform
        const bool full = row0 + 128 <= p.M && n0 + kTileN <= p.N;                           // uniform
        // bf16: lanes exchange values in pairs so that every lane stores two adjacent columns of
        // one row (even lanes the even row of a row pair, odd lanes the odd row)
        const bool pairs = BF16 && full && (p.ldc & 1) == 0 && ((p.strideC * kEsz) & 3) == 0 &&
                           (reinterpret_cast<uintptr_t>(p.out) & 3) == 0;                    // uniform
        const uint32_t lane_off = pairs ? (uint32_t)((4 * h + (r & 1)) * row_bytes + (r & ~1) * kEsz)
                                        : (uint32_t)(4 * h * row_bytes + r * kEsz);
        int ew[4];
#pragma unroll
        for (int n = 0; n < 4; ++n) ew[n] = (int)s_refw[n * 32 + r] - 256;
        auto store_tile = [&](auto full_c, auto pairs_c, int i, int (&v)[16]) {
            constexpr bool kFull = decltype(full_c)::value, kPairs = decltype(pairs_c)::value;
            const int gi = i >> 2, n = i & 3;
            uint8_t* tile_out = wave_out + (int64_t)gi * 32 * row_bytes + n * 32 * kEsz;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t e4 = *reinterpret_cast<const uint32_t*>(&s_refa[wave * 128 + gi * 32 + 8 * q + 4 * h]);
                float f[4];
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    f[j] = ldexpf((float)v[4 * q + j], (int)((e4 >> (8 * j)) & 0xffu) + ew[n]);
                uint8_t* rowp = tile_out + (int64_t)(8 * q) * row_bytes;                    // uniform
                if constexpr (BF16 && kPairs) {
#pragma unroll
                    for (int j = 0; j < 4; j += 2) {
                        const uint32_t b0 = f32_to_bf16_rne(f[j]), b1 = f32_to_bf16_rne(f[j + 1]);
                        const uint32_t send = (r & 1) ? b0 : b1;
                        const uint32_t recv = (uint32_t)__builtin_amdgcn_mov_dpp((int)send, 0xB1, 0xf, 0xf, true);
                        const uint32_t word = (r & 1) ? (recv | (b1 << 16)) : (b0 | (recv << 16));
                        DFP4_OUT_STORE(reinterpret_cast<uint32_t*>(rowp + (int64_t)j * row_bytes + lane_off), word);
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        if (kFull || (row0 + gi * 32 + 8 * q + 4 * h + j < p.M && n0 + n * 32 + r < p.N)) {
                            uint8_t* dst = rowp + (int64_t)j * row_bytes + lane_off;
                            if constexpr (BF16)
                                DFP4_OUT_STORE(reinterpret_cast<uint16_t*>(dst), f32_to_bf16_rne(f[j]));
                            else
                                DFP4_OUT_STORE(reinterpret_cast<float*>(dst), f[j]);
                        }
                    }
                }
            }
        };
#define DFP4_FINISH(G)                                                                              \
        {                                                                                           \
            int v[16];                                                                              \
            DFP4_READ_TILE(G, v);                                                                   \
            store_tile(kFullC, kPairsC, G, v);                                                      \
        }
        if (pairs) {
            constexpr std::true_type kFullC{}, kPairsC{};
            DFP4_FOR_TILES(DFP4_FINISH)
        } else if (full) {
            constexpr std::true_type kFullC{};
            constexpr std::false_type kPairsC{};
            DFP4_FOR_TILES(DFP4_FINISH)
        } else {
            constexpr std::false_type kFullC{}, kPairsC{};
            DFP4_FOR_TILES(DFP4_FINISH)
        }
#undef DFP4_FINISH
    }
    DFP4_STAMP(4)
#undef DFP4_STAMP
#undef DFP4_FOR_TILES
#undef DFP4_READ_TILE
#undef DFP4_READ_ACC
}

// The whole prepared form of an A operand of few rows: the count of declined tiles.
__global__ void clear_count_kernel(uint32_t* count) {
    if (threadIdx.x == 0) *count = 0;
}

}  // namespace

// Largest operands the single-accumulator kernel addresses with its 32-bit offsets: the expanded
// A (all classes) and the 4-bit codes of W each stay below 2 GiB.  Larger products are cut into
// pieces of at most this many rows on the host.
static int64_t max_rows_a(int64_t KB) {
    const int64_t tiles = (((int64_t)1 << 31) - 1) / ((int64_t)(kMaxClass + 1) * kGroups * (KB + 1) * 1024);
    return (tiles < 65535 ? tiles : 65535) * kTileM;
}
static int64_t max_rows_w(int64_t KB) { return ((((int64_t)1 << 31) - 1) / (KB * 16)) / kTileN * kTileN; }

size_t gemm_prepared_bytes(int64_t rows, int64_t K, bool weight) {
    const int64_t KB = K / kBlock;
    if (rows <= 0 || KB <= 0 || KB > kMaxKB) return 0;
    if (!weight && rows < kPreparedMinRows) return 256;    // the count of declined tiles
    return (size_t)(weight ? prep_w_layout(rows, KB).total : prep_a_layout(rows, KB).total);
}

// byte offset, inside a prepared A, of the dword that counts tiles declined since it was prepared
size_t gemm_prepared_declined_offset(int64_t M, int64_t K) {
    return M < kPreparedMinRows ? 0 : (size_t)prep_a_layout(M, K / kBlock).off_cnt + (size_t)kMaxSplitTiles * 4;
}

size_t gemm_prepared_workspace_bytes(int64_t M, int64_t N, int64_t K) {
    const int64_t KB = K / kBlock;
    if (M <= 0 || N <= 0 || !fast_kernel_can(M, KB) || M < kPreparedMinRows) return 0;
    const int64_t cu = device_cu_count();
    return direct_shape(M, N, KB, 1, true, cu) >= 0 ? 0 : (size_t)partial_bytes(M, N, KB, cu);
}

// what gemm_fast_kernel and its prepass need
static size_t fast_workspace_bytes(int64_t M, int64_t N, int64_t KB, int64_t cu) {
    const int64_t Mc = M < max_rows_a(KB) ? M : max_rows_a(KB), Nc = N < max_rows_w(KB) ? N : max_rows_w(KB);
    return (size_t)(prep_a_layout(Mc, KB).total + prep_w_layout(Nc, KB).total + partial_bytes(Mc, Nc, KB, cu));
}

size_t gemm_fast_workspace_bytes(int64_t M, int64_t N, int64_t K) {
    const int64_t KB = K / kBlock;
    return M <= 0 || N <= 0 || !fast_kernel_can(M, KB) ? 0 : fast_workspace_bytes(M, N, KB, device_cu_count());
}

size_t gemm_workspace_bytes(int64_t M, int64_t N, int64_t K) {
    const int64_t KB = K / kBlock;
    if (M <= 0 || N <= 0 || !fast_kernel_can(M, KB)) return 0;
    // nothing but a token where the direct kernel is taken whatever the batch
    const int64_t cu = device_cu_count();
    if (direct_shape(M, N, KB, 1, false, cu) >= 0 && direct_shape(M, N, KB, 65535, false, cu) >= 0) return 256;
    return fast_workspace_bytes(M, N, KB, cu);
}

int gemm_path(int64_t M, int64_t N, int64_t KB, int64_t batch, bool prepared) {
    prepared = prepared && KB > 0 && KB <= kMaxKB;         // otherwise nothing is prepared and the operands are read as they are
    return 1 + direct_shape(M, N, KB, batch, prepared, device_cu_count());
}

size_t gemm_requant_workspace_bytes(int64_t M, int64_t N, int64_t K) {
    if (M <= 0 || N <= 0) return 0;
    return (size_t)align256((int64_t)gemm_fast_workspace_bytes(M, N, K)) + (size_t)align256(M * N * 2);
}

namespace {

void fill_params(GemmParams& p, const dfp4_tensor& A, const dfp4_tensor& W, void* out, int64_t ldc,
                 int64_t strideA_rows, int64_t strideW_rows, int64_t strideC, const dfp4_tensor* rq) {
    p.a_codes = A.codes; p.a_dial = A.dialect; p.a_exp = A.exponent;
    p.w_codes = W.codes; p.w_dial = W.dialect; p.w_exp = W.exponent;
    p.out = out; p.M = (int)A.rows; p.N = (int)W.rows; p.KB = (int)(A.K / kBlock);
    p.ldc = ldc; p.strideA_rows = strideA_rows; p.strideW_rows = strideW_rows; p.strideC = strideC;
    p.tiles_m = (int)((A.rows + kTileM - 1) / kTileM); p.tiles_n = (int)((W.rows + kTileN - 1) / kTileN);
    p.ksplit = 1;
    if (rq) {
        p.q_codes = reinterpret_cast<uint32_t*>(rq->codes); p.q_dial = rq->dialect; p.q_exp = rq->exponent;
    }
}

void set_prepared(GemmParams& p, uint8_t* a_prep, int64_t a_stride, uint8_t* w_prep, int64_t w_stride) {
    const PrepALayout la = prep_a_layout(p.M, p.KB);
    const PrepWLayout lw = prep_w_layout(p.N, p.KB);
    p.a_prep = a_prep; p.a_prep_stride = a_stride;
    p.w_prep = w_prep; p.w_prep_stride = w_stride;
    p.off_refa = la.off_refa; p.off_mask = la.off_mask; p.off_cnt = la.off_cnt; p.off_a8 = la.off_a8;
    p.off_refw = lw.off_refw; p.off_wmask = lw.off_wmask; p.off_wmeta = lw.off_wmeta; p.off_wcodes = lw.off_wcodes;
    p.wmeta_cls_stride = (uint32_t)((int64_t)p.tiles_n * kTileN * p.KB * 4);
}

// prepass: A workgroups (when do_a) and W workgroups (when do_w) in one launch
int launch_prep(bool mx, const GemmParams& p, bool do_a, bool do_w, int64_t batch, hipStream_t stream) {
    const int64_t KB = p.KB;
    const int chunks_a = (int)((KB + 7) / 8);
    const int64_t n_a = do_a ? (int64_t)p.tiles_m * chunks_a : 0;
    const int64_t n_w = do_w ? (int64_t)p.tiles_n * ((KB + 63) / 64) : 0;
    if (n_a + n_w == 0) return DFP4_OK;
    if (n_a + n_w > 0x7fffffff || batch > 65535) return DFP4_ERR_SHAPE;
    dim3 gp((unsigned)(n_a + n_w), 1, (unsigned)batch);
    if (mx)
        hipLaunchKernelGGL((gemm_prep_kernel<true>), gp, dim3(1024), 0, stream, p, (int)n_a, chunks_a);
    else
        hipLaunchKernelGGL((gemm_prep_kernel<false>), gp, dim3(1024), 0, stream, p, (int)n_a, chunks_a);
    return check_launch();
}

// single-accumulator kernel on prepared operands; `part`: room for the partial tiles where K is split
int launch_fast(bool mx, bool bf16, GemmParams& p, int64_t batch, int* part, size_t part_bytes, bool rq,
                hipStream_t stream) {
    const int64_t tiles = (int64_t)p.tiles_m * p.tiles_n;
    p.ksplit = choose_ksplit(tiles * batch, p.KB, device_cu_count());
    const size_t per_batch = (size_t)p.ksplit * tiles * kTileM * kTileN * 4;
    if (p.ksplit > 1 && (!part || per_batch * (size_t)batch > part_bytes)) p.ksplit = 1;   // no room: no split
    p.part = part;
    p.part_stride = (int64_t)(per_batch / 4);
    if (batch * p.ksplit > 65535 || p.tiles_m > 65535) return DFP4_ERR_SHAPE;
    dim3 gf((unsigned)p.tiles_n, (unsigned)p.tiles_m, (unsigned)(batch * p.ksplit));
    if (rq) {
        if (mx) hipLaunchKernelGGL((gemm_fast_kernel<true, true, true>), gf, dim3(256), 0, stream, p);
        else hipLaunchKernelGGL((gemm_fast_kernel<false, true, true>), gf, dim3(256), 0, stream, p);
    } else {
        dispatch_mx_bf16(mx, bf16, [&](auto mxc, auto bc) {
            hipLaunchKernelGGL((gemm_fast_kernel<decltype(mxc)::value, decltype(bc)::value, false>), gf, dim3(256), 0,
                               stream, p);
        });
    }
    return check_launch();
}

// direct kernel, in pieces of at most as many rows as it addresses
int launch_direct(bool mx, bool bf16, dfp4_tensor A, dfp4_tensor W, void* out, int64_t ldc, int64_t batch,
                  int64_t strideA_rows, int64_t strideW_rows, int64_t strideC, hipStream_t stream) {
    const int64_t KB = A.K / kBlock, M = A.rows, N = W.rows, cu = device_cu_count();
    const int64_t mc = gemm_direct_max_rows(KB, false), nc = gemm_direct_max_rows(KB, true);
    for (int64_t m0 = 0; m0 < M; m0 += mc)
        for (int64_t n0 = 0; n0 < N; n0 += nc) {
            dfp4_tensor a = A, w = W;
            a.rows = M - m0 < mc ? M - m0 : mc;
            w.rows = N - n0 < nc ? N - n0 : nc;
            a.codes += m0 * KB * 16; a.exponent += m0 * KB; if (a.dialect) a.dialect += m0 * KB;
            w.codes += n0 * KB * 16; w.exponent += n0 * KB; if (w.dialect) w.dialect += n0 * KB;
            GemmParams p{};
            fill_params(p, a, w, static_cast<uint8_t*>(out) + (size_t)(m0 * ldc + n0) * (bf16 ? 2 : 4), ldc, strideA_rows,
                        strideW_rows, strideC, nullptr);
            const int rc = launch_gemm_direct(mx, bf16, p, batch, choose_direct(p.M, p.N, KB, batch, cu).shape, stream);
            if (rc != DFP4_OK) return rc;
        }
    return DFP4_OK;
}

bool shape_in_range(int64_t M, int64_t N, int64_t KB, int64_t batch, int64_t ldc) {
    return M < (1 << 30) && N < (1 << 30) && KB < (1 << 26) && batch <= 65535 && ldc < (1 << 27);
}

}  // namespace

// Shape limits of launch_gemm, so that callers can refuse a product before they enqueue anything.
int gemm_shape_check(dfp4_tensor A, dfp4_tensor W, int64_t ldc, int64_t batch, bool rq) {
    const int64_t M = A.rows, N = W.rows, KB = A.K / kBlock;
    if (M == 0 || N == 0 || batch == 0) return DFP4_OK;
    if (!shape_in_range(M, N, KB, batch, ldc)) return DFP4_ERR_SHAPE;
    if (fast_kernel_can(M, KB) && (rq || batch > 1) && (M > max_rows_a(KB) || N > max_rows_w(KB)))
        return DFP4_ERR_SHAPE;         // only the plain single product is cut into pieces
    return DFP4_OK;
}

// `rq` (optional): quantize the result along N into *rq.  `out` must then be a bf16 [batch * M, N]
// temporary (ldc = N): it receives the results of every path that does not quantize in its epilogue.
int launch_gemm(bool mx, dfp4_tensor A, dfp4_tensor W, void* out, int out_dtype, int64_t ldc,
                int64_t batch, int64_t strideA_rows, int64_t strideW_rows, int64_t strideC,
                void* workspace, size_t workspace_bytes, hipStream_t stream, const dfp4_tensor* rq) {
    const int64_t M = A.rows, N = W.rows, KB = A.K / kBlock;
    if (M == 0 || N == 0 || batch == 0) return DFP4_OK;
    int rc = gemm_shape_check(A, W, ldc, batch, rq != nullptr);
    if (rc != DFP4_OK) return rc;
    const bool bf16 = out_dtype == DFP4_BF16;
    const int64_t cu = device_cu_count();
    if (!fast_kernel_can(M, KB) || (!rq && (!workspace || workspace_bytes < fast_workspace_bytes(M, N, KB, cu) * (size_t)batch ||
                                            direct_shape(M, N, KB, batch, false, cu) >= 0))) {
        rc = launch_direct(mx, bf16, A, W, out, ldc, batch, strideA_rows, strideW_rows, strideC, stream);
        if (rc != DFP4_OK || !rq) return rc;
        return launch_quantize(mx, out, M * batch, N, ldc, *rq, stream);       // `out` holds the bf16 [batch * M, N]
    }
    // pieces of at most mc x nc outputs (one piece for every product of ordinary size)
    const int64_t mc = M < max_rows_a(KB) ? M : max_rows_a(KB), nc = N < max_rows_w(KB) ? N : max_rows_w(KB);
    const PrepALayout la = prep_a_layout(mc, KB);
    const PrepWLayout lw = prep_w_layout(nc, KB);
    const size_t prep_bytes = (size_t)(la.total + lw.total) * (size_t)batch;
    if (!workspace || prep_bytes > workspace_bytes) return DFP4_ERR_WORKSPACE;
    uint8_t* ws = static_cast<uint8_t*>(workspace);
    const size_t esz = bf16 ? 2 : 4;
    for (int64_t m0 = 0; m0 < M; m0 += mc) {
        for (int64_t n0 = 0; n0 < N; n0 += nc) {
            dfp4_tensor a = A, w = W;
            a.rows = M - m0 < mc ? M - m0 : mc;
            w.rows = N - n0 < nc ? N - n0 : nc;
            a.codes += m0 * KB * 16; a.exponent += m0 * KB; if (a.dialect) a.dialect += m0 * KB;
            w.codes += n0 * KB * 16; w.exponent += n0 * KB; if (w.dialect) w.dialect += n0 * KB;
            GemmParams p{};
            fill_params(p, a, w, static_cast<uint8_t*>(out) + (size_t)(m0 * ldc + n0) * esz, ldc, strideA_rows,
                        strideW_rows, strideC, rq);
            // the piece's own layouts (a last piece may be smaller), always within the room of a full one
            const PrepALayout pa = prep_a_layout(a.rows, KB);
            const PrepWLayout pw = prep_w_layout(w.rows, KB);
            set_prepared(p, ws, pa.total, ws + (size_t)la.total * batch, pw.total);
            rc = launch_prep(mx, p, n0 == 0, true, batch, stream);
            if (rc != DFP4_OK) return rc;
            rc = launch_fast(mx, bf16, p, batch, reinterpret_cast<int*>(ws + prep_bytes), workspace_bytes - prep_bytes,
                             rq != nullptr, stream);
            if (rc != DFP4_OK) return rc;
        }
    }
    return DFP4_OK;
}

// One operand prepared ahead of the product (weights: once; an activation: once for all the
// products that consume it).
int launch_gemm_prepare(bool mx, dfp4_tensor T, bool weight, void* prepared, hipStream_t stream) {
    const int64_t KB = T.K / kBlock;
    if (!weight && T.rows < kPreparedMinRows) {
        hipLaunchKernelGGL(clear_count_kernel, dim3(1), dim3(64), 0, stream, static_cast<uint32_t*>(prepared));
        return check_launch();
    }
    GemmParams p{};
    dfp4_tensor none{};
    none.K = T.K;
    if (weight) {
        if (T.rows > max_rows_w(KB)) return DFP4_ERR_SHAPE;
        fill_params(p, none, T, nullptr, 0, 0, 0, 0, nullptr);
    } else {
        if (T.rows > max_rows_a(KB)) return DFP4_ERR_SHAPE;
        fill_params(p, T, none, nullptr, 0, 0, 0, 0, nullptr);
    }
    set_prepared(p, static_cast<uint8_t*>(prepared), 0, static_cast<uint8_t*>(prepared), 0);
    return launch_prep(mx, p, !weight, weight, 1, stream);
}

int launch_gemm_block16(dfp4_tensor A, bool a16, dfp4_tensor W, bool w16, void* out, int out_dtype, int64_t ldc,
                        hipStream_t stream) {
    const int64_t M = A.rows, N = W.rows, KB = A.K / kBlock;
    if (M == 0 || N == 0) return DFP4_OK;
    if (!shape_in_range(M, N, KB, 1, ldc) || (M + 127) / 128 > 65535) return DFP4_ERR_SHAPE;
    GemmParams p{};
    fill_params(p, A, W, out, ldc, 0, 0, 0, nullptr);
    dim3 gb((unsigned)((N + 127) / 128), (unsigned)((M + 127) / 128), 1);
    if (out_dtype == DFP4_BF16)
        hipLaunchKernelGGL((gemm_block16_kernel<true>), gb, dim3(256), 0, stream, p, a16 ? 1 : 0, w16 ? 1 : 0);
    else
        hipLaunchKernelGGL((gemm_block16_kernel<false>), gb, dim3(256), 0, stream, p, a16 ? 1 : 0, w16 ? 1 : 0);
    return check_launch();
}

int launch_gemm_prepared(bool mx, dfp4_tensor A, void* a_prepared, dfp4_tensor W, const void* w_prepared, void* out,
                         int out_dtype, int64_t ldc, void* workspace, size_t workspace_bytes, hipStream_t stream) {
    const int64_t M = A.rows, N = W.rows, KB = A.K / kBlock;
    if (M == 0 || N == 0) return DFP4_OK;
    if (!shape_in_range(M, N, KB, 1, ldc)) return DFP4_ERR_SHAPE;
    const bool bf16 = out_dtype == DFP4_BF16;
    if (KB == 0 || KB > kMaxKB) return launch_direct(mx, bf16, A, W, out, ldc, 1, 0, 0, 0, stream);
    const int64_t cu = device_cu_count();
    GemmParams p{};
    fill_params(p, A, W, out, ldc, 0, 0, 0, nullptr);
    if (M > max_rows_a(KB) || N > max_rows_w(KB)) return DFP4_ERR_SHAPE;
    if (M < kPreparedMinRows) {
        p.declined = static_cast<uint32_t*>(a_prepared);
        return launch_gemm_direct(mx, bf16, p, 1, choose_direct(M, N, KB, 1, cu).shape, stream);     // one launch: max_rows_w is half of what it takes
    }
    set_prepared(p, static_cast<uint8_t*>(a_prepared), 0, static_cast<uint8_t*>(const_cast<void*>(w_prepared)), 0);
    const int shape = direct_shape(M, N, KB, 1, true, cu);
    if (shape >= 0 && M <= gemm_direct_max_rows(KB, false) && N <= gemm_direct_max_rows(KB, true)) {
        p.declined = reinterpret_cast<uint32_t*>(static_cast<uint8_t*>(a_prepared) + gemm_prepared_declined_offset(M, A.K));
        return launch_gemm_direct(mx, bf16, p, 1, shape, stream);
    }
    return launch_fast(mx, bf16, p, 1, static_cast<int*>(workspace), workspace_bytes, false, stream);
}

}  // namespace dfp4
