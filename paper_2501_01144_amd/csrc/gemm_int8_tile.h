// A tile of A * W^T on operands in their 4-bit form, summed exactly in int32 on the int8 matrix cores (scheme: gemm.hip), or with
// one fp32 scale-and-add per block where its exponents spread too far.  One workgroup computes a tile of
// 32 TI WM x 32 TJ WN outputs: a piece of a tile that gemm_f8.hip or gemm_native.hip cannot sum exactly in fp32.
//
// A workgroup has KG groups of WM x WN waves.  Every group computes the same tile of 32 TI WM x 32 TJ WN
// outputs over its own contiguous range of K; the groups' exact partial sums are added through LDS.
// A group iterates over 4 blocks at a time: a thread takes items (row, block), 4 lanes read the 64 bytes
// of codes of a row.  An item is expanded with the table of its dialect and shift and goes to LDS in MFMA
// operand order, [32-row group][pair of blocks][t][block of the pair][row][16 bytes]; the row slot is
// rotated by twice the block number, which spreads the 4 blocks of a row over the banks.  Lane (h, r) of
// the multiply reads block 2 pair + h, row r.
//
// Classes (exponent offset / 4 of a row's block, see gemm.hip) are kept per row and block.  Where a wave's
// rows have classes other than 0 in a pair of blocks, that pair takes further products, rows of other
// classes zeroed, into a second set of accumulators (class sum 1, weight 16; class sum 2 is added there
// shifted).  Whether the tile can be summed in int32 is decided from the rows' exponents:
// 32 * 120^2 * sum over blocks of 16^(class of A + class of W) must stay below 2^31 for every output.  Bounds of
// rising cost: the largest classes of the tile in every block; the blocks of every row against the largest class of the
// other operand (where that is 0 it is as good as the next; it also takes many rows whose high blocks lie in different
// places); the classes that meet in every block (of the tile's own rows; on prepared operands of 512 x 128 outputs, from masks).  A tile that
// passes none is computed with one fp32 scale-and-add per block.
#pragma once
#include <type_traits>
#include "gemm_common.h"

namespace dfp4 {
namespace {


// ONCE: K is one iteration (attention scores: heads of 64 or 128).  Such a tile is all latency (exponents, codes, LDS,
// stores), so what counts is tiles in flight: one operand buffer instead of two, and one set of accumulators (class
// sums from the highest down, shifted in between), so that three workgroups share a compute unit instead of two.
// Q K^T to fp32 (microseconds; before: a kernel of 512 x 128 tiles with its prepass / the 128 x 128 shape with two buffers):
//   128 heads, 2048 x 2048 x 128    568 / 566 -> 502      the same with heads of 64    545 / 540 -> 371 (5.9 TB/s)
//    16 heads,  700 x 1312 x  64     45 /  28 ->  21       32 heads, 300 x 2048 x 128   54 /  32 ->  26
// The write of the scores is 313 us of the first (a fill of the same size); classes on both operands, up to four
// products per pair of blocks, are most of the rest.
template <int TI_, int TJ_, int WM_, int WN_, int KG_, bool ONCE_ = false>
struct DirectShape {
    static constexpr bool kOnce = ONCE_;
    static constexpr int TI = TI_, TJ = TJ_, WM = WM_, WN = WN_, KG = KG_;
    static constexpr int kGroupThreads = 64 * WM * WN, kThreads = kGroupThreads * KG;
    static constexpr int kTm = 32 * TI * WM, kTn = 32 * TJ * WN, kRows = kTm + kTn, kRowGroups = kRows / 32;
    static constexpr int kItemRows = kGroupThreads / 4;                // rows of one item index
    static constexpr int kItems = kRows / kItemRows, kItemsA = kTm / kItemRows;
    static constexpr bool kPrivate = WM * WN == 1;                     // the group is one wave: no barrier in the loop
    static constexpr int kBufs = kPrivate || kOnce ? 1 : 2;
    static constexpr int kWavesPerSimd = TI * TJ == 1 ? 4 : kOnce ? 3 : 2;         // what the registers allow
    static constexpr int scan_parts() {                                // threads that look for a row's smallest exponent
        int p = 1;
        while (p * 2 * kRows <= kThreads && p < 16) p *= 2;
        return p;
    }
    static_assert(kItemsA * kItemRows == kTm && kItems * kItemRows == kRows, "an item is of one operand");
    static_assert(TI * TJ * 16 % KG == 0, "the groups share the outputs of a tile evenly");
};

template <class S>
struct DirectLds {
    __attribute__((aligned(16))) uint8_t x[S::KG][S::kBufs][S::kRowGroups * 4096];   // expanded operands: groups of A, of W
    __attribute__((aligned(16))) uint32_t tab[kDialects * 16 + 4];     // [dialect][shift] tables, the all-zero table
    uint8_t cls[S::KG][S::kBufs][4][S::kRows];                         // class of (block, row), rows of A then of W
    __attribute__((aligned(4))) uint8_t mn[S::kRows];                  // reference exponent of every row
    int spread[2];                                                     // largest exponent offset of A, of W
    int weight[2];                                                     // largest sum of 16^class over a row of A, of W
    int met;                                                           // sum of 16^(class sum) over the pairs that meet
};

// What a block adds to the bound on a tile's sums, from the classes present among the rows of A and of W (bits);
// more than the bound where a class sum beyond kMaxClass meets
__device__ __forceinline__ int block_weight(uint32_t ma, uint32_t mw) {
    int weight = 0;
    if (31 - __builtin_clz(ma | 1u) + 31 - __builtin_clz(mw | 1u) > kMaxClass) weight = kIntBound + 1;
#pragma unroll
    for (int ct = 0; ct <= kMaxClass; ++ct)
#pragma unroll
        for (int c = 0; c <= ct; ++c)
            if (((ma >> c) & 1u) && ((mw >> (ct - c)) & 1u)) weight += 1 << (4 * ct);
    return weight;
}

// Of prepared operands: the classes of the 512 x 128 outputs that contain (m0, n0), from their masks; of this thread's blocks of K
// the highest class of A and of W, and their weight
template <int THREADS>
__device__ __forceinline__ void mask_weights(const GemmParams& p, int m0, int n0, int& ha, int& hw, int& weight) {
    const int KB = p.KB, group = m0 / 512 * 4, groups = min(4, (p.M + 127) / 128 - group);
    const uint8_t *mask_a = p.mask_a + (int64_t)group * KB, *mask_w = p.mask_w + (int64_t)(n0 / 128) * KB;
    for (int kb = threadIdx.x; kb < KB; kb += THREADS) {
        uint32_t ma = 0;
        for (int i = 0; i < groups; ++i) ma |= mask_a[(int64_t)i * KB + kb];
        const uint32_t mw = mask_w[kb];
        ha = max(ha, 31 - __builtin_clz(ma | 1u));
        hw = max(hw, 31 - __builtin_clz(mw | 1u));
        weight += block_weight(ma, mw);
    }
}

template <class S>
union TileLds {
    DirectLds<S> d;
    SmallTileLds<S::kThreads / 64, S::kOnce ? kDirectOnceBlocks : kSmallMaxKB> small;      // declined tiles
};

// The tile (by, bx) of problem bz, by the S::kThreads threads of a workgroup; `u` is theirs alone, and a barrier lies between two calls
template <bool MX, bool BF16, class S>
__device__ __forceinline__ void int8_tile(const GemmParams& p, TileLds<S>& u, int64_t bz, int by, int bx) {
    constexpr int TI = S::TI, TJ = S::TJ;
    DirectLds<S>& lds = u.d;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6) % (S::WM * S::WN);
    const int kg = __builtin_amdgcn_readfirstlane(tid >> 6) / (S::WM * S::WN);
    const int gt = tid % S::kGroupThreads;
    const int KB = p.KB;
    const int m0 = by * S::kTm, n0 = bx * S::kTn;

    // ---- items of this thread: rows kItemRows j + r4 (the first kItemsA of A), block b4 of the iteration
    const int b4 = gt & 3, r4 = gt >> 2;
    const int per = ((KB + S::KG - 1) / S::KG + 3) & ~3;               // blocks per group
    const int k_lo = kg * per;
    const int64_t a_blk0 = bz * p.strideA_rows * KB, w_blk0 = bz * p.strideW_rows * KB;
    const uint8_t *ac = p.a_codes + a_blk0 * 16, *wc = p.w_codes + w_blk0 * 16;              // uniform bases,
    const uint8_t *ae = p.a_exp + a_blk0, *we = p.w_exp + w_blk0;                            // 32-bit offsets
    const uint8_t *ad = MX ? nullptr : p.a_dial + a_blk0, *wd = MX ? nullptr : p.w_dial + w_blk0;
    uint32_t blk[S::kItems];                                           // first block of item j's row
#pragma unroll
    for (int j = 0; j < S::kItems; ++j) {
        const int row = j * S::kItemRows + r4;
        blk[j] = (uint32_t)(j < S::kItemsA ? min(m0 + row, p.M - 1) : min(n0 + row - S::kTm, p.N - 1)) * (uint32_t)KB;
    }
    struct Item { uint4 c; uint32_t e, d; };
    Item item[S::kItems];                                              // of the next iteration
    auto load = [&](Item& it, int j, int kb0) {
        const uint32_t i = blk[j] + (uint32_t)min(kb0 + b4, KB - 1);   // blocks beyond K read the row's last
        it.c = *reinterpret_cast<const uint4*>((j < S::kItemsA ? ac : wc) + (uint64_t)(i * 16u));
        it.e = (j < S::kItemsA ? ae : we)[i];
        it.d = MX ? 7u : (uint32_t)(j < S::kItemsA ? ad : wd)[i];
    };
    if (KB > 0) {
#pragma unroll
        for (int j = 0; j < S::kItems; ++j) load(item[j], j, k_lo);
    }

    // ---- reference exponents, and whether the tile can be summed in int32
    for (int i = tid; i < kDialects * 16 + 4; i += S::kThreads) lds.tab[i] = i < kDialects * 16 ? (&g_shifted_book.w[0][0][0])[i] : 0u;
    if (tid < 2) {
        lds.spread[tid] = 0;
        lds.weight[tid] = 0;
        lds.met = 0;
    }
    int ca_max, cw_max, ref[S::kItems];
    bool declined;
    if (p.ref_a) {
        // prepared operands: the references are there, and whether a tile is taken is decided per 512 x 128 outputs from
        // the prepared masks
        for (int i = tid; i < S::kRows; i += S::kThreads)
            lds.mn[i] = i < S::kTm ? p.ref_a[min(m0 + i, p.M - 1)] : p.ref_w[min(n0 + i - S::kTm, p.N - 1)];
        int ha = 0, hw = 0, weight = 0;
        __syncthreads();
        mask_weights<S::kThreads>(p, m0, n0, ha, hw, weight);
        if (ha) atomicMax(&lds.spread[0], 4 * ha);
        if (hw) atomicMax(&lds.spread[1], 4 * hw);
        if (weight) atomicAdd(&lds.met, weight);
        __syncthreads();
        ca_max = __builtin_amdgcn_readfirstlane(lds.spread[0]) >> 2;
        cw_max = __builtin_amdgcn_readfirstlane(lds.spread[1]) >> 2;
        declined = lds.met > kIntBound;
    } else {
        // kParts threads per row look through its exponents (rows beyond the operand repeat its last)
        constexpr int kParts = S::scan_parts();
        const int srow = tid / kParts, part = tid % kParts;
        const bool is_a = srow < S::kTm, is_row = srow < S::kRows;
        const int64_t own_row = is_a ? bz * p.strideA_rows + min(m0 + srow, p.M - 1)
                                     : bz * p.strideW_rows + min(n0 + srow - S::kTm, p.N - 1);
        const uint8_t* erow = (is_a ? p.a_exp : p.w_exp) + own_row * KB;
        int mn = 255, mx = 0;
        const int n16 = KB >> 4;
        auto span = [&](uint32_t v) {
            mn = min(mn, min_bytes(v));
            mx = max(mx, max_bytes(v));
        };
        if (is_row) {
            for (int i0 = part; i0 < n16; i0 += 4 * kParts) {
                uint4 v[4];
#pragma unroll
                for (int q = 0; q < 4; ++q)                            // no alignment assumed
                    __builtin_memcpy(&v[q], erow + 16 * min(i0 + q * kParts, n16 - 1), 16);
#pragma unroll
                for (int q = 0; q < 4; ++q) { span(v[q].x); span(v[q].y); span(v[q].z); span(v[q].w); }
            }
            if (KB >= 4) {                                             // the last up to 15 bytes: dwords, the last overlapping
                uint32_t v[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) __builtin_memcpy(&v[q], erow + min(n16 * 16 + 4 * q, KB - 4), 4);
#pragma unroll
                for (int q = 0; q < 4; ++q) span(v[q]);
            } else {
                for (int i = 0; i < KB; ++i) span(erow[i] * 0x01010101u);
            }
#pragma unroll
            for (int o = 1; o < kParts; o <<= 1) {
                mn = min(mn, __shfl_xor(mn, o));
                mx = max(mx, __shfl_xor(mx, o));
            }
            if (part == 0) lds.mn[srow] = (uint8_t)mn;
        }
        __syncthreads();
        if (is_row && part == 0) atomicMax(&lds.spread[is_a ? 0 : 1], mx - mn);
        __syncthreads();
        ca_max = __builtin_amdgcn_readfirstlane(lds.spread[0]) >> 2;
        cw_max = __builtin_amdgcn_readfirstlane(lds.spread[1]) >> 2;
        const bool can = max(ca_max, cw_max) <= kMaxClass && KB <= kIntBound;
        declined = !can || ca_max + cw_max > kMaxClass || (KB << (4 * (ca_max + cw_max))) > kIntBound;
        // the classes of every row's own blocks against the largest class of the other operand
        auto weigh_rows = [&] {
            if (is_row) {
                int weight = 0;
                for (int i = part; i < n16; i += kParts) {
                    uint4 v;
                    __builtin_memcpy(&v, erow + 16 * i, 16);
                    const uint32_t w4[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                    for (int k = 0; k < 16; ++k) weight += 1 << (((int)((w4[k >> 2] >> (8 * (k & 3))) & 0xffu) - mn) & ~3);
                }
                for (int i = n16 * 16 + part; i < KB; i += kParts) weight += 1 << (((int)erow[i] - mn) & ~3);
#pragma unroll
                for (int o = 1; o < kParts; o <<= 1) weight += __shfl_xor(weight, o);
                if (part == 0) atomicMax(&lds.weight[is_a ? 0 : 1], weight << (4 * (is_a ? cw_max : ca_max)));
            }
            __syncthreads();
            declined = min(lds.weight[0], lds.weight[1]) > kIntBound;
        };
        auto weigh_met = [&] {
            // The classes that meet in every block: 8 lanes take 4 blocks, each an eighth of the rows of A and of W, and
            // OR the bits of the classes they find (A's in the low half of a block's byte).  Few outlier channels on both
            // operands end here, all of them from K = 8864.  700 x 4096 x 4096, 0.5 % of the channels of W x 20: 465 us with
            // every such tile declined, 65 so.  It is a chain of latencies: 16 x 4096 x 4096 13.7 us, 10.2 without classes on W.
            int weight = 0;
            if (KB >= 4) {
                const int part8 = tid & 7;
                for (int i = tid >> 3; 4 * i < KB; i += S::kThreads / 8) {
                    const int left = min(KB - 4 * i, 4), at = min(4 * i, KB - 4);      // the last of K with those before them
                    uint32_t met = 0;
                    auto present = [&](const uint8_t* e, int64_t row0, int last, int r0, const uint8_t* ref, int n, int shift) {
#pragma unroll 4
                        for (int j = 0; j < n; ++j) {
                            uint32_t v;
                            __builtin_memcpy(&v, e + (row0 + min(r0 + j, last)) * KB + at, 4);     // no alignment assumed
                            // offset of every byte / 4 (no offset is beyond 11) -> its bit
                            met |= __builtin_amdgcn_perm(0u, 0x00040201u, ((v - ref[j] * 0x01010101u) >> 2) & 0x03030303u) << shift;
                        }
                    };
                    constexpr int kNa = S::kTm / 8, kNw = S::kTn / 8;
                    present(p.a_exp, bz * p.strideA_rows + m0, p.M - 1 - m0, part8 * kNa, &lds.mn[part8 * kNa], kNa, 0);
                    present(p.w_exp, bz * p.strideW_rows + n0, p.N - 1 - n0, part8 * kNw, &lds.mn[S::kTm + part8 * kNw], kNw, 4);
#pragma unroll
                    for (int o = 1; o < 8; o <<= 1) met |= (uint32_t)__shfl_xor((int)met, o);
                    met >>= 8 * (4 - left);
                    if (part8 < left) weight += block_weight((met >> (8 * part8)) & 15u, (met >> (8 * part8 + 4)) & 15u);
                }
            } else {                                                   // up to 3 blocks: a bit per (block, class); the rows' weights are not in use
                if (is_row && part == 0)
                    for (int k = 0; k < KB; ++k) atomicOr(&lds.weight[is_a ? 0 : 1], 1 << (8 * k + ((erow[k] - mn) >> 2)));
                __syncthreads();
                if (tid < KB) weight = block_weight((lds.weight[0] >> (8 * tid)) & 15, (lds.weight[1] >> (8 * tid)) & 15);
            }
            if (weight) atomicAdd(&lds.met, weight);
            __syncthreads();
            declined = lds.met > kIntBound;
        };
        // With classes on both operands the rows are looked at first where K is short (24 x 2904 x 1600: 9.3 us, after the
        // blocks 9.9), the blocks that meet first otherwise (16 x 4096 x 4096: 13.7, after the rows 14.4).  One copy of
        // either, out of the way of the tiles that need neither.
        if (can && declined) {
            // a row with a single block of its operand's largest class, the least that can be found
            const bool rows_may = ca_max + cw_max <= kMaxClass && min((KB - 1 + (1 << (4 * ca_max))) << (4 * cw_max),
                                                                      (KB - 1 + (1 << (4 * cw_max))) << (4 * ca_max)) <= kIntBound;
            const bool both = min(ca_max, cw_max) > 0, rows_first = !both || KB <= 64;
#pragma unroll 1
            for (int pass = 0; pass < 2 && declined; ++pass) {
                if ((pass == 0) == rows_first) {
                    if (rows_may) weigh_rows();
                } else if (both) {
                    weigh_met();
                }
            }
        }
    }
#pragma unroll
    for (int j = 0; j < S::kItems; ++j) ref[j] = lds.mn[j * S::kItemRows + r4];
    if (declined) {                               // the same for every thread
        // counted once per 512 x 128 tile where that is what the masks decide, once per tile otherwise
        if (p.declined && tid == 0 && (!p.ref_a || (m0 % 512 == 0 && n0 % 128 == 0))) atomicAdd(p.declined, 1u);
        __syncthreads();
        if constexpr (S::kTm % 128 == 0 && S::kTn == 128) {
            // 128 rows by each 4 waves (with two groups both compute the same rows: same values)
            constexpr int kPieces = S::kTm / 128;
            uint8_t (&s_exp)[2][256] = *reinterpret_cast<uint8_t (*)[2][256]>(&lds.x[0][0][0] + (tid >> 8) * 512);
            block_flush_tile<MX, BF16>(p, bz, by * kPieces + (tid >> 8) % kPieces, bx, s_exp);
        } else {
            for (int i = 0; i < S::kTm / 32; ++i)
                for (int j = 0; j < S::kTn / 32; ++j) {
                    if (m0 + 32 * i >= p.M || n0 + 32 * j >= p.N) continue;
                    small_tile<MX, BF16>(p, bz, m0 + 32 * i, n0 + 32 * j, u.small);
                    __syncthreads();
                }
        }
        return;
    }

    const int wm = wave / S::WN, wn = wave % S::WN, h = lane >> 5, r = lane & 31;
    const v16i zero16 = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    const v4i zero4 = {0, 0, 0, 0};
    v16i acc[TI][TJ], acc1[TI][TJ];                                    // class sum 0; class sums above 0 (weight 16)
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j) acc[i][j] = acc1[i][j] = zero16;
    // Item j of the iteration at kb0: the table of its dialect and shift, then the expansion into a buffer.
    auto table = [&](const Item& it, int j, int kb0) {
        const uint32_t t = kb0 + b4 < KB ? ((it.d & 15u) * 4u + ((it.e - (uint32_t)ref[j]) & 3u)) * 16u : kZeroTab;
        return *reinterpret_cast<const uint4*>(reinterpret_cast<const uint8_t*>(lds.tab) + t);
    };
    uint8_t* slot = &lds.x[kg][0][0] + (b4 >> 1) * 2048 + (b4 & 1) * 512;
    auto expand = [&](const Item& it, int j, uint4 tab, int buf) {
        const int row = j * S::kItemRows + r4;
        uint8_t* dst = slot + buf * (S::kRowGroups * 4096) + (row >> 5) * 4096 + ((row + 2 * b4) & 31) * 16;
        *reinterpret_cast<v4i*>(dst) = unpack16(it.c.x, it.c.y, tab);
        *reinterpret_cast<v4i*>(dst + 1024) = unpack16(it.c.z, it.c.w, tab);
        lds.cls[kg][buf][b4][row] = (uint8_t)((it.e - (uint32_t)ref[j]) >> 2);
    };
    auto only = [&](bool keep, const v4i (&v)[2], v4i (&o)[2]) {
        o[0] = keep ? v[0] : zero4;
        o[1] = keep ? v[1] : zero4;
    };
    struct Operands { v4i a[TI][2], b[TJ][2]; int ka[TI], kw[TJ]; };   // of a pair, with the class of the lane's row / column
    auto read = [&](Operands& o, int buf, int pr) {
        const int kb = 2 * pr + h;
        const uint8_t* src = &lds.x[kg][buf][0] + pr * 2048 + h * 512 + ((r + 2 * kb) & 31) * 16;
        const uint8_t* cls = &lds.cls[kg][buf][kb][0] + r;
#pragma unroll
        for (int i = 0; i < TI; ++i) {
            o.ka[i] = cls[(TI * wm + i) * 32];
            o.a[i][0] = *reinterpret_cast<const v4i*>(src + (TI * wm + i) * 4096);
            o.a[i][1] = *reinterpret_cast<const v4i*>(src + (TI * wm + i) * 4096 + 1024);
        }
#pragma unroll
        for (int j = 0; j < TJ; ++j) {
            o.kw[j] = cls[S::kTm + (TJ * wn + j) * 32];
            o.b[j][0] = *reinterpret_cast<const v4i*>(src + (S::kTm / 32 + TJ * wn + j) * 4096);
            o.b[j][1] = *reinterpret_cast<const v4i*>(src + (S::kTm / 32 + TJ * wn + j) * 4096 + 1024);
        }
    };
    auto multiply = [&](Operands& o) {
        int any_cls = 0;
#pragma unroll
        for (int i = 0; i < TI; ++i) any_cls |= o.ka[i];
#pragma unroll
        for (int j = 0; j < TJ; ++j) any_cls |= o.kw[j];
        if (__ballot(any_cls != 0) != 0ull) {
            if (ca_max + cw_max >= 2) {
#pragma unroll
                for (int i = 0; i < TI; ++i)
#pragma unroll
                    for (int j = 0; j < TJ; ++j) {
                        v16i s = zero16;
                        bool any = false;
#pragma unroll 1
                        for (int c1 = 0; c1 <= 2; ++c1) {
                            if (__ballot(o.ka[i] == c1) == 0ull || __ballot(o.kw[j] == 2 - c1) == 0ull) continue;
                            v4i x[2], y[2];
                            only(o.ka[i] == c1, o.a[i], x);
                            only(o.kw[j] == 2 - c1, o.b[j], y);
#pragma unroll
                            for (int t = 0; t < 2; ++t) s = __builtin_amdgcn_mfma_i32_32x32x32_i8(x[t], y[t], s, 0, 0, 0);
                            any = true;
                        }
                        if (any) {
#pragma unroll
                            for (int x = 0; x < 16; ++x) acc1[i][j][x] += s[x] << 4;
                        }
                    }
            }
#pragma unroll
            for (int j = 0; j < TJ; ++j)
                if (__ballot(o.kw[j] != 0) != 0ull) {
                    v4i x[TI][2], y[2];
                    only(o.kw[j] == 1, o.b[j], y);
                    only(o.kw[j] == 0, o.b[j], o.b[j]);
#pragma unroll
                    for (int i = 0; i < TI; ++i) only(o.ka[i] == 0, o.a[i], x[i]);
#pragma unroll
                    for (int t = 0; t < 2; ++t)
#pragma unroll
                        for (int i = 0; i < TI; ++i)
                            acc1[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(x[i][t], y[t], acc1[i][j], 0, 0, 0);
                }
#pragma unroll
            for (int i = 0; i < TI; ++i)
                if (__ballot(o.ka[i] != 0) != 0ull) {
                    v4i x[2];
                    only(o.ka[i] == 1, o.a[i], x);
#pragma unroll
                    for (int t = 0; t < 2; ++t)
#pragma unroll
                        for (int j = 0; j < TJ; ++j)
                            acc1[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(x[t], o.b[j][t], acc1[i][j], 0, 0, 0);
                    only(o.ka[i] == 0, o.a[i], o.a[i]);
                }
        }
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int i = 0; i < TI; ++i)
#pragma unroll
                for (int j = 0; j < TJ; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(o.a[i][t], o.b[j][t], acc[i][j], 0, 0, 0);
    };
    if constexpr (S::kOnce) {
        if (KB > 0) {
#pragma unroll
            for (int j = 0; j < S::kItems; ++j) expand(item[j], j, table(item[j], j, 0), 0);
        }
        __syncthreads();
        const int top = min(ca_max + cw_max, kMaxClass);               // higher sums do not meet
#pragma unroll 1
        for (int ct = top; ct >= 0; --ct) {
            if (ct < top) {
#pragma unroll
                for (int i = 0; i < TI; ++i)
#pragma unroll
                    for (int j = 0; j < TJ; ++j)
#pragma unroll
                        for (int x = 0; x < 16; ++x) acc[i][j][x] <<= 4;
            }
#pragma unroll 1
            for (int c1 = max(0, ct - cw_max); c1 <= min(ct, ca_max); ++c1)
#pragma unroll 1
                for (int pr = 0; 2 * pr < KB; ++pr) {
                    Operands o;
                    read(o, 0, pr);
                    bool any_a[TI], any_b[TJ];
#pragma unroll
                    for (int i = 0; i < TI; ++i) {
                        any_a[i] = __ballot(o.ka[i] == c1) != 0ull;
                        only(o.ka[i] == c1, o.a[i], o.a[i]);
                    }
#pragma unroll
                    for (int j = 0; j < TJ; ++j) {
                        any_b[j] = __ballot(o.kw[j] == ct - c1) != 0ull;
                        only(o.kw[j] == ct - c1, o.b[j], o.b[j]);
                    }
#pragma unroll
                    for (int i = 0; i < TI; ++i)
#pragma unroll
                        for (int j = 0; j < TJ; ++j)
                            if (any_a[i] && any_b[j]) {
#pragma unroll
                                for (int t = 0; t < 2; ++t)
                                    acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(o.a[i][t], o.b[j][t], acc[i][j], 0, 0, 0);
                            }
                }
        }
    } else if constexpr (S::kPrivate) {
        // one wave: its LDS operations execute in order, so lanes exchange operands without a barrier; the fences keep
        // the compiler to that order (they cost no instruction).  4 waves per SIMD hide the latencies
        auto in_order = [] {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        };
        for (int k = 0; k < per; k += 4) {
            const int kb0 = k_lo + k;
            if (kb0 >= KB) break;
#pragma unroll
            for (int j = 0; j < S::kItems; ++j) {
                expand(item[j], j, table(item[j], j, kb0), 0);
                load(item[j], j, kb0 + 4);
            }
            in_order();
#pragma unroll
            for (int pr = 0; pr < 2; ++pr) {
                Operands o;
                read(o, 0, pr);
                multiply(o);
            }
            in_order();
        }
    } else {
        // One iteration: multiply the 4 blocks from kb0 (buffer BUF), expand the next 4 into the other buffer,
        // load the 4 after those.  A wave issues the LDS reads of a pair's operands, expands while they are on
        // their way, then multiplies.
        auto iteration = [&](auto buf_c, int k) {
            constexpr int kBuf = decltype(buf_c)::value, kNxt = 1 - kBuf, kHalf = S::kItems / 2;
            const bool more = k + 4 < per;
#pragma unroll
            for (int pr = 0; pr < 2; ++pr) {
                const int j_lo = pr == 0 ? 0 : kHalf, j_hi = pr == 0 ? kHalf : S::kItems;
                uint4 tab[S::kItems];
                if (more) {
#pragma unroll
                    for (int j = j_lo; j < j_hi; ++j) tab[j] = table(item[j], j, k_lo + k + 4);
                }
                Operands o;
                read(o, kBuf, pr);
                __builtin_amdgcn_sched_barrier(0);
                if (more) {
#pragma unroll
                    for (int j = j_lo; j < j_hi; ++j) {
                        expand(item[j], j, tab[j], kNxt);
                        load(item[j], j, k_lo + k + 8);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
                multiply(o);
                __builtin_amdgcn_sched_barrier(0);
            }
            __syncthreads();
        };
        if (KB > 0) {
#pragma unroll
            for (int j = 0; j < S::kItems; ++j) {
                expand(item[j], j, table(item[j], j, k_lo), 0);
                load(item[j], j, k_lo + 4);
            }
            __syncthreads();
            for (int k = 0; k < per; k += 8) {
                iteration(std::integral_constant<int, 0>{}, k);
                if (k + 4 >= per) break;
                iteration(std::integral_constant<int, 1>{}, k + 4);
            }
        }
    }
    if (!S::kOnce && ca_max + cw_max > 0) {
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j)
#pragma unroll
                for (int x = 0; x < 16; ++x) acc[i][j][x] += acc1[i][j][x] << 4;
    }

    // ---- the one rounding: int32 -> fp32, scaled by 2^(refA + refW - 2)
    constexpr int kEsz = BF16 ? 2 : 4;
    const int row0 = m0 + wm * 32 * TI, col0 = n0 + wn * 32 * TJ;      // of this wave
    if constexpr (S::KG > 1) {
        // the groups' exact partial sums, added through LDS; group kg finishes its share of the tile's outputs
        constexpr int kOut = TI * TJ * 16, kShare = kOut / S::KG;
        static_assert(sizeof(int) * S::KG * S::WM * S::WN * kOut * 64 <= sizeof(lds.x), "partial tiles reuse the operands");
        __syncthreads();
        int* red = reinterpret_cast<int*>(&lds.x[0][0][0]);
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j)
#pragma unroll
                for (int x = 0; x < 16; ++x)
                    red[((kg * S::WM * S::WN + wave) * kOut + (i * TJ + j) * 16 + x) * 64 + lane] = acc[i][j][x];
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kShare; ++q) {
            const int o = kg * kShare + q, i = o / (16 * TJ), j = o / 16 % TJ, x = o % 16;
            int sum = 0;
#pragma unroll
            for (int g = 0; g < S::KG; ++g) sum += red[((g * S::WM * S::WN + wave) * kOut + o) * 64 + lane];
            const int lr = 32 * i + 8 * (x >> 2) + 4 * h + (x & 3), lc = 32 * j + r;
            if (row0 + lr < p.M && col0 + lc < p.N) {
                const float f = ldexpf((float)sum, (int)lds.mn[wm * 32 * TI + lr] + (int)lds.mn[S::kTm + wn * 32 * TJ + lc] - 256);
                const int64_t at = bz * p.strideC + (int64_t)(row0 + lr) * p.ldc + col0 + lc;
                if constexpr (BF16) static_cast<uint16_t*>(p.out)[at] = f32_to_bf16_rne(f);
                else static_cast<float*>(p.out)[at] = f;
            }
        }
    } else {
        if (row0 >= p.M || col0 >= p.N) return;
        uint8_t* wave_out = static_cast<uint8_t*>(p.out) + (bz * p.strideC + (int64_t)row0 * p.ldc + col0) * kEsz;
        const int64_t row_bytes = p.ldc * kEsz;
        const bool full = row0 + 32 * TI <= p.M && col0 + 32 * TJ <= p.N;
        // bf16: every lane stores two adjacent columns of one row (as in gemm_native_kernel)
        const bool pairs = BF16 && full && (p.ldc & 1) == 0 && ((p.strideC * kEsz) & 3) == 0 &&
                           (reinterpret_cast<uintptr_t>(p.out) & 3) == 0;
        const uint32_t lane_off = pairs ? (uint32_t)((4 * h + (r & 1)) * row_bytes + (r & ~1) * kEsz)
                                        : (uint32_t)(4 * h * row_bytes + r * kEsz);
        auto store = [&](auto full_c, auto pairs_c) {
            constexpr bool kFull = decltype(full_c)::value, kPairs = decltype(pairs_c)::value;
#pragma unroll
            for (int i = 0; i < TI; ++i)
#pragma unroll
                for (int j = 0; j < TJ; ++j) {
                    const int ew = (int)lds.mn[S::kTm + (wn * TJ + j) * 32 + r] - 256;
                    uint8_t* tile_out = wave_out + (int64_t)i * 32 * row_bytes + j * 32 * kEsz;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const uint32_t e4 = *reinterpret_cast<const uint32_t*>(&lds.mn[(wm * TI + i) * 32 + 8 * q + 4 * h]);
                        float f[4];
#pragma unroll
                        for (int x = 0; x < 4; ++x)
                            f[x] = ldexpf((float)acc[i][j][4 * q + x], (int)((e4 >> (8 * x)) & 0xffu) + ew);
                        uint8_t* rowp = tile_out + (int64_t)(8 * q) * row_bytes;
                        if constexpr (kPairs) {
#pragma unroll
                            for (int x = 0; x < 4; x += 2) {
                                const uint32_t b0 = f32_to_bf16_rne(f[x]), b1 = f32_to_bf16_rne(f[x + 1]);
                                const uint32_t send = (r & 1) ? b0 : b1;
                                const uint32_t recv = (uint32_t)__builtin_amdgcn_mov_dpp((int)send, 0xB1, 0xf, 0xf, true);
                                const uint32_t word = (r & 1) ? (recv | (b1 << 16)) : (b0 | (recv << 16));
                                DFP4_OUT_STORE(reinterpret_cast<uint32_t*>(rowp + (int64_t)x * row_bytes + lane_off), word);
                            }
                        } else {
#pragma unroll
                            for (int x = 0; x < 4; ++x) {
                                if (kFull || (row0 + i * 32 + 8 * q + 4 * h + x < p.M && col0 + j * 32 + r < p.N)) {
                                    uint8_t* dst = rowp + (int64_t)x * row_bytes + lane_off;
                                    if constexpr (BF16) DFP4_OUT_STORE(reinterpret_cast<uint16_t*>(dst), f32_to_bf16_rne(f[x]));
                                    else DFP4_OUT_STORE(reinterpret_cast<float*>(dst), f[x]);
                                }
                            }
                        }
                    }
                }
        };
        if (BF16 && pairs) store(std::true_type{}, std::integral_constant<bool, BF16>{});
        else if (full) store(std::true_type{}, std::false_type{});
        else store(std::false_type{}, std::false_type{});
    }
}

}  // namespace
}  // namespace dfp4
