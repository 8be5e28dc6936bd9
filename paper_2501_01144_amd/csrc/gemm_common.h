// Shared by the GEMM kernels (gemm.hip, gemm_f8.hip, gemm_native.hip): operand tables, the expansion of 4-bit codes
// to int8, launch parameters, and the tiles computed with one fp32 scale-and-add per block.
#pragma once
#include <type_traits>
#include "common.h"
#include "formatbook.h"

namespace dfp4 {

// [dialect][shift] -> {magnitudes lo, hi, negated magnitudes lo, hi}, bytes u << shift
struct ShiftedBook { uint32_t w[kDialects][4][4]; };
constexpr ShiftedBook make_shifted_book() {
    ShiftedBook b{};
    for (int d = 0; d < kDialects; ++d)
        for (int s = 0; s < 4; ++s)
            for (int j = 0; j < 8; ++j) {
                const uint32_t u = (uint32_t)kBook[d][j] << s;
                b.w[d][s][j / 4] |= u << (8 * (j % 4));
                b.w[d][s][2 + j / 4] |= ((256u - u) & 0xffu) << (8 * (j % 4));
            }
    return b;
}
static __device__ const ShiftedBook g_shifted_book = make_shifted_book();

struct GemmParams {
    const uint8_t *a_codes, *a_dial, *a_exp, *w_codes, *w_dial, *w_exp;
    void* out;
    int M, N, KB;
    int64_t ldc, strideA_rows, strideW_rows, strideC;
    // prepared operands (per problem of a batch: base + problem * stride; gemm_native.hip)
    uint8_t* a_prep;
    uint8_t* w_prep;
    int64_t a_prep_stride, w_prep_stride;
    // prepared operands in gemm_f8_kernel (batch 1; otherwise null): smallest exponent of every row, and per (128 rows,
    // block) the classes present
    const uint8_t *ref_a, *mask_a, *ref_w, *mask_w;
    uint32_t* declined;               // counts tiles computed with one fp32 scale-and-add per block (may be null)
    // requantizing epilogue: the quantized [M, N] output (blocks of 32 along N)
    uint32_t* q_codes;
    uint8_t *q_dial, *q_exp;
};

constexpr int kDirectOnceBlocks = 4;         // K, in blocks, that the direct kernels take in one iteration

namespace {

// Results leave the kernel once and are not read again by it: stored with the non-temporal hint so
// that they do not push the operands other workgroups still need out of the caches.
#if defined(DFP4_TIMING_NO_OUT_STORES)   // timing experiments only: results are computed and dropped
__device__ int g_timing_store_results = 0;
#define DFP4_OUT_STORE(PTR, VAL) do { if (g_timing_store_results) *(PTR) = (VAL); } while (0)
#elif defined(DFP4_PLAIN_OUT_STORES)
#define DFP4_OUT_STORE(PTR, VAL) (*(PTR) = (VAL))
#else
#define DFP4_OUT_STORE(PTR, VAL) __builtin_nontemporal_store((VAL), (PTR))
#endif

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int kMaxClass = 2;          // classes 0..2, i.e. exponent offsets 0..11
constexpr int kIntBound = 4660;       // n0 + 16 n1 + 256 n2 <= 2^31 / (32 * 120 * 120)
constexpr uint32_t kZeroTab = kDialects * 4 * 16;   // byte offset of the all-zero table behind the shifted book in LDS


// 8 codes (one dword) -> 8 signed int8 through one dialect table:
// returns the even-numbered elements in one dword and the odd ones in another.
// Magnitudes and negated magnitudes are looked up with v_perm_b32 (selector =
// 3-bit index); the per-byte choice between them uses v_perm_b32's
// sign-replication selectors (8..11 = 0x00 / 0xff from bit 7 of bytes 1, 3, 5, 7
// of the source pair), which turn the code's sign bits into byte masks.
__device__ __forceinline__ void unpack8(uint32_t c, uint32_t plo, uint32_t phi, uint32_t nlo,
                                        uint32_t nhi, uint32_t& even, uint32_t& odd) {
    const uint32_t ie = c & 0x07070707u, io = (c >> 4) & 0x07070707u;
    const uint32_t pe = __builtin_amdgcn_perm(phi, plo, ie), po = __builtin_amdgcn_perm(phi, plo, io);
    const uint32_t ne = __builtin_amdgcn_perm(nhi, nlo, ie), no = __builtin_amdgcn_perm(nhi, nlo, io);
    // result byte k <- sign of byte k of x: bytes 1, 3 come from x, bytes 0, 2 from x << 8
    constexpr uint32_t kSignSel = 0x090b080au;
    const uint32_t c4 = c << 4;                                   // index sign bit 3 -> bit 7
    const uint32_t mo = __builtin_amdgcn_perm(c << 8, c, kSignSel);
    const uint32_t me = __builtin_amdgcn_perm(c4 << 8, c4, kSignSel);
    even = (ne & me) | (pe & ~me);
    odd = (no & mo) | (po & ~mo);
}

__device__ __forceinline__ v4i unpack16(uint32_t c0, uint32_t c1, uint4 tab) {
    uint32_t a, b, e, f;
    unpack8(c0, tab.x, tab.y, tab.z, tab.w, a, b);
    unpack8(c1, tab.x, tab.y, tab.z, tab.w, e, f);
    return v4i{(int)a, (int)b, (int)e, (int)f};
}

__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f) {
    uint32_t u = __builtin_bit_cast(uint32_t, f);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ __forceinline__ int min_bytes(uint32_t x) {
    return min(min((int)(x & 0xffu), (int)((x >> 8) & 0xffu)), min((int)((x >> 16) & 0xffu), (int)(x >> 24)));
}
__device__ __forceinline__ int max_bytes(uint32_t x) {
    return max(max((int)(x & 0xffu), (int)((x >> 8) & 0xffu)), max((int)((x >> 16) & 0xffu), (int)(x >> 24)));
}

// ---------------------------------------------------------------------------
// Per-block flush (always correct): 128 x 128 outputs per workgroup of 256 threads,
// operands straight from global memory, one fp32 scale-and-add per block as in the
// paper's MAC (Section 3.3).  For the tiles that the
// single-accumulator kernels decline.
// ---------------------------------------------------------------------------
template <bool MX, bool BF16>
__device__ __forceinline__ void block_flush_tile(const GemmParams& p, int64_t bz, int by, int bx,
                                                 uint8_t (&s_exp)[2][256]) {
    const int KB = p.KB;
    const int lane = threadIdx.x & 63, wave = (threadIdx.x >> 6) & 3;        // 4 waves, also where a larger workgroup calls
    const int wm = wave >> 1, wn = wave & 1;
    const int m0 = by * 128, n0 = bx * 128;
    const int64_t a_row0 = bz * p.strideA_rows, w_row0 = bz * p.strideW_rows;
    const int half = lane >> 5, l32 = lane & 31;

    int64_t a_row[2], w_row[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        a_row[i] = a_row0 + min(m0 + wm * 64 + i * 32 + l32, p.M - 1);
        w_row[i] = w_row0 + min(n0 + wn * 64 + i * 32 + l32, p.N - 1);
    }
    const int t = threadIdx.x & 255;
    const int64_t e_row = t < 128 ? a_row0 + min(m0 + t, p.M - 1) : w_row0 + min(n0 + t - 128, p.N - 1);
    const uint8_t* e_src = (t < 128 ? p.a_exp : p.w_exp) + e_row * KB;

    float acc[2][2][16];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int x = 0; x < 16; ++x) acc[i][j][x] = 0.0f;

    // operands of one block, loaded one iteration ahead so that the memory latency of block kb + 1
    // passes behind the arithmetic of block kb
    struct BlockOperands { uint2 ca[2], cw[2]; uint32_t da[2], dw[2], e; };
    auto load_block = [&](int kb) {
        BlockOperands o;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            o.ca[i] = *reinterpret_cast<const uint2*>(p.a_codes + (a_row[i] * KB + kb) * 16 + half * 8);
            o.cw[i] = *reinterpret_cast<const uint2*>(p.w_codes + (w_row[i] * KB + kb) * 16 + half * 8);
            o.da[i] = MX ? 7u : ((uint32_t)p.a_dial[a_row[i] * KB + kb] & 15u);
            o.dw[i] = MX ? 7u : ((uint32_t)p.w_dial[w_row[i] * KB + kb] & 15u);
        }
        o.e = e_src[kb];
        return o;
    };
    BlockOperands nxt{};
    if (KB > 0) nxt = load_block(0);              // K = 0: nothing to read, the outputs are zeros
    for (int kb = 0; kb < KB; ++kb) {
        const BlockOperands cur = nxt;
        if (kb + 1 < KB) nxt = load_block(kb + 1);
        uint8_t* se = s_exp[kb & 1];
        se[t] = (uint8_t)cur.e;
        v4i a[2], b[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            a[i] = unpack16(cur.ca[i].x, cur.ca[i].y, *reinterpret_cast<const uint4*>(g_shifted_book.w[cur.da[i]][0]));
            b[i] = unpack16(cur.cw[i].x, cur.cw[i].y, *reinterpret_cast<const uint4*>(g_shifted_book.w[cur.dw[i]][0]));
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                v16i pr = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
                pr = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[i], b[j], pr, 0, 0, 0);
                const int ew = se[128 + wn * 64 + j * 32 + l32];
#pragma unroll
                for (int x = 0; x < 16; ++x) {
                    const int row = 8 * (x >> 2) + 4 * half + (x & 3);
                    const int ea = se[wm * 64 + i * 32 + row];
                    acc[i][j][x] += ldexpf((float)pr[x], ea + ew - 256);
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
                    const int64_t o = bz * p.strideC + (int64_t)m * p.ldc + n;
                    if constexpr (BF16)
                        static_cast<uint16_t*>(p.out)[o] = f32_to_bf16_rne(acc[i][j][x]);
                    else
                        static_cast<float*>(p.out)[o] = acc[i][j][x];
                }
            }
        }
}

// ---------------------------------------------------------------------------
// A 32 x 32 output tile by a workgroup of NW (4, 8 or 16) waves that share K in contiguous ranges, one fp32
// scale-and-add per block as in the paper's MAC; the partial tiles are added in a fixed order through LDS.
// Small tiles that int8_tile declines.
// ---------------------------------------------------------------------------
constexpr int kSmallMaxKB = 512;      // LDS holds the 32 rows' exponent bytes of all blocks

template <int NW, int MAX_KB>
struct SmallTileLds {
    __attribute__((aligned(16))) uint32_t tab[kDialects * 4];   // shift-0 tables
    __attribute__((aligned(4))) uint8_t ea[MAX_KB * 32];        // [block][row] exponent bytes of A (a longer K: read where they are)
    float red[NW / 2][16][64];
};

template <bool MX, bool BF16, int NW, int MAX_KB>
__device__ __forceinline__ void small_tile(const GemmParams& p, int64_t bz, int m0, int n0, SmallTileLds<NW, MAX_KB>& lds) {
    uint32_t (&s_tab)[kDialects * 4] = lds.tab;
    uint8_t (&s_ea)[MAX_KB * 32] = lds.ea;
    float (&s_red)[NW / 2][16][64] = lds.red;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int h = lane >> 5, r = lane & 31;
    const int KB = p.KB;
    const int64_t a_row0 = bz * p.strideA_rows, w_row0 = bz * p.strideW_rows;

    const int64_t arow = a_row0 + min(m0 + r, p.M - 1), wrow = w_row0 + min(n0 + r, p.N - 1);
    const uint8_t* ac = p.a_codes + arow * KB * 16 + h * 8;
    const uint8_t* wc = p.w_codes + wrow * KB * 16 + h * 8;
    const uint8_t* ad = MX ? nullptr : p.a_dial + arow * KB;
    const uint8_t* wd = MX ? nullptr : p.w_dial + wrow * KB;
    const uint8_t* we = p.w_exp + wrow * KB;
    const int per = (KB + NW - 1) / NW;
    const int kb_lo = wave * per, kb_hi = min(KB, kb_lo + per);

    for (int i = tid; i < kDialects * 4; i += NW * 64) s_tab[i] = g_shifted_book.w[i >> 2][0][i & 3];
    const bool staged = KB <= MAX_KB;
    if (staged) {
        for (int i = tid; i < 32 * KB; i += NW * 64) {
            const int row = i / KB, kb = i - row * KB;
            s_ea[kb * 32 + row] = p.a_exp[(a_row0 + min(m0 + row, p.M - 1)) * KB + kb];
        }
    }
    __syncthreads();

    float acc[16];
#pragma unroll
    for (int x = 0; x < 16; ++x) acc[x] = 0.0f;
    constexpr int kU = 4;              // blocks whose loads are issued together
    for (int kb0 = kb_lo; kb0 < kb_hi; kb0 += kU) {
        uint2 ca[kU], cw[kU];
        uint32_t da[kU], dw[kU], ew[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int kb = min(kb0 + u, kb_hi - 1);            // the tail repeats the last block (not used)
            ca[u] = *reinterpret_cast<const uint2*>(ac + (int64_t)kb * 16);
            cw[u] = *reinterpret_cast<const uint2*>(wc + (int64_t)kb * 16);
            da[u] = MX ? 7u : ((uint32_t)ad[kb] & 15u);
            dw[u] = MX ? 7u : ((uint32_t)wd[kb] & 15u);
            ew[u] = we[kb];
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int kb = kb0 + u;
            if (kb >= kb_hi) break;                            // wave-uniform
            const v4i a = unpack16(ca[u].x, ca[u].y, *reinterpret_cast<const uint4*>(&s_tab[da[u] * 4]));
            const v4i b = unpack16(cw[u].x, cw[u].y, *reinterpret_cast<const uint4*>(&s_tab[dw[u] * 4]));
            v16i pr = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
            pr = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, pr, 0, 0, 0);
            const int ewc = (int)ew[u] - 256;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                uint32_t e4 = 0;
                if (staged) {
                    e4 = *reinterpret_cast<const uint32_t*>(&s_ea[kb * 32 + 8 * q + 4 * h]);
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        e4 |= (uint32_t)p.a_exp[(a_row0 + min(m0 + 8 * q + 4 * h + j, p.M - 1)) * KB + kb] << (8 * j);
                }
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[4 * q + j] += ldexpf((float)pr[4 * q + j], (int)((e4 >> (8 * j)) & 0xffu) + ewc);
            }
        }
    }
    // the NW partial tiles, added in a fixed order: the upper half of the waves hands theirs to the lower
    if (wave >= NW / 2) {
#pragma unroll
        for (int x = 0; x < 16; ++x) s_red[wave - NW / 2][x][lane] = acc[x];
    }
    __syncthreads();
    if (wave < NW / 2) {
#pragma unroll
        for (int x = 0; x < 16; ++x) s_red[wave][x][lane] += acc[x];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 16 / NW; ++i) {
        const int x = wave + i * NW;                           // thread (x, lane) finishes one output
        float sum = 0.0f;
#pragma unroll
        for (int w = 0; w < NW / 2; ++w) sum += s_red[w][x][lane];
        const int m = m0 + 8 * (x >> 2) + 4 * h + (x & 3), n = n0 + r;
        if (m < p.M && n < p.N) {
            const int64_t o = bz * p.strideC + (int64_t)m * p.ldc + n;
            if constexpr (BF16)
                static_cast<uint16_t*>(p.out)[o] = f32_to_bf16_rne(sum);
            else
                static_cast<float*>(p.out)[o] = sum;
        }
    }
}


template <typename F>
void dispatch_mx_bf16(bool mx, bool bf16, F&& f) {
    if (mx) {
        if (bf16) f(std::true_type{}, std::true_type{}); else f(std::true_type{}, std::false_type{});
    } else {
        if (bf16) f(std::false_type{}, std::true_type{}); else f(std::false_type{}, std::false_type{});
    }
}

}  // namespace

// gemm_native.hip: products whose operands are packed beforehand (exact_operand_bytes each; A with the counters)
constexpr int kExactSplitTiles = 2048;        // K is split only below this many tiles
constexpr int kExactCounters = kExactSplitTiles + 1;      // arrivals at every such tile, and the count of declined tiles
int64_t exact_operand_bytes(int64_t rows, int64_t KB, bool fp6, bool counters);
int64_t exact_split_bytes(int64_t M, int64_t N, int64_t KB, int64_t batch);
int launch_exact_prep(bool mx, const GemmParams& p, int64_t batch, bool classes, hipStream_t stream);
void set_prepared_classes(bool mx, GemmParams& p, const uint8_t* a_prep, const uint8_t* w_prep);
int launch_exact(bool mx, bool bf16, const GemmParams& g, int64_t batch, float* part, size_t part_bytes, bool rq, hipStream_t stream);

// gemm_f8.hip: any product of at most gemm_direct_max_rows(KB, false) rows of A and (KB, true) of W, with the operands as
// they are; a shape and the microseconds it is estimated to take on `cu` compute units
struct DirectChoice { int shape; float us; };
int launch_gemm_f8(bool mx, bool bf16, const GemmParams& p, int64_t batch, int shape, hipStream_t stream);
DirectChoice choose_direct(int64_t M, int64_t N, int64_t KB, int64_t batch, int64_t cu);
int64_t gemm_direct_max_rows(int64_t KB, bool weight);

}  // namespace dfp4
