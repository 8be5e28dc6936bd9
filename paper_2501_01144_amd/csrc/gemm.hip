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
//   gemm_native_kernel   (gemm_native.hip) large products: both operands packed for the block-scaled matrix instruction by
//                        exact_prep_kernel, once per call (dfp4_gemm) or once per tensor (dfp4_gemm_prepare), 256 x 256
//                        or 128 x 256 outputs per workgroup.  That instruction applies the exponents itself, at twice the
//                        int8 rate, and sums in fp32; the kernel keeps the result where norms of the rows show that no
//                        partial sum was rounded, and computes the tile again by the scheme above where they do not.
//                        (It replaced a kernel that ran the scheme above on operands expanded to int8 beforehand:
//                        2048 x 14336 x 4096 prepared 142 -> 83 us, 2048 x 4096 x 14336 125 -> 75, 4096 x 12288 x 4096
//                        202 -> 117; with the prepass 150 -> 100, 162 -> 108, 220 -> 144.)
//   gemm_f8_kernel       (gemm_f8.hip) both operands expanded inside the kernel to FP8 for the block-scaled instruction, under the
//                        same proof, in tiles from 32 x 32 to 256 x 128: few rows, few tiles, long K, batches whose packed A
//                        would be read only once.  Products of prepared operands of more than 256 rows that are too small for
//                        the large kernel take it too;
//   gemm_block16_kernel  operands quantized in blocks of 16: per-block fp32 flush.
//
// The order of the elements inside an MFMA operand does not matter as long
// as A and W use the same order; both sides go through unpack8() below.
#include <type_traits>
#include "common.h"
#include "formatbook.h"
#include "gemm_common.h"

namespace dfp4 {

namespace {

constexpr int kTileM = 512, kTileN = 128;   // fast_cost: tiles of the kernel it was fitted to
constexpr int kMaxKB = 512;           // prepared operands: K <= 16384

__host__ __device__ inline int64_t align256(int64_t x) { return (x + 255) & ~(int64_t)255; }

// fast_cost: workgroups per output tile
inline int choose_ksplit(int64_t tiles, int64_t KB, int64_t cu) {
    int s = 1;
    while (s < 8 && tiles * s * 2 <= cu && KB / (2 * s) >= 16) s *= 2;
    return tiles <= kExactSplitTiles ? s : 1;
}
// Which kernel.  The large kernel multiplies packed operands; gemm_f8_kernel ("direct") expands in the kernel and
// takes everything the large one is not for (few rows, K beyond 16384), and the products it is estimated to finish sooner:
// those with few output tiles, and batches whose packed A would be read only once or twice (P V of attention).  K of one
// iteration of the direct kernel (Q K^T) goes there unless it is prepared already.  fast_cost is of the int8 kernel that
// the large one replaced and choose_direct's estimates of int8 operands, so the line lies where it lay between those two.  The
// large kernel gained more than the direct one, which leaves products on the direct side that it would finish sooner, up to
// 1.7 times (microseconds, large with its prepass / direct):
//   2048 x 4096 x 4096  40 / 59     512 x 4096 x 14336  70 / 101     1188 x 2211 x 9472  63 / 81     3000 x 5000 x 992  32 / 44
//    777 x 3001 x 2080  33 / 24     512 x 4096 x  4096  45 /  29     1024 x 1024 x 4096  56 / 18     P V, 128 x 2048 x 128 x 2048  308 / 153
//   prepared: 1024 x 4096 x 4096  25 / 43     400 x 2759 x 6592  34 / 44     512 x 4096 x 4096  30 / 29     300 x 4096 x 4096  28 / 27
// and of the sizes measured none on the large side the other way (4096 x 4096 x 4096 55 / 114, 2048 x 2048 x 14336 72 / 124).
// An A operand of fewer rows than kPreparedMinRows is not packed ahead: its products read it as it is.
constexpr int kPreparedMinRows = 257;
inline bool large_kernel_can(int64_t M, int64_t KB) { return M > 64 && KB > 0 && KB <= kMaxKB; }
// Estimated microseconds of that int8 kernel (512 x 128 outputs per workgroup), fitted like those of the direct shapes: per
// round of workgroups a fixed part, and per block of a workgroup's share of K more where the chip is full, growing beyond 128
// blocks; the results; the exchange of partial tiles between s workgroups; the prepass unless the operands are prepared
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
// the shape of gemm_f8_kernel that is taken, -1: the large kernel
inline int direct_shape(int64_t M, int64_t N, int64_t KB, int64_t batch, bool prepared, int64_t cu) {
    const DirectChoice d = choose_direct(M, N, KB, batch, cu);
    const bool direct = !large_kernel_can(M, KB) || (prepared ? M < kPreparedMinRows : KB <= kDirectOnceBlocks) ||
                        d.us <= fast_cost(M, N, KB, batch, prepared, cu);
    return direct ? d.shape : -1;
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

// The whole prepared form of an A operand of few rows: the count of declined tiles.
__global__ void clear_count_kernel(uint32_t* count) {
    if (threadIdx.x == 0) *count = 0;
}

}  // namespace

// Largest operands of a single launch: larger products are cut into pieces of at most this many rows on the host, larger
// prepared operands are refused.  The bound of A is the documented one (its operand was once int8, 49152 bytes per 512 rows and block, with 31-bit
// offsets); what the kernels index in 32 bits, rows x K / 32 x 16 bytes of codes and 65535 tiles of 256 rows, lies beyond both.
static int64_t max_rows_a(int64_t KB) {
    const int64_t tiles = (((int64_t)1 << 31) - 1) / ((KB + 1) * 49152);
    return (tiles < 65535 ? tiles : 65535) * 512;
}
static int64_t max_rows_w(int64_t KB) { return ((((int64_t)1 << 31) - 1) / (KB * 16)) / 128 * 128; }

// Prepared operands are of either format: bytes of the larger (DialectFP4, FP6 E2M3)
size_t gemm_prepared_bytes(int64_t rows, int64_t K, bool weight) {
    const int64_t KB = K / kBlock;
    if (rows <= 0 || KB <= 0 || KB > kMaxKB) return 0;
    if (!weight && rows < kPreparedMinRows) return 256;    // the count of declined tiles
    return (size_t)exact_operand_bytes(rows, KB, true, !weight);
}

// byte offset, inside a prepared A, of the dword that counts tiles declined since it was prepared
size_t gemm_prepared_declined_offset(int64_t M, int64_t) {
    return M < kPreparedMinRows ? 0 : (size_t)kExactSplitTiles * 4;
}

size_t gemm_prepared_workspace_bytes(int64_t M, int64_t N, int64_t K) {
    const int64_t KB = K / kBlock;
    if (M <= 0 || N <= 0 || !large_kernel_can(M, KB) || M < kPreparedMinRows) return 0;
    return direct_shape(M, N, KB, 1, true, device_cu_count()) >= 0 ? 0 : (size_t)exact_split_bytes(M, N, KB, 1);
}

// what the large kernel and its prepass need for one problem of a batch
static size_t large_workspace_bytes(int64_t M, int64_t N, int64_t KB) {
    const int64_t Mc = M < max_rows_a(KB) ? M : max_rows_a(KB), Nc = N < max_rows_w(KB) ? N : max_rows_w(KB);
    return (size_t)(align256(exact_operand_bytes(Mc, KB, true, true)) + align256(exact_operand_bytes(Nc, KB, true, false)) +
                    align256(exact_split_bytes(Mc, Nc, KB, 1)));
}

size_t gemm_large_workspace_bytes(int64_t M, int64_t N, int64_t K) {
    const int64_t KB = K / kBlock;
    return M <= 0 || N <= 0 || !large_kernel_can(M, KB) ? 0 : large_workspace_bytes(M, N, KB);
}

size_t gemm_workspace_bytes(int64_t M, int64_t N, int64_t K) {
    const int64_t KB = K / kBlock;
    if (M <= 0 || N <= 0 || !large_kernel_can(M, KB)) return 0;
    // nothing but a token where the direct kernel is taken whatever the batch
    const int64_t cu = device_cu_count();
    if (direct_shape(M, N, KB, 1, false, cu) >= 0 && direct_shape(M, N, KB, 65535, false, cu) >= 0) return 256;
    return large_workspace_bytes(M, N, KB);
}

int gemm_path(int64_t M, int64_t N, int64_t KB, int64_t batch, bool prepared) {
    prepared = prepared && KB > 0 && KB <= kMaxKB;         // otherwise nothing is prepared and the operands are read as they are
    return 1 + direct_shape(M, N, KB, batch, prepared, device_cu_count());
}

size_t gemm_requant_workspace_bytes(int64_t M, int64_t N, int64_t K) {
    if (M <= 0 || N <= 0) return 0;
    return (size_t)align256((int64_t)gemm_large_workspace_bytes(M, N, K)) + (size_t)align256(M * N * 2);
}

namespace {

void fill_params(GemmParams& p, const dfp4_tensor& A, const dfp4_tensor& W, void* out, int64_t ldc,
                 int64_t strideA_rows, int64_t strideW_rows, int64_t strideC, const dfp4_tensor* rq) {
    p.a_codes = A.codes; p.a_dial = A.dialect; p.a_exp = A.exponent;
    p.w_codes = W.codes; p.w_dial = W.dialect; p.w_exp = W.exponent;
    p.out = out; p.M = (int)A.rows; p.N = (int)W.rows; p.KB = (int)(A.K / kBlock);
    p.ldc = ldc; p.strideA_rows = strideA_rows; p.strideW_rows = strideW_rows; p.strideC = strideC;
    if (rq) {
        p.q_codes = reinterpret_cast<uint32_t*>(rq->codes); p.q_dial = rq->dialect; p.q_exp = rq->exponent;
    }
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
            const int rc = launch_gemm_f8(mx, bf16, p, batch, choose_direct(p.M, p.N, KB, batch, cu).shape, stream);
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
    if (large_kernel_can(M, KB) && (rq || batch > 1) && (M > max_rows_a(KB) || N > max_rows_w(KB)))
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
    if (!large_kernel_can(M, KB) || (!rq && (!workspace || workspace_bytes < large_workspace_bytes(M, N, KB) * (size_t)batch ||
                                            direct_shape(M, N, KB, batch, false, cu) >= 0))) {
        rc = launch_direct(mx, bf16, A, W, out, ldc, batch, strideA_rows, strideW_rows, strideC, stream);
        if (rc != DFP4_OK || !rq) return rc;
        return launch_quantize(mx, out, M * batch, N, ldc, *rq, stream);       // `out` holds the bf16 [batch * M, N]
    }
    // pieces of at most mc x nc outputs (one piece for every product of ordinary size)
    const int64_t mc = M < max_rows_a(KB) ? M : max_rows_a(KB), nc = N < max_rows_w(KB) ? N : max_rows_w(KB);
    const int64_t a_bytes = align256(exact_operand_bytes(mc, KB, !mx, true)), w_bytes = align256(exact_operand_bytes(nc, KB, !mx, false));
    const size_t prep_bytes = (size_t)(a_bytes + w_bytes) * (size_t)batch;
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
            // (a last piece may be smaller: within the room of a full one)
            p.a_prep = ws; p.a_prep_stride = a_bytes;
            p.w_prep = ws + (size_t)a_bytes * (size_t)batch; p.w_prep_stride = w_bytes;
            GemmParams prep = p;
            if (n0 > 0) prep.a_prep = nullptr;                 // this piece of A is there already
            rc = launch_exact_prep(mx, prep, batch, false, stream);
            if (rc != DFP4_OK) return rc;
            rc = launch_exact(mx, bf16, p, batch, reinterpret_cast<float*>(ws + prep_bytes), workspace_bytes - prep_bytes, rq != nullptr, stream);
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
    (weight ? p.w_prep : p.a_prep) = static_cast<uint8_t*>(prepared);
    return launch_exact_prep(mx, p, 1, true, stream);
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
        return launch_gemm_f8(mx, bf16, p, 1, choose_direct(M, N, KB, 1, cu).shape, stream);     // one launch: max_rows_w is half of what it takes
    }
    p.declined = reinterpret_cast<uint32_t*>(static_cast<uint8_t*>(a_prepared) + gemm_prepared_declined_offset(M, A.K));
    const int shape = direct_shape(M, N, KB, 1, true, cu);
    if (shape >= 0 && M <= gemm_direct_max_rows(KB, false) && N <= gemm_direct_max_rows(KB, true)) {
        set_prepared_classes(mx, p, static_cast<const uint8_t*>(a_prepared), static_cast<const uint8_t*>(w_prepared));
        return launch_gemm_f8(mx, bf16, p, 1, shape, stream);
    }
    p.a_prep = static_cast<uint8_t*>(a_prepared);
    p.w_prep = static_cast<uint8_t*>(const_cast<void*>(w_prepared));
    return launch_exact(mx, bf16, p, 1, static_cast<float*>(workspace), workspace_bytes, false, stream);
}

}  // namespace dfp4
