// Exact products of few rows, few tiles, short or very long K, and thin batches, with both operands in their 4-bit form: the
// block-scaled matrix instruction on operands expanded to FP8 inside the kernel.
//
// Every DialectFP4 magnitude 0.5 u (u <= 15) is an FP8 E4M3 number, and the exponent byte is the instruction's scale, so an item
// (row, block of 32 codes) is expanded by two table lookups and a sign bit per byte, with no reference exponent, no shift and
// no class, and a pair of blocks is one instruction per 32 x 32 outputs.  Sums are fp32 and exact under the rule of
// gemm_native.hip: with the norms of the rows in units of their smallest block exponent, sum |a||w| <= ||a|| ||w|| <= 2^24 units means that no
// partial sum rounds (3.2 million outputs of single FP8 instructions below that bound checked: none off).  The norms are
// taken while the items are expanded: of A from its codes, of W, which has most of the rows where A has few, up to K = 6144 from its
// exponents alone (||w||^2 <= sum over blocks of 32 15^2 4^offset: about three times the norm of Gaussian data, more with outliers) and
// beyond from its codes.  A tile without a proof looks at the codes a second time, first W's, then A's, for the three bounds of
// gemm_native.hip, over all of K or over every group's share of it (the groups' sums are added with one rounding); one that passes none is computed
// again in int32 (gemm_int8_tile.h), in pieces small enough that they do not set the kernel's register count.  Microseconds of a call, plain inputs / outlier channels on A (x 50) and W (x 20), or A alone (x 200), without a second look,
// so that such tiles were multiplied twice / with it:
//   32 x 4096 x 4096  9.2 / 21.2, 20.6 / 12.9, 12.8      1500 x 4000 x 1120                20.3 / 113 / 24
//   777 x 3001 x 2080  24 /   91,   85 / 30, 30          P V, 128 x 2048 x 128 x 2048       155 / 637 / 181
// The bound of every group's share (without it / with it): channels x 1000 on A, 16 x 4096 x 14336 104 / 46, 700 x 1024 x 8192 217 / 53; W x 100 and
// A x 50, 250 x 4096 x 4096 120 / 29.  The second look is vector-ALU work (a third of a product's time for either operand) and lost where it finds no
// proof: channels x 1000 on A, 512 x 4096 x 14336 616 -> 697.
//
// This took the place of int8 operands with classes (gemm_int8_tile.h).  There a pass over the exponents came first, and classes on
// both operands cost up to four products per pair of blocks.  Microseconds of a call with int8 / with FP8 operands (A with 0.5 %
// outlier channels x 50, scores with two outlier dimensions on both):
//   16 x 4096 x 4096      10.7 /  9.5     777 x 3001 x 2080     28.6 / 24.1     2048 x 4096 x 4096            78.7 / 65.7
//   16 x 14336 x 4096     17.2 / 14.6     512 x 4096 x 4096     37.2 / 30.7     scores, 128 x 2048 x 2048 x 128  487 / 366
//   36 x 7898 x 1344      10.9 /  9.0     512 x 4096 x 14336     110 / 100      P V, 128 x 2048 x 128 x 2048     210 / 155
// and, on prepared operands of more than 256 rows (where the references and classes were there already),
//   300 x 4096 x 4096     32.7 / 26.9     777 x 3001 x 2080     30.1 / 25.4     1500 x 4000 x 1120            23.5 / 20.3
// What bounds it: as before nothing alone.  An item is about 60 vector-ALU instructions, and the expansion, the LDS traffic and the
// products of a workgroup's few waves overlap only in part.  Tried: one operand buffer and three or four waves per SIMD for the
// 128 x 128 and 256 x 128 tiles (3 to 18 % slower); four waves per SIMD for the tiles of one iteration (scores above 369, but 16 x 700 x 1312 x
// 64 18.6 instead of 16.7 us); the second look with the sums in registers, which the compiler then spilled (scores 399 -> 1086 us): they are in LDS
// meanwhile, and what follows the products takes the thread's place anew.  The exponents' ends are kept as one packed maximum per row: as two values
// they cost registers, and the last shape above 15 % of its time.
//
// Tiles, groups and the loop are those of gemm_int8_tile.h: KG groups of WM x WN waves, each with its contiguous range of K, 4
// blocks per iteration, expanded operands in LDS as [32-row group][pair of blocks][half of a block][block of the pair][row][16
// bytes], the row slot rotated by twice the block number.  The instruction wants in lane (h, r) half h of both blocks of row r, and the
// scale of block h.
#include "exact_norms.h"
#include "gemm_int8_tile.h"

namespace dfp4 {
namespace {

// Tables of a dialect: FP8 E4M3 bit patterns of its 8 magnitudes, and the magnitudes u themselves
constexpr uint8_t e4m3_of_half_units(int u) {
    int e = -1;                                                        // floor(log2(0.5 u))
    for (int v = u; v > 1; v >>= 1) ++e;
    return u == 0 ? 0 : (uint8_t)(((e + 7) << 3) | (((u << 3) >> (e + 1)) & 7));
}
struct F8Book { uint32_t w[kDialects + 1][4]; };                       // the last: all zeros
constexpr F8Book make_f8_book() {
    F8Book b{};
    for (int d = 0; d < kDialects; ++d)
        for (int j = 0; j < 8; ++j) {
            b.w[d][j / 4] |= (uint32_t)e4m3_of_half_units(kBook[d][j]) << (8 * (j % 4));
            b.w[d][2 + j / 4] |= (uint32_t)kBook[d][j] << (8 * (j % 4));
        }
    return b;
}
__device__ const F8Book g_f8_book = make_f8_book();

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int kMaxExp = 190;          // of any block: 4^(e - 127) is built as a float, and 2 e - 127 is its exponent byte

template <class S>
struct F8Lds {
    union {
        __attribute__((aligned(16))) uint8_t x[S::KG][S::kBufs][S::kRowGroups * 4096]; // expanded operands: groups of A, of W
        float sums[S::kOnce ? 1 : S::KG * S::kTm * S::kTn];            // of the groups, [group][wave][register][lane], once the operands are done with
    };
    __attribute__((aligned(16))) uint32_t tab[kDialects + 1][4];
    __attribute__((aligned(4))) uint8_t sc[S::KG][S::kBufs][S::kRows][4];              // exponent bytes of the 4 blocks of a row
    float sq[S::KG][S::kRows];                                         // per row: sum of squares in units of 2^-127 ...
    uint8_t lo[S::KG][S::kRows];                                       // ... smallest exponent byte (255: all zero) ...
    uint8_t ok[S::KG][S::kRows];                                       // ... and whether all are in range
    ExactStat part[S::KG > 1 ? S::KG : 1][S::KG > 1 ? S::kRows : 1];   // of the groups, second look
    int norm[2][8];                                                    // of A's, of W's rows in their units, the largest (bits): squared norm; ExactStat; [0][5] groups without a proof
};

template <int CTRL>
__device__ __forceinline__ int quad_dpp(int v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true); }

// S: tile; F: the shape a tile is computed again with, of as many threads
template <bool MX, bool BF16, class S, class F>
__global__ __launch_bounds__(S::kThreads, S::kWavesPerSimd) void gemm_f8_kernel(GemmParams p) {
    static_assert(S::kThreads == F::kThreads && S::kTm % F::kTm == 0 && S::kTn % F::kTn == 0);
    constexpr int TI = S::TI, TJ = S::TJ;
    __shared__ union {
        F8Lds<S> d;
        TileLds<F> again;
    } u;
    F8Lds<S>& lds = u.d;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6) % (S::WM * S::WN);
    const int kg = __builtin_amdgcn_readfirstlane(tid >> 6) / (S::WM * S::WN);
    const int gt = tid % S::kGroupThreads;
    const int KB = p.KB;
    const int64_t bz = blockIdx.z;
    const int m0 = (int)blockIdx.y * S::kTm, n0 = (int)blockIdx.x * S::kTn;

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
    float sq[S::kItems];                                               // of the items expanded so far
    typedef uint16_t v2u __attribute__((ext_vector_type(2)));
    v2u ends[S::kItems];                                               // 255 - smallest exponent of nonzero blocks (0: none), largest exponent
    auto load = [&](Item& it, int j, int kb0) {
        const uint32_t i = blk[j] + (uint32_t)min(kb0 + b4, KB - 1);   // blocks beyond K read the row's last
        it.c = *reinterpret_cast<const uint4*>((j < S::kItemsA ? ac : wc) + (uint64_t)(i * 16u));
        it.e = (j < S::kItemsA ? ae : we)[i];
        it.d = MX ? 7u : (uint32_t)(j < S::kItemsA ? ad : wd)[i];
    };
#pragma unroll
    for (int j = 0; j < S::kItems; ++j) {
        if (KB > 0) load(item[j], j, k_lo);
        sq[j] = 0.0f;
        ends[j] = v2u{0, 0};
    }
    for (int i = tid; i < (kDialects + 1) * 4; i += S::kThreads) (&lds.tab[0][0])[i] = (&g_f8_book.w[0][0])[i];
    if (tid < 16) (&lds.norm[0][0])[tid] = 0;
    __syncthreads();

    const int wm = wave / S::WN, wn = wave % S::WN, h = lane >> 5, r = lane & 31;
    v16f acc[TI][TJ];
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j)
#pragma unroll
            for (int x = 0; x < 16; ++x) acc[i][j][x] = 0.0f;
    // Item j of the iteration at kb0: the table of its dialect, then the expansion into a buffer, and its part of the row's norm
    auto table = [&](const Item& it, int kb0) {
        return *reinterpret_cast<const uint4*>(&lds.tab[kb0 + b4 < KB ? (it.d & 15u) : (uint32_t)kDialects][0]);
    };
    // Of W the norm is taken from its codes only where K is long, where the looser one of ordinary data comes near the limit (Gaussian W, 0.5 %
    // outlier channels x 50 on A: 2^22.5 units at K = 4096, 2^24 at 14336); the 16 instructions of 60 are the second look's otherwise.
    const bool w_codes = KB > 192;
    uint8_t* slot = &lds.x[kg][0][0] + (b4 >> 1) * 2048 + (b4 & 1) * 512;
    auto expand = [&](const Item& it, int j, uint4 tab, int buf, int kb0) {
        const int row = j * S::kItemRows + r4;
        const uint32_t c4[4] = {it.c.x, it.c.y, it.c.z, it.c.w};
        uint32_t v[8], s2 = 32 * 15 * 15;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[2 * k] = __builtin_amdgcn_perm(tab.y, tab.x, c4[k] & 0x07070707u) | ((c4[k] << 4) & 0x80808080u);
            v[2 * k + 1] = __builtin_amdgcn_perm(tab.y, tab.x, (c4[k] >> 4) & 0x07070707u) | (c4[k] & 0x80808080u);
        }
        if (j < S::kItemsA || w_codes) {
            s2 = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t ue = __builtin_amdgcn_perm(tab.w, tab.z, c4[k] & 0x07070707u), uo = __builtin_amdgcn_perm(tab.w, tab.z, (c4[k] >> 4) & 0x07070707u);
                s2 = __builtin_amdgcn_udot4(ue, ue, __builtin_amdgcn_udot4(uo, uo, s2, false), false);
            }
        }
        uint8_t* dst = slot + buf * (S::kRowGroups * 4096) + (row >> 5) * 4096 + ((row + 2 * b4) & 31) * 16;
        *reinterpret_cast<uint4*>(dst) = make_uint4(v[0], v[1], v[2], v[3]);
        *reinterpret_cast<uint4*>(dst + 1024) = make_uint4(v[4], v[5], v[6], v[7]);
        lds.sc[kg][buf][row][b4] = (uint8_t)it.e;
        // 4^(e - 127) while e is in range (otherwise the tile is refused)
        const bool some = kb0 + b4 < KB && ((it.c.x | it.c.y | it.c.z | it.c.w) & 0x77777777u) != 0;      // not an all-zero block
        const float unit2 = __builtin_bit_cast(float, ((it.e << 1) - 127u) << 23);
        sq[j] += some ? (float)s2 * unit2 : 0.0f;
        ends[j] = __builtin_elementwise_max(ends[j], __builtin_bit_cast(v2u, (it.e << 16) | (some ? 255u - it.e : 0u)));
    };
    // the rows' norms over the 4 blocks' lanes; over the groups once all are there
    auto row_norm = [&](float s, uint32_t lo, bool ok) {
        const float v = lo == 255 ? 0.0f : ldexpf(s, 2 * (127 - (int)lo));
        return ok ? v : __builtin_inff();
    };
    // the largest of a wave's values, whose quads hold equal ones (not negative: ordered like their bits); no LDS
    auto take_norm = [&](int v, int side, int which) {
        v = max(v, quad_dpp<0x141>(v));
        v = max(v, quad_dpp<0x140>(v));
        v = max(max(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
                max(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
        if (lane == 0) atomicMax(&lds.norm[side][which], v);
    };
    auto finish_norms = [&] {
        int most[2] = {0, 0};
#pragma unroll
        for (int j = 0; j < S::kItems; ++j) {
            float s = sq[j];
            s += __builtin_bit_cast(float, quad_dpp<0xB1>(__builtin_bit_cast(int, s)));
            s += __builtin_bit_cast(float, quad_dpp<0x4E>(__builtin_bit_cast(int, s)));
            v2u e = ends[j];
            e = __builtin_elementwise_max(e, __builtin_bit_cast(v2u, quad_dpp<0xB1>(__builtin_bit_cast(int, e))));
            e = __builtin_elementwise_max(e, __builtin_bit_cast(v2u, quad_dpp<0x4E>(__builtin_bit_cast(int, e))));
            const uint32_t lo = 255u - e.x, hi = e.y;
            const bool ok = lo >= (uint32_t)kMinRef && (lo == 255 || lo <= (uint32_t)kMaxRef) && hi <= (uint32_t)kMaxExp;
            if constexpr (S::KG == 1) {
                int& m = most[j < S::kItemsA ? 0 : 1];
                m = max(m, __builtin_bit_cast(int, row_norm(s, lo, ok)));
            } else {
                const int row = j * S::kItemRows + r4;
                if (b4 == 0) {
                    lds.sq[kg][row] = s;
                    lds.lo[kg][row] = (uint8_t)lo;
                    lds.ok[kg][row] = ok ? 1 : 0;
                }
            }
        }
        if constexpr (S::KG == 1) {
            take_norm(most[0], 0, 0);
            take_norm(most[1], 1, 0);
        }
    };
    struct Operands { v8i a[TI], b[TJ]; };                             // of a pair of blocks
    struct Scales { int a[TI], b[TJ]; };                               // byte 0: of block h of the first pair, byte 2: of the second
    auto read_scales = [&](Scales& o, int buf) {
        const uint32_t* sc = reinterpret_cast<const uint32_t*>(&lds.sc[kg][buf][0][0]) + r;
#pragma unroll
        for (int i = 0; i < TI; ++i) o.a[i] = (int)(sc[(TI * wm + i) * 32] >> (8 * h));
#pragma unroll
        for (int j = 0; j < TJ; ++j) o.b[j] = (int)(sc[S::kTm + (TJ * wn + j) * 32] >> (8 * h));
    };
    auto read = [&](Operands& o, int buf, int pr) {
        const uint8_t* src = &lds.x[kg][buf][0] + pr * 2048 + h * 1024;
        const int s0 = ((r + 4 * pr) & 31) * 16, s1 = 512 + ((r + 4 * pr + 2) & 31) * 16;
        auto both = [&](int group) {
            const v4i x = *reinterpret_cast<const v4i*>(src + group * 4096 + s0), y = *reinterpret_cast<const v4i*>(src + group * 4096 + s1);
            return v8i{x[0], x[1], x[2], x[3], y[0], y[1], y[2], y[3]};
        };
#pragma unroll
        for (int i = 0; i < TI; ++i) o.a[i] = both(TI * wm + i);
#pragma unroll
        for (int j = 0; j < TJ; ++j) o.b[j] = both(S::kTm / 32 + TJ * wn + j);
    };
    auto multiply = [&](const Operands& o, const Scales& s, auto pr_c) {
        constexpr int kByte = 2 * decltype(pr_c)::value;
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(o.a[i], o.b[j], acc[i][j], 0, 0, kByte, s.a[i], kByte, s.b[j]);
        // The operands are in use until here.  Where the sums change registers the compiler has let the result overlap an operand
        // that it saw no further use of, which the instruction overwrites before it has read it for the last rows (the build checks).
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j) asm volatile("" : "+v"(acc[i][j]) : "v"(o.a[i]), "v"(o.b[j]));
    };
    using First = std::integral_constant<int, 0>;
    using Second = std::integral_constant<int, 1>;
    if constexpr (S::kOnce) {
        if (KB > 0) {
#pragma unroll
            for (int j = 0; j < S::kItems; ++j) expand(item[j], j, table(item[j], 0), 0, 0);
        }
        finish_norms();
        __syncthreads();                                               // (its products follow once it is known whether they are wanted)
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
                expand(item[j], j, table(item[j], kb0), 0, kb0);
                load(item[j], j, kb0 + 4);
            }
            in_order();
            Scales s;
            read_scales(s, 0);
            Operands o;
            read(o, 0, 0);
            multiply(o, s, First{});
            read(o, 0, 1);
            multiply(o, s, Second{});
            in_order();
        }
        finish_norms();
    } else {
        // One iteration: multiply the 4 blocks from kb0 (buffer BUF), expand the next 4 into the other buffer,
        // load the 4 after those.  A wave issues the LDS reads of a pair's operands, expands while they are on
        // their way, then multiplies.
        auto iteration = [&](auto buf_c, int k) {
            constexpr int kBuf = decltype(buf_c)::value, kNxt = 1 - kBuf, kHalf = S::kItems / 2;
            const bool more = k + 4 < per;
            Scales s;
            read_scales(s, kBuf);
            auto pair = [&](auto pr_c) {
                constexpr int kPr = decltype(pr_c)::value;
                constexpr int j_lo = kPr == 0 ? 0 : kHalf, j_hi = kPr == 0 ? kHalf : S::kItems;
                uint4 tab[S::kItems];
                if (more) {
#pragma unroll
                    for (int j = j_lo; j < j_hi; ++j) tab[j] = table(item[j], k_lo + k + 4);
                }
                Operands o;
                read(o, kBuf, kPr);
                __builtin_amdgcn_sched_barrier(0);
                if (more) {
#pragma unroll
                    for (int j = j_lo; j < j_hi; ++j) {
                        expand(item[j], j, tab[j], kNxt, k_lo + k + 4);
                        load(item[j], j, k_lo + k + 8);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
                multiply(o, s, pr_c);
                __builtin_amdgcn_sched_barrier(0);
            };
            pair(First{});
            pair(Second{});
            __syncthreads();
        };
        if (KB > 0) {
#pragma unroll
            for (int j = 0; j < S::kItems; ++j) {
                expand(item[j], j, table(item[j], k_lo), 0, k_lo);
                load(item[j], j, k_lo + 4);
            }
            __syncthreads();
            for (int k = 0; k < per; k += 8) {
                iteration(std::integral_constant<int, 0>{}, k);
                if (k + 4 >= per) break;
                iteration(std::integral_constant<int, 1>{}, k + 4);
            }
        }
        finish_norms();
    }
    if constexpr (!S::kOnce) __syncthreads();
    // the thread's place, where registers are short taken anew: nothing of it is kept through the products for what follows
    int tid_ = threadIdx.x;
    if constexpr (S::KG > 1) asm volatile("" : "+v"(tid_));
    const int lane_ = tid_ & 63, h_ = lane_ >> 5, r_ = lane_ & 31;
    constexpr int kOut = TI * TJ * 16;
    float* sums = lds.sums + (S::kOnce ? 0 : (kg * S::WM * S::WN + wave) * kOut * 64 + lane_);          // of this lane
    auto put_sums = [&] {
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j)
#pragma unroll
                for (int x = 0; x < 16; ++x) sums[((i * TJ + j) * 16 + x) * 64] = acc[i][j][x];
    };
    // NV values of every row from row_lo to row_hi, over the groups: the largest of A's and of W's rows
    auto over_groups = [&](auto nv_c, int which, int row_lo, int row_hi, auto&& of_row) {
        constexpr int NV = decltype(nv_c)::value;
        static_assert(S::kTm % 32 == 0 && S::kTn % 32 == 0, "half a wave holds rows of one operand");
        for (int i = tid_; i < (row_hi - row_lo + 63) / 64 * 64; i += S::kThreads) {      // whole waves
            const int row = row_lo + i;
            float v[NV] = {};
            if (row < row_hi) of_row(row, v);
#pragma unroll
            for (int q = 0; q < NV; ++q) {
                int b = __builtin_bit_cast(int, v[q]);
#pragma unroll
                for (int o = 1; o < 32; o <<= 1) b = max(b, __shfl_xor(b, o));
                if ((lane_ & 31) == 0 && row < row_hi) atomicMax(&lds.norm[row < S::kTm ? 0 : 1][which + q], b);
            }
        }
    };
    // The groups' sums go to LDS ahead of the norms' barrier, which saves one, where they are few; 64 registers delay it (249 x 11523 x 640 13.4 -> 14.0 us)
    constexpr bool kPutEarly = S::KG > 1 && TI * TJ == 1;
    if constexpr (S::KG > 1) {
        if constexpr (kPutEarly) put_sums();
        over_groups(std::integral_constant<int, 1>{}, 0, 0, S::kRows, [&](int row, float (&v)[1]) {
            uint32_t lo = 255;
            bool ok = true;
#pragma unroll
            for (int g = 0; g < S::KG; ++g) {
                lo = min(lo, (uint32_t)lds.lo[g][row]);
                ok = ok && lds.ok[g][row] != 0;
                v[0] += lds.sq[g][row];
            }
            v[0] = row_norm(v[0], lo, ok);
        });
        __syncthreads();
    }
    auto norm = [&](int side, int which) { return __builtin_bit_cast(float, lds.norm[side][which]); };
    // the same for every thread
    bool proven = sqrtf(norm(0, 0)) * sqrtf(norm(1, 0)) <= kExactUnits;
    const bool looked = !proven && fmaxf(norm(0, 0), norm(1, 0)) < __builtin_inff();
    if (looked) {
        // A second look at the codes: what exact_prep_kernel keeps of a prepared operand (ExactStat), first of W, whose norm was a
        // bound, then of A.  The sums are in LDS meanwhile and set no register count (K of one iteration: there are none yet).
        if constexpr (!kPutEarly && !S::kOnce) put_sums();
        auto look = [&](auto side_c) {
            constexpr int kSide = decltype(side_c)::value, kFirst = kSide == 0 ? 0 : S::kItemsA;
            constexpr int kN = kSide == 0 ? S::kItemsA : S::kItems - S::kItemsA;
            constexpr int kAhead = S::KG == 1 ? 1 : 2;                 // iterations whose loads are on their way
            Item next[kAhead][kN];
            float sq2[kN], low[kN], high[kN];                          // of this thread's blocks of the rows
            int ref[kN], far[kN];
#pragma unroll
            for (int j = 0; j < kN; ++j) {
#pragma unroll
                for (int d = 0; d < kAhead; ++d) load(next[d][j], kFirst + j, k_lo + 4 * d);
                sq2[j] = low[j] = high[j] = 0.0f;
                far[j] = 0;
                if constexpr (S::KG == 1) {
                    int e = (int)ends[kFirst + j].x;
                    e = max(e, quad_dpp<0xB1>(e));
                    ref[j] = 255 - max(e, quad_dpp<0x4E>(e));
                } else {
                    ref[j] = 255;
#pragma unroll
                    for (int g = 0; g < S::KG; ++g) ref[j] = min(ref[j], (int)lds.lo[g][(kFirst + j) * S::kItemRows + r4]);
                }
            }
            const int k_hi = min(k_lo + per, KB);
#pragma unroll 1
            for (int k = k_lo; k < k_hi; k += 4 * kAhead) {
#pragma unroll
                for (int d = 0; d < kAhead; ++d) {
                    const int kb0 = k + 4 * d;
                    if (kb0 >= k_hi) break;
#pragma unroll
                    for (int j = 0; j < kN; ++j) {
                        const uint4 tab = table(next[d][j], kb0);
                        const uint32_t c4[4] = {next[d][j].c.x, next[d][j].c.y, next[d][j].c.z, next[d][j].c.w};
                        const int delta = (int)next[d][j].e - ref[j];
                        uint32_t u[8], s2 = 0;
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            u[2 * q] = __builtin_amdgcn_perm(tab.w, tab.z, c4[q] & 0x07070707u);
                            u[2 * q + 1] = __builtin_amdgcn_perm(tab.w, tab.z, (c4[q] >> 4) & 0x07070707u);
                        }
#pragma unroll
                        for (int q = 0; q < 8; ++q) s2 = __builtin_amdgcn_udot4(u[q], u[q], s2, false);
                        load(next[d][j], kFirst + j, kb0 + 4 * kAhead);
                        const bool some = s2 != 0, is_high = some && delta >= 4;               // (beyond K the table is all zeros)
                        const float v = some ? ldexpf((float)s2, 2 * delta) : 0.0f;
                        sq2[j] += v;
                        low[j] += is_high ? 0.0f : v;
                        far[j] = max(far[j], some ? delta : 0);
                        if (__ballot(is_high) != 0ull) {
                            uint32_t s1 = 0;
#pragma unroll
                            for (int q = 0; q < 8; ++q) s1 = __builtin_amdgcn_udot4(u[q], 0x01010101u, s1, false);
                            high[j] += is_high ? ldexpf((float)s1, delta) : 0.0f;
                        }
                    }
                }
            }
            auto over_quad = [&](float a) {
                a += __builtin_bit_cast(float, quad_dpp<0xB1>(__builtin_bit_cast(int, a)));
                return a + __builtin_bit_cast(float, quad_dpp<0x4E>(__builtin_bit_cast(int, a)));
            };
            ExactStat most{0, 0, 0, 0};
#pragma unroll
            for (int j = 0; j < kN; ++j) {
                int f = far[j];
                f = max(f, quad_dpp<0xB1>(f));
                f = max(f, quad_dpp<0x4E>(f));
                const ExactStat v{over_quad(sq2[j]), over_quad(low[j]), over_quad(high[j]), ldexpf(15.0f, f)};
                if constexpr (S::KG == 1) most = ExactStat{fmaxf(most.sq, v.sq), fmaxf(most.sq_low, v.sq_low), fmaxf(most.sum_high, v.sum_high), fmaxf(most.top, v.top)};
                else if (b4 == 0) lds.part[kg][(kFirst + j) * S::kItemRows + r4] = v;
            }
            if constexpr (S::KG == 1) {
                take_norm(__builtin_bit_cast(int, most.sq), kSide, 1);
                take_norm(__builtin_bit_cast(int, most.sq_low), kSide, 2);
                take_norm(__builtin_bit_cast(int, most.sum_high), kSide, 3);
                take_norm(__builtin_bit_cast(int, most.top), kSide, 4);
            } else {
                __syncthreads();
                over_groups(std::integral_constant<int, 4>{}, 1, kSide == 0 ? 0 : S::kTm, kSide == 0 ? S::kTm : S::kRows, [&](int row, float (&o)[4]) {
#pragma unroll
                    for (int g = 0; g < S::KG; ++g) {
                        const ExactStat v = lds.part[g][row];
                        o[0] += v.sq;
                        o[1] += v.sq_low;
                        o[2] += v.sum_high;
                        o[3] = fmaxf(o[3], v.top);
                    }
                });
            }
            __syncthreads();
            return ExactStat{norm(kSide, 1), norm(kSide, 2), norm(kSide, 3), norm(kSide, 4)};
        };
        const ExactStat w = look(std::integral_constant<int, 1>{});
        const float inf = __builtin_inff();
        proven = sums_exactly(ExactStat{norm(0, 0), inf, inf, sqrtf(norm(0, 0))}, w);          // (an element is at most the norm of its row)
        if (!proven) proven = sums_exactly(look(std::integral_constant<int, 0>{}), w);
        if constexpr (S::KG > 1) {
            if (!proven) {
                // It is enough that every group's sums are exact, if adding them rounds once: every wave bounds its group's
                ExactStat a{0, 0, 0, 0}, b{0, 0, 0, 0};
#pragma unroll
                for (int row = 0; row < S::kRows; row += 32) {
                    const ExactStat v = lds.part[kg][row + (lane_ & 31)];
                    ExactStat& m = row < S::kTm ? a : b;
                    m = ExactStat{fmaxf(m.sq, v.sq), fmaxf(m.sq_low, v.sq_low), fmaxf(m.sum_high, v.sum_high), fmaxf(m.top, v.top)};
                }
#pragma unroll
                for (int o = 1; o < 32; o <<= 1) {
                    a = ExactStat{fmaxf(a.sq, __shfl_xor(a.sq, o)), fmaxf(a.sq_low, __shfl_xor(a.sq_low, o)), fmaxf(a.sum_high, __shfl_xor(a.sum_high, o)), fmaxf(a.top, __shfl_xor(a.top, o))};
                    b = ExactStat{fmaxf(b.sq, __shfl_xor(b.sq, o)), fmaxf(b.sq_low, __shfl_xor(b.sq_low, o)), fmaxf(b.sum_high, __shfl_xor(b.sum_high, o)), fmaxf(b.top, __shfl_xor(b.top, o))};
                }
                if (!sums_exactly(a, b) && lane_ == 0) atomicOr(&lds.norm[0][5], 1);
                __syncthreads();
                proven = lds.norm[0][5] == 0;
                if (S::KG > 2 && proven) {
                    // (two are: one addition.)  The outputs that this thread finishes below, at most 2^27 units: added here, zeros left for there
#pragma unroll 1
                    for (int o = kg * (kOut / S::KG); o < (kg + 1) * (kOut / S::KG); ++o) {
                        double sum = 0.0;
#pragma unroll
                        for (int g = S::KG - 1; g >= 0; --g) {
                            float& part = lds.sums[((g * S::WM * S::WN + wave) * kOut + o) * 64 + lane_];
                            sum += (double)part;
                            part = g == 0 ? (float)sum : 0.0f;
                        }
                    }
                }
            }
        }
        if (S::KG == 1 && !S::kOnce && proven) {
#pragma unroll
            for (int i = 0; i < TI; ++i)
#pragma unroll
                for (int j = 0; j < TJ; ++j)
#pragma unroll
                    for (int x = 0; x < 16; ++x) acc[i][j][x] = sums[((i * TJ + j) * 16 + x) * 64];
        }
    }
    if (!proven) {
        __syncthreads();
#pragma unroll 1
        for (int i = 0; i < (S::kTm / F::kTm) * (S::kTn / F::kTn); ++i) {
            int piece = i;
            asm volatile("" : "+s"(piece));                            // nothing of a piece is kept in registers for the next
            const int by = (int)blockIdx.y * (S::kTm / F::kTm) + piece / (S::kTn / F::kTn);
            const int bx = (int)blockIdx.x * (S::kTn / F::kTn) + piece % (S::kTn / F::kTn);
            if (by * F::kTm >= p.M || bx * F::kTn >= p.N) continue;
            int8_tile<MX, BF16, F>(p, u.again, bz, by, bx);
            __syncthreads();
        }
        return;
    }

    if constexpr (S::kOnce) {
        if (KB > 0) {
            Scales s;
            read_scales(s, 0);
            Operands o;
            read(o, 0, 0);
            multiply(o, s, First{});
            if (KB > 2) {
                read(o, 0, 1);
                multiply(o, s, Second{});
            }
        }
    }

    // ---- results
    constexpr int kEsz = BF16 ? 2 : 4;
    const int row0 = m0 + wm * 32 * TI, col0 = n0 + wn * 32 * TJ;      // of this wave
    if constexpr (S::KG > 1) {
        if constexpr (!kPutEarly) {
            if (!looked) put_sums();
            __syncthreads();
        }
        // the groups' exact partial sums are added; group kg finishes its share of the tile's outputs
        constexpr int kShare = kOut / S::KG;
#pragma unroll
        for (int q = 0; q < kShare; ++q) {
            const int o = kg * kShare + q, i = o / (16 * TJ), j = o / 16 % TJ, x = o % 16;
            float sum = 0.0f;
#pragma unroll
            for (int g = 0; g < S::KG; ++g) sum += lds.sums[((g * S::WM * S::WN + wave) * kOut + o) * 64 + lane_];
            const int lr = 32 * i + 8 * (x >> 2) + 4 * h_ + (x & 3), lc = 32 * j + r_;
            if (row0 + lr < p.M && col0 + lc < p.N) {
                const int64_t at = bz * p.strideC + (int64_t)(row0 + lr) * p.ldc + col0 + lc;
                if constexpr (BF16) static_cast<uint16_t*>(p.out)[at] = f32_to_bf16_rne(sum);
                else static_cast<float*>(p.out)[at] = sum;
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
        const uint32_t lane_off = pairs ? (uint32_t)((4 * h_ + (r_ & 1)) * row_bytes + (r_ & ~1) * kEsz)
                                        : (uint32_t)(4 * h_ * row_bytes + r_ * kEsz);
        auto store = [&](auto full_c, auto pairs_c) {
            constexpr bool kFull = decltype(full_c)::value, kPairs = decltype(pairs_c)::value;
#pragma unroll
            for (int i = 0; i < TI; ++i)
#pragma unroll
                for (int j = 0; j < TJ; ++j) {
                    uint8_t* tile_out = wave_out + (int64_t)i * 32 * row_bytes + j * 32 * kEsz;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        uint8_t* rowp = tile_out + (int64_t)(8 * q) * row_bytes;
                        if constexpr (kPairs) {
#pragma unroll
                            for (int x = 0; x < 4; x += 2) {
                                const uint32_t b0 = f32_to_bf16_rne(acc[i][j][4 * q + x]), b1 = f32_to_bf16_rne(acc[i][j][4 * q + x + 1]);
                                const uint32_t send = (r_ & 1) ? b0 : b1;
                                const uint32_t recv = (uint32_t)__builtin_amdgcn_mov_dpp((int)send, 0xB1, 0xf, 0xf, true);
                                const uint32_t word = (r_ & 1) ? (recv | (b1 << 16)) : (b0 | (recv << 16));
                                DFP4_OUT_STORE(reinterpret_cast<uint32_t*>(rowp + (int64_t)x * row_bytes + lane_off), word);
                            }
                        } else {
#pragma unroll
                            for (int x = 0; x < 4; ++x) {
                                if (kFull || (row0 + i * 32 + 8 * q + 4 * h_ + x < p.M && col0 + j * 32 + r_ < p.N)) {
                                    uint8_t* dst = rowp + (int64_t)x * row_bytes + lane_off;
                                    if constexpr (BF16) DFP4_OUT_STORE(reinterpret_cast<uint16_t*>(dst), f32_to_bf16_rne(acc[i][j][4 * q + x]));
                                    else DFP4_OUT_STORE(reinterpret_cast<float*>(dst), acc[i][j][4 * q + x]);
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
    // Prepared operands of more than 256 rows: 512 x 128 outputs that the masks decline are counted once, by the first wave of their
    // first tile (where that tile is computed again in int32: there).  Behind the stores, where it delays nobody: before the
    // products 598 x 6742 x 288 took 15.6 us instead of 15.1.
    if (p.ref_a && p.declined && m0 % 512 == 0 && n0 % 128 == 0 && tid_ < 64) {
        int ha = 0, hw = 0, weight = 0;
        mask_weights<64>(p, m0, n0, ha, hw, weight);
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) weight += __shfl_xor(weight, o);
        if (tid_ == 0 && weight > kIntBound) atomicAdd(p.declined, 1u);
    }
}

// The tile shapes and what a product takes with each, in microseconds: `base`; per round of workgroups `fixed`, and for
// every 4 blocks of a group's share of K `step` + `fill` x the share of the chip that the round fills (the last round's
// rest counts as much as it fills), growing with K beyond 128 blocks by `grow` per 384; `store` per MB of fp32
// results, where their rows begin inside a line (N % 16) `ragged`.  1: one workgroup per compute unit, 2: two, which
// shapes that fit take as soon as there are more tiles than compute units.
// Fitted to 21000 products timed with int8 operands on 256 compute units (gemm_f8_kernel is 0 to 20 % faster in all shapes, which
// leaves the order of the shapes as it is), M 1..4096, N 64..14336, K 32..16384, 1 to 128 problems, each with
// every shape: the estimates are within 10 % (rms).  Microseconds of 32 / 64 (KG 4) / 64 (KG 2) / 128 (KG 2) / 128 / 256 rows, and of the int8
// kernel that the large one replaced, with its prepass:
//   16 x 4096 x 4096       10.1   17.5   20.0   36.5   49.0      -      -
//   512 x 4096 x 4096      60.6   40.1   33.8   39.6   50.3   57.0    112
//   777 x 3001 x 2080      54.1   40.0   31.8   27.1   31.0   35.4     72
//   2048 x 4096 x 4096        -    156    123   87.8   76.1   66.9   75.5
//   2048 x 4096 x 14336       -    487    439    300    305    262    171
struct DirectCost {
    int tm, tn, kg, resident;
    bool any_k;
    float base, fixed1, step1, fill1, fixed2, step2, fill2, store, ragged, grow;
};
constexpr DirectCost kDirectCost[] = {
    {32, 32, 8, 2, false, 2.63f, 0.53f, 1.67f, 0.27f, 0.0f, 3.07f, 0.61f, 0.351f, 0.378f, 0.0f},
    {64, 64, 4, 1, false, 2.11f, 2.46f, 1.58f, 0.53f, 0, 0, 0, 0.221f, 0.235f, 0.0f},
    {64, 64, 2, 2, false, 3.32f, 0.72f, 0.985f, 0.177f, 1.77f, 1.43f, 0.434f, 0.167f, 0.180f, 0.059f},
    {128, 128, 2, 1, true, 3.02f, 3.32f, 1.93f, 0.404f, 0, 0, 0, 0.239f, 0.233f, 0.074f},
    {128, 128, 1, 2, true, 2.90f, 2.31f, 1.38f, 0.162f, 3.11f, 1.76f, 0.335f, 0.047f, 0.262f, 0.152f},
    {256, 128, 1, 1, true, 1.29f, 4.71f, 1.56f, 0.216f, 0, 0, 0, 0.065f, 0.322f, 0.188f},
};
constexpr int kOnceShape = 6;                          // the one-iteration form of the 128 x 128 tile

template <class S, class F = S>
int launch(bool mx, bool bf16, const GemmParams& p, int64_t batch, hipStream_t stream) {
    dim3 g((unsigned)((p.N + S::kTn - 1) / S::kTn), (unsigned)((p.M + S::kTm - 1) / S::kTm), (unsigned)batch);
    dispatch_mx_bf16(mx, bf16, [&](auto mxc, auto bc) {
        hipLaunchKernelGGL((gemm_f8_kernel<decltype(mxc)::value, decltype(bc)::value, S, F>), g, dim3(S::kThreads), 0, stream, p);
    });
    return check_launch();
}

}  // namespace

DirectChoice choose_direct(int64_t M, int64_t N, int64_t KB, int64_t batch, int64_t cu) {
    const float outputs = (float)M * (float)N * (float)batch * 4e-6f, beyond = (float)(KB > 128 ? KB - 128 : 0) / 384.0f;
    const bool ragged = N % 16 != 0;
    DirectChoice best{0, 3e38f};
#pragma unroll
    for (int i = 0; i < (int)(sizeof(kDirectCost) / sizeof(kDirectCost[0])); ++i) {
        const DirectCost& c = kDirectCost[i];
        if (KB > kSmallMaxKB && !c.any_k) continue;    // their declined tiles keep all exponents of A in LDS
        if (KB <= kDirectOnceBlocks && c.any_k) continue;      // the large tiles take a K of one iteration in one form
        const int64_t tiles = ((M + c.tm - 1) / c.tm) * ((N + c.tn - 1) / c.tn) * batch;
        const float steps = (float)(((KB + c.kg - 1) / c.kg + 3) / 4), grow = 1.0f + c.grow * beyond;
        const bool two = c.resident == 2 && tiles > cu;
        const int64_t slots = two ? 2 * cu : cu, rounds = tiles / slots, rest = tiles - rounds * slots;
        auto round_us = [&](bool pair, float fill) {
            return pair ? c.fixed2 + steps * (c.step2 + c.fill2 * fill) * grow : c.fixed1 + steps * (c.step1 + c.fill1 * fill) * grow;
        };
        float t = c.base + outputs * (ragged ? c.ragged : c.store) + (float)rounds * round_us(two, 1.0f);
        if (rest > 0) t += two && rest > cu ? round_us(true, (float)rest / (float)slots) : round_us(false, (float)rest / (float)cu);
        if (t < best.us) best = {i, t};
    }
    if (KB <= kDirectOnceBlocks) {
        // tiles of one iteration flow through the chip rather than in rounds: latency, then tiles and outputs.  (12 %
        // below the fit: where it is close to the small tiles it wins more often than they do.)
        const float tiles = (float)(((M + 127) / 128) * ((N + 127) / 128) * batch) / (float)cu, more = tiles > 1.61f ? tiles - 1.61f : 0.0f;
        const float t = 5.1f + 0.34f * (float)KB + more * (1.30f + 0.147f * (float)KB) + outputs * (ragged ? 0.40f : 0.071f);
        if (t < best.us) best = {kOnceShape, t};
    }
    return best;
}

// At most this many rows of A or of W in one launch: the kernel addresses an operand with 32-bit byte offsets, the rows
// of A give at most 65535 tiles of the smallest shape along the grid's y, and those of W at most 2^22 along its x, of
// 512 threads each.  Whole tiles while that many rows fit; at least 4 rows for any K / 32 < 2^26.
int64_t gemm_direct_max_rows(int64_t KB, bool weight) {
    const int64_t offsets = ((int64_t)1 << 28) / (KB > 0 ? KB : 1), grid = weight ? (int64_t)1 << 27 : (int64_t)65535 * 32;
    const int64_t rows = offsets < grid ? offsets : grid;
    return rows >= 512 ? rows / 512 * 512 : rows;
}

int launch_gemm_f8(bool mx, bool bf16, const GemmParams& p, int64_t batch, int shape, hipStream_t stream) {
    switch (shape) {
        case 0: return launch<DirectShape<1, 1, 1, 1, 8>>(mx, bf16, p, batch, stream);
        case 1: return launch<DirectShape<1, 1, 2, 2, 4>>(mx, bf16, p, batch, stream);
        case 2: return launch<DirectShape<1, 1, 2, 2, 2>>(mx, bf16, p, batch, stream);
        case 3: return launch<DirectShape<2, 2, 2, 2, 2>, DirectShape<1, 1, 2, 2, 2>>(mx, bf16, p, batch, stream);
        case 4: return launch<DirectShape<2, 2, 2, 2, 1>, DirectShape<1, 1, 2, 2, 1>>(mx, bf16, p, batch, stream);
        case 5: return launch<DirectShape<2, 2, 4, 2, 1>, DirectShape<1, 1, 2, 2, 2>>(mx, bf16, p, batch, stream);
        default: return launch<DirectShape<2, 2, 2, 2, 1, true>, DirectShape<1, 1, 2, 2, 1, true>>(mx, bf16, p, batch, stream);
    }
}

}  // namespace dfp4
