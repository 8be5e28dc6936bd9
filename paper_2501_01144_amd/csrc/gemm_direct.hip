// Products of prepared operands of more than 256 rows that are too small for the large kernel, on the int8 matrix cores (the
// tile: gemm_int8_tile.h), and the choice of a tile shape for these and for gemm_f8_kernel (gemm_f8.hip), which takes the
// same shapes.  Here whether a tile is summed exactly in int32 or block by block is decided, and counted, from masks that were prepared with
// the operands.
#include "gemm_int8_tile.h"

namespace dfp4 {
namespace {

template <bool MX, bool BF16, class S>
__global__ __launch_bounds__(S::kThreads, S::kWavesPerSimd) void gemm_direct_kernel(GemmParams p) {
    __shared__ TileLds<S> u;
    int8_tile<MX, BF16, S>(p, u, blockIdx.z, (int)blockIdx.y, (int)blockIdx.x);
}

template <class S>
int launch(bool mx, bool bf16, const GemmParams& p, int64_t batch, hipStream_t stream) {
    dim3 g((unsigned)((p.N + S::kTn - 1) / S::kTn), (unsigned)((p.M + S::kTm - 1) / S::kTm), (unsigned)batch);
    dispatch_mx_bf16(mx, bf16, [&](auto mxc, auto bc) {
        hipLaunchKernelGGL((gemm_direct_kernel<decltype(mxc)::value, decltype(bc)::value, S>), g, dim3(S::kThreads), 0, stream, p);
    });
    return check_launch();
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

int launch_gemm_direct(bool mx, bool bf16, const GemmParams& p, int64_t batch, int shape, hipStream_t stream) {
    if (!p.ref_a) return launch_gemm_f8(mx, bf16, p, batch, shape, stream);
    switch (shape) {
        case 0: return launch<DirectShape<1, 1, 1, 1, 8>>(mx, bf16, p, batch, stream);
        case 1: return launch<DirectShape<1, 1, 2, 2, 4>>(mx, bf16, p, batch, stream);
        case 2: return launch<DirectShape<1, 1, 2, 2, 2>>(mx, bf16, p, batch, stream);
        case 3: return launch<DirectShape<2, 2, 2, 2, 2>>(mx, bf16, p, batch, stream);
        case 4: return launch<DirectShape<2, 2, 2, 2, 1>>(mx, bf16, p, batch, stream);
        case 5: return launch<DirectShape<2, 2, 4, 2, 1>>(mx, bf16, p, batch, stream);
        default: return launch<DirectShape<2, 2, 2, 2, 1, true>>(mx, bf16, p, batch, stream);
    }
}

}  // namespace dfp4
