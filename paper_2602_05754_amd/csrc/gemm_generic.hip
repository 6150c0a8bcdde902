// Grouped GEMM for every shape, on the matrix cores: the fp32 configuration and whatever bf16
// problems the 256 x 256-tile kernel does not take (fewer than 256 rows or columns, pitches or
// extents that are no multiple of 8).  Computes both halves of a backward action (TimelyFreeze
// Sec. 3.2.1): the input gradient dX = dY W^T (layout kNT) and the parameter gradient dW = X^T dY
// (layout kTN); frozen tensors never reach this file.
//
// fp32 operands go through v_mfma_f32_16x16x4_f32 (true fp32 products and sums, twice the rate of
// the vector FMA; in the smallest tiles through the 64-bit form), bf16 operands through
// v_mfma_f32_16x16x32_bf16.
//
// Against plain fp32 vector FMAs in 64 x 64 tiles (what this file held before): fp32 stage of width 1024,
// 1000 tokens, input gradients of two blocks 740 -> 375 us (59 -> 118 TFLOP/s); bf16, 200 tokens of a
// LLaMA-1B block pair, input gradients 1195 -> 104 us; bf16, weight gradients over 3001 tokens 9435 ->
// 870 us.  Counters: fp32 has the matrix pipe busy 77 % of the cycles (weight gradients 70 %).  bf16 has no unit
// full (3001 tokens: matrix pipe 44 %, LDS 45 %, address unit 50 %, no bank conflicts), two waves per SIMD that wait
// half of the time for operands on their way through L1, registers and LDS; 200 tokens: a unit holds a
// tile 65 % of the time, matrix pipe 24 %: chains of up to 128 steps in few tiles.
//
// One output tile per workgroup of four waves in a 2 x 2 grid.  The contraction advances 128 bytes
// per operand row (64 bf16 or 32 fp32 values) through two LDS stages; the 16-byte pieces of the
// steps ahead travel through registers, so that no element needs an alignment beyond its own
// (a global 128-bit load takes any address) and what lies outside the contraction can be zeroed.
//   kNT stage: [row][128 bytes of contraction], 16-byte chunks of a row XOR-swizzled; an operand
//              is one 128-bit LDS read per lane.
//   kTN stage: [contraction][rows] as in memory.  bf16: operands by the LDS transpose read; fp32:
//              by four 32-bit reads.  32- / 64-byte units XOR-swizzled against bank conflicts.
// Nothing is ever read outside a matrix: rows past its end are clamped to the last one (their
// outputs are not stored); pieces that run over the end of a row stay inside the matrix except in
// its last row, and the last contraction step checks that and zeroes the values past the contraction.
#include "gemm_tile.h"

namespace tf {
namespace {

template <typename TIn, bool kContig, bool kOutBf16, bool kAccumulate, int kTileM, int kTileN>
__global__ __launch_bounds__(kThreads, 2) void gemm_generic_kernel(GemmBatch batch) {
    __shared__ __attribute__((aligned(1024))) char lds[2 * (kTileM + kTileN) * kStepBytes];
    const int lt = logical_tile(int(blockIdx.x), batch.total_tiles);
    const GemmProblem& P = batch.p[find_problem(batch, lt)];
    contract_tile<TIn, kContig, kOutBf16, kAccumulate, kTileM, kTileN>(P, tile_at<kTileM, kTileN>(P, lt), lds);
}

// The launch shapes.  step_us, chain_us: a step's share of a compute unit when all are full, and its
// time in a workgroup that has the unit to itself; tile_steps: what a tile costs beside its steps.
// Measured (LLaMA-1B, LLaMA-8B and small widths, 32 to 3001 tokens, both layouts): the bf16 steps wait
// for the L1 and LDS traffic of their operands (input gradients of a LLaMA-1B block, 3001
// tokens: 128 x 128 tiles 906 TFLOP/s, 128 x 64 753, 64 x 64 598), the fp32 steps by the matrix pipe
// (2048 tokens, width 1024: 64 x 64 tiles 545 us, 32 x 64 558, 128 x 64 553; width 512, 512 tokens: 32 x 64
// 47 us, 64 x 64 64, 32 x 32 in 64 bits 78).  Small tiles are for calls with few of them: an
// fp32 chain of 64 steps takes 30 us in 32 x 32 and 32 x 64 tiles, 46 in 64 x 64 and 155 in 128 x 128.
constexpr GenericShape kShapes16[] = {{64, 64, 0.222f, 0.40f, 2.7f}, {128, 64, 0.348f, 0.45f, 3.1f}, {128, 128, 0.575f, 0.60f, 3.5f}};
constexpr GenericShape kShapes32[] = {{32, 32, 0.28f, 0.43f, 1.0f}, {32, 64, 0.275f, 0.42f, 1.2f}, {64, 64, 0.53f, 0.62f, 1.5f}};
static_assert(sizeof(kShapes16) == kGenericShapes * sizeof(GenericShape) && sizeof(kShapes32) == sizeof(kShapes16), "as many for both types");

// Both halves of an fp32 backward in one launch: neither waits for the other, and a launch of few tiles, or the end of a longer
// one, leaves most units idle.  Each half has its own tiles.  Whole calls, us, against two launches: one block of widths 1024 / 512 / 3000, 20 tokens
// 68 -> 49, 150 tokens 90 -> 70, 2000 tokens 693 -> 682; 512 / 256 / 1700, 150 tokens 49 -> 34, 700 tokens 90 -> 79; two blocks of 1024 /
// 256 / 2731, 1000 tokens 604 -> 591; calls that wait for the host (128 / 32 / 400) 27 -> 23.
template <bool kAccumulate, int kShapeX, int kShapeW>
__global__ __launch_bounds__(kThreads, 2) void gemm_generic_both_kernel(GemmBatch batch) {
    constexpr int kXm = kShapes32[kShapeX].tile_m, kXn = kShapes32[kShapeX].tile_n, kWm = kShapes32[kShapeW].tile_m, kWn = kShapes32[kShapeW].tile_n;
    __shared__ __attribute__((aligned(1024))) char lds[2 * (kXm + kXn > kWm + kWn ? kXm + kXn : kWm + kWn) * kStepBytes];
    const int lt = logical_tile(int(blockIdx.x), batch.total_tiles);
    const int pi = find_problem(batch, lt);
    const GemmProblem& P = batch.p[pi];
    if (batch.tn >> pi & 1) contract_tile<float, false, false, kAccumulate, kWm, kWn>(P, tile_at<kWm, kWn>(P, lt), lds);
    else contract_tile<float, true, false, false, kXm, kXn>(P, tile_at<kXm, kXn>(P, lt), lds);
}

template <typename TIn, bool kContig, bool kOutBf16, bool kAccumulate>
void launch(hipStream_t stream, const GemmBatch& batch, int shape) {
    const dim3 grid(batch.total_tiles), block(kThreads);
    constexpr bool k16 = sizeof(TIn) == 2;
    constexpr const GenericShape* kS = k16 ? kShapes16 : kShapes32;
    if (shape == 0)
        hipLaunchKernelGGL((gemm_generic_kernel<TIn, kContig, kOutBf16, kAccumulate, kS[0].tile_m, kS[0].tile_n>), grid, block, 0, stream, batch);
    else if (shape == 1)
        hipLaunchKernelGGL((gemm_generic_kernel<TIn, kContig, kOutBf16, kAccumulate, kS[1].tile_m, kS[1].tile_n>), grid, block, 0, stream, batch);
    else
        hipLaunchKernelGGL((gemm_generic_kernel<TIn, kContig, kOutBf16, kAccumulate, kS[2].tile_m, kS[2].tile_n>), grid, block, 0, stream, batch);
}

}  // namespace

const GenericShape& generic_shape(Dtype in_dtype, int shape) { return in_dtype == Dtype::BF16 ? kShapes16[shape] : kShapes32[shape]; }

hipError_t launch_gemm_generic(hipStream_t stream, GemmBatch& batch, int n_problems, int shape,
                               Layout layout, Dtype in_dtype, Dtype out_dtype, bool accumulate) {
    batch.n_problems = n_problems;
    if (n_problems == 0 || batch.total_tiles == 0) return hipSuccess;
    const bool contig = layout == Layout::kNT;
    if (in_dtype == Dtype::F32) {
        if (out_dtype != Dtype::F32) return hipErrorInvalidValue;
        if (contig) accumulate ? launch<float, true, false, true>(stream, batch, shape) : launch<float, true, false, false>(stream, batch, shape);
        else        accumulate ? launch<float, false, false, true>(stream, batch, shape) : launch<float, false, false, false>(stream, batch, shape);
    } else if (contig) {
        if (out_dtype != Dtype::BF16 || accumulate) return hipErrorInvalidValue;       // an input gradient has the inputs' type
        launch<uint16_t, true, true, false>(stream, batch, shape);
    } else if (out_dtype == Dtype::BF16) {
        launch<uint16_t, false, true, false>(stream, batch, shape);
    } else {
        accumulate ? launch<uint16_t, false, false, true>(stream, batch, shape) : launch<uint16_t, false, false, false>(stream, batch, shape);
    }
    return hipGetLastError();
}

hipError_t launch_gemm_generic_both(hipStream_t stream, GemmBatch& batch, int n_problems, int shape_x, int shape_w, bool accumulate) {
    batch.n_problems = n_problems;
    if (n_problems == 0 || batch.total_tiles == 0) return hipSuccess;
    const dim3 grid(batch.total_tiles), block(kThreads);
    static_for<2 * kGenericShapes * kGenericShapes>([&](auto i) {
        constexpr bool kAdd = i % 2;
        constexpr int kX = i / 2 / kGenericShapes, kW = i / 2 % kGenericShapes;
        if (kAdd == accumulate && kX == shape_x && kW == shape_w) hipLaunchKernelGGL((gemm_generic_both_kernel<kAdd, kX, kW>), grid, block, 0, stream, batch);
    });
    return hipGetLastError();
}

}  // namespace tf
