// Weight gradients of few tokens, dW = X^T dY (TimelyFreeze Sec. 3.2.1) in bf16: from 64 tokens to the some hundred
// from which on a tile of 256 x 256 has enough steps to be worth its epilogue.  The outputs are as large as the weights and a
// tile has 2 to 16 steps: what the 256 x 256-tile kernel spends its time on is storing (and fetching what it adds to) with
// its matrix cores idle, one workgroup per compute unit.  Here three or four workgroups of smaller tiles share a unit, so that
// one stores while others contract, and the values to be added to are on their way before a tile's last steps.
//
// What bounds it: 64 tokens, HBM (243 MB stored in 47 us where the outputs' old lines are in the memory-side cache, 58 where they are not,
// as for all figures from here on).  More tokens: tiles of 128 x 128 read 32 KB of LDS and fill 16 KB for 256 cycles of MFMAs a step, so LDS,
// matrix cores and the unit's one memory path are each half busy (counters, 200 tokens: 55 %, 34 %, 51 %) and three workgroups do not
// fill any; stores that wait for HBM hold the loads behind them.  256 x 128 tiles, two workgroups per unit, load less; with values to add
// to they need more registers than there are.  Workgroups that stay for several tiles and fetch the next one's first steps ahead of the
// stores: 128 x 128 tiles 105 us instead of 96, 256 x 128 88 instead of 91, outputs in the cache 79 instead of 76: not worth a second
// scheme.  Four workgroups of 128 x 128 with two stages (93), raised wave priority around the MFMAs: no gain.  Ordinary stores instead
// of non-temporal ones: 100 instead of 79.
//
// us, in brackets the better one of the 256 x 256-tile and the generic kernel; two LLaMA-1B blocks, bf16 outputs, 64 tokens 58 (62), 200 90 (92); fp32, 64
// tokens 85 (110); added to fp32, 64 tokens 165 (214), 200 176 (214), 512 229 (244); two blocks of widths 1024 / 256 / 2816, bf16, 64 tokens 14
// (21), 200 21 (29), 512 32 (37); added to, 200 tokens 41 (59), 1024 79 (85); one block of widths 2816 / 1408 / 8200, added to, 200 tokens 150 (207).
//
// The sums are those of the other kernels, in the same order: the same bits.
#include "gemm_device.h"

#include <cmath>

namespace tf {
namespace {

constexpr int kWaves = 4, kThreads = 64 * kWaves;
constexpr int kGroupM = 8;                      // tile rows per L2 locality group

enum Out { kBf16 = 0, kF32 = 1, kAdd = 2 };

template <int kRows, int kCols>
struct Short {
    static constexpr int kRowsW = kRows / 2, kColsW = kCols / 2;                     // a wave's part of the tile, 2 x 2
    static constexpr int kFragA = kRowsW / 16, kFragB = kColsW / 16;
    static constexpr int kLoadsA = kRows / 64, kLoads = kLoadsA + kCols / 64;         // per wave and step, 1 KB each
    static constexpr int kPitchA = kRows * 2, kPitchB = kCols * 2;                   // bytes of a stage row
    static constexpr int kStageA = kRows * 64, kStage = kStageA + kCols * 64;
    static constexpr int kDeep = 3;                                                 // stages: two steps ahead
    static constexpr int kLds = kDeep * kStage;
};

// Stage: [32 contraction rows][rows of the operand], as in memory; 32-byte units of a row XOR-swizzled.  The transpose
// read of a 16-row block takes a unit of contraction rows 8 G + x, x = 0..3, G = lane / 16, 32 lanes at a time: 8 rows
// whose units must fall into different banks (a pitch of 256 bytes is all banks, one of 128 half of them).
template <int kPitch>
__device__ __forceinline__ constexpr int unit_xor(int t) {
    return kPitch >= 256 ? 4 * ((t >> 3) & 1) + (t & 3) : 2 * ((t >> 3) & 1) + ((t >> 1) & 1);
}

template <int kRows, int kCols, int kOut, int kPerUnit>
__global__ __launch_bounds__(kThreads, kPerUnit) void gemm_short_kernel(GemmBatch batch) {
    typedef Short<kRows, kCols> S;
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    static_assert(kMaxProblemsPerLaunch == 64, "one lane per problem");
    const int lt = logical_tile(int(blockIdx.x), batch.total_tiles);
    const bool started = lane < batch.n_problems && batch.p[lane].tile_start <= lt;
    const int pi = __builtin_amdgcn_readfirstlane(__popcll(__ballot(started)) - 1);
    const GemmProblem& P = batch.p[pi];
    const int M = P.M, N = P.N, Kc = P.Kc;
    const int tiles_m = (M + kRows - 1) / kRows, tiles_n = (N + kCols - 1) / kCols;
    int t = lt - P.tile_start;
    const int per_group = kGroupM * tiles_n;
    const int first_m = (t / per_group) * kGroupM;
    const int gsz = min(tiles_m - first_m, kGroupM);
    t %= per_group;
    const int m0 = (first_m + t % gsz) * kRows, n0 = (t / gsz) * kCols;

    // Steps of 32 values.  A contraction that is no multiple of 64 ends in its last 64 values, those contracted before
    // masked out, as on the other kernels; where that masks a whole step, the step is left out.
    const int whole = (Kc / 64) * 2, rest = Kc % 64;
    const int steps = whole + (rest > 32 ? 2 : rest > 0 ? 1 : 0);
    const int masked = rest > 32 ? 64 - rest : rest > 0 ? 32 - rest : 0;     // values masked out of step `whole`
    auto at_step = [&](int s) { return s < whole ? 32 * s : Kc - 32 * (steps - s); };

    const uint32_t lds_base = __builtin_amdgcn_readfirstlane(uint32_t(reinterpret_cast<uintptr_t>(TF_LPTR(lds))));
    // Load p of a step: 1 KB of whole stage rows of X (p < kLoadsA) or of dY, straight to LDS.  What lies past the end of a row
    // is the row's last piece (its outputs are not stored).
    uint32_t off[S::kLoads];
#pragma unroll
    for (int p = 0; p < S::kLoads; ++p) {
        const bool of_a = p < S::kLoadsA;
        const int pieces = (of_a ? S::kPitchA : S::kPitchB) / 16;
        const int at = (wave + kWaves * (of_a ? p : p - S::kLoadsA)) * 64 + lane;        // piece of the operand's stage
        const int k = at / pieces, c = at % pieces;
        const int x = of_a ? unit_xor<S::kPitchA>(k) : unit_xor<S::kPitchB>(k);
        const int col = (((c >> 1) ^ x) << 4) + ((c & 1) << 3);
        off[p] = uint32_t(k) * uint32_t((of_a ? P.lda : P.ldb) * 2) + uint32_t(min((of_a ? m0 : n0) + col, (of_a ? M : N) - 8)) * 2;
    }
    auto load_stage = [&](int s, uint32_t stage) __attribute__((always_inline)) {
        const int64_t k = at_step(s);
        const char* const X = static_cast<const char*>(P.A) + k * (int64_t(P.lda) * 2);
        const char* const dY = static_cast<const char*>(P.B) + k * (int64_t(P.ldb) * 2);
        static_for<S::kLoads>([&](auto p) __attribute__((always_inline)) {
            constexpr int kTo = p < S::kLoadsA ? p * kWaves * 1024 : S::kStageA + (p - S::kLoadsA) * kWaves * 1024;
            direct_load_16B<kTo>(p < S::kLoadsA ? X : dY, off[p], stage + wave * 1024);
        });
    };

    f32x4 acc[S::kFragA][S::kFragB];
#pragma unroll
    for (int i = 0; i < S::kFragA; ++i)
#pragma unroll
        for (int j = 0; j < S::kFragB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int wm = wave >> 1, wn = wave & 1;
    const int q = lane >> 4, tr = 8 * q + ((lane & 15) >> 2);          // contraction row of this lane's transpose reads
    auto fragment = [&](uint32_t at, int pitch) __attribute__((always_inline)) {
        typedef __attribute__((address_space(3))) char* P3;
        const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LdsBf16x4Ptr)(P3)(uintptr_t)at);
        const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LdsBf16x4Ptr)(P3)(uintptr_t)(at + 4 * pitch));
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    };
    uint32_t a_at[S::kFragA], b_at[S::kFragB];
#pragma unroll
    for (int i = 0; i < S::kFragA; ++i) a_at[i] = tr * S::kPitchA + (((wm * S::kFragA + i) ^ unit_xor<S::kPitchA>(tr)) << 5) + ((lane & 3) << 3);
#pragma unroll
    for (int j = 0; j < S::kFragB; ++j) b_at[j] = S::kStageA + tr * S::kPitchB + (((wn * S::kFragB + j) ^ unit_xor<S::kPitchB>(tr)) << 5) + ((lane & 3) << 3);
    auto contract = [&](uint32_t stage, int drop) __attribute__((always_inline)) {
        bf16x8 fa[S::kFragA], fb[S::kFragB];
#pragma unroll
        for (int j = 0; j < S::kFragB; ++j) fb[j] = fragment(stage + b_at[j], S::kPitchB);
#pragma unroll
        for (int i = 0; i < S::kFragA; ++i) fa[i] = fragment(stage + a_at[i], S::kPitchA);
        if (drop > 0) {                                 // of a lane's 8 values 8 q + 0..7
            const int n = drop - 8 * q;
            U4 keep;
#pragma unroll
            for (int d = 0; d < 4; ++d) keep[d] = (2 * d >= n ? 0xffffu : 0u) | (2 * d + 1 >= n ? 0xffff0000u : 0u);
#pragma unroll
            for (int i = 0; i < S::kFragA; ++i) fa[i] = __builtin_bit_cast(bf16x8, U4(__builtin_bit_cast(U4, fa[i]) & keep));
#pragma unroll
            for (int j = 0; j < S::kFragB; ++j) fb[j] = __builtin_bit_cast(bf16x8, U4(__builtin_bit_cast(U4, fb[j]) & keep));
        }
        // D rows <- n (rows of dY^T), D columns <- m: a lane then owns 4 consecutive n of one output row
#pragma unroll
        for (int i = 0; i < S::kFragA; ++i)
#pragma unroll
            for (int j = 0; j < S::kFragB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
    };

    // Outputs leave by whole rows of the tile, 16 bytes per lane; fp32 values that are added to come the same way, all of
    // them on their way before the last steps are contracted.
    constexpr int kOutE = kOut == kBf16 ? 8 : 4, kLanes = kCols / kOutE, kRowsPass = kThreads / kLanes, kPasses = kRows / kRowsPass;
    const int oc = int(threadIdx.x) % kLanes, orow = int(threadIdx.x) / kLanes, on = n0 + oc * kOutE;
    // turned around in the stages, the waves' first and second halves one after the other if all does not fit
    constexpr int kChunk = kOut == kBf16 ? 8 : 16, kRow = kCols / 4 * kChunk, kTurn = kCols / 4 < 16 ? kCols / 4 - 1 : 15;
    constexpr int kParts = (kRows * kRow + S::kLds - 1) / S::kLds, kFragsPart = S::kFragA / kParts, kRowsPart = kRows / kParts;
    static_assert(kParts == 1 || kParts == 2, "one half of each wave's rows at a time");
    constexpr int kPassesPart = kPasses / kParts, kOld = kOut == kAdd ? kPassesPart : 0;
    auto out_row = [&](int p) __attribute__((always_inline)) {         // of the tile, in pass p
        const int r = (p % kPassesPart) * kRowsPass + orow;
        return kParts == 1 ? r : (r / (kRowsPart / 2)) * S::kRowsW + (p / kPassesPart) * (kRowsPart / 2) + r % (kRowsPart / 2);
    };
    f32x4 old[kPassesPart];                             // of one part; the second part's, each where one of the first has been used
    auto fetch_old = [&](int p) __attribute__((always_inline)) {
        // (past the tensor's end: its last whole piece)
        const float* const c = static_cast<const float*>(P.C) + int64_t(min(m0 + out_row(p), M - 1)) * N + min(on, N - 4);
        old[p % kPassesPart] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(c));
    };

    for (int s = 0; s < S::kDeep - 1 && s < steps; ++s) load_stage(s, lds_base + s * S::kStage);
    uint32_t stage = lds_base, filled = lds_base + (S::kDeep - 1) * S::kStage;
    auto next = [&](uint32_t s) { return s + S::kStage == lds_base + S::kLds ? lds_base : s + S::kStage; };
    int s = 0;
    for (; s + S::kDeep <= steps; ++s) {
        wait_loads<S::kLoads * (S::kDeep - 2)>();
        __syncthreads();                                // step s is there; every wave has read step s - 1
        load_stage(s + S::kDeep - 1, filled);
        contract(stage, 0);                             // (what is masked is among the last two steps)
        filled = stage;
        stage = next(stage);
    }
    if constexpr (kOut == kAdd) {                       // behind all of the stages' loads, and counted as such below
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int p = 0; p < kPassesPart; ++p) fetch_old(p);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    }
    for (; s < steps; ++s) {
        wait_stages<S::kLoads, S::kDeep - 2, kOld>(steps - 1 - s);
        __syncthreads();
        contract(stage, s == whole ? masked : 0);
        stage = next(stage);
    }
    __syncthreads();
    wait_for_sums(acc);

    // Epilogue.  acc[i][j][e] is C[m][n], m = 16 i + lane % 16, n = 16 j + 4 (lane / 16) + e of the wave's part (chunks of
    // 4 values, XOR-swizzled).
#pragma unroll
    for (int h = 0; h < kParts; ++h) {
        if (h > 0) __syncthreads();
#pragma unroll
        for (int i = 0; i < kFragsPart; ++i)
#pragma unroll
            for (int j = 0; j < S::kFragB; ++j) {
                const int r = wm * (kRowsPart / 2) + 16 * i + (lane & 15), c = wn * (S::kColsW / 4) + 4 * j + q;
                char* const to = lds + r * kRow + ((c ^ (r & kTurn)) * kChunk);
                const f32x4 v = acc[h * kFragsPart + i][j];
                if constexpr (kOut == kBf16) *reinterpret_cast<U2*>(to) = U2{f32x2_to_bf16x2(v[0], v[1]), f32x2_to_bf16x2(v[2], v[3])};
                else *reinterpret_cast<f32x4*>(to) = v;
            }
        __syncthreads();
#pragma unroll
        for (int p = 0; p < kPassesPart; ++p) {
            const int r = p * kRowsPass + orow;
            const int m = m0 + out_row(h * kPassesPart + p);
            if constexpr (kOut == kBf16) {
                // chunks 2 oc and 2 oc + 1 sit in one aligned pair, swapped in odd rows
                const U4 v = *reinterpret_cast<const U4*>(lds + r * kRow + (((2 * oc) ^ (r & (kTurn - 1))) * kChunk));
                const U4 x = (r & 1) ? U4{v.z, v.w, v.x, v.y} : v;
                if (m < M && on < N) __builtin_nontemporal_store(x, reinterpret_cast<U4*>(static_cast<uint16_t*>(P.C) + int64_t(m) * N + on));
            } else {
                f32x4 v = *reinterpret_cast<const f32x4*>(lds + r * kRow + ((oc ^ (r & kTurn)) * kChunk));
                if constexpr (kOut == kAdd) {
                    v += old[p];
                    if (h + 1 < kParts) fetch_old(kPassesPart + p);
                }
                if (m < M && on < N) __builtin_nontemporal_store(v, reinterpret_cast<f32x4*>(static_cast<float*>(P.C) + int64_t(m) * N + on));
            }
        }
    }
}

template <int kRows, int kCols, int kOut, int kPerUnit>
hipError_t launch_kernel(hipStream_t stream, const GemmBatch& batch) {
    auto kern = gemm_short_kernel<kRows, kCols, kOut, kPerUnit>;
    constexpr int kLds = Short<kRows, kCols>::kLds;
    if constexpr (kLds > 65536) {
        // more than 64 KB of dynamic LDS are allowed once per kernel and device
        constexpr int kMaxDevices = 64;
        static bool lds_allowed[kMaxDevices] = {false};
        int dev = -1;
        if (hipGetDevice(&dev) != hipSuccess || dev >= kMaxDevices) dev = -1;
        if (dev < 0 || !lds_allowed[dev]) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
            if (e != hipSuccess) return e;
            if (dev >= 0) lds_allowed[dev] = true;
        }
    }
    hipLaunchKernelGGL(kern, dim3(batch.total_tiles), dim3(kThreads), kLds, stream, batch);
    return hipGetLastError();
}
template <int kRows, int kCols, int kPerUnit>
hipError_t launch_shape(hipStream_t stream, const GemmBatch& batch, int out) {
    switch (out) {
        case kBf16: return launch_kernel<kRows, kCols, kBf16, kPerUnit>(stream, batch);
        case kF32: return launch_kernel<kRows, kCols, kF32, kPerUnit>(stream, batch);
        default: return launch_kernel<kRows, kCols, kAdd, kPerUnit>(stream, batch);
    }
}

// The launch shapes.  A step's and a tile's share of a compute unit when all are full, a step in a launch's longest chain, what a
// launch takes beside them; for each kind of output how much of the smaller of computing and storing is left, and the stores per
// MB (those added to counted once), in whole cache lines and not; see short_launch_us().
constexpr ShortShape kShapes[kShortShapes] = {
    {128, 64, 0.185f, 0.43f, 0.211f, 5.5f, {{0.213f, 0.11f, 0.6f}, {0.468f, 0.125f, 0.309f}, {0.438f, 0.3f, 0.455f}}},
    {128, 128, 0.263f, 1.07f, 0.287f, 6.3f, {{0.064f, 0.11f, 0.443f}, {0.496f, 0.117f, 0.235f}, {0.459f, 0.29f, 0.381f}}},
    {256, 128, 0.417f, 2.46f, 0.474f, 7.1f, {{0.083f, 0.11f, 0.469f}, {0.497f, 0.127f, 0.242f}, {0, HUGE_VALF, HUGE_VALF}}}};

}  // namespace

const ShortShape& short_shape(int shape) { return kShapes[shape]; }

bool short_shape_ok(int64_t M, int64_t N, int64_t Kc, int64_t lda, int64_t ldb) {
    // 16-byte direct loads: rows on 16-byte boundaries, a step's rows within 32-bit offsets
    constexpr int64_t kMaxPitch = int64_t(1) << 22;
    return M > 0 && N > 0 && M % 8 == 0 && N % 8 == 0 && Kc >= 64 && lda % 8 == 0 && ldb % 8 == 0 && lda <= kMaxPitch && ldb <= kMaxPitch;
}
hipError_t launch_gemm_short(hipStream_t stream, GemmBatch& batch, int n_problems, int shape, Dtype out_dtype, bool accumulate) {
    batch.n_problems = n_problems;
    if (n_problems == 0 || batch.total_tiles == 0) return hipSuccess;
    if (accumulate && out_dtype != Dtype::F32) return hipErrorInvalidValue;
    for (int i = 0; i < n_problems; ++i) {
        const GemmProblem& p = batch.p[i];
        if (p.n_seg != 1 || ~p.row_bits != 0 || !short_shape_ok(p.M, p.N, p.Kc, p.lda, p.ldb)) return hipErrorInvalidValue;
    }
    const int out = out_dtype == Dtype::BF16 ? kBf16 : accumulate ? kAdd : kF32;
    switch (shape) {
        case 0: return launch_shape<128, 64, 4>(stream, batch, out);
        case 1: return launch_shape<128, 128, 3>(stream, batch, out);
        case 2: return out == kAdd ? hipErrorInvalidValue : out == kBf16 ? launch_kernel<256, 128, kBf16, 2>(stream, batch) : launch_kernel<256, 128, kF32, 2>(stream, batch);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace tf
