// Input gradients of few tokens, dX = dY W^T (TimelyFreeze Sec. 3.2.1) in bf16: from one row to the thousand or two
// from which on the 256 x 256-tile kernel has enough tiles.  Most of the bytes are weights that are read once, and
// a launch is a few hundred tiles, each a chain of Kc / 64 short steps: what it takes is how long a step takes.
//
// What bounds a step, measured: (a) a compute unit gets about 60 GB/s of lines that miss its L2 (130 of those that hit),
// whatever the number of loads asked for ahead, and a load that hits waits for those that miss in front of it: rows of
// dY, which all workgroups share, arrive no earlier than the weights.  So both come from one ring of stages, as deep as the
// LDS allows, straight to LDS.  A second, deeper ring for the weights alone, touches of dY further ahead, and the steps ahead in
// registers (six stages, but stores to LDS at half its rate) were each slower.  (b) The LDS: 128 x 128 tiles read 64 KB
// and are filled with 32 KB a step, 750 cycles of 128 bytes, against 512 of MFMAs.  Four waves, 2 x 2, each a quarter of the
// tile; the reads of the next half step's fragments and the loads ride behind the MFMAs of this one, one by one: issued
// in one go they hold the wave until the LDS has taken them (256 x 128 tiles, operands in L2: 0.64 -> 0.53 us a step).
// Waves of their own for the loads: no difference.
//
// us, in brackets with the generic kernel's 64 x 64 to 128 x 128 tiles through registers: two LLaMA-1B blocks (243 MB of
// weights), 64 tokens 51 (70), 128 61 (78), 200 71 (103), 256 81 (108), 512 118 (150), 1024 218 (253 on 256 x 256 tiles); one
// LLaMA-8B block, 64 tokens 96 (124), 256 151 (192), 512 207 (243); one block of widths 1024 / 256 / 2816, 64 tokens 16
// (22); of width 256, 5.2 (8.0).  With three sets of buffers in turn, which leave less of the weights in the memory-side cache, the two LLaMA-1B
// blocks take 58 (72) at 64 tokens, 80 (104) at 200, 134 (159) at 512.
//   stage: [row][64 contraction values], 16-byte chunks of a row XOR-swizzled (nt_swizzle).
// The contraction's last step, where it is no multiple of 64, is the last 64 values with those contracted
// before masked out, as on the other two kernels: the same sums in the same order, the same bits.
#include "gemm_device.h"

namespace tf {
namespace {

constexpr int kWaves = 4, kThreads = 64 * kWaves;

template <int kRows, int kCols>
struct Narrow {
    static constexpr int kWavesM = 2, kWavesN = 2;
    static constexpr int kRowsW = kRows / kWavesM, kColsW = kCols / kWavesN;        // a wave's part of the tile
    static constexpr int kFragA = kRowsW / 16, kFragB = kColsW / 16;
    static constexpr int kLoadsA = kRows / 32, kLoads = kLoadsA + kCols / 32;        // per wave and step, 1 KB each
    static constexpr int kStageA = kRows * 128, kStage = kStageA + kCols * 128;
    static constexpr int kDeep = kRows == 64 ? 5 : kRows == 256 ? 3 : kCols == 64 ? 6 : 5;
    static constexpr int kLds = kDeep * kStage;         // 80 KB of the smallest shape, two workgroups per unit; else one
    static_assert(kLoads % 2 == 0 && kFragA * kFragB >= kLoads / 2, "a load behind an MFMA");
    static_assert(kWaves * kRowsW * kColsW * 2 <= kLds, "the output is turned around in the stages");
};

template <int kRows, int kCols>
__global__ __launch_bounds__(kThreads, 2) void gemm_narrow_kernel(GemmBatch batch) {       // (2: the sums stay in vector registers)
    typedef Narrow<kRows, kCols> S;
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    static_assert(kMaxProblemsPerLaunch == 64, "one lane per problem");
    const int lt = logical_tile(int(blockIdx.x), batch.total_tiles);
    const bool started = lane < batch.n_problems && batch.p[lane].tile_start <= lt;
    const int pi = __builtin_amdgcn_readfirstlane(__popcll(__ballot(started)) - 1);
    const GemmProblem& P = batch.p[pi];
    const int M = P.M, N = P.N, Kc = P.Kc;
    const int tiles_m = (M + kRows - 1) / kRows;
    const int t = lt - P.tile_start;
    const int m0 = (t % tiles_m) * kRows, n0 = (t / tiles_m) * kCols;
    const int steps = (Kc + 63) / 64;
    const int back = steps * 64 - Kc;                   // contraction values of the last step that were contracted before
    const uint32_t lds_base = __builtin_amdgcn_readfirstlane(uint32_t(reinterpret_cast<uintptr_t>(TF_LPTR(lds))));

    // byte offset of step s's contraction values in a row
    auto at_step = [&](int s) { return int64_t(min(s * 64, Kc - 64)) * 2; };
    const int r8 = lane >> 3, c8 = lane & 7;            // a load of 1 KB: 8 rows of 8 chunks

    const int wm = wave / S::kWavesN, wn = wave % S::kWavesN;

    // Load p of a step: 8 rows of dY (p < kLoadsA) or of W, 128 bytes each, straight to LDS.
    const char* const dY = static_cast<const char*>(P.A) + int64_t(m0) * P.lda * 2;
    const char* const W = static_cast<const char*>(P.B) + int64_t(n0) * P.ldb * 2;
    uint32_t off[S::kLoads];
#pragma unroll
    for (int p = 0; p < S::kLoads; ++p) {
        const bool of_a = p < S::kLoadsA;
        const int r = 8 * (wave + kWaves * (of_a ? p : p - S::kLoadsA)) + r8;
        off[p] = uint32_t(min(r, (of_a ? M - m0 : N - n0) - 1)) * uint32_t((of_a ? P.lda : P.ldb) * 2) + uint32_t((c8 ^ nt_swizzle(r)) << 4);
    }
    auto load = [&](auto p, int64_t at, uint32_t stage) __attribute__((always_inline)) {
        constexpr int q = (p + S::kLoadsA) % S::kLoads;         // the weights first, they come from furthest away
        direct_load_16B<q * kWaves * 1024>(q < S::kLoadsA ? dY + at : W + at, off[q], stage + wave * 1024);
    };
    constexpr int kHalf = S::kLoads / 2;                        // a step is fetched in two halves, behind the MFMAs of two half steps
    auto load_half = [&](auto half, int64_t at, uint32_t stage) __attribute__((always_inline)) {
        static_for<kHalf>([&](auto p) __attribute__((always_inline)) { load(std::integral_constant<int, p + half * kHalf>{}, at, stage); });
    };
    constexpr std::integral_constant<int, 0> u0{};
    constexpr std::integral_constant<int, 1> u1{};
    for (int s = 0; s < S::kDeep && s < steps; ++s) {
        load_half(u0, at_step(s), lds_base + s * S::kStage);
        if (s + 1 < S::kDeep) load_half(u1, at_step(s), lds_base + s * S::kStage);       // the last stage's second half: in step 0
    }

    f32x4 acc[S::kFragA][S::kFragB];
#pragma unroll
    for (int i = 0; i < S::kFragA; ++i)
#pragma unroll
        for (int j = 0; j < S::kFragB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // a lane's 16 bytes of 16-row block b, half step u: row 16 b + lane % 16, chunk (4 u + lane / 16) swizzled
    const uint32_t in_stage = uint32_t((lane & 15) * 128 + (((lane >> 4) ^ nt_swizzle(lane & 15)) << 4));
    const uint32_t a0 = wm * S::kRowsW * 128 + in_stage, b0 = S::kStageA + wn * S::kColsW * 128 + in_stage;
    typedef __attribute__((address_space(3))) const bf16x8* LdsBf16x8Ptr;
    bf16x8 fa[S::kFragA], fb[2][S::kFragB];
    // LDS addresses of half step u's fragments: formed well ahead of the reads, which add a constant
    uint32_t at_a, at_b;
    auto address = [&](auto u, uint32_t stage) __attribute__((always_inline)) {
        at_a = (a0 ^ (u << 6)) + stage;
        at_b = (b0 ^ (u << 6)) + stage;
        asm volatile("" : "+v"(at_a), "+v"(at_b));
    };
    // fragment q of half step u, in the order in which the MFMAs want them
    auto read_one = [&](auto u, auto q) __attribute__((always_inline)) {
        if constexpr (q < S::kFragB) fb[u][q] = *(LdsBf16x8Ptr)(uintptr_t)(at_b + q * 2048);
        else fa[q - S::kFragB] = *(LdsBf16x8Ptr)(uintptr_t)(at_a + (q - S::kFragB) * 2048);
    };
    constexpr int kFrags = S::kFragA + S::kFragB, kMfmas = S::kFragA * S::kFragB;
    // The MFMAs of half step u, and behind them, one by one, the reads of the next half step's fragments: issued
    // in one go they hold the wave until the LDS, which four waves share, has taken them, and its MFMAs with it.
    // And the loads of half a step, if any, spread over them.
    auto contract = [&](auto u, uint32_t next_stage, auto loads, int64_t at, uint32_t filled) __attribute__((always_inline)) {
        constexpr std::integral_constant<int, 1 - u> other{};
        address(other, next_stage);
        __builtin_amdgcn_sched_barrier(0);
        // D rows <- n (rows of W), D columns <- m: a lane then owns 4 consecutive n of one output row
        static_for<kMfmas>([&](auto k) __attribute__((always_inline)) {
            constexpr int i = k / S::kFragB, j = (i & 1) ? S::kFragB - 1 - k % S::kFragB : k % S::kFragB;
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[u][j], fa[i], acc[i][j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            constexpr int first = k * kFrags / kMfmas, end = (k + 1) * kFrags / kMfmas;
            // (a fragment of dY into the registers of the one before it, whose MFMAs have been issued)
            static_assert(end <= S::kFragB || (end - S::kFragB) * S::kFragB <= k + 1, "row by row");
            static_for<end - first>([&](auto q) __attribute__((always_inline)) { read_one(other, std::integral_constant<int, first + q>{}); });
            if constexpr (loads) {
                // a half step's loads: the second half of a step behind u = 0, the first half of the next behind u = 1
                constexpr int from = k * kHalf / kMfmas, to = (k + 1) * kHalf / kMfmas;
                static_for<to - from>([&](auto p) __attribute__((always_inline)) { load(std::integral_constant<int, (1 - u) * kHalf + from + p>{}, at, filled); });
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    auto mask = [&](auto u) __attribute__((always_inline)) {         // of a lane's 8 values 32 u + 8 (lane / 16) + 0..7
        const int n = back - 32 * u - 8 * (lane >> 4);
        U4 keep;
#pragma unroll
        for (int d = 0; d < 4; ++d) keep[d] = (2 * d >= n ? 0xffffu : 0u) | (2 * d + 1 >= n ? 0xffff0000u : 0u);
#pragma unroll
        for (int i = 0; i < S::kFragA; ++i) fa[i] = __builtin_bit_cast(bf16x8, U4(__builtin_bit_cast(U4, fa[i]) & keep));
#pragma unroll
        for (int j = 0; j < S::kFragB; ++j) fb[u][j] = __builtin_bit_cast(bf16x8, U4(__builtin_bit_cast(U4, fb[u][j]) & keep));
    };
    if (steps < S::kDeep) wait_stages<S::kLoads, S::kDeep - 1>(steps - 1);
    else wait_loads<S::kLoads * (S::kDeep - 2) + kHalf>();
    __syncthreads();
    uint32_t stage = lds_base;                          // of the step being contracted
    uint32_t filled = lds_base + (S::kDeep - 1) * S::kStage;    // being fetched to
    auto next = [&](uint32_t s) { return s + S::kStage == lds_base + S::kLds ? lds_base : s + S::kStage; };
    address(u0, stage);
    static_for<kFrags>([&](auto q) __attribute__((always_inline)) { read_one(u0, q); });
    // The barrier in the middle of step g: every wave has read all of step g, whose stage may be filled again; step
    // g + 1, of which every wave has awaited its own loads in front of it, may be read.
    int g = 0;
    for (; g + S::kDeep < steps; ++g) {
        contract(u0, stage, std::true_type{}, at_step(g + S::kDeep - 1), filled);
        wait_loads<S::kLoads * (S::kDeep - 2)>();
        __syncthreads();
        filled = stage;
        stage = next(stage);
        contract(u1, stage, std::true_type{}, at_step(g + S::kDeep), filled);
    }
    if (steps >= S::kDeep) load_half(u1, at_step(steps - 1), filled);
    for (; g < steps; ++g) {
        const bool masked = g + 1 == steps && back > 0;
        if (masked) mask(u0);
        contract(u0, stage, std::false_type{}, 0, 0);
        if (masked) mask(u1);
        wait_stages<S::kLoads, S::kDeep - 2>(steps - 2 - g);
        __syncthreads();
        stage = next(stage);
        contract(u1, stage, std::false_type{}, 0, 0);   // (behind the last step: reads what lies in the next stage, for nothing)
    }
    __syncthreads();

    // Epilogue.  acc[i][j][e] is C[m][n], m = 16 i + lane % 16, n = 16 j + 4 (lane / 16) + e of the wave's part: turned
    // around in the wave's own part of the stages (nothing is in flight towards them, every wave is past the last
    // barrier) and stored 16 bytes per lane, whole rows of the part.
    wait_for_sums(acc);
    constexpr int kRowBytes = S::kColsW * 2, kChunks = kRowBytes / 8, kLanes = kRowBytes / 16, kRowsPass = 64 / kLanes;
    char* const turn = lds + wave * (S::kRowsW * kRowBytes);
#pragma unroll
    for (int i = 0; i < S::kFragA; ++i)
#pragma unroll
        for (int j = 0; j < S::kFragB; ++j) {
            const int r = 16 * i + (lane & 15), c = 4 * j + (lane >> 4);
            *reinterpret_cast<U2*>(turn + r * kRowBytes + ((c ^ (r & (kChunks - 1))) << 3)) =
                U2{f32x2_to_bf16x2(acc[i][j][0], acc[i][j][1]), f32x2_to_bf16x2(acc[i][j][2], acc[i][j][3])};
        }
    const int cb = lane % kLanes, n = n0 + wn * S::kColsW + cb * 8;
#pragma unroll
    for (int r0 = 0; r0 < S::kRowsW; r0 += kRowsPass) {
        const int r = r0 + lane / kLanes, m = m0 + wm * S::kRowsW + r;
        // chunks 2 cb and 2 cb + 1 sit in one aligned pair, swapped in odd rows
        const U4 v = *reinterpret_cast<const U4*>(turn + r * kRowBytes + (((2 * cb) ^ (r & (kChunks - 2))) << 3));
        const U4 x = (r & 1) ? U4{v.z, v.w, v.x, v.y} : v;
        if (m >= M || n >= N) continue;
        uint16_t* const out = static_cast<uint16_t*>(P.C) + int64_t(m) * N + n;
        if (n + 8 <= N) {
            __builtin_nontemporal_store(x, reinterpret_cast<U4any*>(out));
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (n + e < N) out[e] = uint16_t(x[e >> 1] >> (16 * (e & 1)));
        }
    }
}

template <int kRows, int kCols>
hipError_t launch_shape(hipStream_t stream, const GemmBatch& batch) {
    auto kern = gemm_narrow_kernel<kRows, kCols>;
    constexpr int kLds = Narrow<kRows, kCols>::kLds;
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
    hipLaunchKernelGGL(kern, dim3(batch.total_tiles), dim3(kThreads), kLds, stream, batch);
    return hipGetLastError();
}

// The launch shapes.  step_us, chain_us, tile_steps: a step's share of a compute unit when all are full, its time in a
// launch's longest chain, what a tile costs beside its steps (and a chain at its ends); fitted to 372 launches (nine sets
// of layers of widths 256 to 4096, 32 to 2048 tokens, all four shapes: 19 % rms).
constexpr NarrowShape kShapes[kNarrowShapes] = {{64, 64, 0.257f, 0.272f, 2.3f, 0.1f}, {128, 64, 0.411f, 0.343f, 6.2f, 0.7f},
                                                {128, 128, 0.612f, 0.559f, 4.5f, 0.1f}, {256, 128, 0.825f, 0.73f, 7.8f, 0.5f}};

}  // namespace

const NarrowShape& narrow_shape(int shape) { return kShapes[shape]; }

bool narrow_shape_ok(int64_t M, int64_t N, int64_t Kc, int64_t lda, int64_t ldb) {
    // 16-byte direct loads: rows on 16-byte boundaries, 64 contraction values, a tile's rows within 32-bit offsets
    constexpr int64_t kMaxPitch = int64_t(1) << 22;
    return M > 0 && N > 0 && Kc >= 64 && Kc % 8 == 0 && lda % 8 == 0 && ldb % 8 == 0 && lda <= kMaxPitch && ldb <= kMaxPitch;
}
hipError_t launch_gemm_narrow(hipStream_t stream, GemmBatch& batch, int n_problems, int shape) {
    batch.n_problems = n_problems;
    if (n_problems == 0 || batch.total_tiles == 0) return hipSuccess;
    for (int i = 0; i < n_problems; ++i) {
        const GemmProblem& p = batch.p[i];
        if (p.n_seg != 1 || ~p.row_bits != 0 || !narrow_shape_ok(p.M, p.N, p.Kc, p.lda, p.ldb)) return hipErrorInvalidValue;
    }
    switch (shape) {
        case 0: return launch_shape<64, 64>(stream, batch);
        case 1: return launch_shape<128, 64>(stream, batch);
        case 2: return launch_shape<128, 128>(stream, batch);
        case 3: return launch_shape<256, 128>(stream, batch);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace tf
