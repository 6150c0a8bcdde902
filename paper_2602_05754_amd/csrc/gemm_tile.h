// The tiles of the generic kernel as device functions: how an operand travels from memory through registers into an LDS stage and from
// there to the matrix cores, a whole tile's contraction and output (contract_tile), which problem and which tile a
// block has.  Used by the generic kernel and by the fp32 kernel of bf16 pieces.
#pragma once
#include "gemm_device.h"

namespace tf {
namespace {

constexpr int kThreads = 256;           // four waves, 2 x 2 over the tile
constexpr int kStepBytes = 128;         // contraction bytes of an operand row per step
constexpr int kDepth = 2;               // steps whose pieces are on their way in registers
constexpr int kGroupM = 8;              // tile rows per L2 locality group

// A thread's number among the kThreads that share a tile.
__device__ __forceinline__ int tile_thread() { return int(threadIdx.x) & (kThreads - 1); }

typedef f32x4 F4any __attribute__((aligned(4)));

// One operand of a workgroup's tile: kRows rows of it, kRows x 128 bytes per stage.
template <typename TIn, bool kContig, int kRows>
struct Operand {
    static constexpr int kSize = int(sizeof(TIn));
    static constexpr int kE = 16 / kSize;                       // elements of a 16-byte piece
    static constexpr int kBK = kStepBytes / kSize;              // contraction values per step
    static constexpr int kPieces = kRows * kStepBytes / 16 / kThreads;      // per thread and step
    static constexpr int kPitch = kContig ? kStepBytes : kRows * kSize;     // bytes of a stage row
    static constexpr int kRowPieces = kPitch / 16;              // pieces of a stage row
    static constexpr int kStageBytes = kRows * kStepBytes;
    static constexpr int kFrags = kRows / 32;                   // 16-row blocks of a wave (it owns half of the rows)
    static_assert(kPieces >= 1, "at least one piece per thread");

    const TIn* p[kPieces];      // this thread's pieces of the step to be loaded next
    int k[kPieces];             // contraction index of the piece's first element (kNT) or of its row (kTN), inside a step
    int lds[kPieces];           // byte offset of the piece inside a stage
    int64_t step;               // elements from one step to the next
    const TIn* matrix;
    int over;                   // kTN: elements by which this thread's pieces run over the end of their rows
    bool narrow;                // rows shorter than a piece: fetched element by element

    __device__ __forceinline__ Operand(const void* base, int64_t ld, int extent, int kc, int origin)
        : matrix(static_cast<const TIn*>(base)), narrow(kContig ? kc < kE : ld < kE || extent < kE) {
        step = kContig ? int64_t(kBK) : int64_t(kBK) * ld;
        const int tid = tile_thread(), c = tid % kRowPieces;     // the same piece of every kThreads / kRowPieces-th row
        static_assert(kThreads % kRowPieces == 0, "a thread's pieces lie below each other");
        const int col = origin + c * kE < extent ? origin + c * kE : 0;
        over = max(col + kE - extent, 0);
#pragma unroll
        for (int i = 0; i < kPieces; ++i) {
            const int r = tid / kRowPieces + i * (kThreads / kRowPieces);      // stage row
            k[i] = kContig ? c * kE : r;
            lds[i] = kContig ? r * kPitch + ((c ^ nt_swizzle(r)) << 4) : piece_tn(r, c);
            p[i] = matrix + (kContig ? int64_t(min(origin + r, extent - 1)) * ld + k[i] : int64_t(k[i]) * ld + col);
        }
    }

    // kTN stage: byte offset of 16-byte piece c of contraction row t.  bf16: the transpose read of a
    // 16-row block takes 32 bytes (a unit) of contraction rows 8 G + x, x = 0..3, G = lane / 16, 32
    // lanes at a time: 8 rows, whose units must differ (128 rows: pitch = all banks; 64 rows: half
    // of them).  fp32: a read takes 64 bytes of rows 4 q + j, q = lane / 16: 4 rows to keep apart.
    __device__ __forceinline__ static int unit_xor(int t) {
        if (kSize == 4) return (t >> 2) & (kRows >= 64 ? 3 : 1);
        return kRows >= 128 ? 4 * ((t >> 3) & 1) + (t & 3) : 2 * ((t >> 3) & 1) + ((t >> 1) & 1);
    }
    __device__ __forceinline__ static int piece_tn(int t, int c) {
        if (kSize == 4) return t * kPitch + (((c >> 2) ^ unit_xor(t)) << 6) + ((c & 3) << 4);
        return t * kPitch + (((c >> 1) ^ unit_xor(t)) << 5) + ((c & 1) << 4);
    }

    // A step of whole pieces that all lie inside the matrix.
    __device__ __forceinline__ void load(U4 (&v)[kPieces]) {
#pragma unroll
        for (int i = 0; i < kPieces; ++i) {
            v[i] = *reinterpret_cast<const U4any*>(p[i]);
            p[i] += step;
        }
    }
    // How many elements of piece i have to be fetched from in front of it, `left` being what is left of
    // the contraction from the step's first value on: what runs over the end of a row (kNT) or of the
    // matrix (kTN: of its last row).
    __device__ __forceinline__ int past(int i, int left) const {
        if (kContig) return max(k[i] + kE - left, 0);
        return k[i] < left - 1 ? 0 : over;
    }
    // Any step: nothing outside the matrix is read; finish() puts the values in their places.  The step begins
    // `back` contraction values early (not in narrow matrices).
    __device__ __forceinline__ void load_inside(U4 (&v)[kPieces], int left) {
#pragma unroll
        for (int i = 0; i < kPieces; ++i) {
            if (!narrow) {
                const TIn* q = p[i] - past(i, left);
                if (!kContig && k[i] >= left) q = matrix;
                v[i] = *reinterpret_cast<const U4any*>(q);
            } else {
                uint64_t lo = 0, hi = 0;
                for (int e = (kContig ? min(left - k[i], kE) : k[i] < left ? kE - over : 0) - 1; e >= 0; --e) {
                    const uint64_t x = kSize == 4 ? reinterpret_cast<const uint32_t*>(p[i])[e] : reinterpret_cast<const uint16_t*>(p[i])[e];
                    hi = hi << (8 * kSize) | lo >> (64 - 8 * kSize);
                    lo = lo << (8 * kSize) | x;
                }
                v[i] = U4{uint32_t(lo), uint32_t(lo >> 32), uint32_t(hi), uint32_t(hi >> 32)};
            }
            p[i] += step;
        }
    }
    // What load_inside() fetched, moved down; zeros past the end of the contraction and for the `back`
    // values that the step before has contracted.
    __device__ __forceinline__ void finish(U4 (&v)[kPieces], int left) const {
        if (narrow) return;
#pragma unroll
        for (int i = 0; i < kPieces; ++i) {
            const int n = past(i, left);
            if (kContig ? n >= kE : k[i] >= left) {
                v[i] = U4{0, 0, 0, 0};
            } else if (n > 0) {
                const int bits = n * (8 * kSize);
                uint64_t lo = v[i][0] | uint64_t(v[i][1]) << 32, hi = v[i][2] | uint64_t(v[i][3]) << 32;
                if (bits >= 64) { lo = hi; hi = 0; }
                if (bits & 63) { lo = lo >> (bits & 63) | hi << (64 - (bits & 63)); hi >>= bits & 63; }
                v[i] = U4{uint32_t(lo), uint32_t(lo >> 32), uint32_t(hi), uint32_t(hi >> 32)};
            }
        }
    }
    // The next step begins `back` contraction values early ...
    __device__ __forceinline__ void rewind(int back) {
#pragma unroll
        for (int i = 0; i < kPieces; ++i) p[i] -= kContig ? int64_t(back) : back * (step / kBK);
    }
    // ... and those are masked out of it.
    __device__ __forceinline__ void drop(U4 (&v)[kPieces], int back) const {
#pragma unroll
        for (int i = 0; i < kPieces; ++i) {
            const int n = back - k[i];                  // kNT: that many of the piece's values; kTN: the row, if any
#pragma unroll
            for (int d = 0; d < 4; ++d)
                v[i][d] &= kContig ? (2 * d >= n ? 0xffffu : 0u) | (2 * d + 1 >= n ? 0xffff0000u : 0u) : n > 0 ? 0u : ~0u;
        }
    }
    __device__ __forceinline__ void store(const U4 (&v)[kPieces], char* stage) const {
#pragma unroll
        for (int i = 0; i < kPieces; ++i) *reinterpret_cast<U4*>(stage + lds[i]) = v[i];
    }

    // The 16 bytes that a lane contributes to the matrix instructions of 16-row block b and half
    // step u: one instruction of 32 contraction values (bf16) or four of 4 (fp32: instruction j takes
    // contraction values 16 u + 4 (lane / 16) + j, the same for both operands).
    __device__ __forceinline__ static U4 fragment(const char* stage, int b, int u) {
        const int lane = threadIdx.x & 63, q = lane >> 4;
        if (kContig) {
            const int r = b * 16 + (lane & 15);
            return *reinterpret_cast<const U4*>(stage + r * kPitch + (((4 * u + q) ^ nt_swizzle(r)) << 4));
        }
        if (kSize == 2) {
            const int ii = lane & 15, t = 8 * q + (ii >> 2);
            const char* a = stage + (32 * u + t) * kPitch + ((b ^ unit_xor(t)) << 5) + ((ii & 3) << 3);
            const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LdsBf16x4Ptr)TF_LPTR(a));
            const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LdsBf16x4Ptr)TF_LPTR(a + 4 * kPitch));
            return __builtin_bit_cast(U4, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        }
        const char* a = stage + (16 * u + 4 * q) * kPitch + ((b ^ unit_xor(4 * q)) << 6) + ((lane & 15) << 2);
        U4 x;
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j] = *reinterpret_cast<const uint32_t*>(a + j * kPitch);
        return x;
    }
};

// First row and column of tile lt of a launch, one of the problem's: groups of kGroupM tile rows, column by column.
struct TileAt { int m, n; };
template <int kTileM, int kTileN>
__device__ __forceinline__ TileAt tile_at(const GemmProblem& P, int lt) {
    const int tiles_m = (P.M + kTileM - 1) / kTileM, tiles_n = (P.N + kTileN - 1) / kTileN;
    int t = lt - P.tile_start;
    const int per_group = kGroupM * tiles_n;
    const int first_m = (t / per_group) * kGroupM;
    const int gsz = min(tiles_m - first_m, kGroupM);
    t %= per_group;
    return {(first_m + t % gsz) * kTileM, (t / gsz) * kTileN};
}

// The output is stored past the caches.  What that is for are weight gradients of few tokens, as large as the
// weights, which they push out of the memory-side cache: a whole call, us, in brackets with ordinary stores: 32 tokens,
// widths of LLaMA-8B 241 (284), LLaMA-1B 74 (76; over six layers' operands in turn 97 (104)), 1024 / 256 / 2816 27 (35 in
// turn).  The next reader of the outputs pays for it with 1 to 2 us a call (LLaMA-1B block, 200 tokens, dX read
// once 80.1 (78.6)); from 200 tokens on the rest makes no difference.
template <typename TIn, bool kContig, bool kOutBf16, bool kAccumulate, int kTileM, int kTileN>
__device__ __forceinline__ void contract_tile(const GemmProblem& P, TileAt at, char* const lds) {
    typedef Operand<TIn, kContig, kTileM> OpA;
    typedef Operand<TIn, kContig, kTileN> OpB;
    constexpr int kStage = OpA::kStageBytes + OpB::kStageBytes;
    static_assert(kTileM * kTileN * 4 <= 2 * kStage, "the sums are turned around in the stages");
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tile_thread() >> 6);
    const int M = P.M, N = P.N, Kc = P.Kc, m0 = at.m, n0 = at.n;

    OpA a(P.A, P.lda, M, Kc, m0);
    OpB b(P.B, P.ldb, N, Kc, n0);
    U4 va[kDepth][OpA::kPieces], vb[kDepth][OpB::kPieces];
    const int steps = Kc / OpA::kBK + (Kc % OpA::kBK != 0);
    // steps whose pieces are whole: all but the last one
    const int free_steps = a.narrow || b.narrow ? 0 : steps - 1;
    constexpr bool kWide = sizeof(TIn) == 2;            // 32 contraction values per instruction, not 4
    // bf16, a contraction of 64 or more that is no multiple of 64: the last step is the last 64 values, those contracted
    // already masked out - the step that the 256 x 256-tile kernel does, so that the bits are the same on both.
    // (Functions of their own: inside load_inside() and finish() they changed the main loop's schedule, 2 % of 104 us at
    // 200 tokens, LLaMA-1B block pair.)
    const int back = kWide && Kc > OpA::kBK && !a.narrow && !b.narrow ? (OpA::kBK - Kc % OpA::kBK) % OpA::kBK : 0;
    // fp32: the products of a step (8 instructions of 4) are summed by themselves and then added to the sums
    // so far.  The smallest tiles, for calls that wait for memory and the host more than for the matrix
    // pipe, contract in 64 bits (half the fp32 rate): one rounding, also of a sum that has cancelled.
    // Error against 64 bits, contraction 256: 1.2e-7 and 2.5e-8 (one chain of fp32 additions: 2.9e-7).
    constexpr bool kExact = !kWide && OpA::kFrags * OpB::kFrags == 1;
    typedef std::conditional_t<kExact, double, float> Sum;
    typedef Sum Sum4 __attribute__((ext_vector_type(4)));
    Sum4 acc[OpA::kFrags][OpB::kFrags];
#pragma unroll
    for (int i = 0; i < OpA::kFrags; ++i)
#pragma unroll
        for (int j = 0; j < OpB::kFrags; ++j) acc[i][j] = Sum4{0, 0, 0, 0};

    Sum4 second[1][1] = {{Sum4{0, 0, 0, 0}}};            // kExact: the second half steps' sums, so that two chains alternate

    const int wm = wave >> 1, wn = wave & 1;
    auto contract = [&](const char* stage) {
        U4 fa[2][OpA::kFrags], fb[2][OpB::kFrags];
        auto fragments = [&](int u) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < OpA::kFrags; ++i) fa[u][i] = OpA::fragment(stage, wm * OpA::kFrags + i, u);
#pragma unroll
            for (int j = 0; j < OpB::kFrags; ++j) fb[u][j] = OpB::fragment(stage + OpA::kStageBytes, wn * OpB::kFrags + j, u);
        };
        // D rows <- n (B rows), D columns <- m: a lane then owns 4 consecutive n of one output row
        if constexpr (kWide) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                fragments(u);
#pragma unroll
                for (int i = 0; i < OpA::kFrags; ++i)
#pragma unroll
                    for (int j = 0; j < OpB::kFrags; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, fb[u][j]),
                                                                           __builtin_bit_cast(bf16x8, fa[u][i]), acc[i][j], 0, 0, 0);
            }
        } else if constexpr (kExact) {
            fragments(0);
            fragments(1);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                auto wide = [](uint32_t x) { return double(__uint_as_float(x)); };
                acc[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(wide(fb[0][0][e]), wide(fa[0][0][e]), acc[0][0], 0, 0, 0);
                second[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(wide(fb[1][0][e]), wide(fa[1][0][e]), second[0][0], 0, 0, 0);
            }
        } else {
            f32x4 part[OpA::kFrags][OpB::kFrags];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                fragments(u);
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int i = 0; i < OpA::kFrags; ++i)
#pragma unroll
                        for (int j = 0; j < OpB::kFrags; ++j)
                            part[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(fb[u][j][e]), __uint_as_float(fa[u][i][e]),
                                                                              u == 0 && e == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : part[i][j], 0, 0, 0);
            }
            wait_for_sums(part);
#pragma unroll
            for (int i = 0; i < OpA::kFrags; ++i)
#pragma unroll
                for (int j = 0; j < OpB::kFrags; ++j) acc[i][j] += part[i][j];
        }
    };

    // Step s sits in stage s % 2, the kDepth steps after it in registers (set s % kDepth) or on their
    // way there while step s is contracted.  One barrier per step: a stage is written one step after
    // every wave has read it.
    // (what is left of the contraction from step s on, as far as it matters; with `back` only the last step asks)
    auto left = [&](int s) { return int(min(int64_t(Kc) - int64_t(s) * OpA::kBK, int64_t(0x10000))) + back; };
    auto put = [&](int s, auto q) __attribute__((always_inline)) {
        if (s >= free_steps) { a.finish(va[q], left(s)); b.finish(vb[q], left(s)); }
        if (kWide && back > 0 && s == steps - 1) { a.drop(va[q], back); b.drop(vb[q], back); }
        a.store(va[q], lds + (s & 1) * kStage);
        b.store(vb[q], lds + (s & 1) * kStage + OpA::kStageBytes);
    };
    auto fetch = [&](int s, auto q) __attribute__((always_inline)) {
        if (s >= steps) return;
        if (s < free_steps) { a.load(va[q]); b.load(vb[q]); }
        else {
            if (kWide && back > 0) { a.rewind(back); b.rewind(back); }
            a.load_inside(va[q], left(s));
            b.load_inside(vb[q], left(s));
        }
    };
    static_for<kDepth>([&](auto q) __attribute__((always_inline)) { fetch(q, q); });
    put(0, std::integral_constant<int, 0>{});
    __syncthreads();
    // The long part has no branch around a load: with one, the wait in front of a store is for the
    // loads just issued instead of the oldest ones.
    int s0 = 0;
    for (; s0 + 2 * kDepth <= free_steps; s0 += kDepth)
        static_for<kDepth>([&](auto q) __attribute__((always_inline)) {
            constexpr int now = decltype(q)::value, nxt = (now + 1) % kDepth;
            const int s = s0 + now;
            a.load(va[now]);
            b.load(vb[now]);
            contract(lds + (s & 1) * kStage);
            a.store(va[nxt], lds + (~s & 1) * kStage);
            b.store(vb[nxt], lds + (~s & 1) * kStage + OpA::kStageBytes);
            __syncthreads();
        });
    for (; s0 < steps; s0 += kDepth)
        static_for<kDepth>([&](auto q) __attribute__((always_inline)) {
            constexpr int now = decltype(q)::value, nxt = (now + 1) % kDepth;
            const int s = s0 + now;
            if (s >= steps) return;
            fetch(s + kDepth, q);
            contract(lds + (s & 1) * kStage);
            if (s + 1 < steps) put(s + 1, std::integral_constant<int, nxt>{});
            __syncthreads();
        });

    if constexpr (kWide || kExact) wait_for_sums(acc);
    if constexpr (kExact) wait_for_sums(second);
    // Epilogue: acc[i][j][e] is C[m][n], m = 16 i + lane % 16, n = 16 j + 4 (lane / 16) + e (kExact: lane / 16
    // + 4 e) of the wave's part.  The sums are turned around in LDS ([row][16-byte chunks, XOR-swizzled]) and whole
    // rows of the tile are stored, 16 bytes per lane.
    constexpr int kRow = kTileN * 4, kTurn = kTileN / 4 < 16 ? kTileN / 4 - 1 : 15;
#pragma unroll
    for (int i = 0; i < OpA::kFrags; ++i)
#pragma unroll
        for (int j = 0; j < OpB::kFrags; ++j) {
            const int r = wm * (kTileM / 2) + 16 * i + (lane & 15), c = wn * (kTileN / 8) + 4 * j + (lane >> 4);
            if constexpr (kExact) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    *reinterpret_cast<float*>(lds + r * kRow + (((c - (lane >> 4) + e) ^ (r & kTurn)) << 4) + (lane >> 4) * 4) = float(acc[0][0][e] + second[0][0][e]);
            } else {
                *reinterpret_cast<f32x4*>(lds + r * kRow + ((c ^ (r & kTurn)) << 4)) = acc[i][j];
            }
        }
    __syncthreads();
    constexpr int kOutE = kOutBf16 ? 8 : 4, kLanes = kTileN / kOutE, kRowsPerPass = kThreads / kLanes;
    const int c = tile_thread() % kLanes, n = n0 + c * kOutE;
#pragma unroll
    for (int r0 = 0; r0 < kTileM; r0 += kRowsPerPass) {
        const int r = r0 + tile_thread() / kLanes, m = m0 + r;
        f32x4 v[kOutE / 4];
#pragma unroll
        for (int h = 0; h < kOutE / 4; ++h)
            v[h] = *reinterpret_cast<const f32x4*>(lds + r * kRow + (((c * (kOutE / 4) + h) ^ (r & kTurn)) << 4));
        if (m >= M || n >= N) continue;
        if constexpr (kOutBf16) {
            const U4 x = {f32x2_to_bf16x2(v[0][0], v[0][1]), f32x2_to_bf16x2(v[0][2], v[0][3]),
                          f32x2_to_bf16x2(v[1][0], v[1][1]), f32x2_to_bf16x2(v[1][2], v[1][3])};
            uint16_t* out = static_cast<uint16_t*>(P.C) + int64_t(m) * N + n;
            if (n + kOutE <= N) {
                __builtin_nontemporal_store(x, reinterpret_cast<U4any*>(out));
            } else {
#pragma unroll
                for (int e = 0; e < kOutE; ++e)
                    if (n + e < N) out[e] = uint16_t(x[e >> 1] >> (16 * (e & 1)));
            }
        } else {
            float* out = static_cast<float*>(P.C) + int64_t(m) * N + n;
            if (n + kOutE <= N) {
                if (kAccumulate) v[0] += *reinterpret_cast<const F4any*>(out);
                __builtin_nontemporal_store(v[0], reinterpret_cast<F4any*>(out));
            } else {
#pragma unroll
                for (int e = 0; e < kOutE; ++e)
                    if (n + e < N) out[e] = kAccumulate ? out[e] + v[0][e] : v[0][e];
            }
        }
    }
}

// This block's problem: lane i looks at the first tile of problem i.
__device__ __forceinline__ int find_problem(const GemmBatch& batch, int lt) {
    static_assert(kMaxProblemsPerLaunch == 64, "one lane per problem");
    const int lane = threadIdx.x & 63;
    const bool started = lane < batch.n_problems && batch.p[lane].tile_start <= lt;
    return __builtin_amdgcn_readfirstlane(__popcll(__ballot(started)) - 1);
}

}  // namespace
}  // namespace tf
