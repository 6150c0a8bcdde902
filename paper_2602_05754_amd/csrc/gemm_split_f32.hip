// fp32 products on the bf16 matrix cores, for launches of the fp32 configuration that the fp32 matrix pipe bounds (TimelyFreeze
// Sec. 3.2.1, both halves of a backward action).
//
// A value is the sum of three bf16 ones, exactly: x = x0 + x1 + x2, x0 the value rounded to bf16, x1 what is left rounded to bf16, x2 the
// rest (Henry, Tang, Heinecke, "Leveraging the bfloat16 artificial intelligence datatype for higher-precision computations", 2019).  Of
// the nine products of two values' pieces the six of 2^-16 and more are contracted, 32 values per instruction, in 96 cycles per 16 x 16 block
// where v_mfma_f32_16x16x4_f32 takes 256.  For x in [1, 2) |x1| <= 2^-8 and |x2| <= 2^-17, of either sign: the three products left out are
// 2 * 2^-25 of the product and little more, as often too much as too little.  (Pieces cut off and not rounded have the value's sign, x1 <
// 2^-7 and x2 < 2^-15: 2^-21, always too little.)  A step's products are summed by themselves, the small ones first, and then added to
// the sums so far, as in the generic kernel.
// Errors against 64 bits, relative rms, in brackets those of the generic kernel's sums in 32 bits.  Normal operands: contraction 64 4.7e-8
// (1.06e-7), 200 6.8e-8 (1.16e-7), 1000 1.19e-7 (1.48e-7), 2731 1.84e-7 (1.98e-7), 4900 2.42e-7 (2.48e-7); their absolute values: 200 5.0e-8
// (5.9e-8), 1000 9.2e-8 (9.3e-8), 2731 1.33e-7 (1.34e-7).  On top of that the instruction aligns small products by cutting them off: sums are
// too low by 1.7e-9 of the sum of the products' magnitudes.  From some 7000 values of either sign on that is more than the generic
// kernel's own roundings inside a step: 6000 2.66e-7 (2.69e-7), 8192 3.08e-7 (3.06e-7), 32768 6.06e-7 (5.81e-7).
// (All six products chained into one sum: 2.2e-7 and more at 200; the instruction rounds four times, after every 8 values.)
//
// What bounds it: the vector instructions that split, 11 per pair of values, and add, beside the matrix instructions.  A wave's
// own two per matrix instruction cost nothing, a third 4 cycles; another wave's get every eighth cycle or so while matrix
// instructions run.  So larger tiles are faster - a value is split once per tile and step - and every wave does everything: loads, splits,
// stores to LDS and contracts, its splitting spread evenly behind its matrix instructions, one barrier per step.  256 x 128 tiles
// of eight waves have 2.1 vector instructions per matrix instruction, 128 x 128 ones 2.6.  Two blocks of widths 1024 / 256 / 2731, 1000 tokens, us:
// input gradients 231 (128 x 128 tiles 248, generic kernel 368), weight gradients 252 (288, 391), both in one launch 455 (739).
// Measured besides, the same input gradients (238 then): two workgroups of 128 x 128 tiles per unit that split and contract in turn 270; four
// waves that load and split beside four that contract 267; the remainders by v_dot2_f32_bf16, exact and half as many instructions, but
// on the matrix cores' hardware: 290; 64 x 64 tiles 320.
#include "gemm_tile.h"

#include <algorithm>

namespace tf {
namespace {

constexpr int kPiecesOf = 3;                    // bf16 pieces of a value
constexpr int kSplitThreads = 512;              // eight waves
constexpr int kBK = 32;                         // contraction values per step
typedef U4 U4any4 __attribute__((aligned(4)));

// Takes the next bf16 pieces off two values; returns them packed.  Rounded to nearest even, what is left is at most half of the
// piece's last place, of either sign; the last piece is all that is left, 8 bits (of values of 2^-110 and more: see `lost`).
__device__ __forceinline__ uint32_t take_piece(uint32_t& x0, uint32_t& x1, bool last) {
    if (last) return __builtin_amdgcn_perm(x1, x0, 0x07060302u);
    const uint32_t piece = f32x2_to_bf16x2(__uint_as_float(x0), __uint_as_float(x1));
    x0 = __float_as_uint(__uint_as_float(x0) - __uint_as_float(piece << 16));
    x1 = __float_as_uint(__uint_as_float(x1) - __uint_as_float(piece & 0xffff0000u));
    return piece;
}

// The thread's number, for what is worked out where it is needed and not once in front of the loop into registers that it has not.
__device__ __forceinline__ int this_thread() {
    int t = int(threadIdx.x);
    asm volatile("" : "+v"(t));
    return t;
}

// One operand of a workgroup's tile: kWaves waves contract kFrags blocks of 16 rows of it each, block i of wave w being number kWaves i + w.
template <bool kContig, int kWaves, int kFrags>
struct SplitOperand {
    static constexpr int kRows = 16 * kWaves * kFrags;
    static constexpr int kLoads = kRows * kBK / 4 / kSplitThreads;      // 16-byte loads per thread and step
    static constexpr int kAcross = kContig ? kBK / 4 : kRows / 4;       // loads across a stage row
    static constexpr int kDown = kSplitThreads / kAcross;               // a thread's loads lie that many stage rows apart
    static constexpr bool kPadded = !kContig && kRows == 128;           // (256 rows, padded as well, would not fit)
    static constexpr int kPitch = kContig ? kBK * 2 : kRows * 2 + (kPadded ? 32 : 0);     // bytes of a stage row
    static constexpr int kPlane = kContig ? kRows * kPitch : kBK * kPitch + (kPadded ? kBK / 8 * 128 : 0);    // of one bf16 piece of a stage
    static constexpr int kStageBytes = kPiecesOf * kPlane;
    static_assert(kLoads >= 1 && kRows >= 128, "every thread loads; a contraction row covers all banks");

    const char* matrix;
    int64_t unit;               // bytes from one contraction value to the next
    uint32_t off[kContig ? kLoads : 1];
    int extent, origin;
    int to, from;               // bytes inside a stage: of load 0's first piece, of this lane's part of a wave's first fragment

    __device__ __forceinline__ SplitOperand(const void* base, int64_t ld, int ext, int org, int w) : extent(ext), origin(org) {
        const int thread = int(threadIdx.x), c = thread % kAcross;
        const int lane = threadIdx.x & 63, q = lane >> 4;
        matrix = static_cast<const char*>(base) + (kContig ? int64_t(origin) * ld * 4 : 0);
        unit = kContig ? 4 : ld * 4;
        if (kContig) {
#pragma unroll
            for (int i = 0; i < kLoads; ++i) off[kContig ? i : 0] = uint32_t(min(row(i, thread), extent - 1 - origin)) * uint32_t(ld * 4) + c * 16;
            to = row(0, thread) * kPitch + chunk(row(0, thread), c >> 1) + ((c & 1) << 3);
            from = (w * 16 + (lane & 15)) * kPitch + chunk(lane & 15, q);
        } else {
            off[0] = uint32_t(row(0, thread)) * uint32_t(ld * 4) + uint32_t(col(thread)) * 4;
            const int r = 8 * q + ((lane & 15) >> 2);
            to = at(c >> 2, row(0, thread)) + ((c & 3) << 3);
            from = at(w, r) + ((lane & 3) << 3);
        }
    }
    __device__ __forceinline__ static int row(int i, int thread) { return thread / kAcross + i * kDown; }
    // kNT stage: byte offset in a row of its 16-byte chunk c.  (The LDS takes 16 lanes of a 128-bit read at a time: lanes 0-3, 8-11, 20-23 and
    // 28-31, the others of the first 32, and so on: rows r and r + 8 of a chunk beside rows r + 4 and r + 12 of its neighbour, four rows to
    // all banks.  Without the exchange of halves every read takes twice its cycles: a third of the LDS' busy time was conflicts, 238 us
    // where it is 233 now, 128 x 128 tiles 270 and 264.)
    __device__ __forceinline__ static int chunk(int r, int c) { return (c ^ ((r >> 3) & 1) << 1) << 4; }
    // kTN stage: byte offset of contraction row r, 16-row block u.  A transpose read takes 32 bytes (a unit) of contraction
    // rows 8 G + x, x = 0..3, G = lane / 16, 32 lanes at a time: 8 rows whose units must fall into different banks.  128 rows: a unit of
    // padding per row and four per eight rows; 256 rows: units XOR-swizzled.  (Either: no conflicts, LDS busy a quarter of the time.)
    __device__ __forceinline__ static int at(int u, int r) {
        if (kPadded) return r * kPitch + (r >> 3) * 128 + u * 32;
        return r * kPitch + (((u & 7) ^ (4 * ((r >> 3) & 1) + (r & 3))) << 5) + ((u >> 3) << 8);
    }
    // kTN: first column of a thread's loads; elements by which load i of the contraction's last row would run over the end of the matrix
    __device__ __forceinline__ int col(int thread) const {
        const int c = origin + thread % kAcross * 4;
        return c < extent ? c : 0;
    }
    __device__ __forceinline__ int over(int i, int thread) const { return !kContig && row(i, thread) == kBK - 1 ? max(col(thread) + 4 - extent, 0) : 0; }
    // Load i of the 32 contraction values from k on; `last`: they are the contraction's last ones.
    __device__ __forceinline__ U4 load(int i, int k, bool last) const {
        uint32_t o = kContig ? off[kContig ? i : 0] : off[0] - (over(i, this_thread()) * 4 & -int(last));
        asm volatile("" : "+v"(o));             // (a 32-bit offset to a scalar base: widened outside of the loop it takes two registers and an addition)
        return *reinterpret_cast<const U4any4*>(matrix + (kContig ? k : k + i * kDown) * unit + o);
    }
    // What it fetched, in its place, the first `back` contraction values zero.  (No branches: selections only.)
    __device__ __forceinline__ U4 finish(int i, U4 v, int back, bool last) const {
        const int thread = this_thread();
        if constexpr (kContig) {
            const int n = back - thread % kAcross * 4;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = e < n ? 0 : v[e];
        } else {
            const int n = over(i, thread) & -int(last);
            v[0] = n & 1 ? v[1] : v[0]; v[1] = n & 1 ? v[2] : v[1]; v[2] = n & 1 ? v[3] : v[2];
            v[0] = n & 2 ? v[2] : v[0]; v[1] = n & 2 ? v[3] : v[1];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = row(i, thread) < back ? 0 : v[e];
        }
        return v;
    }
    __device__ __forceinline__ char* place(char* stage, int i, int t) const {        // of bf16 piece t of load i
        static_assert(kDown % (kContig ? 16 : 8) == 0, "a thread's rows differ in one bit of the swizzle, kNT: in none");
        if (kPadded) return stage + to + (t * kPlane + i * kDown * kPitch + i * kDown / 8 * 128);
        const int flip = kContig ? 0 : ((i * kDown >> 3) & 1) << 7;
        return stage + (to ^ flip) + (t * kPlane + i * kDown * kPitch);
    }
    __device__ __forceinline__ bf16x8 fragment(const char* stage, int i, int t) const {
        if (kContig) return *reinterpret_cast<const bf16x8*>(stage + from + (t * kPlane + kWaves * i * 16 * kPitch));
        const char* a = kPadded ? stage + from + (t * kPlane + kWaves * i * 32)
                                : stage + (from ^ ((kWaves * i & 7) << 5)) + (t * kPlane + ((kWaves * i >> 3) << 8));
        const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LdsBf16x4Ptr)TF_LPTR(a));
        const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LdsBf16x4Ptr)TF_LPTR(a + 4 * kPitch));
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    }
};

// What three pieces cannot hold: an infinity meets zeros among the other value's pieces, a first piece rounds to infinity or a sum of
// pieces leaves the range where the sum does not, a piece below bf16's smallest value loses bits.  (The matrix instructions keep
// subnormal pieces and sums: nothing else is lost from 2^-110 on.)  Outputs that this may have reached are computed again from fp32 products, in
// blocks of 32 x 64 that lie where they lie in either tile, by the contents of the block's own rows and columns: neither
// the tile nor anything else in the launch says which way an element is computed.
// What it costs: a tile that notices anything reads its rows and columns once more, a fifth of its time and more; a pair of blocks takes a
// chain of fp32 steps of 0.8 us.  Two blocks of widths 1024 / 256 / 2731, 1000 tokens, us (generic kernel): ordinary values 467 (739); every dY
// with one tiny value 559 (738), with one in every row 679 (740), with one infinity 719 (740), all NaN 566 (725); all infinite 1797 (724),
// all tiny 1855 (742): every product twice, once in fp32 with two tiles of 32 x 64 per unit.  Worst where a launch has a tile per unit:
// 864 / 864 / 2798, 475 tokens, input gradients alone 98 (101), one tiny value 151 (106), one infinity 215 (110), all infinite 418 (98).
constexpr int kBlockM = 32, kBlockN = 64;
__device__ __forceinline__ bool finite(float x) { return __builtin_fabsf(x) < __builtin_huge_valf(); }
// Do pieces lose bits of one of the values?
__device__ __forceinline__ bool lose_bits(f32x4 v) {
    uint32_t smallest = ~0u;            // magnitude but zero, doubled, minus one
#pragma unroll
    for (int e = 0; e < 4; ++e) smallest = min(smallest, (__float_as_uint(v[e]) << 1) - 1);
    if (smallest >= (__float_as_uint(0x1p-110f) << 1) - 1) return false;
    uint32_t left = 0;
#pragma unroll
    for (int e = 0; e < 4; e += 2) {
        uint32_t x0 = __float_as_uint(v[e]), x1 = __float_as_uint(v[e + 1]);
        take_piece(x0, x1, false);
        take_piece(x0, x1, false);
        left |= x0 | x1;
    }
    return (left & 0xffffu) != 0;
}
// What a row or column of the tile holds: its largest magnitude, doubled (a NaN is larger than everything), and whether pieces lose
// bits of one of its values.
struct RowNotes { uint32_t largest, lost; };
__device__ __forceinline__ uint32_t twice_magnitude(f32x4 v) {
    uint32_t m = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) m = max(m, __float_as_uint(v[e]) << 1);
    return m;
}
// The notes of kRows rows of an operand from `origin` on.  One pass over them, eight loads on their way; what would lie beyond the
// matrix is shifted back inside (at least 32 contraction values, kTN: at least 4 rows).
template <bool kContig, int kRows>
__device__ __forceinline__ void look_at_rows(const void* base, int64_t ld, int extent, int origin, int Kc, RowNotes* notes) {
    const float* const matrix = static_cast<const float*>(base);
    const int thread = this_thread(), lane = thread & 63, wave = thread >> 6;
    constexpr int kMany = 8;
    if constexpr (kContig) {            // a wave: eight rows, 256 contraction values of each at a time
        for (int r0 = wave * kMany; r0 < kRows; r0 += kSplitThreads / 64 * kMany) {
            bool found[kMany] = {};
            uint32_t largest[kMany] = {};
            for (int k = lane * 4; k < Kc; k += 256) {
                f32x4 v[kMany];
#pragma unroll
                for (int i = 0; i < kMany; ++i) v[i] = *reinterpret_cast<const F4any*>(matrix + int64_t(min(origin + r0 + i, extent - 1)) * ld + min(k, Kc - 4));
#pragma unroll
                for (int i = 0; i < kMany; ++i) {
                    largest[i] = max(largest[i], twice_magnitude(v[i]));
                    found[i] = found[i] || lose_bits(v[i]);
                }
            }
#pragma unroll
            for (int i = 0; i < kMany; ++i) {
#pragma unroll
                for (int d = 32; d > 0; d >>= 1) largest[i] = max(largest[i], uint32_t(__shfl_xor(int(largest[i]), d)));
                if (lane == 0) notes[r0 + i].largest = largest[i];
                if (found[i]) notes[r0 + i].lost = 1;
            }
        }
    } else {                            // a thread: four rows, every kDown-th contraction value
        constexpr int kAcross = kRows / 4, kDown = kSplitThreads / kAcross;
        const int first = min(origin + thread % kAcross * 4, extent - 4);
        uint32_t found = 0, largest[4] = {};
        for (int k0 = thread / kAcross; k0 < Kc; k0 += kDown * kMany) {
            f32x4 v[kMany];
#pragma unroll
            for (int i = 0; i < kMany; ++i) v[i] = *reinterpret_cast<const F4any*>(matrix + int64_t(min(k0 + i * kDown, Kc - 1)) * ld + first);
#pragma unroll
            for (int i = 0; i < kMany; ++i) {
#pragma unroll
                for (int e = 0; e < 4; ++e) largest[e] = max(largest[e], __float_as_uint(v[i][e]) << 1);
                if (lose_bits(v[i])) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) found |= uint32_t(lose_bits(f32x4{v[i][e], 0.f, 0.f, 0.f})) << e;
                }
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (first + e >= origin) {
                atomicMax(&notes[first + e - origin].largest, largest[e]);
                if (found >> e & 1) notes[first + e - origin].lost = 1;
            }
    }
}
// Is a sum of row x and column y to be computed again?  Not if one of them holds a NaN: it is one either way.  Else if it is not
// finite, or if the lost bits, less than 2^-133 of a value each, could change it by 2^-30 of itself (which a single tiny value
// among ordinary ones does not do).
__device__ __forceinline__ bool sum_is_odd(float sum, RowNotes x, RowNotes y, float n_values) {
    const uint32_t infinite = __float_as_uint(__builtin_huge_valf()) << 1;
    if (x.largest > infinite || y.largest > infinite) return false;
    const float reach = (x.lost ? __uint_as_float(y.largest >> 1) : 0.f) + (y.lost ? __uint_as_float(x.largest >> 1) : 0.f);
    return !finite(sum) || !(n_values * 0x1p-103f * reach <= __builtin_fabsf(sum));
}
// The blocks of a tile to be computed again, bit 2 (row / 32) + column / 64.  The tile's sums lie in `lds`, `side` is free LDS behind them.
template <int kTileM, int kTileN>
constexpr int kNotes = 2 + 2 * (kTileM + kTileN);       // words of `side`
template <bool kContig, int kTileM, int kTileN>
__device__ __forceinline__ uint32_t odd_blocks(const GemmProblem& P, TileAt at, const char* lds, uint32_t* side) {
    static_assert(kTileM / kBlockM * (kTileN / kBlockN) <= 32 && kTileN == 2 * kBlockN, "a bit per block");
    uint32_t* const blocks = side;
    RowNotes* const of_row = reinterpret_cast<RowNotes*>(side + 2);
    RowNotes* const of_col = of_row + kTileM;
    const int thread = this_thread();
    __syncthreads();
    for (int i = thread; i < kNotes<kTileM, kTileN>; i += kSplitThreads) side[i] = 0;
    __syncthreads();
    look_at_rows<kContig, kTileM>(P.A, P.lda, P.M, at.m, P.Kc, of_row);
    look_at_rows<kContig, kTileN>(P.B, P.ldb, P.N, at.n, P.Kc, of_col);
    __syncthreads();
    constexpr int kLanes = kTileN / 4;
    const int c = thread % kLanes;
    for (int r = thread / kLanes; r < kTileM && at.m + r < P.M; r += kSplitThreads / kLanes) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(lds + r * kTileN * 4 + ((c ^ (r & 15)) << 4));
        bool odd = false;
#pragma unroll
        for (int e = 0; e < 4; ++e) odd = odd || (at.n + c * 4 + e < P.N && sum_is_odd(v[e], of_row[r], of_col[c * 4 + e], float(P.Kc)));
        if (odd) atomicOr(blocks, 1u << (r / kBlockM * 2 + c / (kBlockN / 4)));
    }
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(*blocks);
}

// (the layout kTN has the larger stages)
template <int kTileM, int kTileN, int kWavesM>
constexpr int split_lds() {
    return 2 * (SplitOperand<false, kWavesM, kTileM / 16 / kWavesM>::kStageBytes + SplitOperand<false, 8 / kWavesM, kTileN / 16 / (8 / kWavesM)>::kStageBytes);
}

template <bool kContig, int kTileM, int kTileN, int kWavesM>
__device__ __forceinline__ void contract_split(const GemmProblem& P, TileAt at, bool add, char* const lds) {
    constexpr int kWavesN = kSplitThreads / 64 / kWavesM, kFragA = kTileM / kWavesM / 16, kFragB = kTileN / kWavesN / 16;
    typedef SplitOperand<kContig, kWavesM, kFragA> OpA;
    typedef SplitOperand<kContig, kWavesN, kFragB> OpB;
    constexpr int kStage = OpA::kStageBytes + OpB::kStageBytes, kLoads = OpA::kLoads + OpB::kLoads;
    static_assert(kFragA % 2 == 0, "the last row of a step and the first of the next hold piece 0 in different registers");
    static_assert(kTileM * kTileN * 4 + kNotes<kTileM, kTileN> * 4 <= 2 * kStage, "the sums are turned around in the stages, with odd_blocks()' notes behind them");
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave / kWavesN, wn = wave % kWavesN;
    const int M = P.M, N = P.N, Kc = P.Kc, m0 = at.m, n0 = at.n;
    const int steps = (Kc + kBK - 1) / kBK, back = steps * kBK - Kc;
    f32x4 acc[kFragA][kFragB];
#pragma unroll
    for (int i = 0; i < kFragA; ++i)
#pragma unroll
        for (int j = 0; j < kFragB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    const OpA a(P.A, P.lda, M, m0, wm);
    const OpB b(P.B, P.ldb, N, n0, wn);
    uint32_t lost = 0;              // its lower half: bits that are in none of the three pieces (of values below 2^-110)
    U4 raw[kLoads];                 // values of the steps ahead: load 0 of the next but one, the others of the next
    uint32_t packed[2];
    // (Step `steps` - 1 is the contraction's last 32 values, those contracted before masked out; what would come after it is that
    // step again, for nothing.)
    auto load = [&](auto i, int s) __attribute__((always_inline)) {
        const int k = min(s * kBK, Kc - kBK);
        const bool last = s >= steps - 1;
        if constexpr (i < OpA::kLoads) raw[i] = a.load(i, k, last);
        else raw[i] = b.load(i - OpA::kLoads, k, last);
    };
    auto load_whole = [&](auto i, int s) __attribute__((always_inline)) {
        if constexpr (i < OpA::kLoads) raw[i] = a.load(i, s * kBK, false);
        else raw[i] = b.load(i - OpA::kLoads, s * kBK, false);
    };
    auto finish = [&](auto i, int s) __attribute__((always_inline)) {
        const bool last = s >= steps - 1;
        if constexpr (i < OpA::kLoads) raw[i] = a.finish(i, raw[i], last ? back : 0, last);
        else raw[i] = b.finish(i - OpA::kLoads, raw[i], last ? back : 0, last);
    };
    // part n of 6 of splitting load i into a stage
    constexpr int kParts = 2 * kPiecesOf;
    auto split = [&](auto i, auto n, char* stage) __attribute__((always_inline)) {
        constexpr int t = n / 2, h = n % 2;
        uint32_t x0 = raw[i][2 * h], x1 = raw[i][2 * h + 1];
        packed[h] = take_piece(x0, x1, t == kPiecesOf - 1);
        // (left to itself the compiler gathers these at a step's end, with all of their operands held until then)
        if constexpr (t == kPiecesOf - 1) asm volatile("v_or3_b32 %0, %0, %1, %2" : "+v"(lost) : "v"(x0), "v"(x1));
        raw[i][2 * h] = x0;
        raw[i][2 * h + 1] = x1;
        if constexpr (h == 1) {
            char* const to = i < OpA::kLoads ? a.place(stage, i, t) : b.place(stage + OpA::kStageBytes, i - OpA::kLoads, t);
            *reinterpret_cast<U2*>(to) = U2{packed[0], packed[1]};
        }
    };
    bf16x8 fb[kFragB][kPiecesOf], fa[2], fa_low[2];     // of A: piece 0 of this row of blocks and of the next; pieces 1 and 2
    // A row of blocks' products of one step; added to the sums behind some matrix instructions of the next row, where the last of them
    // is done (rows of two blocks: a row more to wait in).
    constexpr int kBuffers = kFragB < 4 ? 2 : 1, kSumAt = kBuffers == 2 ? 5 : 0;
    f32x4 part[kBuffers][kFragB];
    auto read_a = [&](const char* stage, auto i, auto t) __attribute__((always_inline)) {
        if constexpr (t == 0) fa[i % 2] = a.fragment(stage, i, 0);
        else fa_low[t - 1] = a.fragment(stage, i, t);
    };
    auto read_b = [&](const char* stage, auto j, auto t) __attribute__((always_inline)) { fb[j][t] = b.fragment(stage + OpA::kStageBytes, j, t); };
    constexpr std::integral_constant<int, 0> k0;

    auto split_load = [&](auto i, int s, char* stage) __attribute__((always_inline)) {
        finish(i, s);
        static_for<kParts>([&](auto n) __attribute__((always_inline)) { split(i, n, stage); });
    };
    // Step s.  kWhole: whatever is loaded and split meanwhile are whole steps; kLast: nothing is, no step follows.
    auto step = [&](int s, auto whole, auto last) __attribute__((always_inline)) {
        constexpr bool kWhole = decltype(whole)::value, kLast = decltype(last)::value;
        char* const now = lds + (s & 1) * kStage;
        char* const then = lds + (~s & 1) * kStage;
        constexpr int kRow = 6 * kFragB, kBefore = (kFragA - 1) * kRow;          // MFMAs of a row, and in front of the barrier
        static_for<kFragA * kRow>([&](auto m) __attribute__((always_inline)) {
            constexpr int order[6][2] = {{0, 2}, {1, 1}, {0, 1}, {2, 0}, {1, 0}, {0, 0}};        // pieces of A and B
            constexpr int i = m / kRow, n = m % kRow, g = n / kFragB, j = n % kFragB, pa = order[g][0], pb = order[g][1];
            // the sums of the row before (in the first row: of the last one of the step before)
            constexpr int was = (i + kFragA - 1) % kFragA;
            if constexpr (g == kSumAt) acc[was][j] += part[was % kBuffers][j];
            f32x4& sum = part[i % kBuffers][j];
            sum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j][pb], pa == 0 ? fa[i % 2] : fa_low[pa == 0 ? 0 : pa - 1], g == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : sum, 0, 0, 0);
            // the next fragments, each where the one in its place has been used
            constexpr std::integral_constant<int, (i + 1) % kFragA> row;
            constexpr std::integral_constant<int, 1> k1;
            constexpr std::integral_constant<int, 2> k2;
            char* const from_a = i + 1 < kFragA ? now : then;
            if constexpr (i + 1 < kFragA || !kLast) {
                if constexpr (g == 2 && j == 0) read_a(from_a, row, k0);
                if constexpr (g == 4 && j == 0) read_a(from_a, row, k2);
                if constexpr (g == 5 && j == 0) read_a(from_a, row, k1);
            }
            if constexpr (i + 1 == kFragA && !kLast) {
                if constexpr (g == 1) read_b(then, j, k2);
                if constexpr (g == 3) read_b(then, j, k1);
                if constexpr (g == 5) read_b(then, j, k0);
            }
            // the values of the steps ahead: load 0 of step s + 2 behind the last row, the others of step s + 1 before it
            constexpr int kItems = i + 1 < kFragA ? (kLoads - 1) * kParts : kParts, kOver = i + 1 < kFragA ? kBefore : kRow, x = i + 1 < kFragA ? int(m) : n;
            constexpr int from = x * kItems / kOver, to = kLast ? from : (x + 1) * kItems / kOver;
            static_for<to - from>([&](auto d) __attribute__((always_inline)) {
                constexpr int item = from + d;
                constexpr std::integral_constant<int, i + 1 < kFragA ? 1 + item / kParts : 0> which;
                constexpr std::integral_constant<int, item % kParts> n_th;
                const int ahead = i + 1 < kFragA ? s + 1 : s + 2;
                if constexpr (!kWhole && n_th == 0) finish(which, ahead);
                split(which, n_th, i + 1 < kFragA ? then : now);
                if constexpr (n_th == kParts - 1) {
                    if constexpr (kWhole) load_whole(which, ahead + 1);
                    else load(which, ahead + 1);
                }
            });
            if constexpr (m == kBefore - 1 && !kLast) __syncthreads();      // step s + 1 is there, step s has been read
            __builtin_amdgcn_sched_barrier(4);         // (scalar instructions may pass)
        });
    };

    auto each_load = [&](auto f) __attribute__((always_inline)) {
        static_for<kLoads>([&](auto i) __attribute__((always_inline)) {
            f(i);
            __builtin_amdgcn_sched_barrier(0);      // in the order in which they are waited for
        });
    };
    each_load([&](auto i) __attribute__((always_inline)) { load(i, 0); });
    each_load([&](auto i) __attribute__((always_inline)) {
        split_load(i, 0, lds);
        load(i, 1);
    });
    split_load(k0, 1, lds + kStage);
    __builtin_amdgcn_sched_barrier(0);
    load(k0, 2);
    __syncthreads();
    static_for<kPiecesOf>([&](auto t) __attribute__((always_inline)) { read_a(lds, k0, t); });
    static_for<kPiecesOf * kFragB>([&](auto n) __attribute__((always_inline)) {
        read_b(lds, std::integral_constant<int, n % kFragB>{}, std::integral_constant<int, kPiecesOf - 1 - n / kFragB>{});
    });
#pragma unroll
    for (int j = 0; j < kFragB; ++j) part[(kFragA - 1) % kBuffers][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    int s = 0;
    for (; s < steps - 4; ++s) step(s, std::true_type{}, std::false_type{});
    // The last step without the loads and splits of none: 3 % of launches of 86 steps, 7 % of 7 (widths 800 / 400 / 2400, input gradients,
    // 512 tokens, 86.4 -> 82.4 us; width 256, weight gradients, 200 tokens, 17.1 -> 15.7).  (Four blocks across and nothing to split in
    // between, the sums would be read too early; waited for they leave the registers short: eleven spilled.)
    constexpr bool kBare = kBuffers == 2;
    for (; s < steps - int(kBare); ++s) step(s, std::false_type{}, std::false_type{});
    if constexpr (kBare) step(s, std::false_type{}, std::true_type{});
    wait_for_sums(part);
#pragma unroll
    for (int j = 0; j < kFragB; ++j) acc[kFragA - 1][j] += part[(kFragA - 1) % kBuffers][j];
    __syncthreads();

    // The sums are turned around in LDS; beside them the waves say whether pieces may have failed: a sum that is not finite, bits lost.
    constexpr int kRow = kTileN * 4, kTurn = 15;
    uint32_t* const side = reinterpret_cast<uint32_t*>(lds + kTileM * kRow);
    bool odd = (lost & 0xffffu) != 0;
#pragma unroll
    for (int i = 0; i < kFragA; ++i)
#pragma unroll
        for (int j = 0; j < kFragB; ++j) {
            const int r = 16 * (kWavesM * i + wm) + (lane & 15), c = 4 * (kWavesN * j + wn) + (lane >> 4);
            *reinterpret_cast<f32x4*>(lds + r * kRow + ((c ^ (r & kTurn)) << 4)) = acc[i][j];
#pragma unroll
            for (int e = 0; e < 4; ++e) odd = odd || !finite(acc[i][j][e]);
        }
    const bool wave_odd = __ballot(odd) != 0;
    if (lane == 0) side[wave] = wave_odd;
    __syncthreads();
    bool any_odd = false;
#pragma unroll
    for (int w = 0; w < kSplitThreads / 64; ++w) any_odd = any_odd || side[w] != 0;
    uint32_t again = 0;
    if (__builtin_amdgcn_readfirstlane(any_odd)) again = odd_blocks<kContig, kTileM, kTileN>(P, at, lds, side);

    constexpr int kLanes = kTileN / 4, kRowsPerPass = kSplitThreads / kLanes;
    const int c = int(threadIdx.x) % kLanes, n = n0 + c * 4;
    const uint32_t skip = again >> (c / (kBlockN / 4));
#pragma unroll
    for (int r0 = 0; r0 < kTileM; r0 += kRowsPerPass) {
        const int r = r0 + int(threadIdx.x) / kLanes, m = m0 + r;
        f32x4 v = *reinterpret_cast<const f32x4*>(lds + r * kRow + ((c ^ (r & kTurn)) << 4));
        if (m >= M || n >= N || (skip >> (r0 / kBlockM * (kTileN / kBlockN)) & 1)) continue;
        float* out = static_cast<float*>(P.C) + int64_t(m) * N + n;
        if (n + 4 <= N) {
            if (add) v += *reinterpret_cast<const F4any*>(out);
            __builtin_nontemporal_store(v, reinterpret_cast<F4any*>(out));
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (n + e < N) out[e] = add ? out[e] + v[e] : v[e];
        }
    }
    // Two blocks at a time, each by four waves; without a second one those contract one that lies beyond the matrix, of which nothing is stored.
    const int half = wave >> 2;
    while (again != 0) {
        __syncthreads();
        const int first = __builtin_ctz(again);
        again &= again - 1;
        const int second = again != 0 ? __builtin_ctz(again) : -1;
        again &= again - 1;             // (of 0: 0)
        const int mine = half == 0 ? first : second;
        const TileAt block = mine < 0 ? TileAt{M, n0} : TileAt{m0 + mine / (kTileN / kBlockN) * kBlockM, n0 + mine % (kTileN / kBlockN) * kBlockN};
        char* const stages = lds + half * (2 * (kBlockM + kBlockN) * kStepBytes);
        if (add) contract_tile<float, kContig, false, true, kBlockM, kBlockN>(P, block, stages);
        else contract_tile<float, kContig, false, false, kBlockM, kBlockN>(P, block, stages);
    }
}

template <int kTileM, int kTileN, int kWavesM>
__global__ __launch_bounds__(kSplitThreads, 2) void gemm_split_kernel(GemmBatch batch) {
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    const int lt = logical_tile(int(blockIdx.x), batch.total_tiles);
    const int pi = find_problem(batch, lt);
    const GemmProblem& P = batch.p[pi];
    const TileAt at = tile_at<kTileM, kTileN>(P, lt);
    if (batch.tn >> pi & 1) contract_split<false, kTileM, kTileN, kWavesM>(P, at, batch.add >> pi & 1, lds);
    else contract_split<true, kTileM, kTileN, kWavesM>(P, at, batch.add >> pi & 1, lds);
}

template <int kTileM, int kTileN, int kWavesM>
hipError_t launch_shape(hipStream_t stream, const GemmBatch& batch) {
    auto kern = gemm_split_kernel<kTileM, kTileN, kWavesM>;
    constexpr int kLds = split_lds<kTileM, kTileN, kWavesM>();
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
    hipLaunchKernelGGL(kern, dim3(batch.total_tiles), dim3(kSplitThreads), kLds, stream, batch);
    return hipGetLastError();
}

// The launch shapes, with the numbers of the estimate of a launch's time: a step's share of a compute unit when all are busy and its
// time in a launch's longest chain, steps added for a tile and for the longest chain, how much of the smaller of the two is added to the larger, and what is
// added to a launch.  They are one fit to launches' times and mean something together only: -0.7 steps for a chain and 12 us for a launch are no costs of either.
constexpr SplitShape kShapes[kSplitShapes] = {{128, 128, 1.38f, 0.96f, 4.6f, 2.9f, 0.07f, 4.3f}, {256, 128, 2.37f, 1.63f, 3.9f, -0.7f, 0.15f, 12.f}};

}  // namespace

const SplitShape& split_shape(int shape) { return kShapes[shape]; }

bool split_shape_ok(Layout layout, int64_t M, int64_t N, int64_t Kc, int64_t lda, int64_t ldb) {
    // 32-bit offsets inside a tile, contraction indices up to two steps past the end.  The last step reads 32 contraction values back from
    // the end, and a load at the end of a row 4 values back: neither may begin before the matrix.
    constexpr int64_t kMaxPitch = int64_t(1) << 22;
    return Kc >= kBK && Kc <= (int64_t(1) << 30) && lda <= kMaxPitch && ldb <= kMaxPitch && (layout == Layout::kNT || std::min(M, N) >= 4);
}

hipError_t launch_gemm_split(hipStream_t stream, GemmBatch& batch, int n_problems, int shape) {
    batch.n_problems = n_problems;
    if (n_problems == 0 || batch.total_tiles == 0) return hipSuccess;
    for (int i = 0; i < n_problems; ++i) {
        const GemmProblem& p = batch.p[i];
        const Layout layout = batch.tn >> i & 1 ? Layout::kTN : Layout::kNT;
        if (p.n_seg != 1 || ~p.row_bits != 0 || !split_shape_ok(layout, p.M, p.N, p.Kc, p.lda, p.ldb)) return hipErrorInvalidValue;
    }
    switch (shape) {
        case 0: return launch_shape<128, 128, 2>(stream, batch);
        case 1: return launch_shape<256, 128, 4>(stream, batch);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace tf
