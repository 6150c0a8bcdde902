// Device side of the metric-aware selection steps that sit next to the hot path.
//
// 1. AutoFreeze (TimelyFreeze Sec. 2.3): the score of a layer compares the norms of
//    its cumulative updates Delta_{K-1}, Delta_K between stability checks.  Delta_K is
//    p_now - p_at_the_previous_check, so one pass per check over the master weights
//    and a snapshot gives sum((p - snapshot)^2) per tensor and renews the snapshot.
//    HBM-bound: 8 B read + 4 B written per element; nothing is paid between checks.
//
// 2. Budget reconciliation of the hybrid variants (App. "Hybrid Variants Algorithm",
//    Alg. 2): a base element mask is brought to exactly N_freeze ones by adding
//    uniformly drawn zeros or removing uniformly drawn ones.  "Uniformly drawn" is made
//    reproducible by ranking candidates by the image of their stage-wide index under a
//    keyed permutation of [0, 2^32) (6-round Feistel network on 16-bit halves, round
//    function: top half of ((half ^ key) + 1) * 0x9E3779B1 mod 2^32) and taking the
//    lowest ranks.  The rank threshold is found by a radix select over the keys (digits of 11, 11
//    and 10 bits): a histogram of the first digit over all candidates; then the permutation is run
//    BACKWARDS over the 2^21 keys with that digit, and over the 2^10 with the first two - a key's
//    element is looked up in the mask - so that only the first digit and the final comparison take
//    a pass over the elements.  All of it on the stream: the host never waits.
//    ALU-bound: two keys at a time in 16-bit halves, 5 instructions per round and pair (see Halves),
//    the top half of a key needs five rounds, and the first round is worked out once for all the
//    words that a thread visits.  Large masks guess their threshold and need one pass over the elements
//    instead of two (rc_try_kernel).  1.74e9 elements, 30 % -> 50 %: 6.2 ms with four passes of six rounds each,
//    key by key; 1.47 with the two passes (0.67 and 0.74); 0.78 with the guess, of which the keyed pass takes 0.65.
#include "tf_internal.h"

namespace tf {
namespace {

constexpr int kThreads = 256;

// ------------------------------------------------------------------------------------------
// AutoFreeze norms
// ------------------------------------------------------------------------------------------
// The launch shape follows the fused optimizer pass (what decides the rate is how the three
// streams meet in the memory system): a block is ONE wave and each of its accesses is 1 KB of one
// array (whole 128-byte lines); an unused 8.75 KB of dynamic LDS per block caps a compute unit at 18
// blocks; every access is non-temporal.  Measured on the 8B stage's 1.74e9 elements: 6.6 TB/s
// with 2 iterations per block and 18 blocks per unit (1 iteration: 5.4; 4: 6.5; 8: 5.9; 9 blocks
// per unit: 4.7 .. 6.1), against 5.5 for blocks of four waves and 8 iterations.
// With 3.4 million blocks the per-tensor sums are gathered in two levels like the optimizer's
// score sums: a block adds to one of 64 slots of its tensor, a second kernel adds up the slots.
constexpr int kNormThreads = 64;
constexpr int kNormGroup = 4, kNormIters = 2;
constexpr int kNormResidencyLds = residency_lds(18);
constexpr int kNormSlotDouble = 2;          // which double of a 64-byte slot (0 and 1 are the optimizer's)
constexpr int64_t kNormElemsPerBlock = int64_t(kNormThreads) * kNormGroup * kNormIters;
typedef float F4 __attribute__((ext_vector_type(4)));

// One wave per tensor: adds up the tensor's slots, writes the sum and leaves the slots zero for
// the next launch.
__global__ __launch_bounds__(kSumSlots) void norm_finish_kernel(NormBatch batch) {
    static_assert(kSumSlots == 64, "one wave reads one tensor's slots");
    double* slot = batch.partials + (int64_t(blockIdx.x) * kSumSlots + threadIdx.x) * kSumSlotDoubles + kNormSlotDouble;
    double x = *slot;
    *slot = 0.0;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) x += __shfl_down(x, off, 64);
    if (threadIdx.x == 0) *batch.t[blockIdx.x].out = x;
}

__global__ __launch_bounds__(kNormThreads) void norm_kernel(NormBatch batch) {
    int ti = 0;
    const int bid = blockIdx.x;
    for (int i = 1; i < batch.n_tensors; ++i)
        if (bid >= batch.t[i].block_start) ti = i;
    const NormTensor& T = batch.t[ti];
    const int64_t numel = T.numel;
    const int local_block = bid - T.block_start;
    const int64_t chunk = int64_t(local_block) * kNormElemsPerBlock;
    double acc = 0.0;
#pragma unroll
    for (int it = 0; it < kNormIters; ++it) {
        const int64_t j = chunk + (int64_t(it) * kNormThreads + threadIdx.x) * kNormGroup;
        if (j + kNormGroup <= numel) {
            // streamed once: non-temporal accesses measured 5 % faster
            const F4 p = __builtin_nontemporal_load(reinterpret_cast<const F4*>(T.p + j));
            const F4 s = __builtin_nontemporal_load(reinterpret_cast<const F4*>(T.snap + j));
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const double d = double(p[e]) - double(s[e]);      // exact
                acc += d * d;
            }
            if (batch.update_snapshot) __builtin_nontemporal_store(p, reinterpret_cast<F4*>(T.snap + j));
        } else {
            for (int64_t q = j; q < numel; ++q) {                  // ragged tail
                const double d = double(T.p[q]) - double(T.snap[q]);
                acc += d * d;
                if (batch.update_snapshot) T.snap[q] = T.p[q];
            }
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
    if (threadIdx.x == 0)
        unsafeAtomicAdd(batch.partials + (int64_t(ti) * kSumSlots + local_block % kSumSlots) * kSumSlotDoubles + kNormSlotDouble, acc);
}

// ------------------------------------------------------------------------------------------
// Budget reconciliation
// ------------------------------------------------------------------------------------------
constexpr int kBins = 2048;
// A thread visits words that lie 2^16 elements apart: their elements share the low halves of their
// indices.  A task is 256 neighbouring words in each of kRows such rows of a tensor.
constexpr int kRowWords = 65536 / 32;
constexpr int kColumns = kRowWords / kThreads;      // tasks side by side
constexpr int kRows = 16;
constexpr int kWindowTops = 64;                      // guessed thresholds: at most this many top halves of keys, 2^22 keys
constexpr int kGrid = 256 * 8;                      // blocks walk the tasks (keyed passes, 4 per compute unit at a time: 2048 blocks 0.67 ms, 1024 0.71)

struct RcTask {
    uint32_t* bits;       // the tensor's words
    uint32_t* undo;       // where rc_try_kernel() leaves them as they were
    int64_t n_words, first;     // first: this thread's first word
    int64_t numel;
    uint32_t index0;      // stage-wide index of that word's bit 0
};
__device__ __forceinline__ RcTask rc_task(const RcBatch& batch, int task) {
    int ti = 0;
#pragma unroll
    for (int step = kMaxRcTensors / 2; step > 0; step >>= 1)
        if (ti + step < batch.n_tensors && batch.t[ti + step].block_start <= task) ti += step;
    const RcTensor& T = batch.t[ti];
    const int t = task - T.block_start;
    RcTask r;
    r.bits = T.bits;
    r.undo = T.undo;
    r.numel = T.numel;
    r.n_words = (T.numel + 31) >> 5;
    r.first = int64_t(t / kColumns) * kRows * kRowWords + (t % kColumns) * kThreads + threadIdx.x;
    r.index0 = uint32_t(T.goff + (r.first << 5));
    return r;
}
// Bits of the word that are elements of the tensor (0 past its end).
__device__ __forceinline__ uint32_t rc_valid(const RcTask& r, int64_t word) {
    const int64_t left = r.numel - (word << 5);
    return left >= 32 ? 0xffffffffu : left > 0 ? (1u << int(left)) - 1u : 0u;
}

typedef unsigned short U16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) { return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96); }

// The top halves of the keys of a word's 32 elements, two per register: element p in the low half of register
// p, element p + 16 in its high half, so that 16 results of one bit each make a word without being interleaved.
// With x0 = high half of the index, x1 = low half, x[r + 2] = x[r] ^ F(x[r + 1] ^ key r), the key is x6 : x7.
struct Halves {
    uint32_t a[16];       // x2 without x0, ^ key 1: the first round, the same for all words of a thread
    uint32_t l[16];       // x1 ^ key 2
    uint32_t k13, k24, k3, c;
    bool carry;           // an element of the word has a low half of 0: those from there on have x0 + 1
    uint32_t low0;

    __device__ __forceinline__ void init(uint32_t index0, const RcKeys& k) {
        auto twice = [](uint32_t x) { return x * 0x10001u; };
        c = 0x9E3779B1u;
        asm("" : "+v"(c));
        low0 = index0 & 0xffffu;
        carry = low0 + 31 > 0xffffu;
#pragma unroll
        for (int p = 0; p < 16; p += 2) {
            uint32_t z[2], q[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const uint32_t e = low0 + p + j, x1 = (e & 0xffffu) | (e + 16) << 16;
                z[j] = x1 ^ twice(k.k[0]);
                l[p + j] = x1 ^ twice(k.k[2]);
            }
            round_pairs(z, q);
            a[p] = q[0] ^ twice(k.k[1]);
            a[p + 1] = q[1] ^ twice(k.k[1]);
        }
        k13 = twice(k.k[1] ^ k.k[3]);
        k24 = twice(k.k[2] ^ k.k[4]);
        k3 = twice(k.k[3]);
    }
    // Registers p and p + 1, step by step side by side: an instruction that reads the one before it waits.
    template <bool kCarry>
    __device__ __forceinline__ void top(int p, uint32_t high2, uint32_t (&x)[2]) const {
        uint32_t z2[2], z3[2], z4[2], z5[2], q[2];
        auto each = [](auto f) __attribute__((always_inline)) { f(0); f(1); };
        each([&](int j) __attribute__((always_inline)) {
            const uint32_t e = low0 + p + j;
            z2[j] = a[p + j] ^ (kCarry ? high2 + (e >> 16 | (e + 16) >> 16 << 16) : high2);
        });
        round_pairs(z2, q);
        each([&](int j) __attribute__((always_inline)) { z3[j] = l[p + j] ^ q[j]; });
        round_pairs(z3, q);
        each([&](int j) __attribute__((always_inline)) { z4[j] = xor3(z2[j], q[j], k13); });
        round_pairs(z4, q);
        each([&](int j) __attribute__((always_inline)) { z5[j] = xor3(z3[j], q[j], k24); });
        round_pairs(z5, q);
        each([&](int j) __attribute__((always_inline)) { x[j] = xor3(z4[j], q[j], k3); });
    }
    // The round function of the permutation on two 16-bit halves in each of two registers: z -> bits 16..31 of
    // (z + 1) C, C = 0x9E3779B1 = Chi 2^16 + Clo.  With p = z Clo + C these are Chi z + (p >> 16), mod 2^16.
    __device__ __forceinline__ void round_pairs(const uint32_t (&z)[2], uint32_t (&q)[2]) const {
        uint32_t p0, p1, r0, r1;
        asm("v_mad_u32_u16 %0, %4, %6, %7\n\t"
            "v_mad_u32_u16 %1, %4, %6, %7 op_sel:[1,0,0,0]\n\t"
            "v_mad_u32_u16 %2, %5, %6, %7\n\t"
            "v_mad_u32_u16 %3, %5, %6, %7 op_sel:[1,0,0,0]"
            : "=&v"(p0), "=&v"(p1), "=&v"(r0), "=&v"(r1) : "v"(z[0]), "v"(z[1]), "s"(0x79B1u), "v"(c));
        const U16x2 h0 = __builtin_bit_cast(U16x2, __builtin_amdgcn_perm(p1, p0, 0x07060302u));
        const U16x2 h1 = __builtin_bit_cast(U16x2, __builtin_amdgcn_perm(r1, r0, 0x07060302u));
        q[0] = __builtin_bit_cast(uint32_t, U16x2(__builtin_bit_cast(U16x2, z[0]) * (unsigned short)0x9E37u + h0));
        q[1] = __builtin_bit_cast(uint32_t, U16x2(__builtin_bit_cast(U16x2, z[1]) * (unsigned short)0x9E37u + h1));
    }
};

// The permutation backwards: the index whose key this is.
__device__ __forceinline__ uint32_t unperm32(uint32_t key, const RcKeys& keys) {
    uint32_t hi = key >> 16, lo = key & 0xffffu;
#pragma unroll
    for (int r = 5; r >= 0; --r) {                                 // (hi, lo) = (x[r + 1], x[r + 2]) -> (x[r], x[r + 1])
        const uint32_t x = lo ^ (((hi ^ keys.k[r]) + 1u) * 0x9E3779B1u >> 16);
        lo = hi;
        hi = x;
    }
    return hi << 16 | lo;
}
// Where the batch's tensors begin in the stage, and the end of the last one.  (Whole block; one barrier.)
__device__ __forceinline__ void tensor_starts(const RcBatch& batch, int64_t* start) {
    if (threadIdx.x < kMaxRcTensors) {
        const int n = batch.n_tensors, i = threadIdx.x;
        start[i] = i < n ? batch.t[i].goff : INT64_MAX;
        if (i == n - 1) start[kMaxRcTensors] = batch.t[i].goff + batch.t[i].numel;
    }
    __syncthreads();
}
// The word that holds an element, its address and the element's bit; null if the element is not one of the batch's.
__device__ __forceinline__ uint32_t* find_element(const RcBatch& batch, const int64_t* start, uint32_t element, uint32_t* word, uint32_t* bit) {
    const int64_t index = int64_t(element);
    if (index < start[0] || index >= start[kMaxRcTensors]) return nullptr;
    int t = 0;
#pragma unroll
    for (int step = kMaxRcTensors / 2; step > 0; step >>= 1)
        if (start[t + step] <= index) t += step;
    const int64_t e = index - start[t];
    *bit = uint32_t(e & 31);
    uint32_t* const at = batch.t[t].bits + (e >> 5);
    *word = *at;
    return at;
}

__global__ void rc_reset_kernel(RcState* st) {
    for (int i = threadIdx.x; i < kBins; i += blockDim.x) st->hist[i] = 0;
    if (threadIdx.x == 0) {
        st->count = 0; st->mode = 0; st->need = 0; st->prefix = 0;
        st->drawn = 0; st->rank = 0; st->window_lo = 0; st->window_hi = 0; st->probe = 0; st->done = 0;
    }
}

// *sum += the block's threads' counts, in one addition: with one per wave the queue at the one address took twice
// the time of the counting pass.
__device__ __forceinline__ void add_block_count(unsigned long long* sum, uint32_t c) {
    __shared__ uint32_t part[kThreads / 64];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) c += __shfl_down(c, off, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long all = 0;
        for (int i = 0; i < kThreads / 64; ++i) all += part[i];
        if (all) atomicAdd(sum, all);
    }
}
__global__ __launch_bounds__(kThreads) void rc_count_kernel(RcBatch batch, RcState* st) {
    uint32_t c = 0;                                                // a thread's share of fewer than 2^32 elements
    for (int task = blockIdx.x; task < batch.total_blocks; task += gridDim.x) {
        const RcTask r = rc_task(batch, task);
#pragma unroll
        for (int i = 0; i < kRows; ++i) {
            const int64_t w = r.first + i * kRowWords;            // past the end: the last word, of which nothing counts
            c += __popc(r.bits[w < r.n_words ? w : r.n_words - 1] & rc_valid(r, w));
        }
    }
    add_block_count(&st->count, c);
}

// mode 0: the base mask already holds n_freeze ones; 1: add `need` of its zeros; 2: remove `need` of its ones
// n: elements of the stage if the threshold may be guessed (rc_try_kernel()), or 0.
__global__ void rc_decide_kernel(RcState* st, unsigned long long n_freeze, unsigned long long n, long long* stats) {
    if (threadIdx.x != 0) return;
    const unsigned long long c = st->count;
    st->mode = c == n_freeze ? 0u : (c < n_freeze ? 1u : 2u);
    st->need = c < n_freeze ? n_freeze - c : c - n_freeze;
    st->prefix = 0;
    if (stats) { stats[0] = (long long)c; stats[1] = st->mode; stats[2] = 0; }
    if (n == 0 || st->mode == 0) return;
    // The need-th smallest of `all` keys drawn from [0, 2^32): six standard deviations on either side.
    const double all = double(st->mode == 1 ? n - c : c), share = double(st->need) / all;
    const double half = 6 * 65536 * sqrt(share * (1 - share) / all);                 // in top halves of a key
    const int lo = int(share * 65536 - half) - 1, hi = min(int(share * 65536 + half) + 2, 65536);
    if (lo < 1 || hi - lo > kWindowTops) return;
    st->window_lo = uint32_t(lo);
    st->window_hi = uint32_t(hi);
}

// Is the mask what the guess takes it for, one that has nothing to do with the keys?  (A mask that the same seed has
// made is not: its candidates' keys begin where the last threshold was.)  Of the keys below the expected threshold 2^15, spread evenly, are
// looked up: those of candidates have to be as many as expected, to six standard deviations.  However few candidates are to
// be drawn, that tells 16 % of them for 2^28 elements, 6.5 % for 1.74e9, seven in ten of them candidates.  (2^16 keys: 10 us more of 955; 2^15: 4.)
constexpr int kProbeBits = 15;
__device__ __forceinline__ uint64_t probed_keys(const RcState* st) { return uint64_t(st->window_lo + st->window_hi) << 15; }       // < 2^32
__global__ __launch_bounds__(kThreads) void rc_probe_kernel(RcBatch batch, RcState* st, RcKeys keys) {
    __shared__ int64_t start[kMaxRcTensors + 1];
    if (st->window_hi == 0) return;
    tensor_starts(batch, start);
    const uint32_t i = blockIdx.x * kThreads + threadIdx.x;        // grid: 2^kProbeBits threads
    const uint32_t key = uint32_t((uint64_t(i << (32 - kProbeBits) | ((i * 0x9E3779B1u) >> kProbeBits)) * probed_keys(st)) >> 32);
    uint32_t word, bit;
    uint32_t* const at = find_element(batch, start, unperm32(key, keys), &word, &bit);
    const unsigned long long ones = __ballot(at && ((word >> bit) & 1u) == (st->mode == 2 ? 1u : 0u));
    if ((threadIdx.x & 63) == 0 && ones) atomicAdd(&st->probe, uint32_t(__popcll(ones)));
}
__device__ __forceinline__ bool guess_holds(const RcState* st) {
    if (st->window_hi == 0) return false;
    const double expected = double(1 << kProbeBits) * double(st->need) / double(probed_keys(st));
    return fabs(double(st->probe) - expected) <= 6 * sqrt(expected) + 8;
}

// No lane's word has more than kFew candidates: key by key is then quicker than all 32 in pairs (a loop of as many
// rounds as the fullest word has candidates).  1.74e9 elements, 5 % candidates 1.51 -> 0.85 ms, 1 % 0.45; 61e6
// elements, 0.1 %: 119 -> 72 us.  From a task's first fuller word on nothing is asked any more (asking at each
// word took 0.8 % of the time at 30 % candidates), and the 32 registers of a Halves are filled only then.
constexpr int kFew = 7;
__device__ __forceinline__ bool few_candidates(uint32_t cand) { return __ballot(__popc(cand) > kFew) == 0; }

// Histogram of the candidates' first digit, the top 11 bits of the key.
template <bool kCarry>
__device__ __forceinline__ void rc_hist_word(const Halves& h, uint32_t cand, uint32_t high2, uint32_t* bins) {
#pragma unroll
    for (int p = 0; p < 16; p += 2) {
        uint32_t x[2];
        h.top<kCarry>(p, high2, x);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            atomicAdd(&bins[(x[j] >> 5) & 0x7ffu], (cand >> (p + j)) & 1u);
            atomicAdd(&bins[x[j] >> 21], (cand >> (p + j + 16)) & 1u);
        }
    }
}
__global__ __launch_bounds__(kThreads) void rc_hist_kernel(RcBatch batch, RcState* st, RcKeys keys) {
    __shared__ uint32_t bins[kBins];
    const uint32_t mode = st->mode;
    if (mode == 0 || st->done) return;                              // block-uniform
    for (int i = threadIdx.x; i < kBins; i += kThreads) bins[i] = 0;
    __syncthreads();
    for (int task = blockIdx.x; task < batch.total_blocks; task += gridDim.x) {
        const RcTask r = rc_task(batch, task);
        uint32_t next = r.first < r.n_words ? r.bits[r.first] : 0u;
        int i = 0;
#pragma unroll 1
        for (; i < kRows; ++i) {                                   // as long as the words have few candidates
            const int64_t w = r.first + i * kRowWords;
            uint32_t cand = (mode == 1 ? ~next : next) & rc_valid(r, w);
            if (!few_candidates(cand)) break;
            if (i + 1 < kRows && w + kRowWords < r.n_words) next = r.bits[w + kRowWords];
            for (; cand; cand &= cand - 1)
                atomicAdd(&bins[perm32(r.index0 + (uint32_t(i) << 16) + uint32_t(__ffs(cand) - 1), keys) >> 21], 1u);
        }
        if (i == kRows) continue;
        Halves h;
        h.init(r.index0, keys);
        const bool any_carry = __ballot(h.carry) != 0;
#pragma unroll 1
        for (; i < kRows; ++i) {
            const int64_t w = r.first + i * kRowWords;
            const uint32_t word = next;
            if (i + 1 < kRows && w + kRowWords < r.n_words) next = r.bits[w + kRowWords];
            const uint32_t cand = (mode == 1 ? ~word : word) & rc_valid(r, w);
            if (__ballot(cand != 0) == 0) continue;
            const uint32_t high2 = ((r.index0 >> 16) + i) * 0x10001u;
            if (any_carry) rc_hist_word<true>(h, cand, high2, bins);
            else rc_hist_word<false>(h, cand, high2, bins);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kBins; i += kThreads)
        if (bins[i]) atomicAdd(&st->hist[i], bins[i]);
}

// Histogram of the digit behind the prefix, over the candidates whose key starts with the prefix: the
// 2^open keys are taken back to their indices and those looked up in the mask.  One key per thread;
// the digit is the top nbits of the open ones.
__global__ __launch_bounds__(kThreads) void rc_enum_kernel(RcBatch batch, RcState* st, RcKeys keys, int open, int nbits) {
    __shared__ int64_t start[kMaxRcTensors + 1];
    const uint32_t mode = st->mode;
    if (mode == 0 || st->done) return;
    tensor_starts(batch, start);
    const uint32_t k = blockIdx.x * kThreads + threadIdx.x;        // grid: 2^open threads
    uint32_t word, bit;
    const bool cand = find_element(batch, start, unperm32(st->prefix << open | k, keys), &word, &bit) && ((word >> bit) & 1u) == (mode == 2 ? 1u : 0u);
    const int below = open - nbits;
    if (below >= 6) {                                              // a wave's keys have one digit
        const unsigned long long ones = __ballot(cand);
        if ((threadIdx.x & 63) == 0 && ones) atomicAdd(&st->hist[k >> below], uint32_t(__popcll(ones)));
    } else if (cand) {
        atomicAdd(&st->hist[k >> below], 1u);
    }
}

// The bin in which the rank-th smallest key lies; *before: keys in the bins in front of it, *total: in all of them.
// One block of 256 threads: each sums 8 neighbouring bins, thread 0 walks the 256 partial sums
// and then the 8 bins of the one that holds the rank; all of them clear the histogram.  (Thread 0 has the results.)
__device__ __forceinline__ int find_bin(RcState* st, int bins, unsigned long long rank, unsigned long long* before, unsigned long long* total) {
    __shared__ unsigned long long part[kThreads];
    constexpr int kPer = kBins / kThreads;
    unsigned long long mine = 0;
    for (int q = 0; q < kPer; ++q) mine += st->hist[threadIdx.x * kPer + q];
    part[threadIdx.x] = mine;
    __syncthreads();
    int b = 0;
    if (threadIdx.x == 0) {
        *before = *total = 0;
        int g = 0;
        for (; g < kThreads - 1 && (g + 1) * kPer < bins; ++g) {
            if (*before + part[g] >= rank) break;
            *before += part[g];
        }
        *total = *before;
        for (int i = g; i < kThreads; ++i) *total += part[i];
        for (b = g * kPer; b < bins - 1; ++b) {
            const unsigned long long hb = st->hist[b];
            if (*before + hb >= rank) break;
            *before += hb;
        }
    }
    __syncthreads();
    for (int q = 0; q < kPer; ++q) st->hist[threadIdx.x * kPer + q] = 0;
    return b;
}
// Extend the prefix by the digit of the need-th smallest key.
__global__ __launch_bounds__(kThreads) void rc_pick_kernel(RcState* st, int nbits, int last, long long* stats) {
    if (st->done) return;
    unsigned long long before, total;
    const int b = find_bin(st, 1 << nbits, st->need, &before, &total);
    if (threadIdx.x != 0) return;
    if (st->mode != 0) {
        st->need -= before;                      // rank inside the bin, >= 1
        st->prefix = (st->prefix << nbits) | uint32_t(b);
    }
    if (last && stats) stats[2] = st->mode == 0 ? 0 : (long long)st->prefix;
}

// After the last digit the prefix is a full key: the need-th smallest.  Candidates with a key
// not above it are the drawn ones.  The top halves of the keys decide, but for those that equal
// the threshold's: a word that has one is looked at element by element (one word in 2000).
// Two keys at a time: (top - x, not below 0; at most 1) is shifted into the halves of `drawn` - 3 instructions
// where comparing them one by one took 5.
template <bool kCarry, bool kTie>
__device__ __forceinline__ uint32_t rc_drawn(const Halves& h, uint32_t high2, uint32_t top, bool& tie) {
    const uint32_t top2 = top * 0x10001u;
    uint32_t drawn = 0;
    U16x2 nearest = {0xffff, 0xffff};
#pragma unroll
    for (int p = 14; p >= 0; p -= 2) {
        uint32_t x[2], less0, less1;
        h.top<kCarry>(p, high2, x);
        // (left to itself the compiler makes comparisons of the halves again)
        asm("v_pk_sub_u16 %1, %5, %3 clamp\n\t"
            "v_pk_sub_u16 %2, %5, %4 clamp\n\t"
            "v_pk_min_u16 %1, %1, %6\n\t"
            "v_pk_min_u16 %2, %2, %6\n\t"
            "v_pk_mad_u16 %0, %0, %7, %2\n\t"
            "v_pk_mad_u16 %0, %0, %7, %1"
            : "+&v"(drawn), "=&v"(less0), "=&v"(less1) : "v"(x[0]), "v"(x[1]), "s"(top2), "s"(0x10001u), "s"(0x20002u));
        if (kTie) {
#pragma unroll
            for (int j = 0; j < 2; ++j) nearest = __builtin_elementwise_min(nearest, __builtin_bit_cast(U16x2, x[j] ^ top2));
        }
    }
    tie = kTie && (nearest.x == 0 || nearest.y == 0);
    return drawn;
}
// The drawn ones of a word's candidates, one by one.
__device__ __forceinline__ uint32_t rc_drawn_each(uint32_t cand, uint32_t index0, const RcKeys& keys, uint32_t threshold) {
    uint32_t drawn = 0;
    for (; cand; cand &= cand - 1) {
        const int b = __ffs(cand) - 1;
        if (perm32(index0 + uint32_t(b), keys) <= threshold) drawn |= 1u << b;
    }
    return drawn;
}
__global__ __launch_bounds__(kThreads) void rc_apply_kernel(RcBatch batch, const RcState* st, RcKeys keys) {
    const uint32_t mode = st->mode;
    if (mode == 0 || st->done) return;
    const uint32_t threshold = st->prefix;
    for (int task = blockIdx.x; task < batch.total_blocks; task += gridDim.x) {
        const RcTask r = rc_task(batch, task);
        uint32_t next = r.first < r.n_words ? r.bits[r.first] : 0u;
        int i = 0;
#pragma unroll 1
        for (; i < kRows; ++i) {                                   // as long as the words have few candidates
            const int64_t w = r.first + i * kRowWords;
            const uint32_t old = next;
            const uint32_t cand = (mode == 1 ? ~old : old) & rc_valid(r, w);
            if (!few_candidates(cand)) break;
            if (i + 1 < kRows && w + kRowWords < r.n_words) next = r.bits[w + kRowWords];
            const uint32_t drawn = rc_drawn_each(cand, r.index0 + (uint32_t(i) << 16), keys, threshold);
            if (drawn) r.bits[w] = mode == 1 ? (old | drawn) : (old & ~drawn);
        }
        if (i == kRows) continue;
        Halves h;
        h.init(r.index0, keys);
        const bool any_carry = __ballot(h.carry) != 0;
#pragma unroll 1
        for (; i < kRows; ++i) {
            const int64_t w = r.first + i * kRowWords;
            const uint32_t old = next;
            if (i + 1 < kRows && w + kRowWords < r.n_words) next = r.bits[w + kRowWords];
            const uint32_t cand = (mode == 1 ? ~old : old) & rc_valid(r, w);
            if (__ballot(cand != 0) == 0) continue;
            const uint32_t high2 = ((r.index0 >> 16) + i) * 0x10001u;
            bool tie;
            uint32_t drawn = any_carry ? rc_drawn<true, true>(h, high2, threshold >> 16, tie) : rc_drawn<false, true>(h, high2, threshold >> 16, tie);
            drawn &= cand;
            if (tie) drawn = rc_drawn_each(cand, r.index0 + (uint32_t(i) << 16), keys, threshold);
            if (drawn) r.bits[w] = mode == 1 ? (old | drawn) : (old & ~drawn);
        }
    }
}

// ---- a large mask: one keyed pass instead of two ----
// Keys have nothing to do with a mask that was made without them, so how many candidates lie below a threshold is
// known to a few parts in 10^5 before any key is worked out.  rc_try_kernel() draws, in place, what lies below the
// lower end of a window around the expected threshold, counts it and keeps the words as they were; the window's keys
// (at most 2^22) are taken back to their elements, which gives the threshold and the rest of the drawing.  Where the
// count shows that the threshold was not in the window, rc_restore_kernel() puts the mask back and the passes
// above do it all; where it was, they return at once.  The result is the same in any case; a guess that the probe let pass and
// the count did not costs its pass and the restoring: 1.74e9 elements, 5 % of the candidates below the threshold taken out, 2.30 ms instead of 1.47.
// The pass takes 13.5 vector instructions per element (the histogram pass 14.5, the apply pass 15.1), 93 % of the vector units' slots (97 %, 92 %).
__global__ __launch_bounds__(kThreads) void rc_try_kernel(RcBatch batch, RcState* st, RcKeys keys) {
    if (!guess_holds(st)) return;
    const uint32_t mode = st->mode, top = st->window_lo;           // top >= 1
    const uint32_t last = (top << 16) - 1;                          // the largest key to be drawn
    uint32_t count = 0;
    for (int task = blockIdx.x; task < batch.total_blocks; task += gridDim.x) {
        const RcTask r = rc_task(batch, task);
        uint32_t next = r.first < r.n_words ? r.bits[r.first] : 0u;
        int i = 0;
        auto done = [&](int64_t w, uint32_t old, uint32_t drawn) __attribute__((always_inline)) {
            if (w < r.n_words) r.undo[w] = old;
            if (drawn) r.bits[w] = mode == 1 ? (old | drawn) : (old & ~drawn);
            count += __popc(drawn);
        };
#pragma unroll 1
        for (; i < kRows; ++i) {                                   // as long as the words have few candidates
            const int64_t w = r.first + i * kRowWords;
            const uint32_t old = next;
            const uint32_t cand = (mode == 1 ? ~old : old) & rc_valid(r, w);
            if (!few_candidates(cand)) break;
            if (i + 1 < kRows && w + kRowWords < r.n_words) next = r.bits[w + kRowWords];
            done(w, old, rc_drawn_each(cand, r.index0 + (uint32_t(i) << 16), keys, last));
        }
        if (i == kRows) continue;
        Halves h;
        h.init(r.index0, keys);
        const bool any_carry = __ballot(h.carry) != 0;
#pragma unroll 1
        for (; i < kRows; ++i) {
            const int64_t w = r.first + i * kRowWords;
            const uint32_t old = next;
            if (i + 1 < kRows && w + kRowWords < r.n_words) next = r.bits[w + kRowWords];
            const uint32_t cand = (mode == 1 ? ~old : old) & rc_valid(r, w);
            uint32_t drawn = 0;
            if (__ballot(cand != 0) != 0) {
                const uint32_t high2 = ((r.index0 >> 16) + i) * 0x10001u;
                bool tie;
                drawn = any_carry ? rc_drawn<true, false>(h, high2, top, tie) : rc_drawn<false, false>(h, high2, top, tie);
            }
            done(w, old, drawn & cand);
        }
    }
    add_block_count(&st->drawn, count);
}

// The window's keys, taken back to their elements.  level 0: how many are candidates, in bins of 2^11 keys;
// 1: in the bin found, key by key; 2: draws those up to the threshold.
__global__ __launch_bounds__(kThreads) void rc_window_kernel(RcBatch batch, RcState* st, RcKeys keys, int level) {
    __shared__ int64_t start[kMaxRcTensors + 1];
    if (level == 0 ? !guess_holds(st) : level == 1 ? st->rank == 0 : st->done == 0) return;
    tensor_starts(batch, start);
    const uint32_t first = (st->window_lo << 16) + (level == 1 ? st->prefix << 11 : 0u);
    const uint32_t n = level == 0 ? (st->window_hi - st->window_lo) << 16 : level == 1 ? 2048u : st->prefix - first + 1;
    const uint32_t one = st->mode == 2 ? 1u : 0u;
    for (uint32_t k = blockIdx.x * kThreads + threadIdx.x; k < n; k += gridDim.x * kThreads) {      // n: a multiple of 64 but at level 2
        uint32_t word = 0, bit = 0;
        uint32_t* const at = find_element(batch, start, unperm32(first + k, keys), &word, &bit);
        const bool cand = at && ((word >> bit) & 1u) == one;
        if (level == 0) {                                          // a wave's keys share their bin
            const unsigned long long ones = __ballot(cand);
            if ((threadIdx.x & 63) == 0 && ones) atomicAdd(&st->hist[k >> 11], uint32_t(__popcll(ones)));
        } else if (cand) {
            if (level == 1) atomicAdd(&st->hist[k], 1u);
            else if (one) atomicAnd(at, ~(1u << bit));
            else atomicOr(at, 1u << bit);
        }
    }
}
// Level 0: is the threshold in the window, and in which bin; 1: the threshold.
__global__ __launch_bounds__(kThreads) void rc_window_pick_kernel(RcState* st, int level, long long* stats) {
    if (level == 0 ? !guess_holds(st) : st->rank == 0) return;
    const bool below = level == 1 || st->drawn < st->need;
    const unsigned long long rank = level == 1 ? st->rank : below ? st->need - st->drawn : 1;
    unsigned long long before, total;
    const uint32_t b = uint32_t(find_bin(st, kBins, rank, &before, &total));
    if (threadIdx.x != 0 || !below || total < rank) return;        // st->rank stays 0
    st->rank = rank - before;                                       // >= 1
    if (level == 0) {
        st->prefix = b;
    } else {
        st->prefix = (st->window_lo << 16) + (st->prefix << 11) + b;
        st->done = 1;
        if (stats) stats[2] = (long long)st->prefix;
    }
}
// The guess was wrong: the mask as it was.
__global__ __launch_bounds__(kThreads) void rc_restore_kernel(RcBatch batch, RcState* st) {
    if (st->done || !guess_holds(st)) return;
    for (int task = blockIdx.x; task < batch.total_blocks; task += gridDim.x) {
        const RcTask r = rc_task(batch, task);
#pragma unroll
        for (int i = 0; i < kRows; ++i) {
            const int64_t w = r.first + i * kRowWords;
            if (w < r.n_words) r.bits[w] = r.undo[w];
        }
    }
}

// grid: (chunks, runs).  Run blockIdx.y, words [blockIdx.x * 4096 ...) four per thread and sweep.
__global__ __launch_bounds__(kThreads) void fill_words_kernel(FillBatch batch) {
    const FillRunDesc& R = batch.r[blockIdx.y];
    for (int64_t w = int64_t(blockIdx.x) * kThreads + threadIdx.x; w < R.n_words; w += int64_t(gridDim.x) * kThreads)
        R.dst[w] = R.value;
}

int rc_grid(const RcBatch& batch) { return batch.total_blocks < kGrid ? batch.total_blocks : kGrid; }

}  // namespace

hipError_t launch_fill_words(hipStream_t stream, const FillBatch& batch) {
    if (batch.n_runs == 0) return hipSuccess;
    int64_t longest = 0;
    for (int i = 0; i < batch.n_runs; ++i) longest = batch.r[i].n_words > longest ? batch.r[i].n_words : longest;
    int64_t bx = (longest + kThreads * 4 - 1) / (kThreads * 4);
    if (bx < 1) bx = 1;
    if (bx > 4096) bx = 4096;
    hipLaunchKernelGGL(fill_words_kernel, dim3(unsigned(bx), unsigned(batch.n_runs)), dim3(kThreads), 0, stream, batch);
    return hipGetLastError();
}

int64_t norm_elems_per_block() { return kNormElemsPerBlock; }
int rc_tasks(int64_t numel) {
    const int64_t rows = ((numel + 31) / 32 + kRowWords - 1) / kRowWords;
    return int((rows + kRows - 1) / kRows * kColumns);
}
size_t rc_state_bytes() { return sizeof(RcState); }

hipError_t launch_autofreeze_norms(hipStream_t stream, NormBatch& batch, int n_tensors, bool update_snapshot) {
    batch.n_tensors = n_tensors;
    batch.update_snapshot = update_snapshot ? 1 : 0;
    if (n_tensors == 0 || batch.total_blocks == 0) return hipSuccess;
    if (!batch.partials) return hipErrorInvalidValue;
    hipLaunchKernelGGL(norm_kernel, dim3(batch.total_blocks), dim3(kNormThreads), kNormResidencyLds, stream, batch);
    hipLaunchKernelGGL(norm_finish_kernel, dim3(n_tensors), dim3(kSumSlots), 0, stream, batch);
    return hipGetLastError();
}

hipError_t launch_rc_begin(hipStream_t stream, RcState* st) {
    hipLaunchKernelGGL(rc_reset_kernel, dim3(1), dim3(256), 0, stream, st);
    return hipGetLastError();
}
hipError_t launch_rc_count(hipStream_t stream, RcBatch& batch, RcState* st) {
    if (batch.n_tensors == 0 || batch.total_blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(rc_count_kernel, dim3((rc_grid(batch) + 1) / 2), dim3(kThreads), 0, stream, batch, st);
    return hipGetLastError();
}
hipError_t launch_rc_decide(hipStream_t stream, RcState* st, uint64_t n_freeze, uint64_t guess_of, int64_t* stats) {
    hipLaunchKernelGGL(rc_decide_kernel, dim3(1), dim3(64), 0, stream, st, (unsigned long long)n_freeze, (unsigned long long)guess_of,
                       reinterpret_cast<long long*>(stats));
    return hipGetLastError();
}
hipError_t launch_rc_probe(hipStream_t stream, RcBatch& batch, RcState* st, const RcKeys& keys) {
    if (batch.n_tensors == 0 || batch.total_blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(rc_probe_kernel, dim3((1 << kProbeBits) / kThreads), dim3(kThreads), 0, stream, batch, st, keys);
    return hipGetLastError();
}
hipError_t launch_rc_try(hipStream_t stream, RcBatch& batch, RcState* st, const RcKeys& keys) {
    if (batch.n_tensors == 0 || batch.total_blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(rc_try_kernel, dim3(rc_grid(batch)), dim3(kThreads), 0, stream, batch, st, keys);
    return hipGetLastError();
}
hipError_t launch_rc_window(hipStream_t stream, RcBatch& batch, RcState* st, const RcKeys& keys, int level) {
    if (batch.n_tensors == 0 || batch.total_blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(rc_window_kernel, dim3(level == 1 ? 2048 / kThreads : kGrid), dim3(kThreads), 0, stream, batch, st, keys, level);
    return hipGetLastError();
}
hipError_t launch_rc_window_pick(hipStream_t stream, RcState* st, int level, int64_t* stats) {
    hipLaunchKernelGGL(rc_window_pick_kernel, dim3(1), dim3(kThreads), 0, stream, st, level, reinterpret_cast<long long*>(stats));
    return hipGetLastError();
}
hipError_t launch_rc_restore(hipStream_t stream, RcBatch& batch, RcState* st) {
    if (batch.n_tensors == 0 || batch.total_blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(rc_restore_kernel, dim3((rc_grid(batch) + 1) / 2), dim3(kThreads), 0, stream, batch, st);
    return hipGetLastError();
}
hipError_t launch_rc_hist(hipStream_t stream, RcBatch& batch, RcState* st, const RcKeys& keys) {
    if (batch.n_tensors == 0 || batch.total_blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(rc_hist_kernel, dim3(rc_grid(batch)), dim3(kThreads), 0, stream, batch, st, keys);
    return hipGetLastError();
}
hipError_t launch_rc_enum(hipStream_t stream, RcBatch& batch, RcState* st, const RcKeys& keys, int open, int nbits) {
    if (batch.n_tensors == 0 || batch.total_blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(rc_enum_kernel, dim3((1u << open) / kThreads), dim3(kThreads), 0, stream, batch, st, keys, open, nbits);
    return hipGetLastError();
}
hipError_t launch_rc_pick(hipStream_t stream, RcState* st, int nbits, bool last, int64_t* stats) {
    hipLaunchKernelGGL(rc_pick_kernel, dim3(1), dim3(kThreads), 0, stream, st, nbits, last ? 1 : 0,
                       reinterpret_cast<long long*>(stats));
    return hipGetLastError();
}
hipError_t launch_rc_apply(hipStream_t stream, RcBatch& batch, RcState* st, const RcKeys& keys) {
    if (batch.n_tensors == 0 || batch.total_blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(rc_apply_kernel, dim3(rc_grid(batch)), dim3(kThreads), 0, stream, batch, st, keys);
    return hipGetLastError();
}

}  // namespace tf
