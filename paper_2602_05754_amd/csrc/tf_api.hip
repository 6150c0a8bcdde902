// C ABI of libtf.so: argument validation, host-side planning (which layers go
// into which grouped launch; frozen tensors are left out of the weight-gradient
// plan entirely) and kernel launches.  Declarations and contracts: include/tf.h.
#include "../../include/tf.h"
#include "tf_internal.h"

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <new>
#include <vector>

struct tf_prof_rec {
    int kind;
    hipEvent_t start, stop;
};

// Sizes, in words, of the copies of their masks that large reconciliations keep: 2^24 << i and some for partly filled words.
constexpr int kUndoSizes = 4;
constexpr int64_t undo_words(int i) { return (int64_t(1) << (24 + i)) + (1 << 20); }

struct tf_ctx {
    int device_id;
    int last_hip_error;
    bool profiling;
    std::vector<tf_prof_rec> recs;      // events recorded since the last tf_profile_collect
    std::vector<hipEvent_t> pool;       // events ready for reuse
    tf::RcState* rc_state;              // device memory of tf_reconcile_mask (radix-select state)
    tf::RcState* rc_state_static;       // this device's static scratch array (tf_reconcile_mask_static)
    uint32_t* rc_undo[kUndoSizes];      // device memory of large reconciliations, each size made when first needed
    bool lowp_is_rounded_master;        // tf_assume_lowp_is_rounded_master
    double* ew_partials;                // device memory of the score sums' first level (zero between launches)
    int gemm_route;                     // tf_internal_gemm_route
    std::atomic<int> common_tiles{-1};  // tf_internal_common_tiles
};

// Device memory of tf_reconcile_mask_static: one array per GPU, part of the loaded code object,
// alive until the process ends.  In host code this name is only a handle for
// hipGetSymbolAddress; kernels get the address that call returned for the current device.
constexpr size_t kStaticScratchBytes = 8448;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
static_assert(sizeof(tf::RcState) <= kStaticScratchBytes, "the rank-search state must fit the static scratch array");

namespace {

using namespace tf;

constexpr int kMaxDevices = 64;
void* g_scratch_addr[kMaxDevices] = {nullptr};      // address of `scratch` on each device, set by tf_create

// With `device` current: the address of this device's copy of `scratch` (asked for once per device).
hipError_t static_scratch_address(int device, void** out) {
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    if (!g_scratch_addr[device]) {
        void* ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!ptr) return hipErrorInvalidSymbol;
        g_scratch_addr[device] = ptr;
    }
    *out = g_scratch_addr[device];
    return hipSuccess;
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline bool valid_dtype(int d) { return d == TF_F32 || d == TF_BF16; }
inline Dtype to_dtype(tf_dtype d) { return d == TF_BF16 ? Dtype::BF16 : Dtype::F32; }

int hip_fail(tf_ctx* ctx, hipError_t e) {
    ctx->last_hip_error = static_cast<int>(e);
    return TF_ERR_HIP;
}

// Optional per-kernel timing: a start/stop event pair around one launch, on the launch stream.
struct ProfScope {
    tf_ctx* ctx;
    hipStream_t stream;
    tf_prof_rec rec;
    bool on;
    ProfScope(tf_ctx* c, hipStream_t s, int kind) : ctx(c), stream(s), on(c->profiling) {
        if (!on) return;
        rec.kind = kind;
        for (hipEvent_t* e : {&rec.start, &rec.stop}) {
            if (!ctx->pool.empty()) { *e = ctx->pool.back(); ctx->pool.pop_back(); }
            else if (hipEventCreate(e) != hipSuccess) { on = false; return; }
        }
        (void)hipEventRecord(rec.start, stream);
    }
    ~ProfScope() {
        if (!on) return;
        (void)hipEventRecord(rec.stop, stream);
        ctx->recs.push_back(rec);
    }
};

// One planned GEMM: which layer, as which problem.
struct Planned {
    const void* A;
    const void* B;
    void* C;
    int64_t M, N, Kc;
    int64_t lda, ldb;       // row pitch of A, B in elements
    uint64_t row_bits;      // 256-row blocks that exist (MFMA kernel); all ones = dense
    // further contraction segments whose products are summed into the same C (layers that
    // share their input); matrix-core kernel only
    std::vector<Planned> more;
    int64_t rows_before = 0, rows_after = 0;   // operand rows in memory around the problem's own (sub-tensor problems)

    int64_t total_kc() const {
        int64_t k = Kc;
        for (const Planned& q : more) k += q.Kc;
        return k;
    }
};

inline bool planned_mfma_ok(const Planned& it, Layout layout, Dtype in_dtype) {
    return in_dtype == Dtype::BF16 && mfma_shape_ok(layout, it.M, it.N, it.Kc, it.lda, it.ldb, it.rows_before, it.rows_after) &&
           aligned16(it.A) && aligned16(it.B) && aligned16(it.C);
}

inline bool planned_tail_ok(const Planned& it, Layout layout, Dtype in_dtype) {
    return in_dtype == Dtype::BF16 && mfma_tail_shape_ok(layout, it.M, it.N, it.Kc, it.lda, it.ldb, it.rows_before, it.rows_after) &&
           aligned16(it.A) && aligned16(it.B) && aligned16(it.C);
}

inline uint32_t parts_of(int64_t extent, uint32_t size) { return (uint32_t(extent) + size - 1) / size; }       // extents have 31 bits
inline int64_t tiles_of(const Planned& it, uint32_t tile_m, uint32_t tile_n) { return int64_t(parts_of(it.M, tile_m)) * parts_of(it.N, tile_n); }

// What a launch is expected to take.  Its work spread evenly over the compute units and its longest
// chain of steps overlap for the most part; `overlap` says how much of the smaller of the two is left.
struct Estimate {
    double work = 0, longest = 0, tiles = 0, most_tiles = 0;      // most_tiles: of one problem
    // `part_tiles` of the problem's tiles take `part_steps` more
    void add(const Planned& it, int tile_m, int tile_n, int per_step, double tile_steps, double chain_steps, double part_tiles = 0, double part_steps = 0) {
        const double steps = parts_of(it.Kc, per_step);
        const double n = double(tiles_of(it, tile_m, tile_n));
        tiles += n;
        most_tiles = std::max(most_tiles, n);
        work += n * (steps + tile_steps) + part_tiles * part_steps;
        longest = std::max(longest, steps + chain_steps + (part_tiles > 0 ? part_steps : 0));
    }
    static double us(double even, double chain, double overlap) { return std::max(even, chain) + overlap * std::min(even, chain); }
};

// A launch of the generic kernel has a block of 256 threads per tile, and fewer than 2^32 threads.  (An extent
// is then at most that many tiles of 128: rounded up to whole tiles it still fits 31 bits.)
constexpr int64_t kMaxGenericTiles = (int64_t(1) << 24) - 1;
constexpr int64_t kMaxTiles256 = 0x3fffffff;       // tile indices are 32-bit on the device

// Launch shape of the generic kernel for these problems: the one with the least estimated time.  The
// estimates were within 15 % of the measured times (to which a launch adds some 4 us) and in their order (input gradients of a LLaMA-1B
// block, 200 tokens: 64 x 64 tiles 65 us, 128 x 64 69, 128 x 128 91; 3001 tokens: 605, 485, 400).
int pick_generic_shape(const std::vector<const Planned*>& items, Dtype in_dtype, double* best_us) {
    int best = 0;
    *best_us = 0;
    if (items.empty()) return best;
    bool any = false;
    for (int i = 0; i < kGenericShapes; ++i) {
        const GenericShape& s = generic_shape(in_dtype, i);
        Estimate e;
        for (const Planned* it : items) e.add(*it, s.tile_m, s.tile_n, in_dtype == Dtype::BF16 ? 64 : 32, s.tile_steps, s.tile_steps);
        if (e.most_tiles > kMaxGenericTiles) continue;
        const double us = Estimate::us(e.work / compute_units() * s.step_us, e.longest * s.chain_us, 0.25);
        if (!any || us < *best_us) { best = i; *best_us = us; }
        any = true;
        // The smallest fp32 tiles contract in 64 bits (error 2.5e-8, not 1.2e-7, at 256 values: the optimizer divides by
        // the root of such a sum's square).  Launches this short keep that: called step by step they wait for the
        // host (30 us a call with its other half).  On the GPU alone it costs them up to 7 us: two blocks of width
        // 256, 256 tokens, input gradients 25.3 (21.2 with 32 x 64 tiles), weight gradients 25.4 (18.1); width 128, 64
        // tokens 9.6 (10.7) and 7.3 (6.7).
        if (i == 0 && in_dtype == Dtype::F32 && us < 20) break;
    }
    if (!any) { best = kGenericShapes - 1; *best_us = HUGE_VAL; }      // too large for a launch: refused there
    return best;
}

// Input gradients on the 256 x 256-tile kernel.  A step takes 1.45 us when all units are busy (the power
// limit), 1.15 in the long tiles at a launch's end, 1.0 when there are fewer tiles than units; a tile's
// epilogue is worth 4.5 steps and, at the end of a chain, 6 with the fill of its first stages; where the tile is
// no whole one (masked stores) 3 more.  Measured in turn with the generic kernel, us, in
// brackets the latter: LLaMA-1B block, 256 tokens 136 (54), 512 140 (96), 1024 192 (144),
// 2048 251 (287); LLaMA-8B block 512 tokens 345 (259), 1024 440 (495).  (Weight gradients: tile256_launch_us().)
double tile256_us(const std::vector<const Planned*>& items, bool tail) {
    if (items.empty()) return 0;
    Estimate e;
    const uint32_t tile = gemm_mfma_tile();
    for (const Planned* it : items) e.add(*it, tile, tile, 64, tail ? 5.5 : 4.5, tail ? 7 : 6, double(tiles_of(*it, tile, tile) - int64_t(uint32_t(it->M) / tile) * (uint32_t(it->N) / tile)), 3);
    const int units = compute_units();
    return Estimate::us(e.work / units * 1.45, e.longest * (e.tiles <= units ? 1.0 : 1.15), 0.4);
}

// Launch shapes beyond the generic kernel's: the kernel for input gradients of few rows.
constexpr int64_t kMaxNarrowTiles = kMaxGenericTiles;      // blocks of 256 threads, too

inline bool planned_narrow_ok(const Planned& it, Layout layout, Dtype in_dtype) {
    return in_dtype == Dtype::BF16 && layout == Layout::kNT && ~it.row_bits == 0 && it.more.empty() &&
           narrow_shape_ok(it.M, it.N, it.Kc, it.lda, it.ldb) && aligned16(it.A) && aligned16(it.B);
}

// As pick_generic_shape(), of the shapes of the kernel for few rows; also no less than the weights take at the rate of
// a stream of them.  Rows that do not begin on cache lines cost its largest tile 15 % more than the others.
int pick_narrow_shape(const std::vector<const Planned*>& items, double* best_us) {
    int best = 0;
    *best_us = HUGE_VAL;
    double weights_us = 0;
    bool lines = true;
    for (const Planned* it : items) {
        weights_us += double(it->N) * double(it->Kc) * 2 / 5.6e6;
        lines = lines && it->ldb % 64 == 0;
    }
    for (int i = 0; i < kNarrowShapes; ++i) {
        const NarrowShape& s = narrow_shape(i);
        Estimate e;
        for (const Planned* it : items) e.add(*it, s.rows, s.cols, 64, s.tile_steps, s.chain_steps);
        if (e.most_tiles > kMaxNarrowTiles) continue;
        double us = std::max(Estimate::us(e.work / compute_units() * s.step_us, e.longest * s.chain_us, 0.25), weights_us);
        if (!lines && s.rows == 256) us *= 1.15;
        if (us < *best_us) { best = i; *best_us = us; }
    }
    return kGenericShapes + best;
}

inline bool planned_short_ok(const Planned& it, Layout layout, Dtype in_dtype) {
    return in_dtype == Dtype::BF16 && layout == Layout::kTN && ~it.row_bits == 0 && it.more.empty() &&
           short_shape_ok(it.M, it.N, it.Kc, it.lda, it.ldb) && aligned16(it.A) && aligned16(it.B) && aligned16(it.C);
}

// What the outputs of weight gradients take: written, fp32 ones added to.
double outputs_us(const std::vector<const Planned*>& items, int out_bytes, const OutputCost& cost) {
    double sum = 0;
    for (const Planned* it : items) sum += 1e-6 * double(it->M) * double(it->N) * out_bytes * (it->N * out_bytes % 128 != 0 ? cost.broken_us : cost.whole_us);
    return sum;
}
inline int output_kind(int out_bytes, bool accumulate) { return out_bytes == 2 ? 0 : accumulate ? 2 : 1; }

// Launch time, events included, of weight gradients in bf16 on the kernel for few tokens (its best launch shape) and on the 256 x 256-tile
// kernel.  Fitted to 264 launches of 64 to 1024 tokens (eleven sets of layers of widths 256 to 4096, four of them without k and v, four
// with rows that are no whole cache lines, bf16, fp32 and added fp32 outputs, three sets of buffers in turn).  A unit then takes its
// next tile whenever it is done with one; longer chains end in rounds (kRounds): 256 x 256 tiles, 172 of them 73 us at 3001 tokens, 344 144.
// The choice among all three kernels, over 708 launches of widths 256 to 4096, 64 to 8192 tokens: 1.6 % more than the fastest on average (with
// the fit to few tokens alone, 7 % from 2100 tokens on; of the other two kernels the better one, 8 to 21 %), at worst 1.34 times (1280 / 640 / 3400,
// 320 tokens, fp32: 37 us, 28).  Against the choice between those two it takes 12 % less on average, and 3 to 18 % more in some 20 launches
// whose tiles just fill the units once (widths 1024 / 4096 without k and v, 128 tokens, bf16: 16.3 us, 13.8): counting rounds there as well
// lost more elsewhere.
constexpr int kRounds = 1024;
double tiles_per_unit(double tiles, int64_t longest) {
    tiles /= compute_units();
    return longest > kRounds ? std::ceil(tiles) : tiles;
}
int64_t longest_contraction(const std::vector<const Planned*>& items) {
    int64_t kc = 0;
    for (const Planned* it : items) kc = std::max(kc, it->Kc);
    return kc;
}
double short_launch_us(const std::vector<const Planned*>& items, int out_bytes, bool accumulate, int* shape) {
    const int64_t kc = longest_contraction(items);
    const double steps = double(kc / 64 * 2 + (kc % 64 > 32 ? 2 : kc % 64 > 0 ? 1 : 0));
    double best = HUGE_VAL;
    for (int i = 0; i < kShortShapes; ++i) {
        const ShortShape& s = short_shape(i);
        const OutputCost& out = s.out[output_kind(out_bytes, accumulate)];
        double most = 0, tiles = 0;
        for (const Planned* it : items) {
            const double n = double(tiles_of(*it, s.rows, s.cols));
            most = std::max(most, n);
            tiles += n;
        }
        if (most > kMaxGenericTiles) continue;
        const double us = std::max(tiles_per_unit(tiles, kc) * (steps * s.step_us + s.tile_us), steps * s.chain_us);
        const double all_us = s.launch_us + Estimate::us(us, outputs_us(items, out_bytes, out), out.overlap);
        if (all_us < best) { best = all_us; *shape = kGenericShapes + kNarrowShapes + i; }
    }
    return best;
}
double tile256_launch_us(const std::vector<const Planned*>& items, int out_bytes, bool accumulate) {
    // a tile's epilogue in steps; up to 1024 tokens what a launch adds, and the share of tile256_us()'s time for a step
    struct { double tile_steps, launch_us, scale; OutputCost out; } constexpr kCost[3] = {
        {3.3, 10.6, 0.935, {0.131f, 0.05f, 0.45f}}, {3.25, 11.7, 0.946, {0.417f, 0.149f, 0.33f}}, {8, 20.3, 0.865, {0.469f, 0.268f, 0.561f}}};
    const auto& c = kCost[output_kind(out_bytes, accumulate)];
    const int tile = gemm_mfma_tile(), units = compute_units();
    const int64_t kc = longest_contraction(items);
    const double steps = double(parts_of(kc, 64)) + c.tile_steps, stores = outputs_us(items, out_bytes, c.out);
    double tiles = 0;
    for (const Planned* it : items) tiles += double(tiles_of(*it, tile, tile));
    if (kc > kRounds) return 10.6 + Estimate::us(tiles_per_unit(tiles, kc) * steps * 1.22, stores, c.out.overlap);
    const double us = c.scale * Estimate::us(tiles / units * steps * 1.45, (steps + 1.5) * (tiles <= units ? 1.0 : 1.15), 0.4);
    return 0.965 * (c.launch_us + Estimate::us(us, stores, c.out.overlap));
}

// The same on the generic kernel.  Up to 1024 tokens it is slower than the kernel for few tokens (1.01 to 2.3 times in 168 launches), but
// a step of 64 in a chain that has its unit to itself takes it 0.29 us, that one 0.38: from some 1500 tokens on it is the faster
// one where there are few tiles.  us, in brackets the latter: two blocks of widths 64 / 64 / 176, bf16, 1024 tokens 12.3 (11.6), 2048 17.0
// (17.9), 8192 44.9 (54.2); 128 / 64 / 344, 4096 tokens 27.6 (31.3), 8192 54.5 (70.7); 384 / 128 / 1024, 3001 tokens 45.9 (40.7).
double generic_launch_us(const std::vector<const Planned*>& items, int out_bytes, bool accumulate, int* shape) {
    double us;
    *shape = pick_generic_shape(items, Dtype::BF16, &us);
    if (us == HUGE_VAL) return us;
    constexpr double kOut[3] = {0.01, 0.05, 0.34};             // per MB of outputs
    const GenericShape& s = generic_shape(Dtype::BF16, *shape);
    const int64_t kc = longest_contraction(items);
    const double steps = double(parts_of(kc, 64)) + s.tile_steps;
    double tiles = 0, mb = 0;
    for (const Planned* it : items) {
        tiles += double(tiles_of(*it, s.tile_m, s.tile_n));
        mb += 1e-6 * double(it->M) * double(it->N) * out_bytes;
    }
    us = Estimate::us(1.1 * tiles_per_unit(tiles, kc) * steps * s.step_us, 0.75 * steps * s.chain_us, kc > kRounds ? 0 : 0.25);
    return 7.3 + us + kOut[output_kind(out_bytes, accumulate)] * mb;
}

constexpr int kFirstNarrow = kGenericShapes, kFirstShort = kFirstNarrow + kNarrowShapes, kFirstSplit = kFirstShort + kShortShapes;     // numbers of their launch shapes

// Rows and columns of a launch shape's tile (-1: the 256 x 256-tile kernel).
void tile_of(int shape, Dtype in_dtype, uint32_t* m, uint32_t* n) {
    if (shape < 0) *m = *n = gemm_mfma_tile();
    else if (shape >= kFirstSplit) { *m = split_shape(shape - kFirstSplit).tile_m; *n = split_shape(shape - kFirstSplit).tile_n; }
    else if (shape >= kFirstShort) { *m = short_shape(shape - kFirstShort).rows; *n = short_shape(shape - kFirstShort).cols; }
    else if (shape >= kGenericShapes) { *m = narrow_shape(shape - kGenericShapes).rows; *n = narrow_shape(shape - kGenericShapes).cols; }
    else { *m = generic_shape(in_dtype, shape).tile_m; *n = generic_shape(in_dtype, shape).tile_n; }
}

// tf_internal_gemm_route: by the estimates; 256 x 256 tiles for every problem that they take, but for the masked
// last steps (kRouteWhole256) or with them; the generic kernel for every problem that it takes.
// From kRouteNarrow and kRouteShort on the kernels for few rows and few tokens, by their shapes; from kRouteF32 on fp32 calls in the
// generic kernel's tiles x (input gradients) and w (weight gradients), kRouteF32 + kGenericShapes x + w; from kRouteSplit on fp32 calls on the
// kernel of bf16 pieces, by its shapes, where it takes all problems of a half.
enum { kRouteEstimated = 0, kRouteWhole256 = 1, kRouteAll256 = 2, kRouteGeneric = 3, kRouteNarrow = 4, kRouteShort = kRouteNarrow + kNarrowShapes,
       kRouteF32 = kRouteShort + kShortShapes, kRouteSplit = kRouteF32 + kGenericShapes * kGenericShapes, kRouteEnd = kRouteSplit + kSplitShapes };

// problems for 256 x 256 tiles; those whose contraction is no multiple of 64; all others
enum { kWhole = 0, kTail = 1, kOther = 2, kClasses = 3 };

// Which kernel takes which problems: on the 256 x 256-tile kernel what it takes, on one with smaller tiles the
// rest - and what it takes when the smaller tiles are expected to be done first (few tiles, or
// few long ones).
struct Routes {
    std::vector<const Planned*> cls[kClasses];
    int shape[kClasses] = {-1, -1, -1};         // launch shape; -1: 256 x 256 tiles
};

// Input gradients in bf16.
void find_input_routes(int route, bool plain, Routes& r) {
    auto smaller = [&](const std::vector<const Planned*>& v, int* shape) {
        double us;
        *shape = pick_generic_shape(v, Dtype::BF16, &us);
        if (v.empty() || route == kRouteGeneric) return us;
        for (const Planned* it : v)
            if (!planned_narrow_ok(*it, Layout::kNT, Dtype::BF16)) return us;
        double narrow_us;
        const int narrow = pick_narrow_shape(v, &narrow_us);
        if (route >= kRouteNarrow && route < kRouteShort) { *shape = kGenericShapes + route - kRouteNarrow; return 0.0; }
        // (both kernels' estimates leave out what a launch adds, of which the generic kernel has 2 us more: over nine sets of
        // layers of widths 256 to 4096, 32 to 2048 tokens, the choice among all three kernels is 3 % off the best on average,
        // 16 % faster than without the one for few rows, and at worst 4 % slower, at 768 tokens of a LLaMA-1B block.  Between 136 and
        // 391 tokens, which those sets leave out but for 200 and 256, it misses more: us, chosen and fastest, three sets of buffers in turn: two
        // LLaMA-1B blocks, 264 tokens 112 and 106; one LLaMA-8B block 200 and 184; widths 3328 / 832 / 11000, 136 tokens 154 and 136, 320 tokens
        // 257 and 199)
        if (narrow_us < us + 2) { *shape = narrow; us = narrow_us; }
        return us;
    };
    if (plain && route != kRouteWhole256 && route != kRouteAll256) {
        int s;
        if (smaller(r.cls[kWhole], &s) < tile256_us(r.cls[kWhole], false) || route == kRouteGeneric) r.shape[kWhole] = s;
    }
    if (!r.cls[kTail].empty() && route != kRouteAll256) {
        std::vector<const Planned*> both = r.cls[kTail];
        both.insert(both.end(), r.cls[kOther].begin(), r.cls[kOther].end());
        int s;
        const double together = smaller(both, &s);
        if (together < tile256_us(r.cls[kTail], true) + smaller(r.cls[kOther], &s) || route == kRouteGeneric) {
            r.cls[kOther] = both;
            r.cls[kTail].clear();
        }
    }
    smaller(r.cls[kOther], &r.shape[kOther]);
}

// Weight gradients in bf16: each class on 256 x 256 tiles, on smaller ones in a launch of its own, or in one with those
// that 256 x 256 tiles do not take, whichever is expected to be done first.
void find_weight_routes(int out_bytes, bool accumulate, int route, Routes& r) {
    auto can_move = [](const std::vector<const Planned*>& v) {
        for (const Planned* it : v)
            if (!planned_short_ok(*it, Layout::kTN, Dtype::BF16)) return false;
        return true;
    };
    auto smaller = [&](const std::vector<const Planned*>& v, int* shape) {
        if (v.empty()) return 0.0;
        if (route >= kRouteShort && route < kRouteF32 && can_move(v)) { *shape = kFirstShort + route - kRouteShort; return 0.0; }
        const bool few = route != kRouteGeneric && can_move(v);
        double few_us = HUGE_VAL;
        int s = 0;
        if (few) few_us = short_launch_us(v, out_bytes, accumulate, &s);
        if (few_us < HUGE_VAL && longest_contraction(v) <= kRounds) { *shape = s; return few_us; }      // (see generic_launch_us())
        const double us = generic_launch_us(v, out_bytes, accumulate, shape);
        if (few_us < us) *shape = s;
        return std::min(us, few_us);
    };
    double other_us = smaller(r.cls[kOther], &r.shape[kOther]);
    for (const int c : {kTail, kWhole}) {
        std::vector<const Planned*>& v = r.cls[c];
        if (v.empty() || !can_move(v) || route == kRouteAll256 || (route == kRouteWhole256 && c == kWhole)) continue;
        int alone = -1, joint = -1;
        double alone_us = HUGE_VAL, joint_us;
        std::vector<const Planned*> both = r.cls[kOther];
        both.insert(both.end(), v.begin(), v.end());
        joint_us = smaller(both, &joint);
        if (!can_move(r.cls[kOther])) {
            // The others are for the generic kernel only: it takes all of them if it would take these too, or if that saves more
            // than a launch: its estimate is up to a fifth short of launches of three to six tiles per unit.  us, whole calls, together
            // and in two launches: widths 256 / 256 / 688 and an output of 1001, 320 tokens 24.2, 29.4; 2048 x 2048 and 36 x 256, 320 tokens 25.1,
            // 26.6, 4096 tokens 106, 96.
            alone_us = smaller(v, &alone);
            if (alone >= kGenericShapes) joint_us = longest_contraction(v) <= 512 ? 1.2 * joint_us : HUGE_VAL;
        }
        const bool forced = route == kRouteGeneric || (route >= kRouteShort && route < kRouteF32);
        if (!forced && tile256_launch_us(v, out_bytes, accumulate) + other_us <= std::min(alone_us + other_us, joint_us)) continue;
        if (alone_us + other_us < joint_us) {
            r.shape[c] = alone;
        } else {
            r.cls[kOther] = both;
            r.shape[kOther] = joint;
            other_us = joint_us;
            v.clear();
        }
    }
}

// (fp32: all are kOther, for a launch shape that choose_f32() gives them)
hipError_t find_routes(const std::vector<Planned>& items, Layout layout, Dtype in_dtype, Dtype out_dtype, bool accumulate, int route, Routes& r) {
    bool plain = true;                          // no row bits, no segments: the kernels with smaller tiles could take them too
    for (const Planned& it : items) {
        bool ok = planned_mfma_ok(it, layout, in_dtype);
        for (const Planned& q : it.more) ok = ok && planned_mfma_ok(q, layout, in_dtype);
        const bool special = ~it.row_bits != 0 || !it.more.empty();
        if (ok) { r.cls[kWhole].push_back(&it); plain = plain && !special; }
        else if (special) return hipErrorInvalidValue;          // only the 256 x 256-tile kernel knows these
        else r.cls[planned_tail_ok(it, layout, in_dtype) ? kTail : kOther].push_back(&it);
    }
    if (in_dtype == Dtype::F32) return hipSuccess;
    if (layout == Layout::kTN) find_weight_routes(out_dtype == Dtype::BF16 ? 2 : 4, accumulate, route, r);
    else find_input_routes(route, plain, r);
    return hipSuccess;
}

void fill(GemmProblem& gp, const Planned& it, int64_t tile_start, int n_seg) {
    gp.A = it.A; gp.B = it.B; gp.C = it.C;
    gp.M = int32_t(it.M); gp.N = int32_t(it.N); gp.Kc = int32_t(it.Kc);
    gp.lda = int32_t(it.lda); gp.ldb = int32_t(it.ldb); gp.row_bits = it.row_bits;
    gp.tile_start = int32_t(tile_start);
    gp.n_seg = n_seg;
    // a problem narrower than one tile window: prefer running over its end to starting before its beginning
    const int64_t short_by = it.M < gemm_mfma_tile() ? gemm_mfma_tile() - it.M : 0;
    const int64_t after = std::min(it.rows_after, short_by), before = std::min(it.rows_before, short_by - after);
    gp.m_slack = uint32_t(before) | (uint32_t(after) << 16);
}

// Launches of the kernel of bf16 pieces have blocks of 512 threads, fewer than 2^32 in all.
constexpr int64_t kMaxSplitTiles = (int64_t(1) << 23) - 1;

// As pick_generic_shape(), of the shapes of the kernel of bf16 pieces.  Fitted to 210 launches on each (seven sets of layers of widths 128
// to 1280, 20 to 2048 tokens, input gradients, weight gradients and both): 6 and 7 % off the measured times.
int pick_split_shape(const std::vector<const Planned*>& items, double* best_us) {
    int best = 0;
    *best_us = HUGE_VAL;
    for (int i = 0; i < kSplitShapes; ++i) {
        const SplitShape& s = split_shape(i);
        Estimate e;
        for (const Planned* it : items) e.add(*it, s.tile_m, s.tile_n, 32, s.tile_steps, s.chain_steps);
        if (e.most_tiles > kMaxSplitTiles) continue;
        const double us = s.launch_us + Estimate::us(e.work / compute_units() * s.step_us, e.longest * s.chain_us, s.overlap);
        if (us < *best_us) { best = i; *best_us = us; }
    }
    return kFirstSplit + best;
}

// What the two halves of an fp32 call, input gradients `x` and weight gradients `w`, run on: launch shapes, and whether they share a
// launch.  The input gradients go to the kernel of bf16 pieces where that is expected to be done first, by themselves - their bits
// must not depend on which tensors are frozen.  The weight gradients join them in one launch or have one of their own on the other
// kernel, as is expected to be done first.  A launch of the generic kernel takes some 4 us that its estimate leaves out.  (Widths 864 / 864 /
// 2798, 475 tokens, where the two kernels' input gradients are level: 98 and 100 us, with all weight gradients 139 and 193.  Where
// the generic kernel's are ahead they stay there, 440 tokens 90 and 98 us, though with the weight gradients it is 178 and 134.)
// What the generic kernel would contract in 64 bits (its smallest tiles) stays there: the other's error is less than that of sums in
// 32 bits (6.8e-8 and 1.16e-7 at 200 values, 1.84e-7 and 1.98e-7 at 2731), not than 2.5e-8.
struct ChoiceF32 { int x, w; bool together; };
ChoiceF32 choose_f32(const std::vector<const Planned*>& x, const std::vector<const Planned*>& w, int route) {
    constexpr double kLaunch = 4;
    struct Half { int generic, split; double generic_us, split_us; };
    auto half = [&](const std::vector<const Planned*>& v, Layout layout) {
        Half h{0, kFirstSplit, 0, HUGE_VAL};
        h.generic = pick_generic_shape(v, Dtype::F32, &h.generic_us);
        h.generic_us += kLaunch;
        if (route >= kRouteF32 && route < kRouteSplit) h.generic = layout == Layout::kNT ? (route - kRouteF32) / kGenericShapes : (route - kRouteF32) % kGenericShapes;
        if (v.empty() || route == kRouteGeneric || (route < kRouteSplit && (route >= kRouteF32 || h.generic == 0))) return h;
        for (const Planned* it : v)
            if (!split_shape_ok(layout, it->M, it->N, it->Kc, it->lda, it->ldb)) return h;
        h.split = pick_split_shape(v, &h.split_us);
        if (route >= kRouteSplit) { h.split = kFirstSplit + route - kRouteSplit; h.split_us = 0; }
        return h;
    };
    const Half hx = half(x, Layout::kNT), hw = half(w, Layout::kTN);
    const bool x_split = hx.split_us < hx.generic_us, w_split = hw.split_us < hw.generic_us;
    const ChoiceF32 apart{x_split ? hx.split : hx.generic, w_split ? hw.split : hw.generic, false};
    if (x.empty() || w.empty() || x.size() + w.size() > size_t(kMaxProblemsPerLaunch)) return apart;
    if (!x_split) {
        const ChoiceF32 joint{hx.generic, hw.generic, true};
        if (!w_split) return joint;
        Estimate e;
        auto add = [&](const std::vector<const Planned*>& v, int shape) {
            const GenericShape& s = generic_shape(Dtype::F32, shape);
            Estimate steps;
            for (const Planned* it : v) steps.add(*it, s.tile_m, s.tile_n, 32, s.tile_steps, s.tile_steps);
            e.work += steps.work * s.step_us;
            e.longest = std::max(e.longest, steps.longest * s.chain_us);
        };
        add(x, hx.generic);
        add(w, hw.generic);
        // (two launches have to promise a tenth: the estimates are up to 8 us short of short launches)
        const double joint_us = kLaunch + Estimate::us(e.work / compute_units(), e.longest, 0.25);
        return 0.9 * joint_us <= hx.generic_us + hw.split_us ? joint : apart;
    }
    if (hw.split_us == HUGE_VAL) return apart;
    std::vector<const Planned*> both = x;
    both.insert(both.end(), w.begin(), w.end());
    double joint_us = 0;
    const int shape = route >= kRouteSplit ? hx.split : pick_split_shape(both, &joint_us);
    return w_split || joint_us <= hx.split_us + hw.generic_us ? ChoiceF32{shape, shape, true} : apart;
}
std::vector<const Planned*> pointers(const std::vector<Planned>& v) {
    std::vector<const Planned*> p;
    p.reserve(v.size());
    for (const Planned& it : v) p.push_back(&it);
    return p;
}

// fp32: the input gradients `x` and the weight gradients `w` in one launch, in the tiles that `choice` gives them - every sum is what it
// would have been in a launch of each half.  *done: false if there are too many tiles.
hipError_t launch_both(tf_ctx* ctx, hipStream_t stream, const std::vector<Planned>& x, const std::vector<Planned>& w, bool accumulate, const ChoiceF32& choice, bool* done) {
    *done = false;
    const bool split = choice.x >= kFirstSplit;
    // longest contraction first
    struct Item { const Planned* it; bool tn; };
    std::vector<Item> items;
    items.reserve(x.size() + w.size());
    for (const Planned& it : x) items.push_back(Item{&it, false});
    for (const Planned& it : w) items.push_back(Item{&it, true});
    std::stable_sort(items.begin(), items.end(), [](const Item& a, const Item& b) { return a.it->Kc > b.it->Kc; });
    const int64_t max_tiles = split ? kMaxSplitTiles : kMaxGenericTiles;
    GemmBatch batch;
    batch.tn = 0;
    int64_t tiles = 0;
    for (size_t i = 0; i < items.size(); ++i) {
        fill(batch.p[i], *items[i].it, std::min(tiles, max_tiles), 1);
        if (items[i].tn) batch.tn |= uint64_t(1) << i;
        uint32_t tile_m, tile_n;
        tile_of(items[i].tn ? choice.w : choice.x, Dtype::F32, &tile_m, &tile_n);
        tiles += tiles_of(*items[i].it, tile_m, tile_n);
    }
    if (tiles > max_tiles) return hipSuccess;
    batch.total_tiles = int32_t(tiles);
    batch.add = accumulate ? batch.tn : 0;
    *done = true;
    ctx->common_tiles.store(split ? kGenericShapes * kGenericShapes + choice.x - kFirstSplit : kGenericShapes * choice.x + choice.w, std::memory_order_relaxed);
    return split ? launch_gemm_split(stream, batch, int(items.size()), choice.x - kFirstSplit)
                 : launch_gemm_generic_both(stream, batch, int(items.size()), choice.x, choice.w, accumulate);
}

// Launch `items` in batches of at most kMaxProblemsPerLaunch, each on the kernel that find_routes() gives it; fp32 ones in launch shape
// f32_shape, or in one chosen for them alone (-1).
hipError_t launch_planned(tf_ctx* ctx, hipStream_t stream, std::vector<Planned>& items, Layout layout,
                          Dtype in_dtype, Dtype out_dtype, bool accumulate, int f32_shape = -1) {
    Routes routes;
    const hipError_t found = find_routes(items, layout, in_dtype, out_dtype, accumulate, ctx->gemm_route, routes);
    if (found != hipSuccess) return found;
    if (in_dtype == Dtype::F32 && !items.empty()) {
        if (f32_shape < 0) {
            const std::vector<const Planned*> v = pointers(items), none;
            f32_shape = layout == Layout::kNT ? choose_f32(v, none, ctx->gemm_route).x : choose_f32(none, v, ctx->gemm_route).w;
        }
        routes.shape[kOther] = f32_shape;
    }
    std::vector<const Planned*>* const cls = routes.cls;
    const int* const shape = routes.shape;

    GemmBatch batch;
    for (int c = 0; c < kClasses; ++c) {
        std::vector<const Planned*>& v = cls[c];
        // Longest contraction first: the tail of a launch is then made of the cheapest tiles.
        std::stable_sort(v.begin(), v.end(), [](const Planned* a, const Planned* b) { return a->total_kc() > b->total_kc(); });
        uint32_t tile_m, tile_n;
        tile_of(shape[c], in_dtype, &tile_m, &tile_n);
        const int64_t max_tiles = shape[c] < 0 ? kMaxTiles256 : shape[c] >= kFirstSplit ? kMaxSplitTiles : shape[c] >= kGenericShapes ? kMaxNarrowTiles : kMaxGenericTiles;
        size_t i = 0;
        while (i < v.size()) {
            int n = 0;
            int64_t tiles = 0;
            while (i < v.size()) {
                const Planned& it = *v[i];
                const int slots = 1 + int(it.more.size());
                if (slots > kMaxProblemsPerLaunch) return hipErrorInvalidValue;
                if (n + slots > kMaxProblemsPerLaunch) break;
                const int64_t nt = tiles_of(it, tile_m, tile_n);
                if (nt > max_tiles) return hipErrorInvalidValue;
                if (n > 0 && tiles + nt > max_tiles) break;
                fill(batch.p[n], it, tiles, slots);
                tiles += nt;
                ++n;
                for (const Planned& q : it.more) { fill(batch.p[n], q, tiles, 1); ++n; }     // own no tiles
                ++i;
            }
            batch.total_tiles = int32_t(tiles);
            batch.tn = layout == Layout::kTN ? ~0ull : 0;
            batch.add = accumulate ? ~0ull : 0;
            const int kind = (layout == Layout::kNT ? TF_KERNEL_DX_MFMA : TF_KERNEL_DW_MFMA) + (shape[c] < 0 ? 0 : 2);     // the kernel that runs
            ProfScope prof(ctx, stream, kind);
            const hipError_t e = shape[c] < 0
                ? launch_gemm_mfma_bf16(stream, batch, n, layout, out_dtype, accumulate, c == kTail)
                : shape[c] >= kFirstSplit
                ? launch_gemm_split(stream, batch, n, shape[c] - kFirstSplit)
                : shape[c] >= kFirstShort
                ? launch_gemm_short(stream, batch, n, shape[c] - kFirstShort, out_dtype, accumulate)
                : shape[c] >= kGenericShapes
                ? launch_gemm_narrow(stream, batch, n, shape[c] - kGenericShapes)
                : launch_gemm_generic(stream, batch, n, shape[c], layout, in_dtype, out_dtype, accumulate);
            if (e != hipSuccess) return e;
        }
    }
    return hipSuccess;
}

// Byte ranges of a stage backward's tensors: an output may overlap neither an input nor
// another output (inputs may overlap each other).  Sweep over the ranges sorted by start.
struct ByteRange { uintptr_t lo, hi; bool output; };
bool outputs_overlap_something(std::vector<ByteRange>& r) {
    std::sort(r.begin(), r.end(), [](const ByteRange& a, const ByteRange& b) { return a.lo < b.lo; });
    uintptr_t end_any = 0, end_out = 0;          // furthest end among the ranges seen so far: all / outputs
    for (const ByteRange& x : r) {
        if (x.output ? x.lo < end_any : x.lo < end_out) return true;
        end_any = std::max(end_any, x.hi);
        if (x.output) end_out = std::max(end_out, x.hi);
    }
    return false;
}

// Later calls may come from another thread, or after the caller made another device current.
inline bool use_device(tf_ctx* ctx) {
    const hipError_t e = hipSetDevice(ctx->device_id);
    if (e != hipSuccess) { ctx->last_hip_error = static_cast<int>(e); return false; }
    return true;
}

int validate_elementwise_common(int32_t n_tensors, const int64_t* numel,
                                void* const* ema, void* const* ema_abs,
                                const uint8_t* tensor_freeze_mask,
                                const uint32_t* const* elem_freeze_bits,
                                const double* score_sums, float ema_decay, bool ema_required) {
    if (n_tensors < 0) return TF_ERR_INVALID_ARG;
    if (n_tensors == 0) return TF_OK;
    if (!numel) return TF_ERR_INVALID_ARG;
    if ((ema == nullptr) != (ema_abs == nullptr)) return TF_ERR_INVALID_ARG;
    if (ema_required && !ema) return TF_ERR_INVALID_ARG;
    if (score_sums && !ema) return TF_ERR_INVALID_ARG;
    if (ema && !(ema_decay >= 0.f && ema_decay <= 1.f)) return TF_ERR_INVALID_ARG;
    if (score_sums && (reinterpret_cast<uintptr_t>(score_sums) & 7u)) return TF_ERR_ALIGN;
    for (int32_t i = 0; i < n_tensors; ++i) {
        if (numel[i] <= 0) return TF_ERR_SHAPE;
        if (numel[i] > (int64_t(1) << 37)) return TF_ERR_SHAPE;      // 2^29 blocks of 256 elements per launch
        if (tensor_freeze_mask && tensor_freeze_mask[i] > 1) return TF_ERR_INVALID_ARG;
        if (tensor_freeze_mask && tensor_freeze_mask[i]) continue;
        if (ema) {
            if (!ema[i] || !ema_abs[i]) return TF_ERR_INVALID_ARG;
            if (!aligned16(ema[i]) || !aligned16(ema_abs[i])) return TF_ERR_ALIGN;
        }
        if (elem_freeze_bits && elem_freeze_bits[i] && !aligned16(elem_freeze_bits[i])) return TF_ERR_ALIGN;
    }
    return TF_OK;
}

// The stage backward behind every entry point.  `accumulate_mask`, when given, says layer by
// layer whether the weight gradient is added to dW_l (1) or overwrites it (0) and replaces
// `accumulate`.
int stage_backward_impl(tf_ctx* ctx, void* hip_stream,
                        int32_t n_layers, const tf_shape* shapes,
                        int64_t T, tf_dtype io_dtype,
                        const void* const* W, const void* const* X, const void* const* dY,
                        const uint8_t* freeze_mask,
                        const uint8_t* const* row_block_mask, int32_t block_rows,
                        const int32_t* input_group,
                        void* const* dX,
                        void* const* dW, tf_dtype dw_dtype,
                        int accumulate, const uint8_t* accumulate_mask) {
    // ---- validation: no HIP call before this block has passed ----
    if (n_layers < 0) return TF_ERR_INVALID_ARG;
    if (!valid_dtype(io_dtype) || !valid_dtype(dw_dtype)) return TF_ERR_DTYPE;
    if (accumulate != 0 && accumulate != 1) return TF_ERR_INVALID_ARG;
    if (accumulate_mask) {
        accumulate = 0;
        for (int32_t l = 0; l < n_layers; ++l) {
            if (accumulate_mask[l] > 1) return TF_ERR_INVALID_ARG;
            if (accumulate_mask[l] && !(freeze_mask && freeze_mask[l] == 1)) accumulate = 1;
        }
    }
    if (accumulate && dw_dtype != TF_F32) return TF_ERR_DTYPE;
    if (io_dtype == TF_F32 && dw_dtype != TF_F32) return TF_ERR_DTYPE;
    if (row_block_mask && block_rows <= 0) return TF_ERR_INVALID_ARG;
    if (n_layers > 0) {
        if (!shapes || !W || !dY || !dX) return TF_ERR_INVALID_ARG;
        if (T <= 0 || T > 0x7fffffff) return TF_ERR_SHAPE;
        bool any_unfrozen = false;
        for (int32_t l = 0; l < n_layers; ++l) {
            if (shapes[l].K <= 0 || shapes[l].N <= 0) return TF_ERR_SHAPE;
            if (shapes[l].K > 0x7fffffff || shapes[l].N > 0x7fffffff) return TF_ERR_SHAPE;
            if (freeze_mask && freeze_mask[l] > 1) return TF_ERR_INVALID_ARG;
            if (!W[l] || !dY[l] || !dX[l]) return TF_ERR_INVALID_ARG;
            if (!aligned16(W[l]) || !aligned16(dY[l]) || !aligned16(dX[l])) return TF_ERR_ALIGN;
            if (!(freeze_mask && freeze_mask[l])) any_unfrozen = true;
        }
        if (any_unfrozen && (!X || !dW)) return TF_ERR_INVALID_ARG;
        if (input_group) {
            // members of a group share their input: same K, same dX buffer; the first member leads
            for (int32_t l = 0; l < n_layers; ++l) {
                const int32_t g = input_group[l];
                if (g < -1 || g >= n_layers) return TF_ERR_INVALID_ARG;
                if (g < 0) continue;
                int32_t lead = l;
                for (int32_t q = 0; q < l; ++q) if (input_group[q] == g) { lead = q; break; }
                if (shapes[lead].K != shapes[l].K) return TF_ERR_SHAPE;
                if (dX[lead] != dX[l]) return TF_ERR_INVALID_ARG;
            }
        }
        for (int32_t l = 0; l < n_layers; ++l) {
            if (freeze_mask && freeze_mask[l]) continue;
            if (!X[l] || !dW[l]) return TF_ERR_INVALID_ARG;
            if (!aligned16(X[l]) || !aligned16(dW[l])) return TF_ERR_ALIGN;
            if (row_block_mask && row_block_mask[l]) {
                if (shapes[l].K % block_rows != 0) return TF_ERR_SHAPE;
                for (int64_t b = 0; b < shapes[l].K / block_rows; ++b)
                    if (row_block_mask[l][b] > 1) return TF_ERR_INVALID_ARG;
            }
        }
    }
    const int64_t in_size = io_dtype == TF_BF16 ? 2 : 4, dw_size = dw_dtype == TF_BF16 ? 2 : 4;
    if (n_layers > 0) {
        // no output may overlap an input or another output (the members of an input group pass
        // one dX buffer: it is listed once, for the member that leads the group)
        std::vector<ByteRange> ranges;
        ranges.reserve(size_t(n_layers) * 5);
        auto add = [&](const void* p, int64_t elems, int64_t size, bool output) {
            const uintptr_t lo = reinterpret_cast<uintptr_t>(p);
            ranges.push_back(ByteRange{lo, lo + uintptr_t(elems) * uintptr_t(size), output});
        };
        std::vector<uint8_t> group_seen(input_group ? n_layers : 0, 0);
        for (int32_t l = 0; l < n_layers; ++l) {
            const int64_t K = shapes[l].K, N = shapes[l].N;
            add(W[l], K * N, in_size, false);
            add(dY[l], T * N, in_size, false);
            const int32_t g = input_group ? input_group[l] : -1;
            if (g < 0 || !group_seen[g]) add(dX[l], T * K, in_size, true);
            if (g >= 0) group_seen[g] = 1;
            if (freeze_mask && freeze_mask[l]) continue;
            add(X[l], T * K, in_size, false);
            add(dW[l], K * N, dw_size, true);
        }
        if (outputs_overlap_something(ranges)) return TF_ERR_ALIAS;
    }
    if (!ctx) return TF_ERR_INVALID_ARG;
    if (n_layers == 0) return TF_OK;
    if (!use_device(ctx)) return TF_ERR_HIP;

    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const Dtype in_dt = to_dtype(io_dtype);

    // input gradients: every layer, whatever the masks say.  Layers that share their input are
    // segments of one problem: their products are summed in the accumulators and rounded once.
    std::vector<Planned> plan;
    plan.reserve(n_layers);
    bool grouped_slow = false;
    {
        std::vector<int32_t> lead_slot(n_layers, -1);          // group id -> index in plan
        for (int32_t l = 0; l < n_layers; ++l) {
            Planned it{dY[l], W[l], dX[l], T, shapes[l].K, shapes[l].N, shapes[l].N, shapes[l].N, ~0ull, {}};
            const int32_t g = input_group ? input_group[l] : -1;
            if (g >= 0 && lead_slot[g] >= 0) plan[lead_slot[g]].more.push_back(it);
            else { if (g >= 0) lead_slot[g] = int32_t(plan.size()); plan.push_back(it); }
        }
        for (const Planned& it : plan) {
            if (it.more.empty()) continue;
            bool ok = planned_mfma_ok(it, Layout::kNT, in_dt);
            for (const Planned& q : it.more) ok = ok && planned_mfma_ok(q, Layout::kNT, in_dt);
            if (!ok) grouped_slow = true;
        }
    }
    // weight gradients: what is frozen - a layer, or a block of rows of one - is simply not
    // in the plan.
    // Layers whose gradient is added to what dW_l holds and layers whose gradient overwrites it
    // are two plans (two kernels: the adding one fetches the old values).
    std::vector<Planned> plan_set, plan_add;
    for (int32_t l = 0; l < n_layers; ++l) {
        if (freeze_mask && freeze_mask[l]) continue;
        const bool add = accumulate_mask ? accumulate_mask[l] != 0 : accumulate != 0;
        std::vector<Planned>& dst = add ? plan_add : plan_set;
        const int64_t K = shapes[l].K, N = shapes[l].N;
        const uint8_t* rm = row_block_mask ? row_block_mask[l] : nullptr;
        if (!rm) {
            dst.push_back(Planned{X[l], dY[l], dW[l], K, N, T, K, N, ~0ull, {}});
            continue;
        }
        const int64_t nb = K / block_rows;
        // Matrix-core path: one problem per tensor whose tile rows are the unfrozen 256-row
        // blocks (a bit per block), so that any pattern of frozen blocks costs one problem.
        const int64_t tile = gemm_mfma_tile();
        if (in_dt == Dtype::BF16 && block_rows % tile == 0 && K / tile <= 64 &&
            mfma_shape_ok(Layout::kTN, tile, N, T, K, N) && aligned16(X[l]) && aligned16(dY[l]) && aligned16(dW[l])) {
            uint64_t bits = 0;
            int64_t rows = 0;
            const int64_t per = block_rows / tile;
            for (int64_t b = 0; b < nb; ++b)
                if (!rm[b])
                    for (int64_t q = 0; q < per; ++q) { bits |= 1ull << (b * per + q); rows += tile; }
            if (rows > 0) dst.push_back(Planned{X[l], dY[l], dW[l], rows, N, T, K, N, rows == K ? ~0ull : bits, {}});
            continue;
        }
        // Otherwise each run of unfrozen row blocks is one problem: columns [k0, k1) of X
        // (pitch K_l) against dY give rows [k0, k1) of dW.
        for (int64_t b = 0; b < nb;) {
            if (rm[b]) { ++b; continue; }
            int64_t e1 = b;
            while (e1 < nb && !rm[e1]) ++e1;
            const int64_t k0 = b * block_rows, rows = (e1 - b) * block_rows;
            Planned run{static_cast<const char*>(X[l]) + k0 * in_size, dY[l],
                        static_cast<char*>(dW[l]) + k0 * N * dw_size, rows, N, T, K, N, ~0ull, {}};
            run.rows_before = k0;                    // columns of X on either side of the run's own
            run.rows_after = K - k0 - rows;
            dst.push_back(run);
            b = e1;
        }
    }
    hipError_t e = hipSuccess;
    bool both = false;
    const bool add_first = plan_set.empty();          // (what overwrites, if there is any, goes with the input gradients)
    ctx->common_tiles.store(-1, std::memory_order_relaxed);
    ChoiceF32 choice{-1, -1, false};
    std::vector<Planned>& first = add_first ? plan_add : plan_set;
    if (in_dt == Dtype::F32 && !input_group) {
        choice = choose_f32(pointers(plan), pointers(first), ctx->gemm_route);
        if (choice.together && !ctx->profiling) {         // (a call whose kernels are timed launches them one by one)
            e = launch_both(ctx, stream, plan, first, add_first, choice, &both);
            if (e != hipSuccess) return hip_fail(ctx, e);
        }
        if (both) first.clear();
    }
    if (both) {
    } else if (!grouped_slow) {
        e = launch_planned(ctx, stream, plan, Layout::kNT, in_dt, in_dt, false, choice.x);
    } else {
        // A group that the matrix-core kernel cannot take: member after member, each launch adding
        // onto the one before.  That needs an fp32 output (the fp32 configuration).
        if (in_dt != Dtype::F32) return TF_ERR_SHAPE;
        size_t depth = 0;
        for (const Planned& it : plan) depth = std::max(depth, it.more.size());
        for (size_t k = 0; k <= depth && e == hipSuccess; ++k) {
            std::vector<Planned> round;
            for (const Planned& it : plan) {
                if (k == 0) { Planned h = it; h.more.clear(); round.push_back(h); }
                else if (k <= it.more.size()) round.push_back(it.more[k - 1]);
            }
            e = launch_planned(ctx, stream, round, Layout::kNT, in_dt, in_dt, k > 0);
        }
    }
    if (e != hipSuccess) return hip_fail(ctx, e);

    e = launch_planned(ctx, stream, plan_set, Layout::kTN, in_dt, to_dtype(dw_dtype), false, add_first ? -1 : choice.w);
    if (e != hipSuccess) return hip_fail(ctx, e);
    e = launch_planned(ctx, stream, plan_add, Layout::kTN, in_dt, to_dtype(dw_dtype), true, add_first ? choice.w : -1);
    if (e != hipSuccess) return hip_fail(ctx, e);
    return TF_OK;
}


}  // namespace

extern "C" {

const char* tf_version(void) { return "0.1.0"; }

const char* tf_strerror(int code) {
    switch (code) {
        case TF_OK: return "ok";
        case TF_ERR_INVALID_ARG: return "invalid argument";
        case TF_ERR_SHAPE: return "invalid shape or size";
        case TF_ERR_DTYPE: return "unsupported dtype or dtype combination";
        case TF_ERR_ALIGN: return "device pointer is not 16-byte aligned";
        case TF_ERR_WORKSPACE: return "workspace allocation failed";
        case TF_ERR_HIP: return "HIP runtime error (see tf_last_hip_error)";
        case TF_ERR_NO_DEVICE: return "no usable gfx950 device";
        case TF_ERR_ALIAS: return "an output buffer overlaps an input or another output";
        default: return "unknown status code";
    }
}

int tf_create(tf_ctx** out, int device_id) {
    if (!out || device_id < 0) return TF_ERR_INVALID_ARG;
    *out = nullptr;
    int count = 0;
    if (hipGetDeviceCount(&count) != hipSuccess || device_id >= count) return TF_ERR_NO_DEVICE;
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, device_id) != hipSuccess) return TF_ERR_NO_DEVICE;
    if (std::strncmp(prop.gcnArchName, "gfx950", 6) != 0) return TF_ERR_NO_DEVICE;
    if (hipSetDevice(device_id) != hipSuccess) return TF_ERR_NO_DEVICE;
    tf_ctx* ctx = new (std::nothrow) tf_ctx;
    if (!ctx) return TF_ERR_WORKSPACE;
    ctx->device_id = device_id;
    ctx->last_hip_error = 0;
    ctx->profiling = false;
    ctx->rc_state = nullptr;
    ctx->rc_state_static = nullptr;
    for (uint32_t*& undo : ctx->rc_undo) undo = nullptr;
    ctx->lowp_is_rounded_master = false;
    ctx->gemm_route = 0;
    ctx->ew_partials = nullptr;
    if (hipMalloc(reinterpret_cast<void**>(&ctx->rc_state), tf::rc_state_bytes()) != hipSuccess) {
        delete ctx;
        return TF_ERR_WORKSPACE;
    }
    void* st = nullptr;
    if (static_scratch_address(device_id, &st) != hipSuccess ||      // device_id is current here
        hipMalloc(reinterpret_cast<void**>(&ctx->ew_partials), tf::ew_partials_bytes()) != hipSuccess ||
        hipMemset(ctx->ew_partials, 0, tf::ew_partials_bytes()) != hipSuccess) {
        if (ctx->ew_partials) (void)hipFree(ctx->ew_partials);
        (void)hipFree(ctx->rc_state);
        delete ctx;
        return TF_ERR_WORKSPACE;
    }
    ctx->rc_state_static = static_cast<tf::RcState*>(st);
    *out = ctx;
    return TF_OK;
}

int tf_destroy(tf_ctx* ctx) {
    if (!ctx) return TF_ERR_INVALID_ARG;
    for (tf_prof_rec& r : ctx->recs) { (void)hipEventDestroy(r.start); (void)hipEventDestroy(r.stop); }
    for (hipEvent_t e : ctx->pool) (void)hipEventDestroy(e);
    if (ctx->rc_state) (void)hipFree(ctx->rc_state);
    for (uint32_t* undo : ctx->rc_undo)
        if (undo) (void)hipFree(undo);
    if (ctx->ew_partials) (void)hipFree(ctx->ew_partials);
    delete ctx;
    return TF_OK;
}

int tf_assume_lowp_is_rounded_master(tf_ctx* ctx, int on) {
    if (!ctx || (on != 0 && on != 1)) return TF_ERR_INVALID_ARG;
    ctx->lowp_is_rounded_master = on != 0;
    return TF_OK;
}

int tf_profile_enable(tf_ctx* ctx, int enable) {
    if (!ctx || (enable != 0 && enable != 1)) return TF_ERR_INVALID_ARG;
    ctx->profiling = enable != 0;
    return TF_OK;
}

int tf_profile_collect(tf_ctx* ctx, int32_t capacity, int32_t* kinds, float* ms, int32_t* n_out) {
    if (!ctx || !n_out || capacity < 0 || (capacity > 0 && (!kinds || !ms))) return TF_ERR_INVALID_ARG;
    int32_t n = 0;
    int rc = TF_OK;
    for (tf_prof_rec& r : ctx->recs) {
        if (n < capacity && rc == TF_OK) {
            hipError_t e = hipEventSynchronize(r.stop);
            float t = 0.f;
            if (e == hipSuccess) e = hipEventElapsedTime(&t, r.start, r.stop);
            if (e != hipSuccess) rc = hip_fail(ctx, e);
            else { kinds[n] = r.kind; ms[n] = t; ++n; }
        }
        ctx->pool.push_back(r.start);
        ctx->pool.push_back(r.stop);
    }
    ctx->recs.clear();
    *n_out = n;
    return rc;
}

int tf_last_hip_error(const tf_ctx* ctx) { return ctx ? ctx->last_hip_error : 0; }

int tf_stage_backward_shared(tf_ctx* ctx, void* hip_stream,
                             int32_t n_layers, const tf_shape* shapes,
                             int64_t T, tf_dtype io_dtype,
                             const void* const* W, const void* const* X, const void* const* dY,
                             const uint8_t* freeze_mask,
                             const uint8_t* const* row_block_mask, int32_t block_rows,
                             const int32_t* input_group,
                             void* const* dX,
                             void* const* dW, tf_dtype dw_dtype,
                             int accumulate) {
    return stage_backward_impl(ctx, hip_stream, n_layers, shapes, T, io_dtype, W, X, dY, freeze_mask,
                               row_block_mask, block_rows, input_group, dX, dW, dw_dtype, accumulate, nullptr);
}

int tf_stage_backward_microbatch(tf_ctx* ctx, void* hip_stream,
                                 int32_t n_layers, const tf_shape* shapes,
                                 int64_t T, tf_dtype io_dtype,
                                 const void* const* W, const void* const* X, const void* const* dY,
                                 const uint8_t* freeze_mask,
                                 void* const* dX,
                                 void* const* dW, tf_dtype dw_dtype,
                                 const uint8_t* accumulate_mask) {
    if (n_layers > 0 && !accumulate_mask) return TF_ERR_INVALID_ARG;
    return stage_backward_impl(ctx, hip_stream, n_layers, shapes, T, io_dtype, W, X, dY, freeze_mask,
                               nullptr, 0, nullptr, dX, dW, dw_dtype, 0, accumulate_mask);
}

int tf_stage_backward(tf_ctx* ctx, void* hip_stream,
                      int32_t n_layers, const tf_shape* shapes,
                      int64_t T, tf_dtype io_dtype,
                      const void* const* W, const void* const* X, const void* const* dY,
                      const uint8_t* freeze_mask,
                      void* const* dX,
                      void* const* dW, tf_dtype dw_dtype,
                      int accumulate) {
    return tf_stage_backward_shared(ctx, hip_stream, n_layers, shapes, T, io_dtype, W, X, dY, freeze_mask,
                                    nullptr, 0, nullptr, dX, dW, dw_dtype, accumulate);
}

int tf_stage_backward_blocks(tf_ctx* ctx, void* hip_stream,
                             int32_t n_layers, const tf_shape* shapes,
                             int64_t T, tf_dtype io_dtype,
                             const void* const* W, const void* const* X, const void* const* dY,
                             const uint8_t* freeze_mask,
                             const uint8_t* const* row_block_mask, int32_t block_rows,
                             void* const* dX,
                             void* const* dW, tf_dtype dw_dtype,
                             int accumulate) {
    return tf_stage_backward_shared(ctx, hip_stream, n_layers, shapes, T, io_dtype, W, X, dY, freeze_mask,
                                    row_block_mask, block_rows, nullptr, dX, dW, dw_dtype, accumulate);
}

int tf_masked_adamw(tf_ctx* ctx, void* hip_stream,
                    int32_t n_tensors, const int64_t* numel,
                    void* const* p_master, void* const* m, void* const* v,
                    const void* const* grad, tf_dtype grad_dtype, float grad_scale,
                    void* const* p_lowp,
                    const uint8_t* tensor_freeze_mask,
                    const uint32_t* const* elem_freeze_bits,
                    const int32_t* step,
                    float lr, float beta1, float beta2, float eps, float weight_decay,
                    void* const* ema, void* const* ema_abs, float ema_decay,
                    double* score_sums) {
    if (!valid_dtype(grad_dtype)) return TF_ERR_DTYPE;
    int rc = validate_elementwise_common(n_tensors, numel, ema, ema_abs, tensor_freeze_mask,
                                         elem_freeze_bits, score_sums, ema_decay, false);
    if (rc != TF_OK) return rc;
    if (n_tensors > 0) {
        if (!p_master || !m || !v || !grad || !step) return TF_ERR_INVALID_ARG;
        if (!(beta1 >= 0.f && beta1 < 1.f) || !(beta2 >= 0.f && beta2 < 1.f)) return TF_ERR_INVALID_ARG;
        if (!(eps >= 0.f) || !std::isfinite(lr) || !std::isfinite(weight_decay) || !std::isfinite(grad_scale))
            return TF_ERR_INVALID_ARG;
        for (int32_t i = 0; i < n_tensors; ++i) {
            if (tensor_freeze_mask && tensor_freeze_mask[i]) continue;
            if (step[i] < 1) return TF_ERR_INVALID_ARG;
            if (!p_master[i] || !m[i] || !v[i] || !grad[i]) return TF_ERR_INVALID_ARG;
            if (!aligned16(p_master[i]) || !aligned16(m[i]) || !aligned16(v[i]) || !aligned16(grad[i]))
                return TF_ERR_ALIGN;
            if (p_lowp && p_lowp[i] && !aligned16(p_lowp[i])) return TF_ERR_ALIGN;
        }
    }
    if (!ctx) return TF_ERR_INVALID_ARG;
    if (n_tensors == 0) return TF_OK;
    if (!use_device(ctx)) return TF_ERR_HIP;

    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    AdamwParams hp;
    hp.grad_scale = grad_scale;
    hp.lr = lr; hp.beta1 = beta1; hp.beta2 = beta2; hp.eps = eps; hp.weight_decay = weight_decay;
    hp.one_minus_beta1 = float(1.0 - double(beta1));
    hp.one_minus_beta2 = float(1.0 - double(beta2));
    hp.ema_decay = ema_decay;
    hp.one_minus_ema_decay = float(1.0 - double(ema_decay));

    const int64_t epb = ew_elems_per_block();
    EwBatch batch;
    batch.lowp_is_rounded_master = ctx->lowp_is_rounded_master ? 1 : 0;
    batch.pad_ = 0;
    batch.partials = ctx->ew_partials;
    int n = 0;
    int64_t blocks = 0;
    auto flush = [&]() -> hipError_t {
        batch.total_blocks = int32_t(blocks);
        ProfScope prof(ctx, stream, TF_KERNEL_ADAMW);
        const hipError_t e = launch_adamw(stream, batch, n, hp, to_dtype(grad_dtype));
        n = 0; blocks = 0;
        return e;
    };
    for (int32_t i = 0; i < n_tensors; ++i) {
        if (tensor_freeze_mask && tensor_freeze_mask[i]) continue;   // frozen: not even read
        const int64_t nb = (numel[i] + epb - 1) / epb;
        if (n == kMaxTensorsPerLaunch || (n > 0 && blocks + nb > 0x3fffffff)) {
            const hipError_t e = flush();
            if (e != hipSuccess) return hip_fail(ctx, e);
        }
        EwTensor& t = batch.t[n];
        t.p = static_cast<float*>(p_master[i]);
        t.m = static_cast<float*>(m[i]);
        t.v = static_cast<float*>(v[i]);
        t.g = grad[i];
        t.p_lowp = p_lowp ? static_cast<uint16_t*>(p_lowp[i]) : nullptr;
        t.bits = elem_freeze_bits ? elem_freeze_bits[i] : nullptr;
        t.E = ema ? static_cast<float*>(ema[i]) : nullptr;
        t.A = ema ? static_cast<float*>(ema_abs[i]) : nullptr;
        t.sums = score_sums ? score_sums + 2 * int64_t(i) : nullptr;
        t.numel = numel[i];
        t.rbc1 = float(1.0 / (1.0 - std::pow(double(beta1), double(step[i]))));
        t.rbc2 = float(1.0 / (1.0 - std::pow(double(beta2), double(step[i]))));
        batch.block_start[n] = int32_t(blocks);
        blocks += nb;
        ++n;
    }
    if (n > 0) {
        const hipError_t e = flush();
        if (e != hipSuccess) return hip_fail(ctx, e);
    }
    return TF_OK;
}

int tf_stability_update(tf_ctx* ctx, void* hip_stream,
                        int32_t n_tensors, const int64_t* numel,
                        const void* const* delta,
                        void* const* ema, void* const* ema_abs, float ema_decay,
                        const uint8_t* tensor_freeze_mask,
                        const uint32_t* const* elem_freeze_bits,
                        double* score_sums) {
    int rc = validate_elementwise_common(n_tensors, numel, ema, ema_abs, tensor_freeze_mask,
                                         elem_freeze_bits, score_sums, ema_decay, true);
    if (rc != TF_OK) return rc;
    if (n_tensors > 0) {
        if (!delta) return TF_ERR_INVALID_ARG;
        for (int32_t i = 0; i < n_tensors; ++i) {
            if (tensor_freeze_mask && tensor_freeze_mask[i]) continue;
            if (!delta[i]) return TF_ERR_INVALID_ARG;
            if (!aligned16(delta[i])) return TF_ERR_ALIGN;
        }
    }
    if (!ctx) return TF_ERR_INVALID_ARG;
    if (n_tensors == 0) return TF_OK;
    if (!use_device(ctx)) return TF_ERR_HIP;

    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    AdamwParams hp;
    std::memset(&hp, 0, sizeof(hp));
    hp.ema_decay = ema_decay;
    hp.one_minus_ema_decay = float(1.0 - double(ema_decay));

    const int64_t epb = ew_elems_per_block();
    EwBatch batch;
    batch.lowp_is_rounded_master = 0;
    batch.pad_ = 0;
    batch.partials = ctx->ew_partials;
    int n = 0;
    int64_t blocks = 0;
    auto flush = [&]() -> hipError_t {
        batch.total_blocks = int32_t(blocks);
        ProfScope prof(ctx, stream, TF_KERNEL_STABILITY);
        const hipError_t e = launch_stability(stream, batch, n, hp);
        n = 0; blocks = 0;
        return e;
    };
    for (int32_t i = 0; i < n_tensors; ++i) {
        if (tensor_freeze_mask && tensor_freeze_mask[i]) continue;
        const int64_t nb = (numel[i] + epb - 1) / epb;
        if (n == kMaxTensorsPerLaunch || (n > 0 && blocks + nb > 0x3fffffff)) {
            const hipError_t e = flush();
            if (e != hipSuccess) return hip_fail(ctx, e);
        }
        EwTensor& t = batch.t[n];
        std::memset(&t, 0, sizeof(t));
        t.g = delta[i];
        t.bits = elem_freeze_bits ? elem_freeze_bits[i] : nullptr;
        t.E = static_cast<float*>(ema[i]);
        t.A = static_cast<float*>(ema_abs[i]);
        t.sums = score_sums ? score_sums + 2 * int64_t(i) : nullptr;
        t.numel = numel[i];
        batch.block_start[n] = int32_t(blocks);
        blocks += nb;
        ++n;
    }
    if (n > 0) {
        const hipError_t e = flush();
        if (e != hipSuccess) return hip_fail(ctx, e);
    }
    return TF_OK;
}

int tf_stability_scores(const double* score_sums, int32_t n, double* scores) {
    if (n < 0 || (n > 0 && (!score_sums || !scores))) return TF_ERR_INVALID_ARG;
    for (int32_t i = 0; i < n; ++i) {
        const double se = score_sums[2 * i], sa = score_sums[2 * i + 1];
        scores[i] = (sa == 0.0) ? 1.0 : se / sa;
    }
    return TF_OK;
}

int tf_select_lowest(const double* scores, int32_t n, int32_t n_freeze, uint8_t* out_mask) {
    if (n < 0 || n_freeze < 0 || n_freeze > n) return TF_ERR_INVALID_ARG;
    if (n > 0 && (!scores || !out_mask)) return TF_ERR_INVALID_ARG;
    for (int32_t i = 0; i < n; ++i)
        if (std::isnan(scores[i])) return TF_ERR_INVALID_ARG;
    std::vector<int32_t> order(n);
    for (int32_t i = 0; i < n; ++i) order[i] = i;
    std::stable_sort(order.begin(), order.end(),
                     [&](int32_t a, int32_t b) { return scores[a] < scores[b]; });
    for (int32_t i = 0; i < n; ++i) out_mask[i] = 0;
    for (int32_t i = 0; i < n_freeze; ++i) out_mask[order[i]] = 1;
    return TF_OK;
}

int tf_microbatch_plan(int32_t n_microbatches, int32_t n_layers, const uint8_t* freeze_masks,
                       uint8_t* accumulate_masks, uint8_t* step_freeze_mask) {
    if (n_microbatches < 0 || n_layers < 0) return TF_ERR_INVALID_ARG;
    if (n_layers == 0) return TF_OK;
    if (!step_freeze_mask || (n_microbatches > 0 && (!freeze_masks || !accumulate_masks))) return TF_ERR_INVALID_ARG;
    for (int64_t i = 0; i < int64_t(n_microbatches) * n_layers; ++i)
        if (freeze_masks[i] > 1) return TF_ERR_INVALID_ARG;
    for (int32_t l = 0; l < n_layers; ++l) {
        uint8_t seen = 0;                       // unfrozen in an earlier microbatch
        for (int32_t m = 0; m < n_microbatches; ++m) {
            accumulate_masks[int64_t(m) * n_layers + l] = seen;
            if (!freeze_masks[int64_t(m) * n_layers + l]) seen = 1;
        }
        step_freeze_mask[l] = seen ? 0 : 1;
    }
    return TF_OK;
}

int32_t tf_num_frozen(double r, int32_t n) {
    if (n <= 0 || !(r > 0.0)) return 0;
    const double x = std::ceil(r * double(n) - 1e-9);
    if (x >= double(n)) return n;
    return x < 0.0 ? 0 : int32_t(x);
}

int tf_autofreeze_norms(tf_ctx* ctx, void* hip_stream,
                        int32_t n_tensors, const int64_t* numel,
                        const void* const* p_master, void* const* snapshot,
                        const uint8_t* tensor_freeze_mask, int update_snapshot,
                        double* sq_norms) {
    if (n_tensors < 0 || (update_snapshot != 0 && update_snapshot != 1)) return TF_ERR_INVALID_ARG;
    if (n_tensors > 0) {
        if (!numel || !p_master || !snapshot || !sq_norms) return TF_ERR_INVALID_ARG;
        if (reinterpret_cast<uintptr_t>(sq_norms) & 7u) return TF_ERR_ALIGN;
        for (int32_t i = 0; i < n_tensors; ++i) {
            if (numel[i] <= 0 || numel[i] > (int64_t(1) << 40)) return TF_ERR_SHAPE;
            if (tensor_freeze_mask && tensor_freeze_mask[i] > 1) return TF_ERR_INVALID_ARG;
            if (tensor_freeze_mask && tensor_freeze_mask[i]) continue;
            if (!p_master[i] || !snapshot[i]) return TF_ERR_INVALID_ARG;
            if (!aligned16(p_master[i]) || !aligned16(snapshot[i])) return TF_ERR_ALIGN;
        }
    }
    if (!ctx) return TF_ERR_INVALID_ARG;
    if (n_tensors == 0) return TF_OK;
    if (!use_device(ctx)) return TF_ERR_HIP;

    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const int64_t epb = norm_elems_per_block();
    NormBatch batch;
    batch.partials = ctx->ew_partials;
    int n = 0;
    int64_t blocks = 0;
    auto flush = [&]() -> hipError_t {
        if (n == 0) return hipSuccess;
        batch.total_blocks = int32_t(blocks);
        ProfScope prof(ctx, stream, TF_KERNEL_AUTOFREEZE);
        const hipError_t e = launch_autofreeze_norms(stream, batch, n, update_snapshot != 0);
        n = 0; blocks = 0;
        return e;
    };
    for (int32_t i = 0; i < n_tensors; ++i) {
        if (tensor_freeze_mask && tensor_freeze_mask[i]) continue;
        const int64_t nb = (numel[i] + epb - 1) / epb;
        if (n == kMaxTensorsPerLaunch || blocks + nb > 0x3fffffff) {
            const hipError_t e = flush();
            if (e != hipSuccess) return hip_fail(ctx, e);
        }
        NormTensor& t = batch.t[n];
        t.p = static_cast<const float*>(p_master[i]);
        t.snap = static_cast<float*>(snapshot[i]);
        t.out = sq_norms + i;
        t.numel = numel[i];
        t.block_start = int32_t(blocks);
        t.pad_ = 0;
        blocks += nb;
        ++n;
    }
    const hipError_t e = flush();
    if (e != hipSuccess) return hip_fail(ctx, e);
    return TF_OK;
}

int tf_autofreeze_scores(const double* sq_prev, const double* sq_cur, int32_t n, double* scores) {
    if (n < 0 || (n > 0 && (!sq_prev || !sq_cur || !scores))) return TF_ERR_INVALID_ARG;
    for (int32_t i = 0; i < n; ++i)
        if (!(sq_prev[i] >= 0.0) || !(sq_cur[i] >= 0.0)) return TF_ERR_INVALID_ARG;
    for (int32_t i = 0; i < n; ++i) {
        const double a = std::sqrt(sq_prev[i]), b = std::sqrt(sq_cur[i]);
        if (a == 0.0) scores[i] = b == 0.0 ? 0.0 : INFINITY;
        else scores[i] = std::fabs(a - b) / a;
    }
    return TF_OK;
}

int tf_autofreeze_select(const double* scores, int32_t n, int32_t n_already_frozen,
                         double percentile, uint8_t* out_mask) {
    if (n < 0 || n_already_frozen < 0 || n_already_frozen > n) return TF_ERR_INVALID_ARG;
    if (!(percentile >= 0.0 && percentile <= 100.0)) return TF_ERR_INVALID_ARG;
    if (n > 0 && (!scores || !out_mask)) return TF_ERR_INVALID_ARG;
    for (int32_t i = 0; i < n; ++i)
        if (std::isnan(scores[i])) return TF_ERR_INVALID_ARG;
    for (int32_t i = 0; i < n; ++i) out_mask[i] = i < n_already_frozen ? 1 : 0;
    const int32_t n_active = n - n_already_frozen;
    if (n_active == 0) return TF_OK;
    std::vector<double> active(scores + n_already_frozen, scores + n);
    std::sort(active.begin(), active.end());
    const int32_t rank = int32_t(std::ceil(percentile / 100.0 * double(n_active) - 1e-9));
    if (rank <= 0) return TF_OK;
    const double tau = active[std::min(rank, n_active) - 1];
    for (int32_t l = n_already_frozen; l < n && scores[l] <= tau; ++l) out_mask[l] = 1;
    return TF_OK;
}

// Validation shared by the two reconciliation entry points (no HIP call).
static int validate_reconcile(int32_t n_tensors, const int64_t* numel, uint32_t* const* elem_bits,
                              int64_t n_freeze, const int64_t* stats) {
    if (n_tensors < 0 || n_freeze < 0) return TF_ERR_INVALID_ARG;
    if (n_tensors > 0 && (!numel || !elem_bits)) return TF_ERR_INVALID_ARG;
    if (stats && (reinterpret_cast<uintptr_t>(stats) & 7u)) return TF_ERR_ALIGN;
    int64_t total = 0;
    for (int32_t i = 0; i < n_tensors; ++i) {
        if (numel[i] <= 0) return TF_ERR_SHAPE;
        total += numel[i];
        if (total >= (int64_t(1) << 32)) return TF_ERR_SHAPE;
        if (!elem_bits[i]) return TF_ERR_INVALID_ARG;
        if (reinterpret_cast<uintptr_t>(elem_bits[i]) & 3u) return TF_ERR_ALIGN;
    }
    if (n_freeze > total) return TF_ERR_INVALID_ARG;
    return TF_OK;
}

// Masks of this many elements guess their threshold (rc_try_kernel()).  Both ways timed, us, 30 % -> 50 %: 61e6 elements
// 122 (general passes 138), 122e6 151 (189), 218e6 193 (263), 436e6 270 (428), 1.74e9 771 (1475).  Where the window would be
// too wide the launches that go with a guess cost 20 us for nothing: from 2^28 elements on that takes fewer than 15 %
// candidates, half of them to be drawn.
constexpr int64_t kGuessFrom = int64_t(1) << 28;

// Room for a copy of the mask, for a reconciliation that guesses its threshold, or null where it does not: masks too
// small for it, or of so many small tensors that their words are far more than their elements; streams that are being captured; no memory
// left.  What a context has once taken it keeps, a larger mask's copy beside a smaller one's: to free one would wait for the device.
static uint32_t* reconcile_undo(tf_ctx* ctx, hipStream_t stream, int32_t n_tensors, const int64_t* numel) {
    int64_t elements = 0, words = 0;
    for (int32_t i = 0; i < n_tensors; ++i) { elements += numel[i]; words += (numel[i] + 31) / 32; }
    if (elements < kGuessFrom) return nullptr;
    int size = 0;
    while (size < kUndoSizes && words > undo_words(size)) ++size;
    if (size == kUndoSizes) return nullptr;
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &status) != hipSuccess || status != hipStreamCaptureStatusNone) {
        (void)hipGetLastError();
        return nullptr;
    }
    uint32_t*& undo = ctx->rc_undo[size];
    if (!undo) {
        // another thread's capture has to live through an allocation here
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        const bool exchanged = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
        if (hipMalloc(reinterpret_cast<void**>(&undo), size_t(undo_words(size)) * 4) != hipSuccess) undo = nullptr;
        if (exchanged) (void)hipThreadExchangeStreamCaptureMode(&mode);
        (void)hipGetLastError();
    }
    return undo;
}

// The passes of the reconciliation on the state `st`.  Allocates nothing, on the host or on the
// device: the tensor descriptors of a launch are built on the stack, pass after pass.
static hipError_t reconcile_passes(hipStream_t stream, int32_t n_tensors, const int64_t* numel,
                                   uint32_t* const* elem_bits, int64_t n_freeze, uint64_t seed,
                                   int64_t* stats, RcState* st, uint32_t* undo) {
    const RcKeys keys = perm32_keys(seed);
    int64_t total = 0;
    for (int32_t i = 0; i < n_tensors; ++i) total += numel[i];
    // calls fn(batch) for every launch-sized group of tensors, in order
    auto for_each_batch = [&](auto&& fn) -> hipError_t {
        RcBatch b;
        b.n_tensors = 0; b.total_blocks = 0;
        int64_t goff = 0, blocks = 0, words = 0;
        for (int32_t i = 0; i < n_tensors; ++i) {
            const int nb = rc_tasks(numel[i]);
            if (b.n_tensors == kMaxRcTensors) {
                b.total_blocks = int32_t(blocks);
                const hipError_t e = fn(b);
                if (e != hipSuccess) return e;
                b.n_tensors = 0; blocks = 0;
            }
            RcTensor& t = b.t[b.n_tensors++];
            t.bits = elem_bits[i]; t.numel = numel[i]; t.goff = goff;
            t.block_start = int32_t(blocks); t.pad_ = 0;
            t.undo = undo ? undo + words : nullptr;
            blocks += nb;
            goff += numel[i];
            words += (numel[i] + 31) / 32;
        }
        if (b.n_tensors > 0) { b.total_blocks = int32_t(blocks); return fn(b); }
        return hipSuccess;
    };
    hipError_t e = launch_rc_begin(stream, st);               // a kernel clears the state: nothing survives from the call before
    if (e == hipSuccess) e = for_each_batch([&](RcBatch& b) { return launch_rc_count(stream, b, st); });
    if (e == hipSuccess) e = launch_rc_decide(stream, st, uint64_t(n_freeze), undo ? uint64_t(total) : 0, stats);
    if (undo) {
        if (e == hipSuccess) e = for_each_batch([&](RcBatch& b) { return launch_rc_probe(stream, b, st, keys); });
        if (e == hipSuccess) e = for_each_batch([&](RcBatch& b) { return launch_rc_try(stream, b, st, keys); });
        for (int level = 0; level < 3; ++level) {
            if (e == hipSuccess) e = for_each_batch([&](RcBatch& b) { return launch_rc_window(stream, b, st, keys, level); });
            if (e == hipSuccess && level < 2) e = launch_rc_window_pick(stream, st, level, stats);
        }
        if (e == hipSuccess) e = for_each_batch([&](RcBatch& b) { return launch_rc_restore(stream, b, st); });
    }
    const int open[3] = {32, 21, 10}, widths[3] = {11, 11, 10};        // key bits not fixed yet, bits of the digit
    for (int pass = 0; pass < 3; ++pass) {
        if (e == hipSuccess)
            e = for_each_batch([&](RcBatch& b) {
                return pass == 0 ? launch_rc_hist(stream, b, st, keys) : launch_rc_enum(stream, b, st, keys, open[pass], widths[pass]);
            });
        if (e == hipSuccess) e = launch_rc_pick(stream, st, widths[pass], pass == 2, stats);
    }
    if (e == hipSuccess) e = for_each_batch([&](RcBatch& b) { return launch_rc_apply(stream, b, st, keys); });
    return e;
}

int tf_reconcile_mask(tf_ctx* ctx, void* hip_stream,
                      int32_t n_tensors, const int64_t* numel,
                      uint32_t* const* elem_bits,
                      int64_t n_freeze, uint64_t seed,
                      int64_t* stats) {
    const int rc = validate_reconcile(n_tensors, numel, elem_bits, n_freeze, stats);
    if (rc != TF_OK) return rc;
    if (!ctx) return TF_ERR_INVALID_ARG;
    if (!use_device(ctx)) return TF_ERR_HIP;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    ProfScope prof(ctx, stream, TF_KERNEL_RECONCILE);
    const hipError_t e = reconcile_passes(stream, n_tensors, numel, elem_bits, n_freeze, seed, stats, ctx->rc_state,
                                          reconcile_undo(ctx, stream, n_tensors, numel));
    if (e != hipSuccess) return hip_fail(ctx, e);
    return TF_OK;
}

int tf_reconcile_mask_static(tf_ctx* ctx, void* hip_stream,
                             int32_t n_tensors, const int64_t* numel,
                             uint32_t* const* elem_bits,
                             int64_t n_freeze, uint64_t seed,
                             int64_t* stats) {
    const int rc = validate_reconcile(n_tensors, numel, elem_bits, n_freeze, stats);     // sizes beyond 2^32 - 1 elements: TF_ERR_SHAPE
    if (rc != TF_OK) return rc;
    if (!ctx || !ctx->rc_state_static) return TF_ERR_INVALID_ARG;
    if (!use_device(ctx)) return TF_ERR_HIP;
    // no timing events here: creating one allocates
    const hipError_t e = reconcile_passes(static_cast<hipStream_t>(hip_stream), n_tensors, numel, elem_bits, n_freeze,
                                          seed, stats, ctx->rc_state_static, nullptr);
    if (e != hipSuccess) return hip_fail(ctx, e);
    return TF_OK;
}

int tf_select_row_blocks(int32_t n_layers, const tf_shape* shapes, int32_t block_rows,
                         double r, uint64_t seed, uint8_t* masks, int64_t* frozen_params) {
    if (n_layers < 0 || block_rows <= 0 || !(r >= 0.0 && r <= 1.0)) return TF_ERR_INVALID_ARG;
    if (n_layers > 0 && (!shapes || !masks)) return TF_ERR_INVALID_ARG;
    struct Unit { uint32_t key; int64_t size; int64_t pos; };
    std::vector<Unit> units;
    const RcKeys keys = perm32_keys(seed);
    int64_t total = 0;
    for (int32_t l = 0; l < n_layers; ++l) {
        if (shapes[l].K <= 0 || shapes[l].N <= 0 || shapes[l].K % block_rows != 0) return TF_ERR_SHAPE;
        for (int64_t b = 0; b < shapes[l].K / block_rows; ++b) {
            if (units.size() >= 0xffffffffull) return TF_ERR_SHAPE;
            const int64_t pos = int64_t(units.size());
            units.push_back(Unit{perm32(uint32_t(pos), keys), int64_t(block_rows) * shapes[l].N, pos});
            total += units.back().size;
        }
    }
    const int64_t budget = int64_t(std::floor(r * double(total) + 1e-9));
    std::sort(units.begin(), units.end(), [](const Unit& a, const Unit& b) { return a.key < b.key; });
    for (size_t i = 0; i < units.size(); ++i) masks[i] = 0;
    int64_t frozen = 0;
    for (const Unit& u : units)
        if (frozen + u.size <= budget) { frozen += u.size; masks[u.pos] = 1; }
    if (frozen_params) *frozen_params = frozen;
    return TF_OK;
}

int tf_row_blocks_to_bits(tf_ctx* ctx, void* hip_stream,
                          int32_t n_layers, const tf_shape* shapes,
                          const uint8_t* const* row_block_mask, int32_t block_rows,
                          uint32_t* const* elem_bits) {
    if (n_layers < 0 || block_rows <= 0) return TF_ERR_INVALID_ARG;
    if (n_layers > 0 && (!shapes || !elem_bits)) return TF_ERR_INVALID_ARG;
    for (int32_t l = 0; l < n_layers; ++l) {
        if (shapes[l].K <= 0 || shapes[l].N <= 0) return TF_ERR_SHAPE;
        if (!elem_bits[l]) return TF_ERR_INVALID_ARG;
        if (reinterpret_cast<uintptr_t>(elem_bits[l]) & 3u) return TF_ERR_ALIGN;
        const uint8_t* rm = row_block_mask ? row_block_mask[l] : nullptr;
        if (rm) {
            if (shapes[l].K % block_rows != 0) return TF_ERR_SHAPE;
            if ((int64_t(block_rows) * shapes[l].N) % 32 != 0) return TF_ERR_SHAPE;     // blocks must end on word boundaries
            for (int64_t b = 0; b < shapes[l].K / block_rows; ++b)
                if (rm[b] > 1) return TF_ERR_INVALID_ARG;
        }
    }
    if (!ctx) return TF_ERR_INVALID_ARG;
    if (!use_device(ctx)) return TF_ERR_HIP;

    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    FillBatch batch;
    batch.n_runs = 0; batch.pad_ = 0;
    auto push = [&](uint32_t* dst, int64_t n_words, uint32_t value) -> hipError_t {
        if (n_words <= 0) return hipSuccess;
        FillRunDesc& d = batch.r[batch.n_runs++];
        d.dst = dst; d.n_words = n_words; d.value = value; d.pad_ = 0;
        if (batch.n_runs == kMaxFillRuns) {
            const hipError_t e = launch_fill_words(stream, batch);
            batch.n_runs = 0;
            return e;
        }
        return hipSuccess;
    };
    for (int32_t l = 0; l < n_layers; ++l) {
        const int64_t numel = shapes[l].K * shapes[l].N;
        const uint8_t* rm = row_block_mask ? row_block_mask[l] : nullptr;
        hipError_t e = hipSuccess;
        if (!rm) {
            e = push(elem_bits[l], (numel + 31) / 32, 0u);
        } else {
            const int64_t nb = shapes[l].K / block_rows, wpb = int64_t(block_rows) * shapes[l].N / 32;
            for (int64_t b = 0; b < nb && e == hipSuccess;) {
                int64_t e1 = b;
                while (e1 < nb && rm[e1] == rm[b]) ++e1;
                e = push(elem_bits[l] + b * wpb, (e1 - b) * wpb, rm[b] ? 0xffffffffu : 0u);
                b = e1;
            }
        }
        if (e != hipSuccess) return hip_fail(ctx, e);
    }
    const hipError_t e = launch_fill_words(stream, batch);
    if (e != hipSuccess) return hip_fail(ctx, e);
    return TF_OK;
}

}  // extern "C"

// For the binding, which knows what its tables of device buffers hold: is table t's entry i on the
// device, of the element type and large enough for what a call will index?  Per table eight numbers:
// address of its int64 rows [bytes][type][device][present] of n entries each (type and device -2 =
// unknown), addresses of two int64 arrays whose products a[i * stride] * b[i * stride] * scale are the elements needed
// (b may be 0: just a), stride, scale, element type, skip the entries that `skip` marks.
// Returns -1, or the number of the first table that does not pass.
extern "C" int tf_internal_check_tables(int32_t n_tables, const int64_t* desc, int32_t n, const uint8_t* skip, int32_t device) {
    for (int32_t t = 0; t < n_tables; ++t, desc += 8) {
        const int64_t* info = reinterpret_cast<const int64_t*>(desc[0]);
        const int64_t* a = reinterpret_cast<const int64_t*>(desc[1]);
        const int64_t* b = reinterpret_cast<const int64_t*>(desc[2]);
        const int64_t stride = desc[3], scale = desc[4], dtype = desc[5], size = dtype == TF_BF16 ? 2 : 4;
        for (int32_t i = 0; i < n; ++i) {
            if (!info[3 * int64_t(n) + i] || (desc[6] && skip && skip[i])) continue;
            const int64_t type = info[int64_t(n) + i], dev = info[2 * int64_t(n) + i];
            if (info[i] < int64_t(uint64_t(a[i * stride]) * uint64_t(b ? b[i * stride] : 1) * uint64_t(scale) * uint64_t(size))) return t;
            if ((type != -2 && type != dtype) || (device >= 0 && dev != -2 && dev != device)) return t;
        }
    }
    return -1;
}

// Test hook (not part of the public header): the kernels that this context's GEMM launches take, so that a
// small problem can be sent through each of them.  A context starts with 0, the estimated times.
extern "C" int tf_internal_gemm_route(tf_ctx* ctx, int route) {
    if (!ctx || route < kRouteEstimated || route >= kRouteEnd) return TF_ERR_INVALID_ARG;
    ctx->gemm_route = route;
    return TF_OK;
}

// Test hook (not part of the public header): did the context's last backward call launch both of its halves together?
// kGenericShapes x + w, the tiles they had (see kRouteF32), behind them the launch shapes of the kernel of bf16 pieces; or -1.
extern "C" int tf_internal_common_tiles(const tf_ctx* ctx) { return ctx ? ctx->common_tiles.load(std::memory_order_relaxed) : -1; }

// Test hook (not part of the public header): how the context's last tf_reconcile_mask went, once the device is done with it: the
// window of its guess (top halves of keys; [0, 0): nothing guessed), candidates found by the probe, candidates drawn below
// the window, whether the guess held.
extern "C" int tf_internal_reconcile_outcome(tf_ctx* ctx, int64_t* out) {
    if (!ctx || !out) return TF_ERR_INVALID_ARG;
    RcState* const st = new (std::nothrow) RcState;
    if (!st) return TF_ERR_WORKSPACE;
    hipError_t e = use_device(ctx) ? hipDeviceSynchronize() : hipErrorInvalidDevice;
    if (e == hipSuccess) e = hipMemcpy(st, ctx->rc_state, sizeof(RcState), hipMemcpyDeviceToHost);
    if (e == hipSuccess) {
        out[0] = st->window_lo; out[1] = st->window_hi; out[2] = st->probe;
        out[3] = int64_t(st->drawn); out[4] = st->done;
    }
    delete st;
    return e == hipSuccess ? TF_OK : hip_fail(ctx, e);
}

// Test hook (not part of the public header): kernel[i] of problem i when these problems (operands packed, buffers
// aligned) are launched together, by the estimated times: -1 the 256 x 256-tile kernel, 0.. the launch shapes of the
// generic kernel, behind them those of the kernel for input gradients of few rows, of the kernel for weight
// gradients of few tokens and of the kernel of bf16 pieces.
// after: rows of the tensor behind the problem's own (it is a run of its rows), or NULL.
extern "C" int tf_internal_kernels(int n, const int64_t* M, const int64_t* N, const int64_t* Kc, const int64_t* after, int layout_tn,
                                   int in_dtype, int out_dtype, int accumulate, int32_t* kernel) {
    const Layout layout = layout_tn ? Layout::kTN : Layout::kNT;
    std::vector<Planned> items;
    for (int i = 0; i < n; ++i) {
        const int64_t more = after ? after[i] : 0;
        items.push_back(Planned{nullptr, nullptr, nullptr, M[i], N[i], Kc[i], layout_tn ? M[i] + more : Kc[i], layout_tn ? N[i] : Kc[i], ~0ull, {}});
        items.back().rows_after = more;
    }
    Routes r;
    if (find_routes(items, layout, to_dtype(tf_dtype(in_dtype)), to_dtype(tf_dtype(out_dtype)), accumulate != 0, kRouteEstimated, r) != hipSuccess) return TF_ERR_SHAPE;
    if (in_dtype == TF_F32) {
        const std::vector<const Planned*> v = pointers(items), none;
        r.shape[kOther] = layout_tn ? choose_f32(none, v, kRouteEstimated).w : choose_f32(v, none, kRouteEstimated).x;
    }
    for (int c = 0; c < kClasses; ++c)
        for (const Planned* it : r.cls[c]) kernel[it - items.data()] = r.shape[c];
    return TF_OK;
}

// Test hook (not part of the public header): which launch shape of the generic kernel a launch of these
// problems gets, its tile goes to tile[0..1]; and what it is expected to take, *us.
extern "C" int tf_internal_generic_shape(int n, const int64_t* M, const int64_t* N, const int64_t* Kc, int in_dtype, int32_t* tile, double* us) {
    std::vector<Planned> items;
    for (int i = 0; i < n; ++i) items.push_back(Planned{nullptr, nullptr, nullptr, M[i], N[i], Kc[i], 0, 0, ~0ull, {}});
    std::vector<const Planned*> p;
    for (const Planned& it : items) p.push_back(&it);
    const Dtype dt = to_dtype(tf_dtype(in_dtype));
    const int shape = pick_generic_shape(p, dt, us);
    tile[0] = generic_shape(dt, shape).tile_m;
    tile[1] = generic_shape(dt, shape).tile_n;
    return shape;
}
