// C ABI of the CD-GraB pair-balancing library (see include/cdgrab.h for the
// contract of every entry point).  Host orchestration only: every arithmetic
// step of the path runs in the kernels of balance_kernels.hpp / order_kernels.hpp.
#include "../../include/cdgrab.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <numeric>
#include <string>
#include <vector>

#include "balance_kernels.hpp"
#include "chain_kernels.hpp"
#include "order_kernels.hpp"
#include "herding_kernels.hpp"
#include "band_kernels.hpp"
#include "narrow_kernels.hpp"
#include "train_kernels.hpp"

using namespace cdgrab;

namespace {

thread_local std::string g_create_error;

enum Interval { kGen = 0, kBalance, kPass1, kReduce, kResolve, kPass2, kFinish, kIntervalKinds };

struct Mark {
    hipEvent_t ev;
    int kind_after;  // what runs between this mark and the next one (-1: nothing timed)
};

}  // namespace

struct cdgrab_handle {
    int device = 0;
    hipStream_t stream = nullptr;
    int block_pairs_opt = 0;
    int timing = 0;
    int pass1_groups_opt = 0;
    int apply_mode = 0;  // 0 choose by row length, 1 separate apply launch, 2 apply fused into the next block's launch,
                         // 3 / 4 separate launch, always in the resident / the flat form
    int apply_groups_opt = 0;  // cap on the resident apply grid (0: two workgroups per CU)
    int gram_mode = 0;   // 0 choose, 1 each block's Gram in its own launch, 2 Grams of many blocks ahead in one launch
    int num_cu = 256;
    std::string err;

    double *r_sum = nullptr;   int64_t r_cap = 0;         // doubles
    double *partials = nullptr; int64_t partials_cap = 0; // doubles
    double *reduced = nullptr;                            // kReduceSlices x PartLayout<64>::PART doubles
    int8_t *eps_blk = nullptr; int64_t eps_cap = 0;       // signs of the current block (per walk: of the current step)
    int32_t *flag = nullptr;                              // reorder's bad-sign flag
    int32_t *reorder_counts = nullptr; int64_t reorder_cap = 0;  // reorder: +1 signs per chunk
    double *mean_ws = nullptr; int64_t mean_cap = 0;      // column mean: sums per chunk of rows
    const float *uniforms = nullptr;                      // caller's draws while a randomized epoch runs
    int64_t walks = 1;                                    // independent walks per launch while such an epoch runs
    WalkStrides ws{};                                     // their strides (all zero for one walk)
    float *zero_row = nullptr; int64_t zero_row_cap = 0;  // a zero vector standing in for a missing stale mean
    float *train_delta = nullptr; int64_t train_delta_cap = 0;  // [m][classes] softmax deltas of one step (of a block of steps)
    int64_t *train_order = nullptr; int64_t train_order_cap = 0;  // rows of the examples in visiting order
    double *train_base = nullptr; int64_t train_base_cap = 0;     // logits of a block's examples at its first weights
    double *train_gram = nullptr; int64_t train_gram_cap = 0;     // Gram tiles of a chunk's features ...
    double *train_parts = nullptr; int64_t train_parts_cap = 0;   // ... and shares of those whose elements are split
    int32_t *train_perm = nullptr; int64_t train_perm_cap = 0;  // spare [m][n] order of the multi-epoch driver
    int8_t *train_signs = nullptr; int64_t train_signs_cap = 0; // its [m][n/2] signs when the caller wants none
    double *herd_ws = nullptr; int64_t herd_cap = 0;      // herding evaluator: segment sums, starts, mean
    double *herd_steps = nullptr; int64_t herd_steps_cap = 0;  // its steps' sums over the workers
    double *gram_all = nullptr; int64_t gram_all_cap = 0; // Grams-ahead form: Gram tiles of a batch of steps
    double *gram_parts = nullptr; int64_t gram_parts_cap = 0;      // shares of tiles whose elements are split
    double *dot_partials = nullptr; int64_t dot_partials_cap = 0;  // its per-workgroup dots of one step
    double *bands = nullptr; int64_t bands_cap = 0;       // rows of at most kNarrowMaxD elements: Gram results and differences
                                                          // beforehand.  Not gram_all: that one's address is in recorded chains.
    bool bands_in_graphs = false;                         // recorded launches hold its address ...
    double *bands_kept = nullptr;                         // ... or that of this one, which it has replaced
    float *staging = nullptr;  int64_t staging_cap = 0;   // floats: two staging chunks (the fused pass reads the previous block too)
    bool fixed_workspace = false;                         // the workspace pointers are borrowed: never grow or free them

    hipStream_t side = nullptr;                           // chunks are balanced here while the next one is generated
    hipEvent_t filled = nullptr, balanced[2] = {};        // the order between the two streams

    std::vector<hipEvent_t> event_pool;
    std::vector<Mark> marks;
    size_t events_used = 0;
    bool have_timing = false;
    cdgrab_timing last{};
};

namespace {

int fail(cdgrab_handle *h, int code, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    if (h) h->err = buf; else g_create_error = buf;
    return code;
}

#define HIP_TRY(h, expr)                                                                  \
    do {                                                                                  \
        hipError_t e_ = (expr);                                                           \
        if (e_ != hipSuccess)                                                             \
            return fail(h, CDGRAB_EHIP, "%s failed: %s", #expr, hipGetErrorString(e_));   \
    } while (0)

int64_t round_up(int64_t v, int64_t q) { return (v + q - 1) / q * q; }

// Do the byte ranges [a, a + na) and [b, b + nb) share a byte?  (Null ranges never do.)
bool ranges_overlap(const void *a, int64_t na, const void *b, int64_t nb) {
    if (!a || !b || na <= 0 || nb <= 0) return false;
    const uintptr_t a0 = reinterpret_cast<uintptr_t>(a), b0 = reinterpret_cast<uintptr_t>(b);
    return a0 < b0 + (uintptr_t)nb && b0 < a0 + (uintptr_t)na;
}

int pick_vector_width(int64_t d, int64_t base_align) {
    if (d % 4 == 0 && base_align % 16 == 0) return 4;
    if (d % 2 == 0 && base_align % 8 == 0) return 2;
    return 1;
}

// How the kernels read the rows (kAligned / kAnyRow / kTiny), from the alignment the plan reports.
int row_form(int vector_width, int64_t d) { return vector_width == 4 ? kAligned : d >= 4 ? kAnyRow : kTiny; }

// 32 pairs per block keep the double-precision Gram tiles under the HBM time for
// long rows; short rows are bound by launches, not bytes, and take 64.
int pick_block_pairs(int64_t pairs, int64_t d, int32_t requested) {
    if (requested == 16 || requested == 32 || requested == 64) return requested;
    if (pairs <= 16) return 16;
    if (pairs > 32 && d <= 65536) return 64;
    return 32;
}

// Measured on MI355X: applying a block inside the next block's dot/Gram launch wins up
// to about 1.2M elements per row (one launch and one read of the running sum less: 3 % at
// 1M, 4 % at 512K, 15 % at 8K); beyond that the heavier fused kernel streams 8-12 % slower
// than the dot/Gram launch and the resident apply launch together (1.5M: 158 against 141 us
// per 32-pair block, 2M: 213 against 198, 4M: 423 against 388).
bool fuse_apply_by_default(int64_t d) { return d <= (int64_t)5 << 18; }

// Short rows: a block is bound by its chain of launches, so the Gram matrices (which depend on
// the rows only) are taken off the chain and the chain is cut into steps of 64 .. 256 pairs at
// two launches each (chain_kernels.hpp).
constexpr int64_t kGramBatch = 512;                  // a staging chunk holds at most this many blocks
constexpr int64_t kGramBytes = (int64_t)256 << 20;   // Gram tiles held at a time
// Measured on MI355X (m = 16, 4096 pairs), us per 64 pairs of the per-block form -> this form: d = 256: 16.6 -> 5.1;
// 1024: 17.9 -> 5.5; 4096: 18.2 -> 6.8; 7850: 19.6 -> 8.6; 16 384: 20.7 -> 12.1; 32 768: 30.6 -> 18.3;
// 65 536: 43.4 -> 29.9; 81 920: 43.3 -> 37.0; 98 304: 43.2 -> 42.6; 131 072: 60.7 -> 55.7 (the rows are read three times
// instead of twice).
// That is for chains of many steps.  Fewer pairs, us per epoch: 128 pairs of 57 344 elements 87 -> 65, of 65 536 (where the
// per-block form changes to tiles of 128 elements) 78 -> 69, of 81 920 80 -> 80, of 98 304 82 -> 88; 70 pairs 84 -> 62,
// 73 -> 66, 57 -> 76, 58 -> 83; 257 pairs of 81 920 183 -> 182, of 98 304 189 -> 214.  The two lines below were drawn when
// diagonal Gram tiles took a third longer (98 304 elements: 49.7 per 64 pairs in this form against 46.1; up to 128 pairs of
// 65 536: 103 against 87) and have not moved since: by these figures both could lie near 81 920 elements.
constexpr int64_t kGramAheadMaxD = 65536;     // chosen by default up to here ...
constexpr int64_t kGramAheadEdgePairs = 128;  // ... where, at that length, there are more pairs than this
constexpr int64_t kChunkAheadMaxD = 16384;    // and for staging chunks of several blocks up to here
constexpr int64_t kGramAheadLimitD = 131072;  // refused beyond (gram_mode 2)
bool gram_ahead_by_default(int64_t d, int64_t pairs) {
    return d < kGramAheadMaxD || (d == kGramAheadMaxD && pairs > kGramAheadEdgePairs);
}

int part_size(int bb) {
    return bb == 64 ? PartLayout<64>::PART : bb == 32 ? PartLayout<32>::PART : PartLayout<16>::PART;
}

// How the Grams-ahead form cuts an epoch (per walk: `walks` independent ones run side by side).
struct ChainPlan {
    int sp;             // pairs per step
    int tiles;          // Gram tiles stored per step
    int64_t steps;      // steps whose Gram tiles are computed in one launch
    int ksplit;         // workgroups sharing the elements of a tile
    int groups;         // workgroups of a step's wide launch
    int64_t band_pairs; // rows of at most kNarrowMaxD elements: pairs of a walk whose Gram results are ahead at a time (0: none are)
    int64_t gram_len, parts_len, dots_len, bands_len;  // doubles of workspace, all walks
};

// Time of one step of sp pairs, microseconds, fitted to measured epochs of 64 / 128 / 256 pairs per step.  Those epochs,
// Gram tiles included: 8192 pairs of 66 .. 256 elements 8.1 - 8.4 / 12.0 - 12.8 / 19.8 - 20.7 us per step, of 512 .. 2048
// elements 9.5 - 9.6 / 13.1 - 13.9 / 20.9 - 23.5; 30 000 pairs of 7850 elements 5.54 / 4.35 / 4.83 ms; 64 walks of 468
// pairs of 7850 1.07 / 1.52 / 2.03 ms.  Long chains of one walk want long steps, many walks or long rows short ones.
// Short chains are the model's weak side, because it counts a wide launch for the first step too, which has none: 300 pairs of
// 7850 elements 72.7 / 65.7 / 77.0 us, 71.2 as chosen; of 256 elements 54.0 / 46.2 / 43.1, 46.7 as chosen; 8 walks of 100
// pairs of 7850 50.4 / 46.8 / 45.9, 50.7 as chosen.
double step_cost_us(int64_t sp, int64_t d, int64_t walks) {
    const double blk = (double)(sp / kTilePairs), tiles = blk * (blk + 1) / 2;
    const double launches = (d > 256 ? 5.7 : 3.7) + 0.066 * (double)sp;
    const double rows = (double)walks * 16.0 * (double)sp * (double)d / 6.25e6;
    const double gram = (double)walks * tiles * kTileEntries * 2.0 * (double)d / 40e6;
    return launches + rows + gram;
}

// Workgroups per Gram tile: the launch takes whole rounds of two workgroups per CU, each as long as its
// share of a tile; shares cost a write and two reads of a tile each.  At least four tiles of elements per share (128
// pairs of 1024 elements in 32 shares of one instead of 8 of four: 1.6 us less for the tiles, and 25 us more
// for a workspace four times as large in a handle's first call).
int pick_ksplit(int64_t tiles, int64_t d, int num_cu) {
    const int64_t ktiles = (d + kGramTE - 1) / kGramTE, slots = 2 * (int64_t)num_cu;
    const double tile_us = 2.0 * kTileEntries * (double)d / (45e6 / (double)slots);
    double least = 0.0;
    int best = 1;
    for (int64_t ks = 1; ks <= std::max<int64_t>(1, std::min<int64_t>(ktiles / 4, 64)); ++ks) {
        const double rounds = (double)((tiles * ks + slots - 1) / slots) / (double)ks;
        const double us = rounds * tile_us + (ks > 1 ? 4.0 + (double)(tiles * (2 * ks + 1)) * kTileEntries * 8.0 / 4e6 : 0.0);
        if (ks == 1 || us < 0.98 * least) { least = us; best = (int)ks; }
    }
    return best;
}

// Rows of at most kNarrowMaxD elements: Gram results beforehand (band_kernels.hpp) or inside the walk's workgroup
// (narrow_kernels.hpp).  The first has one launch more and walks faster.  us per epoch of one walk, inside -> beforehand, rows of
// 16 / 32 / 64 elements: 256 pairs 13.4 -> 16.8 / 13.6 -> 17.2 / 19.0 -> 21.7; 384 pairs 16.9 -> 17.0 / 17.2 -> 18.1 /
// 23.9 -> 24.7; 512 pairs 19.7 -> 17.4 / 20.6 -> 19.6 / 29.9 -> 27.9; 4096 pairs 89 -> 71 / 108 -> 75 / 172 -> 107; 200 000
// pairs 3846 -> 2861 / 4814 -> 2925 / 7939 -> 4276.  The results of all walks go through memory: 16 walks of 512 pairs 19.7 -> 19.0 /
// 20.5 -> 22.0 / 28.9 -> 30.4, of 768 24.8 -> 24.3 / 27.0 -> 27.4 / 39.9 -> 38.2, of 1024 29.8 -> 29.2 / 33.2 -> 32.6 / 49.7 ->
// 45.0, of 4000 88 -> 82 / 107 -> 87 / 170 -> 128; 100 walks of 1000 30.6 -> 40.1 / - / 51 -> 95.
// More than 16 walks, of 4000 and 25 000 pairs: 17 walks 88 -> 83 and 497 -> 473 / 107 -> 90 and 628 -> 525 / 169 -> 144 and 1016 ->
// 826; 20 walks 88 -> 82 and 497 -> 484 / 107 -> 91 and 629 -> 555 / 170 -> 152 and 1015 -> 913; 24 walks 88 -> 84 and 498 -> 506 /
// 107 -> 106 and 629 -> 586 / 170 -> 159 and 1018 -> 975; 32 walks 89 -> 99 and 500 -> 547 / 108 -> 114 and 629 -> 687 / 170 -> 167
// and 1018 -> 1077; 64 walks 89 -> 122 and 501 -> 794 / 108 -> 151 and 632 -> 1031 / 172 -> 244 and 1025 -> 1610.  By these the line
// could lie near 20 walks.
constexpr int64_t kBandMinPairs = 512, kBandMinPairsMore = 32;  // of the only walk, per further walk
constexpr int64_t kBandMaxWalks = 16;
constexpr int64_t kBandBytes = (int64_t)64 << 20;  // Gram results and differences held at a time, but for whole strides of blocks
// in doubles, with those: what no epoch exceeds
constexpr int64_t kBandMost = kBandBytes / 8 + kBandMaxWalks * (kBandStride + 1) * band_doubles(kNarrowMaxD);
int narrow_padded(int64_t d) { return d <= 16 ? 16 : d <= 32 ? 32 : 64; }

ChainPlan plan_chain(int64_t pairs, int64_t d, int64_t walks, int64_t chunk_pairs, int num_cu) {
    ChainPlan c{};
    const int64_t longest = chunk_pairs > 0 ? std::min(chunk_pairs, pairs) : pairs;
    if (d <= kNarrowMaxD) {  // a walk is one workgroup
        c.sp = kTilePairs;
        if (walks <= kBandMaxWalks && longest >= kBandMinPairs + kBandMinPairsMore * (walks - 1)) {
            const int64_t per_block = band_doubles(narrow_padded(d));
            const int64_t held = std::max<int64_t>(1, kBandBytes / 8 / per_block / walks);
            const int64_t blocks = round_up(std::min<int64_t>((longest + kBandBlock - 1) / kBandBlock, held), kBandStride);
            c.band_pairs = blocks * kBandBlock;
            c.bands_len = walks * band_walk_doubles(narrow_padded(d), blocks);
        }
        return c;
    }
    double best = 0.0;
    for (int sp = kTilePairs; sp <= kMaxStepPairs; sp *= 2) {
        if (sp > kTilePairs && sp / 2 >= longest) break;  // a shorter step holds them all
        const double cost = (double)((pairs + sp - 1) / sp) * step_cost_us(sp, d, walks);
        if (c.sp == 0 || cost < best) { c.sp = sp; best = cost; }
    }
    const int blk = c.sp / kTilePairs;
    c.tiles = blk * (blk + 1) / 2;
    const int64_t per_step = walks * c.tiles * kTileEntries;
    const int64_t total = (longest + c.sp - 1) / c.sp;
    c.steps = std::max<int64_t>(1, std::min<int64_t>(total, kGramBytes / 8 / per_step));
    c.ksplit = pick_ksplit(c.steps * walks * c.tiles, d, num_cu);
    c.groups = (int)((d + kStepElems - 1) / kStepElems);
    c.gram_len = c.steps * per_step;
    c.parts_len = c.ksplit > 1 ? c.gram_len * c.ksplit : 0;
    c.dots_len = walks * c.groups * c.sp;
    return c;
}

// Two staging chunks when a launch reads the previous block's rows as well and there is a next chunk.
int64_t staging_chunks(int64_t pairs, int64_t chunk_pairs, bool reads_previous) {
    return reads_previous && pairs > chunk_pairs ? 2 : 1;
}

// The launch plan of one epoch.  `chunk_pairs` is the number of flattened pairs staged per
// generator call (streamed input; 0 = one block), `walks` the number of independent epochs side by side.  Every decision an epoch takes is taken
// here, so that cdgrab_plan_epoch reports exactly what a handle with the same options runs.
int plan_epoch(int64_t m, int64_t n, int64_t d, int32_t block_pairs, int32_t streamed,
               int64_t base_align, int num_cu, int32_t pass1_groups_opt, int apply_mode, int gram_mode,
               int64_t chunk_pairs, int64_t walks, cdgrab_plan *plan) {
    if (m < 1 || n < 2 || (n & 1) || d < 1 || !plan) return CDGRAB_EINVAL;
    if (block_pairs != 0 && block_pairs != 16 && block_pairs != 32 && block_pairs != 64) return CDGRAB_EINVAL;
    if (base_align < 4 || (base_align & (base_align - 1))) return CDGRAB_EINVAL;
    if (m > (INT64_MAX / n) / d || m > (1 << 30)) return CDGRAB_EINVAL;
    plan->pairs = m * (n / 2);
    plan->block_pairs = pick_block_pairs(plan->pairs, d, block_pairs);
    const int64_t bb = plan->block_pairs;
    plan->blocks = (plan->pairs + bb - 1) / bb;
    plan->vector_width = pick_vector_width(d, streamed ? 256 : base_align);
    // long rows stream through 128-element tiles with two resident workgroups per CU;
    // short rows use 64-element tiles so that more workgroups share the work
    plan->tile_elems = (d >= (int64_t)128 * 2 * num_cu) ? 128 : 64;
    int64_t ntiles = (d + plan->tile_elems - 1) / plan->tile_elems;
    int64_t want = pass1_groups_opt > 0 ? pass1_groups_opt
                                        : (int64_t)num_cu * (plan->tile_elems == 128 ? 2 : 4);
    plan->pass1_groups = (int32_t)std::max<int64_t>(1, std::min<int64_t>(want, ntiles));
    plan->pass2_groups = (int32_t)((d + kThreads * 4 - 1) / (kThreads * 4));
    if (chunk_pairs <= 0) chunk_pairs = bb;

    // Grams ahead: asked for, or chosen for short rows when the caller left both choices
    // open; for streamed rows when a staging chunk holds more than one block's pairs.
    const bool ahead_dense = !streamed && plan->blocks >= 2 &&
                             (gram_mode == 2 || (gram_mode == 0 && apply_mode == 0 &&
                                                 gram_ahead_by_default(d, plan->pairs * walks)));
    const bool ahead_streamed = streamed && gram_mode != 1 && apply_mode == 0 && d <= kChunkAheadMaxD &&
                                plan->pairs > bb && chunk_pairs > bb && chunk_pairs <= kGramBatch * bb;
    const bool ahead = ahead_dense || ahead_streamed;
    // the ahead form applies a block inside the next block's launch by construction
    const bool fused = !ahead && (apply_mode == 2 || (apply_mode == 0 && fuse_apply_by_default(d)));
    plan->gram_ahead = ahead ? 1 : 0;
    plan->fused_apply = fused ? 1 : 0;
    plan->step_pairs = 0;

    plan->staging_bytes = streamed ? staging_chunks(plan->pairs, chunk_pairs, fused || ahead) * chunk_pairs * 2 * d * 4 : 0;
    const int64_t part = part_size(plan->block_pairs);
    const int64_t partial_doubles = (int64_t)plan->pass1_groups * part;
    int64_t ahead_bytes = 0;
    if (ahead) {
        const ChainPlan c = plan_chain(plan->pairs, d, 1, streamed ? chunk_pairs : 0, num_cu);
        plan->step_pairs = c.sp;
        ahead_bytes = (c.gram_len + c.parts_len + c.dots_len + c.bands_len) * 8 + kMaxStepPairs;
    }
    plan->workspace_bytes = round_up(d, kPadE) * 8 + partial_doubles * 8 +
                            (int64_t)kReduceSlices * PartLayout<64>::PART * 8 + 64 + ahead_bytes +
                            plan->staging_bytes;
    // each row twice; the double running sum read twice and written once per block, or read
    // once and written once when the apply rides in the next block's launch; with the Gram
    // matrices ahead the rows are read three times (less: the first step takes no dots, and a step is
    // at least a block), or once where the walk runs in one workgroup
    plan->bytes_per_example = ahead ? (d <= kNarrowMaxD ? 4.0 * (double)d : 12.0 * (double)d + 8.0 * (double)d / (double)bb)
                                    : 8.0 * (double)d + (fused ? 8.0 : 12.0) * (double)d / (double)bb;
    return CDGRAB_OK;
}

// ---- timing marks ----------------------------------------------------------
int mark(cdgrab_handle *h, int kind_after) {
    if (h->events_used == h->event_pool.size()) {
        hipEvent_t ev;
        HIP_TRY(h, hipEventCreate(&ev));
        h->event_pool.push_back(ev);
    }
    hipEvent_t ev = h->event_pool[h->events_used++];
    HIP_TRY(h, hipEventRecord(ev, h->stream));
    h->marks.push_back({ev, kind_after});
    return CDGRAB_OK;
}

#define MARK(h, level, kind)                                   \
    do {                                                       \
        if ((h)->timing >= (level)) {                          \
            int rc_ = mark((h), (kind));                       \
            if (rc_ != CDGRAB_OK) return rc_;                  \
        }                                                      \
    } while (0)

template <typename T>
int ensure(cdgrab_handle *h, T *&ptr, int64_t &cap, int64_t want) {
    if (cap >= want) return CDGRAB_OK;
    if (h->fixed_workspace)
        return fail(h, CDGRAB_ENOMEM, "the fixed workspace is too small (%lld elements needed, %lld there)",
                    (long long)want, (long long)cap);
    if (ptr) { HIP_TRY(h, hipStreamSynchronize(h->stream)); HIP_TRY(h, hipFree(ptr)); ptr = nullptr; cap = 0; }
    hipError_t e = hipMalloc(reinterpret_cast<void **>(&ptr), (size_t)want * sizeof(T));
    if (e != hipSuccess) {
        ptr = nullptr;
        (void)hipGetLastError();
        return fail(h, CDGRAB_ENOMEM, "workspace allocation of %lld bytes failed: %s",
                    (long long)(want * (int64_t)sizeof(T)), hipGetErrorString(e));
    }
    cap = want;
    return CDGRAB_OK;
}

// The same where the call can do without: no error of the call if there is no room.
template <typename T>
bool room(cdgrab_handle *h, T *&ptr, int64_t &cap, int64_t want) {
    const std::string text = h->err;
    const bool there = ensure(h, ptr, cap, want) == CDGRAB_OK;
    if (!there) h->err = text;
    return there;
}

// Are the handle's launches being recorded?
bool capturing(cdgrab_handle *h) {
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(h->stream, &status) == hipSuccess) return status != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return true;
}

// `want` doubles for the Gram results of long narrow walks, or false: then they go without.  A recorded call allocates nothing
// and takes the buffer that an eager one has left.  That buffer is not given back before the handle is; the one that takes its
// place has room for any epoch, so that there is one such buffer.
bool bands_room(cdgrab_handle *h, int64_t want) {
    if (capturing(h)) {
        if (h->bands_cap < want) return false;
        h->bands_in_graphs = true;
        return true;
    }
    if (h->bands_cap >= want || !h->bands_in_graphs) return room(h, h->bands, h->bands_cap, want);
    double *all = nullptr;
    int64_t cap = 0;
    if (!room(h, all, cap, kBandMost)) return false;
    h->bands_kept = h->bands;
    h->bands = all;
    h->bands_cap = cap;
    return true;
}

template <int BB, int VW>
void launch_pass1(cdgrab_handle *h, const RowMap &rm, const PrevBlock *prev, bool fresh, const cdgrab_plan &plan) {
    PrevBlock none;
    none.rm = rm;
    none.rm.nb = 0;
    none.eps = h->eps_blk;
    const dim3 grid(plan.pass1_groups), block(kThreads);
    const int64_t ntiles = (rm.d + plan.tile_elems - 1) / plan.tile_elems;
    auto launch = [&](auto kernel, const PrevBlock &pb) {
        hipLaunchKernelGGL(kernel, grid, block, 0, h->stream, rm, pb, h->r_sum, h->partials, ntiles);
    };
    auto by_start = [&](auto tile) {
        constexpr int TE = decltype(tile)::value;
        if (prev && fresh) launch(pass1_dots_gram<BB, VW, TE, true, true>, *prev);
        else if (prev) launch(pass1_dots_gram<BB, VW, TE, true, false>, *prev);
        else if (fresh) launch(pass1_dots_gram<BB, VW, TE, false, true>, none);
        else launch(pass1_dots_gram<BB, VW, TE, false, false>, none);
    };
    if (plan.tile_elems == 128) by_start(std::integral_constant<int, 128>{});
    else by_start(std::integral_constant<int, 64>{});
}
// Rows from this length on take the resident form of the apply pass (the running-sum
// traffic in one burst); shorter ones the flat form, whose launch ramps up faster
// (block of 32 pairs, dot/Gram launch included: 1M elements 106 against 115 us, 768K 84
// against 80 us).
constexpr int64_t kResidentMinD = (int64_t)1 << 20;

template <int BB, int VW>
void launch_pass2(cdgrab_handle *h, const RowMap &rm, const SumEnds &ends, int groups) {
    // short rows: too few flat workgroups to hide latency -> split the pairs over thread groups
    if (groups < 2 * h->num_cu && h->apply_mode < 3) {
        const dim3 grid((unsigned)((rm.d + kSplitElems - 1) / kSplitElems));
        if (rm.nb == BB)
            hipLaunchKernelGGL((pass2_apply_split<BB, VW, true>), grid, dim3(kThreads), 0, h->stream, rm,
                               h->eps_blk, ends, h->r_sum);
        else
            hipLaunchKernelGGL((pass2_apply_split<BB, VW, false>), grid, dim3(kThreads), 0, h->stream, rm,
                               h->eps_blk, ends, h->r_sum);
        return;
    }
    if (h->apply_mode == 3 || (h->apply_mode != 4 && rm.d >= kResidentMinD)) {
        // a wholly resident grid: two workgroups per CU, each thread up to kResidentGroups groups of four
        const int64_t quads = (rm.d + 3) / 4;
        int64_t grid = std::min<int64_t>(2 * (int64_t)h->num_cu, (quads + kThreads - 1) / kThreads);
        if (h->apply_groups_opt > 0) grid = std::min<int64_t>(grid, h->apply_groups_opt);
        const int64_t T = grid * kThreads;
        const int64_t per_thread = (quads + T - 1) / T;
        const int64_t slabs = (per_thread + kResidentGroups - 1) / kResidentGroups;
        const int kuse = (int)((per_thread + slabs - 1) / slabs);
        // one launch per slab: the boundary keeps the workgroups in step, so that each slab ends in
        // one burst of running-sum traffic
        for (int64_t sl = 0; sl < slabs; ++sl) {
            if (rm.nb == BB)
                hipLaunchKernelGGL((pass2_apply_resident<BB, VW, true>), dim3((unsigned)grid), dim3(kThreads), 0,
                                   h->stream, rm, h->eps_blk, ends, h->r_sum, kuse, sl * kuse);
            else
                hipLaunchKernelGGL((pass2_apply_resident<BB, VW, false>), dim3((unsigned)grid), dim3(kThreads), 0,
                                   h->stream, rm, h->eps_blk, ends, h->r_sum, kuse, sl * kuse);
        }
        return;
    }
    if (rm.nb == BB)
        hipLaunchKernelGGL((pass2_apply<BB, VW, true>), dim3(groups), dim3(kThreads), 0, h->stream, rm,
                           h->eps_blk, ends, h->r_sum);
    else
        hipLaunchKernelGGL((pass2_apply<BB, VW, false>), dim3(groups), dim3(kThreads), 0, h->stream, rm,
                           h->eps_blk, ends, h->r_sum);
}
template <int BB>
void launch_resolve(cdgrab_handle *h, const RowMap &rm, int8_t *signs_out, double *dots_out) {
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(1), dim3(kResolveThreads<BB>), 0, h->stream, h->reduced, rm.nb, rm.k0, rm.i0,
                           rm.m, rm.n / 2, h->eps_blk, signs_out, dots_out, h->uniforms);
    };
    if (h->uniforms) launch(resolve_signs<BB, true>);
    else launch(resolve_signs<BB, false>);
}

// Dispatch on how the rows are read, which is a template parameter of the kernels.
template <typename F>
void by_row_form(int form, F &&launch) {
    switch (form) {
        case kAligned: launch(std::integral_constant<int, kAligned>{}); break;
        case kAnyRow: launch(std::integral_constant<int, kAnyRow>{}); break;
        default: launch(std::integral_constant<int, kTiny>{}); break;
    }
}

// All of `pairs` consecutive pairs of rows of at most kNarrowMaxD elements.
int run_narrow(cdgrab_handle *h, const StepRows &rows, int64_t first, int64_t pairs, int64_t half_n,
               const ChainPlan &c, int8_t *signs_out, double *dots_out, float *r32, double *r64) {
    MARK(h, 2, kPass1);
    const int64_t most = c.band_pairs > 0 ? c.band_pairs : kNarrowMaxPairs;
    for (int64_t at = 0; at < pairs; at += most) {
        const int fresh = first + at == 0;
        const StepRows part = step_at(rows, at, 0);
        StepRows slots = part;  // (output slots are counted from the flattened pair, whatever the layout)
        slots.k0 = (first + at) / rows.m;
        slots.i0 = (int32_t)((first + at) % rows.m);
        const int count = (int)std::min<int64_t>(most, pairs - at);
        const dim3 walks((unsigned)h->walks);
        auto by_rule = [&](auto dp, auto vw) {
            constexpr int DP = decltype(dp)::value, VW = decltype(vw)::value;
            BandSpace space{};
            auto walk = [&](auto kernel) {
                hipLaunchKernelGGL(kernel, walks, dim3(kNarrowThreads), 0, h->stream, slots, count, half_n, fresh, space,
                                   h->r_sum, r32, r64, signs_out, dots_out, h->uniforms, h->ws);
            };
            if (c.band_pairs > 0) {
                const int blocks = (int)round_up((count + kBandBlock - 1) / kBandBlock, kBandStride);
                space = BandSpace{h->bands, band_walk_doubles(DP, blocks), blocks};
                hipLaunchKernelGGL((narrow_bands<DP, VW>), dim3((unsigned)((blocks + kWaves - 1) / kWaves), walks.x),
                                   dim3(kThreads), 0, h->stream, part, slots.k0, slots.i0, count, half_n, space, h->uniforms, h->ws);
                if (h->uniforms) walk(narrow_walk<DP, VW, true, true>);
                else walk(narrow_walk<DP, VW, false, true>);
            } else {
                if (h->uniforms) walk(narrow_walk<DP, VW, true, false>);
                else walk(narrow_walk<DP, VW, false, false>);
            }
        };
        const std::integral_constant<int, kAnyRow> any{};
        if (rows.d < 4) by_rule(std::integral_constant<int, 16>{}, std::integral_constant<int, kTiny>{});
        else if (rows.d <= 16) by_rule(std::integral_constant<int, 16>{}, any);
        else if (rows.d <= 32) by_rule(std::integral_constant<int, 32>{}, any);
        else by_rule(std::integral_constant<int, 64>{}, any);
    }
    HIP_TRY(h, hipGetLastError());
    return CDGRAB_OK;
}

// Gram tiles of `gb.units` units into out (through parts when the elements of a tile are shared).
template <bool SINGLE>
int run_gram_tiles(cdgrab_handle *h, const GramBatch &gb, double *out, double *parts, int form) {
    const int64_t padded = gb.units >= 8 ? round_up(gb.units, 8) : gb.units;
    by_row_form(form, [&](auto vw) {
        hipLaunchKernelGGL((gram_tiles<decltype(vw)::value, SINGLE>),
                           dim3((unsigned)(padded * gb.tiles), (unsigned)gb.ksplit), dim3(kThreads), 0, h->stream, gb,
                           gb.ksplit > 1 ? parts : out);
    });
    if (gb.ksplit > 1)
        hipLaunchKernelGGL(gram_reduce, dim3((unsigned)(gb.units * gb.tiles), kTileEntries / 2 / kThreads),
                           dim3(kThreads), 0, h->stream, parts, out, gb.ksplit);
    HIP_TRY(h, hipGetLastError());
    return CDGRAB_OK;
}

// Those of the steps of `pairs` pairs per walk, the first at rows, into h->gram_all.
int run_step_grams(cdgrab_handle *h, const StepRows &rows, int64_t pairs, const ChainPlan &c, int form) {
    GramBatch gb{};
    gb.rows = rows;
    gb.pairs = pairs;
    gb.walk_floats = h->ws.rows;
    gb.sp = c.sp;
    gb.steps = (int32_t)((pairs + c.sp - 1) / c.sp);
    gb.units = (int32_t)(gb.steps * h->walks);
    gb.tiles = c.tiles;
    gb.ksplit = c.ksplit;
    gb.ktiles = (int32_t)((rows.d + kGramTE - 1) / kGramTE);
    MARK(h, 2, kPass1);
    return run_gram_tiles<false>(h, gb, h->gram_all, h->gram_parts, form);
}

// Wide launch of a step: applies prev (if it has pairs), dots of cur (if it has pairs).
int run_step_wide(cdgrab_handle *h, const StepRows &cur, const StepRows &prev, const ChainPlan &c, int form, bool fresh,
                  float *r32, double *r64) {
    MARK(h, 2, kPass1);
    by_row_form(form, [&](auto vw) {
        constexpr int VW = decltype(vw)::value;
        auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3((unsigned)(c.groups >= 16 ? round_up(c.groups, 8) : c.groups), (unsigned)h->walks),
                               dim3(kStepThreads), 0, h->stream, cur, prev, h->eps_blk, c.sp, c.groups, fresh ? 1 : 0,
                               h->r_sum, h->dot_partials, r32, r64, h->ws);
        };
        if (c.sp > 128) launch(chain_apply_dots<8, VW>);
        else if (c.sp > 64) launch(chain_apply_dots<4, VW>);
        else launch(chain_apply_dots<2, VW>);
    });
    HIP_TRY(h, hipGetLastError());
    return CDGRAB_OK;
}

// Workgroups that read the next step's rows beside a walk, if those are well below what the L2s hold (32 MB).  us per
// epoch without them, with 32, 64, 120: 30 000 pairs of 7850 elements 4343 / 4177 / 4198 / 4206; 8000 of 2048 747 / 744 / 745 /
// 749, of 4096 909 / 875 / 878 / 880; 4096 of 16 384 782 / 824 / 731 / 737, of 32 768 1172 / 1388 / 1085 / 1080.  Without,
// with 64, 120 on both sides of the line, 300 and 2048 pairs: 32 768 elements (a step is 17 MB) 103.8 / 101.6 / 102.9 and
// 580 / 543 / 543; 36 864 117.1 / 116.5 / 118.4 and 678 / 640 / 649; 20 000, where the 2048 pairs are in steps of 128,
// 91.2 / 90.3 / 91.4 and 461 / 449 / 452; 40 960 118.0 / 119.2 / 121.0 and 696 / 669 / 680; 49 152
// 125.6 / 129.8 / 130.2 and 743 / 791 / 739; 57 344 149.6 / 154.9 / 156.4 and 877 / 920 / 884; 65 533 160.1 / 169.3 / 170.4 and
// 964 / 1020 / 967; 65 536 158.3 / 165.8 / 167.0 and 963 / 997 / 944; 131 072 with 120, 2048 pairs 1740 / - / 1750.
constexpr int kTouchMinGroups = 16;  // (shorter rows have no fixed XCD per element)
constexpr int64_t kTouchBytes = (int64_t)20 << 20;
constexpr unsigned kTouchWorkgroups = 64;
bool touch_next(const StepRows &next, const ChainPlan &c, int64_t walks) {
    return next.nb > 0 && walks == 1 && c.groups >= kTouchMinGroups && 2 * c.sp * next.d * 4 < kTouchBytes;
}

// Serial launch of a step: the walk; the rows of `next` (if it has pairs) are read beside it.  dot_groups 0: the running sum is still zero.
int run_step_walk(cdgrab_handle *h, const StepRows &cur, const StepRows &next, const ChainPlan &c, const double *gram,
                  int dot_groups, int64_t half_n, int8_t *signs_out, double *dots_out) {
    MARK(h, 2, kResolve);
    const unsigned beside = touch_next(next, c, h->walks) ? 8 + kTouchWorkgroups : 1;
    const RowsAhead ahead{next, c.groups};
    auto by_rule = [&](auto sb) {
        constexpr int SB = decltype(sb)::value;
        auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3((unsigned)h->walks, beside), dim3(kWalkThreads), 0,
                               h->stream, gram, h->dot_partials, dot_groups, c.sp, cur, half_n, h->eps_blk, signs_out,
                               dots_out, h->uniforms, h->ws, ahead);
        };
        if (h->uniforms) launch(chain_walk<SB, true>);
        else launch(chain_walk<SB, false>);
    };
    if (c.sp > 128) by_rule(std::integral_constant<int, 256>{});
    else if (c.sp > 64) by_rule(std::integral_constant<int, 128>{});
    else by_rule(std::integral_constant<int, 64>{});
    HIP_TRY(h, hipGetLastError());
    return CDGRAB_OK;
}

template <int BB>
int apply_block_vw(cdgrab_handle *h, const RowMap &rm, const SumEnds &ends, const cdgrab_plan &plan) {
    if (ends.last && !ends.r32 && !ends.r64) return CDGRAB_OK;  // nobody asked for the epoch's running sum
    MARK(h, 2, kPass2);
    switch (row_form(plan.vector_width, rm.d)) {
        case kAligned: launch_pass2<BB, 4>(h, rm, ends, plan.pass2_groups); break;
        case kAnyRow: launch_pass2<BB, 2>(h, rm, ends, plan.pass2_groups); break;
        default: launch_pass2<BB, 1>(h, rm, ends, plan.pass2_groups); break;
    }
    HIP_TRY(h, hipGetLastError());
    return CDGRAB_OK;
}

// One block: dots + Gram (with the previous block applied in the same launch when
// `prev` is given), reduction, sign resolution, and -- unless the apply is left to the
// next block's launch -- the apply pass.  fresh: nothing has been applied before this launch.
template <int BB>
int run_block_vw(cdgrab_handle *h, const RowMap &rm, const PrevBlock *prev, bool fresh, const SumEnds *apply_now,
                 const cdgrab_plan &plan, int8_t *signs_out, double *dots_out) {
    const int part = PartLayout<BB>::PART;
    MARK(h, 2, kPass1);
    switch (row_form(plan.vector_width, rm.d)) {
        case kAligned: launch_pass1<BB, 4>(h, rm, prev, fresh, plan); break;
        case kAnyRow: launch_pass1<BB, 2>(h, rm, prev, fresh, plan); break;
        default: launch_pass1<BB, 1>(h, rm, prev, fresh, plan); break;
    }
    MARK(h, 2, kReduce);
    hipLaunchKernelGGL(reduce_partials,
                       dim3((part + kReduceEntries - 1) / kReduceEntries, kReduceSlices),
                       dim3(kThreads), 0, h->stream, h->partials, h->reduced, part, plan.pass1_groups);
    MARK(h, 2, kResolve);
    launch_resolve<BB>(h, rm, signs_out, dots_out);
    HIP_TRY(h, hipGetLastError());
    return apply_now ? apply_block_vw<BB>(h, rm, *apply_now, plan) : CDGRAB_OK;
}

// Orders of m workers from their signs (flag already cleared).  A grid holds at most 2^23 chunks.
int launch_reorder(cdgrab_handle *h, int64_t m, int64_t n, const int8_t *signs, const int32_t *perm_in,
                   int32_t *perm_out) {
    const int64_t chunks = (n + kReorderChunk - 1) / kReorderChunk;
    const int64_t most = std::max<int64_t>(1, ((int64_t)1 << 23) / chunks);
    if (chunks > 1) {
        const int rc = ensure(h, h->reorder_counts, h->reorder_cap, std::min(m, most) * chunks);
        if (rc) return rc;
    }
    for (int64_t i = 0; i < m; i += most) {
        const dim3 grid((unsigned)(std::min(most, m - i) * chunks)), block(kReorderThreads);
        if (chunks > 1)
            hipLaunchKernelGGL(reorder_count, grid, block, 0, h->stream, signs + i * n, n, chunks, h->reorder_counts);
        auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, grid, block, 0, h->stream, signs + i * n, perm_in ? perm_in + i * n : nullptr,
                               perm_out + i * n, n, chunks, h->reorder_counts, h->flag);
        };
        if (n <= kReorderThreads) launch(reorder_from_signs<1>);
        else if (n <= 4 * kReorderThreads) launch(reorder_from_signs<4>);
        else if (n <= 8 * kReorderThreads) launch(reorder_from_signs<8>);
        else launch(reorder_from_signs<kReorderPer>);
    }
    HIP_TRY(h, hipGetLastError());
    return CDGRAB_OK;
}

// mean_out[d] of n rows: about four workgroups per CU, at least eight rows per thread.
int launch_column_mean(cdgrab_handle *h, int64_t n, int64_t d, const float *rows, float *mean_out) {
    const int64_t quads = (d + 3) / 4;
    const int slots = quads <= 128 ? (int)(256 / quads) : 1;
    const int64_t grid_x = slots > 1 ? 1 : (quads + 255) / 256;
    const int64_t want = std::max<int64_t>(1, std::min<int64_t>((n + 8 * slots - 1) / (8 * slots),
                                                                (4 * (int64_t)h->num_cu + grid_x - 1) / grid_x));
    const int64_t chunk_rows = (n + want - 1) / want, chunks = (n + chunk_rows - 1) / chunk_rows;
    const int form = row_form((d % 4 == 0 && reinterpret_cast<uintptr_t>(rows) % 16 == 0) ? 4 : 1, d);
    if (chunks > 1) {  // (a few times the elements that fill the chip; long rows are one chunk and need none)
        const int rc = ensure(h, h->mean_ws, h->mean_cap, chunks * d);
        if (rc) return rc;
    }
    by_row_form(form, [&](auto vw) {
        constexpr int VW = decltype(vw)::value;
        auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3((unsigned)grid_x, (unsigned)chunks), dim3(256), 0, h->stream, rows, n, d,
                               quads, slots, chunk_rows, h->mean_ws, mean_out);
        };
        if (chunks > 1) launch(column_sums<VW, false>);
        else launch(column_sums<VW, true>);
    });
    if (chunks > 1)
        hipLaunchKernelGGL(column_mean_finish, dim3((unsigned)((d + 15) / 16)), dim3(256), 0, h->stream, h->mean_ws,
                           chunks, n, d, mean_out);
    HIP_TRY(h, hipGetLastError());
    return CDGRAB_OK;
}

}  // namespace

extern "C" {

int cdgrab_create(cdgrab_handle **out, const cdgrab_options *opt) {
    if (!out) return fail(nullptr, CDGRAB_EINVAL, "cdgrab_create: out is NULL");
    *out = nullptr;
    cdgrab_options o{};
    if (opt) o = *opt;
    if (o.block_pairs != 0 && o.block_pairs != 16 && o.block_pairs != 32 && o.block_pairs != 64)
        return fail(nullptr, CDGRAB_EINVAL, "block_pairs must be 0, 16, 32 or 64 (got %d)", o.block_pairs);
    if (o.timing < 0 || o.timing > 2) return fail(nullptr, CDGRAB_EINVAL, "timing must be 0, 1 or 2");
    if (o.pass1_groups < 0 || o.pass1_groups > 65536)
        return fail(nullptr, CDGRAB_EINVAL, "pass1_groups out of range");
    if (o.apply_mode < 0 || o.apply_mode > 4) return fail(nullptr, CDGRAB_EINVAL, "apply_mode must be 0 .. 4");
    if (o.apply_groups < 0 || o.apply_groups > 65536)
        return fail(nullptr, CDGRAB_EINVAL, "apply_groups out of range");
    if (o.gram_mode < 0 || o.gram_mode > 2) return fail(nullptr, CDGRAB_EINVAL, "gram_mode must be 0, 1 or 2");
    int count = 0;
    hipError_t e = hipGetDeviceCount(&count);
    if (e != hipSuccess || o.device < 0 || o.device >= count)
        return fail(nullptr, CDGRAB_EHIP, "no HIP device %d (%d visible): %s", o.device, count,
                    hipGetErrorString(e));
    cdgrab_handle *h = new (std::nothrow) cdgrab_handle();
    if (!h) return fail(nullptr, CDGRAB_ENOMEM, "out of host memory");
    h->device = o.device;
    h->stream = reinterpret_cast<hipStream_t>(o.stream);
    h->block_pairs_opt = o.block_pairs;
    h->timing = o.timing;
    h->pass1_groups_opt = o.pass1_groups;
    h->apply_mode = o.apply_mode;
    h->gram_mode = o.gram_mode;
    h->apply_groups_opt = o.apply_groups;
    hipDeviceProp_t prop;
    if (hipSetDevice(h->device) == hipSuccess && hipGetDeviceProperties(&prop, h->device) == hipSuccess)
        h->num_cu = prop.multiProcessorCount;
    *out = h;
    return CDGRAB_OK;
}

int cdgrab_destroy(cdgrab_handle *h) {
    if (!h) return CDGRAB_OK;
    (void)hipSetDevice(h->device);
    (void)hipStreamSynchronize(h->stream);
    for (hipEvent_t ev : h->event_pool) (void)hipEventDestroy(ev);
    for (hipEvent_t ev : {h->filled, h->balanced[0], h->balanced[1]})
        if (ev) (void)hipEventDestroy(ev);
    if (h->side) (void)hipStreamDestroy(h->side);
    if (h->r_sum) (void)hipFree(h->r_sum);
    if (h->partials) (void)hipFree(h->partials);
    if (h->reduced) (void)hipFree(h->reduced);
    if (h->eps_blk) (void)hipFree(h->eps_blk);
    if (h->flag) (void)hipFree(h->flag);
    if (h->reorder_counts) (void)hipFree(h->reorder_counts);
    if (h->mean_ws) (void)hipFree(h->mean_ws);
    if (h->herd_ws) (void)hipFree(h->herd_ws);
    if (h->herd_steps) (void)hipFree(h->herd_steps);
    if (h->train_delta) (void)hipFree(h->train_delta);
    if (h->train_order) (void)hipFree(h->train_order);
    if (h->train_base) (void)hipFree(h->train_base);
    if (h->train_gram) (void)hipFree(h->train_gram);
    if (h->train_parts) (void)hipFree(h->train_parts);
    if (h->train_perm) (void)hipFree(h->train_perm);
    if (h->train_signs) (void)hipFree(h->train_signs);
    if (h->zero_row) (void)hipFree(h->zero_row);
    if (h->staging) (void)hipFree(h->staging);
    if (h->gram_all) (void)hipFree(h->gram_all);
    if (h->dot_partials) (void)hipFree(h->dot_partials);
    if (h->gram_parts) (void)hipFree(h->gram_parts);
    if (h->bands) (void)hipFree(h->bands);
    if (h->bands_kept) (void)hipFree(h->bands_kept);
    delete h;
    return CDGRAB_OK;
}

const char *cdgrab_last_error(const cdgrab_handle *h) {
    return h ? h->err.c_str() : g_create_error.c_str();
}

int cdgrab_plan_epoch(int64_t m, int64_t n, int64_t d, int32_t block_pairs, int32_t streamed,
                      int64_t base_align, cdgrab_plan *plan) {
    return plan_epoch(m, n, d, block_pairs, streamed, base_align, 256, 0, 0, 0, 0, 1, plan);
}

int cdgrab_pergrad(cdgrab_handle *h, int64_t N, int64_t in_dim, int64_t classes, const float *X,
                   const int32_t *y, const float *W, float *G_out) {
    if (!h) return CDGRAB_EINVAL;
    if (N < 0 || in_dim < 1 || classes < 1 || classes > 1024 || in_dim > (1 << 20))
        return fail(h, CDGRAB_EINVAL, "cdgrab_pergrad: bad sizes N=%lld in_dim=%lld classes=%lld",
                    (long long)N, (long long)in_dim, (long long)classes);
    if (N == 0) return CDGRAB_OK;
    if (!X || !y || !W || !G_out) return fail(h, CDGRAB_EINVAL, "cdgrab_pergrad: null pointer");
    // per-wave staging of one example; fewer wavefronts per workgroup when it is long
    const size_t per_wave = (size_t)(in_dim + 1 + classes) * sizeof(float);
    if (per_wave > 64 * 1024)
        return fail(h, CDGRAB_EINVAL, "cdgrab_pergrad: in_dim + classes too large for LDS staging");
    int waves = kGradWaves;
    while (waves > 1 && waves * per_wave > 64 * 1024) waves >>= 1;
    const size_t lds_waves = waves * per_wave;
    HIP_TRY(h, hipSetDevice(h->device));
    // weights in LDS when they fit beside the per-wave staging (64 KB per workgroup)
    const int wstride = (int)classes | 1;
    const size_t lds_w = (size_t)(in_dim + 1) * (size_t)wstride * sizeof(float);
    const bool wlds = lds_waves + lds_w <= 64 * 1024;
    const size_t lds = lds_waves + (wlds ? lds_w : 0);
    // each wavefront loops over examples: as many workgroups as stay resident
    int64_t per_cu = (int64_t)((160 * 1024) / lds);
    per_cu = std::max<int64_t>(1, std::min<int64_t>(per_cu, 32 / waves));
    int64_t groups = std::min<int64_t>((N + waves - 1) / waves, per_cu * h->num_cu);
    const bool prefetch = in_dim <= 64 * kGradPrefetch;
    auto launch = [&](auto kernel, int stride) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)groups), dim3(waves * 64), lds, h->stream, X, y, W,
                           G_out, N, (int)in_dim, (int)classes, stride);
    };
    if (wlds && prefetch) launch(softmax_pergrad<true, true>, wstride);
    else if (wlds) launch(softmax_pergrad<true, false>, wstride);
    else if (prefetch) launch(softmax_pergrad<false, true>, (int)classes);
    else launch(softmax_pergrad<false, false>, (int)classes);
    HIP_TRY(h, hipGetLastError());
    return CDGRAB_OK;
}

// The herding evaluator keeps the steps' sums over the workers from this many workers on ... Measured, rows read
// twice -> kept: four workers 363 -> 396 us (rows of 100 001 elements), 253 -> 225 (7850), 354 -> 380 (16 384); six
// 362 -> 315, 344 -> 287, 354 -> 296; 32 workers 307 -> 219, 329 -> 226, 292 -> 210; rows of 8 .. 512 elements
// equal up to twelve workers, 100 workers 147 -> 87 (16 elements).
constexpr int64_t kHerdKeepMinWorkers = 6;
constexpr int64_t kHerdKeepBytes = (int64_t)1 << 30;  // ... and up to this size

// The prefix over the segments.  By a workgroup per element where there are few elements: always up to 200 of them
// (400 steps and more of 130 elements 16 - 38 % of the call less than by 64 threads per element, of 200 elements 1 - 23 %),
// up to 512 while segments * elements is small (one worker, 400 steps of 300, 400 and 512 elements 19.8, 21.0 and 22.2 us
// against 23.2, 24.3 and 24.4; 1000 steps 27.8, 32.6 and 39.1 against 31.3, 33.5 and 34.3; 3000 steps 59, 70 and 90 against
// 53, 59 and 61).
constexpr int64_t kHerdScanMaxD = 200, kHerdScanSomeD = 512, kHerdScanEntries = 300000;
bool herding_by_scan(int64_t segments, int64_t d) {
    return d <= kHerdScanMaxD || (d <= kHerdScanSomeD && segments * d <= kHerdScanEntries);
}
// Above, 64 threads share an element where there are many segments, else eight.  A thread that shares an element needs a
// segment of its own, so one thread takes all of fewer than eight (eight threads -> one, whole call: 4 steps of
// 30M elements 1558 -> 695 us, 6 workers x 7 steps of 100 000 32.7 -> 28.5, calls below 20 us equal), and it is the faster
// form up to 24 (one worker: 8 segments of 250 000 elements 57.5 -> 51.8 us, 16 of 150 000 43.5 -> 39.6, 17 of 65 536
// 37.1 -> 34.8, 24 45.3 -> 45.2; 32 54.3 -> 55.6), in three sizes, since it requests all it has room for (10 of
// 100 001 in room for 24 36.8 us, for 16 33.3).
constexpr int64_t kHerdManySegments = 160;
constexpr int kHerdFewSegments = 24;

// Dispatch on the block size, which is a template parameter of the launch helpers.
#define BY_BLOCK_PAIRS(bb, call64, call32, call16) ((bb) == 64 ? (call64) : (bb) == 32 ? (call32) : (call16))

namespace {

// One epoch's state: what the caller gave, the plan, the launch form chosen, and the
// row map of the current and of the previous block.
struct Epoch {
    cdgrab_handle *h;
    int64_t m, n, d;
    const float *grads;        // dense input, or null: rows come from gen
    cdgrab_gen_fn gen;
    void *gen_ctx;
    int64_t chunk_pairs;       // flattened pairs staged per generator call
    const float *center_row;   // dense, m == 1: every row is paired with this one
    int8_t *signs_out;
    double *dots_out;
    float *r_out;              // the running sum's exports, or null
    double *r64_out;

    bool streamed = false;
    cdgrab_plan plan{};
    int bb = 0;
    bool fused = false;        // apply inside the next block's dot/Gram launch
    bool ahead = false;        // Gram matrices of a batch of blocks ahead, one launch per block
    ChainPlan chain{};         // its steps
    int64_t staging_chunk = 0; // floats per staging chunk
    int64_t center_off = 0;    // element offset of center_row from grads
    int64_t walks = 1;         // independent walks of this shape run side by side (m == 1, dense, Grams ahead)

    RowMap rm;
    PrevBlock prev;
    bool have_prev = false;
    int64_t steps_run = 0;     // of the Grams-ahead form
    int64_t blocks_run = 0;    // of the other one

    int prepare();
    void set_block(int64_t p0, int64_t nb, const float *stage_base);
    int generate(int64_t first, int64_t count, float *stage_buf);
    int chain_ahead();
    int chain_blocks();
    int apply_last();
};

// Validation, plan, choice of the launch form, workspace.
int Epoch::prepare() {
    if (m < 1 || n < 2 || (n & 1) || d < 1)
        return fail(h, CDGRAB_EINVAL,
                    "cdgrab_balance_epoch: need m>=1, even n>=2, d>=1 (got m=%lld n=%lld d=%lld)",
                    (long long)m, (long long)n, (long long)d);
    if ((grads == nullptr) == (gen == nullptr))
        return fail(h, CDGRAB_EINVAL, "cdgrab_balance_epoch: give exactly one of grads and gen");
    if (n > INT32_MAX) return fail(h, CDGRAB_EINVAL, "cdgrab_balance_epoch: n exceeds int32 range");
    HIP_TRY(h, hipSetDevice(h->device));

    streamed = grads == nullptr;
    int64_t align = 16;
    if (!streamed) {
        uintptr_t a = reinterpret_cast<uintptr_t>(grads);
        if (center_row) a |= reinterpret_cast<uintptr_t>(center_row);
        align = (a % 16 == 0) ? 16 : (a % 8 == 0) ? 8 : 4;
        if (a % 4) return fail(h, CDGRAB_EINVAL, "cdgrab_balance_epoch: grads is not 4-byte aligned");
    }
    // (One workgroup adds all d / kStepElems shares of a step's dots in the Grams-ahead form, and its
    // Gram tiles are bound by double MFMA work, not bytes: hence refused for long rows.)
    if (h->gram_mode == 2 && !streamed && d > kGramAheadLimitD)
        return fail(h, CDGRAB_EINVAL, "cdgrab_balance_epoch: gram_mode 2 is for rows up to %lld elements (d=%lld)",
                    (long long)kGramAheadLimitD, (long long)d);
    int rc = plan_epoch(m, n, d, h->block_pairs_opt, streamed, align, h->num_cu, h->pass1_groups_opt,
                        h->apply_mode, h->gram_mode, chunk_pairs, walks, &plan);
    if (rc != CDGRAB_OK) return fail(h, rc, "cdgrab_balance_epoch: sizes overflow or are invalid");
    bb = plan.block_pairs;
    if (chunk_pairs <= 0) chunk_pairs = bb;
    staging_chunk = chunk_pairs * 2 * d;
    fused = plan.fused_apply != 0;
    ahead = plan.gram_ahead != 0;
    if (ahead) chain = plan_chain(plan.pairs, d, walks, streamed ? chunk_pairs : 0, h->num_cu);

    // workspace (per walk when several independent walks run side by side)
    const int64_t r_pad = round_up(d, kPadE);
    if (walks > 1 && !(ahead && !streamed && !center_row && m == 1))
        return fail(h, CDGRAB_EINVAL, "several walks per launch need dense short rows (the Grams-ahead form)");
    int64_t fixed_cap = 0;
    rc = ensure(h, h->r_sum, h->r_cap, walks * r_pad);
    if (rc) return rc;
    rc = ensure(h, h->partials, h->partials_cap, (int64_t)plan.pass1_groups * part_size(bb));
    if (rc) return rc;
    if (!h->reduced) { fixed_cap = 0; rc = ensure(h, h->reduced, fixed_cap, (int64_t)kReduceSlices * PartLayout<64>::PART); if (rc) return rc; }
    rc = ensure(h, h->eps_blk, h->eps_cap, ahead ? walks * kMaxStepPairs : (int64_t)kMaxBlockPairs);
    if (rc) return rc;
    if (streamed) {
        // (two chunks: the previous one's rows must outlive the next fill)
        rc = ensure(h, h->staging, h->staging_cap, staging_chunks(plan.pairs, chunk_pairs, fused || ahead) * staging_chunk);
        if (rc) return rc;
    }
    h->ws = WalkStrides{};
    if (ahead) {
        if (chain.band_pairs > 0 && !bands_room(h, chain.bands_len)) chain.band_pairs = 0;
        if (chain.gram_len > 0 && (rc = ensure(h, h->gram_all, h->gram_all_cap, chain.gram_len))) return rc;
        if (chain.parts_len > 0 && (rc = ensure(h, h->gram_parts, h->gram_parts_cap, chain.parts_len))) return rc;
        if (chain.dots_len > 0 && (rc = ensure(h, h->dot_partials, h->dot_partials_cap, chain.dots_len))) return rc;
        if (walks > 1) {
            h->ws.rows = n * d;
            h->ws.r = r_pad;
            h->ws.dots = chain.groups * (int64_t)chain.sp;
            h->ws.out = n / 2;
        }
    }
    h->walks = walks;

    center_off = center_row ? (int64_t)((reinterpret_cast<intptr_t>(center_row) - reinterpret_cast<intptr_t>(grads)) /
                                        (intptr_t)sizeof(float))
                            : 0;
    rm.d = d; rm.m = (int32_t)m; rm.n = n;
    rm.k0 = 0; rm.i0 = 0; rm.nb = 0;
    // (a copy of this map stands in for "no previous block": its rows must be readable)
    rm.base = streamed ? h->staging : grads;
    for (int64_t &o : rm.off) o = 0;
    prev.eps = h->eps_blk;
    prev.rm = rm;
    have_prev = false;
    return CDGRAB_OK;
}

// Row offsets of the block of flattened pairs p0 .. p0+nb-1 (dense input), or of a
// staging chunk's rows [2 q], [2 q + 1] starting at stage_base.
void Epoch::set_block(int64_t p0, int64_t nb, const float *stage_base) {
    rm.k0 = p0 / m;
    rm.i0 = (int32_t)(p0 - rm.k0 * m);
    rm.nb = (int32_t)nb;
    if (stage_base) rm.base = stage_base;
    for (int j = 0; j < rm.nb; ++j) {
        if (stage_base) {
            rm.off[2 * j] = (int64_t)(2 * j) * d;
        } else if (center_row) {
            rm.off[2 * j] = (p0 + j) * d;
            rm.off[2 * j + 1] = center_off;
            continue;
        } else {
            const int64_t p = p0 + j, k = p / m, i = p - k * m;
            rm.off[2 * j] = (i * n + 2 * k) * d;
        }
        rm.off[2 * j + 1] = rm.off[2 * j] + d;
    }
    // The kernels read the table without a branch, also for pairs the block does not have:
    // those entries point at the block's first row, which is always readable (an entry left
    // over from an earlier, fuller block could point past the end of a staging chunk).
    for (int j = rm.nb; j < kMaxBlockPairs; ++j) rm.off[2 * j] = rm.off[2 * j + 1] = 0;
}

int Epoch::generate(int64_t first, int64_t count, float *stage_buf) {
    MARK(h, 1, kGen);
    const int grc = gen(gen_ctx, first, count, stage_buf, h->stream);
    if (grc != 0)
        return fail(h, CDGRAB_EGEN, "generator callback returned %d at pair %lld", grc, (long long)first);
    return CDGRAB_OK;
}

// A training epoch's chunks are generated by a chain of small launches (one workgroup solves the steps), and balanced by
// another one, which needs the rows but not the other way round: while chunk k + 1 is generated, chunk k is balanced on a
// second stream.  16 workers x 1000 steps of 784 -> 10: 3948 -> 3462 us (the training launches alone are
// 2750; the Gram launch of a chunk holds them up).  All of it is ordered before
// whatever follows the call on the handle's stream, however the call ends.
struct Beside {
    cdgrab_handle *h;
    hipStream_t main;
    bool on = false, open = false;

    explicit Beside(cdgrab_handle *handle, bool wanted) : h(handle), main(handle->stream) {
        if (!wanted) return;
        const auto event = [](hipEvent_t &ev) { return ev || hipEventCreateWithFlags(&ev, hipEventDisableTiming) == hipSuccess; };
        on = (h->side || hipStreamCreateWithFlags(&h->side, hipStreamNonBlocking) == hipSuccess) && event(h->filled) &&
             event(h->balanced[0]) && event(h->balanced[1]);
        if (!on) (void)hipGetLastError();
    }
    // The chunk's buffer is free: the chunk two before it has been balanced.
    int before_fill(int64_t chunk) {
        if (on && chunk >= 2) HIP_TRY(h, hipStreamWaitEvent(main, h->balanced[chunk & 1], 0));
        return CDGRAB_OK;
    }
    int enter() {
        if (!on) return CDGRAB_OK;
        HIP_TRY(h, hipEventRecord(h->filled, main));
        HIP_TRY(h, hipStreamWaitEvent(h->side, h->filled, 0));
        h->stream = h->side;
        open = true;
        return CDGRAB_OK;
    }
    int leave(int64_t chunk) {
        if (!on) return CDGRAB_OK;
        h->stream = main;
        HIP_TRY(h, hipEventRecord(h->balanced[chunk & 1], h->side));
        return CDGRAB_OK;
    }
    ~Beside() {
        h->stream = main;
        if (!open) return;
        if (hipEventRecord(h->filled, h->side) != hipSuccess || hipStreamWaitEvent(main, h->filled, 0) != hipSuccess)
            (void)hipStreamSynchronize(h->side);
    }
};

// Gram tiles of a batch of steps in one launch, then two launches per step; the step before is
// applied in the first of them.
int Epoch::chain_ahead() {
    const int form = row_form(plan.vector_width, d);
    const bool narrow = d <= kNarrowMaxD;
    const int64_t batch_pairs = streamed ? chunk_pairs : narrow ? plan.pairs : chain.steps * chain.sp;
    StepRows prev_step{}, none{};
    none.d = d;
    int64_t batch_index = 0;
    bool fresh = true;  // nothing has been applied yet
    int rc = CDGRAB_OK;
    {
    Beside beside(h, streamed && plan.pairs > batch_pairs && h->timing == 0 && !capturing(h));
    for (int64_t first = 0; first < plan.pairs; first += batch_pairs, ++batch_index) {
        const int64_t pairs = std::min(batch_pairs, plan.pairs - first);
        float *stage_buf = streamed ? h->staging + (batch_index & 1) * staging_chunk : nullptr;
        if ((rc = beside.before_fill(batch_index))) return rc;
        if (streamed && (rc = generate(first, pairs, stage_buf))) return rc;
        if ((rc = beside.enter())) return rc;
        MARK(h, 1, kBalance);
        StepRows rows{};
        rows.base = streamed ? stage_buf : center_row ? grads + first * d : grads;
        rows.centre = center_row;
        rows.d = d;
        rows.n = n;
        rows.k0 = first / m;
        rows.i0 = (int32_t)(first % m);
        rows.m = (int32_t)m;
        rows.layout = streamed ? kStaged : center_row ? kCentred : kDense;
        if (narrow) {
            // (every launch exports what it has: the last one's stays)
            if ((rc = run_narrow(h, rows, first, pairs, n / 2, chain, signs_out, dots_out, r_out, r64_out))) return rc;
            steps_run += (pairs + chain.sp - 1) / chain.sp;
            if ((rc = beside.leave(batch_index))) return rc;
            continue;
        }
        // (a chunk of streamed pairs may hold more steps than one launch of Gram tiles)
        for (int64_t at = 0; at < pairs; at += chain.steps * chain.sp) {
            const int64_t count = std::min<int64_t>(chain.steps * chain.sp, pairs - at);
            const StepRows part = step_at(rows, at, 0);
            if ((rc = run_step_grams(h, part, count, chain, form))) return rc;
            const int64_t steps = (count + chain.sp - 1) / chain.sp;
            steps_run += steps;
            h->ws.gram = walks > 1 ? steps * chain.tiles * kTileEntries : 0;
            for (int64_t s = 0; s < steps; ++s) {
                StepRows cur = step_at(part, s * chain.sp, (int)std::min<int64_t>(chain.sp, count - s * chain.sp));
                const bool has_prev = prev_step.nb > 0 || !fresh;  // (a running sum to take dots with)
                if (has_prev) {
                    if ((rc = run_step_wide(h, cur, prev_step, chain, form, fresh, nullptr, nullptr))) return rc;
                    fresh = false;
                }
                // (output slots are counted from the flattened pair, whatever the layout)
                cur.k0 = (first + at + s * chain.sp) / m;
                cur.i0 = (int32_t)((first + at + s * chain.sp) % m);
                const int64_t after = (s + 1) * chain.sp;
                const StepRows next = after < count ? step_at(part, after, (int)std::min<int64_t>(chain.sp, count - after)) : none;
                if ((rc = run_step_walk(h, cur, next, chain, h->gram_all + s * chain.tiles * kTileEntries,
                                        has_prev ? chain.groups : 0, n / 2, signs_out, dots_out))) return rc;
                prev_step = cur;
            }
        }
        if (beside.on && first + pairs < plan.pairs) {  // (its last step too, so that its rows can be overwritten)
            if ((rc = run_step_wide(h, none, prev_step, chain, form, fresh, nullptr, nullptr))) return rc;
            fresh = false;
            prev_step.nb = 0;
        }
        if ((rc = beside.leave(batch_index))) return rc;
    }
    }
    if (narrow) return CDGRAB_OK;
    if (!r_out && !r64_out) return CDGRAB_OK;  // the last step would be applied for nobody
    MARK(h, 1, kBalance);
    return run_step_wide(h, none, prev_step, chain, form, fresh, r_out, r64_out);
}

// Block by block: dot/Gram launch (with the previous block's apply inside it when
// fused), reduction, resolver, and the apply launch when it is not fused.
int Epoch::chain_blocks() {
    const int64_t chunk = streamed ? chunk_pairs : plan.pairs;
    int64_t chunk_index = 0;
    int rc = CDGRAB_OK;
    for (int64_t first = 0; first < plan.pairs; first += chunk, ++chunk_index) {
        const int64_t cnt = std::min<int64_t>(chunk, plan.pairs - first);
        // with the fused pass the previous block's rows must outlive this chunk's staging
        float *stage_buf = h->staging + ((fused && (chunk_index & 1)) ? staging_chunk : 0);
        if (streamed && (rc = generate(first, cnt, stage_buf))) return rc;
        for (int64_t p0 = first; p0 < first + cnt; p0 += bb) {
            set_block(p0, std::min<int64_t>(bb, first + cnt - p0), streamed ? stage_buf + (p0 - first) * 2 * d : nullptr);
            MARK(h, 1, kBalance);
            const PrevBlock *pp = (fused && have_prev) ? &prev : nullptr;
            // A last block of at most 16 pairs in the 16-pair kernels: the 32-pair ones would spend the
            // double MFMA time of three Gram tiles on pairs that do not exist, more than the rows take to
            // read (40 pairs at d = 124M, 8 of them in the last block: 17.8 against 15.1 ms per epoch).
            // Same sums in the same order.
            const int kb = (!fused && bb == 32 && rm.nb <= 16) ? 16 : bb;
            // (fused: the launch of the epoch's second block is the first to write the running sum)
            const bool fresh = blocks_run < (fused ? 2 : 1);
            const SumEnds ends{fresh ? 1 : 0, p0 + rm.nb == plan.pairs ? 1 : 0, r_out, r64_out};
            const SumEnds *now = fused ? nullptr : &ends;
            rc = BY_BLOCK_PAIRS(kb, run_block_vw<64>(h, rm, pp, fresh, now, plan, signs_out, dots_out),
                                run_block_vw<32>(h, rm, pp, fresh, now, plan, signs_out, dots_out),
                                run_block_vw<16>(h, rm, pp, fresh, now, plan, signs_out, dots_out));
            if (rc) return rc;
            ++blocks_run;
            prev.rm = rm;
            have_prev = true;
        }
    }
    return CDGRAB_OK;
}

// The epoch's last block has no successor to apply it.
int Epoch::apply_last() {
    if (!fused || !have_prev) return CDGRAB_OK;
    MARK(h, 1, kBalance);
    const SumEnds ends{blocks_run < 2 ? 1 : 0, 1, r_out, r64_out};
    return BY_BLOCK_PAIRS(bb, apply_block_vw<64>(h, prev.rm, ends, plan), apply_block_vw<32>(h, prev.rm, ends, plan),
                          apply_block_vw<16>(h, prev.rm, ends, plan));
}

}  // namespace

// One epoch.  With a generator, `chunk_pairs` flattened pairs are staged per callback
// (0 = one block) and balanced block by block out of the staging buffer.
// With `center_row` (dense input, m == 1) every row j is paired with that one row
// instead of with its neighbour: "pair" j is (row j, center_row), n pairs in all, and
// the permutation is left to the caller (perm_out may be null).
static int balance_epoch_impl(cdgrab_handle *h, int64_t m, int64_t n, int64_t d, const float *grads,
                              cdgrab_gen_fn gen, void *gen_ctx, int64_t chunk_pairs,
                              const int32_t *perm_in, int8_t *signs_out, int32_t *perm_out,
                              float *r_out, double *r64_out, double *dots_out,
                              const float *center_row = nullptr, int64_t walks = 1) {
    if (!h) return CDGRAB_EINVAL;
    if (!signs_out || (!perm_out && !center_row))
        return fail(h, CDGRAB_EINVAL, "cdgrab_balance_epoch: signs_out and perm_out are required");
    Epoch ep{h, m, n, d, grads, gen, gen_ctx, chunk_pairs, center_row, signs_out, dots_out, r_out, r64_out};
    ep.walks = walks;
    int rc = ep.prepare();
    if (rc) return rc;
    // the permutation kernel reads perm_in while other threads write perm_out
    if (ranges_overlap(perm_in, walks * m * n * 4, perm_out, walks * m * n * 4))
        return fail(h, CDGRAB_EINVAL, "cdgrab_balance_epoch: perm_in and perm_out must not overlap");

    h->marks.clear();
    h->events_used = 0;
    h->have_timing = false;
    rc = ep.ahead ? ep.chain_ahead() : ep.chain_blocks();
    if (rc) return rc;
    rc = ep.apply_last();
    if (rc) return rc;

    MARK(h, 1, kFinish);
    if (!center_row)  // (side-by-side walks are one-worker walks: `walks` rows of signs and orders)
        hipLaunchKernelGGL(build_pair_permutations, dim3((unsigned)((walks * m * (n / 2) + 255) / 256)), dim3(256),
                           0, h->stream, signs_out, perm_in, perm_out, walks * m, n);
    MARK(h, 1, -1);
    HIP_TRY(h, hipGetLastError());
    const int64_t cp = ep.chunk_pairs, bb = ep.bb;
    h->last = cdgrab_timing{};
    if (ep.ahead) {
        h->last.blocks = ep.steps_run;
        h->last.block_pairs = ep.chain.sp;
    } else {
        h->last.blocks = ep.streamed ? ((ep.plan.pairs / cp) * ((cp + bb - 1) / bb) + ((ep.plan.pairs % cp) + bb - 1) / bb)
                                     : ep.plan.blocks;
        h->last.block_pairs = (int32_t)bb;
    }
    h->last.pass1_groups = ep.plan.pass1_groups;
    h->have_timing = h->timing >= 1;
    h->walks = 1;
    h->ws = WalkStrides{};
    return CDGRAB_OK;
}

int cdgrab_balance_epoch(cdgrab_handle *h, int64_t m, int64_t n, int64_t d, const float *grads,
                         cdgrab_gen_fn gen, void *gen_ctx, const int32_t *perm_in,
                         int8_t *signs_out, int32_t *perm_out, float *r_out, double *r64_out,
                         double *dots_out) {
    return balance_epoch_impl(h, m, n, d, grads, gen, gen_ctx, 0, perm_in, signs_out, perm_out, r_out,
                              r64_out, dots_out);
}

// ---- the epoch on a static workspace (for callers that cannot allocate) -------------
namespace {

// Workspace of cdgrab_balance_epoch_static, in doubles: the running sum, the per-workgroup
// partials of the dot/Gram pass, the slice sums of the reduction, and the block's signs.
constexpr int64_t kStaticMaxD = CDGRAB_STATIC_MAX_D;
constexpr int kStaticGroups = 128;  // workgroups of the dot/Gram pass at most
constexpr int64_t kStaticRsum = kStaticMaxD;
constexpr int64_t kStaticPartials = (int64_t)kStaticGroups * PartLayout<64>::PART;
constexpr int64_t kStaticReduced = (int64_t)kReduceSlices * PartLayout<64>::PART;
constexpr int64_t kStaticEps = 64 / 8;
constexpr int64_t kStaticDoubles = kStaticRsum + kStaticPartials + kStaticReduced + kStaticEps;
static_assert(kStaticMaxD % kPadE == 0, "the running sum is padded to whole tiles");

constexpr int kMaxDevices = 64;
double *g_scratch_ptr[kMaxDevices] = {};  // device address of `scratch` on each device, once resolved
std::mutex g_scratch_mutex;

}  // namespace

// Every GPU the library runs on holds its own copy of this array (about 3.9 MB) until the
// process ends.  In host code the name is only a stand-in: its device address comes from
// hipGetSymbolAddress with that device current.
static __device__ __align__(256) double scratch[kStaticDoubles];

namespace {

int static_scratch(cdgrab_handle *h, double **out) {
    if (h->device < 0 || h->device >= kMaxDevices)
        return fail(h, CDGRAB_EINVAL, "cdgrab_balance_epoch_static: device ordinal %d not supported", h->device);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[h->device]) {
        HIP_TRY(h, hipSetDevice(h->device));
        void *ptr = nullptr;
        HIP_TRY(h, hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        if (!ptr) return fail(h, CDGRAB_EHIP, "cdgrab_balance_epoch_static: no device address for the workspace");
        g_scratch_ptr[h->device] = static_cast<double *>(ptr);
    }
    *out = g_scratch_ptr[h->device];
    return CDGRAB_OK;
}

}  // namespace

int cdgrab_balance_epoch_static(cdgrab_handle *h, int64_t m, int64_t n, int64_t d, const float *grads,
                                const int32_t *perm_in, int8_t *signs_out, int32_t *perm_out,
                                float *r_out, double *r64_out, double *dots_out) {
    if (!h) return CDGRAB_EINVAL;
    if (!grads) return fail(h, CDGRAB_EINVAL, "cdgrab_balance_epoch_static: grads is NULL (dense input only)");
    if (d > kStaticMaxD)
        return fail(h, CDGRAB_EINVAL, "cdgrab_balance_epoch_static: d=%lld exceeds the static workspace (at most %lld)",
                    (long long)d, (long long)kStaticMaxD);
    double *base = nullptr;
    int rc = static_scratch(h, &base);
    if (rc) return rc;

    // Borrow the static array as the handle's workspace for this call: the per-block launch
    // form, no timing events, at most kStaticGroups workgroups in the dot/Gram pass.
    struct Saved {
        double *r_sum, *partials, *reduced; int8_t *eps_blk;
        int64_t r_cap, partials_cap, eps_cap; int timing, gram_mode, pass1_groups_opt; bool fixed;
    } sv{h->r_sum, h->partials, h->reduced, h->eps_blk, h->r_cap, h->partials_cap, h->eps_cap,
         h->timing, h->gram_mode, h->pass1_groups_opt, h->fixed_workspace};
    h->r_sum = base;
    h->r_cap = d > 0 ? round_up(d, kPadE) : 0;  // only this much is used
    h->partials = base + kStaticRsum;
    h->partials_cap = kStaticPartials;
    h->reduced = h->partials + kStaticPartials;
    h->eps_blk = reinterpret_cast<int8_t *>(h->reduced + kStaticReduced);
    h->eps_cap = kMaxBlockPairs;
    h->fixed_workspace = true;
    h->timing = 0;
    h->gram_mode = 1;
    h->pass1_groups_opt = (sv.pass1_groups_opt > 0 && sv.pass1_groups_opt < kStaticGroups) ? sv.pass1_groups_opt
                                                                                            : kStaticGroups;
    rc = balance_epoch_impl(h, m, n, d, grads, nullptr, nullptr, 0, perm_in, signs_out, perm_out, r_out,
                            r64_out, dots_out);
    h->r_sum = sv.r_sum; h->partials = sv.partials; h->reduced = sv.reduced; h->eps_blk = sv.eps_blk;
    h->r_cap = sv.r_cap; h->partials_cap = sv.partials_cap; h->eps_cap = sv.eps_cap;
    h->timing = sv.timing; h->gram_mode = sv.gram_mode; h->pass1_groups_opt = sv.pass1_groups_opt;
    h->fixed_workspace = sv.fixed;
    h->have_timing = false;
    return rc;
}

int cdgrab_balance_epoch_randomized(cdgrab_handle *h, int64_t m, int64_t n, int64_t d,
                                    const float *grads, const float *uniforms, const int32_t *perm_in,
                                    int8_t *signs_out, int32_t *perm_out, double *r64_out,
                                    double *dots_out) {
    if (!h) return CDGRAB_EINVAL;
    if (!uniforms) return fail(h, CDGRAB_EINVAL, "cdgrab_balance_epoch_randomized: uniforms is NULL");
    h->uniforms = uniforms;
    int rc = balance_epoch_impl(h, m, n, d, grads, nullptr, nullptr, 0, perm_in, signs_out, perm_out, nullptr,
                                r64_out, dots_out);
    h->uniforms = nullptr;
    return rc;
}

int cdgrab_balance_epoch_stale_mean(cdgrab_handle *h, int64_t n, int64_t d, const float *grads,
                                    const float *stale_mean, const int32_t *perm_in,
                                    int8_t *signs_out, int32_t *perm_out, float *mean_out,
                                    double *r64_out) {
    if (!h) return CDGRAB_EINVAL;
    if (n < 1 || d < 1 || n > INT32_MAX / 2)
        return fail(h, CDGRAB_EINVAL, "cdgrab_balance_epoch_stale_mean: need n>=1, d>=1");
    if (!grads || !signs_out || !perm_out)
        return fail(h, CDGRAB_EINVAL, "cdgrab_balance_epoch_stale_mean: null pointer");
    if (ranges_overlap(perm_in, n * 4, perm_out, n * 4))
        return fail(h, CDGRAB_EINVAL, "cdgrab_balance_epoch_stale_mean: perm_in and perm_out must not overlap");
    if (ranges_overlap(stale_mean, d * 4, mean_out, d * 4))
        return fail(h, CDGRAB_EINVAL, "cdgrab_balance_epoch_stale_mean: stale_mean and mean_out must not overlap");
    HIP_TRY(h, hipSetDevice(h->device));
    int rc = CDGRAB_OK;
    if (!stale_mean) {
        rc = ensure(h, h->zero_row, h->zero_row_cap, d);
        if (rc) return rc;
        hipLaunchKernelGGL(fill_zero_b32, dim3((unsigned)std::min<int64_t>(4096, (d + 255) / 256)), dim3(256), 0,
                           h->stream, reinterpret_cast<uint32_t *>(h->zero_row), d);
        stale_mean = h->zero_row;
    }
    if (!h->flag) { int64_t cap = 0; rc = ensure(h, h->flag, cap, (int64_t)1); if (rc) return rc; }
    // single vectors as pairs (g_j, stale mean): the pair walk then balances
    // mean - g_j = -z_j and its exported sign is minus the sign of z_j, ties included
    rc = balance_epoch_impl(h, 1, 2 * n, d, grads, nullptr, nullptr, 0, nullptr, signs_out, nullptr, nullptr,
                            r64_out, nullptr, stale_mean);
    if (rc) return rc;
    hipLaunchKernelGGL(negate_signs, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, h->stream, signs_out, n);
    hipLaunchKernelGGL(fill_zero_b32, dim3(1), dim3(64), 0, h->stream, reinterpret_cast<uint32_t *>(h->flag), (int64_t)1);
    if ((rc = launch_reorder(h, 1, n, signs_out, perm_in, perm_out))) return rc;
    return mean_out ? launch_column_mean(h, n, d, grads, mean_out) : CDGRAB_OK;
}

int cdgrab_balance_epoch_independent(cdgrab_handle *h, int64_t m, int64_t n, int64_t d,
                                     const float *grads, const int32_t *perm_in, int8_t *signs_out,
                                     int32_t *perm_out) {
    if (!h) return CDGRAB_EINVAL;
    if (m < 1) return fail(h, CDGRAB_EINVAL, "cdgrab_balance_epoch_independent: need m>=1");
    if (!grads || !signs_out || !perm_out)
        return fail(h, CDGRAB_EINVAL, "cdgrab_balance_epoch_independent: null pointer");
    if (n < 2 || (n & 1) || d < 1 || m > (INT64_MAX / n) / d)
        return fail(h, CDGRAB_EINVAL, "cdgrab_balance_epoch_independent: need even n >= 2, d >= 1");
    // Short rows (the Grams-ahead form): the m one-worker walks run side by side, the worker
    // as a grid coordinate, each on its own running sum -- every launch of the chain serves all
    // workers.  The sums are those of a one-worker epoch, perhaps in another order: the length of a step and the
    // shares of a Gram tile go by the number of walks too, and with rows of at most kNarrowMaxD elements the form of
    // the walk and the pairs of a launch.  (A worker's rows start n*d floats after the previous
    // worker's: as aligned as the first worker's whenever d suits the load width.)
    if (m > 1 && m <= 65535) {
        const uintptr_t a = reinterpret_cast<uintptr_t>(grads);
        cdgrab_plan one{};
        const int prc = plan_epoch(1, n, d, h->block_pairs_opt, 0, (a % 16 == 0) ? 16 : (a % 8 == 0) ? 8 : 4,
                                   h->num_cu, h->pass1_groups_opt, h->apply_mode, h->gram_mode, 0, m, &one);
        if (prc == CDGRAB_OK && one.gram_ahead)
            return balance_epoch_impl(h, 1, n, d, grads, nullptr, nullptr, 0, perm_in, signs_out, perm_out,
                                      nullptr, nullptr, nullptr, nullptr, m);
    }
    // long rows: m separate one-worker epochs, each bound by bytes, not by launches
    for (int64_t i = 0; i < m; ++i) {
        int rc = balance_epoch_impl(h, 1, n, d, grads + i * n * d, nullptr, nullptr, 0,
                                    perm_in ? perm_in + i * n : nullptr, signs_out + i * (n / 2),
                                    perm_out + i * n, nullptr, nullptr, nullptr);
        if (rc) return rc;
    }
    return CDGRAB_OK;
}

namespace {
// State of the internal generator of cdgrab_train_epoch_softmax: it produces the rows
// of a chunk of whole step pairs by running the workers' steps at the evolving weights.
struct TrainCtx {
    cdgrab_handle *h;
    int64_t m, n, in_dim, classes, d;
    const float *X; const int32_t *y; const int32_t *perm_in;
    float *W, *velocity, *grads_out, *loss_out;
    float lr, momentum;
    int64_t block_steps;  // steps per block of train_kernels.hpp; 0: a launch pair per step
    int tiles, ksplit;    // Gram tiles per block of steps, workgroups per tile
};

// Workers and classes that the blocks of steps are for: at least four steps per block and one MFMA column
// tile of classes.  (16 workers, 784 -> 10: 2.6 us per step against 11.6 in a launch pair per step; 64
// workers, whose blocks are four steps: 0.56 - 0.69 of the launch pairs' time at 784 .. 2000 -> 2 .. 8.)
int64_t train_block_steps(int64_t m, int64_t n, int64_t classes) {
    const bool fits = m <= kSolveWorkers && classes <= kSolveClasses && n <= INT32_MAX / m;
    return fits ? std::min<int64_t>((kSolveExamples / m) & ~(int64_t)1, n) : 0;
}

// A block of fewer steps than this goes as launch pairs: its logits read all weights once per example, which
// few steps do not repay.  Measured, time of an epoch of one block against its launch pairs (16 workers):
// two steps 1.02 - 1.27 at 31 .. 784 features, 1.2 - 2.45 at 2000 .. 200 000; four steps 0.58 - 1.01 up to 2000
// features and 0.8 - 0.97 beyond with more than eight classes, but 1.0 - 1.8 with 2 .. 8; six steps of those
// 0.74 - 0.96, but 1.1 - 1.3 with four classes and 50 000 features or more; eight 0.58 - 0.95.  With more than
// 32 workers a launch pair takes longer and four steps 0.72 - 0.84 (64 workers, 5000 -> 2).
int64_t train_least_steps(int64_t m, int64_t in_dim, int64_t classes) {
    if (m > 32 || in_dim <= 2048 || classes == 1 || classes > 8) return 4;
    return in_dim > 32768 && classes <= 4 ? 8 : 6;
}

// Flattened pairs staged at a time: whole step pairs, about 64 pairs; for short rows about 1024 pairs, so that
// the Gram tiles of a chunk come from one launch.  There whole steps of the chain are preferred (a ragged
// last one per chunk costs up to 6 %), but whole step pairs and whole steps at once can be many pairs
// (14 080 for 11 workers), so a chunk is held to what the last-level cache holds, 256 MB, or to 1024 pairs,
// and to the epoch.
int64_t train_chunk_pairs(const cdgrab_handle *h, int64_t m, int64_t n, int64_t d) {
    const int64_t pairs = m * (n / 2), bb = pick_block_pairs(pairs, d, h->block_pairs_opt);
    const int64_t base = std::max<int64_t>(1, 64 / m) * m;
    int64_t k = 1;
    if (d <= kChunkAheadMaxD && h->gram_mode != 1 && h->apply_mode == 0) {
        const int64_t sp = plan_chain(pairs, d, 1, 0, h->num_cu).sp;
        k = sp / std::gcd(base, sp);
        k *= std::max<int64_t>(1, 1024 / (base * k));
        k = std::min(k, std::max<int64_t>(1024 / base, ((int64_t)1 << 28) / (2 * d * 4) / base));
        k = std::max<int64_t>(1, std::min(k, kGramBatch * bb / base));
    }
    return std::min(base * k, pairs);
}

// The steps j .. j_end - 1 of a chunk, a launch pair each.
int train_step_launches(TrainCtx *c, int64_t j, int64_t j_end, int64_t k_first, float *staging) {
    cdgrab_handle *h = c->h;
    const size_t lds = (size_t)c->classes * sizeof(float);
    for (; j < j_end; ++j) {
        hipLaunchKernelGGL(train_step_delta, dim3((unsigned)c->m), dim3(kDeltaWaves * 64), lds, h->stream, c->X, c->y,
                           c->perm_in, c->W, h->train_delta, c->loss_out, c->m, c->n, j, (int)c->in_dim,
                           (int)c->classes);
        auto update = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3((unsigned)((c->d + 255) / 256)), dim3(256), 0, h->stream, c->X, c->perm_in,
                               h->train_delta, c->W, c->velocity, staging, c->grads_out, c->m, c->n, j, k_first,
                               (int)c->in_dim, (int)c->classes, c->lr, c->momentum);
        };
        if (c->perm_in) update(train_step_update<true>);
        else update(train_step_update<false>);
    }
    HIP_TRY(h, hipGetLastError());
    return CDGRAB_OK;
}

// The steps j .. j_end - 1 of a chunk, a block at a time; what is left for less than a shortest block, as above.
int train_blocks(TrainCtx *c, int64_t j, int64_t j_end, int64_t k_first, float *staging) {
    cdgrab_handle *h = c->h;
    const int64_t S = c->block_steps, m = c->m, d = c->in_dim, least = train_least_steps(c->m, c->in_dim, c->classes);
    const int64_t rest = (j_end - j) % S, j_blocks = rest < least ? j_end - rest : j_end;
    if (j == j_blocks) return train_step_launches(c, j, j_end, k_first, staging);
    GramBatch gb{};
    gb.rows.base = c->X;
    gb.rows.d = d;
    gb.rows.m = 1;
    gb.rows.layout = kStaged;
    gb.examples = h->train_order + j * m;
    gb.pairs = (j_blocks - j) * m;
    gb.sp = (int32_t)(S * m);
    gb.steps = gb.units = (int32_t)((j_blocks - j + S - 1) / S);
    gb.tiles = c->tiles;
    gb.ksplit = c->ksplit;
    gb.ktiles = (int32_t)((d + kGramTE - 1) / kGramTE);
    const int form = row_form((d % 4 == 0 && reinterpret_cast<uintptr_t>(c->X) % 16 == 0) ? 4 : 1, d);
    const int rc = run_gram_tiles<true>(h, gb, h->train_gram, h->train_parts, form);
    if (rc) return rc;
    const int64_t update_blocks = (c->d + 63) / 64, update_groups = update_blocks >= 16 ? round_up(update_blocks, 8) : update_blocks;
    for (int64_t b = 0; b < gb.units; ++b, j += S) {
        const int steps = (int)std::min(S, j_blocks - j), examples = (int)(steps * m);
        const int64_t *order = h->train_order + j * m;
        hipLaunchKernelGGL(train_base_logits, dim3((unsigned)examples), dim3(512), 0, h->stream, c->X, order, c->W, c->velocity, (int)d, (int)c->classes, h->train_base);
        auto solve = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(1), dim3(kSolveThreads), 0, h->stream, h->train_gram + b * gb.tiles * kTileEntries,
                               h->train_base, c->y, order, h->train_delta, c->loss_out, (int)m, steps, c->n, j,
                               (int)c->classes, (double)c->lr, (double)c->momentum);
        };
        if (m <= 4) solve(train_solve<1>);
        else if (m <= 8) solve(train_solve<2>);
        else solve(train_solve<4>);
        hipLaunchKernelGGL(train_update_block, dim3((unsigned)update_groups), dim3(1024), 0, h->stream, c->X, order,
                           h->train_delta, c->W, c->velocity, staging, c->grads_out, (int)m, steps, c->n, j, k_first,
                           (int)d, (int)c->classes, c->lr, c->momentum);
    }
    HIP_TRY(h, hipGetLastError());
    return train_step_launches(c, j_blocks, j_end, k_first, staging);
}

int train_generate(void *vctx, int64_t first_pair, int64_t count, float *staging, void *) {
    TrainCtx *c = static_cast<TrainCtx *>(vctx);
    if (first_pair % c->m != 0 || count % c->m != 0) return 1;  // chunks are whole step pairs
    const int64_t k_first = first_pair / c->m, j = 2 * k_first, j_end = j + 2 * (count / c->m);
    return c->block_steps > 0 ? train_blocks(c, j, j_end, k_first, staging)
                              : train_step_launches(c, j, j_end, k_first, staging);
}
}  // namespace

int cdgrab_train_epoch_softmax(cdgrab_handle *h, int64_t m, int64_t n, int64_t in_dim, int64_t classes,
                               const float *X, const int32_t *y, const int32_t *perm_in, float *W,
                               float *velocity, float lr, float momentum, int8_t *signs_out,
                               int32_t *perm_out, float *grads_out, float *loss_out) {
    if (!h) return CDGRAB_EINVAL;
    if (m < 1 || n < 2 || (n & 1) || in_dim < 1 || classes < 1 || classes > 1024 || in_dim > (1 << 20))
        return fail(h, CDGRAB_EINVAL, "cdgrab_train_epoch_softmax: bad sizes");
    if (!X || !y || !W || !signs_out || !perm_out)
        return fail(h, CDGRAB_EINVAL, "cdgrab_train_epoch_softmax: null pointer");
    if (ranges_overlap(perm_in, m * n * 4, perm_out, m * n * 4))
        return fail(h, CDGRAB_EINVAL, "cdgrab_train_epoch_softmax: perm_in and perm_out must not overlap");
    if (momentum != 0.0f && !velocity)
        return fail(h, CDGRAB_EINVAL, "cdgrab_train_epoch_softmax: momentum needs a velocity buffer");
    HIP_TRY(h, hipSetDevice(h->device));
    const int64_t chunk = train_chunk_pairs(h, m, n, (in_dim + 1) * classes);
    int64_t block_steps = std::min(train_block_steps(m, n, classes), 2 * (chunk / m));
    if (block_steps < train_least_steps(m, in_dim, classes)) block_steps = 0;
    int rc = ensure(h, h->train_delta, h->train_delta_cap, block_steps > 0 ? block_steps * m * classes : m * classes);
    if (rc) return rc;
    TrainCtx ctx{h, m, n, in_dim, classes, (in_dim + 1) * classes, X, y, perm_in, W, velocity,
                 grads_out, loss_out, lr, momentum, block_steps, 0, 1};
    if (block_steps > 0) {
        const int64_t blocks = (std::min(2 * (chunk / m), n) + block_steps - 1) / block_steps;  // of a chunk
        const int64_t blk = (block_steps * m + kTilePairs - 1) / kTilePairs;
        ctx.tiles = (int)(blk * (blk + 1) / 2);
        ctx.ksplit = pick_ksplit(blocks * ctx.tiles, in_dim, h->num_cu);
        const int64_t entries = blocks * ctx.tiles * kTileEntries;
        if ((rc = ensure(h, h->train_gram, h->train_gram_cap, entries))) return rc;
        if (ctx.ksplit > 1 && (rc = ensure(h, h->train_parts, h->train_parts_cap, entries * ctx.ksplit))) return rc;
        if ((rc = ensure(h, h->train_order, h->train_order_cap, m * n))) return rc;
        if ((rc = ensure(h, h->train_base, h->train_base_cap, (int64_t)kSolveExamples * 2 * kSolveClasses))) return rc;
        hipLaunchKernelGGL(example_order, dim3((unsigned)((m * n + 255) / 256)), dim3(256), 0, h->stream, perm_in, m, n,
                           h->train_order);
    }
    return balance_epoch_impl(h, m, n, ctx.d, nullptr, train_generate, &ctx, chunk, perm_in,
                              signs_out, perm_out, nullptr, nullptr, nullptr);
}

int cdgrab_train_softmax(cdgrab_handle *h, int64_t m, int64_t n, int64_t in_dim, int64_t classes,
                         const float *X, const int32_t *y, int32_t *perm, float *W, float *velocity,
                         float lr, float momentum, int64_t epochs, int8_t *signs_out, float *loss_out) {
    if (!h) return CDGRAB_EINVAL;
    if (epochs < 1 || !perm) return fail(h, CDGRAB_EINVAL, "cdgrab_train_softmax: need epochs>=1 and perm");
    if (m < 1 || n < 2 || (n & 1) || m > INT32_MAX || n > INT32_MAX)
        return fail(h, CDGRAB_EINVAL, "cdgrab_train_softmax: bad sizes");
    HIP_TRY(h, hipSetDevice(h->device));
    int rc = ensure(h, h->train_perm, h->train_perm_cap, m * n);
    if (rc) return rc;
    if (!signs_out) {
        rc = ensure(h, h->train_signs, h->train_signs_cap, m * (n / 2));
        if (rc) return rc;
        signs_out = h->train_signs;
    }
    // the order ping-pongs between the caller's buffer and the spare one
    int32_t *cur = perm, *nxt = h->train_perm;
    for (int64_t t = 0; t < epochs; ++t) {
        rc = cdgrab_train_epoch_softmax(h, m, n, in_dim, classes, X, y, cur, W, velocity, lr, momentum,
                                        signs_out, nxt, nullptr, loss_out ? loss_out + t * m * n : nullptr);
        if (rc) return rc;
        std::swap(cur, nxt);
    }
    if (cur != perm)
        HIP_TRY(h, hipMemcpyAsync(perm, cur, (size_t)(m * n) * sizeof(int32_t), hipMemcpyDeviceToDevice,
                                  h->stream));
    return CDGRAB_OK;
}

int cdgrab_reorder(cdgrab_handle *h, int64_t m, int64_t n, const int8_t *signs,
                   const int32_t *perm_in, int32_t *perm_out) {
    if (!h) return CDGRAB_EINVAL;
    if (m < 1 || n < 1 || n > INT32_MAX || m > INT32_MAX)
        return fail(h, CDGRAB_EINVAL, "cdgrab_reorder: need m>=1, n>=1");
    if (!signs || !perm_out) return fail(h, CDGRAB_EINVAL, "cdgrab_reorder: null pointer");
    if (ranges_overlap(perm_in, m * n * 4, perm_out, m * n * 4))
        return fail(h, CDGRAB_EINVAL, "cdgrab_reorder: perm_in and perm_out must not overlap");
    HIP_TRY(h, hipSetDevice(h->device));
    if (!h->flag) { int64_t cap = 0; int rc = ensure(h, h->flag, cap, (int64_t)1); if (rc) return rc; }
    hipLaunchKernelGGL(fill_zero_b32, dim3(1), dim3(64), 0, h->stream, reinterpret_cast<uint32_t *>(h->flag), (int64_t)1);
    const int rc = launch_reorder(h, m, n, signs, perm_in, perm_out);
    if (rc) return rc;
    int32_t bad = 0;
    HIP_TRY(h, hipMemcpyAsync(&bad, h->flag, sizeof bad, hipMemcpyDeviceToHost, h->stream));
    HIP_TRY(h, hipStreamSynchronize(h->stream));
    if (bad) return fail(h, CDGRAB_EINVAL, "cdgrab_reorder: a sign is neither +1 nor -1");
    return CDGRAB_OK;
}

int cdgrab_herding_bound(cdgrab_handle *h, int64_t m, int64_t n, int64_t d, const float *z,
                         const int32_t *perm, double *bound_out) {
    if (!h) return CDGRAB_EINVAL;
    if (m < 1 || n < 1 || d < 1 || m > (INT64_MAX / n) / d)
        return fail(h, CDGRAB_EINVAL, "cdgrab_herding_bound: need m>=1, n>=1, d>=1");
    if (!z || !bound_out) return fail(h, CDGRAB_EINVAL, "cdgrab_herding_bound: null pointer");
    HIP_TRY(h, hipSetDevice(h->device));
    HerdingShape sh;
    sh.m = m; sh.n = n; sh.d = d;
    // enough (segment, four elements) threads to fill the chip, at least one step per segment
    const int64_t quads = (d + 3) / 4;
    sh.quads = (int32_t)std::min<int64_t>(quads, INT32_MAX);
    // short rows: a workgroup serves several segments (thread = (segment, four elements))
    sh.spw = quads <= 128 ? (int32_t)(256 / quads) : 1;
    int64_t want_threads = (int64_t)h->num_cu * 2048;
    // blockIdx.y counts workgroups of spw segments (at most 65 535 of them)
    int64_t segs = std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(n, (int64_t)65535 * sh.spw),
                                                          (want_threads + quads - 1) / quads));
    sh.seg_len = (n + segs - 1) / segs;
    sh.segments = (n + sh.seg_len - 1) / sh.seg_len;
    int rc = ensure(h, h->herd_ws, h->herd_cap, 2 * sh.segments * d + d);
    if (rc) return rc;
    double *segsum = h->herd_ws, *start = segsum + sh.segments * d, *zbar = start + sh.segments * d;
    const dim3 grid(sh.spw == 1 ? (unsigned)((quads + 255) / 256) : 1u,
                    (unsigned)((sh.segments + sh.spw - 1) / sh.spw));
    unsigned long long *bits = reinterpret_cast<unsigned long long *>(bound_out);
    // the segment's example ids go through LDS when they fit (48 KB)
    const size_t ids_bytes = (size_t)(sh.seg_len * m) * sizeof(int32_t);
    const int lds_ids = (perm && sh.spw == 1 && ids_bytes <= 48 * 1024) ? 1 : 0;
    const size_t lds = lds_ids ? ids_bytes : 0;
    const int form = row_form((d % 4 == 0 && reinterpret_cast<uintptr_t>(z) % 16 == 0) ? 4 : 1, d);
    // where the steps' sums are kept for the second pass (and fit), the rows are read once; not in a launch that is
    // recorded, because their buffer is replaced when a later call has more steps
    const bool keep = m >= kHerdKeepMinWorkers && n <= kHerdKeepBytes / 32 / quads && !capturing(h) &&
                      room(h, h->herd_steps, h->herd_steps_cap, n * quads * 4);
    hipLaunchKernelGGL(herding_clear, dim3(1), dim3(1), 0, h->stream, bits);
    auto launch = [&](auto vw_tag) {
        constexpr int VW = decltype(vw_tag)::value;
        auto sums = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, grid, dim3(256), lds, h->stream, z, perm, sh, lds_ids, segsum, h->herd_steps);
        };
        if (keep) sums(herding_segment_sums<VW, true>);
        else sums(herding_segment_sums<VW, false>);
        auto few = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3((unsigned)((d + 255) / 256)), dim3(256), 0, h->stream, segsum, sh, zbar, start);
        };
        if (herding_by_scan(sh.segments, d))
            hipLaunchKernelGGL(herding_segment_offsets_scan, dim3((unsigned)d), dim3(256), 0, h->stream,
                               segsum, sh, zbar, start);
        else if (sh.segments >= kHerdManySegments)
            hipLaunchKernelGGL((herding_segment_offsets<16, 64>), dim3((unsigned)((d + 15) / 16)), dim3(1024), 0,
                               h->stream, segsum, sh, zbar, start);
        else if (sh.segments <= 8)
            few(herding_segment_offsets_few<8>);
        else if (sh.segments <= 16)
            few(herding_segment_offsets_few<16>);
        else if (sh.segments <= kHerdFewSegments)
            few(herding_segment_offsets_few<kHerdFewSegments>);
        else
            hipLaunchKernelGGL((herding_segment_offsets<32, 8>), dim3((unsigned)((d + 31) / 32)), dim3(256), 0,
                               h->stream, segsum, sh, zbar, start);
        auto replay = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, grid, dim3(256), keep ? 0 : lds, h->stream, z, perm, sh, lds_ids, zbar, start,
                               h->herd_steps, bits);
        };
        if (keep) replay(herding_prefix_max<VW, true>);
        else replay(herding_prefix_max<VW, false>);
    };
    if (form == kAligned) launch(std::integral_constant<int, kAligned>{});
    else if (form == kAnyRow) launch(std::integral_constant<int, kAnyRow>{});
    else launch(std::integral_constant<int, kTiny>{});
    HIP_TRY(h, hipGetLastError());
    return CDGRAB_OK;
}

int cdgrab_get_timing(cdgrab_handle *h, cdgrab_timing *out) {
    if (!h || !out) return CDGRAB_EINVAL;
    if (!h->have_timing) return fail(h, CDGRAB_EINVAL, "cdgrab_get_timing: no timed epoch on this handle");
    HIP_TRY(h, hipSetDevice(h->device));
    HIP_TRY(h, hipStreamSynchronize(h->stream));
    double sum[kIntervalKinds] = {0};
    for (size_t q = 0; q + 1 < h->marks.size(); ++q) {
        int kind = h->marks[q].kind_after;
        if (kind < 0) continue;
        float ms = 0.f;
        HIP_TRY(h, hipEventElapsedTime(&ms, h->marks[q].ev, h->marks[q + 1].ev));
        sum[kind] += ms;
    }
    cdgrab_timing t = h->last;
    t.generator_ms = sum[kGen];
    t.pass1_ms = sum[kPass1];
    t.reduce_ms = sum[kReduce];
    t.resolve_ms = sum[kResolve];
    t.pass2_ms = sum[kPass2];
    t.finish_ms = sum[kFinish];
    // with per-kernel marks the balancer interval is split into its four kernels
    t.balance_ms = sum[kBalance] + sum[kPass1] + sum[kReduce] + sum[kResolve] + sum[kPass2];
    h->last = t;
    *out = t;
    return CDGRAB_OK;
}

}  // extern "C"
