// Blocked pair-balancing kernels for gfx950 (CDNA4).
//
// The greedy walk of CD-GraB (App. B.2 "Balancing without normalization" applied
// pair by pair in the server algorithm's order, Sec. 3.3) decides each sign from
// <r, d_k>, where r already contains the earlier differences.  For a block of Bb
// consecutive differences
//     <r + sum_{j<k} eps_j d_j, d_k> = <r, d_k> + sum_{j<k} eps_j <d_j, d_k>,
// so one pass over the rows yields everything the Bb decisions need: the Bb dots
// with the block-start running sum and the Bb x Bb Gram matrix.  A single
// wavefront then resolves the signs in order, and a second pass applies
// r += sum_k eps_k d_k.  Each gradient row is read from HBM twice per epoch.
//
// Arithmetic: rows are fp32; differences are formed in double (exact), dots with
// r are double FMAs, the Gram matrix is accumulated by the double-precision MFMA
// (products of two exact fp32 differences are exact in double), and all
// cross-lane / cross-workgroup sums are taken in a fixed order.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

namespace cdgrab {

constexpr int kThreads = 256;       // workgroup size of the streaming kernels
constexpr int kWaves = kThreads / 64;
constexpr int kPadE = 128;          // the running sum is padded to a multiple of this many elements

typedef double double4_t __attribute__((ext_vector_type(4)));
typedef float float4_t __attribute__((ext_vector_type(4)));

// Where the rows of the current block live: element offsets from `base` of the
// first and second row of each pair, filled in by the host (dense input [m][n][d]:
// flattened pair p belongs to worker p % m and is its pair p / m; a staging block
// is [Bb][2][d]).  Passed by value: uniform indices become scalar loads.
constexpr int kMaxBlockPairs = 64;

struct RowMap {
    const float *base;
    int64_t d;
    int64_t n;
    int64_t k0;     // pair index (per worker) of the block's first flattened pair
    int32_t i0;     // worker of the block's first flattened pair
    int32_t m;
    int32_t nb;     // valid pairs in this block (<= Bb)
    int64_t off[2 * kMaxBlockPairs];  // off[2 j + which]

    __device__ __forceinline__ const float *row(int j, int which) const { return base + off[2 * j + which]; }
};

// How a kernel reads four consecutive elements of a row (template parameter VW):
//   kAligned  every row start is 16-byte aligned and d is a multiple of 4: one 16 B load;
//   kAnyRow   any row start and any d >= 4: still one 16 B load, which needs only the 4-byte
//             alignment every row has; the group that straddles the end of the row takes its
//             elements one at a time (load4) or from the row's last four (load4_nb);
//   kTiny     rows of fewer than four elements: one 4 B load per element.
// One 16 B load per thread instead of four 4 B loads (or two 8 B ones) matters for every row length
// that is not a multiple of 4: the narrow loads of a wave touch each line up to four times.
// Measured, narrow -> one load: 32-pair block at d = 1 048 575 225 -> 125 us (109 us aligned);
// d = 7850 (8-byte aligned): epoch of 30 000 pairs 7.36 -> 6.78 ms, herding objective of its
// 60 000 rows 0.86 -> 0.70 ms.
constexpr int kAligned = 4, kAnyRow = 2, kTiny = 1;

typedef float float4_any __attribute__((ext_vector_type(4), aligned(4)));

// Four consecutive fp32 elements starting at element e of a row, zero beyond d or
// for a missing row.  Rows are read exactly once per pass, so the loads carry the
// non-temporal hint: the streamed rows then do not evict the running sum, which
// is re-read and rewritten every block, from the last-level cache.
// INSIDE: the caller knows that the group lies inside the row (e + 4 <= d).  The apply kernels decide that once
// per thread, because a branch at every load keeps fewer of them in flight (32-pair block in
// separate launches at d = 1 200 001: 197 us, now 142; 124 aligned).  The dot/Gram pass, whose loads have
// a whole tile's time, gains nothing from it.
template <int VW, bool INSIDE = false>
__device__ __forceinline__ float4 load4(const float *row, int64_t e, int64_t d) {
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (row == nullptr) return v;
    if constexpr (VW == kAnyRow && INSIDE) {
        float4_any t = __builtin_nontemporal_load(reinterpret_cast<const float4_any *>(row + e));
        v = make_float4(t.x, t.y, t.z, t.w);
    } else if constexpr (VW == kAligned) {
        if (e < d) {
            float4_t t = __builtin_nontemporal_load(reinterpret_cast<const float4_t *>(row + e));
            v = make_float4(t.x, t.y, t.z, t.w);
        }
    } else {
        if (VW == kAnyRow && e + 4 <= d) {
            float4_any t = __builtin_nontemporal_load(reinterpret_cast<const float4_any *>(row + e));
            v = make_float4(t.x, t.y, t.z, t.w);
        } else {
            if (e < d) v.x = __builtin_nontemporal_load(row + e);
            if (e + 1 < d) v.y = __builtin_nontemporal_load(row + e + 1);
            if (e + 2 < d) v.z = __builtin_nontemporal_load(row + e + 2);
            if (VW == kTiny && e + 3 < d) v.w = __builtin_nontemporal_load(row + e + 3);
        }
    }
    return v;
}

// The same without a branch, for launches that are bound by latency rather than by
// bytes: `row` must be readable at its first elements whether or not `have` is set,
// out-of-range parts read another part of the row instead and are replaced by zero afterwards.
// (A load inside an `if` ends in a wait for it before the next one is issued; with
// straight-line code all loads of a thread are in flight together.)
// NT: with the non-temporal hint (false where the next launch on the same XCD reads the row again).
template <bool NT>
__device__ __forceinline__ float load_one(const float *p) {
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}

template <bool NT>
__device__ __forceinline__ float4_t load_four(const float *p) {  // 4-byte aligned
    const float4_any *q = reinterpret_cast<const float4_any *>(p);
    if constexpr (NT) return __builtin_nontemporal_load(q);
    else return *q;
}

template <int VW, bool NT = true>
__device__ __forceinline__ float4 load4_nb(const float *row, bool have, int64_t e, int64_t d) {
    float4 v;
    if constexpr (VW == kAligned) {
        const bool in = have && e < d;
        const float4_t t = load_four<NT>(row + (in ? e : 0));
        v = make_float4(in ? t.x : 0.f, in ? t.y : 0.f, in ? t.z : 0.f, in ? t.w : 0.f);
    } else if constexpr (VW == kAnyRow) {
        // a group that reaches beyond the row reads the row's last four elements and moves them down
        const int64_t base = e <= d - 4 ? e : d - 4;
        const int sh = have && e - base < 4 ? (int)(e - base) : 4;
        const float4_t t = load_four<NT>(row + base);
        // (in binary steps: a chain of comparisons on sh becomes branches)
        const bool s1 = sh & 1, s2 = sh & 2, s4 = sh & 4;
        const float x1 = s1 ? t.y : t.x, y1 = s1 ? t.z : t.y, z1 = s1 ? t.w : t.z, w1 = s1 ? 0.f : t.w;
        const float x2 = s2 ? z1 : x1, y2 = s2 ? w1 : y1, z2 = s2 ? 0.f : z1, w2 = s2 ? 0.f : w1;
        v = make_float4(s4 ? 0.f : x2, s4 ? 0.f : y2, s4 ? 0.f : z2, s4 ? 0.f : w2);
    } else {
        float o[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const bool in = have && e + q < d;
            const float t = load_one<NT>(row + (in ? e + q : 0));
            o[q] = in ? t : 0.f;
        }
        v = make_float4(o[0], o[1], o[2], o[3]);
    }
    return v;
}

// Number of doubles one workgroup of the dot/Gram pass emits: the Gram tiles in
// the MFMA accumulator layout (tile * 256 + v * 64 + lane) followed by Bb dots.
template <int BB> struct PartLayout {
    static constexpr int RG = BB / 16;               // 16-row groups
    static constexpr int NT = RG * (RG + 1) / 2;     // upper-triangular 16x16 tiles
    static constexpr int GRAM = NT * 256;
    static constexpr int PART = GRAM + BB;
};

// Row / column of accumulator element v of lane `lane` in the 16x16 result of
// v_mfma_f64_16x16x4_f64: column = lane % 16, row = 4 * v + lane / 16
// (measured on gfx950 with a rank-one probe).
__device__ __forceinline__ void mfma_f64_16x16_coord(int lane, int v, int &i, int &j) {
    j = lane & 15;
    i = 4 * v + (lane >> 4);
}

// ---------------------------------------------------------------------------
// Pass 1: partial dots <r, d_k> and partial Gram <d_j, d_k> over a strided set
// of TE-element tiles of d.  One workgroup = 4 waves; each tile is staged
// through LDS (coalesced 16 B global loads -> row-per-lane MFMA operands), with
// the next tile's loads in flight while the current one is consumed.
// Lane (row = lane % 16, kslot = lane / 16) of wave w owns elements
// (TE/4) w + 16 s + 4 kslot .. +3 (s = 0 .. TE/64-1) of the tile for pair `row`
// of each 16-pair group.  TE = 128 halves the barriers per byte and is the
// streaming configuration; TE = 64 gives short rows more workgroups.
//
// With APPLY the same launch first applies the PREVIOUS block to the tile's slice
// of the running sum (r += sum_k eps_k d_k over prev's rows, the work of pass 2):
// every thread adds up the signed rows it loads, the RPI partial sums per element
// are added in row order through LDS, the new slice is written back and is the one
// the current block's dots are taken against.  The running sum is then read once
// and written once per block, and a block costs one streaming launch instead of two.
struct PrevBlock {
    RowMap rm;           // rows of the previous block
    const int8_t *eps;   // its resolved signs
};

// Several independent walks of the same shape in one launch (the uncoordinated baseline:
// every worker balances its own rows on its own running sum).  The walk is a grid
// coordinate; everything a walk owns lies at a fixed element stride from the first walk's.
// All strides are zero for a single walk.
struct WalkStrides {
    int64_t rows;   // floats from walk w's rows to walk w+1's
    int64_t r;      // doubles between running sums
    int64_t gram;   // doubles between the walks' Gram tiles
    int64_t dots;   // doubles between the walks' per-workgroup dots
    int64_t out;    // entries between the walks' slices of signs_out / dots_out
};

// `group` of `ngroups` workgroups share the tiles; the workgroup's result goes to `out`.
// FRESH: the running sum is zero and r_sum holds nothing yet; the launch that takes dots only then clears r_sum beyond d,
// where the apply launches write nothing.  (As a kernel argument, with the padding masked in every launch: the dots of
// 124M elements 5.24 -> 5.31 ms, of 11.2M 0.478 -> 0.479.)
template <int BB, int VW, int TE, bool APPLY, bool FRESH, bool NB>
__device__ __forceinline__ void pass1_body(const RowMap &rm, const PrevBlock &prev, double *__restrict__ r_sum,
                                           double *__restrict__ out, int64_t ntiles, int group, int ngroups)
{
    using L = PartLayout<BB>;
    constexpr int RG = L::RG;
    constexpr int TPR = TE / 4;               // threads covering one row of the tile
    constexpr int RPI = kThreads / TPR;       // rows covered by one load instruction
    constexpr int LOADS = 2 * BB / RPI;       // 16 B loads per thread per tile
    constexpr int STRIDE = TE + 4;            // floats per LDS row (16 B aligned, bank-skewed)
    constexpr int TILE_FLOATS = BB * STRIDE;
    constexpr int EPW = TE / kWaves;          // elements per wave per tile
    // LDS: two stages of (first rows, second rows, running-sum chunk), with APPLY one
    // buffer of RPI partial sums per element; the final cross-wave reduction reuses
    // the same bytes.
    constexpr int STAGE_BYTES = 2 * TILE_FLOATS * 4 + TE * 8;
    constexpr int APPLY_BYTES = APPLY ? RPI * TE * 8 : 0;
    constexpr int RED_BYTES = kWaves * (L::GRAM + RG * 64) * 8;
    constexpr int SMEM = (2 * STAGE_BYTES + APPLY_BYTES > RED_BYTES) ? 2 * STAGE_BYTES + APPLY_BYTES : RED_BYTES;
    __shared__ __attribute__((aligned(16))) unsigned char smem[SMEM];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int64_t d = rm.d;

    const int lrow = tid / TPR;
    const int chunk = tid % TPR;
    const float *src[LOADS];
    const float *psrc[APPLY ? LOADS : 1];
    float psign[APPLY ? LOADS : 1];
    int lds_off[LOADS];
    uint32_t have_mask = 0;  // bit u: load u's pair exists in this block
#pragma unroll
    for (int u = 0; u < LOADS; ++u) {
        int rr = u * RPI + lrow;       // 0 .. 2*BB-1
        int j = rr >> 1, which = rr & 1;
        // the table is read without a branch (entries of missing pairs are readable rows:
        // zero, or those of an earlier block), so that the lookups overlap
        src[u] = rm.row(j, which);
        if (j < rm.nb) have_mask |= 1u << u;
        lds_off[u] = (which * TILE_FLOATS + j * STRIDE + chunk * 4) * 4;
        if constexpr (APPLY) {
            const bool have = j < prev.rm.nb;
            psrc[u] = prev.rm.row(j, which);
            const float ej = (float)prev.eps[j];  // 64 entries, always readable
            // d_k = second - first, so the second row enters with eps and the first with -eps
            // (a missing pair enters with sign 0)
            psign[u] = have ? ej * (which ? 1.0f : -1.0f) : 0.0f;
        }
    }

    // NB (one block of short rows: one or two tiles per workgroup, the launch is bound by
    // latency): loads without branches; the streaming uses keep the plain loads.  Rows of
    // the previous block that do not exist enter with sign 0, so they need no zeroing.
    auto tile_load = [&](const float *row, bool have, int64_t e) {
        if constexpr (NB) return load4_nb<VW>(row, have, e, d);
        else return load4<VW>(have ? row : nullptr, e, d);
    };

    double4_t acc[L::NT];
#pragma unroll
    for (int q = 0; q < L::NT; ++q) acc[q] = (double4_t){0.0, 0.0, 0.0, 0.0};
    double pdot[RG];
#pragma unroll
    for (int g = 0; g < RG; ++g) pdot[g] = 0.0;

    const int mrow = lane & 15;
    const int kslot = lane >> 4;

    float4 stage_regs[LOADS];
    float4 prev_regs[APPLY ? LOADS : 1];
    double2 stage_s = make_double2(0.0, 0.0);

    auto load_tile = [&](int64_t t) {
#pragma unroll
        for (int u = 0; u < LOADS; ++u) stage_regs[u] = tile_load(src[u], (have_mask >> u) & 1u, t * TE + chunk * 4);
        if constexpr (APPLY) {
#pragma unroll
            for (int u = 0; u < LOADS; ++u) prev_regs[u] = tile_load(psrc[u], true, t * TE + chunk * 4);
        }
        if (!FRESH && tid < TE / 2) stage_s = *reinterpret_cast<const double2 *>(r_sum + t * TE + tid * 2);
    };
    int64_t tile = group;
    if (tile < ntiles) load_tile(tile);
    int buf = 0;
    for (; tile < ntiles; tile += ngroups) {
        unsigned char *stage = smem + buf * STAGE_BYTES;
#pragma unroll
        for (int u = 0; u < LOADS; ++u)
            *reinterpret_cast<float4 *>(stage + lds_off[u]) = stage_regs[u];
        if constexpr (APPLY) {
            // this thread's signed sum of the previous block's rows it holds
            double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
#pragma unroll
            for (int u = 0; u < LOADS; ++u) {
                const double sg = (double)psign[u];
                a0 = __builtin_fma(sg, (double)prev_regs[u].x, a0);
                a1 = __builtin_fma(sg, (double)prev_regs[u].y, a1);
                a2 = __builtin_fma(sg, (double)prev_regs[u].z, a2);
                a3 = __builtin_fma(sg, (double)prev_regs[u].w, a3);
            }
            double *ap = reinterpret_cast<double *>(smem + 2 * STAGE_BYTES) + lrow * TE + chunk * 4;
            *reinterpret_cast<double2 *>(ap) = make_double2(a0, a1);
            *reinterpret_cast<double2 *>(ap + 2) = make_double2(a2, a3);
            __syncthreads();
            if (tid < TE / 2) {
                const double *col = reinterpret_cast<const double *>(smem + 2 * STAGE_BYTES) + tid * 2;
                double s0 = 0.0, s1 = 0.0;
#pragma unroll
                for (int q = 0; q < RPI; ++q) { s0 += col[q * TE]; s1 += col[q * TE + 1]; }
                stage_s.x = (FRESH ? 0.0 : stage_s.x) + s0;
                stage_s.y = (FRESH ? 0.0 : stage_s.y) + s1;
                *reinterpret_cast<double2 *>(r_sum + tile * TE + tid * 2) = stage_s;
            }
        }
        if (FRESH && !APPLY && tile == ntiles - 1 && tid < TE / 2) {
            const int64_t e = tile * TE + tid * 2;
            if (e >= d) r_sum[e] = 0.0;
            if (e + 1 >= d) r_sum[e + 1] = 0.0;
        }
        if (tid < TE / 2)
            *reinterpret_cast<double2 *>(stage + 2 * TILE_FLOATS * 4 + tid * 16) = stage_s;
        __syncthreads();

        // prefetch the next tile while this one is consumed
        int64_t nxt = tile + ngroups;
        if (nxt < ntiles) load_tile(nxt);

        const float *first = reinterpret_cast<const float *>(stage);
        const float *second = first + TILE_FLOATS;
        const double *sv = reinterpret_cast<const double *>(stage + 2 * TILE_FLOATS * 4);
#pragma unroll
        for (int ks = 0; ks < EPW / 16; ++ks) {
            const int eo = EPW * wave + 16 * ks + 4 * kslot;  // element offset inside the tile
            float4 a[RG], b[RG];
#pragma unroll
            for (int g = 0; g < RG; ++g) {
                a[g] = *reinterpret_cast<const float4 *>(first + (16 * g + mrow) * STRIDE + eo);
                b[g] = *reinterpret_cast<const float4 *>(second + (16 * g + mrow) * STRIDE + eo);
            }
            double2 s01 = *reinterpret_cast<const double2 *>(sv + eo);
            double2 s23 = *reinterpret_cast<const double2 *>(sv + eo + 2);
            const double se[4] = {s01.x, s01.y, s23.x, s23.y};
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                double dd[RG];
#pragma unroll
                for (int g = 0; g < RG; ++g) {
                    float fa = (t == 0) ? a[g].x : (t == 1) ? a[g].y : (t == 2) ? a[g].z : a[g].w;
                    float fb = (t == 0) ? b[g].x : (t == 1) ? b[g].y : (t == 2) ? b[g].z : b[g].w;
                    dd[g] = (double)fb - (double)fa;
                    pdot[g] = __builtin_fma(se[t], dd[g], pdot[g]);
                }
                // upper-triangular tiles, row group g (A operand) x row group h >= g (B operand)
                int q = 0;
#pragma unroll
                for (int g = 0; g < RG; ++g)
#pragma unroll
                    for (int h = g; h < RG; ++h) {
                        acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(dd[g], dd[h], acc[q], 0, 0, 0);
                        ++q;
                    }
            }
        }
        buf ^= 1;
    }

    // cross-wave reduction in a fixed order
    __syncthreads();
    double *red = reinterpret_cast<double *>(smem);
    constexpr int PER_WAVE = L::GRAM + RG * 64;
#pragma unroll
    for (int q = 0; q < L::NT; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v) red[wave * PER_WAVE + q * 256 + v * 64 + lane] = acc[q][v];
#pragma unroll
    for (int g = 0; g < RG; ++g) red[wave * PER_WAVE + L::GRAM + g * 64 + lane] = pdot[g];
    __syncthreads();
    for (int idx = tid; idx < L::GRAM; idx += kThreads) {
        double sum = 0.0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) sum += red[w * PER_WAVE + idx];
        out[idx] = sum;
    }
    if (tid < BB) {
        int g = tid >> 4, rw = tid & 15;
        double sum = 0.0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w)
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) sum += red[w * PER_WAVE + L::GRAM + g * 64 + ks * 16 + rw];
        out[L::GRAM + tid] = sum;
    }
}

template <int BB, int VW, int TE, bool APPLY, bool FRESH>
__global__ __launch_bounds__(kThreads) void pass1_dots_gram(RowMap rm, PrevBlock prev,
                                                            double *__restrict__ r_sum,
                                                            double *__restrict__ partials,
                                                            int64_t ntiles)
{
    pass1_body<BB, VW, TE, APPLY, FRESH, TE == 64>(rm, prev, r_sum,
                                                   partials + (int64_t)blockIdx.x * PartLayout<BB>::PART, ntiles,
                                                   (int)blockIdx.x, (int)gridDim.x);
}

// ---------------------------------------------------------------------------
// Fixed-order reduction of the per-workgroup partials, first level: the list of
// workgroups is cut into kReduceSlices slices (blockIdx.y); each workgroup sums
// its slice for 32 consecutive entries, 8 sub-ranges per entry combined in order.
// The resolver adds the kReduceSlices slice sums, again in order.
constexpr int kReduceEntries = 32;
constexpr int kReduceSubs = kThreads / kReduceEntries;
constexpr int kReduceSlices = 8;

__global__ __launch_bounds__(kThreads) void reduce_partials(const double *__restrict__ partials,
                                                            double *__restrict__ sliced, int part,
                                                            int groups)
{
    __shared__ double subsum[kReduceSubs][kReduceEntries];
    const int ent = threadIdx.x % kReduceEntries;
    const int sub = threadIdx.x / kReduceEntries;
    const int entry = blockIdx.x * kReduceEntries + ent;
    const int slice = blockIdx.y;
    const int s0 = (int)((int64_t)slice * groups / kReduceSlices);
    const int s1 = (int)((int64_t)(slice + 1) * groups / kReduceSlices);
    const int g0 = s0 + (int)((int64_t)sub * (s1 - s0) / kReduceSubs);
    const int g1 = s0 + (int)((int64_t)(sub + 1) * (s1 - s0) / kReduceSubs);
    double sum = 0.0;
    if (entry < part) {
        // the loads are independent: keep eight in flight (the adds stay in order)
#pragma unroll 8
        for (int g = g0; g < g1; ++g) sum += partials[(int64_t)g * part + entry];
    }
    subsum[sub][ent] = sum;
    __syncthreads();
    if (sub == 0 && entry < part) {
        double tot = 0.0;
#pragma unroll
        for (int q = 0; q < kReduceSubs; ++q) tot += subsum[q][ent];
        sliced[(int64_t)slice * part + entry] = tot;
    }
}

// ---------------------------------------------------------------------------
// A step of a walk whose lanes hold u = -t, never -0: u loses c where lane LANE's u is not negative (its
// sign is +1), else gains it.  The whole decision is one sign bit: it reaches a scalar register by v_readlane (walk_sign),
// flips the sign of c (sign_flipped_by), and the sum is taken -- three dependent instructions, 22 cycles.  (Compare, vote,
// scalar +-1 and FMA 37.8; sign bit by scalar AND and XOR 41; +-1 made first, read and multiplied 26.5; by DPP row
// broadcast, which reaches sixteen lanes only, 25.3.)  Not for a u that is not a number.
template <int LANE>
__device__ __forceinline__ int walk_sign(double u) { return __builtin_amdgcn_readlane(__double2hiint(u), LANE); }

// x, or -x if the sign bit of `decided` is set.
__device__ __forceinline__ double sign_flipped_by(double x, uint32_t decided) {
    // x ^ (decided & 0x80000000)
    const int hi = (int)__builtin_amdgcn_bitop3_b32((uint32_t)__double2hiint(x), decided, 0x80000000u, 0x78);
    return __hiloint2double(hi, __double2loint(x));
}

// f(integral_constant<int, 0>) .. f(integral_constant<int, N - 1>)
template <int... I, typename F>
__device__ __forceinline__ void static_for(std::integer_sequence<int, I...>, F &&f) {
    (f(std::integral_constant<int, I>{}), ...);
}

// One wavefront walks N pairs: lane k holds t of pair k before them and, in col, column k of their Gram matrix,
// zero at and above the diagonal (so lane k changes at steps j < k only).  Returns the resolved dot; plus: the
// pair's sign is +1.  Straight-line code, 22 cycles per pair by walk_sign; a vote per step instead of it (38) serves
// where a dot is not a number, which has no sign to go by.
// Randomized rule (PairBalance's RandomizedBalance subroutine, Sec. 3.2): with
// c = z1 - z2 = -d, the first row gets +1 with probability p = (1 - <r,c>)/2 =
// (1 + t)/2, so the exported sign (of the second row) is -1 when the draw is below p: the sign of their
// difference (rounded once, so it is zero only where they are equal, and then +0: a draw of -0 is taken as 0).
// A draw that is not a finite number goes by comparison, as a dot that is not a number does.
template <int N, bool RANDOM>
__device__ __forceinline__ double walk_pairs(const double (&col)[N], double t, float draw, bool &plus) {
    auto rule = [&](double tv) { return RANDOM ? !((double)draw < 0.5 * (1.0 + tv)) : (tv <= 0.0); };
    const double of = (double)draw + 0.0;
    double u = 0.0 - t;  // (a difference of equal numbers is +0)
    static_for(std::make_integer_sequence<int, N>{}, [&](auto jj) {
        constexpr int j = decltype(jj)::value;
        u -= sign_flipped_by(col[j], (uint32_t)walk_sign<j>(RANDOM ? __builtin_fma(-0.5, 1.0 - u, of) : u));
    });
    if (__ballot(u != u || (RANDOM && !isfinite(draw)))) {
        u = 0.0 - t;
        static_for(std::make_integer_sequence<int, N>{}, [&](auto jj) {
            constexpr int j = decltype(jj)::value;
            const bool vote = (__ballot(rule(0.0 - u)) >> j) & 1ull;
            u -= vote ? col[j] : -col[j];
        });
    }
    t = 0.0 - u;
    plus = rule(t);
    return t;
}

// ---------------------------------------------------------------------------
// Sequential sign resolution.  All threads of the workgroup finish the reduction and unpack
// the Gram tiles into LDS; then one wavefront walks the block: lane k carries
// t_k = <r, d_k> + sum_{j<k, decided} eps_j G[j][k]; step j fixes eps_j = +1 if t_j <= 0
// else -1 (or, given uniform draws, by the randomized rule) and updates the later lanes (walk_pairs).
// Threads of the resolver's load phase: 1024, but 512 for 64-pair blocks, whose walk
// keeps 64 doubles of the Gram matrix per lane in registers.
template <int BB> constexpr int kResolveThreads = BB > 32 ? 512 : 1024;

// The walk is run by the workgroup's first wavefront.
template <int BB, bool RANDOM>
__global__ __launch_bounds__(kResolveThreads<BB>) void resolve_signs(const double *__restrict__ sliced, int nb,
                                                                     int64_t k0, int32_t i0, int32_t m, int64_t half_n,
                                                                     int8_t *__restrict__ eps_blk,
                                                                     int8_t *__restrict__ signs_out,
                                                                     double *__restrict__ dots_out,
                                                                     const float *__restrict__ uniforms)
{
    // Gram tiles and dots: sums of the kReduceSlices arrays sliced[slice * PART], in order.
    using L = PartLayout<BB>;
    constexpr int NT = kResolveThreads<BB>;
    __shared__ double G[BB][BB + 1];
    __shared__ double P[BB];
    __shared__ double psub[BB][kReduceSlices + 1];
    // A dot's slices are requested before anything else, one per thread, and consumed after the Gram tiles.
    static_assert(BB * kReduceSlices <= NT, "a thread per dot and slice");
    const int dk = (threadIdx.x / kReduceSlices) % BB, dsl = threadIdx.x % kReduceSlices;
    const double dv = sliced[dsl * L::PART + L::GRAM + dk];
    // Two consecutive entries per thread and step (16 B loads; GRAM is even).  All loads
    // of a thread are issued before the first is used: entries beyond the end re-read
    // entry 0 and are dropped.
    constexpr int ITER = (L::GRAM + 2 * NT - 1) / (2 * NT);
    double2 raw[ITER][kReduceSlices];
#pragma unroll
    for (int it = 0; it < ITER; ++it) {
        const int idx = 2 * (int)threadIdx.x + it * 2 * NT;
        const int idc = idx < L::GRAM ? idx : 0;
#pragma unroll
        for (int sl = 0; sl < kReduceSlices; ++sl)
            raw[it][sl] = *reinterpret_cast<const double2 *>(sliced + sl * L::PART + idc);
    }
#pragma unroll
    for (int it = 0; it < ITER; ++it) {
        const int idx = 2 * (int)threadIdx.x + it * 2 * NT;
        if (idx >= L::GRAM) continue;
        double2 val = make_double2(0.0, 0.0);
#pragma unroll
        for (int sl = 0; sl < kReduceSlices; ++sl) {
            val.x += raw[it][sl].x;
            val.y += raw[it][sl].y;
        }
        const int tile = idx >> 8, v = (idx >> 6) & 3, ln = idx & 63;
        // tiles are stored row group by row group, upper triangle only: (0,0), (0,1), .., (1,1), ..
        int tg = 0, th = tile;
        while (th >= L::RG - tg) { th -= L::RG - tg; ++tg; }
        th += tg;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            int i, j;
            mfma_f64_16x16_coord(ln + q, v, i, j);
            const double x = q ? val.y : val.x;
            G[16 * tg + i][16 * th + j] = x;
            if (th != tg) G[16 * th + j][16 * tg + i] = x;
        }
    }
    if (threadIdx.x < BB * kReduceSlices) psub[dk][dsl] = dv;
    __syncthreads();
    if (threadIdx.x < BB) {
        double sum = 0.0;
#pragma unroll
        for (int q = 0; q < kReduceSlices; ++q) sum += psub[threadIdx.x][q];
        P[threadIdx.x] = sum;
    }
    __syncthreads();
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        // lane k keeps column k of the Gram matrix (= row k, it is symmetric) in registers
        // (entries j >= lane are zeroed: lane k is updated at steps j < k only, and the walk
        // then needs no lane test of its own)
        double col[BB];
#pragma unroll
        for (int j = 0; j < BB; ++j) col[j] = (lane < BB && lane > j) ? G[lane][j] : 0.0;
        const double t = (lane < nb) ? P[lane] : 0.0;
        // flattened pair of this lane -> (worker, pair) slot of the [m][n/2] arrays
        int64_t slot = 0;
        if (lane < nb) {
            uint32_t q = (uint32_t)(i0 + lane);
            uint32_t dq = q / (uint32_t)m;
            slot = (int64_t)(q - dq * (uint32_t)m) * half_n + (k0 + dq);
        }
        const float my_u = (RANDOM && lane < nb) ? uniforms[slot] : 0.f;
        // (Steps j >= nb of a short last block run too: they only touch lanes above j, which
        // hold no pair.)
        bool plus;
        const double my_t = walk_pairs<BB, RANDOM>(col, t, my_u, plus);
        const int my_eps = plus ? 1 : -1;
        if (lane < nb) {
            eps_blk[lane] = (int8_t)my_eps;
            signs_out[slot] = (int8_t)my_eps;
            if (dots_out) dots_out[slot] = my_t;
        }
    }
}

// ---------------------------------------------------------------------------
// What an apply launch does besides, so that no launch of its own clears or exports the running sum: the epoch's first
// block starts it (fresh: r_sum holds nothing and is not read), the last one's result leaves as fp32 and / or
// double (r32, r64; last: it goes nowhere else).  Five passes over the running sum less per epoch: 40 pairs of
// 124M elements 15.03 -> 14.07 ms, 128 pairs of 11.2M 3913 -> 3805 us.
struct SumEnds {
    int fresh, last;
    float *r32;
    double *r64;
};

typedef double double2_any __attribute__((ext_vector_type(2), aligned(8)));

// r[e .. e + 3] += acc.  The running sum is padded to the tile, and the padding of these four stays zero because
// elements beyond d load as zero.
__device__ __forceinline__ void update_four(const SumEnds &ends, double *__restrict__ r_sum, int64_t e, int64_t d,
                                            const double (&acc)[4]) {
    double2 lo = make_double2(0.0, 0.0), hi = lo;
    if (!ends.fresh) {
        lo = *reinterpret_cast<double2 *>(r_sum + e);
        hi = *reinterpret_cast<double2 *>(r_sum + e + 2);
    }
    lo.x += acc[0]; lo.y += acc[1]; hi.x += acc[2]; hi.y += acc[3];
    if (!ends.last) {
        *reinterpret_cast<double2 *>(r_sum + e) = lo;
        *reinterpret_cast<double2 *>(r_sum + e + 2) = hi;
        return;
    }
    const double v[4] = {lo.x, lo.y, hi.x, hi.y};
    if (e + 4 <= d) {
        if (ends.r32) *reinterpret_cast<float4_any *>(ends.r32 + e) = (float4_any){(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
        if (ends.r64) {
            *reinterpret_cast<double2_any *>(ends.r64 + e) = (double2_any){v[0], v[1]};
            *reinterpret_cast<double2_any *>(ends.r64 + e + 2) = (double2_any){v[2], v[3]};
        }
    } else {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (e + q < d) {
                if (ends.r32) ends.r32[e + q] = (float)v[q];
                if (ends.r64) ends.r64[e + q] = v[q];
            }
    }
}

// ---------------------------------------------------------------------------
// Pass 2: r += sum_k eps_k d_k.  Each thread owns four consecutive elements and
// streams the block's rows through registers.  FULL = the block holds all BB
// pairs (no per-pair test inside the unrolled loop).
template <int BB, int VW, bool FULL>
__global__ __launch_bounds__(kThreads) void pass2_apply(RowMap rm, const int8_t *__restrict__ eps_blk, SumEnds ends,
                                                        double *__restrict__ r_sum)
{
    const int64_t d = rm.d;
    const int64_t e = ((int64_t)blockIdx.x * kThreads + threadIdx.x) * 4;
    if (e >= d) return;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    auto add_rows = [&](auto inside) {
#pragma unroll 8
        for (int j = 0; j < BB; ++j) {
            if (FULL || j < rm.nb) {
                float4 a = load4<VW, decltype(inside)::value>(rm.row(j, 0), e, d);
                float4 b = load4<VW, decltype(inside)::value>(rm.row(j, 1), e, d);
                double sg = (double)eps_blk[j];
                acc[0] = __builtin_fma(sg, (double)b.x - (double)a.x, acc[0]);
                acc[1] = __builtin_fma(sg, (double)b.y - (double)a.y, acc[1]);
                acc[2] = __builtin_fma(sg, (double)b.z - (double)a.z, acc[2]);
                acc[3] = __builtin_fma(sg, (double)b.w - (double)a.w, acc[3]);
            }
        }
    };
    if (VW == kAnyRow && e + 4 <= d) add_rows(std::true_type{});
    else add_rows(std::false_type{});
    update_four(ends, r_sum, e, d, acc);
}

// ---------------------------------------------------------------------------
// Pass 2 for long rows, with the running-sum traffic gathered into bursts.  The grid is
// wholly resident (two workgroups per CU); a thread owns up to kResidentGroups groups of
// four elements (group g of slab s at element ((s * kuse + g) * T + t) * 4, T threads in
// all), streams all rows of the block for one group after the other and keeps the sums in
// registers; only when all its groups are done does it read, update and write the running
// sum.  All workgroups run in step, so the launch is a long stretch of pure row reads
// followed by one short burst of running-sum reads and writes.  A row longer than the
// registers of the chip hold (kuse * T * 4 elements) is cut into slabs, ONE LAUNCH PER SLAB:
// the launch boundary brings the workgroups back into step -- inside one launch they drift
// apart from slab to slab, the bursts smear out into the row reads, and the gain is lost
// (d = 124M, eleven slabs: 6.06 ms in one launch, the same as the flat form).
// Writes scattered through a read stream cost this chip about 1 us per MB (the flat form
// above: 0.52 ms per 32-pair block at d = 11.2M, of which 0.09 ms for 180 MB of running-sum
// traffic); gathered at the end they cost a third of that (0.46 ms).  Same sums in the
// same order as the flat form: bit-identical results.
constexpr int kResidentGroups = 22;

template <int BB, int VW, bool FULL>
__global__ __launch_bounds__(kThreads, 2) void pass2_apply_resident(RowMap rm, const int8_t *__restrict__ eps_blk,
                                                                    SumEnds ends, double *__restrict__ r_sum,
                                                                    int kuse, int64_t g0)
{
    // this launch: groups g0 .. g0 + kuse - 1 of every thread (one slab)
    constexpr int K = kResidentGroups;
    const int64_t d = rm.d;
    const int64_t T = (int64_t)gridDim.x * kThreads;
    const int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    double acc[K][4];
#pragma unroll
    for (int g = 0; g < K; ++g) {
        acc[g][0] = acc[g][1] = acc[g][2] = acc[g][3] = 0.0;
        const int64_t e = ((g0 + g) * T + t) * 4;
        auto add_rows = [&](auto inside) {
#pragma unroll 2
            for (int j = 0; j < BB; ++j) {
                if (FULL || j < rm.nb) {
                    float4 a = load4<VW, decltype(inside)::value>(rm.row(j, 0), e, d);
                    float4 b = load4<VW, decltype(inside)::value>(rm.row(j, 1), e, d);
                    double sg = (double)eps_blk[j];
                    acc[g][0] = __builtin_fma(sg, (double)b.x - (double)a.x, acc[g][0]);
                    acc[g][1] = __builtin_fma(sg, (double)b.y - (double)a.y, acc[g][1]);
                    acc[g][2] = __builtin_fma(sg, (double)b.z - (double)a.z, acc[g][2]);
                    acc[g][3] = __builtin_fma(sg, (double)b.w - (double)a.w, acc[g][3]);
                }
            }
        };
        if (g < kuse && e < d) {
            if (VW == kAnyRow && e + 4 <= d) add_rows(std::true_type{});
            else add_rows(std::false_type{});
        }
    }
#pragma unroll
    for (int g = 0; g < K; ++g) {
        const int64_t e = ((g0 + g) * T + t) * 4;
        if (g < kuse && e < d) update_four(ends, r_sum, e, d, acc[g]);
    }
}

// ---------------------------------------------------------------------------
// Pass 2 for short rows: a workgroup owns 64 consecutive elements; its 256 threads
// are 16 element-quads x 16 pair groups, each thread sums BB/16 pairs for its quad,
// the 16 partial sums are added in group order through LDS, and 64 threads update
// one element each.  Sixteen times the workgroups and a sixteenth of the loads per
// thread of the flat form, which is what a latency-bound launch needs.
constexpr int kSplitGroups = 16;
constexpr int kSplitElems = (kThreads / kSplitGroups) * 4;  // 64 elements per workgroup

template <int BB, int VW, bool FULL>
__global__ __launch_bounds__(kThreads) void pass2_apply_split(RowMap rm, const int8_t *__restrict__ eps_blk,
                                                              SumEnds ends, double *__restrict__ r_sum)
{
    __shared__ double part[kSplitGroups][kSplitElems];
    const int64_t d = rm.d;
    const int quad = threadIdx.x % (kThreads / kSplitGroups), grp = threadIdx.x / (kThreads / kSplitGroups);
    const int64_t e = (int64_t)blockIdx.x * kSplitElems + quad * 4;
    const int64_t mine = (int64_t)blockIdx.x * kSplitElems + threadIdx.x;
    // the running-sum element is requested first so that its latency overlaps the row loads
    const double r_old = (threadIdx.x < kSplitElems && mine < d && !ends.fresh) ? r_sum[mine] : 0.0;
    constexpr int PER = BB / kSplitGroups;
    float4 a[PER], b[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int j = grp * PER + q;
        // (offsets of missing pairs are readable rows: zero, or those of an earlier block)
        const bool have = FULL || j < rm.nb;
        a[q] = load4_nb<VW>(rm.row(j, 0), have, e, d);
        b[q] = load4_nb<VW>(rm.row(j, 1), have, e, d);
    }
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int j = grp * PER + q;
        const double sg = (FULL || j < rm.nb) ? (double)eps_blk[j] : 0.0;
        acc[0] = __builtin_fma(sg, (double)b[q].x - (double)a[q].x, acc[0]);
        acc[1] = __builtin_fma(sg, (double)b[q].y - (double)a[q].y, acc[1]);
        acc[2] = __builtin_fma(sg, (double)b[q].z - (double)a[q].z, acc[2]);
        acc[3] = __builtin_fma(sg, (double)b[q].w - (double)a[q].w, acc[3]);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) part[grp][quad * 4 + q] = acc[q];
    __syncthreads();
    if (threadIdx.x < kSplitElems && mine < d) {
        double sum = 0.0;
#pragma unroll
        for (int g = 0; g < kSplitGroups; ++g) sum += part[g][threadIdx.x];
        const double r = r_old + sum;
        if (!ends.last) r_sum[mine] = r;
        else {
            if (ends.r32) ends.r32[mine] = (float)r;
            if (ends.r64) ends.r64[mine] = r;
        }
    }
}

// ---------------------------------------------------------------------------
// Clears `count` 32-bit words.  The library clears its flags and scratch with fill
// kernels rather than memset nodes, so that a caller may capture its stream in a graph.
__global__ void fill_zero_b32(uint32_t *p, int64_t count) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < count; i += stride) p[i] = 0u;
}

}  // namespace cdgrab
