// Short rows: the balancing walk as a chain of long steps.
//
// With short rows an epoch is bound by its chain of dependent launches, not by bytes, so the
// chain is made of few long steps.  A step covers `sp` consecutive pairs (64, 128 or 256).  The
// Gram matrices <d_j, d_k> of the pairs of a step depend on the rows only -- not on the running
// sum, not on earlier signs -- and are taken off the chain: gram_tiles computes those of many
// steps in one launch.  What stays on the chain is two launches per step:
//   chain_apply_dots   r += sum eps_j d_j over the previous step, and this step's dots <r, d_k>,
//                      every workgroup on 64 elements of d;
//   chain_walk         one workgroup adds the workgroups' shares of the dots and walks the step:
//                      t_k = <r, d_k> + sum_{j<k} eps_j <d_j, d_k>, eps_k = +1 if t_k <= 0 else -1.
// A longer step has fewer launches per pair and more Gram entries per pair (double MFMA work
// and bytes grow with sp); the host picks sp by a cost model of both.
#pragma once
#include <type_traits>
#include <utility>

#include "balance_kernels.hpp"

namespace cdgrab {

constexpr int kTilePairs = 64;                           // the Gram matrix is stored in 64 x 64 tiles
constexpr int kTileEntries = kTilePairs * kTilePairs;
constexpr int kMaxStepPairs = 256;

// The rows of consecutive flattened pairs, in one of three layouts.
struct StepRows {
    const float *base;    // kDense: the input [m][n][d]; kCentred / kStaged: the first pair's first row
    const float *centre;  // kCentred: every single row is paired with this one
    int64_t d, n;
    int64_t k0;           // kDense: pair index (per worker) of the first pair ...
    int32_t i0;           // ... and its worker
    int32_t m;
    int32_t nb;           // number of pairs
    int32_t layout;
};
enum { kDense = 0, kCentred = 1, kStaged = 2 };

// Walks consecutive pairs without a division per pair.
struct PairCursor {
    int64_t i, k;  // kDense: worker and pair index; else k counts pairs from base
    __device__ __forceinline__ PairCursor(const StepRows &sr, int j) {
        if (sr.layout == kDense) {
            const uint32_t q = (uint32_t)(sr.i0 + j), dk = q / (uint32_t)sr.m;
            i = (int64_t)(q - dk * (uint32_t)sr.m);
            k = sr.k0 + (int64_t)dk;
        } else {
            i = 0;
            k = j;
        }
    }
    __device__ __forceinline__ void next(const StepRows &sr) {
        ++i;
        const bool wrap = sr.layout != kDense || i == sr.m;
        i = wrap ? 0 : i;
        k += wrap ? 1 : 0;
    }
    __device__ __forceinline__ void rows(const StepRows &sr, const float *&a, const float *&b) const {
        const int64_t row = sr.layout == kCentred ? k : i * sr.n + 2 * k;  // (staged pairs: i is 0)
        a = sr.base + row * sr.d;
        b = sr.layout == kCentred ? sr.centre : a + sr.d;
    }
};

// The sub-range of `nb` pairs that starts `first` pairs into sr.
__host__ __device__ inline StepRows step_at(StepRows sr, int64_t first, int nb) {
    if (sr.layout == kDense) {
        const int64_t q = (int64_t)sr.i0 + first;
        sr.k0 += q / sr.m;
        sr.i0 = (int32_t)(q % sr.m);
    } else {
        sr.base += first * (sr.layout == kStaged ? 2 : 1) * sr.d;
    }
    sr.nb = nb;
    return sr;
}

// ---------------------------------------------------------------------------
// Gram tiles of many steps.  One workgroup computes one 64 x 64 tile (ti <= tj) of one step over
// its share of d: tiles of kGramTE elements of the 64 + 64 pair differences are formed in double
// on the way into LDS (an element is used by two wavefronts, so it is converted once instead of
// twice), and the next tile's loads are in flight meanwhile.  Off the diagonal each of the four wavefronts
// owns a 32 x 32 quarter of the tile.  On it only the ten 16 x 16 results of the upper triangle
// are needed, which four quarters cannot share evenly (three whole quarters and an idle wavefront took the
// time of sixteen results), so there each wavefront takes a quarter of the elements and all ten.
// LDS rows are 34 doubles: the sixteen rows a quarter of a
// wavefront reads start four banks apart, so the 16-byte reads do not collide.  Element order
// inside a tile: lane slot s of MFMA step 2q (2q + 1) takes element 8 q + 2 s (+ 1), the same for
// both operands.  The tiles of one step are consecutive workgroups of one XCD where there are
// enough steps, so that the rows they share come from its L2.
// Bound by the matrix instructions: 41 TFLOP/s on 235 steps of 128 pairs of 7850 elements (1.09 -> 0.82 ms),
// 40 on 64 walks of 468 pairs, whose tiles are all diagonal (0.76 -> 0.51 ms), of 48.9 in a loop of nothing else.
struct GramBatch {
    StepRows rows;        // all pairs of the batch (nb unused)
    int64_t pairs;        // pairs in the batch
    int64_t walk_floats;  // floats between the walks' rows
    int32_t sp;           // pairs per step
    int32_t steps;        // steps per walk
    int32_t units;        // walks * steps
    int32_t tiles;        // tiles stored per step
    int32_t ksplit;       // workgroups sharing the elements of a tile
    int32_t ktiles;       // kGramTE-element tiles of a row
    const int64_t *examples;  // not null: the matrix of single rows base + examples[pair] * d instead of differences
};
constexpr int kGramTE = 32;

// Position of tile (ti, tj), ti <= tj, in a step's list: (0,0) (0,1) (1,1) (0,2) (1,2) (2,2) ..
__host__ __device__ constexpr int tile_index(int ti, int tj) { return tj * (tj + 1) / 2 + ti; }

// A thread's share of a tile of elements, N rows of pairs: four elements of both rows each.
template <int N> struct GramPieces { float4 a[N], b[N]; };

template <int VW, bool SINGLE>
__global__ __launch_bounds__(kThreads, 2) void gram_tiles(GramBatch gb, double *__restrict__ out)
{
    constexpr int STRIDE = kGramTE + 2;
    __shared__ __attribute__((aligned(16))) double lds[2][2][kTilePairs * STRIDE];  // [stage][side]
    int unit, tile;
    if (gb.units >= 8) {
        const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
        unit = (slot / gb.tiles) * 8 + xcd;
        tile = slot % gb.tiles;
    } else {
        unit = blockIdx.x / gb.tiles;
        tile = blockIdx.x % gb.tiles;
    }
    if (unit >= gb.units) return;
    const int walk = unit / gb.steps, step = unit - walk * gb.steps;
    int tj = 0;
    while (tile_index(0, tj + 1) <= tile) ++tj;
    const int ti = tile - tile_index(0, tj);
    const int64_t left = gb.pairs - (int64_t)step * gb.sp;
    const int nb = (int)(left < gb.sp ? left : gb.sp);
    if (tj * kTilePairs >= nb) return;
    StepRows rows = gb.rows;
    rows.base += walk * gb.walk_floats;
    rows = step_at(rows, (int64_t)step * gb.sp, nb);
    const int64_t d = rows.d;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int quad = tid & 7, prow = tid >> 3;  // eight threads cover a row's tile, 32 rows at a time
    const float *src[4][2];                     // [side * 2 + half][first / second row]
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const int j = (s < 2 ? ti : tj) * kTilePairs + (s & 1) * 32 + prow;
        if constexpr (SINGLE) {
            src[s][0] = src[s][1] = gb.rows.base + gb.examples[(int64_t)step * gb.sp + (j < nb ? j : nb - 1)] * d;
            continue;
        }
        PairCursor(rows, j < nb ? j : nb - 1).rows(rows, src[s][0], src[s][1]);  // (a missing pair repeats the last one)
    }
    const int kt0 = (int)((int64_t)blockIdx.y * gb.ktiles / gb.ksplit);
    const int kt1 = (int)((int64_t)(blockIdx.y + 1) * gb.ktiles / gb.ksplit);

    double *dst = out + (((int64_t)unit * gb.tiles + tile) * gb.ksplit + blockIdx.y) * kTileEntries;
    const int mrow = lane & 15, kslot = lane >> 4;
    // N 32-row pieces of a tile of elements: the diagonal tile's two, or the four of both sides
    auto load = [&](auto &x, int kt) {
        constexpr int N = sizeof(x.a) / sizeof(x.a[0]);
        const int64_t e = (int64_t)kt * kGramTE + quad * 4;
        if ((int64_t)(kt + 1) * kGramTE <= d) {  // uniform
#pragma unroll
            for (int s = 0; s < N; ++s) {
                const float4_t b = load_four<false>(src[s][1] + e);
                const float4_t a = SINGLE ? (float4_t){0.f, 0.f, 0.f, 0.f} : load_four<false>(src[s][0] + e);
                x.a[s] = make_float4(a.x, a.y, a.z, a.w);
                x.b[s] = make_float4(b.x, b.y, b.z, b.w);
            }
        } else {
#pragma unroll
            for (int s = 0; s < N; ++s) {
                x.a[s] = SINGLE ? make_float4(0.f, 0.f, 0.f, 0.f) : load4_nb<VW>(src[s][0], true, e, d);
                x.b[s] = load4_nb<VW>(src[s][1], true, e, d);
            }
        }
    };
    auto store = [&](const auto &x, int stage) {
        constexpr int N = sizeof(x.a) / sizeof(x.a[0]);
#pragma unroll
        for (int s = 0; s < N; ++s) {
            double2 *p = reinterpret_cast<double2 *>(&lds[stage][s >> 1][((s & 1) * 32 + prow) * STRIDE + quad * 4]);
            p[0] = make_double2((double)x.b[s].x - (double)x.a[s].x, (double)x.b[s].y - (double)x.a[s].y);
            p[1] = make_double2((double)x.b[s].z - (double)x.a[s].z, (double)x.b[s].w - (double)x.a[s].w);
        }
    };

    if (ti == tj) {  // uniform
        // A wavefront takes a quarter of the elements of every tile and all ten results of the upper triangle,
        // two tiles of loads in flight; the quarters' results are added in order through LDS.
        GramPieces<2> even, odd;
        double4_t acc[10];
#pragma unroll
        for (int q = 0; q < 10; ++q) acc[q] = (double4_t){0.0, 0.0, 0.0, 0.0};
        if (kt0 < kt1) {
            load(even, kt0);
            if (kt0 + 1 < kt1) load(odd, kt0 + 1);
            store(even, 0);
            if (kt0 + 2 < kt1) load(even, kt0 + 2);
        }
        __syncthreads();
        auto tile_of = [&](int kt, GramPieces<2> &next) {
            const int stage = (kt - kt0) & 1;
            const double *A = lds[stage][0] + mrow * STRIDE + 8 * wave + 2 * kslot;
            double2 a[4];
#pragma unroll
            for (int g = 0; g < 4; ++g) a[g] = *reinterpret_cast<const double2 *>(A + g * 16 * STRIDE);
#pragma unroll
            for (int h = 0; h < 4; ++h)
#pragma unroll
                for (int g = 0; g <= h; ++g)
                    acc[tile_index(g, h)] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[g].x, a[h].x, acc[tile_index(g, h)], 0, 0, 0);
#pragma unroll
            for (int h = 0; h < 4; ++h)
#pragma unroll
                for (int g = 0; g <= h; ++g)
                    acc[tile_index(g, h)] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[g].y, a[h].y, acc[tile_index(g, h)], 0, 0, 0);
            if (kt + 1 < kt1) store(next, stage ^ 1);
            if (kt + 3 < kt1) load(next, kt + 3);
            __syncthreads();
        };
        for (int kt = kt0; kt < kt1; kt += 2) {
            tile_of(kt, odd);
            if (kt + 1 < kt1) tile_of(kt + 1, even);
        }
        // result q is added by wavefront q % 4, the other three leave theirs in LDS
        double4_t *red = reinterpret_cast<double4_t *>(&lds[0][0][0]);
        static_assert(10 * 3 * 64 * sizeof(double4_t) <= sizeof(lds), "three wavefronts' results");
#pragma unroll
        for (int q = 0; q < 10; ++q)
            if ((q & 3) != wave) red[(q * 3 + wave - (wave > (q & 3) ? 1 : 0)) * 64 + lane] = acc[q];
        __syncthreads();
#pragma unroll
        for (int h = 0; h < 4; ++h)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                // (the walk's columns are zero at and above the diagonal)
                const int q = g <= h ? tile_index(g, h) : g * 4 + h;
                if ((q & 3) != wave) continue;
                double4_t sum = (double4_t){0.0, 0.0, 0.0, 0.0};
                if (g <= h) {
#pragma unroll
                    for (int w = 0; w < 4; ++w)
                        sum += w == (q & 3) ? acc[g <= h ? q : 0] : red[(q * 3 + w - (w > (q & 3) ? 1 : 0)) * 64 + lane];
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    int i, j;
                    mfma_f64_16x16_coord(lane, v, i, j);
                    const int r = 16 * g + i, c = 16 * h + j;
                    dst[r * kTilePairs + c] = r < c ? sum[v] : 0.0;
                }
            }
        return;
    }

    GramPieces<4> x;
    double4_t acc[2][2];
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int h = 0; h < 2; ++h) acc[g][h] = (double4_t){0.0, 0.0, 0.0, 0.0};
    const int wi = wave >> 1, wj = wave & 1;

    if (kt0 < kt1) {
        load(x, kt0);
        store(x, 0);
    }
    __syncthreads();
    for (int kt = kt0; kt < kt1; ++kt) {
        const int stage = (kt - kt0) & 1;
        if (kt + 1 < kt1) load(x, kt + 1);
        const double *A = lds[stage][0] + (32 * wi + mrow) * STRIDE + 2 * kslot;
        const double *B = lds[stage][1] + (32 * wj + mrow) * STRIDE + 2 * kslot;
#pragma unroll
        for (int q = 0; q < kGramTE / 8; ++q) {
            double2 a[2], b[2];
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                a[g] = *reinterpret_cast<const double2 *>(A + g * 16 * STRIDE + 8 * q);
                b[g] = *reinterpret_cast<const double2 *>(B + g * 16 * STRIDE + 8 * q);
            }
#pragma unroll
            for (int g = 0; g < 2; ++g)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    acc[g][h] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[g].x, b[h].x, acc[g][h], 0, 0, 0);
                    acc[g][h] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[g].y, b[h].y, acc[g][h], 0, 0, 0);
                }
        }
        if (kt + 1 < kt1) store(x, stage ^ 1);
        __syncthreads();
    }
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                int i, j;
                mfma_f64_16x16_coord(lane, v, i, j);
                dst[(32 * wi + 16 * g + i) * kTilePairs + 32 * wj + 16 * h + j] = acc[g][h][v];
            }
}

// Sum of the shares of tiles whose elements were split, in order.  One workgroup per tile.
__global__ __launch_bounds__(kThreads) void gram_reduce(const double *__restrict__ parts, double *__restrict__ out,
                                                        int ksplit)
{
    const double2 *src = reinterpret_cast<const double2 *>(parts + (int64_t)blockIdx.x * ksplit * kTileEntries);
    double2 *dst = reinterpret_cast<double2 *>(out + (int64_t)blockIdx.x * kTileEntries);
    const int idx = blockIdx.y * kThreads + threadIdx.x;
    double2 sum = make_double2(0.0, 0.0);
#pragma unroll 8
    for (int q = 0; q < ksplit; ++q) {
        const double2 x = src[(int64_t)q * (kTileEntries / 2) + idx];
        sum.x += x.x;
        sum.y += x.y;
    }
    dst[idx] = sum;
}

// ---------------------------------------------------------------------------
// One step of the chain, wide part: a workgroup owns kStepElems consecutive elements; its 512
// threads are 16 element quads x 32 pair groups of PP pairs (32 PP >= sp).  It applies the
// previous step to its slice of r (partial sums per pair group through LDS, added in group
// order) and writes its share of this step's dots to dots_out[workgroup][sp].  All rows are
// requested up front, so that the launch is one memory round trip long.  Neighbouring workgroups
// share lines (rows need not start on one) and read at the next step what they read at this one, so
// each XCD keeps a contiguous run of workgroups.  Either step may have
// no pairs (the first step has no predecessor, the last apply no successor).  `fresh`: the running sum is
// zero and r_sum holds nothing yet; r32 / r64 (or null): the running sum leaves here as well.  Both spare
// a short epoch a launch of its own (4 x 64 x 1024: 28 us with a fill and an export launch, 25 now).
constexpr int kStepElems = 64;
constexpr int kStepThreads = 512;

template <int PP, int VW>
__global__ __launch_bounds__(kStepThreads, 2) void chain_apply_dots(StepRows cur, StepRows prev,
                                                                    const int8_t *__restrict__ eps, int sp, int groups,
                                                                    int fresh, double *__restrict__ r_sum,
                                                                    double *__restrict__ dots_out,
                                                                    float *__restrict__ r32, double *__restrict__ r64,
                                                                    WalkStrides ws)
{
    constexpr int QUADS = kStepElems / 4;              // 16
    constexpr int GROUPS = kStepThreads / QUADS;       // 32
    constexpr int SUBS = kStepThreads / kStepElems;    // 8
    __shared__ double part[GROUPS][kStepElems];
    __shared__ double part2[SUBS][kStepElems];
    __shared__ __attribute__((aligned(16))) double rnew[kStepElems];
    const int64_t w = blockIdx.y;
    cur.base += w * ws.rows;
    prev.base += w * ws.rows;
    eps += w * kMaxStepPairs;
    r_sum += w * ws.r;
    dots_out += w * ws.dots;
    const int64_t d = cur.d;
    // each XCD takes a contiguous run of element groups, the same one at every step
    const int per_xcd = (groups + 7) >> 3;
    const int block = groups >= 16 ? (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3) : (int)blockIdx.x;
    if (block >= groups) return;
    const int quad = threadIdx.x % QUADS, grp = threadIdx.x / QUADS;
    const int64_t e = (int64_t)block * kStepElems + quad * 4;
    const int el = threadIdx.x % kStepElems, sub = threadIdx.x / kStepElems;
    const int64_t mine = (int64_t)block * kStepElems + el;
    float4 pa[PP], pb[PP], ca[PP], cb[PP];
    int8_t sg[PP];
    if (prev.nb > 0) {  // uniform
        PairCursor at(prev, grp * PP < prev.nb ? grp * PP : prev.nb - 1);
#pragma unroll
        for (int q = 0; q < PP; ++q) {  // (a missing pair enters as zero: 0 times a value that is not finite is not 0)
            const bool have = grp * PP + q < prev.nb;
            const float *a, *b;
            at.rows(prev, a, b);
            pa[q] = load4_nb<VW>(a, have, e, d);
            pb[q] = load4_nb<VW>(b, have, e, d);
            if (grp * PP + q + 1 < prev.nb) at.next(prev);
        }
        __builtin_memcpy(sg, eps + grp * PP, PP);
    }
    if (cur.nb > 0) {  // uniform
        PairCursor at(cur, grp * PP < cur.nb ? grp * PP : cur.nb - 1);
#pragma unroll
        for (int q = 0; q < PP; ++q) {
            const float *a, *b;
            at.rows(cur, a, b);
            ca[q] = load4_nb<VW, false>(a, true, e, d);  // (read again by the next launch)
            cb[q] = load4_nb<VW, false>(b, true, e, d);
            if (grp * PP + q + 1 < cur.nb) at.next(cur);
        }
    }
    const double r_old = sub == 0 && !fresh ? r_sum[mine] : 0.0;  // padded to a multiple of 128
    if (prev.nb > 0) {
        double acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int q = 0; q < PP; ++q) {
            const double s = grp * PP + q < prev.nb ? (double)sg[q] : 0.0;
            acc[0] = __builtin_fma(s, (double)pb[q].x - (double)pa[q].x, acc[0]);
            acc[1] = __builtin_fma(s, (double)pb[q].y - (double)pa[q].y, acc[1]);
            acc[2] = __builtin_fma(s, (double)pb[q].z - (double)pa[q].z, acc[2]);
            acc[3] = __builtin_fma(s, (double)pb[q].w - (double)pa[q].w, acc[3]);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) part[grp][quad * 4 + q] = acc[q];
        __syncthreads();
        double s = 0.0;
#pragma unroll
        for (int g = 0; g < GROUPS / SUBS; ++g) s += part[sub * (GROUPS / SUBS) + g][el];
        part2[sub][el] = s;
        __syncthreads();
    }
    if (sub == 0) {
        double r = r_old;
        if (prev.nb > 0) {
            double s = 0.0;
#pragma unroll
            for (int g = 0; g < SUBS; ++g) s += part2[g][el];
            r += s;  // elements beyond d load as zero, so the padding stays zero
            r_sum[mine] = r;
            if (r32 && mine < d) r32[mine] = (float)r;
            if (r64 && mine < d) r64[mine] = r;
        }
        rnew[el] = r;
    }
    __syncthreads();
    if (cur.nb == 0) return;
    const double2 r01 = *reinterpret_cast<const double2 *>(&rnew[quad * 4]);
    const double2 r23 = *reinterpret_cast<const double2 *>(&rnew[quad * 4 + 2]);
#pragma unroll
    for (int q = 0; q < PP; ++q) {
        double p = r01.x * ((double)cb[q].x - (double)ca[q].x);
        p = __builtin_fma(r01.y, (double)cb[q].y - (double)ca[q].y, p);
        p = __builtin_fma(r23.x, (double)cb[q].z - (double)ca[q].z, p);
        p = __builtin_fma(r23.y, (double)cb[q].w - (double)ca[q].w, p);
#pragma unroll
        for (int off = 1; off < QUADS; off <<= 1) p += __shfl_xor(p, off, 64);
        if (quad == 0 && grp * PP + q < sp) dots_out[(int64_t)block * sp + grp * PP + q] = p;
    }
}

// ---------------------------------------------------------------------------
// One step of the chain, serial part: one workgroup per walk.  Wavefronts 2 .. 9 add the wide
// launch's shares of the dots, in order; then the step is walked 64 pairs at a time.  Every
// wavefront below TILES holds the columns of one Gram tile in registers: the wavefront of a
// diagonal tile (s, s) walks the pairs 64 s .. 64 s + 63, then those of the tiles (s, w) add the
// decided signs' contributions to the t of the pairs of w.
// 64 pairs with what is around them take 0.7 us, 1.05 with a vote per step (walk_pairs).
//
// +1.0 if bit BIT of the (uniform) word is set, else -1.0, in a scalar register pair: a decided sign is then applied
// in two scalar instructions and one FMA (exact: +-1 times the entry).
template <int BIT>
__device__ __forceinline__ double sign_of_bit(uint32_t word) {
    uint32_t hi;
    asm("s_bitcmp1_b32 %1, %2\n\ts_cselect_b32 %0, %3, %4"
        : "=s"(hi) : "s"(word), "n"(BIT), "s"(0x3ff00000u), "s"(0xbff00000u) : "scc");
    return __hiloint2double((int)hi, 0);
}

constexpr int kShareThreads = 512;  // threads that add shares of the dots
constexpr int kWalkThreads = kShareThreads + 128;

// Workgroups (0, 8) .. (0, gridDim.y - 1) read the next step's rows, so that the wide launch after this one finds them in
// the L2 of its XCD (the XCDs take workgroups in turn; one walk).  A walk is one workgroup on an idle chip, and the
// wide launch is one round trip for its rows: 7.5 us of a step of 128 pairs of 7850 elements before, 30 000 such pairs 4334 -> 4198 us.
struct RowsAhead {
    StepRows rows;
    int32_t groups;  // of the wide launch
};

__device__ __forceinline__ void touch_rows(const RowsAhead &ahead, int index) {
    // the workgroups of XCD index % 8 share the lines (128 bytes) of its run of elements
    const int xcd = index & 7, per_xcd = (ahead.groups + 7) >> 3;
    const uint32_t threads = ((gridDim.y >> 3) - 1) * kWalkThreads;
    const int64_t e0 = (int64_t)xcd * per_xcd * kStepElems;
    const int64_t left = ahead.rows.d - e0;
    if (left <= 0) return;
    const uint32_t len = (uint32_t)(left < per_xcd * kStepElems ? left : per_xcd * kStepElems);
    const uint32_t lines = (len + 31) / 32 + 1, items = 2 * (uint32_t)ahead.rows.nb * lines;
    constexpr int FLIGHT = 4;
    for (uint32_t q0 = (uint32_t)((index >> 3) - 1) * kWalkThreads + threadIdx.x; q0 < items; q0 += FLIGHT * threads) {
        float x[FLIGHT];
#pragma unroll
        for (int u = 0; u < FLIGHT; ++u) {
            const uint32_t q = q0 + u * threads < items ? q0 + u * threads : q0, row = q / lines, line = q - row * lines;
            const float *a, *b;
            PairCursor(ahead.rows, (int)(row >> 1)).rows(ahead.rows, a, b);
            x[u] = (row & 1 ? b : a)[e0 + (32 * line < len ? 32 * line : len - 1)];
        }
#pragma unroll
        for (int u = 0; u < FLIGHT; ++u) asm volatile("" :: "v"(x[u]));
    }
}

template <int SB> constexpr int kWalkTiles = (SB / 64) * (SB / 64 + 1) / 2;

template <int SB, bool RANDOM>
__global__ __launch_bounds__(kWalkThreads) void chain_walk(const double *__restrict__ gram,
                                                               const double *__restrict__ dots_in, int dot_groups,
                                                               int sp, StepRows cur, int64_t half_n,
                                                               int8_t *__restrict__ eps_out,
                                                               int8_t *__restrict__ signs_out,
                                                               double *__restrict__ dots_out,
                                                               const float *__restrict__ uniforms, WalkStrides ws,
                                                               RowsAhead ahead)
{
    constexpr int SUBS = kShareThreads / SB;    // threads sharing one dot
    constexpr int FLIGHT = 32;                  // loads in flight per thread
    __shared__ double psub[SUBS][SB];
    __shared__ double tnow[SB];                 // t of every pair not walked yet
    __shared__ unsigned long long votes;        // signs of the tile just walked
    const int64_t w = blockIdx.x;
    // (decided by the workgroup's number alone: an argument to wait for first is 0.4 us more per launch)
    if (blockIdx.y > 0) {
        if (blockIdx.y >= 8) touch_rows(ahead, (int)blockIdx.y);
        return;
    }
    gram += w * ws.gram;
    dots_in += w * ws.dots;
    eps_out += w * kMaxStepPairs;
    signs_out += w * ws.out;
    if (dots_out) dots_out += w * ws.out;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // (uniform: tile addresses stay scalar)
    const int nb = cur.nb;
    const int nblk = (nb + 63) >> 6;            // tiles with pairs
    int tj = 0;
    while (tile_index(0, tj + 1) <= wave) ++tj;
    const int ti = wave - tile_index(0, tj);    // this wavefront's tile, if wave < TILES
    const bool holds = wave < kWalkTiles<SB> && tj < nblk;

    // Every wavefront passes 2 + 2 nblk barriers: after the shares, after their sum, and then two
    // per tile -- before its signs are used and before the next tile is walked.
    int passed = 0;
    auto pass_to = [&](int barriers) {
        for (; passed < barriers; ++passed) __syncthreads();
    };
    if (wave >= 2) {
        const int k = (tid - 128) % SB, s = (tid - 128) / SB;
        const double *src = dots_in + (k < sp ? k : sp - 1);
        double sum = 0.0;
        for (int g0 = s; g0 < dot_groups; g0 += FLIGHT * SUBS) {
            double v[FLIGHT];
#pragma unroll
            for (int u = 0; u < FLIGHT; ++u) {
                const int g = g0 + u * SUBS;
                v[u] = src[(int64_t)(g < dot_groups ? g : dot_groups - 1) * sp];
            }
#pragma unroll
            for (int u = 0; u < FLIGHT; ++u) sum += (g0 + u * SUBS < dot_groups) ? v[u] : 0.0;
        }
        psub[s][k] = sum;
        pass_to(1);
        if (s == 0) {
            double t = 0.0;
#pragma unroll
            for (int q = 0; q < SUBS; ++q) t += psub[q][k];
            tnow[k] = t;
        }
        pass_to(2);
    }
    // (the roles' branches are uniform; a tile is requested one walk before it is needed -- all at
    // once they delay each other -- and the first two before anything else)
    auto load_tile = [&](double (&col)[64]) {
        const double *g = gram + (int64_t)wave * kTileEntries + lane;
#pragma unroll
        for (int j = 0; j < 64; ++j) col[j] = g[j * kTilePairs];
    };
    const int kk = 64 * tj + lane;              // this lane's pair
    if (holds && ti == tj) {
        double col[64];
        pass_to(tj == 0 ? 0 : 2 + 2 * (tj > 2 ? tj - 2 : 0));
        load_tile(col);
        // flattened pair of this lane -> (worker, pair) slot of the [m][n/2] arrays
        int64_t slot = 0;
        if (kk < nb) {
            const uint32_t q = (uint32_t)(cur.i0 + kk);
            const uint32_t dq = q / (uint32_t)cur.m;
            slot = (int64_t)(q - dq * (uint32_t)cur.m) * half_n + (cur.k0 + dq);
        }
        const float my_u = (RANDOM && kk < nb) ? uniforms[slot] : 0.f;
        pass_to(2 + 2 * tj);
        bool plus;
        const double t = walk_pairs<64, RANDOM>(col, tnow[kk], my_u, plus);
        const unsigned long long all = __ballot(plus);
        if (lane == 0) votes = all;
        pass_to(2 + 2 * tj + 1);
        if (kk < nb) {
            eps_out[kk] = plus ? 1 : -1;
            signs_out[slot] = plus ? 1 : -1;
            if (dots_out) dots_out[slot] = t;
        }
    } else if (holds) {
        double col[64];
        pass_to(wave == 1 ? 0 : 2 + 2 * (ti > 1 ? ti - 1 : 0));
        load_tile(col);
        pass_to(2 + 2 * ti + 1);
        const unsigned long long v = votes;
        double t = tnow[kk];
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(v >> 32));
        static_for(std::make_integer_sequence<int, 64>{}, [&](auto jj) {
            constexpr int j = decltype(jj)::value;
            t = __builtin_fma(sign_of_bit<j & 31>(j < 32 ? lo : hi), col[j], t);
        });
        tnow[kk] = t;
    }
    pass_to(2 + 2 * nblk);
}

}  // namespace cdgrab
