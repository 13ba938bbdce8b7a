// Rows of at most 64 elements: a whole walk inside one workgroup (short walks and many of them; long ones: band_kernels.hpp).
//
// With so few elements a block of pairs is a few KB, the running sum is a few hundred bytes, and what
// a chain of launches spends between its steps is many times the work in them.  So one workgroup
// (per independent walk) keeps the running sum and walks all pairs, a block of 64 (rows of up to 16 elements) or
// 32 at a time, one barrier per block:
//   wavefront 0           walks block b, a step per pair, and applies each pair to the running sum in the shadow of
//                         the next step; then takes the dots of block b + 1;
//   the others but 4      meanwhile compute the Gram matrix of block b + 2 by MFMA and leave the differences of
//                         block b + 4, in double, in a ring in LDS (four blocks of loads in flight);
//   wavefront 4           writes the signs of block b - 1.
// Bound by the serial chain of wavefront 0, and there by what it issues: a step is 22 cycles (walk_sign), the pair
// applied to the running sum 12 more, the LDS reads for it and for the next block's columns 8; 450 cycles lie between two
// blocks (signs, barrier, dots).  Per 64 pairs of a long epoch: 1.25 us at 16 elements, 1.57 at 32, 2.57 at 64 (where
// the MFMAs of a block, about 100 cycles each, outlast its walk); 2.2, 2.7 and 3.8 with a vote per step and the
// running sum applied by other wavefronts after each walk.
// The double MFMA and the walk's additions share a SIMD's double-precision unit, so the walk has its SIMD
// nearly to itself: with Gram results computed there a step took 49 cycles.  Signs handed to another wavefront that
// applies them, and two walking wavefronts taking turns: 1.16 us at 16 elements, but 1.9 at 32 and 3.0 at 64.
// The next block's dots kept up to date by the walk itself, for which it needs twice the Gram results: 1.56 us at 16.
#pragma once
#include "band_kernels.hpp"

namespace cdgrab {

// p += x * (r of lane Q of the same row of sixteen lanes).  FIRST: r may be the result of the instruction before
// (a DPP operand needs two wait states).
template <int Q>
__device__ __forceinline__ void fma_row_lane(double &p, double r, double x, bool first) {
    if (first) asm volatile("s_nop 1\n\tv_fmac_f64_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+&v"(p) : "v"(r), "v"(x), "n"(Q));
    else asm volatile("v_fmac_f64_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+&v"(p) : "v"(r), "v"(x), "n"(Q));
}

constexpr int kNarrowAhead = 4;           // a block's differences come this many blocks before its walk

template <int DP, bool RANDOM>
struct NarrowArrays {
    // Blocks of 64 pairs spend less between walks, of 32 fewer Gram results per pair: six 16 x 16 ones per 64 pairs
    // instead of ten, of which three SIMDs take DP / 4 MFMAs each.
    static constexpr int NB = DP == 16 ? 64 : 32;
    static constexpr int DS = DP + 2;     // doubles per difference row in LDS (sixteen rows: distinct banks)
    static constexpr int GS = NB + 2;
    static constexpr int RING = kNarrowAhead + 1;  // blocks b .. b + kNarrowAhead are held
    __attribute__((aligned(16))) double diff[RING][NB * DS];
    double G[3][NB * GS];                 // minus the Gram matrices of blocks b .. b + 2; zero on and below the diagonal
    double walked[2][NB];                 // minus the dots of the block just walked
    float draw[RANDOM ? RING : 1][NB];
    unsigned long long votes[2];          // ... and its signs
};

// DP: padded row length (16, 32 or 64).  `pairs` consecutive pairs of every walk, the first at
// rows; the running sum is read from (fresh: starts at zero) and written back to r_sum, and to r32 / r64
// where they are not null.  BANDS: narrow_bands has filled `space`, walk_window takes all of them, and this walk is for launches with
// a value that is not finite.
template <int DP, int VW, bool RANDOM, bool BANDS>
__global__ __launch_bounds__(kNarrowThreads) void narrow_walk(StepRows rows, int pairs, int64_t half_n, int fresh, BandSpace space,
                                                              double *__restrict__ r_sum, float *__restrict__ r32,
                                                              double *__restrict__ r64,
                                                              int8_t *__restrict__ signs_out,
                                                              double *__restrict__ dots_out,
                                                              const float *__restrict__ uniforms, WalkStrides ws)
{
    constexpr int NB = NarrowArrays<DP, RANDOM>::NB, DS = NarrowArrays<DP, RANDOM>::DS, GS = NarrowArrays<DP, RANDOM>::GS;
    constexpr int AHEAD = kNarrowAhead, RING = NarrowArrays<DP, RANDOM>::RING;
    constexpr int QUADS = DP / 4;
    constexpr int LOADERS = 256;          // threads that bring in rows, PER items of (pair, four elements) each
    constexpr int PER = NB * QUADS / LOADERS;
    constexpr int FLIGHT = 4;             // blocks of loads in flight
    using Arrays = NarrowArrays<DP, RANDOM>;
    // (arrays of their own where there is no window: members of one variable could be each other's neighbours to the compiler, 2 - 4 %)
    __shared__ __attribute__((aligned(16))) double own_diff[RING][NB * DS];
    __shared__ double own_G[3][NB * GS];
    __shared__ double own_walked[2][NB];
    __shared__ float own_draw[RANDOM ? RING : 1][NB];
    __shared__ unsigned long long own_votes[2];
    __shared__ union { BandArrays<DP, RANDOM> window; Arrays inside; } shared;
    auto &diff = *[&] { if constexpr (BANDS) return &shared.inside.diff; else return &own_diff; }();
    auto &G = *[&] { if constexpr (BANDS) return &shared.inside.G; else return &own_G; }();
    auto &walked = *[&] { if constexpr (BANDS) return &shared.inside.walked; else return &own_walked; }();
    auto &draw = *[&] { if constexpr (BANDS) return &shared.inside.draw; else return &own_draw; }();
    auto &votes = *[&] { if constexpr (BANDS) return &shared.inside.votes; else return &own_votes; }();
    const int64_t w = blockIdx.x;
    rows.base += w * ws.rows;
    r_sum += w * ws.r;
    signs_out += w * ws.out;
    if (dots_out) dots_out += w * ws.out;
    if constexpr (BANDS) {
        auto &s = shared.window;
        if (walk_window<DP, RANDOM>(s.ring, s.running, s.verdict, s.walked, s.start, s.draw, &s.strange, rows, pairs, half_n,
                                    fresh, space, r_sum, r32, r64, signs_out, dots_out)) return;
        // what is on its way to LDS has to be there before the place is used again
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        narrow_barrier();
    }
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t d = rows.d;
    const int blocks = (pairs + NB - 1) / NB;

    // Barriers: three before the loop, then one at the end of every block: its signs are there, and what the next
    // block needs.
    if (wave == 0) {
        // A row of sixteen lanes holds sixteen elements of the running sum (rows of 16: all four the same, of 32: the
        // first two and the last two), from where they reach its lanes' dots by DPP.
        constexpr int SETS = DP == 64 ? 2 : 1;  // pairs per lane in the dots
        const int e = DP == 16 ? lane & 15 : DP == 32 ? (lane & 15) + 16 * (lane >> 5) : lane;
        const int k = lane % NB, pair = DP == 64 ? lane & 15 : k;
        double c[NB];            // this lane's column of the Gram matrix, replaced by the next block's as it is used
        double own[SETS][16];    // the next block's differences, of this lane's pairs and its row's elements
        double ahead[8];         // differences of the next eight pairs, this lane's element
        double r = e < d && !fresh ? r_sum[e] : 0.0;
        // u = -t, so that the sign bit is the decision: eps = +1 (t <= 0) where it is clear.  Never -0: differences
        // of equal numbers are +0, and so is every sum with +0.
        double u = 0.0;
        auto own_row = [&](int b, int s) { return &diff[b % RING][(pair + 16 * s) * DS + (e & ~15)]; };
        auto take_dots = [&] {
            double p[SETS][4] = {};
            static_for(std::make_integer_sequence<int, 16>{}, [&](auto qq) {
                constexpr int q = decltype(qq)::value;
#pragma unroll
                for (int s = 0; s < SETS; ++s) fma_row_lane<q>(p[s][q & 3], r, own[s][q], q == 0 && s == 0);
            });
            double sum[SETS];
#pragma unroll
            for (int s = 0; s < SETS; ++s) {
                sum[s] = (p[s][0] + p[s][1]) + (p[s][2] + p[s][3]);
                if (DP == 64) sum[s] = sum_across_16(sum[s]);
                if (DP >= 32) sum[s] = sum_across_32(sum[s]);
            }
            u = 0.0 - ((lane & 16) ? sum[SETS - 1] : sum[0]);
        };
        narrow_barrier();
        narrow_barrier();
#pragma unroll
        for (int j = 0; j < NB; ++j) c[j] = G[0][j * GS + k];
#pragma unroll
        for (int j = 0; j < 8; ++j) ahead[j] = diff[0][j * DS + e];
#pragma unroll
        for (int s = 0; s < SETS; ++s)
#pragma unroll
            for (int q = 0; q < 16; ++q) own[s][q] = own_row(0, s)[q];
        take_dots();
        narrow_barrier();
        for (int b = 0; b < blocks; ++b) {
            // randomized rule (PairBalance's RandomizedBalance subroutine, Sec. 3.2): with
            // c = z1 - z2 = -d, the first row gets +1 with probability p = (1 - <r,c>)/2 =
            // (1 + t)/2, so the exported sign (of the second row) is -1 when the draw is below p:
            // the sign of their difference (as in walk_pairs, which says which draws have one).
            const float dr = RANDOM ? draw[b % RING][k] : 0.f;
            auto rule = [&](double tv) { return RANDOM ? !((double)dr < 0.5 * (1.0 + tv)) : (tv <= 0.0); };
            auto vote = [&](int j) { return ((__ballot(rule(0.0 - u)) >> j) & 1ull) ? 0u : 0x80000000u; };
            const double u0 = u, r0 = r, draw_of = (double)dr + 0.0;
            const double *col = &G[(b + 1) % 3][k];  // (of a block that does not exist: slots of the rings, not used)
            const double *here = &diff[b % RING][e], *next = &diff[(b + 1) % RING][e];
            uint32_t before = 0;
            // what a step has used is replaced a step or two later (two rows per instruction), when the running sum
            // follows it; between a step's v_readlane and the use of what it read are two wait states to fill
            auto follow = [&](auto jj) {
                constexpr int j = decltype(jj)::value;
                r += sign_flipped_by(ahead[j & 7], before);
                asm volatile("" : "+v"(r));  // (here, not all of them at the end)
            };
            auto replace = [&](auto jj) {
                constexpr int j = decltype(jj)::value;  // odd
                c[j - 1] = col[(j - 1) * GS];
                c[j] = col[j * GS];
                const double *from = j + 8 < NB ? here + (j + 7) * DS : next + (j + 7 - NB) * DS;
                ahead[(j - 1) & 7] = from[0];
                ahead[j & 7] = from[DS];
                if constexpr (j < 16 * SETS) {
                    constexpr int s = j / 16, q = j % 16 - 1;
                    own[s][q] = own_row(b + 1, s)[q];
                    own[s][q + 1] = own_row(b + 1, s)[q + 1];
                }
            };
            static_for(std::make_integer_sequence<int, NB>{}, [&](auto jj) {
                constexpr int j = decltype(jj)::value;
                const uint32_t flip = (uint32_t)walk_sign<j>(RANDOM ? __builtin_fma(-0.5, 1.0 - u, draw_of) : u);
                __builtin_amdgcn_sched_barrier(0);  // (left alone, the compiler reads everything at once)
                if constexpr (j > 0) follow(std::integral_constant<int, j - 1>{});
                __builtin_amdgcn_sched_barrier(0);
                u += sign_flipped_by(c[j], flip);
                before = flip;
                if constexpr (j > 0 && j % 2 == 0) replace(std::integral_constant<int, j - 1>{});
                __builtin_amdgcn_sched_barrier(0);
            });
            follow(std::integral_constant<int, NB - 1>{});
            replace(std::integral_constant<int, NB - 1>{});
            // a t that is not a number, or such a draw, has no sign to go by: walk again by comparison
            if (__ballot(u != u || (RANDOM && !isfinite(dr)))) {
                u = u0;
                r = r0;
                if (BANDS && __ballot(r != r)) {  // every dot from here on is not a number: no rule to wait for
                    const uint32_t flip = RANDOM ? 0u : 0x80000000u;
#pragma unroll 8
                    for (int j = 0; j < NB; ++j) r += sign_flipped_by(here[j * DS], flip);
                } else for (int j = 0; j < NB; ++j) {
                    const uint32_t flip = vote(j);
                    u += sign_flipped_by(G[b % 3][j * GS + k], flip);
                    r += sign_flipped_by(here[j * DS], flip);
                }
            }
            const unsigned long long all = __ballot(rule(0.0 - u));
            if (lane == 0) votes[b & 1] = all;
            walked[b & 1][k] = u;
            narrow_barrier();
            take_dots();
        }
        if (e < d && (DP == 64 || (lane & 16) == 0) && (DP != 16 || lane < 16)) {
            r_sum[e] = r;
            if (r32) r32[e] = (float)r;
            if (r64) r64[e] = r;
        }
        return;
    }

    if (wave == 4) {  // (on the walker's SIMD: it issues little)
        narrow_barrier();
        narrow_barrier();
        narrow_barrier();
        for (int b = 0; b < blocks; ++b) {
            narrow_barrier();
            const int kk = b * NB + lane;
            const uint32_t q = (uint32_t)rows.i0 + (uint32_t)kk, dq = q / (uint32_t)rows.m;
            const int64_t slot = (int64_t)(q - dq * (uint32_t)rows.m) * half_n + (rows.k0 + dq);
            if (lane < NB && kk < pairs) {
                signs_out[slot] = (votes[b & 1] >> lane) & 1ull ? 1 : -1;
                if (dots_out) dots_out[slot] = 0.0 - walked[b & 1][lane];
            }
        }
        return;
    }

    // ---- rows
    const int hw = wave < 4 ? wave - 1 : wave - 2, h = hw * 64 + lane;  // of six
    const bool loads = h < LOADERS;  // (uniform per wavefront)
    struct Rows { float4_t a[PER], b[PER]; float u; };  // as loaded: what does not belong is cut off in store()
    // Every thread keeps its pairs of the block and its four elements; from block to block its rows move on by
    // NB pairs, i.e. by a fixed distance plus another one whenever the worker index wraps around.
    const bool dense = rows.layout == kDense;
    const int di = dense ? NB % rows.m : 0, wrap_at = dense ? rows.m : 1;
    const int64_t dk = dense ? NB / rows.m : 0;
    const int64_t row_step = dense ? di * rows.n + 2 * dk : (rows.layout == kStaged ? 2 * NB : NB);
    const int64_t step = row_step * d, wrap = dense ? (2 - rows.m * rows.n) * d : 0;
    const int e = (h & (QUADS - 1)) * 4, dn = (int)d;
    const float *at[PER];
    int64_t at_k[PER];
    int worker[PER], pair[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        pair[u] = ((h + u * LOADERS) / QUADS) % NB;
        const PairCursor p(rows, pair[u]);
        const float *b;
        p.rows(rows, at[u], b);
        worker[u] = (int)p.i;
        at_k[u] = p.k;
    }
    auto load = [&](Rows &x, int blk) {  // called for blocks 0, 1, 2, .. in turn
        if (!loads || blk >= blocks) return;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const bool have = blk * NB + pair[u] < pairs;  // (else the first pair again)
            const float *a = have ? at[u] : rows.base + (dense ? rows.i0 * rows.n + 2 * rows.k0 : 0) * d;
            const float *b = rows.layout == kCentred ? rows.centre : a + d;
            if constexpr (VW == kTiny) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    x.a[u][q] = a[e + q < dn ? e + q : 0];
                    x.b[u][q] = b[e + q < dn ? e + q : 0];
                }
            } else {  // a group that reaches beyond the row reads the row's last four elements
                const int from = e <= dn - 4 ? e : dn - 4;
                x.a[u] = load_four<true>(a + from);
                x.b[u] = load_four<true>(b + from);
            }
            if (RANDOM && (PER == 1 || e < 4 * PER))  // (quad u of a row brings in the draw of its item u)
                if (PER == 1 || e == 4 * u) x.u = uniforms[have ? worker[u] * half_n + at_k[u] : rows.i0 * half_n + rows.k0];
            worker[u] += di;
            at[u] += step;
            at_k[u] += dk;
            if (worker[u] >= wrap_at) {
                worker[u] -= wrap_at;
                at[u] += wrap;
                ++at_k[u];
            }
        }
    };
    auto store = [&](const Rows &x, int blk) {  // (a pair that does not exist becomes zero)
        if (!loads || blk >= blocks) return;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int from = VW == kTiny || e <= dn - 4 ? e : dn - 4;
            const bool have = blk * NB + pair[u] < pairs;
            double v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = (double)x.b[u][q] - (double)x.a[u][q];
            // element e + q sits at position e - from + q of what was loaded (in binary steps)
            const int sh = e - from;
            const bool s1 = sh & 1, s2 = sh & 2;
            const double y0 = s1 ? v[1] : v[0], y1 = s1 ? v[2] : v[1], y2 = s1 ? v[3] : v[2], y3 = v[3];
            const double z0 = s2 ? y2 : y0, z1 = s2 ? y3 : y1;
            double2 *p = reinterpret_cast<double2 *>(&diff[blk % RING][pair[u] * DS + e]);
            p[0] = make_double2(have && e < dn ? z0 : 0.0, have && e + 1 < dn ? z1 : 0.0);
            p[1] = make_double2(have && e + 2 < dn ? y2 : 0.0, have && e + 3 < dn ? y3 : 0.0);
            if (RANDOM && e == 4 * u) draw[blk % RING][pair[u]] = x.u;
        }
    };

    // ---- Gram matrix: this wavefront's 16 x 16 results of a block, of ten (the first four wavefronts two) or of three
    constexpr int RESULTS = NB == 64 ? 2 : 1;
    const int grams = NB == 64 ? (hw < 4 ? 2 : 1) : hw < 3 ? 1 : 0;
    int ti[RESULTS], tj[RESULTS];
#pragma unroll
    for (int i = 0; i < RESULTS; ++i) {
        const int result = hw + 6 * i;
        tj[i] = result >= 6 ? 3 : result >= 3 ? 2 : result >= 1 ? 1 : 0;
        ti[i] = result - tile_index(0, tj[i]);
    }
    const int mrow = lane & 15, kslot = lane >> 4;
    double ga[RESULTS][DP / 4], gb[RESULTS][DP / 4];
    double4_t acc[RESULTS];
    auto gram_read = [&](int blk) {
#pragma unroll
        for (int i = 0; i < RESULTS; ++i)
            if (i < grams) {  // (uniform)
                const double *A = diff[blk % RING] + (16 * ti[i] + mrow) * DS + kslot;
                const double *B = diff[blk % RING] + (16 * tj[i] + mrow) * DS + kslot;
#pragma unroll
                for (int q = 0; q < DP / 4; ++q) {
                    ga[i][q] = A[4 * q];
                    gb[i][q] = B[4 * q];
                }
            }
    };
    auto gram_multiply = [&] {
#pragma unroll
        for (int i = 0; i < RESULTS; ++i)
            if (i < grams) {
                acc[i] = (double4_t){0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int q = 0; q < DP / 4; ++q) acc[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(ga[i][q], gb[i][q], acc[i], 0, 0, 0);
            }
    };
    auto gram_write = [&](int blk) {
#pragma unroll
        for (int i = 0; i < RESULTS; ++i)
            if (i < grams) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    int row, col;
                    mfma_f64_16x16_coord(lane, v, row, col);
                    if (ti[i] != tj[i] || row < col) G[blk % 3][(16 * ti[i] + row) * GS + 16 * tj[i] + col] = 0.0 - acc[i][v];
                }
            }
    };

    Rows x[FLIGHT];
#pragma unroll
    for (int i = 0; i < FLIGHT; ++i) load(x[i], i);
    for (int q = h; q < 3 * NB * GS; q += 384) (&G[0][0])[q] = 0.0;
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) {
        store(x[i % FLIGHT], i);
        load(x[i % FLIGHT], i + FLIGHT);
    }
    narrow_barrier();
#pragma unroll
    for (int blk = 0; blk < 2; ++blk) {
        gram_read(blk);
        gram_multiply();
        gram_write(blk);
    }
    gram_read(2);  // (of a block that does not exist: a slot of the ring, not used)
    narrow_barrier();
    narrow_barrier();  // (the walker has what it needs of block 0)
    for (int b0 = 0; b0 < blocks; b0 += FLIGHT)
#pragma unroll
        for (int i = 0; i < FLIGHT; ++i) {
            const int b = b0 + i;
            if (b < blocks) {  // (uniform)
                gram_multiply();
                store(x[(AHEAD + i) % FLIGHT], b + AHEAD);
                load(x[(AHEAD + i) % FLIGHT], b + AHEAD + FLIGHT);
                gram_read(b + 3);
                gram_write(b + 2);
                narrow_barrier();
            }
        }
}

}  // namespace cdgrab
