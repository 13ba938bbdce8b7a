// Rows of at most 64 elements, long walks: everything that does not wait for signs is computed beforehand by the
// whole chip, and a walk streams it in.
//
// narrow_bands   for every block of sixteen pairs, minus its Gram results with itself and with the next three blocks, and its
//                differences in double, into a workspace, and whether all of its values are finite;
// walk_window    one workgroup per walk, which reads them (the Gram results straight into a ring in LDS):
//   wavefront 0     walks.  Its lanes are a window of 64 pairs, a row of sixteen lanes per block: while block b is
//                   walked, the dots of blocks b + 1 .. b + 3 take its signs too, so that no dot waits for the running
//                   sum.  Little but a step's three instructions and an LDS read per two steps is issued;
//   wavefront 1     (and 6, for rows of more than 32) applies block b - 1 to the running sum while b is walked;
//   wavefront 2     takes the dots of block b + 2 with the running sum that ends before block b - 1;
//   wavefront 5     writes signs and dots, four blocks at a time;
//   wavefronts 3, 7 bring in the Gram results;
//   wavefront 4     looks, before the first block, whether a value of the launch or of the running sum is not finite.  If so, all go
//                   on in narrow_walk, where only the blocks without a sign to go by are walked twice: an infinity in the
//                   first of 25 000 pairs of 16 / 32 / 64 elements 521 / 620 / 1031 us, a draw that is no number 614 / 717 /
//                   1285 (walked pair by pair from there on by wavefront 1: 3819 / 4217 / 4682 and 5727 / 6049 / 6512).
//                   Finite values have finite dots: 64 products of a sum of 2^63 numbers below 2^129 and such a number.
// One barrier per block, half way into its walk: what the block before has left in LDS is there by then, so that nothing of
// it is waited for on the chain.
//
// Bound by the serial chain of wavefront 0: a step is 24.6 cycles of its own (three dependent instructions and the wait states
// between them) and 4 more for its share of an LDS read; what a block adds around its barrier is 5 to 6 per step.  Per 64
// pairs of a long epoch 0.91 us at 16 elements, 0.93 at 32, 1.36 at 64, where 24 KB per block pass through one CU; 1.23, 1.54 and
// 2.54 with everything in one workgroup (narrow_kernels.hpp): 500 000 pairs of 16 elements 9657 -> 7228 us.  A check for dots
// that are not finite in the walk itself cost 40 cycles per block; a window of 64 pairs is three blocks of slack, one for
// each wavefront a sign passes through.
#pragma once
#include "narrow_common.hpp"

namespace cdgrab {

constexpr int kBandBlock = 16;
constexpr int kBandDoubles = kBandBlock * 64;  // Gram results of a block: [pair / 2][lane of the walk][pair % 2]
// doubles of workspace per block: results, differences ([pair / 2][element][pair % 2]), draws
constexpr int64_t band_doubles(int dp) { return kBandDoubles + kBandBlock * dp + kBandBlock / 2; }

// A walk takes a multiple of this many blocks, the last ones of pairs that do not exist and are zero: where the loops of loads
// in flight have no exit in between, the compiler knows how many are.
constexpr int kBandStride = 8;

struct BandSpace {
    double *base;
    int64_t walk;  // doubles between the walks'
    int blocks;    // a multiple of kBandStride
    __device__ __forceinline__ double *band(int64_t w) const { return base + w * walk; }
    __device__ __forceinline__ double *diff(int64_t w) const { return band(w) + (int64_t)blocks * kBandDoubles; }
    template <int DP> __device__ __forceinline__ float *draws(int64_t w) const {
        return reinterpret_cast<float *>(diff(w) + (int64_t)blocks * kBandBlock * DP);
    }
    // per block: 0 where all of its differences and draws are finite, else 1
    template <int DP> __device__ __forceinline__ uint8_t *strange(int64_t w) const {
        return reinterpret_cast<uint8_t *>(draws<DP>(w) + (int64_t)blocks * kBandBlock);
    }
};
// A walk's, in doubles (a multiple of 256 bytes).
constexpr int64_t band_walk_doubles(int dp, int64_t blocks) { return blocks * band_doubles(dp) + (blocks + 255) / 256 * 32; }

// A wavefront per block.  (k0, i0): where the first pair's outputs and draws are.
template <int DP, int VW>
__global__ __launch_bounds__(kThreads) void narrow_bands(StepRows rows, int64_t k0, int32_t i0, int pairs, int64_t half_n,
                                                         BandSpace space, const float *__restrict__ uniforms, WalkStrides ws)
{
    constexpr int PER = DP / 4;  // elements per lane: lane (pair = lane % 16, quarter = lane / 16)
    const int lane = threadIdx.x & 63, mrow = lane & 15, kslot = lane >> 4;
    const int c = blockIdx.x * kWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (c >= space.blocks) return;
    const int64_t w = blockIdx.y;
    rows.base += w * ws.rows;
    auto take = [&](double (&x)[PER], int pair) {  // (a pair that does not exist is zero)
        const bool have = pair < pairs;
        const float *a, *b;
        PairCursor(rows, have ? pair : 0).rows(rows, a, b);
        float4 va[PER / 4], vb[PER / 4];
#pragma unroll
        for (int q = 0; q < PER / 4; ++q) {
            va[q] = load4_nb<VW, false>(a, have, kslot * PER + 4 * q, rows.d);
            vb[q] = load4_nb<VW, false>(b, have, kslot * PER + 4 * q, rows.d);
        }
#pragma unroll
        for (int q = 0; q < PER / 4; ++q) {
            x[4 * q] = (double)vb[q].x - (double)va[q].x;
            x[4 * q + 1] = (double)vb[q].y - (double)va[q].y;
            x[4 * q + 2] = (double)vb[q].z - (double)va[q].z;
            x[4 * q + 3] = (double)vb[q].w - (double)va[q].w;
        }
    };
    // rows of the result are pairs in the order 0 4 8 12 1 5 ..: a lane then holds four consecutive ones
    double A[PER], B[4][PER];
    take(A, c * kBandBlock + 4 * (mrow & 3) + (mrow >> 2));
#pragma unroll
    for (int i = 0; i < 4; ++i) take(B[i], (c + i) * kBandBlock + mrow);
    double *diff = space.diff(w) + (int64_t)c * kBandBlock * DP + ((mrow >> 1) * DP + kslot * PER) * 2 + (mrow & 1);
#pragma unroll
    for (int q = 0; q < PER; ++q) diff[2 * q] = B[0][q];
    double rest = 0.0;  // stays zero if all values are finite
#pragma unroll
    for (int q = 0; q < PER; ++q) rest = __builtin_fma(B[0][q], 0.0, rest);
    if (uniforms && kslot == 0) {
        const int pair = c * kBandBlock + mrow;
        const uint32_t q = (uint32_t)i0 + (uint32_t)(pair < pairs ? pair : 0), dq = q / (uint32_t)rows.m;
        const float draw = uniforms[(int64_t)(q - dq * (uint32_t)rows.m) * half_n + (k0 + dq)];
        space.draws<DP>(w)[pair] = draw;
        rest = __builtin_fma((double)draw, 0.0, rest);
    }
    const unsigned long long strange = __ballot(rest != 0.0);
    if (lane == 0) space.strange<DP>(w)[c] = strange ? 1 : 0;
    double *band = space.band(w) + (int64_t)c * kBandDoubles;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        double4_t acc = (double4_t){0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int q = 0; q < PER; ++q) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(A[q], B[i][q], acc, 0, 0, 0);
        double v[4];  // zero for the block's own pairs up to the one that is walked
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = i == 0 && mrow <= 4 * kslot + q ? 0.0 : 0.0 - acc[q];
        double2 *to = reinterpret_cast<double2 *>(band + 4 * kslot * 64 + (((c + i) & 3) * 16 + mrow) * 2);
        to[0] = make_double2(v[0], v[1]);
        to[64] = make_double2(v[2], v[3]);
    }
}

constexpr int kBandFlight = 8;                  // blocks of Gram results on their way from memory ...
constexpr int kBandRing = kBandFlight + 4;      // ... of those held

template <int DP, bool RANDOM>
struct BandArrays {
    __attribute__((aligned(16))) double ring[kBandRing][kBandDoubles];
    __attribute__((aligned(16))) double running[4][DP];  // the running sum before block b
    // of the last blocks, in their own lanes: sign bit: the pair's sign is -1; minus the dot, unless RANDOM
    __attribute__((aligned(16))) double verdict[2][4][64];
    double walked[RANDOM ? 2 : 1][4][64];  // RANDOM: minus the dot
    double start[4][64];      // minus the dots with the running sum three blocks back, in the block's lanes, else 0
    double draw[4][kBandBlock];
    int strange;              // not all values of the launch are finite
};

// Arguments as of narrow_walk, behind its arrays in LDS.  False, and nothing done, if a value of the launch is not finite.
template <int DP, bool RANDOM>
__device__ __forceinline__ bool walk_window(double (*ring)[kBandDoubles], double (*running)[DP], double (*verdict)[4][64],
                                            double (*walked)[4][64], double (*start)[64], double (*draw)[kBandBlock], int *strange,
                                            const StepRows &rows, int pairs, int64_t half_n, int fresh, const BandSpace &space,
                                            double *__restrict__ r_sum, float *__restrict__ r32, double *__restrict__ r64,
                                            int8_t *__restrict__ signs_out, double *__restrict__ dots_out)
{
    constexpr int NB = kBandBlock;
    constexpr int FLIGHT = kBandFlight, RING = kBandRing;
    constexpr int AHEAD = 8, AHEAD_DOTS = DP == 64 ? 4 : 8;  // blocks of differences on their way
    constexpr int SE = DP < 32 ? DP : 32;    // elements of the running sum per wavefront: rows of 64 take two
    static_assert(kBandStride % AHEAD == 0 && kBandStride % AHEAD_DOTS == 0 && kBandStride % 4 == 0, "whole rounds");
    static_assert(RING % 4 == 0, "the window's four blocks have fixed places");
    const int64_t w = blockIdx.x, d = rows.d;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int blocks = space.blocks;
    auto slot_of = [&](int pair) {  // its place in the [m][n/2] arrays
        const uint32_t q = (uint32_t)rows.i0 + (uint32_t)pair, dq = q / (uint32_t)rows.m;
        return (int64_t)(q - dq * (uint32_t)rows.m) * half_n + (rows.k0 + dq);
    };
    auto finite = [&] { return __builtin_amdgcn_readfirstlane(*strange) == 0; };  // (from the first barrier on)

    // LDS reads right after a barrier meet the walker's.  25 000 pairs of 16 / 32 / 64 elements, without -> with these sixteen cycles in
    // wavefronts 1 and 2: 390 -> 374, 388 -> 380, 548 -> 549 us, randomized 484 -> 471, 486 -> 479, 566 -> 576 (hence not
    // in 2 there); 64 cycles in wavefront 1, which then comes late to the next barrier, 401 at 16 elements.
    auto step_aside = [] { asm volatile("s_nop 15"); };

    // Barriers of every wavefront: one before the first block, one in each, one after the last.
    if (wave == 0) {
        double col[NB];  // this lane's Gram results with the pairs of the block, replaced by the next block's as they are used
        double keep[4];  // 0 in the lanes of row R, else 1
#pragma unroll
        for (int R = 0; R < 4; ++R) keep[R] = (lane >> 4) == R ? 0.0 : 1.0;
        narrow_barrier();
        if (!finite()) return false;
#pragma unroll
        for (int j = 0; j < NB - 2; j += 2) {
            const double2 x = *reinterpret_cast<const double2 *>(&ring[0][j * 64 + 2 * lane]);
            col[j] = x.x;
            col[j + 1] = x.y;
        }
        double u = start[0][lane];  // minus the dot, never -0 (as in narrow_walk)
        double draw_of = RANDOM ? draw[0][lane & 15] : 0.0;
        auto margin = [&] { return RANDOM ? __builtin_fma(-0.5, 1.0 - u, draw_of) : u; };
        int place = 0;  // in the ring, of the four blocks' first
        for (int b0 = 0; b0 < blocks; b0 += 4) {
            const int group = (b0 >> 2) & 1, after = place + 4 == RING ? 0 : place + 4;
            const double *here = &ring[place][2 * lane], *then = &ring[after][2 * lane];
            static_for(std::make_integer_sequence<int, 4>{}, [&](auto row) {
                constexpr int R = decltype(row)::value;
                const double *now = here + R * kBandDoubles, *next = R < 3 ? now + kBandDoubles : then;
                double add = 0.0, draw_next = 0.0;
                static_for(std::make_integer_sequence<int, NB>{}, [&](auto jj) {
                    constexpr int j = decltype(jj)::value;
                    const uint32_t flip = (uint32_t)walk_sign<16 * R + j>(margin());
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (j % 2 == 0) {  // (in the wait for the sign; two steps after their last use)
                        constexpr int at = (j + NB - 2) % NB;
                        const double2 x = *reinterpret_cast<const double2 *>((j == 0 ? now : next) + at * 64);
                        col[at] = x.x;
                        col[at + 1] = x.y;
                    }
                    if constexpr (j == 8) {
                        // five LDS reads have been issued since the last block's verdicts were written
                        asm volatile("s_waitcnt lgkmcnt(4)\n\ts_barrier" ::: "memory");
                        add = start[(R + 1) & 3][lane];
                        if (RANDOM) draw_next = draw[(R + 1) & 3][lane & 15];
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    u += sign_flipped_by(col[j], flip);
                    __builtin_amdgcn_sched_barrier(0);
                });
                verdict[group][R][lane] = margin();
                if (RANDOM) walked[group][R][lane] = u;
                // this block's lanes start at zero again, the next one's take their start
                u = __builtin_fma(u, keep[R], add);
                draw_of = draw_next;
            });
            place = after;
        }
        narrow_barrier();
    } else if (wave == 1 || (DP > SE && wave == 6)) {
        constexpr int PP = NB * SE / 64;  // pairs per lane
        const int e = lane % SE + (wave == 6 ? SE : 0), first = lane / SE * PP;
        const double *diff = space.diff(w) + first * DP + 2 * e;
        double2 x[AHEAD][PP / 2];
        auto load = [&](double2 (&v)[PP / 2], int b) {  // (a block that does not exist: the last one, not used)
            const double2 *p = reinterpret_cast<const double2 *>(diff + (int64_t)(b < blocks ? b : blocks - 1) * NB * DP);
#pragma unroll
            for (int i = 0; i < PP / 2; ++i) v[i] = p[i * DP];
        };
        double r = e < d && !fresh ? r_sum[e] : 0.0;
        if (lane < SE) running[0][e] = r;
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) load(x[i], i);
        narrow_barrier();
        if (!finite()) return false;
        narrow_barrier();
        for (int b0 = 0; b0 < blocks; b0 += AHEAD)
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) {
                const int b = b0 + i;
                narrow_barrier();
                step_aside();
                const uint32_t *signs = reinterpret_cast<const uint32_t *>(&verdict[(b >> 2) & 1][b & 3][16 * (b & 3)] + first);
                double sum[2] = {0.0, 0.0};
#pragma unroll
                for (int q = 0; q < PP / 2; ++q) {
                    sum[0] += sign_flipped_by(x[i][q].x, signs[4 * q + 1]);
                    sum[1] += sign_flipped_by(x[i][q].y, signs[4 * q + 3]);
                }
                double all = sum[0] + sum[1];
                if (SE == 16) all = sum_across_16(all);
                r += sum_across_32(all);
                if (lane < SE) running[(b + 1) & 3][e] = r;
                load(x[i], b + AHEAD);
            }
        if (lane < SE && e < d) {
            r_sum[e] = r;
            if (r32) r32[e] = (float)r;
            if (r64) r64[e] = r;
        }
    } else if (wave == 2) {
        constexpr int PE = DP / 8;  // elements per lane: lane (two pairs, part of the elements)
        const int two = lane & 7, part = lane >> 3, pair = 2 * two + (part & 1);  // (the pair whose dot it ends with)
        const double *diff = space.diff(w) + (two * DP + part * PE) * 2;
        const float *draws = space.draws<DP>(w) + pair;
        double2 y[AHEAD_DOTS][PE];
        double rr[PE];
        float f[AHEAD_DOTS];
        auto load = [&](int i, int b) {
            const int64_t at = b < blocks ? b : blocks - 1;
            const double2 *p = reinterpret_cast<const double2 *>(diff + at * NB * DP);
#pragma unroll
            for (int q = 0; q < PE; ++q) y[i][q] = p[q];
            if (RANDOM) f[i] = draws[at * NB];
        };
        auto dots = [&](int i, int b) {
            double even = 0.0, odd = 0.0;
#pragma unroll
            for (int q = 0; q < PE; ++q) {
                even = __builtin_fma(rr[q], y[i][q].x, even);
                odd = __builtin_fma(rr[q], y[i][q].y, odd);
            }
            even = dpp_add<0x128>(even);  // row_ror 8: the other eight of sixteen
            odd = dpp_add<0x128>(odd);
            const double sum = sum_across_32(sum_across_16((part & 1) ? odd : even));
            start[b & 3][(lane & 48) + pair] = (lane >> 4) == (b & 3) ? 0.0 - sum : 0.0;
            if (RANDOM && lane < NB) draw[b & 3][pair] = (double)f[i] + 0.0;  // (-0 is taken as 0)
        };
#pragma unroll
        for (int i = 0; i < AHEAD_DOTS; ++i) load(i, i);
#pragma unroll
        for (int q = 0; q < PE; ++q) rr[q] = part * PE + q < d && !fresh ? r_sum[part * PE + q] : 0.0;
        dots(0, 0);
        dots(1, 1);
        load(0, AHEAD_DOTS);
        load(1, AHEAD_DOTS + 1);
        narrow_barrier();
        if (!finite()) return false;
        for (int b0 = 0; b0 < blocks; b0 += AHEAD_DOTS)
#pragma unroll
            for (int i = 0; i < AHEAD_DOTS; ++i) {
                const int b = b0 + i;
                narrow_barrier();
                if (DP < 64) step_aside();
                const double2 *src = reinterpret_cast<const double2 *>(&running[b > 0 ? (b - 1) & 3 : 0][part * PE]);
#pragma unroll
                for (int q = 0; q < PE / 2; ++q) {
                    const double2 v = src[q];
                    rr[2 * q] = v.x;
                    rr[2 * q + 1] = v.y;
                }
                dots((i + 2) % AHEAD_DOTS, b + 2);
                load((i + 2) % AHEAD_DOTS, b + 2 + AHEAD_DOTS);
            }
        narrow_barrier();
    } else if (wave == 5) {
        narrow_barrier();
        if (!finite()) return false;
        narrow_barrier();
        for (int b = 0; b < blocks; ++b) {
            narrow_barrier();
            if ((b & 3) != 3) continue;
            const int group = (b >> 2) & 1, kk = (b - 3) * NB + lane;
            const double v = verdict[group][lane >> 4][lane];
            const double u = RANDOM ? walked[RANDOM ? group : 0][lane >> 4][lane] : v;
            if (kk < pairs) {
                const int64_t slot = slot_of(kk);
                signs_out[slot] = __double2hiint(v) < 0 ? -1 : 1;
                if (dots_out) dots_out[slot] = 0.0 - u;
            }
        }
    } else if (wave == 3 || wave == 7) {
        constexpr int LOADS = kBandDoubles / 2 / 128;  // of 1 KB each, per block and wavefront
        const int half = wave == 7 ? kBandDoubles / 2 : 0;
        const double *band = space.band(w) + half + 2 * lane;
        int to = 0;
        auto issue = [&](int b) {
            const double *p = band + (int64_t)(b < blocks ? b : blocks - 1) * kBandDoubles;
#pragma unroll
            for (int i = 0; i < LOADS; ++i)
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(p + 128 * i),
                                                 (__attribute__((address_space(3))) void *)(&ring[to][half + 128 * i]), 16, 0, 0);
            to = to + 1 == RING ? 0 : to + 1;
        };
        // (LOADS per block are in flight, always, so that their number says which block has arrived)
        auto arrived = [&] {
            static_assert(LOADS * FLIGHT == 32, "the number of loads in flight");
            asm volatile("s_waitcnt vmcnt(32)" ::: "memory");
        };
        for (int b = 0; b < FLIGHT + 3; ++b) issue(b);
        arrived();
        narrow_barrier();
        if (!finite()) return false;
        for (int b = 0; b < blocks; ++b) {
            narrow_barrier();
            issue(b + FLIGHT + 3);
            arrived();
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        narrow_barrier();
    } else {
        if (wave == 4) {
            const double sum = !fresh && lane < d ? r_sum[lane] : 0.0;
            const uint64_t *flags = reinterpret_cast<const uint64_t *>(space.strange<DP>(w));  // of eight blocks each
            static_assert(kBandStride % 8 == 0, "whole words");
            constexpr int HELD = 8;
            uint64_t any = !(__builtin_fabs(sum) < __builtin_inf()) ? 1 : 0;
            for (int at = lane; at < blocks / 8; at += 64 * HELD) {
                uint64_t x[HELD];
#pragma unroll
                for (int q = 0; q < HELD; ++q) x[q] = flags[at + 64 * q < blocks / 8 ? at + 64 * q : at];
#pragma unroll
                for (int q = 0; q < HELD; ++q) any |= x[q];
            }
            const unsigned long long found = __ballot(any != 0);
            if (lane == 0) *strange = found ? 1 : 0;
        }
        narrow_barrier();
        return finite();
    }
    return true;
}

}  // namespace cdgrab
