// Rows of at most 64 elements: a whole walk inside one workgroup.
//
// With so few elements a block of 64 pairs is a few KB, the running sum is a few hundred bytes, and what
// a chain of launches spends between its steps is many times the work in them.  So one workgroup
// (per independent walk) keeps the running sum in LDS and walks all pairs, 64 at a time: two
// wavefronts take turns walking a block, ten helpers meanwhile bring in the rows (two blocks
// of loads in flight), form the differences in double and compute the next block's Gram matrix
// by MFMA; then all helpers apply the decided block and take the next block's dots.
// Bound by the serial chain of a block: the walk (20 ns per pair: four dependent instructions, 15 ns, and
// a barrier on the way) and, between two walks, apply + dots through LDS.  At 16 elements a block takes 2.2 us
// of an epoch (in-kernel clocks: walk 1.3, apply 0.4, running sum 0.1, dots 0.2), 5.2 us in the steps of
// chain_kernels.hpp; at 33 .. 64 elements 3.8 us (the next block's Gram matrix, in MFMA time, outlasts the walk).  Longer rows would need
// more LDS than a CU has for three blocks of differences and a Gram matrix.
#pragma once
#include "chain_kernels.hpp"

namespace cdgrab {

constexpr int kNarrowMaxD = 64;
constexpr int kNarrowHelpers = 512;                   // threads that load, apply and take dots
constexpr int kNarrowThreads = 128 + 640;             // two walkers, ten helper wavefronts (a Gram tile each)
constexpr int64_t kNarrowMaxPairs = (int64_t)1 << 30; // per launch and walk

// Sums over lanes that differ in bit 0, 1 or 2 (DPP), or in bit 4 or 5 (row swaps), left in every
// lane: a few cycles each, where a shuffle through LDS costs about a hundred.
template <int CTRL>
__device__ __forceinline__ double dpp_add(double x) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xf, 0xf, true);
    return x + __hiloint2double(hi, lo);
}
__device__ __forceinline__ double sum_of_eight(double x) {
    x = dpp_add<0xB1>(x);   // quad_perm 1 0 3 2
    x = dpp_add<0x4E>(x);   // quad_perm 2 3 0 1
    return dpp_add<0x141>(x);  // row_half_mirror: the other four of eight
}
__device__ __forceinline__ double sum_across_16(double x) {
    const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(x), __double2loint(x), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(x), __double2hiint(x), false, false);
    return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
__device__ __forceinline__ double sum_across_32(double x) {
    const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(x), __double2loint(x), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(x), __double2hiint(x), false, false);
    return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}

// DP: padded row length (16, 32 or 64).  `pairs` consecutive pairs of every walk, the first at
// rows; the running sum is read from (fresh: starts at zero) and written back to r_sum, and to r32 / r64
// where they are not null.
template <int DP, int VW, bool RANDOM>
__global__ __launch_bounds__(kNarrowThreads) void narrow_walk(StepRows rows, int pairs, int64_t half_n, int fresh,
                                                              double *__restrict__ r_sum, float *__restrict__ r32,
                                                              double *__restrict__ r64,
                                                              int8_t *__restrict__ signs_out,
                                                              double *__restrict__ dots_out,
                                                              const float *__restrict__ uniforms, WalkStrides ws)
{
    constexpr int DS = DP + 2;            // doubles per difference row in LDS (sixteen rows: distinct banks)
    constexpr int GS = kTilePairs + 2;
    constexpr int QUADS = DP / 4;
    constexpr int ITEMS = kTilePairs * QUADS;                                  // (pair, four elements) of a block
    constexpr int PER = (ITEMS + kNarrowHelpers - 1) / kNarrowHelpers;         // per helper thread
    __shared__ __attribute__((aligned(16))) double diff[3][kTilePairs * DS];   // blocks b, b + 1, b + 2
    __shared__ double G[kTilePairs * GS];                                      // of block b + 1; zero on and below the diagonal
    __shared__ double part[8][DP];
    __shared__ double r[DP];
    __shared__ double dots[kTilePairs];
    __shared__ unsigned long long votes;
    const int64_t w = blockIdx.x;
    rows.base += w * ws.rows;
    r_sum += w * ws.r;
    signs_out += w * ws.out;
    if (dots_out) dots_out += w * ws.out;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t d = rows.d;
    const int blocks = (pairs + kTilePairs - 1) / kTilePairs;

    // Barriers: three before the loop, then five per block: M (the next block's Gram matrix is there),
    // E1 (signs), E2 (partial sums of the apply), E3 (running sum), E4 (next block's dots).
    if (wave < 2) {
        __syncthreads();
        __syncthreads();
        if (wave == 1) __syncthreads();
        int passed = 0;
        auto pass_to = [&](int barriers) {
            for (; passed < barriers; ++passed) __syncthreads();
        };
        for (int b = wave; b < blocks; b += 2) {
            // columns, draws and output slot of this block, whose Gram matrix is in G from M of the
            // block before on
            if (b > 0) pass_to(5 * (b - 1) + 1);
            double col[64];
#pragma unroll
            for (int j = 0; j < 64; ++j) col[j] = G[j * GS + lane];
            const int kk = b * kTilePairs + lane;
            const uint32_t q = (uint32_t)rows.i0 + (uint32_t)kk;
            const uint32_t dq = q / (uint32_t)rows.m;
            const int64_t slot = (int64_t)(q - dq * (uint32_t)rows.m) * half_n + (rows.k0 + dq);
            // randomized rule (PairBalance's RandomizedBalance subroutine, Sec. 3.2): with
            // c = z1 - z2 = -d, the first row gets +1 with probability p = (1 - <r,c>)/2 =
            // (1 + t)/2, so the exported sign (of the second row) is -1 when u < p.
            const float my_u = (RANDOM && kk < pairs) ? uniforms[slot] : 0.f;
            auto rule = [&](double tv) { return RANDOM ? !((double)my_u < 0.5 * (1.0 + tv)) : (tv <= 0.0); };
            if (b > 0) pass_to(5 * b);
            else __syncthreads();
            double t = dots[lane];
            auto step = [&](auto jj) {
                constexpr int j = decltype(jj)::value;
                const unsigned long long vote = __ballot(rule(t));
                t = __builtin_fma(sign_of_bit<j & 31>(j < 32 ? (uint32_t)vote : (uint32_t)(vote >> 32)), col[j], t);
            };
            static_for(std::make_integer_sequence<int, 48>{}, step);
            __syncthreads();  // M
            static_for(std::make_integer_sequence<int, 16>{},
                       [&](auto jj) { step(std::integral_constant<int, 48 + decltype(jj)::value>{}); });
            const bool plus = rule(t);
            const unsigned long long all = __ballot(plus);
            if (lane == 0) votes = all;
            __syncthreads();  // E1
            if (kk < pairs) {
                signs_out[slot] = plus ? 1 : -1;
                if (dots_out) dots_out[slot] = t;
            }
            passed = 5 * b + 2;
        }
        pass_to(5 * blocks);
        return;
    }

    const int h = tid - 128, hw = wave - 2;
    const bool works = h < kNarrowHelpers;  // (uniform per wavefront: the last two only compute Gram tiles)
    struct Rows { float4_t a[PER], b[PER]; };  // as loaded: what does not belong is cut off in store(), two blocks later
    // Every thread keeps its (pair of the block, four elements); from block to block its rows move on by
    // 64 pairs, i.e. by a fixed distance plus another one whenever the worker index wraps around.
    const bool dense = rows.layout == kDense;
    const int di = dense ? kTilePairs % rows.m : 0, wrap_at = dense ? rows.m : 1;
    const int64_t row_step = dense ? di * rows.n + 2 * (kTilePairs / rows.m)
                                   : (rows.layout == kStaged ? 2 * kTilePairs : kTilePairs);
    const int64_t step = row_step * d, wrap = dense ? (2 - rows.m * rows.n) * d : 0;
    const float *at[PER];
    int worker[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const PairCursor c(rows, ((h + u * kNarrowHelpers) % ITEMS) / QUADS);
        const float *b;
        c.rows(rows, at[u], b);
        worker[u] = (int)c.i;
    }
    auto load = [&](Rows &x, int blk) {  // called for blocks 0, 1, 2, .. in turn
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int item = h + u * kNarrowHelpers;
            const bool have = blk * kTilePairs + (item % ITEMS) / QUADS < pairs;  // (else the first pair again)
            const float *a = have ? at[u] : rows.base + (dense ? rows.i0 * rows.n + 2 * rows.k0 : 0) * d;
            const float *b = rows.layout == kCentred ? rows.centre : a + d;
            const int e = (item % QUADS) * 4, dn = (int)d;
            if constexpr (VW == kTiny) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    x.a[u][q] = a[e + q < dn ? e + q : 0];
                    x.b[u][q] = b[e + q < dn ? e + q : 0];
                }
            } else {  // a group that reaches beyond the row reads the row's last four elements
                const int base = e <= dn - 4 ? e : dn - 4;
                x.a[u] = load_four<true>(a + base);
                x.b[u] = load_four<true>(b + base);
            }
            worker[u] += di;
            at[u] += step;
            if (worker[u] >= wrap_at) {
                worker[u] -= wrap_at;
                at[u] += wrap;
            }
        }
    };
    auto store = [&](const Rows &x, int blk) {  // (a pair that does not exist becomes zero)
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int item = h + u * kNarrowHelpers;
            if (item < ITEMS) {
                const int j = item / QUADS, e = (item % QUADS) * 4, dn = (int)d;
                const int base = VW == kTiny || e <= dn - 4 ? e : dn - 4;
                const bool have = blk * kTilePairs + j < pairs;
                double v[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) v[q] = (double)x.b[u][q] - (double)x.a[u][q];
                // element e + q sits at position e - base + q of what was loaded (in binary steps)
                const int sh = e - base;
                const bool s1 = sh & 1, s2 = sh & 2;
                const double y0 = s1 ? v[1] : v[0], y1 = s1 ? v[2] : v[1], y2 = s1 ? v[3] : v[2], y3 = v[3];
                const double z0 = s2 ? y2 : y0, z1 = s2 ? y3 : y1;
                double2 *p = reinterpret_cast<double2 *>(&diff[blk % 3][j * DS + e]);
                p[0] = make_double2(have && e < dn ? z0 : 0.0, have && e + 1 < dn ? z1 : 0.0);
                p[1] = make_double2(have && e + 2 < dn ? y2 : 0.0, have && e + 3 < dn ? y3 : 0.0);
            }
        }
    };
    // upper 16 x 16 tiles of the Gram matrix of block blk, one per wavefront
    int tj = 0;
    while (tile_index(0, tj + 1) <= hw) ++tj;
    const int ti = hw - tile_index(0, tj);
    auto gram = [&](int blk) {
        const int mrow = lane & 15, kslot = lane >> 4;
        const double *A = diff[blk % 3] + (16 * ti + mrow) * DS + kslot, *B = diff[blk % 3] + (16 * tj + mrow) * DS + kslot;
        double a[DP / 4], b[DP / 4];
#pragma unroll
        for (int q = 0; q < DP / 4; ++q) {
            a[q] = A[4 * q];
            b[q] = B[4 * q];
        }
        double4_t acc = (double4_t){0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int q = 0; q < DP / 4; ++q) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q], b[q], acc, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            int i, j;
            mfma_f64_16x16_coord(lane, v, i, j);
            if (ti != tj || i < j) G[(16 * ti + i) * GS + 16 * tj + j] = acc[v];
        }
    };
    auto take_dots = [&](int blk) {  // eight threads per pair
        const int k = h >> 3, sub = h & 7;
        const double *D = diff[blk % 3] + k * DS;
        double p = 0.0;
#pragma unroll
        for (int q = 0; q < DP / 8; ++q) p = __builtin_fma(r[sub + 8 * q], D[sub + 8 * q], p);
        p = sum_of_eight(p);
        if (sub == 0) dots[k] = p;
    };
    Rows even, odd;
    auto block = [&](int b, Rows &x) {
        if (b + 1 < blocks) gram(b + 1);
        if (works && b + 2 < blocks) store(x, b + 2);
        __syncthreads();  // M
        if (works && b + 4 < blocks) load(x, b + 4);
        __syncthreads();  // E1
        if (works) {
            // a wavefront applies eight pairs: DP elements x 64 / DP pair groups
            constexpr int LG = 64 / DP;
            const unsigned long long v = votes;
            const int e = lane % DP, g = lane / DP;
            const double *D = diff[b % 3] + e;
            double acc = 0.0;
#pragma unroll
            for (int q = 0; q < 8 / LG; ++q) {
                const int j = hw * 8 + g * (8 / LG) + q;
                acc = __builtin_fma((v >> j) & 1ull ? 1.0 : -1.0, D[j * DS], acc);
            }
            if (DP <= 16) acc = sum_across_16(acc);
            if (DP <= 32) acc = sum_across_32(acc);
            if (lane < DP) part[hw][lane] = acc;
        }
        __syncthreads();  // E2
        if (h < DP) {
            double s = 0.0;
#pragma unroll
            for (int q = 0; q < 8; ++q) s += part[q][h];
            r[h] += s;
        }
        __syncthreads();  // E3
        if (works && b + 1 < blocks) take_dots(b + 1);
        __syncthreads();  // E4
    };
    if (works) {
        load(even, 0);
        load(odd, 1);
    }
    for (int q = h; q < kTilePairs * GS; q += kNarrowThreads - 128) G[q] = 0.0;
    if (h < DP) r[h] = h < d && !fresh ? r_sum[h] : 0.0;
    if (works) {
        store(even, 0);
        store(odd, 1);
        load(even, 2);
        load(odd, 3);
    }
    __syncthreads();
    gram(0);
    if (works) take_dots(0);
    __syncthreads();
    __syncthreads();  // (the walker of block 0 has its columns)
    for (int b = 0; b < blocks; b += 2) {
        block(b, even);
        if (b + 1 < blocks) block(b + 1, odd);
    }
    if (h < d) {
        r_sum[h] = r[h];
        if (r32) r32[h] = (float)r[h];
        if (r64) r64[h] = r[h];
    }
}

}  // namespace cdgrab
