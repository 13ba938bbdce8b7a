// Many optimisation steps of the m simulated workers at a time ("CD-GraB Workers" lines 4-7
// with the server's average, "CD-GraB Parameter Server" lines 5-7), softmax-regression model.
//
// Step after step, the logits of an example depend on the weights only through its features' inner
// products with the examples visited since: with W <- W - lr v, v <- momentum v + gbar and
// gbar = (1/m) sum_i x_i delta_i^T,
//     W_{j+1}^T x = W_j^T x - lr v_{j+1}^T x,
//     v_{j+1}^T x = momentum v_j^T x + (1/m) sum_{i in step j} <x_i, x> delta_i.
// So the steps of a block (up to 256 examples) need the logits of its examples at the block's first
// weights and the Gram matrix of their features -- both wide launches, the Gram matrix off the chain
// (gram_tiles) -- and one workgroup then runs the steps on those few thousand numbers
// (train_solve).  With all deltas known, one wide launch writes every gradient row and applies the
// block's steps to the weights in the same arithmetic as a launch per step (train_update_block).
// Three launches per block instead of two per step: 16 workers x 16 steps of 784 -> 10 take
// 41 us (logits 8, solve 21, update 12) instead of 185.
// Products of features are exact in double and summed in double; the deltas and everything
// the weights are made of are fp32 as before.
#pragma once
#include "narrow_kernels.hpp"

namespace cdgrab {

constexpr int kSolveExamples = 256;  // examples of a block: four 64 x 64 tiles' worth of columns
constexpr int kSolveClasses = 16;    // classes at most: one column tile of an MFMA
constexpr int kSolveThreads = 1024;
constexpr int kSolveWorkers = 64;    // workers at most: four steps per block

// Row of every example in visiting order: order[j * m + i] = i * n + perm[i][j].
__global__ __launch_bounds__(256) void example_order(const int32_t *__restrict__ perm, int64_t m, int64_t n,
                                                     int64_t *__restrict__ order)
{
    const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (q >= m * n) return;
    const int64_t i = q / n, j = q - i * n;
    order[j * m + i] = i * n + (perm ? (int64_t)perm[q] : j);
}

// base[e][0][c] = W^T [x_e; 1], base[e][1][c] = v^T [x_e; 1] for the examples of a block, in double.
// One workgroup per example; wavefront (which, quarter) takes a quarter of the classes, its lanes share
// the features.  Bound by latency: two batches of loads, one reduction.  (By MFMA, sixteen examples
// a workgroup: 12 us, the products of so few workgroups being the longer part; this way 8 us.)
__global__ __launch_bounds__(512) void train_base_logits(const float *__restrict__ X,
                                                         const int64_t *__restrict__ order,
                                                         const float *__restrict__ W,
                                                         const float *__restrict__ velocity, int in_dim, int classes,
                                                         double *__restrict__ base)
{
    constexpr int K = 8;  // features per lane and batch
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int which = wave >> 2, quarter = wave & 3;
    const int per = (classes + 3) / 4, c0 = quarter * per;
    const float *x = X + order[blockIdx.x] * in_dim;
    const float *p = which ? velocity : W;
    double *out = base + ((int64_t)blockIdx.x * 2 + which) * kSolveClasses;
    if (!p) {
        if (lane < per && c0 + lane < classes) out[c0 + lane] = 0.0;
        return;
    }
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int f0 = lane; f0 < in_dim; f0 += 64 * K) {
        float xv[K], pv[K][4];
#pragma unroll
        for (int u = 0; u < K; ++u) {
            const int f = f0 + 64 * u < in_dim ? f0 + 64 * u : in_dim - 1;
            xv[u] = x[f];
#pragma unroll
            for (int q = 0; q < 4; ++q) pv[u][q] = p[f * classes + (c0 + q < classes ? c0 + q : classes - 1)];
        }
#pragma unroll
        for (int u = 0; u < K; ++u) {
            const double a = f0 + 64 * u < in_dim ? (double)xv[u] : 0.0;
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[q] = __builtin_fma(a, (double)pv[u][q], acc[q]);
        }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        acc[q] = sum_across_32(sum_across_16(dpp_add<0x140>(sum_of_eight(acc[q]))));  // (row_mirror: the other eight)
        if (lane == 0 && q < per && c0 + q < classes)
            out[c0 + q] = acc[q] + (double)p[in_dim * classes + c0 + q];  // bias input 1
    }
}

// Sum / maximum over the sixteen lanes of a row.
template <typename F>
__device__ __forceinline__ float row_reduce(float x, F &&f) {
    auto from = [&](auto ctrl) {
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value, 0xf, 0xf, true));
    };
    x = f(x, from(std::integral_constant<int, 0xB1>{}));   // quad_perm 1 0 3 2
    x = f(x, from(std::integral_constant<int, 0x4E>{}));   // quad_perm 2 3 0 1
    x = f(x, from(std::integral_constant<int, 0x141>{}));  // row_half_mirror
    return f(x, from(std::integral_constant<int, 0x140>{}));  // row_mirror
}

// The steps of a block, in order, by one workgroup.  Wavefront w keeps the logits (under W and
// under v) of sixteen examples, 16 w .., in registers, as a 16 x 16 MFMA result
// (row = example, column = class), and drops out when they have all been visited.  (Sixteen wavefronts
// of one result each: 1.2 us per step; four of four, whose chains of MFMAs nothing overlaps: 2.0.)  A step: its m examples' logits go through LDS to one lane per (example,
// class), which takes the softmax in fp32; then every later example's logits are updated by one
// rank-m product, features' Gram entries (two steps ahead in registers) x deltas.  MQ: MFMA
// steps of four workers per round; more than 4 MQ workers take several rounds per step.  `steps` is even.
template <int MQ>
__global__ __launch_bounds__(kSolveThreads) void train_solve(const double *__restrict__ gram,
                                                             const double *__restrict__ base,
                                                             const int32_t *__restrict__ y,
                                                             const int64_t *__restrict__ order,
                                                             float *__restrict__ delta_out,
                                                             float *__restrict__ loss_out, int m, int steps, int64_t n,
                                                             int64_t j0, int classes, double lr, double momentum)
{
    __shared__ float logit[kSolveWorkers][kSolveClasses];
    __shared__ double delta[kSolveWorkers + 16][kSolveClasses];  // rows beyond m, columns beyond the classes: zero
    __shared__ int32_t label[kSolveExamples];
    __shared__ float sum_exp[kSolveExamples], margin[kSolveExamples];
    __shared__ float delta_all[kSolveExamples][kSolveClasses];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, kslot = lane >> 4;
    constexpr int WAVES = kSolveThreads / 64, GROUPS = kSolveExamples / 16 / WAVES;
    const int examples = m * steps;
    const int rounds = (m + 4 * MQ - 1) / (4 * MQ);
    const double inv_m = 1.0 / (double)m;
    double lw[GROUPS][4], lv[GROUPS][4];
    int at_step[GROUPS][4];
#pragma unroll
    for (int t = 0; t < GROUPS; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int e = 16 * (WAVES * t + wave) + 4 * v + kslot, ec = e < examples ? e : examples - 1;
            lw[t][v] = base[(ec * 2) * kSolveClasses + col];
            lv[t][v] = base[(ec * 2 + 1) * kSolveClasses + col];
            at_step[t][v] = e < examples ? e / m : steps;  // (a missing example is updated and never read)
        }
    // Gram entries <x_i, x_e> of round f: i = the round's workers, e = this wavefront's examples
    // Does group t still hold an example of a step after s?
    auto later = [&](int t, int s) { return 16 * (WAVES * t + wave) + 15 >= (s + 1) * m && 16 * (WAVES * t + wave) < examples; };
    // (No branch around these loads and no store in the loop: each would end in waiting for all of
    // them at every step.  What a group without later examples reads is not used.)
    const int last_tile = (examples - 1) >> 6;
    const double *column[GROUPS];
#pragma unroll
    for (int t = 0; t < GROUPS; ++t) {
        const int tj = (WAVES * t + wave) >> 2;
        column[t] = gram + (int64_t)tile_index(0, tj < last_tile ? tj : last_tile) * kTileEntries;
    }
    struct Entries { double k[GROUPS][MQ]; };
    auto load = [&](Entries &x, int f) {
        // (tile (ti, t) row j of tile: row 64 ti + j of column tile t, since a column's tiles are stored in order)
        const int s = rounds == 1 ? f : f / rounds, first = s * m + (f - s * rounds) * 4 * MQ;
#pragma unroll
        for (int q = 0; q < MQ; ++q) {
            const int i = first + 4 * q + kslot, most = (s + 1) * m - 1;
            const uint32_t at = (uint32_t)((i < most ? i : most) * kTilePairs + 16 * (wave & 3) + col);
#pragma unroll
            for (int t = 0; t < GROUPS; ++t) x.k[t][q] = column[t][at];
        }
    };
    Entries even, odd;
    const int total = steps * rounds;
    load(even, 0);
    load(odd, 1);
    if (tid < examples) label[tid] = y[order[tid]];
    for (int q = tid; q < (kSolveWorkers + 16) * kSolveClasses; q += kSolveThreads) delta[q / kSolveClasses][q % kSolveClasses] = 0.0;
    double4_t acc[GROUPS];
    int s = 0, round = 0;
    auto advance = [&](Entries &x, int f) {
        if (round == 0) {  // the step's deltas
            const int first = s * m;
#pragma unroll
            for (int t = 0; t < GROUPS; ++t) {
                const int e0 = 16 * (WAVES * t + wave);
                if (e0 + 15 < first || e0 >= first + m) continue;  // (uniform)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (at_step[t][v] == s)
                        logit[16 * (WAVES * t + wave) + 4 * v + kslot - first][col] = (float)lw[t][v];
            }
            __syncthreads();
            for (int i = tid >> 4; i < m; i += kSolveThreads / 16) {
                const float z = col < classes ? logit[i][col] : -INFINITY;
                const float mx = row_reduce(z, [](float a, float b) { return fmaxf(a, b); });
                const float ex = col < classes ? expf(z - mx) : 0.f;
                const float Z = row_reduce(ex, [](float a, float b) { return a + b; });
                if (col < classes) {
                    const bool mine = col == label[first + i];
                    const float dl = ex / Z - (mine ? 1.0f : 0.0f);
                    delta[i][col] = (double)dl;
                    delta_all[first + i][col] = dl;
                    if (mine) {
                        margin[first + i] = z - mx;
                        sum_exp[first + i] = Z;
                    }
                }
            }
            __syncthreads();
#pragma unroll
            for (int t = 0; t < GROUPS; ++t) acc[t] = (double4_t){0.0, 0.0, 0.0, 0.0};
        }
        double b[MQ];
#pragma unroll
        for (int q = 0; q < MQ; ++q) b[q] = delta[round * 4 * MQ + 4 * q + kslot][col];
#pragma unroll
        for (int t = 0; t < GROUPS; ++t)
            if (later(t, s)) {
#pragma unroll
                for (int q = 0; q < MQ; ++q)  // (1: the bias input)
                    acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(x.k[t][q] + 1.0, b[q], acc[t], 0, 0, 0);
            }
        load(x, f + 2 < total ? f + 2 : total - 1);
        if (++round == rounds) {
#pragma unroll
            for (int t = 0; t < GROUPS; ++t)
                if (later(t, s)) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        lv[t][v] = __builtin_fma(momentum, lv[t][v], acc[t][v] * inv_m);
                        lw[t][v] = __builtin_fma(-lr, lv[t][v], lw[t][v]);
                    }
                }
            round = 0;
            ++s;
            // (the next step's logits are written to LDS after everyone has read this step's:
            // the barrier after the deltas)
        }
    };
    __syncthreads();
    for (int f = 0; f < total; f += 2) {
        advance(even, f);
        advance(odd, f + 1);
    }
    __syncthreads();
    for (int q = tid; q < examples * classes; q += kSolveThreads) delta_out[q] = delta_all[q / classes][q % classes];
    // (a label that names no class leaves its loss as it is)
    if (loss_out && tid < examples && (uint32_t)label[tid] < (uint32_t)classes)
        loss_out[(int64_t)(tid % m) * n + j0 + tid / m] = -(margin[tid] - logf(sum_exp[tid]));
}

// Gradient rows and weights of a block of steps whose deltas are known.  A workgroup owns 64
// parameters p = (r, c), its sixteen wavefronts share the steps: each forms a step's m gradients (all
// loads of sixteen workers in flight), writes them into the staging chunk (pair-major: pair (k, i)
// of the chunk holds rows [2q], [2q+1] with q = (k - k_first) m + i) and optionally into
// grads_out[m][n][d], and leaves their sum in LDS; one wavefront then applies the steps in order
// (v <- momentum v + gbar; w <- w - lr v).
__global__ __launch_bounds__(1024) void train_update_block(const float *__restrict__ X,
                                                           const int64_t *__restrict__ order,
                                                           const float *__restrict__ delta, float *__restrict__ W,
                                                           float *__restrict__ velocity, float *__restrict__ staging,
                                                           float *__restrict__ grads_out, int m, int steps, int64_t n,
                                                           int64_t j0, int64_t k_first, int in_dim, int classes,
                                                           float lr, float momentum)
{
    __shared__ float sums[kSolveExamples][64];
    const int64_t d = (int64_t)(in_dim + 1) * classes;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // (neighbours share the lines at their edges: each XCD takes a contiguous run of workgroups)
    const int blocks = (int)((d + 63) / 64), per_xcd = (blocks + 7) >> 3;
    const int block = blocks >= 16 ? (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3) : (int)blockIdx.x;
    if (block >= blocks) return;
    const int64_t p = (int64_t)block * 64 + lane;
    const int64_t pc = p < d ? p : d - 1;
    const int r = (int)(pc / classes), c = (int)(pc - (int64_t)r * classes);
    const int rx = r < in_dim ? r : in_dim - 1;  // the bias row reads a valid feature and drops it
    constexpr int U = 16;
    for (int s = wave; s < steps; s += 16) {
        const int64_t id = order[s * m + (lane < m ? lane : m - 1)];  // the step's examples, one per lane (m <= 64)
        auto example = [&](int i) {  // (i uniform)
            const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)id, i);
            const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)id >> 32), i);
            return (int64_t)(((uint64_t)hi << 32) | lo);
        };
        const int64_t j = j0 + s, k = j >> 1;
        const int which = (int)(j & 1);
        float sum = 0.f;
        for (int i0 = 0; i0 < m; i0 += U) {
            float g[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = i0 + u < m ? i0 + u : m - 1, q = s * m + i;
                const float xv = X[example(i) * in_dim + rx];
                g[u] = (r < in_dim ? xv : 1.0f) * delta[q * classes + c];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = i0 + u;
                if (i < m) {
                    if (p < d) {
                        staging[(2 * ((k - k_first) * m + i) + which) * d + p] = g[u];
                        if (grads_out) grads_out[((int64_t)i * n + j) * d + p] = g[u];
                    }
                    sum += g[u];
                }
            }
        }
        sums[s][lane] = sum;
    }
    __syncthreads();
    if (wave != 0 || p >= d) return;
    float w = W[p], v = velocity ? velocity[p] : 0.f;
    for (int s = 0; s < steps; ++s) {
        const float gbar = sums[s][lane] / (float)m;
        v = velocity ? momentum * v + gbar : gbar;
        w = w - lr * v;
    }
    W[p] = w;
    if (velocity) velocity[p] = v;
}

}  // namespace cdgrab
