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
// BLOCK us instead of 185.
// Products of features are exact in double and summed in double; the deltas and everything
// the weights are made of are fp32 as before.
#pragma once
#include "chain_kernels.hpp"

namespace cdgrab {

constexpr int kSolveExamples = 256;  // examples of a block: four 64 x 64 tiles' worth of columns
constexpr int kSolveClasses = 16;    // classes at most: one column tile of an MFMA
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
// One workgroup per sixteen examples; its sixteen wavefronts share the features (MFMA: examples x
// features x classes), the shares are added in order through LDS.
__global__ __launch_bounds__(1024) void train_base_logits(const float *__restrict__ X,
                                                          const int64_t *__restrict__ order, int examples,
                                                          const float *__restrict__ W,
                                                          const float *__restrict__ velocity, int in_dim, int classes,
                                                          double *__restrict__ base)
{
    __shared__ double red[16][2][256];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 15, kslot = lane >> 4;
    const int e = blockIdx.x * 16 + col;
    const float *x = X + order[e < examples ? e : examples - 1] * in_dim;
    const int cc = col < classes ? col : 0;
    const float *vel = velocity ? velocity : W;
    const int steps = (in_dim + 3) / 4;
    const int q0 = wave * steps / 16, q1 = (wave + 1) * steps / 16;
    double4_t aw = (double4_t){0.0, 0.0, 0.0, 0.0}, av = aw;
    for (int q = q0; q < q1; q += 8) {
        float xv[8], wv[8], vv[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int f = 4 * (q + u < q1 ? q + u : q1 - 1) + kslot, fc = f < in_dim ? f : in_dim - 1;
            xv[u] = x[fc];
            wv[u] = W[fc * classes + cc];
            vv[u] = vel[fc * classes + cc];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const bool in = q + u < q1 && 4 * (q + u) + kslot < in_dim;
            const double a = in ? (double)xv[u] : 0.0;
            aw = __builtin_amdgcn_mfma_f64_16x16x4f64(a, (double)wv[u], aw, 0, 0, 0);
            av = __builtin_amdgcn_mfma_f64_16x16x4f64(a, (double)vv[u], av, 0, 0, 0);
        }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        red[wave][0][v * 64 + lane] = aw[v];
        red[wave][1][v * 64 + lane] = av[v];
    }
    __syncthreads();
    if (threadIdx.x < 512) {
        const int which = threadIdx.x >> 8, idx = threadIdx.x & 255;
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < 16; ++w) s += red[w][which][idx];
        int i, j;
        mfma_f64_16x16_coord(idx & 63, idx >> 6, i, j);
        const int ex = blockIdx.x * 16 + i;
        if (ex < examples && j < classes) {
            const float *p = which ? velocity : W;
            s += p ? (double)p[in_dim * classes + j] : 0.0;  // bias input 1
            base[(ex * 2 + which) * kSolveClasses + j] = p ? s : 0.0;
        }
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
// under v) of the examples 64 w .. 64 w + 63 in registers, as four 16 x 16 MFMA results (row =
// example, column = class).  A step: its m examples' logits go through LDS to one lane per (example,
// class), which takes the softmax in fp32; then every later example's logits are updated by one
// rank-m product, features' Gram entries (two steps ahead in registers) x deltas.  MQ: MFMA
// steps of four workers per round; more than 4 MQ workers take several rounds per step.
template <int MQ>
__global__ __launch_bounds__(256) void train_solve(const double *__restrict__ gram, const double *__restrict__ base,
                                                   const int32_t *__restrict__ y, const int64_t *__restrict__ order,
                                                   float *__restrict__ delta_out, float *__restrict__ loss_out,
                                                   int m, int steps, int64_t n, int64_t j0, int classes, double lr,
                                                   double momentum)
{
    __shared__ float logit[kSolveWorkers][kSolveClasses];
    __shared__ double delta[kSolveWorkers + 16][kSolveClasses];  // rows beyond m, columns beyond the classes: zero
    __shared__ int32_t label[kSolveExamples];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, kslot = lane >> 4;
    const int examples = m * steps;
    const int rounds = (m + 4 * MQ - 1) / (4 * MQ);
    const double inv_m = 1.0 / (double)m;
    double lw[4][4], lv[4][4];
    int at_step[4][4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int e = 64 * wave + 16 * t + 4 * v + kslot, ec = e < examples ? e : examples - 1;
            lw[t][v] = base[(ec * 2) * kSolveClasses + col];
            lv[t][v] = base[(ec * 2 + 1) * kSolveClasses + col];
            at_step[t][v] = e < examples ? e / m : steps;  // (a missing example is updated and never read)
        }
    // Gram entries <x_i, x_e> of round f: i = the round's workers, e = this wavefront's examples
    // (what a wavefront without examples, or with earlier ones only, reads is not used)
    const int last_tile = (examples - 1) >> 6, tile_col = wave < last_tile ? wave : last_tile;
    struct Entries { double k[4][MQ]; };
    auto load = [&](Entries &x, int f) {
        const int s = f / rounds, first = s * m + (f - s * rounds) * 4 * MQ;
#pragma unroll
        for (int q = 0; q < MQ; ++q) {
            const int i = first + 4 * q + kslot, ic = i < examples ? i : examples - 1;
            const double *g = gram + (int64_t)tile_index(ic >> 6, tile_col) * kTileEntries + (ic & 63) * kTilePairs + col;
#pragma unroll
            for (int t = 0; t < 4; ++t) x.k[t][q] = g[16 * t];
        }
    };
    Entries even, odd;
    const int total = steps * rounds;
    load(even, 0);
    load(odd, total > 1 ? 1 : 0);
    if (tid < examples) label[tid] = y[order[tid]];
    for (int q = tid; q < (kSolveWorkers + 16) * kSolveClasses; q += 256) delta[q / kSolveClasses][q % kSolveClasses] = 0.0;
    double4_t acc[4];
    int s = 0, round = 0;
    auto advance = [&](Entries &x, int f) {
        if (round == 0) {  // the step's deltas
            const int first = s * m;
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (at_step[t][v] == s)
                        logit[64 * wave + 16 * t + 4 * v + kslot - first][col] = (float)lw[t][v];
            __syncthreads();
            for (int i = tid >> 4; i < m; i += 16) {
                const int lab = label[first + i];
                const float z = col < classes ? logit[i][col] : -INFINITY;
                const float mx = row_reduce(z, [](float a, float b) { return fmaxf(a, b); });
                const float ex = col < classes ? expf(z - mx) : 0.f;
                const float Z = row_reduce(ex, [](float a, float b) { return a + b; });
                if (col < classes) {
                    const float dl = ex / Z - (col == lab ? 1.0f : 0.0f);
                    delta[i][col] = (double)dl;
                    delta_out[(first + i) * classes + col] = dl;
                    if (col == lab && loss_out) loss_out[(int64_t)i * n + j0 + s] = -(z - mx - logf(Z));
                }
            }
            __syncthreads();
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[t] = (double4_t){0.0, 0.0, 0.0, 0.0};
        }
        const bool later = 64 * wave + 63 >= (s + 1) * m;  // (uniform: examples of later steps here)
        if (later) {
#pragma unroll
            for (int q = 0; q < MQ; ++q) {
                const double b = delta[round * 4 * MQ + 4 * q + kslot][col];
#pragma unroll
                for (int t = 0; t < 4; ++t)  // (1: the bias input)
                    acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(x.k[t][q] + 1.0, b, acc[t], 0, 0, 0);
            }
        }
        if (f + 2 < total) load(x, f + 2);
        if (++round == rounds) {
            if (later) {
#pragma unroll
                for (int t = 0; t < 4; ++t)
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
        if (f + 1 < total) advance(odd, f + 1);
    }
}

// Gradient rows and weights of a block of steps whose deltas are known.  A workgroup owns 64
// parameters p = (r, c), its sixteen wavefronts share the steps: each forms a step's m gradients (all
// loads of eight workers in flight), writes them into the staging chunk (pair-major: pair (k, i)
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
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t p = (int64_t)blockIdx.x * 64 + lane;
    const int64_t pc = p < d ? p : d - 1;
    const int r = (int)(pc / classes), c = (int)(pc - (int64_t)r * classes);
    const int rx = r < in_dim ? r : in_dim - 1;  // the bias row reads a valid feature and drops it
    constexpr int U = 8;
    for (int s = wave; s < steps; s += 16) {
        const int64_t j = j0 + s, k = j >> 1;
        const int which = (int)(j & 1);
        float sum = 0.f;
        for (int i0 = 0; i0 < m; i0 += U) {
            float g[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int q = s * m + (i0 + u < m ? i0 + u : m - 1);
                const float xv = X[order[q] * in_dim + rx];
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
