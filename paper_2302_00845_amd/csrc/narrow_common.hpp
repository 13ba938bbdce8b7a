// Rows of at most 64 elements: what the kernels of narrow_kernels.hpp and band_kernels.hpp share.
#pragma once
#include "chain_kernels.hpp"

namespace cdgrab {

constexpr int kNarrowMaxD = 64;
constexpr int kNarrowThreads = 512;
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

// A barrier of the workgroup: what this wavefront has written to LDS is there, and what it has read from LDS is
// in registers, before it passes; rows on their way from memory stay on their way.
__device__ __forceinline__ void narrow_barrier() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

}  // namespace cdgrab
