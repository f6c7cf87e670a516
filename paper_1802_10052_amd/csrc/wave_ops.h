// Lane exchanges of a 64-wide wavefront in registers, and accesses that workgroups of one launch share.
#pragma once
#include <hip/hip_runtime.h>

namespace ed {

// With lanes paired at distance 32 (16): the lower lane of a pair gets the pair's sum of a, the upper
// lane the pair's sum of b. pair_sum(a, a) is the pair's sum on both.
__device__ __forceinline__ double pair_sum32(double a, double b) {
    const unsigned long long ua = __double_as_longlong(a), ub = __double_as_longlong(b);
    const auto lo = __builtin_amdgcn_permlane32_swap(unsigned(ua), unsigned(ub), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(unsigned(ua >> 32), unsigned(ub >> 32), false, false);
    return __hiloint2double(int(hi[0]), int(lo[0])) + __hiloint2double(int(hi[1]), int(lo[1]));
}
__device__ __forceinline__ double pair_sum16(double a, double b) {
    const unsigned long long ua = __double_as_longlong(a), ub = __double_as_longlong(b);
    const auto lo = __builtin_amdgcn_permlane16_swap(unsigned(ua), unsigned(ub), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(unsigned(ua >> 32), unsigned(ub >> 32), false, false);
    return __hiloint2double(int(hi[0]), int(lo[0])) + __hiloint2double(int(hi[1]), int(lo[1]));
}
__device__ __forceinline__ double2 pair_sum32(double2 a, double2 b) {
    return make_double2(pair_sum32(a.x, b.x), pair_sum32(a.y, b.y));
}
__device__ __forceinline__ double2 pair_sum16(double2 a, double2 b) {
    return make_double2(pair_sum16(a.x, b.x), pair_sum16(a.y, b.y));
}

// the value of the lane that the DPP control names; every lane of the wave must be active
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E;            // quad permutations: lane ^ 1, lane ^ 2
constexpr int kDppHalfMirror = 0x141, kDppMirror = 0x140;  // lane ^ 7, lane ^ 15
constexpr int kDppRor8 = 0x128;                            // lane ^ 8
template <int CTRL>
__device__ __forceinline__ double dpp(double a) {
    return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(a), CTRL, 0xf, 0xf, true),
                            __builtin_amdgcn_update_dpp(0, __double2loint(a), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double2 dpp(double2 a) {
    return make_double2(dpp<CTRL>(a.x), dpp<CTRL>(a.y));
}

// Accesses at agent scope, for what one workgroup writes and another reads within a launch: they pass by
// the caches that are not shared by the whole chip, so no cache has to be written back or invalidated.
__device__ __forceinline__ int ld_shared(const int* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_shared(int* p, int v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double ld_shared(const double* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_shared(double* p, double v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double2 ld_shared(const double2* p) {
    const double* q = reinterpret_cast<const double*>(p);
    return make_double2(ld_shared(q), ld_shared(q + 1));
}
__device__ __forceinline__ void st_shared(double2* p, double2 v) {
    double* q = reinterpret_cast<double*>(p);
    st_shared(q, v.x);
    st_shared(q + 1, v.y);
}
// every access of this wave so far has been performed (and none below is moved above it)
__device__ __forceinline__ void drain() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory"); }

}  // namespace ed
