// Device arithmetic shared by the pair-sum kernels (gfx950).
#pragma once

#include <hip/hip_runtime.h>

namespace mfs {

// 1/sqrt(r2) in FP64.  The hardware estimate y = v_rsq_f64(r2) has a relative
// error of about 2^-24 (measured over 2^20 arguments in [1e-8, 1e8]).  With
// e = 1 - r2 y^2, the exact value is y (1 - e)^(-1/2) = y (1 + e/2 + 3e^2/8 +
// O(e^3)), so one step y + y e (1/2 + 3e/8) leaves a truncation error near
// (5/16) e^3, about 2^-70: below FP64 rounding.  The same arguments give at
// most 0.99 ulp against a long-double reference, as two Newton steps do, in
// five FP64 operations instead of eight.
__device__ __forceinline__ double rsqrt_f64(double r2) {
    const double y = __builtin_amdgcn_rsq(r2);
    const double e = __builtin_fma(-r2 * y, y, 1.0);
    const double c = __builtin_fma(0.375, e, 0.5);
    return __builtin_fma(y * e, c, y);
}

// Brackets around a run of v_rsq_f32.  Two waves of a SIMD issue cheap FP32 operations side by
// side (1.0 ns each per wave and SIMD at full occupancy), but not beside a wave that is in a
// v_rsq_f32 (3.4 ns): with single ones spread over the loop the cheap operations fall to 1.65 ns.
// So the pair loops collect the 1/sqrt of several pairs, and the wave takes priority for them:
// one v_rsq_f32 per 16 multiplies takes 17.4 ns so, 22 to 26 ns with the clusters alone, 22 to
// 30 ns scattered (18.6 ns if nothing overlapped).
__device__ __forceinline__ void rsq_cluster_begin() {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(3);
}
__device__ __forceinline__ void rsq_cluster_end() {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(0);
}

// The next U of p's values, m of them there (1 <= m <= U; the last one is read again), added to s in order
template <int U, class T>
__device__ __forceinline__ void add_group(T &s, const T *__restrict__ p, int64_t stride, int m) {
    T v[U];
#pragma unroll
    for (int q = 0; q < U; ++q) v[q] = p[min(q, m - 1) * stride];
#pragma unroll
    for (int q = 0; q < U; ++q)
        if (q < m) s += v[q];
}

// p[0] + p[stride] + ... (n values) in order, their loads issued up to eight at a time: a loop of n
// dependent loads and adds took 14 us of a launch for 14 split slices, 5 us so.  The last group is of the
// size that holds what is left: with eight loads whatever was left, the projection of one
// FP64 body took 4.7 us (a plain loop 4.1, so 4.0).
template <class T>
__device__ __forceinline__ T strided_sum(const T *__restrict__ p, int64_t stride, int n) {
    T s = T(0);
    for (; n > 4; n -= 8, p += 8 * stride) add_group<8>(s, p, stride, min(n, 8));
    if (n > 2) add_group<4>(s, p, stride, n);
    else if (n > 0) add_group<2>(s, p, stride, n);
    return s;
}

}  // namespace mfs
