// Source records and 1/sqrt by precision, shared by the gradient and field pair sums (gfx950).
#pragma once

#include "device_math.h"
#include "mfs_internal.h"

namespace mfs {

template <bool MIXED>
struct Records {  // arithmetic and source records of a precision
    typedef float R;
    typedef SrcS32 S;
    typedef SrcL32 L;
};
template <>
struct Records<false> {
    typedef double R;
    typedef SrcS64 S;
    typedef SrcL64 L;
};

__device__ __forceinline__ void source(const SrcS32 &s, float (&y)[3], float (&f)[3]) {
    y[0] = s.pos.x; y[1] = s.pos.y; y[2] = s.pos.z;
    f[0] = s.str.x; f[1] = s.str.y; f[2] = s.str.z;
}
__device__ __forceinline__ void source(const SrcS64 &s, double (&y)[3], double (&f)[3]) {
    for (int c = 0; c < 3; ++c) {
        y[c] = s.pos[c];
        f[c] = s.str[c];
    }
}
__device__ __forceinline__ void source(const SrcL32 &s, float (&y)[3], float &q) {
    y[0] = s.x; y[1] = s.y; y[2] = s.z;
    q = s.w;
}
__device__ __forceinline__ void source(const SrcL64 &s, double (&y)[3], double &q) {
    for (int c = 0; c < 3; ++c) y[c] = s.v[c];
    q = s.v[3];
}

// 1/sqrt in place; the FP32 ones as one run (see rsq_cluster_begin)
template <int U>
__device__ __forceinline__ void rsqrt_all(float (&r)[U]) {
    rsq_cluster_begin();
#pragma unroll
    for (int u = 0; u < U; ++u) r[u] = __builtin_amdgcn_rsqf(r[u]);
    rsq_cluster_end();
}
template <int U>
__device__ __forceinline__ void rsqrt_all(double (&r)[U]) {
#pragma unroll
    for (int u = 0; u < U; ++u) r[u] = rsqrt_f64(r[u]);
}

}  // namespace mfs
