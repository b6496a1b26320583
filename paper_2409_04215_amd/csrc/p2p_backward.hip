// Position gradients of the pair sums, gfx950.
//
// For the pairing Phi = sum_i sum_j w_i . G(x_i - y_j) s_j over the pair set of
// the forward sum, with d = x - y, r = |d|:
//   Stokes:  dPhi_ij/dd = [-(w.s) d + (w.d) s + (s.d) w - 3 (w.d)(s.d) d / r^2] / (8 pi mu r^3)
//   Laplace: dPhi_ij/dd = -w s d / (4 pi r^3)
// (derived from the kernels of Sections 2.1-2.2; the paper has no gradients).
//
// One kernel computes, per lane point p carrying vector a_p,
//   g_p = sum_q dPhi/dd (d = p - q; w = a_p, s = b_q)
// over the lane's pair set.  Run on the forward orientation (lanes =
// collocation points with w, sources = proxies with s) it gives dPhi/dx_i.
// Because dPhi_ij/dd is odd in d and symmetric in (w, s), the same kernel run
// on the transposed orientation (lanes = proxies with s, sources = collocation
// points with w) gives dPhi/dy_j = -sum_i dPhi_ij/dd directly.
//
// The walk is the one of the forward sum: an item of 64 lane points, the four
// waves of the workgroup each taking a contiguous quarter of every source body
// (wave-uniform loop, scalar loads, SGPR operands), the partial gradients added
// in wave order through LDS, same-body handling and mixed FP32-pair /
// FP64-accumulation precision exactly as there.
// The transposed orientation gives dPhi/ds_j too (the velocity sum over the pairs
// it has in hand): the three gradients of 60 Stokes bodies of 400 sources and 800
// targets 1735 -> 1532 us, where a sum of its own walked the pairs a third time
// (now 1405 us).
#include "pair_math.h"

namespace mfs {

namespace {

constexpr int BLOCK = 256;
constexpr int WAVES = BLOCK / 64;
// Sources per FP32 run.  Each adds two terms to the sums, so the runs are shorter than the velocity
// sums' 64: at 16 the three gradients of 60 bodies err by 1.43e-7, 2.33e-7 and 2.38e-7 (1405 us), at
// 32 by 1.80e-7, 2.60e-7 and 2.66e-7 (1377 us); with a term's sum added once per source and runs of
// 32 it was 1.48e-7, 2.42e-7 and 2.48e-7 (1519 us).
constexpr int FLUSH = 16;

struct GradArgs {
    const P2PItem *items;
    const double *centre;
    const int32_t *lane_body;
    const int32_t *src_ptr;
    const double *lane_vec;  // lane vectors, indexed like the forward output (out0 + dim*(i - t0))
    double *out;             // [n_lane][3] (split slices of stride out_stride)
    double *sum_out;         // SUM: the lanes' pair sums, like lane_vec (slices of the same stride)
    int64_t out_stride;
    double alpha;
    int skip_same;
    int accumulate;
};

__device__ __forceinline__ float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }

// U Stokes sources: with c = 1/r^3, the pair's gradient is
//   c (-(w.s) - 3 (w.d)(s.d) / r^2) d + c (w.d) s + c (s.d) w.
// The coefficients of w are added up in pw and multiplied once per run, so a pair takes 30
// operations and a 1/sqrt.  SUM: v += s / r + c (s.d) d, the velocity sum over the same pairs, for
// six operations more (a sum of its own takes 17 and the 1/sqrt).
template <bool MIXED, bool SUM, int U, class R>
__device__ __forceinline__ void stokes_grad(const R (&xr)[3], const R (&w)[3], const typename Records<MIXED>::S *src,
                                            R (&p)[3], R &pw, R (&v)[3]) {
    R d[U][3], ri[U], s[U][3];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        R y[3];
        source(src[u], y, s[u]);
#pragma unroll
        for (int c = 0; c < 3; ++c) d[u][c] = xr[c] - y[c];
        ri[u] = d[u][0] * d[u][0] + d[u][1] * d[u][1] + d[u][2] * d[u][2];
    }
    rsqrt_all(ri);
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const R ri2 = ri[u] * ri[u], c3 = ri[u] * ri2;
        const R ws = w[0] * s[u][0] + w[1] * s[u][1] + w[2] * s[u][2];
        const R wd = w[0] * d[u][0] + w[1] * d[u][1] + w[2] * d[u][2];
        const R sd = s[u][0] * d[u][0] + s[u][1] * d[u][1] + s[u][2] * d[u][2];
        const R k = c3 * (R(-3) * (wd * sd * ri2) - ws), a = c3 * wd;
        const R e = c3 * sd;
        pw += e;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            // two FMAs each: added up as written, the two terms would cost a multiplication more
            p[c] = fma_(k, d[u][c], fma_(a, s[u][c], p[c]));
            if (SUM) v[c] = fma_(e, d[u][c], fma_(ri[u], s[u][c], v[c]));
        }
    }
}

// U Laplace sources: p += q d / r^3 (the factor -w follows once per run); SUM: v += q / r
template <bool MIXED, bool SUM, int U, class R>
__device__ __forceinline__ void laplace_grad(const R (&xr)[3], const typename Records<MIXED>::L *src, R (&p)[3], R &v) {
    R d[U][3], ri[U], q[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        R y[3];
        source(src[u], y, q[u]);
#pragma unroll
        for (int c = 0; c < 3; ++c) d[u][c] = xr[c] - y[c];
        ri[u] = d[u][0] * d[u][0] + d[u][1] * d[u][1] + d[u][2] * d[u][2];
    }
    rsqrt_all(ri);
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const R c = q[u] * ri[u] * (ri[u] * ri[u]);
        if (SUM) v += q[u] * ri[u];
#pragma unroll
        for (int e = 0; e < 3; ++e) p[e] += c * d[u][e];
    }
}

template <bool MIXED, bool SUM>
__global__ __launch_bounds__(BLOCK) void p2p_grad_kernel(GradArgs a, const void *__restrict__ lane_off_v,
                                                         const void *__restrict__ srcS_v,
                                                         const void *__restrict__ srcL_v) {
    typedef typename Records<MIXED>::R R;
    constexpr int U = MIXED ? 4 : 2;  // sources per step
    const auto *src_s = reinterpret_cast<const typename Records<MIXED>::S *>(srcS_v);
    const auto *src_l = reinterpret_cast<const typename Records<MIXED>::L *>(srcL_v);
    constexpr int NV = SUM ? 6 : 3;  // gradient, sum
    __shared__ double lds[(WAVES - 1) * NV * 64];
    const P2PItem it = a.items[blockIdx.x];
    const bool stokes = it.kind == MFS_STOKES;
    const int dim = stokes ? 3 : 1;
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i = it.t0 + lane;
    const bool valid = i < it.t1;
    const int ii = valid ? i : it.t0;
    const int body = a.lane_body[ii];
    double ct[3] = {a.centre[3 * body], a.centre[3 * body + 1], a.centre[3 * body + 2]};
    R xt[3];
    if (MIXED) {
        const float4 o = reinterpret_cast<const float4 *>(lane_off_v)[ii];
        xt[0] = o.x; xt[1] = o.y; xt[2] = o.z;
    } else {
        const double4 o = reinterpret_cast<const double4 *>(lane_off_v)[ii];
        xt[0] = (R)o.x; xt[1] = (R)o.y; xt[2] = (R)o.z;
    }
    const int64_t vo = it.out0 + (int64_t)dim * (ii - it.t0);
    R w[3];
    w[0] = (R)a.lane_vec[vo];
    w[1] = stokes ? (R)a.lane_vec[vo + 1] : R(0);
    w[2] = stokes ? (R)a.lane_vec[vo + 2] : R(0);
    double acc[NV] = {};

    for (int b = it.b0; b < it.b1; ++b) {
        const bool use = valid && !(a.skip_same && body == b);
        if (!__any(use)) continue;
        R xr[3];
        for (int c = 0; c < 3; ++c) xr[c] = xt[c] + (R)(ct[c] - a.centre[3 * b + c]);
        // this wave's contiguous quarter of the body's sources
        const int s0 = a.src_ptr[b], s1 = a.src_ptr[b + 1];
        const int qn = (s1 - s0 + WAVES - 1) / WAVES;
        const int j0 = min(s0 + wv * qn, s1), j1 = min(j0 + qn, s1);
        for (int jb = j0; jb < j1; jb += FLUSH) {
            const int je = min(jb + FLUSH, j1);
            R p[3] = {R(0), R(0), R(0)}, v[3] = {R(0), R(0), R(0)}, pw = R(0);
            int j = jb;
            if (stokes) {
                for (; j + U <= je; j += U) stokes_grad<MIXED, SUM, U>(xr, w, src_s + j, p, pw, v);
                for (; j < je; ++j) stokes_grad<MIXED, SUM, 1>(xr, w, src_s + j, p, pw, v);
                for (int c = 0; c < 3; ++c) p[c] += pw * w[c];
            } else {
                for (; j + U <= je; j += U) laplace_grad<MIXED, SUM, U>(xr, src_l + j, p, v[0]);
                for (; j < je; ++j) laplace_grad<MIXED, SUM, 1>(xr, src_l + j, p, v[0]);
                for (int c = 0; c < 3; ++c) p[c] *= -w[0];
            }
            for (int c = 0; c < 3; ++c) acc[c] += use ? (double)p[c] : 0.0;
            if constexpr (SUM)
                for (int c = 0; c < 3; ++c) acc[3 + c] += use ? (double)v[c] : 0.0;
        }
    }
    // waves 1..3 hand their partial gradients to wave 0, which adds them in wave order
    if (wv > 0)
        for (int c = 0; c < NV; ++c) lds[((wv - 1) * NV + c) * 64 + lane] = acc[c];
    __syncthreads();
    if (wv > 0) return;
    for (int w = 1; w < WAVES; ++w)
        for (int c = 0; c < NV; ++c) acc[c] += lds[((w - 1) * NV + c) * 64 + lane];
    if (!valid) return;
    double *out = a.out + (int64_t)it.split * a.out_stride + 3 * (int64_t)i;
    for (int c = 0; c < 3; ++c) {
        double v = a.alpha * it.scale * acc[c];
        if (a.accumulate) v += out[c];
        out[c] = v;
    }
    if constexpr (SUM) {
        double *sum = a.sum_out + (int64_t)it.split * a.out_stride + vo;
        for (int c = 0; c < dim; ++c) {
            double v = a.alpha * it.scale * acc[3 + c];
            if (a.accumulate) v += sum[c];
            sum[c] = v;
        }
    }
}

__global__ void reduce3_kernel(int64_t n, const double *__restrict__ partial, int64_t stride, int n_split,
                               double *__restrict__ out, int accumulate) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    double s = strided_sum(partial + v, stride, n_split);
    if (accumulate) s += out[v];
    out[v] = s;
}

}  // namespace

// lane vectors `lane_vec` indexed in the items' output layout; gradient out [n_lane][3].  sum_out
// (or null): the pair sums at the lanes as well, n_sum values like lane_vec.  L.partial holds
// n_split slices of 3 n_lane + n_sum values.
int launch_p2p_grad(const P2PPlan &pp, const P2PLaunch &L, const double *lane_vec, int64_t n_lane, hipStream_t s,
                    double *sum_out, int64_t n_sum) {
    if (pp.items.empty()) return MFS_OK;
    if (pp.tpl != 1) return fail(MFS_EINVAL, "gradient pair sums take items of one target per lane");
    GradArgs a;
    a.items = pp.d_items.as<P2PItem>();
    a.centre = L.centre;
    a.lane_body = L.trg_body;
    a.src_ptr = L.src_ptr;
    a.lane_vec = lane_vec;
    a.alpha = L.alpha;
    a.skip_same = L.skip_same ? 1 : 0;
    const bool direct = pp.n_split == 1;
    a.out = direct ? L.out : L.partial;
    a.sum_out = direct ? sum_out : L.partial + 3 * n_lane;
    a.out_stride = 3 * n_lane + (sum_out ? n_sum : 0);
    a.accumulate = direct ? (L.accumulate ? 1 : 0) : 0;
    const dim3 grid((unsigned)pp.items.size());
    const bool mixed = L.prec == MFS_MIXED;
    if (sum_out) {
        if (mixed) p2p_grad_kernel<true, true><<<grid, BLOCK, 0, s>>>(a, L.trg_off, L.srcS, L.srcL);
        else p2p_grad_kernel<false, true><<<grid, BLOCK, 0, s>>>(a, L.trg_off, L.srcS, L.srcL);
    } else {
        if (mixed) p2p_grad_kernel<true, false><<<grid, BLOCK, 0, s>>>(a, L.trg_off, L.srcS, L.srcL);
        else p2p_grad_kernel<false, false><<<grid, BLOCK, 0, s>>>(a, L.trg_off, L.srcS, L.srcL);
    }
    MFS_HIP_TRY(hipGetLastError());
    auto reduce = [&](const double *partial, int64_t n, double *out) {
        reduce3_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(n, partial, a.out_stride, pp.n_split, out,
                                                                 L.accumulate ? 1 : 0);
    };
    if (!direct) {
        reduce(L.partial, 3 * n_lane, L.out);
        if (sum_out) reduce(L.partial + 3 * n_lane, n_sum, sum_out);
        MFS_HIP_TRY(hipGetLastError());
    }
    return MFS_OK;
}

}  // namespace mfs
