// All-pairs fundamental-solution sums (the MFS representation), gfx950.
//
// Laplace (Section 2.1):  u_i = sum_j s_j / (4 pi r_ij)
// Stokes  (Section 2.2, eq. (stokeslet)):
//          u_i = sum_j (s_j + (d.s_j) d / r^2) / (8 pi mu r),  d = x_i - y_j
//
// Design (MI355X):
//  * One work item = a block of 64*TPL targets of one system x a range of
//    source bodies of the same system, run by one workgroup of four waves.
//    Every wave holds all the item's targets (TPL per lane, register blocking)
//    and takes a contiguous quarter of each source body; the four FP64
//    partial sums meet in LDS once per item and are added in wave order, so
//    results do not depend on timing.  Splitting the sources rather than the
//    targets keeps items small in targets, so a launch reaches many items
//    with few source splits (each split costs one FP64 slice of the output).
//  * Items are launched largest-first, so the hardware dispatcher hands the
//    long items out before the short ones.
//  * Stokes sources are read with wave-uniform addresses: every lane of a wave
//    walks the same source list, so the compiler turns the reads into scalar
//    loads (s_load) and the VALU instructions take the source coordinates and
//    strengths as SGPR operands.  Laplace sources (16 B, one v_rsq_f32 per 8
//    VALU instructions) are staged per run of 64 in the wave's own LDS slots
//    and read back by broadcast: 15% faster there, 1% slower for Stokes.
//  * Mixed precision: the coordinates are split into a per-body FP64 centre
//    and a small FP32 offset; per (lane, source body) the FP64 centre
//    difference is rounded to FP32 once, so the FP32 rounding of d scales
//    with |d| plus the body size.  Per pair: FP32 arithmetic with the hardware
//    v_rsq_f32; per run of at most FLUSH sources the FP32 partial is added
//    to an FP64 accumulator.
//  * Laplace sources far from all the item's targets go through the matrix cores
//    (far_body): |x - y|^2 = |x|^2 - 2 x.y + |y|^2 is one v_mfma_f32_16x16x32_bf16
//    per 16 targets x 16 sources, from exact three-way splits of FP32 coordinates,
//    which leaves a pair v_rsq_f32 and one FMA of its 8 VALU instructions.
//  * FP64 variant: the same walk in FP64, 1/sqrt from v_rsq_f64 refined by
//    one third-order step (rsqrt_f64 in device_math.h).
//  * Same-body pairs: a source body equal to every active lane's own body is
//    skipped wave-uniformly; a body shared by only some lanes is evaluated
//    and its partial discarded per lane (select, not multiply), so no masking
//    sits inside the pair loop.
#include <type_traits>

#include "device_math.h"
#include "mfs_internal.h"

namespace mfs {

namespace {

constexpr int BLOCK = 256;
constexpr int WAVES = BLOCK / 64;
constexpr int FLUSH = 64;
constexpr int STAGED_ITEMS = 1024;

// Adds the FP64 accumulators of waves 1..WAVES-1 into wave 0's, in wave order.
// lds holds (WAVES-1) * NV * 64 doubles.  Every thread of the workgroup must
// call it; returns true in wave 0, which then owns the sums.
template <int NV>
__device__ __forceinline__ bool reduce_waves(double (&v)[NV], double *lds) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (wv > 0)
#pragma unroll
        for (int q = 0; q < NV; ++q) lds[((wv - 1) * NV + q) * 64 + lane] = v[q];
    __syncthreads();
    if (wv > 0) return false;
    for (int w = 1; w < WAVES; ++w)
#pragma unroll
        for (int q = 0; q < NV; ++q) v[q] += lds[((w - 1) * NV + q) * 64 + lane];
    return true;
}

struct Src4 {
    SrcS32 s[4];
};

// U Stokes sources against the lane's TPL targets, FP32 (eq. (stokeslet) without 1/(8 pi mu)).
template <int TPL, int U>
__device__ __forceinline__ void stokes_pairs(const float (&xr)[TPL][3], const SrcS32 *s, float (&p)[TPL][3]) {
    float d[U][TPL][3], ri[U][TPL];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int t = 0; t < TPL; ++t) {
            const float4 y = s[u].pos;
            float *e = d[u][t];
            e[0] = xr[t][0] - y.x;
            e[1] = xr[t][1] - y.y;
            e[2] = xr[t][2] - y.z;
            ri[u][t] = __builtin_fmaf(e[2], e[2], __builtin_fmaf(e[1], e[1], e[0] * e[0]));
        }
    rsq_cluster_begin();
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int t = 0; t < TPL; ++t) ri[u][t] = __builtin_amdgcn_rsqf(ri[u][t]);
    rsq_cluster_end();
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int t = 0; t < TPL; ++t) {
            const float4 f = s[u].str;
            const float *e = d[u][t], r = ri[u][t];
            const float df = __builtin_fmaf(e[2], f.z, __builtin_fmaf(e[1], f.y, e[0] * f.x));
            const float sc = df * (r * r);
            p[t][0] = __builtin_fmaf(r, __builtin_fmaf(sc, e[0], f.x), p[t][0]);
            p[t][1] = __builtin_fmaf(r, __builtin_fmaf(sc, e[1], f.y), p[t][1]);
            p[t][2] = __builtin_fmaf(r, __builtin_fmaf(sc, e[2], f.z), p[t][2]);
        }
}

// U Laplace sources (LDS) against the lane's TPL targets, FP32 (1/r without 1/(4 pi)).
template <int TPL, int U>
__device__ __forceinline__ void laplace_pairs(const float (&xr)[TPL][3], const float4 *s, float (&p)[TPL]) {
    float q[U], ri[U][TPL];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const float4 y = s[u];
        q[u] = y.w;
#pragma unroll
        for (int t = 0; t < TPL; ++t) {
            const float d0 = xr[t][0] - y.x, d1 = xr[t][1] - y.y, d2 = xr[t][2] - y.z;
            ri[u][t] = __builtin_fmaf(d2, d2, __builtin_fmaf(d1, d1, d0 * d0));
        }
    }
    rsq_cluster_begin();
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int t = 0; t < TPL; ++t) ri[u][t] = __builtin_amdgcn_rsqf(ri[u][t]);
    rsq_cluster_end();
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int t = 0; t < TPL; ++t) p[t] = __builtin_fmaf(q[u], ri[u][t], p[t]);
}

// Orders a wave's LDS stores before its later reads of them (its accesses complete in order).
__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// This wave's contiguous quarter [j0, j1) of the source range [b0, b1).
__device__ __forceinline__ void wave_range(int b0, int b1, int wv, int &j0, int &j1) {
    const int q = (b1 - b0 + WAVES - 1) / WAVES;
    j0 = min(b0 + wv * q, b1);
    j1 = min(j0 + q, b1);
}

typedef float float4v __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t uint4v __attribute__((ext_vector_type(4)));

struct KernelArgs {
    const P2PItem *items;
    const double *centre;      // [n_body][3]
    const int32_t *trg_body;   // [n_trg]
    const int32_t *src_ptr;    // [n_body+1]
    const int32_t *sys_active; // [n_sys] or null
    double *out;               // partial slices or final output
    const double *addend;      // added once (may be null); only when n_split == 1
    int64_t out_stride;        // elements per split slice
    double alpha;              // scale applied to the pair sum (includes 1/(4pi) or 1/(8 pi mu))
    int skip_same;
    int accumulate;
    int *queue;                // persistent mode: work-queue counter (reset to 0 before the launch), else null
    int n_items;
    const uint4v *far_tiles;      // Laplace far tiles (pack_far_tile), 64 per tile
    const int32_t *far_tile_ptr;  // [n_body] first tile of a body
    const double *far_centre;     // [n_body][3] the point a body's tiles are relative to
    const float *far_rho;         // [n_body] largest distance of a source from it
};

// ---------------------------------------------------------------------------
// Laplace sources far from a block of targets
//
// The 32 k slots of the bf16 MFMA hold, for a target x and a source y relative to the mean of
// the body's sources, group by group of eight (lane l holds group l/16):
//   0..2:  coordinate c of x and of -2 y as three bf16 pieces a + m + l, which is FP32 exactly;
//          eight of the nine products of pieces (l l is below 2^-32 of x.y)
//   3:     |x|^2 in four pieces against ones, ones against |y|^2 in four pieces
// with |x|^2 and |y|^2 from the FP64 coordinates.  Products of pieces are exact in FP32 and the
// matrix core adds the slots with a rounding of 0.28 ulp of the largest (measured, rms), so for
// |x| >= 2 |y| r^2 errs by less than the subtracted coordinates' does (0.33e-7 |x|^2, where
// rounding x alone leaves 0.7e-7 |x| r).  Bodies nearer than that, bodies with a target of their
// own in the block and extreme scales take the VALU path.
// Rate: a pair is v_rsq_f32 and one FMA on the VALU (5.2 ns per 64 pairs and SIMD in a bare
// loop, 13.3 with the six operations of r^2), the MFMA (1.7 ns) runs beside them.
// 250 bodies, 389 sources and 777 targets each: 3285 -> 2430 us (7.7e12 pairs/s).
// ---------------------------------------------------------------------------
__device__ __forceinline__ float bf16_head(float x) { return __uint_as_float(__float_as_uint(x) & 0xffff0000u); }
__device__ __forceinline__ uint32_t bf16_pair(float lo, float hi) {  // both exact in bf16
    return __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u);
}
__device__ __forceinline__ void split3(float x, float &a, float &m, float &l) {
    a = bf16_head(x);
    const float r = x - a;
    m = bf16_head(r);
    l = r - m;
}
__device__ __forceinline__ void split4(double x, float (&p)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        p[i] = bf16_head((float)x);
        x -= p[i];
    }
}
constexpr uint32_t BF16_ONES = 0x3f803f80u;

// Column l%16 of tile k of nt is source nt (l%16) + k, so that a lane's sums run over
// neighbouring sources: oscillating strengths cancel early there as in the VALU runs (sources dealt
// out 16 apart left up to twice their error).
__device__ __forceinline__ int far_source(int k, int nt, int lane) { return nt * (lane & 15) + k; }
// A lane's 16 bytes of a tile for its source's offset y from the body's centre.
__device__ __forceinline__ uint4v pack_far_tile(const double (&y)[3], int lane) {
    const int g = lane >> 4;
    if (g < 3) {
        float a, m, l;
        split3(-2.0f * (float)y[g], a, m, l);
        return uint4v{bf16_pair(a, m), bf16_pair(l, a), bf16_pair(m, l), bf16_pair(a, m)};
    }
    float p[4];
    split4(y[0] * y[0] + y[1] * y[1] + y[2] * y[2], p);
    return uint4v{BF16_ONES, BF16_ONES, bf16_pair(p[0], p[1]), bf16_pair(p[2], p[3])};
}

// Sums of one wave's far bodies, value i = 4 t + r: target 16 t + 4 (l/16) + r against the sources
// that lane l has had.
struct FarSums {
    double sum[16];
};

template <int CTRL>
__device__ __forceinline__ double dpp_move(double x) {  // x of another lane of the row of 16
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}

// The values summed over the row's 16 lanes, every exchange halving what a lane carries, which leaves
// lane l value i = l%16.
__device__ __forceinline__ double far_row_sum(double (&v)[16]) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int h = 8; h >= 1; h >>= 1) {
        const bool up = (lane & h) != 0;
#pragma unroll
        for (int i = 0; i < h; ++i) {
            const double lo = v[i], hi = v[i + h];
            const double send = up ? +lo : +hi, keep = up ? +hi : +lo;  // values: a choice of elements is indexing
            double got;
            if (h == 8) got = dpp_move<0x128>(send);       // row_ror:8
            else if (h == 4) got = dpp_move<0x1B>(dpp_move<0x141>(send));  // row_half_mirror, quad_perm [3,2,1,0]
            else if (h == 2) got = dpp_move<0x4E>(send);   // quad_perm [2,3,0,1]
            else got = dpp_move<0xB1>(send);               // quad_perm [1,0,3,2]
            v[i] = keep + got;
        }
    }
    return v[0];
}
__device__ __forceinline__ int far_target(int lane) {  // value i = 4 t + r of row g: target 16 t + 4 g + r
    return 16 * ((lane & 15) >> 2) + 4 * (lane >> 4) + (lane & 3);
}

// All sources of one far body against the wave's 64 targets; x: this lane's target relative to
// the body's centre, frag: 4 KB and str: 1024 floats of the wave's own.  The next tile is fetched
// while this one is summed (two ahead 3% slower, four 17%: registers).
// A lane adds its FP32 sum to FP64 every FAR_RUN tiles and at the end of a body: four neighbouring
// sources, where a run of the walk above has up to 64, because the bf16 r^2 errs from pair to pair.
// Error against 64 bits over the walk without far tiles, of sums over pseudo-inverse strengths of
// smooth data, aspects 2 and 3, 100 to 800 sources (24 suspensions each): 0.72 to 0.97 with runs of 4,
// 0.85 to 1.10 with 8, 0.86 to 1.13 with 16, and 0.86 to 1.19 with an FP32 sum carried over 64 tiles.
// 250 bodies of 389 sources: 2387, 2324, 2283 and 2298 us.
constexpr int FAR_RUN = 4;
__device__ __forceinline__ void far_body(const uint4v *__restrict__ tiles, const SrcL32 *__restrict__ src, int n,
                                         const double (&x)[3], uint4v *frag, float *str, FarSums &fs) {
    const int lane = threadIdx.x & 63, g = lane >> 4, c16 = lane & 15;
    const int nt = (n + 15) / 16;  // at most 64
    uint4v B = tiles[(unsigned)lane];
    for (int j = lane; j < 16 * nt; j += 64) str[j] = j < n ? src[j].w : 0.f;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        float a, m, l;
        split3((float)x[c], a, m, l);
        frag[64 * c + lane] = uint4v{bf16_pair(a, a), bf16_pair(a, m), bf16_pair(m, m), bf16_pair(l, l)};
    }
    float p[4];
    split4(x[0] * x[0] + x[1] * x[1] + x[2] * x[2], p);
    frag[192 + lane] = uint4v{bf16_pair(p[0], p[1]), bf16_pair(p[2], p[3]), BF16_ONES, BF16_ONES};
    wave_lds_order();
    bf16x8 A[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) A[t] = __builtin_bit_cast(bf16x8, frag[64 * g + 16 * t + c16]);
    __builtin_amdgcn_wave_barrier();  // the next body's stores follow these reads
    auto tile = [&](int k, auto add) {  // add(i, strength, 1 / r)
        const bf16x8 Bk = __builtin_bit_cast(bf16x8, B);
        const float q = str[far_source(k, nt, lane)];
        B = (tiles + 64 * (int64_t)min(k + 1, nt - 1))[(unsigned)lane];  // uniform base, 32-bit lane offset
        const float4v zero = {0.f, 0.f, 0.f, 0.f};
        float4v r2[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) r2[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[t], Bk, zero, 0, 0, 0);
        rsq_cluster_begin();
#pragma unroll
        for (int i = 0; i < 16; ++i) r2[i / 4][i % 4] = __builtin_amdgcn_rsqf(r2[i / 4][i % 4]);
        rsq_cluster_end();
#pragma unroll
        for (int i = 0; i < 16; ++i) add(i, q, r2[i / 4][i % 4]);
    };
    for (int kr = 0; kr < nt; kr += FAR_RUN) {
        float part[16];
        tile(kr, [&](int i, float q, float ri) { part[i] = q * ri; });
        for (int k = kr + 1; k < min(kr + FAR_RUN, nt); ++k)
            tile(k, [&](int i, float q, float ri) { part[i] = __builtin_fmaf(q, ri, part[i]); });
#pragma unroll
        for (int i = 0; i < 16; ++i) fs.sum[i] += (double)part[i];
    }
}

// The wave's far sums, lane l: target l
__device__ __forceinline__ double far_total(FarSums &fs, uint4v *frag) {
    const int lane = threadIdx.x & 63;
    double *tot = reinterpret_cast<double *>(frag);
    tot[far_target(lane)] = far_row_sum(fs.sum);
    wave_lds_order();
    return tot[lane];
}

// ---------------------------------------------------------------------------
// Mixed precision, Stokes / Laplace (one kernel; item.kind is wave-uniform)
// ---------------------------------------------------------------------------
// STAGED: Stokes sources through LDS instead of scalar loads.  A launch with few waves per SIMD waits
// for every scalar load (300 ns per four sources), one with many hides it and is faster without the
// LDS reads: up to STAGED_ITEMS items, four waves per SIMD (6 bodies of 400 x 800, 450 items, in a
// matvec of 48.4 us: 44.9; 3 of 1000 x 150 38.2: 28.6; beyond, 16 bodies of 400 x 800 72.4: 75.7).
template <int TPL, bool STAGED>
__device__ __forceinline__ void mixed_item(const KernelArgs &a, const P2PItem it, const float4 *__restrict__ trg_off,
                                           const SrcS32 *__restrict__ srcS, const SrcL32 *__restrict__ srcL,
                                           double *lds, float4 *stage) {
    // an inactive system still writes its epilogue (pair sum 0), so outputs stay finite
    const bool active = !a.sys_active || a.sys_active[it.sys];
    const bool stokes = it.kind == MFS_STOKES;
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    int idx[TPL];
    bool valid[TPL];
    int body[TPL];
    double ct[TPL][3];
    float xt[TPL][3];
    double acc[TPL][3];
#pragma unroll
    for (int t = 0; t < TPL; ++t) {
        idx[t] = it.t0 + lane + t * 64;
        valid[t] = idx[t] < it.t1;
        const int i = valid[t] ? idx[t] : it.t0;
        body[t] = a.trg_body[i];
        const float4 o = trg_off[i];
        xt[t][0] = o.x;
        xt[t][1] = o.y;
        xt[t][2] = o.z;
        ct[t][0] = a.centre[3 * body[t] + 0];
        ct[t][1] = a.centre[3 * body[t] + 1];
        ct[t][2] = a.centre[3 * body[t] + 2];
        acc[t][0] = acc[t][1] = acc[t][2] = 0.0;
    }

    for (int b = it.b0; active && b < it.b1; ++b) {
        bool use[TPL];
        bool any_use = false;
#pragma unroll
        for (int t = 0; t < TPL; ++t) {
            use[t] = valid[t] && !(a.skip_same && body[t] == b);
            any_use |= use[t];
        }
        if (!__any(any_use)) continue;
        const double cs0 = a.centre[3 * b + 0], cs1 = a.centre[3 * b + 1], cs2 = a.centre[3 * b + 2];
        float xr[TPL][3];
#pragma unroll
        for (int t = 0; t < TPL; ++t) {
            xr[t][0] = xt[t][0] + (float)(ct[t][0] - cs0);
            xr[t][1] = xt[t][1] + (float)(ct[t][1] - cs1);
            xr[t][2] = xt[t][2] + (float)(ct[t][2] - cs2);
        }
        int j0, j1;
        wave_range(a.src_ptr[b], a.src_ptr[b + 1], wv, j0, j1);
        if (stokes) {
            for (int jb = j0; jb < j1; jb += FLUSH) {
                const int je = min(jb + FLUSH, j1);
                float p[TPL][3];
#pragma unroll
                for (int t = 0; t < TPL; ++t) p[t][0] = p[t][1] = p[t][2] = 0.f;
                const SrcS32 *__restrict__ ps = srcS + jb;
                const int n = je - jb;
                int k = 0;
                if constexpr (STAGED) {  // one coalesced load per run, as for Laplace below
                    SrcS32 *slot = reinterpret_cast<SrcS32 *>(stage) + 64 * wv;
                    if (lane < n) slot[lane] = ps[lane];
                    wave_lds_order();
                    for (; k + 4 <= n; k += 4) stokes_pairs<TPL, 4>(xr, slot + k, p);
                    for (; k < n; ++k) stokes_pairs<TPL, 1>(xr, slot + k, p);
                    __builtin_amdgcn_wave_barrier();  // the next run's stores follow this run's reads
                } else {
                    // four sources per 128-byte scalar load (s_load_dwordx16 pairs), then the tail
                    for (; k + 4 <= n; k += 4) {
                        const Src4 q = *reinterpret_cast<const Src4 *>(ps + k);
                        stokes_pairs<TPL, 4>(xr, q.s, p);
                    }
                    for (; k < n; ++k) stokes_pairs<TPL, 1>(xr, ps + k, p);
                }
#pragma unroll
                for (int t = 0; t < TPL; ++t) {
                    acc[t][0] += use[t] ? (double)p[t][0] : 0.0;
                    acc[t][1] += use[t] ? (double)p[t][1] : 0.0;
                    acc[t][2] += use[t] ? (double)p[t][2] : 0.0;
                }
            }
        } else {
            // Laplace: each run of up to 64 sources is staged in this wave's own LDS slots by one
            // coalesced load (lane l fetches source jb + l) and read back by every lane
            // (broadcast), so the pair arithmetic takes the sources from VGPRs.  The slots belong
            // to one wave, whose LDS accesses complete in order: no workgroup barrier is needed.
            float4 *slot = stage + 64 * wv;
            for (int jb = j0; jb < j1; jb += FLUSH) {
                const int cnt = min(FLUSH, j1 - jb);
                float p[TPL];
#pragma unroll
                for (int t = 0; t < TPL; ++t) p[t] = 0.f;
                if (lane < cnt) slot[lane] = srcL[jb + lane];
                wave_lds_order();
                int k = 0;
                for (; k + 8 <= cnt; k += 8) laplace_pairs<TPL, 8>(xr, slot + k, p);
                for (; k < cnt; ++k) laplace_pairs<TPL, 1>(xr, slot + k, p);
#pragma unroll
                for (int t = 0; t < TPL; ++t) acc[t][0] += use[t] ? (double)p[t] : 0.0;
                __builtin_amdgcn_wave_barrier();  // the next run's stores follow this run's reads
            }
        }
    }

    double sum[TPL * 3];
#pragma unroll
    for (int t = 0; t < TPL; ++t)
#pragma unroll
        for (int c = 0; c < 3; ++c) sum[3 * t + c] = acc[t][c];
    if (!reduce_waves<TPL * 3>(sum, lds)) return;
    const int dim = stokes ? 3 : 1;
    double *out = a.out + (int64_t)it.split * a.out_stride;
#pragma unroll
    for (int t = 0; t < TPL; ++t) {
        if (!valid[t]) continue;
        const int64_t o = it.out0 + (int64_t)dim * (idx[t] - it.t0);
        for (int c = 0; c < dim; ++c) {
            double v = a.alpha * it.scale * sum[3 * t + c];
            if (a.addend) v += a.addend[o + c];
            if (a.accumulate) v += out[o + c];
            out[o + c] = v;
        }
    }
}

// One Laplace item of a launch with far tiles: 64 targets per wave, so that the four waves read the
// same tiles at about the same time (the tiles of 250 bodies, 6 MB, do not stay in an XCD's L2:
// with one block of targets per item and the far bodies dealt to its waves a 250-body sum took
// 1.08 times as long).  Bodies that are not far are walked eight sources at a time as in mixed_item:
// 40 bodies of 1000 x 1000 points all over the domain, where none is far, take 307 us so, 322 with four
// (316 before there were far tiles).
__device__ __forceinline__ void laplace_far_item(const KernelArgs &a, const P2PItem it,
                                                 const float4 *__restrict__ trg_off, const SrcL32 *__restrict__ srcL,
                                                 float4 *stage, uint4v *frags, float *strs) {
    const bool active = !a.sys_active || a.sys_active[it.sys];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int t0 = it.t0 + 64 * wv;
    if (t0 >= it.t1) return;
    uint4v *frag = frags + 256 * wv;
    float *str = strs + 1024 * wv;
    float4 *slot = stage + 64 * wv;
    const int idx = t0 + lane;
    const bool valid = idx < it.t1;
    const int i = valid ? idx : t0;  // lanes past the last target repeat the wave's first one
    const int body = a.trg_body[i];
    const float4 xt = trg_off[i];
    const double ct0 = a.centre[3 * body], ct1 = a.centre[3 * body + 1], ct2 = a.centre[3 * body + 2];
    double acc = 0.0;
    FarSums fs;
#pragma unroll
    for (int q = 0; q < 16; ++q) fs.sum[q] = 0.0;
    for (int b = it.b0; active && b < it.b1; ++b) {
        const int s0 = a.src_ptr[b], s1 = a.src_ptr[b + 1];
        const bool use = !(a.skip_same && body == b);
        if (s1 == s0 || !__any(use)) continue;
        const double x[3] = {(ct0 - a.far_centre[3 * b]) + (double)xt.x, (ct1 - a.far_centre[3 * b + 1]) + (double)xt.y,
                             (ct2 - a.far_centre[3 * b + 2]) + (double)xt.z};
        const float f0 = (float)x[0], f1 = (float)x[1], f2 = (float)x[2];
        const float n2 = f0 * f0 + f1 * f1 + f2 * f2, rho = a.far_rho[b];
        const bool far = n2 >= 4.0f * rho * rho && n2 > 1e-24f && n2 < 1e24f && use;  // false for NaN
        if (__all(far)) {
            far_body(a.far_tiles + 64 * (int64_t)a.far_tile_ptr[b], srcL + s0, s1 - s0, x, frag, str, fs);
            continue;
        }
        const float xr[1][3] = {{xt.x + (float)(ct0 - a.centre[3 * b]), xt.y + (float)(ct1 - a.centre[3 * b + 1]),
                                 xt.z + (float)(ct2 - a.centre[3 * b + 2])}};
        const int run = min(FLUSH, (s1 - s0 + WAVES - 1) / WAVES);  // no longer than a wave's of mixed_item
        for (int jb = s0; jb < s1; jb += run) {
            const int cnt = min(run, s1 - jb);
            float p[1] = {0.f};
            if (lane < cnt) slot[lane] = srcL[jb + lane];
            wave_lds_order();
            int k = 0;
            for (; k + 8 <= cnt; k += 8) laplace_pairs<1, 8>(xr, slot + k, p);
            for (; k < cnt; ++k) laplace_pairs<1, 1>(xr, slot + k, p);
            acc += use ? (double)p[0] : 0.0;
            __builtin_amdgcn_wave_barrier();  // the next run's stores follow this run's reads
        }
    }
    acc += far_total(fs, frag);
    if (!valid) return;
    double *out = a.out + (int64_t)it.split * a.out_stride;
    const int64_t o = it.out0 + (idx - it.t0);
    double v = a.alpha * it.scale * acc;
    if (a.addend) v += a.addend[o];
    if (a.accumulate) v += out[o];
    out[o] = v;
}

// ---------------------------------------------------------------------------
// Mixed precision, short sums in one launch
//
// A sum of a few bodies is a chain of launches of a few microseconds each (operands, pairs, the sum
// over source splits), most of them latency.  Here a workgroup of 16 waves takes 64 targets and all
// sources of their system, wave w the w-th sixteenth, so there is nothing left to add up, and makes
// the operands from the caller's points: the sources of a run on their way to LDS, the target's
// offset from a body's first source directly (one rounding where the two offsets of
// operands_kernel have two).  4 Stokes bodies, 300 sources and 600 targets each: 19.1 -> 13.7 us.
// ---------------------------------------------------------------------------
struct RawPoints {
    const double *trg, *src, *str;  // [n][3], [n][3], [n][3] or [n]
};

constexpr int WIDE = 16;  // waves
union WideShared {
    SrcS32 stokes[WIDE][FLUSH];
    SrcL32 laplace[WIDE][FLUSH];
    double part[WIDE][3][64];
};

template <bool STOKES>
__device__ __forceinline__ void wide_item(const KernelArgs &a, const P2PItem it, const RawPoints &raw, WideShared &sh) {
    constexpr int NW = WIDE, DIM = STOKES ? 3 : 1;
    using Rec = std::conditional_t<STOKES, SrcS32, SrcL32>;
    const bool active = !a.sys_active || a.sys_active[it.sys];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int idx = it.t0 + lane;
    const bool valid = idx < it.t1;
    const int i = valid ? idx : it.t0;
    const int body = a.trg_body[i];
    const double x[3] = {raw.trg[3 * (int64_t)i], raw.trg[3 * (int64_t)i + 1], raw.trg[3 * (int64_t)i + 2]};
    Rec *rec;  // the wave's own
    if constexpr (STOKES) rec = sh.stokes[wv];
    else rec = sh.laplace[wv];
    double acc[DIM] = {};
    const int s0 = a.src_ptr[it.b0], ns = a.src_ptr[it.b1] - s0;
    int j = s0 + (int)((int64_t)ns * wv / NW);
    const int j1 = active ? s0 + (int)((int64_t)ns * (wv + 1) / NW) : j;
    int b = it.b0;  // the body of source j
    for (int b64 = it.b0; j < j1 && b64 < it.b1; b64 += 64) {
        const int k = b64 + lane;
        b += __popcll(__ballot(k < it.b1 && a.src_ptr[min(k + 1, it.b1)] <= j));
        if (b < min(b64 + 64, it.b1)) break;
    }
    for (; j < j1; ++b) {
        const int end = min(a.src_ptr[b + 1], j1);
        const bool use = valid && !(a.skip_same && body == b);
        if (end <= j) continue;
        if (!__any(use)) {
            j = end;
            continue;
        }
        const double *first = raw.src + 3 * (int64_t)a.src_ptr[b];
        const double c0 = first[0], c1 = first[1], c2 = first[2];
        const float xr[1][3] = {{(float)(x[0] - c0), (float)(x[1] - c1), (float)(x[2] - c2)}};
        // runs no longer than the quarter of a body that a wave of p2p_mixed_kernel sums in FP32
        const int run = min(FLUSH, (a.src_ptr[b + 1] - a.src_ptr[b] + WAVES - 1) / WAVES);
        for (; j < end; j += run) {
            const int cnt = min(run, end - j);
            if (lane < cnt) {
                const int k = j + lane;
                const double *y = raw.src + 3 * (int64_t)k;
                const float d0 = (float)(y[0] - c0), d1 = (float)(y[1] - c1), d2 = (float)(y[2] - c2);
                if constexpr (STOKES) {
                    const double *f = raw.str + 3 * (int64_t)k;
                    rec[lane] = SrcS32{make_float4(d0, d1, d2, 0.f), make_float4((float)f[0], (float)f[1], (float)f[2], 0.f)};
                } else {
                    rec[lane] = make_float4(d0, d1, d2, (float)raw.str[k]);
                }
            }
            wave_lds_order();
            int k = 0;
            if constexpr (STOKES) {
                float p[1][3] = {{0.f, 0.f, 0.f}};
                for (; k + 4 <= cnt; k += 4) stokes_pairs<1, 4>(xr, rec + k, p);
                for (; k < cnt; ++k) stokes_pairs<1, 1>(xr, rec + k, p);
                for (int c = 0; c < 3; ++c) acc[c] += use ? (double)p[0][c] : 0.0;
            } else {
                float p[1] = {0.f};
                for (; k + 8 <= cnt; k += 8) laplace_pairs<1, 8>(xr, rec + k, p);
                for (; k < cnt; ++k) laplace_pairs<1, 1>(xr, rec + k, p);
                acc[0] += use ? (double)p[0] : 0.0;
            }
            __builtin_amdgcn_wave_barrier();  // the next run's stores follow this run's reads
        }
        j = end;
    }
    __syncthreads();  // the records are done with
    for (int c = 0; c < DIM; ++c) sh.part[wv][c][lane] = acc[c];
    __syncthreads();
    if (wv >= DIM || !valid) return;  // wave c: component c, the waves' sums in order
    double sum = sh.part[0][wv][lane];
    for (int w = 1; w < NW; ++w) sum += sh.part[w][wv][lane];
    const int64_t o = it.out0 + (int64_t)DIM * (idx - it.t0) + wv;
    double v = a.alpha * it.scale * sum;
    if (a.addend) v += a.addend[o];
    if (a.accumulate) v += a.out[o];
    a.out[o] = v;
}

__global__ __launch_bounds__(64 * WIDE) void p2p_wide_kernel(KernelArgs a, RawPoints raw) {
    __shared__ WideShared sh;
    const P2PItem it = a.items[blockIdx.x];
    if (it.kind == MFS_STOKES) wide_item<true>(a, it, raw, sh);
    else wide_item<false>(a, it, raw, sh);
}

// ---------------------------------------------------------------------------
// FP64
// ---------------------------------------------------------------------------
template <int TPL>
__device__ __forceinline__ void f64_item(const KernelArgs &a, const P2PItem it, const double4 *__restrict__ trg_off,
                                         const SrcS64 *__restrict__ srcS, const SrcL64 *__restrict__ srcL,
                                         double *lds) {
    // an inactive system still writes its epilogue (pair sum 0), so outputs stay finite
    const bool active = !a.sys_active || a.sys_active[it.sys];
    const bool stokes = it.kind == MFS_STOKES;
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    int idx[TPL];
    bool valid[TPL];
    int body[TPL];
    double ct[TPL][3];
    double xt[TPL][3];
    double acc[TPL][3];
#pragma unroll
    for (int t = 0; t < TPL; ++t) {
        idx[t] = it.t0 + lane + t * 64;
        valid[t] = idx[t] < it.t1;
        const int i = valid[t] ? idx[t] : it.t0;
        body[t] = a.trg_body[i];
        const double4 o = trg_off[i];
        xt[t][0] = o.x;
        xt[t][1] = o.y;
        xt[t][2] = o.z;
        ct[t][0] = a.centre[3 * body[t] + 0];
        ct[t][1] = a.centre[3 * body[t] + 1];
        ct[t][2] = a.centre[3 * body[t] + 2];
        acc[t][0] = acc[t][1] = acc[t][2] = 0.0;
    }

    for (int b = it.b0; active && b < it.b1; ++b) {
        bool use[TPL];
        bool any_use = false;
#pragma unroll
        for (int t = 0; t < TPL; ++t) {
            use[t] = valid[t] && !(a.skip_same && body[t] == b);
            any_use |= use[t];
        }
        if (!__any(any_use)) continue;
        const double cs0 = a.centre[3 * b + 0], cs1 = a.centre[3 * b + 1], cs2 = a.centre[3 * b + 2];
        double xr[TPL][3];
#pragma unroll
        for (int t = 0; t < TPL; ++t) {
            xr[t][0] = xt[t][0] + (ct[t][0] - cs0);
            xr[t][1] = xt[t][1] + (ct[t][1] - cs1);
            xr[t][2] = xt[t][2] + (ct[t][2] - cs2);
        }
        int j0, j1;
        wave_range(a.src_ptr[b], a.src_ptr[b + 1], wv, j0, j1);
        double p[TPL][3];
#pragma unroll
        for (int t = 0; t < TPL; ++t) p[t][0] = p[t][1] = p[t][2] = 0.0;
        if (stokes) {
const SrcS64 *__restrict__ ps = srcS + j0;
#pragma unroll 2
            for (int k = 0; k < j1 - j0; ++k) {
                const SrcS64 &sj = ps[k];
                const double y0 = sj.pos[0], y1 = sj.pos[1], y2 = sj.pos[2];
                const double f0 = sj.str[0], f1 = sj.str[1], f2 = sj.str[2];
#pragma unroll
                for (int t = 0; t < TPL; ++t) {
                    const double d0 = xr[t][0] - y0, d1 = xr[t][1] - y1, d2 = xr[t][2] - y2;
                    const double r2 = __builtin_fma(d2, d2, __builtin_fma(d1, d1, d0 * d0));
                    const double ri = rsqrt_f64(r2);
                    const double df = __builtin_fma(d2, f2, __builtin_fma(d1, f1, d0 * f0));
                    const double s = df * (ri * ri);
                    p[t][0] = __builtin_fma(ri, __builtin_fma(s, d0, f0), p[t][0]);
                    p[t][1] = __builtin_fma(ri, __builtin_fma(s, d1, f1), p[t][1]);
                    p[t][2] = __builtin_fma(ri, __builtin_fma(s, d2, f2), p[t][2]);
                }
            }
        } else {
const SrcL64 *__restrict__ ps = srcL + j0;
#pragma unroll 4
            for (int k = 0; k < j1 - j0; ++k) {
                const SrcL64 &sj = ps[k];
                const double y0 = sj.v[0], y1 = sj.v[1], y2 = sj.v[2], q = sj.v[3];
#pragma unroll
                for (int t = 0; t < TPL; ++t) {
                    const double d0 = xr[t][0] - y0, d1 = xr[t][1] - y1, d2 = xr[t][2] - y2;
                    const double r2 = __builtin_fma(d2, d2, __builtin_fma(d1, d1, d0 * d0));
                    p[t][0] = __builtin_fma(q, rsqrt_f64(r2), p[t][0]);
                }
            }
        }
#pragma unroll
        for (int t = 0; t < TPL; ++t) {
            acc[t][0] += use[t] ? p[t][0] : 0.0;
            acc[t][1] += use[t] ? p[t][1] : 0.0;
            acc[t][2] += use[t] ? p[t][2] : 0.0;
        }
    }

    double sum[TPL * 3];
#pragma unroll
    for (int t = 0; t < TPL; ++t)
#pragma unroll
        for (int c = 0; c < 3; ++c) sum[3 * t + c] = acc[t][c];
    if (!reduce_waves<TPL * 3>(sum, lds)) return;
    const int dim = stokes ? 3 : 1;
    double *out = a.out + (int64_t)it.split * a.out_stride;
#pragma unroll
    for (int t = 0; t < TPL; ++t) {
        if (!valid[t]) continue;
        const int64_t o = it.out0 + (int64_t)dim * (idx[t] - it.t0);
        for (int c = 0; c < dim; ++c) {
            double v = a.alpha * it.scale * sum[3 * t + c];
            if (a.addend) v += a.addend[o + c];
            if (a.accumulate) v += out[o + c];
            out[o + c] = v;
        }
    }
}

// One work item per workgroup, or (persistent mode) a fixed grid whose
// workgroups claim items from a counter until the list is exhausted; every
// workgroup ends with the claim that runs past the end, so the grid drains.
template <int TPL, bool STAGED>
__global__ __launch_bounds__(BLOCK) void p2p_mixed_kernel(KernelArgs a, const float4 *__restrict__ trg_off,
                                                          const SrcS32 *__restrict__ srcS,
                                                          const SrcL32 *__restrict__ srcL) {
    __shared__ double lds[(WAVES - 1) * 3 * TPL * 64];
    __shared__ float4 stage[WAVES * 64 * (STAGED ? 2 : 1)];
    if (!a.queue) {
        mixed_item<TPL, STAGED>(a, a.items[blockIdx.x], trg_off, srcS, srcL, lds, stage);
        return;
    }
    __shared__ int slot;
    for (;;) {
        __syncthreads();  // also orders the previous item's LDS reads before the next item's writes
        if (threadIdx.x == 0) slot = atomicAdd(a.queue, 1);
        __syncthreads();
        const int k = slot;
        if (k >= a.n_items) break;
        mixed_item<TPL, STAGED>(a, a.items[k], trg_off, srcS, srcL, lds, stage);
    }
}

// The same for launches with far tiles (Laplace items of 256 targets).
__global__ __launch_bounds__(BLOCK, 4) void p2p_far_kernel(KernelArgs a, const float4 *__restrict__ trg_off,
                                                        const SrcL32 *__restrict__ srcL) {
    __shared__ float4 stage[WAVES * 64];
    __shared__ uint4v frag[WAVES * 256];
    __shared__ float str[WAVES * 1024];
    __shared__ int slot;
    int k = blockIdx.x;
    for (;;) {  // one item, or until the queue is empty
        if (a.queue) {
            __syncthreads();  // also orders the previous item's LDS reads before the next item's writes
            if (threadIdx.x == 0) slot = atomicAdd(a.queue, 1);
            __syncthreads();
            k = slot;
        }
        if (k >= a.n_items) break;
        const P2PItem it = a.items[k];
        laplace_far_item(a, it, trg_off, srcL, stage, frag, str);
        if (!a.queue) break;
    }
}

template <int TPL>
__global__ __launch_bounds__(BLOCK) void p2p_f64_kernel(KernelArgs a, const double4 *__restrict__ trg_off,
                                                        const SrcS64 *__restrict__ srcS,
                                                        const SrcL64 *__restrict__ srcL) {
    __shared__ double lds[(WAVES - 1) * 3 * TPL * 64];
    if (!a.queue) {
        f64_item<TPL>(a, a.items[blockIdx.x], trg_off, srcS, srcL, lds);
        return;
    }
    __shared__ int slot;
    for (;;) {
        __syncthreads();  // also orders the previous item's LDS reads before the next item's writes
        if (threadIdx.x == 0) slot = atomicAdd(a.queue, 1);
        __syncthreads();
        const int k = slot;
        if (k >= a.n_items) break;
        f64_item<TPL>(a, a.items[k], trg_off, srcS, srcL, lds);
    }
}

__global__ void reset_counter_kernel(int *c) { *c = 0; }

// Sum of split slices: out = (acc ? out : 0) + addend + sum_s partial[s]
__global__ void reduce_split_kernel(int64_t n, const double *__restrict__ partial, int64_t stride, int n_split,
                                    const double *__restrict__ addend, double *__restrict__ out, int accumulate) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    double s = strided_sum(partial + v, stride, n_split);
    if (addend) s += addend[v];
    if (accumulate) s += out[v];
    out[v] = s;
}

// Far centre (the mean of the body's sources), radius and tiles of every body; one workgroup per
// body.  pos: [n][stride] from the body's base point (null: the origin).  A body with a source that
// is not finite or further than 1e12 gets an infinite radius: no target is far from it.
__global__ __launch_bounds__(256) void far_pack_kernel(const int32_t *__restrict__ ptr, const double *__restrict__ pos,
                                                       int stride, const double *__restrict__ base,
                                                       const int32_t *__restrict__ tile_ptr,
                                                       double *__restrict__ centre, uint4v *__restrict__ tiles,
                                                       float *__restrict__ rho) {
    __shared__ double part[4][3];
    __shared__ float sh[4];
    const int b = blockIdx.x, s0 = ptr[b], n = ptr[b + 1] - s0;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const double *y = pos + stride * (int64_t)s0;
    double c[3] = {0.0, 0.0, 0.0};
    for (int j = threadIdx.x; j < n; j += 256)
        for (int e = 0; e < 3; ++e) c[e] += y[stride * j + e];
    for (int e = 0; e < 3; ++e) {
        for (int d = 32; d > 0; d >>= 1) c[e] += __shfl_down(c[e], d, 64);
        if (lane == 0) part[wv][e] = c[e];
    }
    __syncthreads();
    for (int e = 0; e < 3; ++e) c[e] = (part[0][e] + part[1][e] + part[2][e] + part[3][e]) / max(n, 1);
    float r2 = 0.f;
    for (int j = threadIdx.x; j < n; j += 256) {
        const double d[3] = {y[stride * j] - c[0], y[stride * j + 1] - c[1], y[stride * j + 2] - c[2]};
        const double e = d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
        r2 = fmaxf(r2, e <= 1e24 ? (float)e : __builtin_inff());
    }
    for (int d = 32; d > 0; d >>= 1) r2 = fmaxf(r2, __shfl_down(r2, d, 64));
    if (lane == 0) sh[wv] = r2;
    __syncthreads();
    if (threadIdx.x == 0) rho[b] = 1.0001f * sqrtf(fmaxf(fmaxf(sh[0], sh[1]), fmaxf(sh[2], sh[3])));
    if (threadIdx.x < 3) {
        const int e = threadIdx.x;
        centre[3 * b + e] = (base ? base[3 * b + e] : 0.0) + (e == 0 ? c[0] : e == 1 ? c[1] : c[2]);
    }
    uint4v *t = tiles + 64 * (int64_t)tile_ptr[b];
    const int nt = (n + 15) / 16;
    for (int e = threadIdx.x; e < 64 * nt; e += 256) {
        const double *yj = y + stride * min(far_source(e >> 6, nt, e & 63), n - 1);  // past the last: no strength
        const double d[3] = {yj[0] - c[0], yj[1] - c[1], yj[2] - c[2]};
        t[e] = pack_far_tile(d, e & 63);
    }
}

__global__ void fill_ids_kernel(int64_t n_body, const int32_t *__restrict__ ptr, int32_t *__restrict__ ids) {
    const int64_t b = blockIdx.x;
    if (b >= n_body) return;
    for (int32_t i = ptr[b] + threadIdx.x; i < ptr[b + 1]; i += blockDim.x) ids[i] = (int32_t)b;
}

// Operands of a standalone call in one launch: thread k makes target k's offset, then source
// k - n_trg's record, then body k - n_trg - n_src's reference point (its first source point, or
// its first target point if it has no sources), which every point of the body reads for itself.
__device__ __forceinline__ const double *body_ref(const StandaloneOperands &o, int b) {
    if (o.src_ptr[b + 1] > o.src_ptr[b]) return o.src_xyz + 3 * (int64_t)o.src_ptr[b];
    if (o.trg_ptr[b + 1] > o.trg_ptr[b]) return o.trg_xyz + 3 * (int64_t)o.trg_ptr[b];
    return nullptr;
}

template <bool MIXED, bool STOKES>
__global__ __launch_bounds__(256) void operands_kernel(StandaloneOperands o) {
    int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < o.n_trg) {
        const double *c = body_ref(o, o.trg_body[k]), *x = o.trg_xyz + 3 * k;
        const double d0 = x[0] - c[0], d1 = x[1] - c[1], d2 = x[2] - c[2];
        if constexpr (MIXED) reinterpret_cast<float4 *>(o.trg_off)[k] = make_float4((float)d0, (float)d1, (float)d2, 0.f);
        else reinterpret_cast<double4 *>(o.trg_off)[k] = make_double4(d0, d1, d2, 0.0);
        return;
    }
    k -= o.n_trg;
    if (k < o.n_src) {
        const double *c = body_ref(o, o.src_body[k]), *y = o.src_xyz + 3 * k;
        const double d0 = y[0] - c[0], d1 = y[1] - c[1], d2 = y[2] - c[2];
        if constexpr (STOKES) {
            const double *f = o.str + 3 * k;
            if constexpr (MIXED)
                reinterpret_cast<SrcS32 *>(o.src_ops)[k] =
                    SrcS32{make_float4((float)d0, (float)d1, (float)d2, 0.f),
                           make_float4((float)f[0], (float)f[1], (float)f[2], 0.f)};
            else
                reinterpret_cast<SrcS64 *>(o.src_ops)[k] = SrcS64{{d0, d1, d2, 0.0}, {f[0], f[1], f[2], 0.0}};
        } else {
            const double q = o.str[k];
            if constexpr (MIXED)
                reinterpret_cast<SrcL32 *>(o.src_ops)[k] = make_float4((float)d0, (float)d1, (float)d2, (float)q);
            else
                reinterpret_cast<SrcL64 *>(o.src_ops)[k] = SrcL64{{d0, d1, d2, q}};
        }
        return;
    }
    k -= o.n_src;
    if (k >= o.n_body) return;
    const double *c = body_ref(o, (int)k);
    for (int e = 0; e < 3; ++e) o.centre[3 * k + e] = c ? c[e] : 0.0;
}

}  // namespace

P2PItems items_of(const P2PPlan &pp) {
    P2PItems it;
    it.items = pp.d_items.as<P2PItem>();
    it.n_items = (int)pp.items.size();
    it.n_split = pp.n_split;
    it.tpl = pp.tpl;
    it.far = pp.far;
    it.wide = pp.wide;
    it.persistent = pp.persistent;
    it.persistent_grid = pp.persistent_grid;
    it.counter = pp.d_counter.as<int>();
    return it;
}

int launch_p2p(const P2PItems &pp, const P2PLaunch &L, hipStream_t s) {
    if (pp.n_items == 0) return MFS_OK;
    if (pp.wide && pp.far) return fail(MFS_EINVAL, "pair sum: items of one walk given to another");
    KernelArgs a;
    a.items = pp.items;
    a.centre = L.centre;
    a.trg_body = L.trg_body;
    a.src_ptr = L.src_ptr;
    a.sys_active = L.sys_active;
    a.alpha = L.alpha;
    a.skip_same = L.skip_same ? 1 : 0;
    const bool direct = pp.n_split == 1;
    a.out = direct ? L.out : L.partial;
    a.addend = direct ? L.addend : nullptr;
    a.accumulate = direct ? (L.accumulate ? 1 : 0) : 0;
    a.out_stride = L.n_val;
    a.n_items = pp.n_items;
    a.queue = nullptr;
    dim3 grid((unsigned)pp.n_items);
    if (pp.persistent) {
        a.queue = pp.counter;
        grid = dim3((unsigned)std::min(pp.n_items, pp.persistent_grid));
        reset_counter_kernel<<<1, 1, 0, s>>>(a.queue);
        MFS_HIP_TRY(hipGetLastError());
    }
    if (L.ev_start) MFS_HIP_TRY(hipEventRecord(L.ev_start, s));
    if (L.prec == MFS_MIXED) {
        a.far_tiles = (const uint4v *)L.far.tiles;
        a.far_tile_ptr = L.far.tile_ptr;
        a.far_centre = L.far.centre;
        a.far_rho = L.far.rho;
        if (pp.wide)
            p2p_wide_kernel<<<grid, 64 * WIDE, 0, s>>>(a, RawPoints{L.raw_trg, L.raw_src, L.raw_str});
        else if (pp.tpl == 2)
            p2p_mixed_kernel<2, false><<<grid, BLOCK, 0, s>>>(a, (const float4 *)L.trg_off, (const SrcS32 *)L.srcS,
                                                              (const SrcL32 *)L.srcL);
        else if (pp.far)
            p2p_far_kernel<<<grid, BLOCK, 0, s>>>(a, (const float4 *)L.trg_off, (const SrcL32 *)L.srcL);
        else if (pp.n_items <= STAGED_ITEMS)
            p2p_mixed_kernel<1, true><<<grid, BLOCK, 0, s>>>(a, (const float4 *)L.trg_off, (const SrcS32 *)L.srcS,
                                                             (const SrcL32 *)L.srcL);
        else
            p2p_mixed_kernel<1, false><<<grid, BLOCK, 0, s>>>(a, (const float4 *)L.trg_off, (const SrcS32 *)L.srcS,
                                                              (const SrcL32 *)L.srcL);
    } else {
        if (pp.tpl == 2)
            p2p_f64_kernel<2><<<grid, BLOCK, 0, s>>>(a, (const double4 *)L.trg_off, (const SrcS64 *)L.srcS,
                                                     (const SrcL64 *)L.srcL);
        else
            p2p_f64_kernel<1><<<grid, BLOCK, 0, s>>>(a, (const double4 *)L.trg_off, (const SrcS64 *)L.srcS,
                                                     (const SrcL64 *)L.srcL);
    }
    MFS_HIP_TRY(hipGetLastError());
    if (L.ev_stop) MFS_HIP_TRY(hipEventRecord(L.ev_stop, s));
    if (!direct) {
        const int64_t n = L.n_val;
        reduce_split_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(n, L.partial, L.n_val, pp.n_split, L.addend,
                                                                      L.out, L.accumulate ? 1 : 0);
        MFS_HIP_TRY(hipGetLastError());
    }
    return MFS_OK;
}

int launch_fill_body_ids(int64_t n_body, const int32_t *ptr, int32_t *ids, hipStream_t s) {
    if (n_body == 0) return MFS_OK;
    fill_ids_kernel<<<(unsigned)n_body, 256, 0, s>>>(n_body, ptr, ids);
    MFS_HIP_TRY(hipGetLastError());
    return MFS_OK;
}

int launch_operands(const StandaloneOperands &o, int kind, int prec, hipStream_t s) {
    const int64_t n = o.n_trg + o.n_src + o.n_body;
    if (n == 0) return MFS_OK;
    const unsigned grid = (unsigned)((n + 255) / 256);
    if (prec == MFS_MIXED) {
        if (kind == MFS_STOKES) operands_kernel<true, true><<<grid, 256, 0, s>>>(o);
        else operands_kernel<true, false><<<grid, 256, 0, s>>>(o);
    } else {
        if (kind == MFS_STOKES) operands_kernel<false, true><<<grid, 256, 0, s>>>(o);
        else operands_kernel<false, false><<<grid, 256, 0, s>>>(o);
    }
    MFS_HIP_TRY(hipGetLastError());
    return MFS_OK;
}

int launch_far_pack(int64_t n_body, const int32_t *ptr, const double *pos, int stride, const double *base,
                    const FarTiles &far, hipStream_t s) {
    if (n_body == 0) return MFS_OK;
    far_pack_kernel<<<(unsigned)n_body, 256, 0, s>>>(ptr, pos, stride, base, far.tile_ptr, far.centre,
                                                     (uint4v *)far.tiles, far.rho);
    MFS_HIP_TRY(hipGetLastError());
    return MFS_OK;
}

}  // namespace mfs
