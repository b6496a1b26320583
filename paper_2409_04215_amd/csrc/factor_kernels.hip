// Batched FP64 QR factorisation of the one-body blocks on the GPU (gfx950).
//
// The pseudo-inverse of a full-column-rank m x n matrix A (m >= n) is
// A^+ = R^-1 Q^T with A = Q R (Q m x n with orthonormal columns, R n x n
// upper triangular): the same operator as V Sigma^-1 U^T from the SVD of
// Section 2.3, applied in the same two steps (Q^T, then R^-1).
//
// Blocked Householder QR (compact WY form).  The columns are taken in panels
// of NB = 16; the reflectors H_j = I - tau_j v_j v_j^T of one panel (v_j[j] = 1,
// stored below the diagonal of column j, R on and above it) multiply to
// H_k0 ... H_k0+kb-1 = I - V T V^T with T kb x kb upper triangular:
//   * panel_qr_kernel: one workgroup per matrix factors the panel column by
//     column (v_j, tau_j, R_jj, then H_j applied to the panel's later columns,
//     half a wave per column) and forms T from tau and the Gram matrix V^T V
//     (T_jj = tau_j, T[0:j, j] = -tau_j T[0:j, 0:j] (V^T v_j)[0:j]);
//   * wy_apply_kernel: the trailing columns C = A[k0:m, k0+kb:n] take
//     C <- (I - V T^T V^T) C, i.e. H_k0+kb-1 ... H_k0 applied at once, as
//     P = V^T C, W = T^T P, C -= V W, both products on the FP64 matrix cores
//     (v_mfma_f64_16x16x4f64); one workgroup per 16 columns.
// Q = H_0 H_1 ... H_{n-1} [I; 0] is accumulated panel by panel from the last
// one in the same way (C <- (I - V T V^T) C on rows k0..m-1 of columns
// k0..n-1; earlier columns of Q are still unit vectors there), and
// X = R^-1 comes from n independent triangular solves R x_i = e_i.  These are
// the kernels for many rows; most matrices take the ones further down.
// Reductions add in a fixed order: results do not depend on timing.
#include <algorithm>
#include <type_traits>

#include "mfs_internal.h"

namespace mfs {

namespace {

constexpr int FB = 256;   // threads per workgroup (inverse, ratio, WY update)
// Panel width: one 16-column MFMA tile.  In the kernels for many rows 16 columns
// beat 32 (2400 x 1200 through them: panels 20.6 ms + updates 10.4 ms against
// 33 ms + 7.6 ms): the one-workgroup panel factorisation does half the work per
// column and the MFMA updates take the rest.
constexpr int NB = 16;
constexpr int PT = 32 * NB;  // threads of the panel kernel: half a wave per panel column
constexpr int PW = PT / 64;
constexpr int CT = 16;    // columns per workgroup of the WY update

typedef double doublex4 __attribute__((ext_vector_type(4)));

// sum over the workgroup in a fixed order (wave shuffles, then the waves in order)
template <int NW>
__device__ double block_sum_fixed(double x, double *sh) {
    for (int off = 32; off > 0; off >>= 1) x += __shfl_down(x, off, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = x;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) t += sh[w];
    __syncthreads();
    return t;
}

// One panel (columns k0 .. k0+kb-1, rows k0 .. m-1) of every matrix; T of the panel to
// Tp[b][NB][NB] (row-major, zero outside the leading kb x kb upper triangle).
// Step j (column c = k0 + j): the norm of the column below the diagonal (all threads,
// fixed-order block sum), v_j and tau_j, then one pass over the panel's other columns:
// wave w owns columns 2w and 2w+1, lane l column 2w + l/32 and rows c+1 + l%32 + 32 i,
// so a column's partial sums are added by a 32-lane butterfly inside the wave (every lane
// gets the sum) and the same lanes apply H_j to that column without a barrier.  The same
// pass gives the Gram entries G[i][j] = v_i . v_j of the earlier columns (v_j is 1 at row
// c and zero above), from which T follows:
// T_jj = tau_j, T[0:j, j] = -tau_j T[0:j, 0:j] G[0:j, j].
__global__ __launch_bounds__(PT) void panel_qr_kernel(double *__restrict__ A, int m, int lda, int64_t stride, int k0,
                                                      int kb, double *__restrict__ tau, int n, double *__restrict__ Tp) {
    __shared__ double sh[PW];
    __shared__ double G[NB][NB + 1];
    __shared__ double Ts[NB][NB + 1];
    __shared__ double tl[NB];
    const int b = blockIdx.x, t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int q = 2 * wave + (lane >> 5), g = lane & 31;  // this lane's panel column and row phase
    double *a = A + (int64_t)b * stride;
    double *xq = a + (int64_t)(k0 + q) * lda;  // dereferenced only for q < kb
    for (int j = 0; j < kb; ++j) {
        const int c = k0 + j;
        double *col = a + (int64_t)c * lda;
        const double alpha = col[c];  // read before the reduction's barriers: thread 0 overwrites it below
        double ss = 0.0;
        for (int r = c + 1 + t; r < m; r += PT) ss += col[r] * col[r];
        ss = block_sum_fixed<PW>(ss, sh);
        double tj = 0.0, scal = 1.0;  // nothing below the diagonal: H_j = I, R_jj = A_jj
        if (ss != 0.0) {
            const double nrm = sqrt(alpha * alpha + ss);
            const double beta = alpha >= 0.0 ? -nrm : nrm;  // no cancellation in alpha - beta
            scal = 1.0 / (alpha - beta);
            tj = (beta - alpha) / beta;
            for (int r = c + 1 + t; r < m; r += PT) col[r] *= scal;
            if (t == 0) col[c] = beta;
        }
        if (t == 0) {
            tau[(int64_t)b * n + c] = tj;
            tl[j] = tj;
        }
        __syncthreads();  // v_j in place
        if (q < kb && q != j) {
            double d = 0.0;
            int r = c + 1 + g;
            for (; r + 96 < m; r += 128) {  // four rows in flight per lane
                const double v0 = col[r], v1 = col[r + 32], v2 = col[r + 64], v3 = col[r + 96];
                const double x0 = xq[r], x1 = xq[r + 32], x2 = xq[r + 64], x3 = xq[r + 96];
                d += v0 * x0;
                d += v1 * x1;
                d += v2 * x2;
                d += v3 * x3;
            }
            for (; r < m; r += 32) d += col[r] * xq[r];
#pragma unroll
            for (int off = 16; off > 0; off >>= 1) d += __shfl_xor(d, off, 64);
            const double xc = xq[c];
            if (q < j) {
                if (g == 0) G[q][j] = d + xc;  // v_q . v_j
            } else if (tj != 0.0) {
                const double w = (d + xc) * tj;
                for (int rr = c + 1 + g; rr < m; rr += 32) xq[rr] -= w * col[rr];
                if (g == 0) xq[c] = xc - w;
            }
        }
        __syncthreads();
    }
    // T column by column in wave 0: lane i owns row i, so it reads only its own earlier entries
    if (wave == 0 && lane < NB) {
        const int i = lane;
        for (int j = 0; j < NB; ++j) {
            double v = 0.0;
            if (j < kb) {
                if (i < j) {
                    double s = 0.0;
                    for (int l = i; l < j; ++l) s += Ts[i][l] * G[l][j];
                    v = -tl[j] * s;
                } else if (i == j) {
                    v = tl[j];
                }
            }
            Ts[i][j] = v;
        }
    }
    __syncthreads();
    double *T = Tp + (int64_t)b * NB * NB;
    for (int e = t; e < NB * NB; e += PT) T[e] = Ts[e / NB][e % NB];
}

// V[r][i] of the panel at k0 (unit lower trapezoidal, zero past kb columns or m rows)
__device__ __forceinline__ double panel_v(const double *__restrict__ v, int lda, int m, int k0, int kb, int r, int i) {
    if (i >= kb || r >= m) return 0.0;
    const int d = k0 + i;
    if (r < d) return 0.0;
    if (r == d) return 1.0;
    return v[(int64_t)d * lda + r];
}

// C[k0:m, c0:c1] <- (I - V op(T) V^T) C[k0:m, c0:c1] with V, T of the panel at k0;
// op(T) = T^T (TRANS: the QR's trailing update) or T (accumulating Q).
// Grid (column tiles of CT, batch); four waves.
//  1. P = V^T C (NB x CT): each wave sums a quarter of the rows in steps of 16;
//     MFMA A = V^T (lane l: V[r][k0 + l%16]), B = C (lane l: C[r][col l%16]),
//     the k slot l/16 of MFMA t standing for row r = r0 + 4 (l/16) + t in both;
//     D layout (16x16x4 f64): lane l, reg q -> row l/16 + 4 q, col l%16.
//  2. The four partial P added in wave order, W = op(T) P in LDS.
//  3. C -= V W by 16-row blocks as D^T = W^T V^T (16 columns x 16 rows): lane l gives
//     W[k][l%16] and V[r0 + l%16][k0 + k] for k = 4 t + l/16, and holds C rows
//     r0 + l%16 of columns l/16 + 4 q: 16 consecutive rows of one column per
//     16 lanes, so the read-modify-write of C is coalesced.
template <bool TRANS>
__global__ __launch_bounds__(FB) void wy_apply_kernel(const double *__restrict__ V, int m, int lda, int64_t stride_v,
                                                      int k0, int kb, const double *__restrict__ Tp,
                                                      double *__restrict__ C, int ldc, int64_t stride_c, int c0,
                                                      int c1) {
    __shared__ double Pw[4][NB][CT];
    __shared__ double Ps[NB][CT];
    __shared__ double Wl[NB][CT];
    __shared__ double Ts[NB][NB + 1];
    const int b = blockIdx.y, t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int q = lane >> 4, c16 = lane & 15;
    const int cbase = c0 + (int)blockIdx.x * CT;
    const double *v = V + (int64_t)b * stride_v;
    double *cm = C + (int64_t)b * stride_c;
    const double *T = Tp + (int64_t)b * NB * NB;
    for (int e = t; e < NB * NB; e += FB) Ts[e / NB][e % NB] = T[e];

    // 1. P = V^T C
    const int col = cbase + c16;
    const bool cok = col < c1;
    const double *ccol = cm + (int64_t)(cok ? col : c0) * ldc;
    doublex4 acc = {0.0, 0.0, 0.0, 0.0};
    for (int r0 = k0 + 16 * wave; r0 < m; r0 += 64) {
        const int rb = r0 + 4 * q;
        double cv[4], va[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int r = rb + u;
            cv[u] = (cok && r < m) ? ccol[r] : 0.0;
            va[u] = panel_v(v, lda, m, k0, kb, r, c16);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(va[u], cv[u], acc, 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) Pw[wave][q + 4 * r][c16] = acc[r];
    __syncthreads();
    // 2. P summed over the waves in order, W = op(T) P
    for (int e = t; e < NB * CT; e += FB) {
        const int i = e / CT, j = e % CT;
        Ps[i][j] = ((Pw[0][i][j] + Pw[1][i][j]) + Pw[2][i][j]) + Pw[3][i][j];
    }
    __syncthreads();
    for (int e = t; e < NB * CT; e += FB) {
        const int i = e / CT, j = e % CT;
        double s = 0.0;
        if (TRANS) {
            for (int l = 0; l <= i; ++l) s += Ts[l][i] * Ps[l][j];  // (T^T)[i][l] = T[l][i], l <= i
        } else {
            for (int l = i; l < NB; ++l) s += Ts[i][l] * Ps[l][j];
        }
        Wl[i][j] = s;
    }
    __syncthreads();
    // 3. C -= V W
    for (int r0 = k0 + 16 * wave; r0 < m; r0 += 64) {
        const int r = r0 + c16;
        doublex4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int u = 0; u < NB / 4; ++u) {
            const int k = 4 * u + q;
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(Wl[k][c16], panel_v(v, lda, m, k0, kb, r, k), acc, 0, 0, 0);
        }
        if (r < m) {
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) {
                const int cc = cbase + q + 4 * rr;
                if (cc < c1) cm[(int64_t)cc * ldc + r] -= acc[rr];
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Steps for matrices whose rows fit one workgroup's registers (at most
// QT * QR_MAX_RPT = 2560 rows; larger ones take the kernels above).
//
// A panel is a serial chain, column after column, so its time is latency:
// panel_qr_kernel, which re-reads the panel from L2 in every column step, took
// 0.27 ms per panel at 2400 rows, and wy_apply_kernel 69 us, its loads one
// block of rows in flight per wave.  Here
//  * the panel stays in registers, 16 columns of RPT rows in each of 512
//    threads (a CU's 512 KB of registers against 0.3 MB of panel);
//  * a column step is one pass, one barrier: the sums x_j . X_q over the rows
//    below the diagonal give the norm, v_j . X_q (by scaling, with the row of the
//    diagonal added) and the Gram entries of T together.  The columns rotate by
//    one place per step, so the step is a loop body and not 16 unrolled copies
//    (200 KB of code, run once, took 129 us per panel in instruction fetches);
//  * the WY update has six blocks of rows in flight per wave;
//  * one launch per panel: workgroup 0 updates the next panel's columns and
//    factors them, both in the panel's registers, the others update the rest
//    meanwhile (52 to 67 us a step);
//  * Q and R^-1 are one launch each, 16 columns per workgroup in registers.
// 2400 x 1200 (QR, Q and R^-1): 32.0 ms before, 6.4 ms now (4.4, 1.55 and 0.37), plan
// creation 34.6 -> 7.7 ms.  sqrt and the divisions are not what a column step waits
// for: through v_rsq_f64 and v_rcp_f64 a panel took the same 40 us.
// ---------------------------------------------------------------------------
constexpr int QT = 512;        // threads
constexpr int QW = QT / 64;    // waves
constexpr int QR_MAX_RPT = 5;  // rows per thread: 16 columns x 5 rows are 160 registers
constexpr int QU = 6;          // row blocks in flight per wave of the WY update
static_assert(NB == 16 && CT == 16, "one 16 x 16 tile of P, four lanes per panel column");

struct QrShared {
    double Pw[QW][NB][CT];  // partial V^T C of every wave
    double W[NB][CT];
    double Ts[NB][NB + 1];
    double red[2][QW][NB];  // partial sums of a column step, double-buffered
    double row[2][NB];      // the diagonal's row
    double G[NB][NB + 1];
    double tl[NB];
};

__device__ __forceinline__ double lane_value(double x, int lane) {  // lane: uniform
    const int lo = __builtin_amdgcn_readlane(__double2loint(x), lane);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(x), lane);
    return __hiloint2double(hi, lo);
}

// x of another lane of the row of 16: CTRL a DPP control that is a permutation of the row
template <int CTRL>
__device__ __forceinline__ double dpp_move(double x) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}

// a summed over a lane and its partner 32 (16) away in the lower half, b in the upper one
template <int DIST>
__device__ __forceinline__ double swap_add(double a, double b) {
    typedef unsigned uint2v __attribute__((ext_vector_type(2)));
    uint2v lo, hi;
    if constexpr (DIST == 32) {
        lo = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
        hi = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
    } else {
        lo = __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
        hi = __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
    }
    return __hiloint2double(hi.x, lo.x) + __hiloint2double(hi.y, lo.y);
}

// Sums of v[0..15] over the wave; lane l returns the sum of v[l / 4].  Every exchange halves
// the values a lane still carries (8 + 4 + 2 + 1), the last two add the four lanes of a value.
__device__ __forceinline__ double wave_sums16(double (&v)[16], int lane) {
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = swap_add<32>(v[q], v[q + 8]);
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = swap_add<16>(v[q], v[q + 4]);
    const bool up8 = (lane & 8) != 0, up4 = (lane & 4) != 0;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const double send = up8 ? v[q] : v[q + 2], keep = up8 ? v[q + 2] : v[q];
        v[q] = keep + dpp_move<0x128>(send);  // row_ror:8
    }
    const double send = up4 ? v[0] : v[1], keep = up4 ? v[1] : v[0];
    double r = keep + dpp_move<0x141>(send);  // row_half_mirror: the other four of the eight
    r += dpp_move<0xB1>(r);                   // quad_perm [1,0,3,2]
    r += dpp_move<0x4E>(r);                   // quad_perm [2,3,0,1]
    return r;
}

// The panel at k0 (kb columns, rows k0..m-1) in registers: thread t holds rows k0 + t + QT i.
template <int RPT>
__device__ __forceinline__ void panel_load(const double *__restrict__ a, int m, int lda, int k0, int kb,
                                           double (&X)[RPT][NB]) {
    const unsigned rows = (unsigned)(m - k0);
#pragma unroll
    for (int q = 0; q < NB; ++q) {
        const double *x = a + (int64_t)(k0 + (q < kb ? q : 0)) * lda + k0;
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            const unsigned r = threadIdx.x + QT * i;
            X[i][q] = (r < rows && q < kb) ? x[r] : 0.0;
        }
    }
}

// Applies the panel before (its NB columns at k0 - NB, T in T) to the panel in X, and to its rows
// k0 - NB..k0-1 in memory: P = V^T C, W = T^T P, C -= V W.  The panel then goes on to its
// factorisation from registers; through wy_update and memory a step of the 2400 x 1200 QR took
// 72 us (at 2048 to 1537 rows), now 60.
template <int RPT>
__device__ __forceinline__ void panel_update(double *__restrict__ a, int m, int lda, int k0, int kb,
                                             const double *__restrict__ T, double (&X)[RPT][NB], QrShared &sh) {
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, ql = lane >> 2;
    const unsigned rows = (unsigned)(m - k0);
    const int p0 = k0 - NB, tr = t % NB, tc = t / NB;  // row and column of a 16 x 16 block, t < 256
    double *top = a + (int64_t)(k0 + min(tc, kb - 1)) * lda + p0 + tr;
    double c_top = 0.0;
    if (t < NB * NB) {
        c_top = *top;
        const double v = a[(int64_t)(p0 + tc) * lda + p0 + tr];
        sh.Ts[t / NB][t % NB] = T[t];
        sh.W[tr][tc] = c_top;
        sh.G[tr][tc] = tr < tc ? 0.0 : (tr == tc ? 1.0 : v);  // the unit lower triangle of V
    }
    auto load_v = [&](double (&v)[RPT], int j) {
        const double *x = a + (int64_t)(p0 + min(j, NB - 1)) * lda + k0;
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            const unsigned r = t + QT * i;
            v[i] = r < rows ? x[r] : 0.0;
        }
    };
    double v[RPT], next[RPT];
    load_v(next, 0);
#pragma unroll 1
    for (int j = 0; j < NB; ++j) {
#pragma unroll
        for (int i = 0; i < RPT; ++i) v[i] = next[i];
        load_v(next, j + 1);
        double d[NB];
#pragma unroll
        for (int q = 0; q < NB; ++q) d[q] = v[0] * X[0][q];
#pragma unroll
        for (int i = 1; i < RPT; ++i)
#pragma unroll
            for (int q = 0; q < NB; ++q) d[q] += v[i] * X[i][q];
        const double part = wave_sums16(d, lane);
        if ((lane & 3) == 0) sh.Pw[wave][j][ql] = part;
    }
    __syncthreads();
    if (t < NB * NB) {  // P summed over the waves in order, then the rows above
        double s = sh.Pw[0][tr][tc];
#pragma unroll
        for (int w = 1; w < QW; ++w) s += sh.Pw[w][tr][tc];
#pragma unroll
        for (int r = 0; r < NB; ++r) s += sh.G[r][tr] * sh.W[r][tc];
        sh.Pw[0][tr][tc] = s;
    }
    __syncthreads();
    if (t < NB * NB) {
        double s = 0.0;
        for (int l = 0; l <= tr; ++l) s += sh.Ts[l][tr] * sh.Pw[0][l][tc];
        sh.W[tr][tc] = s;
    }
    __syncthreads();
    if (t < NB * NB && tc < kb) {
        double o = 0.0;
#pragma unroll
        for (int j = 0; j < NB; ++j) o += sh.G[tr][j] * sh.W[j][tc];
        *top = c_top - o;
    }
#pragma unroll 1
    for (int j = 0; j < NB; j += 4) {  // four columns of V at a time: X is rounded four times
        double u[4][RPT];
#pragma unroll
        for (int e = 0; e < 4; ++e) load_v(u[e], j + e);
#pragma unroll
        for (int q = 0; q < NB; ++q) {
            double w[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e] = sh.W[j + e][q];
#pragma unroll
            for (int i = 0; i < RPT; ++i) X[i][q] -= u[0][i] * w[0] + u[1][i] * w[1] + u[2][i] * w[2] + u[3][i] * w[3];
        }
    }
    __syncthreads();  // the factorisation writes G and Ts
}

// Factors the panel in X (panel_load) and forms T, as panel_qr_kernel does.  At step j the
// registers hold the columns j, j+1, ..., 15, 0, ..., j-1, the last j of them reflectors already.
template <int RPT>
__device__ __forceinline__ void panel_registers(double *__restrict__ a, int m, int lda, int k0, int kb,
                                                double (&X)[RPT][NB], double *__restrict__ tau, double *__restrict__ T,
                                                QrShared &sh) {
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, ql = lane >> 2;
    const unsigned rows = (unsigned)(m - k0);
#pragma unroll 1
    for (int j = 0; j < NB; ++j) {
        double d[NB];
        {
            const double x = t > j ? X[0][0] : 0.0;  // the rows at and above the diagonal are in the first block
#pragma unroll
            for (int q = 0; q < NB; ++q) d[q] = x * X[0][q];
        }
#pragma unroll
        for (int i = 1; i < RPT; ++i)
#pragma unroll
            for (int q = 0; q < NB; ++q) d[q] += X[i][0] * X[i][q];
        const int buf = j & 1;
        if (t == j)
#pragma unroll
            for (int q = 0; q < NB; ++q) sh.row[buf][q] = X[0][q];
        const double part = wave_sums16(d, lane);
        if ((lane & 3) == 0) sh.red[buf][wave][ql] = part;
        // one barrier per step: a buffer is written again two steps later, after the next
        // step's barrier, which every thread reaches past its reads here
        __syncthreads();
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < QW; ++w) s += sh.red[buf][w][ql];  // x_j . X_ql below the diagonal
        const double rq = sh.row[buf][ql], alpha = sh.row[buf][0];
        const double ss = lane_value(s, 0);
        double tj = 0.0, scal = 1.0, beta = alpha;  // nothing below the diagonal: H_j = I, R_jj = A_jj
        if (ss != 0.0) {
            const double nrm = sqrt(alpha * alpha + ss);
            beta = alpha >= 0.0 ? -nrm : nrm;  // no cancellation in alpha - beta
            scal = 1.0 / (alpha - beta);
            tj = (beta - alpha) / beta;
        }
        const double gq = scal * s + rq;  // v_j . X_ql, the diagonal's row included
        const bool later = ql < NB - j;   // else X_ql is reflector ql - (NB - j)
        const double wq = later ? tj * gq : 0.0;
        if (wave == 0 && (lane & 3) == 0 && !later) sh.G[ql - (NB - j)][j] = gq;
        if (t == 0) {
            sh.tl[j] = tj;
            if (j < kb) tau[k0 + j] = tj;
        }
        double v[RPT];
        const double x0 = X[0][0];
        v[0] = t > j ? x0 * scal : (t == j ? 1.0 : 0.0);
#pragma unroll
        for (int i = 1; i < RPT; ++i) v[i] = X[i][0] * scal;
#pragma unroll
        for (int q = 1; q < NB; ++q) {  // H_j applied to the later columns, each one place on
            const double w = lane_value(wq, 4 * q);
#pragma unroll
            for (int i = 0; i < RPT; ++i) X[i][q - 1] = X[i][q] - w * v[i];
        }
        X[0][NB - 1] = t > j ? v[0] : (t == j ? beta : x0);
#pragma unroll
        for (int i = 1; i < RPT; ++i) X[i][NB - 1] = v[i];
    }
#pragma unroll
    for (int q = 0; q < NB; ++q) {
        double *x = a + (int64_t)(k0 + (q < kb ? q : 0)) * lda + k0;
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            const unsigned r = t + QT * i;
            if (r < rows && q < kb) x[r] = X[i][q];
        }
    }
    __syncthreads();  // G and tl complete
    if (wave == 0 && lane < NB) {  // T column by column: lane i owns row i
        const int i = lane;
        for (int j = 0; j < NB; ++j) {
            double v = 0.0;
            if (j < kb) {
                if (i < j) {
                    double s = 0.0;
                    for (int l = i; l < j; ++l) s += sh.Ts[i][l] * sh.G[l][j];
                    v = -sh.tl[j] * s;
                } else if (i == j) {
                    v = sh.tl[j];
                }
            }
            sh.Ts[i][j] = v;
        }
        for (int j = 0; j < NB; ++j) T[i * NB + j] = sh.Ts[i][j];
    }
}

struct __attribute__((packed, aligned(8))) Rows4 { double v[4]; };  // four rows of a column

// C[k0:m, cbase : min(cbase + 16, c1)] <- (I - V T^T V^T) C, as wy_apply_kernel.  Lane l of a
// 16-row block r0 holds rows r0 + 4 (l/16) + (0..3) of column l%16: the k slots of V^T C (MFMA u
// takes row u of the four), and the D layout of V W when row i of the A operand there is row
// 4 (i%4) + i/4 of the block.  Block b is wave b % QW's.
__device__ __forceinline__ void wy_update(const double *__restrict__ v, int m, int lda, int k0, int kb,
                                          const double *__restrict__ T, double *__restrict__ cm, int ldc, int cbase,
                                          int c1, QrShared &sh) {
    const int t = threadIdx.x, lane = t & 63, q = lane >> 4, c16 = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int full = (m - k0) / 16;  // whole blocks; one more may hold the last rows
    const int col = cbase + c16;
    const bool cok = col < c1, vok = c16 < kb;
    double *ccol = cm + (int64_t)(cok ? col : cbase) * ldc + k0 + 4 * q;
    const double *vcol = v + (int64_t)(k0 + (vok ? c16 : 0)) * lda + k0 + 4 * q;
    for (int e = t; e < NB * NB; e += QT) sh.Ts[e / NB][e % NB] = T[e];
    // 1. P = V^T C; a block past the last whole one reads the last whole one and counts as zero
    doublex4 acc[2] = {};
    auto add = [&](const Rows4 &c, const Rows4 &x, int b) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            double y = vok ? x.v[u] : 0.0;
            if (b == 0) {  // the unit lower triangle
                const int r = 4 * q + u;
                y = (r < c16 || !vok) ? 0.0 : (r == c16 ? 1.0 : y);
            }
            acc[u & 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(y, c.v[u], acc[u & 1], 0, 0, 0);
        }
    };
    for (int b0 = wave; b0 < full; b0 += QW * QU) {
        Rows4 c[QU], x[QU];
#pragma unroll
        for (int i = 0; i < QU; ++i) {
            const int b = min(b0 + QW * i, full - 1);
            c[i] = *reinterpret_cast<const Rows4 *>(ccol + 16 * b);
            x[i] = *reinterpret_cast<const Rows4 *>(vcol + 16 * b);
        }
#pragma unroll
        for (int i = 0; i < QU; ++i)
            if (b0 + QW * i < full) add(c[i], x[i], b0 + QW * i);
    }
    if (k0 + 16 * full < m && wave == full % QW) {
        Rows4 c, x;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const bool ok = k0 + 16 * full + 4 * q + u < m;
            c.v[u] = ok ? ccol[16 * full + u] : 0.0;
            x.v[u] = ok ? vcol[16 * full + u] : 0.0;
        }
        add(c, x, full);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) sh.Pw[wave][q + 4 * r][c16] = acc[0][r] + acc[1][r];
    __syncthreads();
    if (t < NB * CT) {  // P summed over the waves in order
        const int i = t / CT, j = t % CT;
        double p = sh.Pw[0][i][j];
#pragma unroll
        for (int w = 1; w < QW; ++w) p += sh.Pw[w][i][j];
        sh.Pw[0][i][j] = p;
    }
    __syncthreads();
    if (t < NB * CT) {  // 2. W = T^T P
        const int i = t / CT, j = t % CT;
        double s = 0.0;
        for (int l = 0; l <= i; ++l) s += sh.Ts[l][i] * sh.Pw[0][l][j];
        sh.W[i][j] = s;
    }
    __syncthreads();
    // 3. C -= V W
    double wv[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) wv[u] = sh.W[4 * u + q][c16];
    const int rho = 4 * (c16 & 3) + (c16 >> 2);
    const double *vk[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) vk[u] = v + (int64_t)(k0 + min(4 * u + q, kb - 1)) * lda + k0 + rho;
    auto product = [&](const double (&x)[4], int b) {
        doublex4 o = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int k = 4 * u + q;
            double y = k < kb ? x[u] : 0.0;
            if (b == 0) y = (rho < k || k >= kb) ? 0.0 : (rho == k ? 1.0 : y);
            o = __builtin_amdgcn_mfma_f64_16x16x4f64(y, wv[u], o, 0, 0, 0);
        }
        return o;
    };
    for (int b0 = wave; b0 < full; b0 += QW * QU) {
        Rows4 c[QU];
        double x[QU][4];
#pragma unroll
        for (int i = 0; i < QU; ++i) {
            const int b = min(b0 + QW * i, full - 1);
            c[i] = *reinterpret_cast<const Rows4 *>(ccol + 16 * b);
#pragma unroll
            for (int u = 0; u < 4; ++u) x[i][u] = vk[u][16 * b];
        }
#pragma unroll
        for (int i = 0; i < QU; ++i) {
            const int b = b0 + QW * i;
            if (b >= full) continue;
            const doublex4 o = product(x[i], b);
#pragma unroll
            for (int u = 0; u < 4; ++u) c[i].v[u] -= o[u];
            if (cok) *reinterpret_cast<Rows4 *>(ccol + 16 * b) = c[i];
        }
    }
    if (k0 + 16 * full < m && wave == full % QW) {
        double x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = k0 + 16 * full + rho < m ? vk[u][16 * full] : 0.0;
        const doublex4 o = product(x, full);
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (cok && k0 + 16 * full + 4 * q + u < m) ccol[16 * full + u] -= o[u];
    }
}

// First panel.
template <int RPT>
__global__ __launch_bounds__(QT) void qr_first_kernel(double *__restrict__ A, int m, int64_t stride, int kb,
                                                      double *__restrict__ tau, int n, double *__restrict__ Tp) {
    __shared__ QrShared sh;
    const int b = blockIdx.x;
    double *a = A + (int64_t)b * stride, X[RPT][NB];
    panel_load<RPT>(a, m, m, 0, kb, X);
    panel_registers<RPT>(a, m, m, 0, kb, X, tau + (int64_t)b * n, Tp + (int64_t)b * NB * NB, sh);
}

// One step of the QR: the panel at k0 (factored, T in Tp) is applied to the columns after it,
// one workgroup per 16 columns; workgroup 0, whose columns are the next panel, factors them.
template <int RPT>
__global__ __launch_bounds__(QT) void qr_step_kernel(double *__restrict__ A, int m, int64_t stride, int k0, int n,
                                                     const double *__restrict__ Tp, double *__restrict__ tau,
                                                     double *__restrict__ Tnext) {
    __shared__ QrShared sh;
    const int b = blockIdx.y, c = k0 + NB + (int)blockIdx.x * CT;
    double *a = A + (int64_t)b * stride;
    if (blockIdx.x != 0) {  // uniform over the workgroup
        wy_update(a, m, m, k0, NB, Tp + (int64_t)b * NB * NB, a, m, c, n, sh);
        return;
    }
    const int kb = min(NB, n - c);
    double X[RPT][NB];
    panel_load<RPT>(a, m, m, c, kb, X);
    panel_update<RPT>(a, m, m, c, kb, Tp + (int64_t)b * NB * NB, X, sh);
    panel_registers<RPT>(a, m, m, c, kb, X, tau + (int64_t)b * n, Tnext + (int64_t)b * NB * NB, sh);
}

// 16 columns of Q = H_0 H_1 ... [I; 0] in one workgroup's registers through all panels that reach
// them (panel p touches columns 16 p and later), last panel first.  Block b (rows 16 b ..) is wave
// b % QW's slot b / QW, in the layout of wy_update: V^T C and C - V W both take it as it lies, so
// only V moves (twice per panel, from L2).  A launch per panel with C in memory took 38 us a panel,
// 2.8 ms for 2400 x 1200; now 1.55.
template <int RPT>
__global__ __launch_bounds__(QT) void q_kernel(const double *__restrict__ A, int m, int64_t stride_a, int n,
                                               const double *__restrict__ Tall, int batch, double *__restrict__ Q,
                                               int64_t stride_q) {
    constexpr int SLOTS = RPT * QT / 16 / QW, GR = 4;  // blocks per wave, blocks in flight
    __shared__ QrShared sh;
    const int t = threadIdx.x, lane = t & 63, q = lane >> 4, c16 = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int cb = (int)(gridDim.x - 1 - blockIdx.x), b = blockIdx.y;  // the longest chains first
    const int col = 16 * cb + c16;
    const int blocks = (m + 15) / 16, whole = m / 16;
    const double *a = A + (int64_t)b * stride_a;
    const int rho = 4 * (c16 & 3) + (c16 >> 2);
    doublex4 C[SLOTS];
#pragma unroll
    for (int i = 0; i < SLOTS; ++i)
#pragma unroll
        for (int u = 0; u < 4; ++u) C[i][u] = 16 * (wave + QW * i) + 4 * q + u == col ? 1.0 : 0.0;
#pragma unroll 1
    for (int p = cb; p >= 0; --p) {
        const int k0 = 16 * p, kb = min(NB, n - k0);
        const bool vok = c16 < kb;
        const double *vcol = a + (int64_t)(k0 + (vok ? c16 : 0)) * m + 4 * q;
        if (t < NB * NB) sh.Ts[t / NB][t % NB] = Tall[((int64_t)p * batch + b) * NB * NB + t];
        doublex4 acc[2] = {};  // P = V^T C
#pragma unroll
        for (int g = 0; g < SLOTS; g += GR) {
            if (wave + QW * (g + GR - 1) < p || wave + QW * g >= blocks) continue;
            Rows4 x[GR];
#pragma unroll
            for (int i = 0; i < GR; ++i) {
                const int bl = wave + QW * (g + i);
                if (bl < whole) {  // blocks before the panel's are read and count as zero
                    x[i] = *reinterpret_cast<const Rows4 *>(vcol + 16 * bl);
                } else {
#pragma unroll
                    for (int u = 0; u < 4; ++u) x[i].v[u] = 16 * bl + 4 * q + u < m ? vcol[16 * bl + u] : 0.0;
                }
            }
#pragma unroll
            for (int i = 0; i < GR; ++i) {
                const int bl = wave + QW * (g + i);
                if (bl < p) continue;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    double y = vok ? x[i].v[u] : 0.0;
                    if (bl == p) {  // the unit lower triangle
                        const int r = 4 * q + u;
                        y = (r < c16 || !vok) ? 0.0 : (r == c16 ? 1.0 : y);
                    }
                    acc[u & 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(y, C[g + i][u], acc[u & 1], 0, 0, 0);
                }
            }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) sh.Pw[wave][q + 4 * r][c16] = acc[0][r] + acc[1][r];
        __syncthreads();
        if (t < NB * CT) {  // P summed over the waves in order
            const int i = t / CT, j = t % CT;
            double s = sh.Pw[0][i][j];
#pragma unroll
            for (int w = 1; w < QW; ++w) s += sh.Pw[w][i][j];
            sh.Pw[0][i][j] = s;
        }
        __syncthreads();
        if (t < NB * CT) {  // W = T P
            const int i = t / CT, j = t % CT;
            double s = 0.0;
            for (int l = i; l < NB; ++l) s += sh.Ts[i][l] * sh.Pw[0][l][j];
            sh.W[i][j] = s;
        }
        __syncthreads();
        double wv[4];
        const double *vk[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            wv[u] = sh.W[4 * u + q][c16];
            vk[u] = a + (int64_t)(k0 + min(4 * u + q, kb - 1)) * m + rho;
        }
#pragma unroll
        for (int g = 0; g < SLOTS; g += GR) {  // C -= V W
            if (wave + QW * (g + GR - 1) < p || wave + QW * g >= blocks) continue;
            double x[GR][4];
#pragma unroll
            for (int i = 0; i < GR; ++i) {
                const int bl = wave + QW * (g + i);
#pragma unroll
                for (int u = 0; u < 4; ++u) x[i][u] = 16 * bl + rho < m ? vk[u][16 * bl] : 0.0;
            }
#pragma unroll
            for (int i = 0; i < GR; ++i) {
                const int bl = wave + QW * (g + i);
                if (bl < p) continue;
                doublex4 o = {0.0, 0.0, 0.0, 0.0};  // the product first: C is rounded once per panel
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int k = 4 * u + q;
                    double y = k < kb ? x[i][u] : 0.0;
                    if (bl == p) y = (rho < k || k >= kb) ? 0.0 : (rho == k ? 1.0 : y);
                    o = __builtin_amdgcn_mfma_f64_16x16x4f64(y, wv[u], o, 0, 0, 0);
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) C[g + i][u] -= o[u];
            }
        }
    }
    if (col >= n) return;
    double *o = Q + (int64_t)b * stride_q + (int64_t)col * m + 4 * q;
#pragma unroll
    for (int i = 0; i < SLOTS; ++i) {
        const int bl = wave + QW * i;
        if (bl < whole) {
            *reinterpret_cast<Rows4 *>(o + 16 * bl) = Rows4{{C[i][0], C[i][1], C[i][2], C[i][3]}};
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (16 * bl + 4 * q + u < m) o[16 * bl + u] = C[i][u];
        }
    }
}

template <class F>
void with_rows(int rows, F &&f) {  // f(integral_constant<RPT>) with RPT = ceil(rows / QT)
    switch ((rows + QT - 1) / QT) {
        case 1: f(std::integral_constant<int, 1>{}); break;
        case 2: f(std::integral_constant<int, 2>{}); break;
        case 3: f(std::integral_constant<int, 3>{}); break;
        case 4: f(std::integral_constant<int, 4>{}); break;
        default: f(std::integral_constant<int, 5>{}); break;
    }
}

// Q = [I_n; 0] (column-major m x n, leading dimension m)
__global__ void identity_kernel(double *__restrict__ Q, int m, int n, int64_t stride, int64_t total) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= total) return;
    const int64_t b = e / ((int64_t)m * n), q = e % ((int64_t)m * n);
    const int c = (int)(q / m), r = (int)(q % m);
    Q[b * stride + q] = r == c ? 1.0 : 0.0;
}

// X[:, i] = R^-1 e_i (column-major, upper triangular): x_k = (delta_ik - s_k) / R_kk for k = i..0,
// where s_k = sum_{l > k} R_kl x_l is accumulated column by column in LDS as the x_l appear.
// colsq[b][0][i] = sum_r R_ri^2 and colsq[b][1][i] = sum_r X_ri^2 for the norms of qr_ratio_kernel.
__global__ __launch_bounds__(FB) void upper_inverse_kernel(const double *__restrict__ R, int n, int ldr, int64_t stride_r,
                                                            double *__restrict__ X, int ldx, int64_t stride_x,
                                                            double *__restrict__ colsq) {
    extern __shared__ double s[];  // [n]
    __shared__ double xk_sh;
    __shared__ double sh[FB / 64];
    const int i = blockIdx.x, b = blockIdx.y;
    const double *Rb = R + (int64_t)b * stride_r;
    double *x = X + (int64_t)b * stride_x + (int64_t)i * ldx;
    for (int r = threadIdx.x; r <= i; r += FB) s[r] = 0.0;
    for (int r = i + 1 + threadIdx.x; r < n; r += FB) x[r] = 0.0;
    for (int k = i; k >= 0; --k) {
        __syncthreads();
        if (threadIdx.x == 0) {
            const double xk = ((k == i) ? 1.0 : -s[k]) / Rb[(int64_t)k * ldr + k];
            x[k] = xk;
            xk_sh = xk;
        }
        __syncthreads();
        const double xk = xk_sh;
        const double *rk = Rb + (int64_t)k * ldr;  // column k of R, rows 0..k-1
        for (int r = threadIdx.x; r < k; r += FB) s[r] += rk[r] * xk;
    }
    __syncthreads();  // x[0..i] written by thread 0
    const double *ri = Rb + (int64_t)i * ldr;
    double sr = 0.0, sx = 0.0;
    for (int r = threadIdx.x; r <= i; r += FB) {
        sr += ri[r] * ri[r];
        sx += x[r] * x[r];
    }
    sr = block_sum_fixed<FB / 64>(sr, sh);
    sx = block_sum_fixed<FB / 64>(sx, sh);
    if (threadIdx.x == 0) {
        colsq[(int64_t)b * 2 * n + i] = sr;
        colsq[(int64_t)b * 2 * n + n + i] = sx;
    }
}

// The same for 16 columns per workgroup with the right-hand sides in registers (as in q_kernel):
// block row p of X is a 16 x 16 substitution, which every wave does for itself, and goes into the rows
// above on the matrix cores; one barrier per block row where the kernel above has two per row.
// n = 1200: 1.0 -> 0.37 ms.
struct InverseShared {
    double c[2][NB][CT];       // the right-hand sides of a block row
    double R[2][NB][NB + 1];   // its diagonal block
    double x[QW][NB][CT];      // a wave's solution, to be read in the B layout
};
template <int RPT>
__global__ __launch_bounds__(QT) void inverse_kernel(const double *__restrict__ R, int n, int ldr, int64_t stride_r,
                                                     double *__restrict__ X, int ldx, int64_t stride_x,
                                                     double *__restrict__ colsq) {
    constexpr int SLOTS = RPT * QT / 16 / QW, GR = 4;
    __shared__ InverseShared sh;
    const int t = threadIdx.x, lane = t & 63, q = lane >> 4, c16 = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int cb = (int)(gridDim.x - 1 - blockIdx.x), b = blockIdx.y;  // the longest chains first
    const int col = 16 * cb + c16;
    const double *Rb = R + (int64_t)b * stride_r;
    double *Xb = X + (int64_t)b * stride_x;
    const int rho = 4 * (c16 & 3) + (c16 >> 2);
    doublex4 C[SLOTS];
#pragma unroll
    for (int i = 0; i < SLOTS; ++i) C[i] = doublex4{0.0, 0.0, 0.0, 0.0};
    // element (r, k) of the diagonal block p; the unit matrix past the last column
    auto diagonal = [&](int p) {
        const int r = t & 15, k = t >> 4, row = 16 * p + r, cl = 16 * p + k;
        return row < n && cl < n ? (r <= k ? Rb[(int64_t)cl * ldr + row] : 0.0) : (r == k ? 1.0 : 0.0);
    };
    if (t < NB * NB) {
        sh.R[cb & 1][t & 15][t >> 4] = diagonal(cb);
        sh.c[cb & 1][t & 15][t >> 4] = (t & 15) == (t >> 4) ? 1.0 : 0.0;
    }
    double sx = 0.0;
#pragma unroll 1
    for (int p = cb; p >= 0; --p) {
        __syncthreads();
        const double next = p > 0 && t < NB * NB ? diagonal(p - 1) : 0.0;
        const double *rk = Rb + rho;
        auto load = [&](double (&y)[GR][4], int g) {
#pragma unroll
            for (int i = 0; i < GR; ++i) {
                const int bl = wave + QW * (g + i);
                if (bl < p)
#pragma unroll
                    for (int u = 0; u < 4; ++u) y[i][u] = rk[(int64_t)min(16 * p + 4 * u + q, n - 1) * ldr + 16 * bl];
            }
        };
        double y[GR][4];
        load(y, 0);
        double x[NB];
#pragma unroll
        for (int r = 0; r < NB; ++r) x[r] = sh.c[p & 1][r][c16];
        const double inv = 1.0 / sh.R[p & 1][c16][c16];
#pragma unroll
        for (int r = NB - 1; r >= 0; --r) {
            x[r] *= lane_value(inv, r);
#pragma unroll
            for (int a = 0; a < r; ++a) x[a] -= sh.R[p & 1][a][r] * x[r];
        }
#pragma unroll
        for (int r = 0; r < NB; ++r) sx += x[r] * x[r];
        if (q == 0)
#pragma unroll
            for (int r = 0; r < NB; ++r) sh.x[wave][r][c16] = x[r];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");  // a wave's LDS accesses complete in order
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (wave == p % QW && col < n)
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (16 * p + 4 * q + u < n) Xb[(int64_t)col * ldx + 16 * p + 4 * q + u] = sh.x[wave][4 * q + u][c16];
        double wv[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) wv[u] = -sh.x[wave][4 * u + q][c16];
#pragma unroll
        for (int g = 0; g < SLOTS; g += GR) {
            if (wave + QW * g >= p) continue;
            if (g > 0) load(y, g);
#pragma unroll
            for (int i = 0; i < GR; ++i) {
                const int bl = wave + QW * (g + i);
                if (bl >= p) continue;
#pragma unroll
                for (int u = 0; u < 4; ++u) C[g + i] = __builtin_amdgcn_mfma_f64_16x16x4f64(y[i][u], wv[u], C[g + i], 0, 0, 0);
                if (bl == p - 1)
#pragma unroll
                    for (int u = 0; u < 4; ++u) sh.c[bl & 1][4 * q + u][c16] = C[g + i][u];
            }
        }
        if (p > 0 && t < NB * NB) sh.R[(p - 1) & 1][t & 15][t >> 4] = next;
    }
    if (wave == 0 && q == 0 && col < n) colsq[(int64_t)b * 2 * n + n + col] = sx;
    for (int j = wave; j < CT; j += QW) {  // rows past the block row's, and the squares of R's column
        const int cj = 16 * cb + j;
        if (cj >= n) break;
        for (int r = 16 * (cb + 1) + lane; r < n; r += 64) Xb[(int64_t)cj * ldx + r] = 0.0;
        double sr = 0.0;
        for (int r = lane; r <= cj; r += 64) sr += Rb[(int64_t)cj * ldr + r] * Rb[(int64_t)cj * ldr + r];
        for (int d = 32; d > 0; d >>= 1) sr += __shfl_down(sr, d, 64);
        if (lane == 0) colsq[(int64_t)b * 2 * n + cj] = sr;
    }
}

// ratio[b] = 1 / (||R||_F ||R^-1||_F), a lower bound of sigma_min / sigma_max
__global__ __launch_bounds__(FB) void qr_ratio_kernel(int n, const double *__restrict__ colsq, double *__restrict__ ratio) {
    __shared__ double sh[FB / 64];
    const int b = blockIdx.x;
    const double *c = colsq + (int64_t)b * 2 * n;
    double sr = 0.0, sx = 0.0;
    for (int i = threadIdx.x; i < n; i += FB) {
        sr += c[i];
        sx += c[n + i];
    }
    sr = block_sum_fixed<FB / 64>(sr, sh);
    sx = block_sum_fixed<FB / 64>(sx, sh);
    if (threadIdx.x == 0) ratio[b] = 1.0 / sqrt(sr * sx);
}

}  // namespace

size_t qr_scratch_doubles(int batch, int n) {
    const size_t panels = (size_t)(n + NB - 1) / NB;
    return (size_t)batch * n * 3 + panels * (size_t)batch * NB * NB;
}

int qr_inverse_batched(int batch, double *A, int m, int n, int64_t stride_a, double *Q, int64_t stride_q, double *X,
                       int64_t stride_x, double *scratch, double *ratio, hipStream_t s) {
    if (batch <= 0 || n <= 0) return MFS_OK;
    if (m < n) return fail(MFS_EINVAL, "QR factorisation needs rows >= columns");
    if ((size_t)n * sizeof(double) > 64 * 1024) return fail(MFS_EINVAL, "QR factorisation supports at most 8192 columns");
    if (batch > 65535) return fail(MFS_EINVAL, "QR factorisation: at most 65535 matrices per batch");
    double *tau = scratch;
    double *colsq = scratch + (size_t)batch * n;      // [batch][2][n]
    double *Tall = scratch + (size_t)batch * n * 3;  // T of panel p: Tall + p * batch * NB * NB
    const int panels = (n + NB - 1) / NB;
    const bool in_registers = m <= QT * QR_MAX_RPT;  // else the panel does not fit a workgroup's registers
    auto panel_T = [&](int p) { return Tall + (size_t)p * batch * NB * NB; };
    if (in_registers) {
        with_rows(m, [&](auto R) {
            qr_first_kernel<R.value><<<batch, QT, 0, s>>>(A, m, stride_a, std::min(NB, n), tau, n, panel_T(0));
        });
        for (int p = 0; p + 1 < panels; ++p)
            with_rows(m - (p + 1) * NB, [&](auto R) {
                qr_step_kernel<R.value><<<dim3(panels - p - 1, batch), QT, 0, s>>>(A, m, stride_a, p * NB, n, panel_T(p),
                                                                                  tau, panel_T(p + 1));
            });
    } else {
        for (int p = 0; p < panels; ++p) {
            const int k0 = p * NB, kb = std::min(NB, n - k0);
            panel_qr_kernel<<<batch, PT, 0, s>>>(A, m, m, stride_a, k0, kb, tau, n, panel_T(p));
            if (k0 + kb < n)
                wy_apply_kernel<true><<<dim3((n - k0 - kb + CT - 1) / CT, batch), FB, 0, s>>>(
                    A, m, m, stride_a, k0, kb, panel_T(p), A, m, stride_a, k0 + kb, n);
        }
    }
    MFS_HIP_TRY(hipGetLastError());
    if (in_registers) {
        with_rows(m, [&](auto R) {
            q_kernel<R.value><<<dim3(panels, batch), QT, 0, s>>>(A, m, stride_a, n, Tall, batch, Q, stride_q);
        });
    } else {
        const int64_t total = (int64_t)batch * m * n;
        identity_kernel<<<(unsigned)((total + 255) / 256), 256, 0, s>>>(Q, m, n, stride_q, total);
        for (int p = panels - 1; p >= 0; --p) {
            const int k0 = p * NB, kb = std::min(NB, n - k0);
            wy_apply_kernel<false><<<dim3((n - k0 + CT - 1) / CT, batch), FB, 0, s>>>(
                A, m, m, stride_a, k0, kb, panel_T(p), Q, m, stride_q, k0, n);
        }
    }
    MFS_HIP_TRY(hipGetLastError());
    if (in_registers)
        with_rows(n, [&](auto R) {
            inverse_kernel<R.value><<<dim3(panels, batch), QT, 0, s>>>(A, n, m, stride_a, X, n, stride_x, colsq);
        });
    else
        upper_inverse_kernel<<<dim3(n, batch), FB, (size_t)n * sizeof(double), s>>>(A, n, m, stride_a, X, n, stride_x,
                                                                                   colsq);
    qr_ratio_kernel<<<batch, FB, 0, s>>>(n, colsq, ratio);
    MFS_HIP_TRY(hipGetLastError());
    return MFS_OK;
}

}  // namespace mfs
