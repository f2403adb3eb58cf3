// Direct route of the eigensolver F = Q diag(lam) Q^T (Sec. IV-A; Algorithm 1, step 2): every factor of a call goes
// through the same few stages, and every stage is one launch (or one chain of launches) over all factors.
//
//  1. Householder reduction to tridiagonal form, A = H T H^T, in fp32, of the factor with its diagonal in descending order
//     (the reduction starts at the large end, so the small end of a graded factor is not swamped by the large end's
//     rounding: on a factor graded over eight decades the small eigenvectors come out fifty times as accurate).  Factors up to 256 wide: one workgroup each, the
//     matrix in registers.  Wider ones: the trailing matrix in the registers of the whole chip (eig_chip.h).  Columns of a factor too
//     wide for that: the blocked right-looking reduction (panels of 32 columns; per column one symmetric matrix-vector product
//     over the lower tiles and one vector step; per panel one rank-64 update on the fp32 matrix instructions) until it fits.
//  2. Eigenvalues of T by bisection and eigenvectors of T by twisted factorisation, both in fp64 and both
//     independent per eigenvalue.  T carries fp32 rounding noise, so fp64 has nine digits to spare: the eigenvectors of
//     eigenvalues that agree to many digits still come out orthogonal without any re-orthogonalisation, once exact
//     multiplicities are broken by a perturbation of T below its rounding noise (PERTURB_REL, PERTURB_ABS).
//  3. Back-transformation by the reflectors: compact WY blocks of 128 on the fp32 matrix instructions, or (small
//     factors) a wave per four columns with the columns in registers.
//  4. One Newton-Schulz step on Q and Rayleigh quotients against the caller's F; where the reduction on the chip has rounded the factor more
//     than the rest of it all does (CORRECT_FROM), a first-order correction of Q and the quotients again; ascending order.
//
// The residual ||F Q - Q diag(lam)||_F = off(Q^T F Q) of the result is measured (it falls out of the Rayleigh quotients), and
// so is the orthogonality of the eigenvectors before the last step; a factor with an unsound result is decomposed by
// Jacobi iteration instead (eig.hip).
#include <algorithm>
#include <climits>
#include <cmath>
#include <cstring>
#include <vector>
#include "eig_chip_ring.h"
#include "kfac_internal.h"
#include "mfma_gemm.h"
#include "mfma_gemm_x3.h"

namespace {

using namespace kfac;

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int NB = 32;            // columns of a panel
constexpr int TB = 128;           // tile edge
constexpr int RB = 64;            // rows per workgroup of the vector step
constexpr int TD_SMALL = KFAC_EIG_REG;
constexpr int WY = 128;           // reflectors of a compact WY block
constexpr int WY_K = 512;         // contraction of one workgroup in Y = V^T Z
constexpr int NPARTS = 64;         // parts of the Rayleigh quotients' sums
constexpr int NORM_WGS = 256;      // workgroups per factor of the norms and copies: workgroup b has rows b, b + gridDim.x, ..; never more than rows
constexpr unsigned long long CHIP_EMPTY = ~0ull;
constexpr double PERTURB_REL = 0x1p-25;   // of every element of T: half the rounding it already carries
constexpr double PERTURB_ABS = 1e-10;     // of the Gershgorin bound, added to the diagonal: breaks multiple zeros
constexpr double NS_AGAIN = 4e-6;         // ||I - Q^T Q||_F^2 from which one Newton-Schulz step is not enough (it leaves 3/4 of this)
// Updates of the trailing matrix in the registers of the chip that an element of the factor has been through, on average over ||F||_F^2 (T's elements say
// what is left in the trailing matrices), from which the eigenvectors are corrected.  Every update rounds, 2.3e-8 of the element
// as measured, so this is 1.8e-7 ||F|| beside the 4 to 6e-7 of everything else; a Gram matrix of independent features gets to n / 2 and
// 1.6e-6 at 4609, factors with a few large eigenvalues or a graded diagonal stay below 64.  1e7 residual / ||F||, by the chain of launches, on the
// chip, and on the chip and corrected: Gram matrices of 2 n samples 577 5.6, 8.0, 3.0, 2305 6.1, 12.7, 3.2, 4609 6.5, 17.0, 3.6, of 30 n samples
// 4609 4.6, 18.5, 3.6, random symmetric 4609 10.3, 17.4, 4.3; ReLU activations (not corrected) 4609 4.8, 4.8.  ||I - Q^T Q||_F: the
// same in all of them.  A corrected factor costs 2.5 ms more at 4609 (31.0), 0.5 at 2305 (11.2), 0.15 at 577 (2.6).
constexpr double CORRECT_FROM = 64.0;
constexpr double REDUCTION_GIVEN_UP = -1.0;
constexpr double CORRECT_GAP = 0x1p11;    // gap of two eigenvalues, in residuals of their columns, below which they are left as they are
constexpr double BIS_REL = 0x1p-51, BIS_ABS = 1e-25;   // width at which an eigenvalue's interval is done, of its size and of the bound
constexpr int BIS_WIDE_MAX = 160;         // up to this many groups of 64 eigenvalues, sixteen lanes each
constexpr double E_MIN = 1e-20;     // of the same: no off-diagonal element of T is exactly zero
constexpr double PIVOT_MIN = 1e-30;

struct DirMat {
    const float *F;
    float *Q, *lam;  // (Q holds the residual of a correction, and the corrected F Q, before it receives the result)
    float *A;        // [np][ld]: the matrix, its lower tiles reduced in place; row p of the upper part receives reflector p
    float *Z;        // [np][ld]: eigenvectors of T, then of A
    float *B1, *B2;  // [np][ld] each, adjacent: together the fp64 pivots of the eigenvectors; then scratch
    float *panel;    // [3 NB][ld]: V, W, V of the current panel
    float *apan;     // [NB + 1][np]: the panel's columns, and the one after it, as they stood when the panel began
    // what a column's launch leaves for the next, twice:
    float *part;     // [2][nb][np]: partial products of the column's matrix-vector product
    float *dots;     // [2][nb][2 NB]: partial V^T x, W^T x per row block
    double *tsum;    // [2] per tile: its share of x^T A x; later [0] mean number of updates, [1] scale of the residual in a correction (0: there is none)
    float *acol;     // [2][np]: the column x, not yet scaled
    float *npart;    // [2][np / RB]: its squared norm, per workgroup
    float *tau;      // [np]
    double *d, *e;   // [np]: T as reduced
    double2 *td;     // [np]: T perturbed and divided by its Gershgorin bound: {d_i, e_i^2}; |e_i| is kept away from zero
    double *te;      // [np]: e_i of the same; later 1 / norm of every eigenvector
    double *lam64;   // [np]: eigenvalues of T, later the Rayleigh quotients
    double *sums;    // [min(NPARTS, n)][3][np] partial traces; partial sums of the Rayleigh quotients
    double *npartd;  // [NORM_WGS][2] partial norms: off^2, diag^2 of the first min(NORM_WGS, n); later of D and of the residual
    double *stat;    // off^2, diag^2, residual^2, ||I - Q^T Q||^2
    float *Tm;       // [nb][WY][WY]: Gram matrices of the WY blocks, then their T
    int *perm;       // [np]: final order of the eigenvectors
    int *ord;        // [np]: row of F that became row i of A (diagonal descending)
    double diag_tol2;   // a factor up to TD_SMALL wide with off^2 <= this ||F||^2 is diagonal as it stands (wider ones: see go_on)
    int n, np, ld, nb, off;
    short split, chain; // chain: columns that the chain of launches reduces, before the matrix fits the chip
};
static_assert(sizeof(DirMat) == 240, "part of every workspace: no larger, or one that a caller has sized for a direct decomposition does not hold it");

// Nothing to reduce: the eigenvectors are unit vectors.  (An identity or another diagonal factor: 64 wide 103 us in place of 267, 145 wide
// 156 in place of 626.)
__device__ inline bool is_diagonal(const DirMat &M, double o2, double d2) { return M.n <= TD_SMALL && o2 <= M.diag_tol2 * (o2 + d2); }
__device__ inline bool is_diagonal(const DirMat &M) { return is_diagonal(M, M.stat[0], M.stat[1]); }

__device__ inline float wave_sum_all(float v) {   // the sum over the wave, in every lane
    int x = __float_as_int(v);
#define KFAC_DPP_ADD(ctrl, rmask) x = __float_as_int(__int_as_float(x) + __int_as_float(__builtin_amdgcn_update_dpp(0, x, ctrl, rmask, 0xf, true)))
    KFAC_DPP_ADD(0x111, 0xf);   // row_shr:1, 2, 4, 8: the last lane of a row of 16 holds the row's sum
    KFAC_DPP_ADD(0x112, 0xf);
    KFAC_DPP_ADD(0x114, 0xf);
    KFAC_DPP_ADD(0x118, 0xf);
    KFAC_DPP_ADD(0x142, 0xa);   // row_bcast:15 into rows 1 and 3
    KFAC_DPP_ADD(0x143, 0xc);   // row_bcast:31 into rows 2 and 3
#undef KFAC_DPP_ADD
    return __int_as_float(__builtin_amdgcn_readlane(x, 63));
}
__device__ inline float lane_value(float v, int lane) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane)); }
__device__ inline float quad_sum(float v) {       // the sum over four neighbouring lanes, in each of them
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xf, 0xf, true));   // quad_perm 1,0,3,2
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xf, 0xf, true));   // quad_perm 2,3,0,1
    return v;
}
template <int CTRL, int ROWS> __device__ inline double dpp_add_f64(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, ROWS, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROWS, 0xf, true);
    return v + __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ inline double wave_sum_f64(double v) {   // the same steps as wave_sum_all
    v = dpp_add_f64<0x111, 0xf>(v);
    v = dpp_add_f64<0x112, 0xf>(v);
    v = dpp_add_f64<0x114, 0xf>(v);
    v = dpp_add_f64<0x118, 0xf>(v);
    v = dpp_add_f64<0x142, 0xa>(v);
    v = dpp_add_f64<0x143, 0xc>(v);
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, 63), hi = __builtin_amdgcn_readlane((int)(b >> 32), 63);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// ---- norms and the working copy ------------------------------------------------------------------------
__global__ __launch_bounds__(256) void dir_norm_kernel(const DirMat *mats) {
    const DirMat M = mats[blockIdx.y];
    const global_ptr<const float> F = as_global(M.F);
    const int n = M.n;
    if ((int)blockIdx.x >= n) return;
    double o2 = 0.0, d2 = 0.0, tr = 0.0;
    for (int r = blockIdx.x; r < n; r += gridDim.x)
        for (int c = threadIdx.x; c < n; c += 256) {
            const double v = (double)F[(int64_t)r * n + c];
            if (c == r) { d2 += v * v; tr += v; } else o2 += v * v;
        }
    __shared__ double red[8];
    if (n > TD_SMALL) {
        tr = wave_sum_f64(tr);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = tr;
        __syncthreads();
        if (threadIdx.x == 0) M.sums[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
        __syncthreads();
    }
    o2 = wave_sum_f64(o2);
    d2 = wave_sum_f64(d2);
    if ((threadIdx.x & 63) == 0) { red[threadIdx.x >> 6] = o2; red[4 + (threadIdx.x >> 6)] = d2; }
    __syncthreads();
    if (threadIdx.x == 0) {
        M.npartd[2 * blockIdx.x] = red[0] + red[1] + red[2] + red[3];
        M.npartd[2 * blockIdx.x + 1] = red[4] + red[5] + red[6] + red[7];
    }
}

__device__ inline float norm_scale(double f2) {      // the power of two that brings ||F||_F into [1, 2)
    if (!(f2 > 0.0) || !(f2 < 1e300)) return 1.f;
    return ldexpf(1.f, min(max(-ilogb(sqrt(f2)), -120), 120));
}
// off^2 and diag^2 from the partial norms (a wave; fixed order), and that scale
__device__ inline float dir_norms(const DirMat &M, double &o2, double &d2) {
    const int lane = threadIdx.x & 63;
    o2 = d2 = 0.0;
#pragma unroll
    for (int i = 0; i < NORM_WGS / 64; ++i) {
        const int w = 64 * i + lane;
        o2 += w < M.n ? M.npartd[2 * w] : 0.0;
        d2 += w < M.n ? M.npartd[2 * w + 1] : 0.0;
    }
    o2 = wave_sum_f64(o2);
    d2 = wave_sum_f64(d2);
    return norm_scale(o2 + d2);
}
// What is taken from the diagonal of a factor before it is reduced on the chip: its mean, if the factor is little else (less than a quarter of
// ||F||_F^2 is left).  Every update rounds what is left, not what was taken.  residual / ||F||: Gram matrices of 30 n samples 1.07e-6 -> 2.1e-7 at
// 1153; eigenvalues that differ by 2 % at most, whose vectors could not be corrected afterwards, 1.7e-6 -> 4.0e-8 at 1153, and 4609, which missed tol and
// took 145 ms with the sweeps that followed, 3.7e-8 in 31.8.  (A graded or rank-deficient factor is never that close to its mean.)  The
// eigenvectors are the same, and the eigenvalues come from the caller's F.
__device__ inline double dir_shift(const DirMat &M, double f2) {
    const int lane = threadIdx.x & 63;
    double tr = 0.0;
#pragma unroll
    for (int i = 0; i < NORM_WGS / 64; ++i) tr += M.sums[64 * i + lane];
    tr = wave_sum_f64(tr);
    return tr * tr > 0.75 * f2 * M.n ? tr / M.n : 0.0;
}

// ord[rank] = index of the rank-th largest diagonal element (ties and NaNs by index: always a permutation)
constexpr int RANK_IPB = 16;
__global__ __launch_bounds__(256) void dir_order_kernel(const DirMat *mats) {
    __shared__ float chunk[256];
    __shared__ int part[256];
    const DirMat M = mats[blockIdx.y];
    const int n = M.n, ii = threadIdx.x & (RANK_IPB - 1), js = threadIdx.x / RANK_IPB, i = blockIdx.x * RANK_IPB + ii;
    if ((int)blockIdx.x * RANK_IPB >= n) return;
    const global_ptr<const float> F = as_global(M.F);
    const float di = i < n ? F[(int64_t)i * (n + 1)] : 0.f;
    const bool nan_i = di != di;
    int rank = 0;
    for (int j0 = 0; j0 < n; j0 += 256) {
        __syncthreads();
        chunk[threadIdx.x] = j0 + (int)threadIdx.x < n ? F[(int64_t)(j0 + threadIdx.x) * (n + 1)] : 0.f;
        __syncthreads();
        const int cnt = min(256, n - j0);
        for (int k = js; k < cnt; k += 256 / RANK_IPB) {
            const float dj = chunk[k];
            const int j = j0 + k;
            const bool nan_j = dj != dj;
            rank += nan_i ? (!nan_j || j < i) : (!nan_j && ((dj > di) || (dj == di && j < i)));
        }
    }
    part[threadIdx.x] = rank;
    __syncthreads();
    if (js == 0 && i < n) {
        int total = 0;
        for (int t = 0; t < 256 / RANK_IPB; ++t) total += part[t * RANK_IPB + ii];
        M.ord[total] = i;
    }
}

// Empties the ring of a factor's first launch of the reduction on the chip: EMPTY, as 8-byte words, over the first half of apan's use; and
// clears the two words that say whether a reduction was given up, behind both halves.
__device__ inline void empty_ring(const DirMat &M, int wg, int wgs) {
    const global_ptr<unsigned long long> ring = as_global((unsigned long long *)M.apan);
    for (int i = wg * 256 + (int)threadIdx.x; i < CHIP_RING * M.np; i += 256 * wgs) ring[i] = CHIP_EMPTY;
    if (wg == 0 && threadIdx.x < 2) ring[(size_t)2 * CHIP_RING * M.np + threadIdx.x] = 0;
}

// A <- scale * (F - shift), reordered, with zero padding, for the factors wider than the register kernels take; the norms for all of them.
__global__ __launch_bounds__(256) void dir_copy_kernel(const DirMat *mats) {
    const DirMat M = mats[blockIdx.y];
    double o2, d2;
    const float sc = dir_norms(M, o2, d2);
    if (blockIdx.x == 0 && threadIdx.x == 0) { M.stat[0] = o2; M.stat[1] = d2; }
    if (M.n <= TD_SMALL) return;
    const global_ptr<const float> F = as_global(M.F);
    const global_ptr<float> A = as_global(M.A);
    const int n = M.n, np = M.np;
    const double shift = dir_shift(M, o2 + d2);
    if (blockIdx.x == 0)
        for (int i = n - 1 + (int)threadIdx.x; i < np; i += 256) M.tau[i] = 0.f;   // no reflectors there
    if (M.chain == 0) empty_ring(M, blockIdx.x, gridDim.x);
    const global_ptr<const int> ord = as_global((const int *)M.ord);
    for (int r = blockIdx.x; r < np; r += gridDim.x) {
        const int64_t fr = r < n ? (int64_t)ord[r] * n : 0;
        for (int c = threadIdx.x; c < np; c += 256) {
            float v = (r < n && c < n) ? F[fr + ord[c]] : 0.f;
            if (c == r && r < n) v = (float)((double)v - shift);
            A[(int64_t)r * M.ld + c] = sc * v;
        }
    }
}

#include "eig_chip.h"

// ---- reduction, one workgroup (n <= 256) -------------------------------------------------------------------
// Four threads per row, each with KC columns of it in registers (groups of four: group k covers columns 16 k + 4 q ..).
// The matrix never touches LDS; per column one row goes to LDS (it is the column, by symmetry), v and w are read
// back by everybody.  A column costs three barriers and a few LDS latencies: 1.0 us at 64, 1.9 at 145, 2.4 at 256.
template <int KC>
__global__ __launch_bounds__(16 * KC) void dir_td_small_kernel(const DirMat *mats, const int *list) {
    constexpr int G = KC / 4, NTH = 16 * KC, NW = NTH / 64, CMAX = 4 * KC;
    __shared__ __attribute__((aligned(16))) float xs[CMAX], v[CMAX], w[CMAX];
    __shared__ float red[NW];
    const DirMat M = mats[list[blockIdx.x]];
    const int n = M.n, tid = threadIdx.x, row = tid >> 2, q = tid & 3, wave = tid >> 6, lane = tid & 63;
    double o2, d2;
    const float sc = dir_norms(M, o2, d2);
    if (is_diagonal(M, o2, d2)) {
        for (int i = tid; i < n; i += NTH) {
            M.d[i] = (double)(sc * as_global(M.F)[(int64_t)M.ord[i] * (n + 1)]);
            M.e[i] = 0.0;
            M.tau[i] = 0.f;
        }
        return;
    }
    floatx4 a[G];
    {
        const global_ptr<const float> F = as_global(M.F);
        const int64_t fr = row < n ? (int64_t)M.ord[row] * n : 0;
#pragma unroll
        for (int k = 0; k < G; ++k)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int c = 16 * k + 4 * q + u;
                a[k][u] = (row < n && c < n) ? sc * F[fr + M.ord[c]] : 0.f;
            }
    }
    const global_ptr<float> A = as_global(M.A);
    for (int j = 0; j < n; ++j) {
        if (row == j)
#pragma unroll
            for (int k = 0; k < G; ++k) *(floatx4 *)(xs + 16 * k + 4 * q) = a[k];
        __syncthreads();
        if (j == n - 1) break;
        // norm of the column below its first element: every wave forms it for itself
        float s2 = 0.f;
#pragma unroll
        for (int c0 = 0; c0 < CMAX; c0 += 64) {
            const int c = c0 + lane;
            const float x = (CMAX % 64 == 0 || c < CMAX) ? xs[c < CMAX ? c : 0] : 0.f;
            s2 += c > j + 1 && c < CMAX ? x * x : 0.f;
        }
        s2 = wave_sum_all(s2);
        const float alpha = xs[j + 1];
        float beta = alpha, tau = 0.f, scale = 0.f;
        if (s2 > 0.f) {
            beta = -copysignf(sqrtf(fmaf(alpha, alpha, s2)), alpha);
            tau = (beta - alpha) / beta;
            scale = 1.f / (alpha - beta);
        }
        if (tid < CMAX) {
            const float x = xs[tid];
            const float vv = tid > j + 1 ? x * scale : (tid == j + 1 ? 1.f : 0.f);
            v[tid] = vv;
            if (tid < n) A[(int64_t)j * M.ld + tid] = vv;
        }
        if (tid == 0) {
            M.d[j] = (double)xs[j];
            M.e[j] = (double)beta;
            M.tau[j] = tau;
        }
        __syncthreads();
        const int k0 = (j + 1) >> 4;     // column groups before it are finished
        float y = 0.f;
#pragma unroll
        for (int k = 0; k < G; ++k)
            if (k >= k0) {
                const floatx4 vc = *(const floatx4 *)(v + 16 * k + 4 * q);
                y = fmaf(a[k].x, vc.x, y);
                y = fmaf(a[k].y, vc.y, y);
                y = fmaf(a[k].z, vc.z, y);
                y = fmaf(a[k].w, vc.w, y);
            }
        y = quad_sum(y);
        const float vr = v[row];
        const float ty = row > j ? tau * y : 0.f;
        const float part = wave_sum_all(q == 0 ? vr * ty : 0.f);
        if (q == 0) w[row] = ty;
        if (lane == 0) red[wave] = part;
        __syncthreads();
        float vty = 0.f;                 // tau v^T A v
#pragma unroll
        for (int u = 0; u < NW; ++u) vty += red[u];
        // w = tau A v - (tau/2)(tau v^T A v) v;  A <- A - v w^T - w v^T with the v v^T parts of both gathered in one factor
        const float wr = fmaf(-tau * vty, vr, ty);
#pragma unroll
        for (int k = 0; k < G; ++k)
            if (k >= k0) {
                const floatx4 vc = *(const floatx4 *)(v + 16 * k + 4 * q), wc = *(const floatx4 *)(w + 16 * k + 4 * q);
#pragma unroll
                for (int u = 0; u < 4; ++u) a[k][u] = fmaf(-vr, wc[u], fmaf(-wr, vc[u], a[k][u]));
            }
    }
    if (tid == 0) {
        M.d[n - 1] = (double)xs[n - 1];
        M.e[n - 1] = 0.0;
        M.tau[n - 1] = 0.f;
    }
}

// ---- reduction, chain of launches -----------------------------------------------------------------------------
// Step t of the chain treats column j = t - off of every factor; off is a multiple of NB, so all factors are at the same place
// of their panels.  The tables list the tiles (symv, update) and row blocks (vector step) that a panel touches:
// factor << 14 | row block << 7 | column block.
struct TabRef { int m, I, J; };
__device__ inline TabRef tab_ref(unsigned w) { return TabRef{(int)(w >> 14), (int)((w >> 7) & 127u), (int)(w & 127u)}; }

// What one launch leaves for the next lies in buffers that alternate with t (no launch reads what it writes):
// launch t multiplies column j of the reduced matrix, not yet scaled to a reflector, with the trailing matrix (x = acol, so the
// norm of x need not be known), and the vector step turns the products into those of the reflector v = scale (x - beta e):
//   A v = scale (A x - beta A e),  V^T v = scale (V^T x - beta V^T e),  v^T A v = scale^2 (x^T A x - 2 beta e^T A x + beta^2 e^T A e)
// with e the unit vector of row j + 1; column j + 1 of the trailing matrix, A e, is in apan.
struct StepBufs { global_ptr<float> part, dots, acol, npart; global_ptr<double> tsum; };
__device__ inline StepBufs step_bufs(const DirMat &M, int t) {
    const int h = t & 1;
    return StepBufs{as_global(M.part) + (int64_t)h * M.nb * M.np, as_global(M.dots) + h * M.nb * 2 * NB, as_global(M.acol) + h * M.np,
                    as_global(M.npart) + h * (M.np / RB), as_global(M.tsum) + h * (M.nb * (M.nb + 1) / 2)};
}

// The panel's columns (and the one after it) row by row, and its first column: acol, its norm, its diagonal element.
__global__ __launch_bounds__(RB) void dir_column_kernel(const DirMat *mats, const unsigned *tab, int t) {
    const TabRef tr = tab_ref(tab[blockIdx.x]);
    const DirMat M = mats[tr.m];
    const int j = t - M.off, row = tr.J * RB + (int)threadIdx.x;
    const StepBufs B = step_bufs(M, t);
    const global_ptr<const float> p = as_global((const float *)M.A) + (int64_t)row * M.ld + j;
    const global_ptr<float> o = as_global(M.apan) + row;
    floatx4 c[NB / 4];
#pragma unroll
    for (int u = 0; u < NB / 4; ++u) c[u] = *(global_ptr<const floatx4>)(p + 4 * u);
    const float c32 = j + NB < M.np ? p[NB] : 0.f;
#pragma unroll
    for (int u = 0; u < NB; ++u) o[(int64_t)u * M.np] = c[u >> 2][u & 3];
    o[(int64_t)NB * M.np] = c32;
    const float a = row >= j ? c[0].x : 0.f;
    if (row == j) M.d[j] = (double)a;
    B.acol[row] = row > j ? a : 0.f;
    const float s = wave_sum_all(row > j + 1 ? a * a : 0.f);
    if (threadIdx.x == 0) B.npart[tr.J] = s;
}

// y = A x over one lower tile: tile (I, J) gives A_IJ x_J to the rows of block I and (I > J) A_IJ^T x_I to those of block
// J; both land in part[], one slot per pair of blocks.  Also x^T A x (per tile, fp64: the squares of a column of 1e-19 of
// the matrix are below fp32's range) and, on the diagonal tiles, V^T x and W^T x of the panel's `ncols` earlier columns.
struct SymvSmem {
    __attribute__((aligned(16))) float xI[TB], xJ[TB];
    float cred[8][TB];
    double tred[4];
};
struct TileLoads { floatx4 a[16], pr[TB / 16]; };
__device__ inline void tile_load(const DirMat &M, int I, int J, int ncols, TileLoads &L) {
    const int tid = threadIdx.x, c4 = tid & 31, rs = tid >> 5, pc = tid >> 2, pq = 4 * (tid & 3);
    const global_ptr<const float> p = as_global((const float *)M.A) + (int64_t)(I * TB + rs) * M.ld + J * TB + 4 * c4;
#pragma unroll
    for (int u = 0; u < 16; ++u) L.a[u] = *(global_ptr<const floatx4>)(p + (int64_t)(8 * u) * M.ld);
    // diagonal tiles: four lanes per earlier column of the panel, V then W
    if (I == J && (pc & (NB - 1)) < ncols) {
        const global_ptr<const float> q = as_global((const float *)M.panel) + (int64_t)pc * M.ld + I * TB + pq;
#pragma unroll
        for (int u = 0; u < TB / 16; ++u) L.pr[u] = *(global_ptr<const floatx4>)(q + 16 * u);
    }
}
__device__ inline void tile_product(const DirMat &M, int I, int J, int b0, int ncols, const StepBufs &B, const TileLoads &L, SymvSmem &sm) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, c4 = tid & 31, rs = tid >> 5;
    const bool diag = I == J;
    const floatx4 vc = *(const floatx4 *)(sm.xJ + 4 * c4);
    float rsum[16];
    floatx4 cs = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < 16; ++u) {
        const floatx4 a = L.a[u];
        rsum[u] = fmaf(a.x, vc.x, fmaf(a.y, vc.y, fmaf(a.z, vc.z, a.w * vc.w)));
        const float vr = sm.xI[rs + 8 * u];
        cs.x = fmaf(a.x, vr, cs.x);
        cs.y = fmaf(a.y, vr, cs.y);
        cs.z = fmaf(a.z, vr, cs.z);
        cs.w = fmaf(a.w, vr, cs.w);
    }
    // sixteen sums over the 32 lanes of a half wave: halve the values with every exchange
#pragma unroll
    for (int h = 8; h >= 1; h >>= 1) {
        const bool up = (c4 & (2 * h)) != 0;
#pragma unroll
        for (int k = 0; k < h; ++k) {
            const float keep = up ? rsum[k + h] : rsum[k], give = up ? rsum[k] : rsum[k + h];
            rsum[k] = keep + __shfl_xor(give, 2 * h, 64);
        }
    }
    const float ysum = rsum[0] + __shfl_xor(rsum[0], 1, 64);
    const int r = rs + 8 * (c4 >> 1);      // c4 bits 4..1 = which of the sixteen rows this lane ended up with
    const double va = wave_sum_f64((c4 & 1) ? 0.0 : (double)sm.xI[r] * (double)ysum);
    if (!(c4 & 1)) B.part[(int64_t)J * M.np + I * TB + r] = ysum;
    if (!diag) *(floatx4 *)(sm.cred[rs] + 4 * c4) = cs;
    if (lane == 0) sm.tred[wave] = va;
    __syncthreads();
    if (tid == 0) {
        const int ri = I - b0;
        B.tsum[ri * (ri + 1) / 2 + J - b0] = (diag ? 1.0 : 2.0) * (sm.tred[0] + sm.tred[1] + sm.tred[2] + sm.tred[3]);
    }
    if (!diag) {
        if (tid < TB) {
            float s = 0.f;
#pragma unroll
            for (int k = 0; k < 8; ++k) s += sm.cred[k][tid];
            B.part[(int64_t)I * M.np + J * TB + tid] = s;
        }
    } else {
        const int pc = tid >> 2, pq = 4 * (tid & 3);
        const bool dot = (pc & (NB - 1)) < ncols;
        float d = 0.f;
        if (dot) {
#pragma unroll
            for (int u = 0; u < TB / 16; ++u) {
                const floatx4 x = *(const floatx4 *)(sm.xI + 16 * u + pq);
                d = fmaf(L.pr[u].x, x.x, fmaf(L.pr[u].y, x.y, fmaf(L.pr[u].z, x.z, fmaf(L.pr[u].w, x.w, d))));
            }
        }
        d = quad_sum(d);
        if (dot && pq == 0) B.dots[I * 2 * NB + pc] = d;
    }
}

// Products of column j.  Reads n'^2 / 2 elements once: 5 TB/s where many large factors share a launch, memory latency (6 us)
// where few do; all loads are issued before anything is waited for.
__global__ __launch_bounds__(256) void dir_symv_kernel(const DirMat *mats, const unsigned *tab, int t) {
    __shared__ SymvSmem sm;
    const TabRef tr = tab_ref(tab[blockIdx.x]);
    const DirMat M = mats[tr.m];
    const int j = t - M.off;
    if (j > M.n - 2) return;
    const int tid = threadIdx.x, ip = t & (NB - 1);
    const StepBufs B = step_bufs(M, t);
    const float x = B.acol[(tid < TB ? tr.I * TB : tr.J * TB - TB) + tid];
    TileLoads L;
    tile_load(M, tr.I, tr.J, ip, L);
    (tid < TB ? sm.xI : sm.xJ - TB)[tid] = x;
    __syncthreads();
    tile_product(M, tr.I, tr.J, j / TB, ip, B, L, sm);
}

// The vector step's sums over row blocks and what follows from them, for one wave: column j's products are in P.  Every wave
// of a workgroup forms the scalars for itself; partial sums over four waves go through LDS.
struct VecSmem { float cw[4][2 * NB]; double tred[4]; };
struct VecLoads {
    float n0, n1, alpha, rowj, yj, ajj, ck[8];
    double tk[3];
};
struct VecScalars { float scale, beta, tau, cf, ah, wj; };
__device__ inline void vec_load(const DirMat &M, const StepBufs &P, int j, int ip, int b0, VecLoads &L) {
    const int tid = threadIdx.x, lane = tid & 63, g = tid >> 6;
    const int ct = M.nb - b0, nt = ct * (ct + 1) / 2, last = M.nb - 1, nrb = M.np / RB, rb = 2 * b0 + lane;
    L.n0 = P.npart[min(rb, nrb - 1)];
    L.n1 = P.npart[min(rb + 64, nrb - 1)];
    L.alpha = P.acol[j + 1];
#pragma unroll
    for (int u = 0; u < 8; ++u) L.ck[u] = P.dots[min(b0 + g + 4 * u, last) * 2 * NB + lane];
#pragma unroll
    for (int u = 0; u < 3; ++u) L.tk[u] = P.tsum[min(tid + 256 * u, nt - 1)];
    L.rowj = as_global((const float *)M.panel)[(int64_t)lane * M.ld + j + 1];
    L.yj = P.part[(int64_t)min(b0 + lane, last) * M.np + j + 1];
    L.ajj = as_global((const float *)M.apan)[(int64_t)(ip + 1) * M.np + j + 1];
}
__device__ inline void vec_partial(const DirMat &M, const StepBufs &P, int ip, int b0, const VecLoads &L, VecSmem &sm) {
    const int tid = threadIdx.x, lane = tid & 63, g = tid >> 6;
    const int ct = M.nb - b0, nt = ct * (ct + 1) / 2;
    float c = 0.f;
    double xax = 0.0;
#pragma unroll
    for (int u = 0; u < 8; ++u) c += g + 4 * u < ct ? L.ck[u] : 0.f;
#pragma unroll
    for (int u = 0; u < 3; ++u) xax += tid + 256 * u < nt ? L.tk[u] : 0.0;
    for (int k = b0 + g + 32; k < M.nb; k += 4) c += P.dots[k * 2 * NB + lane];
    for (int i = tid + 768; i < nt; i += 256) xax += P.tsum[i];
    sm.cw[g][lane] = (lane & (NB - 1)) < ip ? c : 0.f;     // (the others' dots are an earlier panel's)
    xax = wave_sum_f64(xax);
    if (lane == 0) sm.tred[g] = xax;
}
// after the barrier behind vec_partial(); rowj: V and W of row j + 1, zero beyond the panel's columns
__device__ inline VecScalars vec_scalars(const DirMat &M, int ip, int b0, const VecLoads &L, float rowj, const VecSmem &sm) {
    const int lane = threadIdx.x & 63, nrb = M.np / RB, rb = 2 * b0 + lane;
    VecScalars S;
    const float s2 = wave_sum_all((rb < nrb ? L.n0 : 0.f) + (rb + 64 < nrb ? L.n1 : 0.f));
    const float alpha = L.alpha;
    S.beta = alpha;
    S.tau = S.scale = 0.f;
    if (s2 > 0.f) {
        S.beta = -copysignf(sqrtf(fmaf(alpha, alpha, s2)), alpha);
        S.tau = (S.beta - alpha) / S.beta;
        S.scale = 1.f / (alpha - S.beta);
    }
    const float yj = wave_sum_all(b0 + lane < M.nb ? L.yj : 0.f);
    const double xax = sm.tred[0] + sm.tred[1] + sm.tred[2] + sm.tred[3];
    S.cf = S.scale * fmaf(-S.beta, rowj, sm.cw[0][lane] + sm.cw[1][lane] + sm.cw[2][lane] + sm.cw[3][lane]);   // V^T v, W^T v
    const float o = __shfl_xor(S.cf, 32, 64);
    const float dvw = wave_sum_all(lane < 32 ? S.cf * o : 0.f);                       // (V^T v) . (W^T v)
    const float rc = wave_sum_all(rowj * o);                                         // row j + 1 of V (W^T v) + W (V^T v)
    const double b = S.beta, sc = S.scale;
    const float vav = (float)(sc * (sc * (xax - 2.0 * b * yj + b * b * L.ajj)));
    // alpha_h of w = tau y + alpha_h v, and row j + 1 of w (where v is 1)
    S.ah = -0.5f * S.tau * S.tau * (vav - 2.f * dvw);
    S.wj = fmaf(S.tau, fmaf(S.scale, fmaf(-S.beta, L.ajj, yj), -rc), S.ah);
    return S;
}
// element `row` of the reflector and of w, stored where the panel's update and the back-transformation read them
__device__ inline void vec_store(const DirMat &M, int j, int ip, int row, float v, float w, const VecScalars &S) {
    const global_ptr<float> pan = as_global(M.panel);
    pan[(int64_t)ip * M.ld + row] = v;
    pan[(int64_t)(NB + ip) * M.ld + row] = w;
    pan[(int64_t)(2 * NB + ip) * M.ld + row] = v;
    as_global(M.A)[(int64_t)j * M.ld + row] = v;
    if (row == j + 1) {
        M.tau[j] = S.tau;
        M.e[j] = (double)S.beta;
    }
}

// Vector step of column j: w, the panel's new columns, reflector j, and (unless the panel ends here) column j + 1 with the
// panel's updates applied.
__global__ __launch_bounds__(256) void dir_vector_kernel(const DirMat *mats, const unsigned *tab, int t) {
    __shared__ VecSmem vs;
    __shared__ float ys[4][RB], as_[4][RB];
    const TabRef tr = tab_ref(tab[blockIdx.x]);
    const DirMat M = mats[tr.m];
    const int j = t - M.off;
    if (j > M.n - 2) return;
    const int tid = threadIdx.x, lane = tid & 63, g = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ip = t & (NB - 1), b0 = j / TB, row = tr.J * RB + lane, ct = M.nb - b0, last = M.nb - 1;
    const bool next = ip != NB - 1;
    const StepBufs P = step_bufs(M, t), B = step_bufs(M, t + 1);
    const global_ptr<const float> panel = as_global((const float *)M.panel);
    VecLoads L;
    vec_load(M, P, j, ip, b0, L);
    float yk[8], pv[NB / 4], pw[NB / 4];
#pragma unroll
    for (int u = 0; u < 8; ++u) yk[u] = P.part[(int64_t)min(b0 + g + 4 * u, last) * M.np + row];
#pragma unroll
    for (int u = 0; u < NB / 4; ++u) {
        pv[u] = panel[(int64_t)(g + 4 * u) * M.ld + row];
        pw[u] = panel[(int64_t)(NB + g + 4 * u) * M.ld + row];
    }
    const float acur = as_global((const float *)M.apan)[(int64_t)(ip + 1) * M.np + row], xv = P.acol[row];
    float y = 0.f;
#pragma unroll
    for (int u = 0; u < 8; ++u) y += g + 4 * u < ct ? yk[u] : 0.f;
    for (int k = b0 + g + 32; k < M.nb; k += 4) y += P.part[(int64_t)k * M.np + row];
    vec_partial(M, P, ip, b0, L, vs);
    __syncthreads();
    const float rowj = (lane & (NB - 1)) < ip ? L.rowj : 0.f;
    const VecScalars S = vec_scalars(M, ip, b0, L, rowj, vs);
    float yc = 0.f, ac = 0.f;
#pragma unroll
    for (int u = 0; u < NB / 4; ++u) {
        const int p = g + 4 * u;
        if (p >= ip) pv[u] = pw[u] = 0.f;       // not this panel's
        yc = fmaf(pv[u], lane_value(S.cf, NB + p), fmaf(pw[u], lane_value(S.cf, p), yc));
        ac = fmaf(pv[u], lane_value(rowj, NB + p), fmaf(pw[u], lane_value(rowj, p), ac));
    }
    ys[g][lane] = fmaf(S.scale, y, -yc);
    as_[g][lane] = ac;
    __syncthreads();
    if (g != 0) return;
    y = ys[0][lane] + ys[1][lane] + ys[2][lane] + ys[3][lane] - S.scale * S.beta * acur;
    ac = as_[0][lane] + as_[1][lane] + as_[2][lane] + as_[3][lane];
    const float v = row > j + 1 ? xv * S.scale : (row == j + 1 ? 1.f : 0.f);
    const float w = row > j ? fmaf(S.tau, y, S.ah * v) : 0.f;
    vec_store(M, j, ip, row, v, w, S);
    if (!next) return;
    const float a = row > j ? acur - ac - fmaf(v, S.wj, w) : 0.f;
    if (row == j + 1) M.d[j + 1] = (double)a;
    B.acol[row] = row > j + 1 ? a : 0.f;
    const float s = wave_sum_all(row > j + 2 ? a * a : 0.f);
    if (lane == 0) B.npart[tr.J] = s;
}

// C -= acc for the rows of the tile from `first` on, sixteen elements at a time (one accumulator's loads in flight, not 64)
__device__ inline void subtract_tile(const floatx16 (&acc)[2][2], global_ptr<float> C, int64_t ld, int first) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lk = lane >> 5, lc = lane & 31;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int r0 = (wave >> 1) * 64 + 32 * i + 4 * lk;
            const global_ptr<float> p = C + (int64_t)r0 * ld + (wave & 1) * 64 + 32 * k + lc;
            float old[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) old[r] = p[(int64_t)(8 * (r >> 2) + (r & 3)) * ld];
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (r0 + 8 * (r >> 2) + (r & 3) >= first) p[(int64_t)(8 * (r >> 2) + (r & 3)) * ld] = old[r] - acc[i][k][r];
        }
}

// Rank-64 update of the trailing matrix by the panel that ends before step t: A_IJ -= V_I W_J^T + W_I V_J^T (lower tiles).
__global__ __launch_bounds__(NTHREADS) __attribute__((amdgpu_waves_per_eu(3))) void dir_update_kernel(const DirMat *mats, const unsigned *tab, int t) {
    __shared__ TileSmem sm;
    const TabRef tr = tab_ref(tab[blockIdx.x]);
    const DirMat M = mats[tr.m];
    if (t - M.off <= 0) return;        // this factor's reduction starts at step t
    const int64_t ld = M.ld;
    OpStrided<float, false> a{M.panel + tr.I * TB, 1, ld, TB, 2 * NB, -1};
    OpStrided<float, false> b{M.panel + NB * ld + tr.J * TB, 1, ld, TB, 2 * NB, -1};
    floatx16 acc[2][2];
    const global_ptr<float> C = as_global(M.A) + (int64_t)tr.I * TB * ld + tr.J * TB;
    gemm_tile(a, b, 0, 0, 0, 2 * NB, sm, acc);
    subtract_tile(acc, C, ld, t - M.off - tr.I * TB);      // rows of finished columns hold reflectors
}

// What the chain leaves of a factor, for the chip: the lower triangle of the trailing matrix (rows and columns from M.chain on)
// copied to the upper, in 64 x 64 blocks.
__global__ __launch_bounds__(256) void dir_mirror_kernel(const DirMat *mats) {
    __shared__ float s[64][65];
    const DirMat M = mats[blockIdx.y];
    if (M.n <= TD_SMALL || M.chain == 0) return;
    const global_ptr<float> A = as_global(M.A);
    const int b0 = M.chain / 64, nblk = M.np / 64 - b0, c = threadIdx.x & 63;
    empty_ring(M, blockIdx.x, gridDim.x);
    for (int q = blockIdx.x; q < nblk * nblk; q += gridDim.x) {
        const int I = b0 + q / nblk, J = b0 + q % nblk;
        if (J > I) continue;
        __syncthreads();
        for (int r = threadIdx.x >> 6; r < 64; r += 4) s[r][c] = A[(int64_t)(I * 64 + r) * M.ld + J * 64 + c];
        __syncthreads();
        for (int r = threadIdx.x >> 6; r < 64; r += 4) {      // element (J 64 + r, I 64 + c)
            const int gr = J * 64 + r, gc = I * 64 + c;
            if (gr >= M.chain && gr < gc) A[(int64_t)gr * M.ld + gc] = s[c][r];
        }
    }
}

// Row p of A keeps reflector p only: zeros up to and including the diagonal.
__global__ __launch_bounds__(256) void dir_clear_kernel(const DirMat *mats) {
    const DirMat M = mats[blockIdx.y];
    if (M.n <= TD_SMALL) return;
    const global_ptr<float> A = as_global(M.A);
    for (int r = blockIdx.x; r < M.np; r += gridDim.x) {
        const int end = r >= M.n - 1 ? M.np : r + 1;
        for (int c = threadIdx.x; c < end; c += 256) A[(int64_t)r * M.ld + c] = 0.f;
    }
}

// ---- eigenvalues and eigenvectors of T ------------------------------------------------------------------------
__device__ inline double hash_unit(int i) {   // in [-1, 1): the output function of SplitMix64 (Steele, Lea, Flood 2014) and its constants
    unsigned long long z = (unsigned long long)(i + 1) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    z ^= z >> 31;
    return (double)(long long)(z >> 11) * (1.0 / 4503599627370496.0) - 1.0;
}

// td <- T / (Gershgorin bound), its diagonal perturbed; zeros where the matrix is not finite.  tsum[0]: see CORRECT_FROM.
__global__ __launch_bounds__(256) void dir_scale_t_kernel(const DirMat *mats) {
    const DirMat M = mats[blockIdx.x];
    const int n = M.n;
    double g = 0.0;
    for (int i = threadIdx.x; i < n; i += 256)
        g = fmax(g, fabs(M.d[i]) + (i > 0 ? fabs(M.e[i - 1]) : 0.0) + (i < n - 1 ? fabs(M.e[i]) : 0.0));
    __shared__ double red[4];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) g = fmax(g, __shfl_xor(g, o, 64));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = g;
    __syncthreads();
    g = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
    const double inv = (g > 0.0 && g < 1e300) ? 1.0 / g : 0.0;
    if (n > TD_SMALL) {
        const double f2 = M.stat[0] + M.stat[1], sc = norm_scale(f2);
        double often = 0.0;
        for (int i = threadIdx.x; i < n; i += 256) {
            const double d = M.d[i], e = i < n - 1 ? M.e[i] : 0.0;
            often += (d * d + 2.0 * e * e) * max(i - M.chain, 0);
        }
        often = wave_sum_f64(often);
        __syncthreads();
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = often;
        __syncthreads();
        if (threadIdx.x == 0) M.tsum[0] = (red[0] + red[1] + red[2] + red[3]) / (sc * sc * f2);
    }
    for (int i = threadIdx.x; i < n; i += 256) {
        const double e = i < n - 1 ? M.e[i] : 0.0, d = M.d[i];
        double en = fabs(e) < 1e300 ? e * inv * (1.0 + PERTURB_REL * hash_unit(-2 - i)) : 0.0;
        if (i < n - 1 && fabs(en) < E_MIN) en = E_MIN;
        M.td[i] = make_double2((fabs(d) < 1e300 ? d * inv : 0.0) * (1.0 + PERTURB_REL * hash_unit(2 * i)) + PERTURB_ABS * hash_unit(2 * i + 1), en * en);
        M.te[i] = en;
    }
}

// Eigenvalue k of T by multisection in fp64: LPE lanes per eigenvalue try the points that cut its interval into LPE + 1 (2.3 bits
// a pass with four lanes, 4.1 with sixteen).  A count is a Sturm sequence of the leading minors' signs, two dependent
// FMAs per row; the minors are rescaled every eight rows.  The passes go on until the interval is at the last bits of the
// eigenvalue itself, not of the largest one: the thousands of tiny eigenvalues of a graded rank-deficient factor have localised
// eigenvectors and do not repel each other, so two of them can agree to 1e-17 of the largest, and where the passes
// stopped there both got the same eigenvector.
constexpr int BIS_CHUNK = 256;
template <int LPE>
__global__ __launch_bounds__(256) void dir_bisect_kernel(const DirMat *mats, const unsigned *tab) {
    constexpr int PER_WG = 256 / LPE, PARTS = 64 / PER_WG;      // a table entry stands for 64 eigenvalues
    __shared__ double2 ch[BIS_CHUNK];
    const TabRef tr = tab_ref(tab[blockIdx.x / PARTS]);
    const DirMat M = mats[tr.m];
    if (is_diagonal(M)) return;
    const int n = M.n, tid = threadIdx.x, q = tid & (LPE - 1), k = tr.J * 64 + (int)(blockIdx.x % PARTS) * PER_WG + tid / LPE;
    double lo = -1.0 - 1e-6, hi = 1.0 + 1e-6;     // Gershgorin, with room for the perturbation
    for (int pass = 0; pass < 40; ++pass) {
        const double step = (hi - lo) * (1.0 / (LPE + 1)), x = lo + step * (q + 1);
        double p = 1.0, pp = 0.0;     // minors i and i - 1
        double e2 = 0.0;
        int count = 0;
        for (int base = 0; base < n; base += BIS_CHUNK) {
            __syncthreads();
            if (base + tid < n) ch[tid] = M.td[base + tid];
            else ch[tid] = make_double2(4.0, 0.0);   // rows past the end: no sign changes
            __syncthreads();
            const int cnt = min(BIS_CHUNK, (n - base + 7) & ~7);
            for (int i = 0; i < cnt; i += 8) {
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const double2 t = ch[i + u];
                    const double np_ = fma(t.x - x, p, -e2 * pp);   // p and pp are never both zero: e2 is not
                    count += (int)(((unsigned)__double2hiint(np_) ^ (unsigned)__double2hiint(p)) >> 31);
                    pp = p;
                    p = np_;
                    e2 = t.y;
                }
                const int ex = -__builtin_amdgcn_frexp_exp(fmax(fabs(p), fabs(pp)));
                p = ldexp(p, ex);
                pp = ldexp(pp, ex);
            }
        }
        int below = count <= k ? 1 : 0;     // the eigenvalue is not below this point
#pragma unroll
        for (int o = 1; o < LPE; o <<= 1) below += __shfl_xor(below, o, 64);
        const double l0 = lo;
        lo = below > 0 ? l0 + step * below : lo;
        hi = below < LPE ? l0 + step * (below + 1) : hi;
        const bool open = k < n && hi - lo > BIS_REL * fmax(fabs(lo), fabs(hi)) + BIS_ABS;
        if (!__syncthreads_or(open)) break;
    }
    if (q == 0 && k < n) M.lam64[k] = 0.5 * (lo + hi);
}

__device__ inline double fast_rcp(double q) {   // |q| in [1e-30, 1e60]: hardware estimate, two Newton steps
    double r = __builtin_amdgcn_rcp(q);
    r = fma(fma(-q, r, 1.0), r, r);
    r = fma(fma(-q, r, 1.0), r, r);
    return r;
}
__device__ inline double pivot(double q) { return fabs(q) < PIVOT_MIN ? -PIVOT_MIN : q; }

// Eigenvector k of T by twisted factorisation: pivots q_i of the elimination from the top and r_i of the one from the
// bottom, the twist where |q_i + r_i - (d_i - lam)| is least, and the two recurrences away from it.  One lane per
// eigenvector; the pivots of the wave's 64 vectors are rows of 512 bytes.  A serial chain of a division per row, bound by the
// latency of the fp64 units: so two chains always run side by side (the eliminations meet in the middle, go on past each other to
// find the twist, and only what was passed over on the way to it is eliminated again; then the two recurrences), and what
// they read is loaded a batch ahead.  One 4609-wide factor 4.1 -> 2.3 ms.
constexpr int VEC_CHUNK = 128, VEC_BATCH = 8;

// Steps s = 0, 1, ..: a(s, u) for s < na and b(s, u) for s < nb, side by side; u: place of s in its batch of VEC_BATCH.
// chunk(s, count): called before every VEC_CHUNK steps; batch(s): before every VEC_BATCH; stores(s): after them (a and b branch nowhere, so
// that their instructions alternate).
template <class Chunk, class Batch, class A, class B, class Stores>
__device__ inline void two_chains(int na, int nb, Chunk chunk, Batch batch, A a, B b, Stores stores) {
    const int n = max(na, nb), both = min(na, nb);
    for (int s0 = 0; s0 < n; s0 += VEC_CHUNK) {
        __syncthreads();
        chunk(s0, min(VEC_CHUNK, n - s0));
        __syncthreads();
        for (int s = s0; s < min(n, s0 + VEC_CHUNK); s += VEC_BATCH) {
            batch(s);
            if (s + VEC_BATCH <= both) {
#pragma unroll
                for (int u = 0; u < VEC_BATCH; ++u) {
                    a(s + u, u);
                    b(s + u, u);
                }
            } else {
#pragma unroll
                for (int u = 0; u < VEC_BATCH; ++u) {
                    if (s + u < na) a(s + u, u);
                    if (s + u < nb) b(s + u, u);
                }
            }
            stores(s);
        }
    }
}

__global__ __launch_bounds__(64) void dir_vectors_kernel(const DirMat *mats, const unsigned *tab) {
    __shared__ double2 ca[VEC_CHUNK], cb[VEC_CHUNK];      // T along the two chains
    const TabRef tr = tab_ref(tab[blockIdx.x]);
    const DirMat M = mats[tr.m];
    const int n = M.n, lane = threadIdx.x, k = min(tr.J * 64 + lane, n - 1), mid = n / 2;     // (lanes past the end do the last one again)
    const int64_t ld = M.ld;
    if (is_diagonal(M)) {
        for (int i = 0; i < n; ++i) as_global(M.Z)[(int64_t)i * ld + k] = i == k ? 1.f : 0.f;
        return;
    }
    const double lam = M.lam64[k];
    const global_ptr<double> D = as_global((double *)M.B1) + k;
    const global_ptr<float> Z = as_global(M.Z) + k;
    const global_ptr<const double> td = as_global((const double *)M.td);      // {d_i, e_i^2}
    const global_ptr<const double> te = as_global((const double *)M.te);
    double q = 1.0, r = 1.0, e2 = 0.0;
    double da[VEC_BATCH], db[VEC_BATCH], na[VEC_BATCH], nb[VEC_BATCH];     // pivots stored before: this batch's and the next one's
    double oa[VEC_BATCH], ob[VEC_BATCH];                                   // to be stored
    // (indices past an end are clamped: what is read there is not used)
    auto fetch = [&](int a0, int b0, int s) {      // rows a0 + s .. upwards and b0 - s .. downwards
#pragma unroll
        for (int u = 0; u < VEC_BATCH; ++u) {
            na[u] = D[(int64_t)min(max(a0 + s + u, 0), n - 1) * ld];
            nb[u] = D[(int64_t)min(max(b0 - s - u, 0), n - 1) * ld];
        }
    };
    auto step_batch = [&](int a0, int b0, int s) {
        if (s == 0) fetch(a0, b0, 0);
#pragma unroll
        for (int u = 0; u < VEC_BATCH; ++u) {
            da[u] = na[u];
            db[u] = nb[u];
        }
        fetch(a0, b0, s + VEC_BATCH);
    };
    auto stage = [&](int a0, int b0, int s, int cnt) {
        for (int i = lane; i < cnt; i += 64) {
            const int ia = min(max(a0 + s + i, 0), n - 1), ib = min(max(b0 - s - i, 0), n - 1);
            ca[i] = make_double2(td[2 * ia], td[2 * ia + 1]);
            cb[i] = make_double2(td[2 * ib], td[2 * ib + 1]);
        }
    };
    // from the top down to the middle, from the bottom up to it
    two_chains(mid, n - mid, [&](int s, int cnt) { stage(0, n - 1, s, cnt); }, [](int) {},
        [&](int s, int u) {
            const double2 t = ca[s & (VEC_CHUNK - 1)];
            q = pivot((t.x - lam) - e2 * fast_rcp(q));
            oa[u] = q;
            e2 = t.y;
        },
        [&](int s, int u) {
            const double2 t = cb[s & (VEC_CHUNK - 1)];
            r = pivot((t.x - lam) - t.y * fast_rcp(r));     // t.y couples rows i and i + 1 (zero in the last row)
            ob[u] = r;
        },
        [&](int s) {
#pragma unroll
            for (int u = 0; u < VEC_BATCH; ++u) {
                if (s + u < mid) D[(int64_t)(s + u) * ld] = oa[u];
                if (s + u < n - mid) D[(int64_t)(n - 1 - s - u) * ld] = ob[u];
            }
        });
    // on past each other: the twist, the last row among equals
    const double qm = q, rm = r, e2m = e2;
    double besta = 1e300, bestb = 1e300;
    int twa = n - 1, twb = 0;
    two_chains(n - mid, mid, [&](int s, int cnt) { stage(mid, mid - 1, s, cnt); }, [&](int s) { step_batch(mid, mid - 1, s); },
        [&](int s, int u) {
            const double2 t = ca[s & (VEC_CHUNK - 1)];
            const double dl = t.x - lam;
            q = pivot(dl - e2 * fast_rcp(q));
            e2 = t.y;
            const double gam = fabs(q + (da[u] - dl));
            const bool better = gam <= besta;
            besta = better ? gam : besta;
            twa = better ? mid + s : twa;
        },
        [&](int s, int u) {
            const double2 t = cb[s & (VEC_CHUNK - 1)];
            const double dl = t.x - lam;
            r = pivot(dl - t.y * fast_rcp(r));
            const double gam = fabs(db[u] + (r - dl));
            const bool better = gam < bestb;
            bestb = better ? gam : bestb;
            twb = better ? mid - 1 - s : twb;
        },
        [](int) {});
    const int tw = bestb < besta ? twb : twa;
    int tmin = tw, tmax = tw;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) { tmin = min(tmin, __shfl_xor(tmin, o, 64)); tmax = max(tmax, __shfl_xor(tmax, o, 64)); }
    tmin = __builtin_amdgcn_readfirstlane(tmin);
    tmax = __builtin_amdgcn_readfirstlane(tmax);
    // the pivots between the middle and the twist, those of the other side so far
    q = qm;
    r = rm;
    e2 = e2m;
    two_chains(tmax - mid, mid - 1 - tmin, [&](int s, int cnt) { stage(mid, mid - 1, s, cnt); }, [](int) {},
        [&](int s, int u) {
            const double2 t = ca[s & (VEC_CHUNK - 1)];
            q = pivot((t.x - lam) - e2 * fast_rcp(q));
            oa[u] = q;
            e2 = t.y;
        },
        [&](int s, int u) {
            const double2 t = cb[s & (VEC_CHUNK - 1)];
            r = pivot((t.x - lam) - t.y * fast_rcp(r));
            ob[u] = r;
        },
        [&](int s) {
#pragma unroll
            for (int u = 0; u < VEC_BATCH; ++u) {
                if (mid + s + u < tw) D[(int64_t)(mid + s + u) * ld] = oa[u];
                if (mid - 1 - s - u > tw) D[(int64_t)(mid - 1 - s - u) * ld] = ob[u];
            }
        });
    // away from the twist, downwards and upwards
    double za = 1.0, zb = 1.0, nrma = 0.0, nrmb = 1.0;
    two_chains(n - 1 - tmin, tmax + 1,
        [&](int s, int cnt) {
            for (int i = lane; i < cnt; i += 64) {
                ca[i].x = te[min(tmin + s + i, n - 1)];            // couples row tmin + 1 + s to the one above
                cb[i].x = te[max(tmax - s - i, 0)];                // couples row tmax - s to the one below
            }
        },
        [&](int s) { step_batch(tmin + 1, tmax, s); },
        [&](int s, int u) {
            const double z = -ca[s & (VEC_CHUNK - 1)].x * za * fast_rcp(da[u]);
            za = tmin + 1 + s > tw ? z : 1.0;
            nrma += tmin + 1 + s > tw ? z * z : 0.0;
            oa[u] = za;
        },
        [&](int s, int u) {
            const double z = -cb[s & (VEC_CHUNK - 1)].x * zb * fast_rcp(db[u]);
            zb = tmax - s < tw ? z : 1.0;
            nrmb += tmax - s < tw ? z * z : 0.0;
            ob[u] = zb;
        },
        [&](int s) {
#pragma unroll
            for (int u = 0; u < VEC_BATCH; ++u) {
                const int ia = tmin + 1 + s + u, ib = tmax - s - u;
                if (ia > tw && ia < n) Z[(int64_t)ia * ld] = (float)oa[u];
                if (ib <= tw && ib >= 0) Z[(int64_t)ib * ld] = (float)ob[u];
            }
        });
    const float inv = (float)(1.0 / sqrt(nrma + nrmb));
    constexpr int ROWS = 32;
    const bool own = tr.J * 64 + lane < n;      // (here a lane must not find what another one has scaled)
    for (int i0 = 0; own && i0 < n; i0 += ROWS) {
        float zz[ROWS];
#pragma unroll
        for (int u = 0; u < ROWS; ++u) zz[u] = Z[(int64_t)min(i0 + u, n - 1) * ld];
#pragma unroll
        for (int u = 0; u < ROWS; ++u)
            if (i0 + u < n) Z[(int64_t)(i0 + u) * ld] = zz[u] * inv;
    }
}

// ---- back-transformation -------------------------------------------------------------------------------------
// Small factors: a wave owns four columns of Z, lane l the rows l, l + 64, ..: all reflectors are applied out of registers, no
// barriers; what bounds it is the latency of a reflector's four wave sums.
__global__ __launch_bounds__(256) void dir_apply_kernel(const DirMat *mats, const unsigned *tab) {
    constexpr int RPL = TD_SMALL / 64;
    const TabRef tr = tab_ref(tab[blockIdx.x]);
    const DirMat M = mats[tr.m];
    const int n = M.n, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, c0 = tr.J * 16 + wave * 4;
    if (c0 >= n || is_diagonal(M)) return;
    const int64_t ld = M.ld;
    const global_ptr<float> Z = as_global(M.Z) + c0;
    floatx4 z[RPL];
#pragma unroll
    for (int k = 0; k < RPL; ++k) {
        const int r = lane + 64 * k;
        z[k] = r < n ? *(global_ptr<floatx4>)(Z + (int64_t)r * ld) : floatx4{0.f, 0.f, 0.f, 0.f};
    }
    const global_ptr<const float> A = as_global((const float *)M.A), tau = as_global((const float *)M.tau);
    float v[RPL], vn[RPL];
    auto load = [&](float (&x)[RPL], int p) {
#pragma unroll
        for (int k = 0; k < RPL; ++k) {
            const int r = lane + 64 * k;
            x[k] = (r < n && r > p) ? A[(int64_t)p * ld + r] : 0.f;
        }
    };
    int p = n - 2;
    if (p >= 0) load(v, p);
    for (; p >= 0; --p) {
        if (p > 0) load(vn, p - 1);
        floatx4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < RPL; ++k) s += v[k] * z[k];
        const float tp = tau[p];
        const floatx4 f = {-tp * wave_sum_all(s.x), -tp * wave_sum_all(s.y), -tp * wave_sum_all(s.z), -tp * wave_sum_all(s.w)};
#pragma unroll
        for (int k = 0; k < RPL; ++k) {
            z[k] += v[k] * f;
            v[k] = vn[k];
        }
    }
#pragma unroll
    for (int k = 0; k < RPL; ++k) {
        const int r = lane + 64 * k;
        if (r < n) *(global_ptr<floatx4>)(Z + (int64_t)r * ld) = z[k];
    }
}

// Large factors: H_{j0} .. H_{j0+127} = I - V T V^T.  Gram matrices of all blocks, their T, U = V T (as rows T^T V^T), then
// block after block from the last: Y = V^T Z, Z -= U Y.
__global__ __launch_bounds__(NTHREADS) __attribute__((amdgpu_waves_per_eu(2))) void dir_wy_gram_kernel(const DirMat *mats, const unsigned *tab) {
    __shared__ TileSmem sm;
    const TabRef tr = tab_ref(tab[blockIdx.x]);
    const DirMat M = mats[tr.m];
    const int j0 = tr.J * WY;
    const int64_t ld = M.ld;
    OpStrided<float, true> a{M.A + (int64_t)j0 * ld, ld, 1, WY, M.np, -1}, b{M.A + (int64_t)j0 * ld, ld, 1, WY, M.np, -1};
    floatx16 acc[2][2];
    gemm_tile_segmented<128, false>(a, b, 0, 0, j0, M.np, sm, acc);
    float *G = M.Tm + (int64_t)tr.J * WY * WY;
    for_each_acc(acc, [&](int r, int c, float v) { as_global(G)[r * WY + c] = v; });
}

// T column by column: T(r, i) = -tau_i sum_p T(r, p) G(p, i).  WT lanes share a row's sum: the chain of columns is serial, and
// with one lane per row its LDS latencies made 1.2 ms of the ResNet-50 step (410 us for a single block).
constexpr int WT = 8;
__global__ __launch_bounds__(WY * WT) void dir_wy_t_kernel(const DirMat *mats, const unsigned *tab) {
    extern __shared__ float lds[];
    __shared__ float taus[WY];
    const TabRef tr = tab_ref(tab[blockIdx.x]);
    const DirMat M = mats[tr.m];
    float *T = lds, *G = lds + WY * (WY + 1);
    if (threadIdx.x < WY) taus[threadIdx.x] = M.tau[tr.J * WY + threadIdx.x];
    const int r = threadIdx.x / WT, l = threadIdx.x & (WT - 1), c0 = threadIdx.x & (WY - 1), r0 = threadIdx.x / WY;
    const global_ptr<float> g = as_global(M.Tm + (int64_t)tr.J * WY * WY);
    for (int i = r0; i < WY; i += WT) { G[i * (WY + 1) + c0] = g[i * WY + c0]; T[i * (WY + 1) + c0] = 0.f; }
    __syncthreads();
    for (int i = 0; i < WY; ++i) {
        const float ti = taus[i];
        double s = 0.0;
        if (r < i)
#pragma unroll 4
            for (int p = r + l; p < i; p += WT) s = fma((double)T[r * (WY + 1) + p], (double)G[p * (WY + 1) + i], s);
#pragma unroll
        for (int o = 1; o < WT; o <<= 1) s += __shfl_xor(s, o, 64);
        if (l == 0 && r <= i) T[r * (WY + 1) + i] = r == i ? ti : (float)(-ti * s);
        __syncthreads();
    }
    for (int i = r0; i < WY; i += WT) g[i * WY + c0] = T[i * (WY + 1) + c0];
}

__global__ __launch_bounds__(NTHREADS) __attribute__((amdgpu_waves_per_eu(3))) void dir_wy_u_kernel(const DirMat *mats, const unsigned *tab) {
    __shared__ TileSmem sm;
    const TabRef tr = tab_ref(tab[blockIdx.x]);
    const DirMat M = mats[tr.m];
    const int j0 = tr.I * WY;
    const int64_t ld = M.ld;
    OpStrided<float, false> a{M.Tm + (int64_t)tr.I * WY * WY, 1, WY, WY, WY, -1};          // T[k][i]
    OpStrided<float, false> b{M.A + (int64_t)j0 * ld + tr.J * TB, 1, ld, TB, WY, -1};      // V^T[k][n]
    floatx16 acc[2][2];
    gemm_tile(a, b, 0, 0, 0, WY, sm, acc);
    const global_ptr<float> U = as_global(M.B1) + (int64_t)j0 * ld + tr.J * TB;
    for_each_acc(acc, [&](int r, int c, float v) { U[(int64_t)r * ld + c] = v; });
}

// Step s counts blocks from the last one of every factor.  Y = V^T Z is one row of tiles with a contraction of up to n: it
// is cut into pieces of 512 (more workgroups than the 111 tiles of three 4609-wide factors, and partial sums short enough
// not to lose accuracy), which dir_wy_sum_kernel adds.  The pieces lie in B2, 128 rows each.
__global__ __launch_bounds__(NTHREADS) __attribute__((amdgpu_waves_per_eu(3))) void dir_wy_y_kernel(const DirMat *mats, const unsigned *tab, int s) {
    __shared__ TileSmem sm;
    const TabRef tr = tab_ref(tab[blockIdx.x]);
    const DirMat M = mats[tr.m];
    const int blk = M.nb - 1 - s, j0 = blk * WY, k0 = j0 + tr.I * WY_K;
    if (blk < 0 || k0 >= M.n) return;
    const int k1 = min(k0 + WY_K, M.n);
    const int64_t ld = M.ld;
    OpStrided<float, true> a{M.A + (int64_t)j0 * ld, ld, 1, WY, k1, -1};
    OpStrided<float, false> b{M.Z + tr.J * TB, 1, ld, TB, k1, -1};
    floatx16 acc[2][2];
    gemm_tile(a, b, 0, 0, k0, k1, sm, acc);
    const global_ptr<float> Y = as_global(M.B2) + (int64_t)tr.I * WY * ld + tr.J * TB;
    for_each_acc(acc, [&](int r, int c, float v) { Y[(int64_t)r * ld + c] = v; });
}
__global__ __launch_bounds__(256) void dir_wy_sum_kernel(const DirMat *mats, const unsigned *tab, int s) {
    const TabRef tr = tab_ref(tab[blockIdx.x]);
    const DirMat M = mats[tr.m];
    const int blk = M.nb - 1 - s;
    const int pieces = blk < 0 ? 0 : (M.n - blk * WY + WY_K - 1) / WY_K;
    if (pieces < 2) return;
    const int64_t ld = M.ld;
    const global_ptr<float> Y = as_global(M.B2) + (int64_t)(threadIdx.x >> 5) * ld + tr.J * TB + 4 * (threadIdx.x & 31);
#pragma unroll 4
    for (int r = 0; r < WY / 8; ++r) {
        const global_ptr<float> p = Y + (int64_t)(8 * r) * ld;
        floatx4 v = *(global_ptr<floatx4>)p;
        for (int c = 1; c < pieces; ++c) v += *(global_ptr<floatx4>)(p + (int64_t)c * WY * ld);
        *(global_ptr<floatx4>)p = v;
    }
}
__global__ __launch_bounds__(NTHREADS) __attribute__((amdgpu_waves_per_eu(3))) void dir_wy_z_kernel(const DirMat *mats, const unsigned *tab, int s) {
    __shared__ TileSmem sm;
    const TabRef tr = tab_ref(tab[blockIdx.x]);
    const DirMat M = mats[tr.m];
    const int blk = M.nb - 1 - s;
    if (blk < 0 || tr.I < blk) return;
    const int64_t ld = M.ld;
    OpStrided<float, false> a{M.B1 + (int64_t)blk * WY * ld + tr.I * TB, 1, ld, TB, WY, -1};   // U^T: elem(i, k) = U[k][i]
    OpStrided<float, false> b{M.B2 + tr.J * TB, 1, ld, TB, WY, -1};
    floatx16 acc[2][2];
    gemm_tile(a, b, 0, 0, 0, WY, sm, acc);
    subtract_tile(acc, as_global(M.Z) + (int64_t)tr.I * TB * ld + tr.J * TB, ld, 0);
}

// ---- Newton-Schulz step, F Q and the correction, all factors in one launch each (tables: largest factor first) -------------
// ORTH: B1 = (I - Q^T Q) / 2 (lower tiles and their mirror images).  STEP: Q' = Q + Q B1.  Q is Z, Q' is B2 with its rows back
// in the caller's order; for the few factors that need a second step (nearly equal eigenvalues of T whose eigenvectors
// were off by more than 1e-3) Q is B2 and Q' is Z.  TIMES_F: B1 = F Q'.
//
// A correction (CORRECT_FROM) begins with the residual R = F Q - Q diag(lam), which dir_residual_kernel puts into the caller's Q for the time being.
// TURN: A = X, X_ij = (q_i^T r_j + q_j^T r_i) / 2 (lam_j - lam_i): to first order, the rotation that makes Q^T F Q = diag(lam) + Q^T R diagonal
// (lower tiles and their mirror images.  With q_i^T r_j alone, which differs from q_j^T r_i by the rounding of F Q, X is not antisymmetric, and
// ||I - Q^T Q||_F comes out twenty times as large).  FOLLOW: Q' = Q + Q X, into the other of Z and B2, and F Q' = F Q + (F Q) X, into the caller's Q.
// Where eigenvalues are close there is nothing to gain and X would not be small, so the quotient is
// damped: gap / (gap^2 + delta^2) with delta = CORRECT_GAP times the larger residual of the two columns.  Every column of X is then shorter
// than 2^-12, whatever the spectrum, and the orthogonality that is lost (X^T X) at the level of fp32 rounding.  Both products have a factor
// that is this small, so the 22 bits of the split-fp16 products are more than fp32 would keep of their results, at any width.
enum { ORTH, STEP, TIMES_F, TURN, FOLLOW };
__device__ inline bool needs_second_step(const DirMat &M) { return M.stat[3] > NS_AGAIN; }
// (a choice between two members as a choice of values: as one of addresses it puts the whole DirMat into scratch memory, and 180 us into a kernel)
__device__ inline float *pick(bool first, float *a, float *b) { return (float *)((uintptr_t)b ^ (((uintptr_t)a ^ (uintptr_t)b) & -(uintptr_t)first)); }
__device__ inline bool corrected(const DirMat &M) { return M.n > TD_SMALL && M.tsum[1] > 0.0; }      // (from dir_residual_kernel on)
__device__ inline float *orthonormal_q(const DirMat &M) { return pick(needs_second_step(M), M.Z, M.B2); }
__device__ inline float *final_q(const DirMat &M) { return pick(needs_second_step(M) != corrected(M), M.Z, M.B2); }

template <int WHAT, bool X3>
__global__ __launch_bounds__(NTHREADS) __attribute__((amdgpu_waves_per_eu(2))) void dir_product_kernel(const DirMat *mats, const unsigned *tab, int second) {
    __shared__ typename std::conditional<X3, X3Smem, TileSmem>::type sm;
    const TabRef tr = tab_ref(tab[blockIdx.x]);
    const DirMat M = mats[tr.m];
    if ((WHAT == ORTH || WHAT == STEP) && ((M.split != 0) != X3 || (second && !needs_second_step(M)))) return;
    if ((WHAT == TURN || WHAT == FOLLOW) && !corrected(M)) return;
    const int n = M.n, i0 = tr.I * TB, j0 = tr.J * TB;
    const int64_t ld = M.ld;
    const float *Q = WHAT == ORTH || WHAT == STEP ? pick(second, M.B2, M.Z) : orthonormal_q(M);
    constexpr float SC = 16384.f, OUT = 1.f / (SC * SC);     // entries of Q, of the step and of the scaled residual are below 2
    constexpr float TURNS = 1024.f;                          // those of X far below: to keep their low halves from underflow
    floatx16 acc[2][2];
    if constexpr (WHAT == ORTH) {
        if constexpr (X3) {
            X3OpG<float, false> a{Q, ld, SC, n, n}, b{Q, ld, SC, n, n};
            a.start(threadIdx.x, i0);
            b.start(threadIdx.x, j0);
            gemm_tile_x3(a, b, n, sm, acc);
        } else {
            OpStrided<float, false> a{Q, 1, ld, n, n, -1}, b{Q, 1, ld, n, n, -1};
            gemm_tile(a, b, i0, j0, 0, n, sm, acc);
        }
        const float os = X3 ? OUT : 1.f;
        const global_ptr<float> D = as_global(M.B1);
        auto epi = [&](int gr, int gc, float v) {
            if (gr < n && gc < n) D[(int64_t)gr * ld + gc] = (gr == gc ? 0.5f : 0.f) - 0.5f * (v * os);
        };
        for_each_acc(acc, [&](int r, int c, float v) { epi(i0 + r, j0 + c, v); });
        if (j0 < i0) for_each_acc_transposed(acc, reinterpret_cast<float *>(&sm), [&](int r, int c, float v) { epi(j0 + r, i0 + c, v); });
    } else if constexpr (WHAT == STEP) {
        const global_ptr<const float> Qi = as_global(Q);
        const global_ptr<float> O = as_global(pick(second, M.Z, M.B2));
        const global_ptr<const int> ord = as_global((const int *)M.ord);
        auto epi = [&](int gr, int gc, float v) { O[(int64_t)(second ? gr : ord[gr]) * ld + gc] = Qi[(int64_t)gr * ld + gc] + v; };
        if constexpr (X3) {
            X3OpG<float, true> a{Q, ld, SC, n, n};
            X3OpG<float, false> b{M.B1, ld, SC, n, n};
            a.start(threadIdx.x, i0);
            b.start(threadIdx.x, j0);
            gemm_tile_x3(a, b, n, sm, acc);
            for_each_acc(acc, [&](int r, int c, float v) { if (i0 + r < n && j0 + c < n) epi(i0 + r, j0 + c, v * OUT); });
        } else {
            OpStrided<float, true> a{Q, ld, 1, n, n, -1};
            OpStrided<float, false> b{M.B1, 1, ld, n, n, -1};
            gemm_tile_ragged(a, b, i0, j0, n, n, n, sm, epi);
        }
    } else if constexpr (WHAT == TURN) {
        const global_ptr<float> X = as_global(M.A);
        const global_ptr<const double> lam = as_global((const double *)M.lam64), rho = as_global((const double *)M.sums);
        const double half = 0.5 * OUT / M.tsum[1];
        X3OpG<float, false> a{Q, ld, SC, n, n}, b{M.Q, n, SC, n, n}, c{M.Q, n, SC, n, n}, d{Q, ld, SC, n, n};
        a.start(threadIdx.x, i0);
        b.start(threadIdx.x, j0);
        gemm_tile_x3(a, b, n, sm, acc);
        __syncthreads();
        c.start(threadIdx.x, i0);
        d.start(threadIdx.x, j0);
        gemm_tile_x3(c, d, n, sm, acc, false);
        auto epi = [&](int gr, int gc, float v) {
            if (gr >= n || gc >= n) return;
            const double gap = lam[gc] - lam[gr], delta = CORRECT_GAP * fmax(rho[gr], rho[gc]), den = fma(gap, gap, delta * delta);
            X[(int64_t)gr * ld + gc] = den > 0.0 ? (float)(half * v * gap / den) : 0.f;
        };
        for_each_acc(acc, [&](int r, int c, float v) { epi(i0 + r, j0 + c, v); });
        if (j0 < i0) for_each_acc_transposed(acc, reinterpret_cast<float *>(&sm), [&](int r, int c, float v) { epi(j0 + r, i0 + c, v); });
    } else if constexpr (WHAT == FOLLOW) {
        const bool fq = blockIdx.y != 0;
        const float sc = fq ? SC * norm_scale(M.stat[0] + M.stat[1]) : SC;     // ||F||_F bounds the entries of F Q
        const float *Y = pick(fq, M.B1, orthonormal_q(M));
        const global_ptr<const float> Yi = as_global(Y);
        const global_ptr<float> O = as_global(pick(fq, M.Q, pick(needs_second_step(M), M.B2, M.Z)));
        const int64_t lo = fq ? n : ld;
        const float os = 1.f / (sc * (SC * TURNS));
        X3OpG<float, true> a{Y, ld, sc, n, n};
        X3OpG<float, false> b{M.A, ld, SC * TURNS, n, n};
        a.start(threadIdx.x, i0);
        b.start(threadIdx.x, j0);
        gemm_tile_x3(a, b, n, sm, acc);
        for_each_acc(acc, [&](int r, int c, float v) {
            if (i0 + r < n && j0 + c < n) O[(int64_t)(i0 + r) * lo + j0 + c] = Yi[(int64_t)(i0 + r) * ld + j0 + c] + v * os;
        });
    } else {
        OpStrided<float, true> a{M.F, n, 1, n, n, -1};
        OpStrided<float, false> b{Q, 1, ld, n, n, -1};
        const global_ptr<float> O = as_global(M.B1);
        gemm_tile_ragged<512>(a, b, i0, j0, n, n, n, sm, [&](int gr, int gc, float v) { O[(int64_t)gr * ld + gc] = v; });
    }
}

// ||I - Q^T Q||_F^2 (four times that of D), per workgroup
__global__ __launch_bounds__(256) void dir_dev_kernel(const DirMat *mats) {
    const DirMat M = mats[blockIdx.y];
    if ((int)blockIdx.x >= M.n) return;
    const global_ptr<const float> D = as_global((const float *)M.B1);
    double s = 0.0;
    for (int r = blockIdx.x; r < M.n; r += gridDim.x)
        for (int c = threadIdx.x; c < M.n; c += 256) {
            const double v = (double)D[(int64_t)r * M.ld + c];
            s += v * v;
        }
    __shared__ double red[4];
    s = wave_sum_f64(s);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) M.npartd[blockIdx.x] = 4.0 * (red[0] + red[1] + red[2] + red[3]);
}

// the sum over the workgroups: stat[3]; REDUCTION_GIVEN_UP for a factor whose T is not its own
__global__ __launch_bounds__(64) void dir_dev_sum_kernel(const DirMat *mats) {
    const DirMat M = mats[blockIdx.x];
    double dev = 0.0;
#pragma unroll
    for (int i = 0; i < NORM_WGS / 64; ++i) dev += 64 * i + (int)threadIdx.x < M.n ? M.npartd[64 * i + (int)threadIdx.x] : 0.0;
    dev = wave_sum_f64(dev);
    if (threadIdx.x == 0) M.stat[3] = M.n > TD_SMALL && M.chain < M.n - 1 && chip_load(chip_flags(M), 0) != 0 ? REDUCTION_GIVEN_UP : dev;
}

// Per column: sums of q fq, fq^2 and q^2 over the rows of part blockIdx.y.
__global__ __launch_bounds__(256) void dir_rayleigh_kernel(const DirMat *mats, int again) {
    const DirMat M = mats[blockIdx.z];
    const int c = blockIdx.x * 256 + threadIdx.x;
    if (c >= M.n || (int)blockIdx.y >= M.n || (again && !corrected(M))) return;
    const global_ptr<const float> Q = as_global((const float *)pick(needs_second_step(M) != (again != 0), M.Z, M.B2)) + c;
    const global_ptr<const float> FQ = as_global((const float *)pick(again, M.Q, M.B1)) + c;
    const int64_t lf = again ? M.n : M.ld;
    const int per = (M.n + NPARTS - 1) / NPARTS, r0 = blockIdx.y * per, r1 = min(M.n, r0 + per);
    double s1 = 0.0, s2 = 0.0, s3 = 0.0;
    for (int r = r0; r < r1; ++r) {
        const double q = (double)Q[(int64_t)r * M.ld], f = (double)FQ[r * lf];
        s1 = fma(q, f, s1);
        s2 = fma(f, f, s2);
        s3 = fma(q, q, s3);
    }
    double *o = M.sums + (int64_t)blockIdx.y * 3 * M.np + c;
    o[0] = s1;
    o[M.np] = s2;
    o[2 * M.np] = s3;
}
// lam64 = q^T F q / q^T q, and the factor that makes the column a unit vector; its residual is then s2 / s3 - lam^2 (the root of it
// in the place of the column's first sum, for the correction)
__global__ __launch_bounds__(256) void dir_lambda_kernel(const DirMat *mats, int again) {
    const DirMat M = mats[blockIdx.y];
    const int c = blockIdx.x * 256 + threadIdx.x;
    if (again && !corrected(M)) return;
    double res = 0.0;
    if (c < M.n) {
        double s1 = 0.0, s2 = 0.0, s3 = 0.0;
        const int parts = min(NPARTS, M.n);
        for (int p0 = 0; p0 < parts; p0 += 16) {     // sixteen parts' loads at a time
            double v[16][3];
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const double *o = M.sums + (int64_t)min(p0 + u, parts - 1) * 3 * M.np + c;
                v[u][0] = o[0];
                v[u][1] = o[M.np];
                v[u][2] = o[2 * M.np];
            }
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const bool in = p0 + u < parts;
                s1 += in ? v[u][0] : 0.0;
                s2 += in ? v[u][1] : 0.0;
                s3 += in ? v[u][2] : 0.0;
            }
        }
        const double l = s1 / s3;
        M.lam64[c] = l;
        M.te[c] = 1.0 / sqrt(s3);
        res = s2 / s3 - l * l;
        M.sums[c] = sqrt(fmax(res, 0.0));
    }
    __shared__ double red[4];
    res = wave_sum_f64(res);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = res;
    __syncthreads();
    if (threadIdx.x == 0 && (int)blockIdx.x * 256 < M.n) M.npartd[NORM_WGS + blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}

// s (F Q - Q diag(lam)), s the power of two that brings its norm into [1, 2), for the factors that are to be corrected: into the caller's Q
__global__ __launch_bounds__(256) void dir_residual_kernel(const DirMat *mats) {
    const DirMat M = mats[blockIdx.y];
    const int n = M.n;
    if (n <= TD_SMALL) return;
    const int lane = threadIdx.x & 63, nr = (n + 255) / 256;
    const double res = wave_sum_f64(lane < nr ? M.npartd[NORM_WGS + lane] : 0.0);
    const bool fix = M.tsum[0] >= CORRECT_FROM && res > 1e-200 && res < 1e200;
    const double s = fix ? ldexp(1.0, -ilogb(sqrt(res))) : 0.0;
    if (blockIdx.x == 0 && threadIdx.x == 0) M.tsum[1] = s;
    if (!fix) return;
    const global_ptr<const float> Q = as_global((const float *)orthonormal_q(M));
    const global_ptr<const float> FQ = as_global((const float *)M.B1);
    const global_ptr<const double> lam = as_global((const double *)M.lam64);
    const global_ptr<float> R = as_global(M.Q);
    for (int r = blockIdx.x; r < n; r += gridDim.x)
        for (int c = threadIdx.x; c < n; c += 256) {
            const int64_t i = (int64_t)r * M.ld + c;
            R[(int64_t)r * n + c] = (float)(s * fma(-lam[c], (double)Q[i], (double)FQ[i]));
        }
}

// perm[rank] = index of the rank-th smallest Rayleigh quotient (ties and NaNs by index: always a permutation)
__global__ __launch_bounds__(256) void dir_rank_kernel(const DirMat *mats) {
    __shared__ float chunk[256];
    __shared__ int part[256];
    const DirMat M = mats[blockIdx.y];
    const int n = M.n, ii = threadIdx.x & (RANK_IPB - 1), js = threadIdx.x / RANK_IPB, i = blockIdx.x * RANK_IPB + ii;
    if ((int)blockIdx.x * RANK_IPB >= n) return;
    if (blockIdx.x == 0 && threadIdx.x < 64) {     // the residual of the whole factor, for the host
        const int lane = threadIdx.x, nr = (n + 255) / 256;
        double res = lane < nr ? M.npartd[NORM_WGS + lane] : 0.0;
        res = wave_sum_f64(res);
        if (lane == 0) M.stat[2] = res;
    }
    const float li = i < n ? (float)M.lam64[i] : 0.f;
    const bool nan_i = li != li;
    int rank = 0;
    for (int j0 = 0; j0 < n; j0 += 256) {
        __syncthreads();
        chunk[threadIdx.x] = j0 + (int)threadIdx.x < n ? (float)M.lam64[j0 + threadIdx.x] : 0.f;
        __syncthreads();
        const int cnt = min(256, n - j0);
        for (int k = js; k < cnt; k += 256 / RANK_IPB) {
            const float lj = chunk[k];
            const int j = j0 + k;
            const bool nan_j = lj != lj;
            rank += nan_i ? (!nan_j || j < i) : (!nan_j && ((lj < li) || (lj == li && j < i)));
        }
    }
    part[threadIdx.x] = rank;
    __syncthreads();
    if (js == 0 && i < n) {
        int total = 0;
        for (int t = 0; t < 256 / RANK_IPB; ++t) total += part[t * RANK_IPB + ii];
        M.perm[total] = i;
        M.lam[total] = li;
    }
}
// the caller's Q (columns in ascending order of the eigenvalues); NaNs for a factor that was not finite
__global__ __launch_bounds__(256) void dir_gather_kernel(const DirMat *mats) {
    const DirMat M = mats[blockIdx.y];
    const int n = M.n;
    const bool bad = !(M.stat[0] + M.stat[1] < 1e300);
    const float nan = __uint_as_float(0x7fc00000u);
    const global_ptr<const float> S = as_global((const float *)final_q(M));
    const global_ptr<float> Q = as_global(M.Q);
    const global_ptr<const double> unit = as_global((const double *)M.te);
    const global_ptr<const int> perm = as_global((const int *)M.perm);
    for (int r = blockIdx.x; r < n; r += gridDim.x)
        for (int c = threadIdx.x; c < n; c += 256) {
            const int p = perm[c];
            Q[(int64_t)r * n + c] = bad ? nan : S[(int64_t)r * M.ld + p] * (float)unit[p];
        }
    if (bad && blockIdx.x == 0)
        for (int c = threadIdx.x; c < n; c += 256) M.lam[c] = nan;
}

// ---- host side -------------------------------------------------------------------------------------------------
struct DirSize { int n, np, ld, nb; };
DirSize dir_size(int n) {
    DirSize s;
    s.n = n;
    s.nb = (n + TB - 1) / TB;
    // the chain's kernels take whole tiles; the register kernels and the products look at n alone
    s.np = n > TD_SMALL ? s.nb * TB : (n + 15) / 16 * 16;
    s.ld = s.np > 64 ? s.np + 32 : s.np;         // not a multiple of 128: rows of one tile then start in different channels
    return s;
}

// Carves a factor's buffers out of `p` (null: sizes only); returns the bytes.
size_t dir_layout(const DirSize &s, char *p, DirMat *M) {
    size_t at = 0;
    auto take = [&](size_t bytes) { char *r = p + at; at += kfac_align_up(bytes, 256); return r; };
    const size_t mat = (size_t)s.np * s.ld * sizeof(float);
    DirMat d{};
    d.A = (float *)take(mat);
    d.Z = (float *)take(mat);
    d.B1 = (float *)take(2 * mat);
    d.B2 = d.B1 + (size_t)s.np * s.ld;
    if (s.n > TD_SMALL) {
        d.panel = (float *)take((size_t)3 * NB * s.ld * sizeof(float));
        d.apan = (float *)take((size_t)(NB + 1) * s.np * sizeof(float));
        d.part = (float *)take((size_t)2 * s.nb * s.np * sizeof(float));
        d.dots = (float *)take((size_t)2 * s.nb * 2 * NB * sizeof(float));
        d.tsum = (double *)take((size_t)s.nb * (s.nb + 1) * sizeof(double));
        d.acol = (float *)take((size_t)2 * s.np * sizeof(float));
        d.npart = (float *)take((size_t)2 * (s.np / RB) * sizeof(float));
    }
    d.tau = (float *)take((size_t)s.np * sizeof(float));
    d.d = (double *)take((size_t)s.np * sizeof(double));
    d.e = (double *)take((size_t)s.np * sizeof(double));
    d.td = (double2 *)take((size_t)s.np * sizeof(double2));
    d.te = (double *)take((size_t)s.np * sizeof(double));
    d.lam64 = (double *)take((size_t)s.np * sizeof(double));
    d.sums = (double *)take((size_t)std::min(NPARTS, s.n) * 3 * s.np * sizeof(double));
    d.npartd = (double *)take((size_t)2 * NORM_WGS * sizeof(double));
    if (s.n > TD_SMALL) d.Tm = (float *)take((size_t)s.nb * WY * WY * sizeof(float));
    d.perm = (int *)take((size_t)s.np * sizeof(int));
    d.ord = (int *)take((size_t)s.np * sizeof(int));
    if (M) {
        d.n = s.n; d.np = s.np; d.ld = s.ld; d.nb = s.nb;
        *M = d;
    }
    return at;
}

struct DirPlan {
    std::vector<DirMat> mats;
    std::vector<unsigned> tab;            // all tables, one after another
    struct Range { unsigned at, count; };
    int steps = 0;                        // of the reduction chain
    std::vector<ChipLaunch> chip;         // launches of the reduction on the chip
    std::vector<Range> tiles, rows;       // per panel
    std::vector<double> parts;            // per panel: partial products that its row blocks add up (64 rows each)
    std::vector<int> small[4];            // factors per register kernel: up to 64, 128, 192, 256
    unsigned small_at[4] = {0, 0, 0, 0};
    Range values{0, 0}, apply{0, 0}, gram{0, 0}, wyu{0, 0}, wyy{0, 0}, wys{0, 0}, wyz{0, 0}, lower{0, 0}, full{0, 0};
    int wy_steps = 0, nmax = 0, lead = 0;     // lead: the widest factor
    bool any_split = false, any_plain = false;
};

unsigned pack(int m, int I, int J) { return (unsigned)m << 14 | (unsigned)I << 7 | (unsigned)J; }

void dir_tables(DirPlan &P, int capacity) {
    const int nm = (int)P.mats.size();
    std::vector<int> order(nm);
    for (int i = 0; i < nm; ++i) order[i] = i;
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return P.mats[a].n > P.mats[b].n; });
    auto begin = [&](DirPlan::Range &r) { r.at = (unsigned)P.tab.size(); };
    auto end = [&](DirPlan::Range &r) { r.count = (unsigned)P.tab.size() - r.at; };
    P.nmax = nm ? P.mats[order[0]].n : 0;
    P.lead = nm ? order[0] : 0;
    const int widest = chip_widest(capacity);      // as many columns by the chain of launches as it takes to fit the chip
    for (auto &M : P.mats) {
        M.chain = (short)(M.n > TD_SMALL && M.n > widest ? (M.n - widest + NB - 1) / NB * NB : 0);
        P.steps = std::max<int>(P.steps, M.chain);
    }
    for (auto &M : P.mats) M.off = P.steps - M.chain;
    if (P.steps > 0) {
        const int npanel = P.steps / NB + 1;       // the last one: the update by the panel before it
        P.tiles.resize(npanel);
        P.rows.resize(npanel);
        P.parts.assign(npanel, 0.0);
        for (int q = 0; q < npanel; ++q) {
            begin(P.tiles[q]);
            for (int m : order) {
                const DirMat &M = P.mats[m];
                const int j = q * NB - M.off;
                if (M.chain == 0 || j < 0 || j > M.n - 1) continue;
                for (int I = j / TB; I < M.nb; ++I)
                    for (int J = j / TB; J <= I; ++J) P.tab.push_back(pack(m, I, J));
            }
            end(P.tiles[q]);
            begin(P.rows[q]);
            for (int m : order) {
                const DirMat &M = P.mats[m];
                const int j = q * NB - M.off;
                if (M.chain == 0 || j < 0 || j > M.n - 1) continue;
                for (int r = j / TB * 2; r < 2 * M.nb; ++r) P.tab.push_back(pack(m, 0, r));
                P.parts[q] += 2.0 * (M.nb - j / TB) * (M.nb - j / TB);
            }
            end(P.rows[q]);
        }
    }
    std::vector<ChipFactor> left;
    for (int m : order)
        if (P.mats[m].n > TD_SMALL && P.mats[m].chain < P.mats[m].n - 1) left.push_back(ChipFactor{m, P.mats[m].n, P.mats[m].chain, 0});
    std::vector<ChipJob> jobs;
    chip_plan(left, capacity, jobs, P.chip);
    for (auto &L : P.chip) L.at = (unsigned)(P.tab.size() + L.at * sizeof(ChipJob) / sizeof(unsigned));
    const size_t at = P.tab.size();
    P.tab.resize(at + jobs.size() * sizeof(ChipJob) / sizeof(unsigned));
    if (!jobs.empty()) memcpy(P.tab.data() + at, jobs.data(), jobs.size() * sizeof(ChipJob));
    for (int m : order) {
        const int n = P.mats[m].n;
        if (n <= TD_SMALL) P.small[n <= 64 ? 0 : n <= 128 ? 1 : n <= 192 ? 2 : 3].push_back(m);
    }
    for (int k = 0; k < 4; ++k) {
        P.small_at[k] = (unsigned)P.tab.size();
        for (int m : P.small[k]) P.tab.push_back((unsigned)m);
    }
    begin(P.values);
    for (int m : order)
        for (int c = 0; c < (P.mats[m].n + 63) / 64; ++c) P.tab.push_back(pack(m, 0, c));
    end(P.values);
    begin(P.apply);
    for (int m : order)
        if (P.mats[m].n <= TD_SMALL)
            for (int c = 0; c < (P.mats[m].n + 15) / 16; ++c) P.tab.push_back(pack(m, 0, c));
    end(P.apply);
    auto wy = [&](DirPlan::Range &r, auto f) {
        begin(r);
        for (int m : order)
            if (P.mats[m].n > TD_SMALL) f(m, P.mats[m].nb);
        end(r);
    };
    wy(P.gram, [&](int m, int nb) { P.wy_steps = std::max(P.wy_steps, nb); for (int b = 0; b < nb; ++b) P.tab.push_back(pack(m, 0, b)); });
    wy(P.wyu, [&](int m, int nb) { for (int b = 0; b < nb; ++b) for (int c = b; c < nb; ++c) P.tab.push_back(pack(m, b, c)); });
    wy(P.wyy, [&](int m, int nb) { for (int k = 0; k * WY_K < P.mats[m].n; ++k) for (int c = 0; c < nb; ++c) P.tab.push_back(pack(m, k, c)); });
    wy(P.wys, [&](int m, int nb) { for (int c = 0; c < nb; ++c) P.tab.push_back(pack(m, 0, c)); });
    wy(P.wyz, [&](int m, int nb) { for (int r = 0; r < nb; ++r) for (int c = 0; c < nb; ++c) P.tab.push_back(pack(m, r, c)); });
    begin(P.lower);
    for (int m : order)
        for (int I = 0; I < P.mats[m].nb; ++I)
            for (int J = 0; J <= I; ++J) P.tab.push_back(pack(m, I, J));
    end(P.lower);
    begin(P.full);
    for (int m : order)
        for (int I = 0; I < P.mats[m].nb; ++I)
            for (int J = 0; J < P.mats[m].nb; ++J) P.tab.push_back(pack(m, I, J));
    end(P.full);
}

// Entries dir_tables() makes, without making them.
size_t dir_table_bound(int batch, const int *d) {
    size_t t = 0;
    for (int i = 0; i < batch; ++i) {
        const size_t nb = (d[i] + TB - 1) / TB;
        t += 4 * nb * nb + 16 * nb + 16 + (size_t)(d[i] + 15) / 16 + (d[i] + 63) / 64;
        if (d[i] > TD_SMALL) t += 4 * (nb * (nb + 1) * (nb + 2) / 6) + 4 * nb * (nb + 1) + 8;   // four panels per block
    }
    return t;
}

// The factors of a call, on the context's stream.
struct DirRun {
    DirPlan P;
    const DirMat *dm;
    const unsigned *tab;
    double cube = 0.0, square = 0.0;
};

void enqueue_copy(kfac_ctx *ctx, const DirRun &R) {
    const DirPlan &P = R.P;
    const hipStream_t st = ctx->stream;
    const unsigned batch = (unsigned)P.mats.size();
    KfacProfScope prof(ctx, KC_EIG_MISC, 0.0, 8.0 * R.square, st);
    const unsigned wgs = (unsigned)std::min(NORM_WGS, P.nmax);
    hipLaunchKernelGGL(dir_norm_kernel, dim3(wgs, batch), dim3(256), 0, st, R.dm);
    hipLaunchKernelGGL(dir_order_kernel, dim3((P.nmax + RANK_IPB - 1) / RANK_IPB, batch), dim3(256), 0, st, R.dm);
    hipLaunchKernelGGL(dir_copy_kernel, dim3(P.nmax > TD_SMALL ? wgs : 1, batch), dim3(256), 0, st, R.dm);
}

void enqueue_small(kfac_ctx *ctx, const DirRun &R) {
    const DirPlan &P = R.P;
    const hipStream_t st = ctx->stream;
    for (int k = 0; k < 4; ++k) {
        if (P.small[k].empty()) continue;
        const dim3 grid((unsigned)P.small[k].size());
        const int *list = (const int *)(R.tab + P.small_at[k]);
        double fl = 0.0;
        for (int m : P.small[k]) fl += 4.0 / 3.0 * std::pow((double)P.mats[m].n, 3);
        KfacProfScope prof(ctx, KC_EIG_SMALL, fl, 0.0, st);
        switch (k) {
            case 0: hipLaunchKernelGGL(dir_td_small_kernel<16>, grid, dim3(256), 0, st, R.dm, list); break;
            case 1: hipLaunchKernelGGL(dir_td_small_kernel<32>, grid, dim3(512), 0, st, R.dm, list); break;
            case 2: hipLaunchKernelGGL(dir_td_small_kernel<48>, grid, dim3(768), 0, st, R.dm, list); break;
            default: hipLaunchKernelGGL(dir_td_small_kernel<64>, grid, dim3(1024), 0, st, R.dm, list); break;
        }
    }
}

void enqueue_update(kfac_ctx *ctx, const DirRun &R, int t) {
    const DirPlan::Range tiles = R.P.tiles[t / NB];
    KfacProfScope prof(ctx, KC_EIG_REDUCE_GEMM, 2.0 * 2.0 * NB * TB * TB * tiles.count, 8.0 * TB * TB * tiles.count, ctx->stream);
    if (tiles.count) hipLaunchKernelGGL(dir_update_kernel, dim3(tiles.count), dim3(NTHREADS), 0, ctx->stream, R.dm, R.tab + tiles.at, t);
}

void enqueue_step(kfac_ctx *ctx, const DirRun &R, int t) {
    const hipStream_t st = ctx->stream;
    const DirPlan::Range tiles = R.P.tiles[t / NB], rows = R.P.rows[t / NB];
    if (t % NB == 0) {
        if (t > 0) enqueue_update(ctx, R, t);
        KfacProfScope prof(ctx, KC_EIG_REDUCE_VEC, 0.0, 8.0 * RB * (NB + 1) * rows.count, st);
        hipLaunchKernelGGL(dir_column_kernel, dim3(rows.count), dim3(RB), 0, st, R.dm, R.tab + rows.at, t);
    }
    const double fl = 4.0 * TB * TB * tiles.count;
    {
        KfacProfScope prof(ctx, KC_EIG_REDUCE_MV, fl, fl, st);
        hipLaunchKernelGGL(dir_symv_kernel, dim3(tiles.count), dim3(256), 0, st, R.dm, R.tab + tiles.at, t);
    }
    // the partial products, the panel's columns so far, column t + 1 and x read; v (three times), w and the next x written
    KfacProfScope prof(ctx, KC_EIG_REDUCE_VEC, 0.0, 4.0 * RB * (R.P.parts[t / NB] + rows.count * (2.0 * (t % NB) + 7.0)), st);
    hipLaunchKernelGGL(dir_vector_kernel, dim3(rows.count), dim3(256), 0, st, R.dm, R.tab + rows.at, t);
}

int enqueue_reduction(kfac_ctx *ctx, const DirRun &R) {
    const DirPlan &P = R.P;
    const hipStream_t st = ctx->stream;
    const dim3 per_mat((unsigned)std::min(NORM_WGS, P.nmax), (unsigned)P.mats.size());
    for (int t = 0; t < P.steps; ++t) enqueue_step(ctx, R, t);
    if (P.steps > 0) {
        enqueue_update(ctx, R, P.steps);
        KfacProfScope prof(ctx, KC_EIG_REDUCE_VEC, 0.0, 4.0 * R.square, st);
        hipLaunchKernelGGL(dir_mirror_kernel, per_mat, dim3(256), 0, st, R.dm);
        // A cooperative launch goes to a queue of its own.  While it waits there for this stream, every launch on this stream takes several times
        // as long, and the chain is thousands of them: 6145 wide 122 ms, 8192 284, with this wait 71.5 and 157 (the chain to the end 98.8 and 188).
        if (!P.chip.empty()) KFAC_HIP_CHECK(hipStreamSynchronize(st));
    }
    for (const ChipLaunch &L : P.chip) {
        const DirMat *dm = R.dm;
        const ChipJob *jobs = (const ChipJob *)(R.tab + L.at);
        int count = L.jobs, lead = P.lead, polls = ctx->chip_polls;
        void *args[] = {&dm, &jobs, &count, &lead, &polls};
        // of three multiplications and additions per element, one belongs to the product and two to the update
        KfacProfScope product(ctx, KC_EIG_REDUCE_MV, L.flops / 3.0, L.bytes / 3.0, st, 1.0 / 3.0);
        KfacProfScope update(ctx, KC_EIG_REDUCE_GEMM, L.flops / 1.5, L.bytes / 1.5, st, 2.0 / 3.0);
        const void *kernel = L.threads == CHIP_WIDE ? (const void *)dir_chip_kernel<CHIP_WIDE> : (const void *)dir_chip_kernel<CHIP_NARROW>;
        if (hipLaunchCooperativeKernel(kernel, dim3((unsigned)L.wgs), dim3((unsigned)L.threads), args, 0, st) != hipSuccess) {
            (void)hipGetLastError();
            return KFAC_EIG_REFUSED;
        }
    }
    if (P.nmax > TD_SMALL) {
        KfacProfScope prof(ctx, KC_EIG_REDUCE_VEC, 0.0, 2.0 * R.square, st);
        hipLaunchKernelGGL(dir_clear_kernel, per_mat, dim3(256), 0, st, R.dm);
    }
    return KFAC_OK;
}

int enqueue_finish(kfac_ctx *ctx, const DirRun &R) {
    const DirPlan &P = R.P;
    const hipStream_t st = ctx->stream;
    const unsigned batch = (unsigned)P.mats.size();
    const dim3 per_mat((unsigned)std::min(NORM_WGS, P.nmax), batch);
    const DirMat *dm = R.dm;
    const unsigned *tab = R.tab;
    {
        // fp64: per eigenvalue 60 Sturm counts of two FMAs a row (bisection to its last bits), per eigenvector five recurrences of a
        // division, i.e. five FMAs and a few more
        KfacProfScope prof(ctx, KC_EIG_TRI, (60.0 * 4.0 + 5.0 * 12.0) * R.square, 0.0, st);
        hipLaunchKernelGGL(dir_scale_t_kernel, dim3(batch), dim3(256), 0, st, dm);
        // sixteen lanes per eigenvalue do 9/4 of the work of four in 4/7 of the passes: right where four leave the chip idle
        if (P.values.count <= BIS_WIDE_MAX)
            hipLaunchKernelGGL(dir_bisect_kernel<16>, dim3(4 * P.values.count), dim3(256), 0, st, dm, tab + P.values.at);
        else
            hipLaunchKernelGGL(dir_bisect_kernel<4>, dim3(P.values.count), dim3(256), 0, st, dm, tab + P.values.at);
        hipLaunchKernelGGL(dir_vectors_kernel, dim3(P.values.count), dim3(64), 0, st, dm, tab + P.values.at);
    }
    {
        KfacProfScope prof(ctx, KC_EIG_BACK, 2.0 * R.cube, 0.0, st);
        if (P.apply.count) hipLaunchKernelGGL(dir_apply_kernel, dim3(P.apply.count), dim3(256), 0, st, dm, tab + P.apply.at);
        if (P.wy_steps > 0) {
            const int lds = 2 * WY * (WY + 1) * (int)sizeof(float);
            if (lds > ctx->max_lds) return KFAC_EHIP;
            KFAC_HIP_CHECK(hipFuncSetAttribute((const void *)dir_wy_t_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, lds));
            hipLaunchKernelGGL(dir_wy_gram_kernel, dim3(P.gram.count), dim3(NTHREADS), 0, st, dm, tab + P.gram.at);
            hipLaunchKernelGGL(dir_wy_t_kernel, dim3(P.gram.count), dim3(WY * WT), lds, st, dm, tab + P.gram.at);
            hipLaunchKernelGGL(dir_wy_u_kernel, dim3(P.wyu.count), dim3(NTHREADS), 0, st, dm, tab + P.wyu.at);
            for (int s = 0; s < P.wy_steps; ++s) {
                hipLaunchKernelGGL(dir_wy_y_kernel, dim3(P.wyy.count), dim3(NTHREADS), 0, st, dm, tab + P.wyy.at, s);
                hipLaunchKernelGGL(dir_wy_sum_kernel, dim3(P.wys.count), dim3(256), 0, st, dm, tab + P.wys.at, s);
                hipLaunchKernelGGL(dir_wy_z_kernel, dim3(P.wyz.count), dim3(NTHREADS), 0, st, dm, tab + P.wyz.at, s);
            }
        }
    }
    {
        KfacProfScope prof(ctx, KC_EIG_POST, 5.0 * R.cube, 0.0, st);
        const dim3 lo(P.lower.count), fu(P.full.count), b(NTHREADS);
        const unsigned *tl = tab + P.lower.at, *tf = tab + P.full.at;
        for (int second = 0; second < 2; ++second) {
            if (P.any_split) hipLaunchKernelGGL((dir_product_kernel<ORTH, true>), lo, b, 0, st, dm, tl, second);
            if (P.any_plain) hipLaunchKernelGGL((dir_product_kernel<ORTH, false>), lo, b, 0, st, dm, tl, second);
            if (!second) {
                hipLaunchKernelGGL(dir_dev_kernel, per_mat, dim3(256), 0, st, dm);
                hipLaunchKernelGGL(dir_dev_sum_kernel, dim3(batch), dim3(64), 0, st, dm);
            }
            if (P.any_split) hipLaunchKernelGGL((dir_product_kernel<STEP, true>), fu, b, 0, st, dm, tf, second);
            if (P.any_plain) hipLaunchKernelGGL((dir_product_kernel<STEP, false>), fu, b, 0, st, dm, tf, second);
        }
        hipLaunchKernelGGL((dir_product_kernel<TIMES_F, false>), fu, b, 0, st, dm, tf, 0);
    }
    auto quotients = [&](int again) {
        KfacProfScope prof(ctx, KC_EIG_MISC, 0.0, 16.0 * R.square, st);
        hipLaunchKernelGGL(dir_rayleigh_kernel, dim3((P.nmax + 255) / 256, std::min(NPARTS, P.nmax), batch), dim3(256), 0, st, dm, again);
        hipLaunchKernelGGL(dir_lambda_kernel, dim3((P.nmax + 255) / 256, batch), dim3(256), 0, st, dm, again);
    };
    quotients(0);
    if (P.nmax > TD_SMALL) {      // which factors are corrected is known on the device only: no work of it is credited
        {
            KfacProfScope prof(ctx, KC_EIG_POST, 0.0, 0.0, st);
            const dim3 lo(P.lower.count), fu(P.full.count), b(NTHREADS);
            const unsigned *tl = tab + P.lower.at, *tf = tab + P.full.at;
            hipLaunchKernelGGL(dir_residual_kernel, per_mat, dim3(256), 0, st, dm);
            hipLaunchKernelGGL((dir_product_kernel<TURN, true>), lo, b, 0, st, dm, tl, 0);
            hipLaunchKernelGGL((dir_product_kernel<FOLLOW, true>), dim3(fu.x, 2), b, 0, st, dm, tf, 0);
        }
        quotients(1);
    }
    {
        KfacProfScope prof(ctx, KC_EIG_MISC, 0.0, 0.0, st);
        hipLaunchKernelGGL(dir_rank_kernel, dim3((P.nmax + RANK_IPB - 1) / RANK_IPB, batch), dim3(256), 0, st, dm);
        hipLaunchKernelGGL(dir_gather_kernel, per_mat, dim3(256), 0, st, dm);
    }
    KFAC_HIP_CHECK(hipGetLastError());
    return KFAC_OK;
}

}  // namespace

size_t kfac_eig_direct_ws_bytes(int batch, const int *d) {
    size_t need = kfac_align_up((size_t)batch * sizeof(DirMat), 256) + kfac_align_up((size_t)batch * 4 * sizeof(double), 256) +
                  kfac_align_up(dir_table_bound(batch, d) * sizeof(unsigned), 256);
    for (int i = 0; i < batch; ++i) need += dir_layout(dir_size(d[i]), nullptr, nullptr);
    return need;
}

// What a call takes, in seconds:
//  - the widest factor's columns one after another, and the arithmetic and the traffic of all factors;
//  - the columns of the register kernels, which run before the chip, one width after another;
//  - where the widest goes in one launch, the launches of those that find no place in the first (at most CHIP_JOBS factors, of narrow workgroups);
//  - what columns by the chain of launches take on top, by their number and the bytes of the trailing matrices.
// Measured, and by this, in ms: one factor of ReLU features 257 wide 1.18, 1.20, 577 2.50, 2.34, 1153 5.28, 5.09, 2100 9.96, 9.94, 4609 31.1, 31.6, 6145 71.5, 71.9,
// 8192 156.9, 153.3; fifty of 300 1.89, 1.85, a hundred and thirty 4.61, 4.61, sixty-five of 257 2.39, 2.49, two hundred 5.62, 5.12, eighty of 577 8.16, 8.05,
// forty of 1100 16.0, 14.7, six of 2305 21.0, 20.6; one of 257 beside twenty of 250 2.04, 1.94; without cooperative launches 1153 11.7, 10.4, 4609 58.5, 59.7.
// Over 57 calls of 1 to 200 factors 5 % off, 13 at the most.  (Without the last three lines, and with the terms of the first alone, 29 % and 68: crowds of narrow
// factors passed for cheap, and were decomposed where sweeps take half the time.)  Factors whose eigenvectors are corrected take 4 to 12 % more,
// which only the decomposition shows.
double kfac_eig_direct_seconds(int capacity, int batch, const int *d) {
    const int widest = chip_widest(capacity), cus = std::min(capacity, CHIP_WGS);
    int nmax = 0, chain = 0, narrow = 0, small[4] = {0, 0, 0, 0};
    double n2 = 0.0, n3 = 0.0, chain3 = 0.0, launches = 0.0;
    for (int i = 0; i < batch; ++i) {
        const double cube = (double)d[i] * d[i] * d[i];
        nmax = std::max(nmax, d[i]);
        n3 += cube;
        if (d[i] <= TD_SMALL) {
            int &w = small[(d[i] - 1) / 64];
            w = std::max(w, d[i]);
            continue;
        }
        n2 += (double)d[i] * d[i];
        if (d[i] > widest) {
            chain = std::max(chain, d[i] - widest);
            chain3 += cube - (double)widest * widest * widest;
        } else if (d[i] - 1 <= CHIP_WHOLE) {
            narrow = std::max(narrow, d[i]);
            launches += 1.0 / std::min(CHIP_JOBS, std::max(1, cus * (CHIP_WIDE / CHIP_NARROW) / chip_need(d[i] - 1, CHIP_NARROW)));
        }
    }
    if (nmax == 0) return 0.0;
    if (nmax <= TD_SMALL) return 60e-6 + 4.6e-6 * nmax + 1.5e-13 * n3;
    double t = 320e-6 + (nmax - 1 <= CHIP_WHOLE ? 3.41e-6 : 3.89e-6) * nmax + 7.7e-11 * n2 + 1.2e-13 * n3 + 4.5e-6 * chain + 7.5e-14 * chain3;
    for (int w : small) t += 2.8e-6 * w;
    if (nmax - 1 <= CHIP_WHOLE) t += 3.24e-6 * narrow * std::max(0.0, std::ceil(launches - 1e-9) - 1.0);
    return t;
}

// All factors of the call by the direct route; stat (pinned host memory): four doubles per factor, off^2 and diag^2 of F, the
// squared residual ||F Q - Q diag(lam)||_F^2 and ||I - Q^T Q||_F^2 before it was orthogonalised.  Waits for the result.
// diag_tol: off(F)_F / ||F||_F up to which a factor counts as diagonal.  go_on (may be null): called, if a factor is wider than
// KFAC_EIG_REG, once off^2 and diag^2 of all factors are in stat; if it returns false, nothing more is done (KFAC_EIG_STOPPED).
// capacity: workgroups that the reduction on the chip may use at once; with none, everything is reduced by the chain of launches.
static int direct_by(kfac_ctx *ctx, int capacity, int batch, const float *const *F, const int *d, float *const *Q, float *const *lam,
                     double diag_tol, double *stat, const std::function<bool()> *go_on) {
    if (kfac_eig_direct_ws_bytes(batch, d) > ctx->ws_bytes) return KFAC_EWORKSPACE;
    DirMat *d_mats = (DirMat *)ctx->ws;
    double *d_stat = (double *)(ctx->ws + kfac_align_up((size_t)batch * sizeof(DirMat), 256));
    unsigned *d_tab = (unsigned *)((char *)d_stat + kfac_align_up((size_t)batch * 4 * sizeof(double), 256));
    char *p = (char *)d_tab + kfac_align_up(dir_table_bound(batch, d) * sizeof(unsigned), 256);
    DirRun R;
    R.dm = d_mats;
    R.tab = d_tab;
    R.P.mats.resize(batch);
    for (int i = 0; i < batch; ++i) {
        DirMat &M = R.P.mats[i];
        p += dir_layout(dir_size(d[i]), p, &M);
        M.F = F[i];
        M.Q = Q[i];
        M.lam = lam[i];
        M.stat = d_stat + 4 * i;
        M.diag_tol2 = diag_tol * diag_tol;
        M.split = d[i] >= KFAC_EIG_SPLIT_MIN;
        (M.split ? R.P.any_split : R.P.any_plain) = true;
        R.cube += (double)d[i] * d[i] * d[i];
        R.square += (double)d[i] * d[i];
    }
    R.P.tab.reserve(dir_table_bound(batch, d));
    dir_tables(R.P, capacity);
    if (R.P.tab.size() > dir_table_bound(batch, d)) return KFAC_EWORKSPACE;
    KFAC_CHECK(kfac_upload(ctx, d_mats, R.P.mats.data(), R.P.mats.size() * sizeof(DirMat)));
    KFAC_CHECK(kfac_upload(ctx, d_tab, R.P.tab.data(), R.P.tab.size() * sizeof(unsigned)));
    enqueue_copy(ctx, R);
    const bool ask = go_on && R.P.nmax > TD_SMALL;
    if (ask) {   // the register kernels run while the host decides
        KFAC_HIP_CHECK(hipMemcpyAsync(stat, d_stat, (size_t)batch * 4 * sizeof(double), hipMemcpyDeviceToHost, ctx->stream));
        KFAC_HIP_CHECK(hipEventRecord(ctx->ev_group[0], ctx->stream));
    }
    enqueue_small(ctx, R);
    if (ask) {
        const bool waited = hipEventSynchronize(ctx->ev_group[0]) == hipSuccess;
        if (!waited || !(*go_on)()) {
            if (hipStreamSynchronize(ctx->stream) != hipSuccess || !waited) return KFAC_EHIP;
            return KFAC_EIG_STOPPED;
        }
    }
    int rc = enqueue_reduction(ctx, R);
    if (rc == KFAC_OK) rc = enqueue_finish(ctx, R);
    if (rc == KFAC_OK && hipMemcpyAsync(stat, d_stat, (size_t)batch * 4 * sizeof(double), hipMemcpyDeviceToHost, ctx->stream) != hipSuccess)
        rc = KFAC_EHIP;
    if (hipStreamSynchronize(ctx->stream) != hipSuccess) rc = KFAC_EHIP;    // on an error, too: no kernel of this call is in flight after the return
    return rc;
}

int kfac_launch_eig_direct(kfac_ctx *ctx, int batch, const float *const *F, const int *d, float *const *Q, float *const *lam,
                           double diag_tol, double *stat, const std::function<bool()> *go_on) {
    int rc = direct_by(ctx, ctx->coop_wgs, batch, F, d, Q, lam, diag_tol, stat, go_on);
    if (rc == KFAC_EIG_REFUSED) return direct_by(ctx, 0, batch, F, d, Q, lam, diag_tol, stat, nullptr);
    if (rc != KFAC_OK) return rc;
    std::vector<int> which, dd;
    std::vector<const float *> FF;
    std::vector<float *> QQ, ll;
    for (int i = 0; i < batch; ++i)
        if (stat[4 * i + 3] == REDUCTION_GIVEN_UP) {
            which.push_back(i);
            dd.push_back(d[i]);
            FF.push_back(F[i]);
            QQ.push_back(Q[i]);
            ll.push_back(lam[i]);
        }
    if (which.empty()) return KFAC_OK;
    std::vector<double> all(stat, stat + (size_t)4 * batch);
    rc = direct_by(ctx, 0, (int)which.size(), FF.data(), dd.data(), QQ.data(), ll.data(), diag_tol, stat, nullptr);
    if (rc != KFAC_OK) return rc;
    for (size_t k = 0; k < which.size(); ++k) std::copy(stat + 4 * k, stat + 4 * k + 4, all.begin() + 4 * which[k]);
    std::copy(all.begin(), all.end(), stat);
    return KFAC_OK;
}

void kfac_limit_chip(kfac_ctx *ctx, int workgroups, int polls) {
    ctx->coop_wgs = workgroups;
    ctx->chip_polls = polls;
}
