// Entry point of the batched symmetric eigensolver (Sec. IV-A; Algorithm 1, step 2): which factors of a call are decomposed directly
// (eig_direct.hip) and which by Jacobi sweeps (eig.hip).
//
// The direct decomposition costs the same for every factor of a size.  Jacobi sweeps cost by how far the factor is from diagonal in
// the basis they start from: none from the eigenvectors of a factor that has not moved since (7 ms at 4609, where the direct
// decomposition takes 30), four and more after a running average moved by 5 % (88 ms).  So with a start basis, that distance is
// estimated first (probe kernels below: 18 us at 145, 64 at 2100, and a wait), and the sweeps take the factors with which the call is cheaper.  Without one, it
// is off(F)_F, which the direct route forms anyway: running averages that are still diagonal need no sweep (0.55 ms at 577, 1.4 at
// 2100, in place of 2.4 and 9.3), and a very loose tol needs few.
#include <algorithm>
#include <climits>
#include <cmath>
#include <functional>
#include <vector>
#include "kfac_internal.h"

namespace {

constexpr int PC = 64;        // columns of the start basis that are looked at: the last PTOP (those of the largest eigenvalues, which
constexpr int PTOP = 16;      // hold half of the off-diagonal norm) and the rest spread evenly
constexpr int PR = 8;         // rows of F per workgroup
constexpr int PK = 256;       // contraction per step of a workgroup
constexpr int PV = 3 * PC + 1;   // sums per workgroup: q fq, fq^2, q^2 for every column, and its share of ||F||_F^2

struct ProbeItem {
    const float *F, *Q;
    float *S;             // [ns][PC]: the columns looked at, rows past n zero
    double *part;         // [ceil(n / PR)][PV]
    double *out;          // estimate of ||F Q - Q diag(lam)||_F^2, ||F||_F^2, share of columns more than 30 % off
    int n, ns;
};

__device__ inline int probe_column(int n, int c) { return c < PTOP ? n - 1 - c : (int)(((c - PTOP) + 0.5f) * (float)(n - PTOP) / (float)(PC - PTOP)); }

__global__ __launch_bounds__(256) void probe_gather_kernel(const ProbeItem *items) {
    const ProbeItem P = items[blockIdx.y];
    const int c = threadIdx.x & (PC - 1), col = probe_column(P.n, c);
    const global_ptr<const float> Q = as_global(P.Q);
    for (int k = blockIdx.x * 4 + (threadIdx.x >> 6); k < P.ns; k += 4 * gridDim.x)
        as_global(P.S)[(int64_t)k * PC + c] = k < P.n ? Q[(int64_t)k * P.n + col] : 0.f;
}

// F q for the PC columns and PR rows: the four waves of a workgroup share the contraction, lane = column.
__global__ __launch_bounds__(256) void probe_rows_kernel(const ProbeItem *items) {
    __shared__ __attribute__((aligned(16))) float fs[PR][PK];
    __shared__ float acc_s[4][PR][PC];
    __shared__ double sums[4][3][PC], f2s[4];
    const ProbeItem P = items[blockIdx.y];
    const int n = P.n, r0 = blockIdx.x * PR, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    if (r0 >= n) return;
    const global_ptr<const float> F = as_global(P.F), S = as_global((const float *)P.S);
    float acc[PR];
    double f2 = 0.0;
#pragma unroll
    for (int r = 0; r < PR; ++r) acc[r] = 0.f;
    for (int k0 = 0; k0 < P.ns; k0 += PK) {     // ns is a multiple of PK
        float v[PR];
#pragma unroll
        for (int r = 0; r < PR; ++r) v[r] = (r0 + r < n && k0 + tid < n) ? F[(int64_t)(r0 + r) * n + k0 + tid] : 0.f;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < PR; ++r) {
            fs[r][tid] = v[r];
            f2 += (double)v[r] * (double)v[r];
        }
        __syncthreads();
#pragma unroll 4
        for (int k = 0; k < 64; k += 4) {
            const global_ptr<const float> s = S + (int64_t)(k0 + 64 * w + k) * PC + lane;
            const float s0 = s[0], s1 = s[PC], s2 = s[2 * PC], s3 = s[3 * PC];
#pragma unroll
            for (int r = 0; r < PR; ++r) {
                const float4 f = *(const float4 *)(&fs[r][64 * w + k]);
                acc[r] = fmaf(f.x, s0, fmaf(f.y, s1, fmaf(f.z, s2, fmaf(f.w, s3, acc[r]))));
            }
        }
    }
#pragma unroll
    for (int r = 0; r < PR; ++r) acc_s[w][r][lane] = acc[r];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) f2 += __shfl_xor(f2, o, 64);
    if (lane == 0) f2s[w] = f2;
    __syncthreads();
    double s1 = 0.0, s2 = 0.0, s3 = 0.0;
#pragma unroll
    for (int r = PR / 4 * w; r < PR / 4 * (w + 1); ++r) {
        const double fq = (double)(acc_s[0][r][lane] + acc_s[1][r][lane] + acc_s[2][r][lane] + acc_s[3][r][lane]);
        const double q = r0 + r < n ? (double)S[(int64_t)(r0 + r) * PC + lane] : 0.0;
        s1 = fma(q, fq, s1);
        s2 = fma(fq, fq, s2);
        s3 = fma(q, q, s3);
    }
    sums[w][0][lane] = s1;
    sums[w][1][lane] = s2;
    sums[w][2][lane] = s3;
    __syncthreads();
    double *o = P.part + (int64_t)blockIdx.x * PV;
    if (tid < 3 * PC) o[tid] = sums[0][tid / PC][lane] + sums[1][tid / PC][lane] + sums[2][tid / PC][lane] + sums[3][tid / PC][lane];
    if (tid == 3 * PC) o[tid] = f2s[0] + f2s[1] + f2s[2] + f2s[3];
}

// One workgroup per factor: a column's residual is s2 / s3 - (s1 / s3)^2, and the columns looked at stand for all.
__global__ __launch_bounds__(256) void probe_sum_kernel(const ProbeItem *items) {
    __shared__ double tot[PV];
    const ProbeItem P = items[blockIdx.x];
    const int tid = threadIdx.x, nb = (P.n + PR - 1) / PR;
    if (tid < PV) {
        double s = 0.0;
        const double *p = P.part + tid;
#pragma unroll 8
        for (int b = 0; b < nb; ++b) s += p[(int64_t)b * PV];
        tot[tid] = s;
    }
    __syncthreads();
    if (tid >= PC) return;
    const double l = tot[tid] / tot[2 * PC + tid], raw = tot[PC + tid] / tot[2 * PC + tid] - l * l;
    double res = raw > 0.0 ? raw : 0.0;
    if (!(fabs(tot[2 * PC + tid] - 1.0) <= 1e-3) || !(raw < 1e300)) res = 1e300;     // zeros, not a number, ..: no basis to start from
    const int lost = __popcll(__ballot(tid >= PTOP && res > 0.09 * l * l));
    res *= tid < PTOP ? 1.0 : (double)(P.n - PTOP) / (double)(PC - PTOP);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) res += __shfl_xor(res, o, 64);
    if (tid == 0) {
        P.out[0] = res;
        P.out[1] = tot[3 * PC];
        P.out[2] = (double)lost / (PC - PTOP);
    }
}

// How far a factor is from diagonal in the basis it would start from.
struct StartBasis {
    double rel = -1.0;      // off(Q^T F Q)_F / ||F||_F; negative: not known
    double lost = 0.0;      // share of the columns whose residual is more than 30 % of their Rayleigh quotient
};


// The start bases of the factors listed in `which`, into start (by index of the call), which stays as it is if the workspace
// has no room.  Waits for the result.
int probe_start_bases(kfac_ctx *ctx, const std::vector<int> &which, const float *const *F, const int *d, const float *const *Q,
                      std::vector<StartBasis> &start) {
    const int m = (int)which.size();
    std::vector<ProbeItem> items(m);
    char *p = ctx->ws;
    auto take = [&](size_t bytes) { char *r = p; p += kfac_align_up(bytes, 256); return r; };
    ProbeItem *d_items = (ProbeItem *)take(m * sizeof(ProbeItem));
    double *d_out = (double *)take((size_t)3 * m * sizeof(double));
    int nmax = 0;
    for (int k = 0; k < m; ++k) {
        const int n = d[which[k]], ns = (n + PK - 1) / PK * PK;
        items[k] = ProbeItem{F[which[k]], Q[which[k]], (float *)take((size_t)ns * PC * sizeof(float)), nullptr, d_out + 3 * k, n, ns};
        items[k].part = (double *)take((size_t)((n + PR - 1) / PR) * PV * sizeof(double));
        nmax = std::max(nmax, n);
    }
    if ((size_t)(p - ctx->ws) > ctx->ws_bytes || (size_t)3 * m * sizeof(double) > ctx->pinned_bytes) return KFAC_OK;
    KFAC_CHECK(kfac_upload(ctx, d_items, items.data(), m * sizeof(ProbeItem)));
    {
        KfacProfScope prof(ctx, KC_EIG_MISC, 0.0, 0.0);
        hipLaunchKernelGGL(probe_gather_kernel, dim3((nmax + 63) / 64, m), dim3(256), 0, ctx->stream, (const ProbeItem *)d_items);
        hipLaunchKernelGGL(probe_rows_kernel, dim3((nmax + PR - 1) / PR, m), dim3(256), 0, ctx->stream, (const ProbeItem *)d_items);
        hipLaunchKernelGGL(probe_sum_kernel, dim3(m), dim3(256), 0, ctx->stream, (const ProbeItem *)d_items);
    }
    KFAC_HIP_CHECK(hipGetLastError());
    KFAC_HIP_CHECK(hipMemcpyAsync(ctx->pinned, d_out, (size_t)3 * m * sizeof(double), hipMemcpyDeviceToHost, ctx->stream));
    KFAC_HIP_CHECK(hipStreamSynchronize(ctx->stream));
    for (int k = 0; k < m; ++k) {
        const double *o = ctx->pinned + 3 * k;
        if (!(o[0] < 1e299) || !(o[1] < 1e300)) continue;
        start[which[k]].rel = o[1] > 0.0 ? std::sqrt(o[0] / o[1]) : 0.0;
        start[which[k]].lost = o[2];
    }
    return KFAC_OK;
}

// The direct route diagonalises by construction; what is left is the fp32 rounding of the reduction.  Measured through F Q: 3e-7 ||F||
// at 129 to 7e-7 at 8192 for Gram matrices, 4.5e-7 at 64 to 1.2e-6 at 8192 for dense ones with random entries.  It serves stopping
// rules down to DIRECT_TOL_MIN, and a factor that comes out further off than the caller's tol is left to Jacobi like one whose
// result is not sound; tighter rules are Jacobi's from the start, whose sweeps go on until the rotated matrix itself is that close to
// diagonal.
constexpr float DIRECT_TOL_MIN = 1e-6f;
constexpr double DIRECT_MAX_RES = 5e-6;    // measured residual / ||F||_F of a sound result
constexpr double DIRECT_MAX_DEV2 = 1e-3;   // ||I - Q^T Q||_F^2 that two Newton-Schulz steps bring below fp32 rounding

// Sweeps down to tol.  A sweep gains a factor of 8 as long as the columns of the basis still are what they were, and the last one of a
// short run more, since the sweeps converge quadratically at the end.  Over 34 factors of 577 to 2100 from 1.1e-5 to 5e-3 off at 2e-6,
// one sweep served up to ln(rel / tol) = 2.0 ln 8 (two from 2.1), two up to 3.03 ln 8 (three from 2.85), three up to 3.47 ln 8 (four from
// 3.49).  The gain is 3.5 where many columns are not what they were: the null space of a rank-deficient factor, which any
// movement makes a dense block (5e-3 at 4609 took 8, 2e-2 at 1624 took 7, 8e-3 at 964 took 8), or no basis at all (0.2 at
// 577 took 1 to 0.1, 4 to 0.01, 6 to 1e-3 and 9 to 2e-6).
int sweeps_needed(const StartBasis &b, double tol) {
    if (b.rel <= tol) return 0;
    const double l = std::log(b.rel / tol);
    if (b.lost >= 0.2) return (int)std::ceil(l / std::log(3.5));
    const double s = l / std::log(8.0);
    return std::max(1, (int)std::lround(s < 3.05 ? s - 0.55 : s));
}

// A factor list of its own: part of a call.
struct EigPart {
    std::vector<int> idx, d;
    std::vector<const float *> F;
    std::vector<float *> Q, lam;
    std::vector<kfac_eig_info> info;
    EigPart(const std::vector<int> &which, const float *const *F_, const int *d_, float *const *Q_, float *const *lam_) : idx(which), info(which.size()) {
        for (int i : which) { d.push_back(d_[i]); F.push_back(F_[i]); Q.push_back(Q_[i]); lam.push_back(lam_[i]); }
    }
    int size() const { return (int)idx.size(); }
    void report(kfac_eig_info *to) const {
        for (size_t k = 0; to && k < idx.size(); ++k) to[idx[k]] = info[k];
    }
};

// The factors (wider than KFAC_EIG_SMALL: the others gain nothing from a start) to iterate rather than to decompose directly, given
// the bases they would start from.  Those that need the fewest sweeps first, as many as make the call
// cheapest, if that is cheaper than all of them directly by the 5 % that the two estimates are good for: a chain of launches is
// shared by all factors of its kind.
std::vector<int> choose_sweeps(kfac_ctx *ctx, int batch, const int *d, const std::vector<StartBasis> &start, double tol, int max_sweeps) {
    std::vector<int> need(batch, INT_MAX), levels, best;
    for (int i = 0; i < batch; ++i) {
        if (d[i] <= KFAC_EIG_SMALL || !(start[i].rel >= 0.0)) continue;
        const int s = sweeps_needed(start[i], tol);
        if (max_sweeps > 0 && s > max_sweeps) continue;
        need[i] = s;
        levels.push_back(s);
    }
    std::sort(levels.begin(), levels.end());
    levels.erase(std::unique(levels.begin(), levels.end()), levels.end());
    double least = 0.95 * kfac_eig_direct_seconds(ctx->coop_wgs, batch, d);
    for (int level : levels) {
        std::vector<int> which, dj, sj, dd;
        for (int i = 0; i < batch; ++i) {
            if (need[i] <= level) { which.push_back(i); dj.push_back(d[i]); sj.push_back(need[i]); }
            else dd.push_back(d[i]);
        }
        const double t = kfac_eig_jacobi_seconds((int)dj.size(), dj.data(), sj.data()) + kfac_eig_direct_seconds(ctx->coop_wgs, (int)dd.size(), dd.data());
        if (t < least && kfac_eig_jacobi_ws_bytes((int)dj.size(), dj.data()) <= ctx->ws_bytes) {
            least = t;
            best = which;
        }
    }
    return best;
}

// Direct decomposition of a part of a call; what is not sound, or not as close as the caller asks, goes on to Jacobi sweeps.
int run_direct(kfac_ctx *ctx, EigPart &P, const kfac_eig_opts *opts, double tol, const std::function<bool()> *go_on) {
    const int batch = P.size();
    if ((size_t)batch * 4 * sizeof(double) > ctx->pinned_bytes) return KFAC_EINVAL;
    const double *stat = ctx->pinned;
    const double max_res = std::min(tol, DIRECT_MAX_RES);
    const int drc = kfac_launch_eig_direct(ctx, batch, P.F.data(), P.d.data(), P.Q.data(), P.lam.data(), max_res, ctx->pinned, go_on);
    if (drc != KFAC_OK) return drc;
    std::vector<int> left;
    bool bad = false;
    for (int i = 0; i < batch; ++i) {
        const double off2 = stat[4 * i], f2 = off2 + stat[4 * i + 1], res2 = std::max(stat[4 * i + 2], 0.0), dev2 = stat[4 * i + 3];
        const double max_res2 = max_res * max_res * f2;
        const bool finite = f2 < 1e300;
        const bool ok = finite && res2 <= max_res2 && dev2 <= DIRECT_MAX_DEV2;
        if (finite && !ok) left.push_back(i);
        bad |= !finite;
        const bool untouched = P.d[i] <= KFAC_EIG_REG && off2 <= max_res2;     // diagonal as it stood
        P.info[i] = kfac_eig_info{!ok || untouched ? 0 : 1, finite ? (f2 > 0.0 ? (float)std::sqrt(res2 / f2) : 0.f) : NAN, ok ? 1 : 0};
    }
    if (left.empty()) return bad ? KFAC_ENOCONV : KFAC_OK;
    EigPart L(left, P.F.data(), P.d.data(), P.Q.data(), P.lam.data());
    kfac_eig_opts o{};
    if (opts) o = *opts;
    o.warm_start = 0;      // the start basis is overwritten
    const int rc = kfac_launch_eig_jacobi(ctx, L.size(), L.F.data(), L.d.data(), L.Q.data(), L.lam.data(), &o, L.info.data());
    if (rc == KFAC_OK || rc == KFAC_ENOCONV) L.report(P.info.data());
    return rc == KFAC_OK && bad ? KFAC_ENOCONV : rc;
}

}  // namespace

size_t kfac_eig_ws_bytes_impl(int batch, const int *d) {
    return std::max(kfac_eig_jacobi_ws_bytes(batch, d), kfac_eig_direct_ws_bytes(batch, d));   // the two routes run one after the other
}

int kfac_launch_eig(kfac_ctx *ctx, int batch, const float *const *F, const int *d, float *const *Q,
                    float *const *lam, const kfac_eig_opts *opts, kfac_eig_info *info) {
    const float tol = (opts && opts->tol > 0.f) ? opts->tol : 2e-6f;
    // fp32_only asks for small eigenvalues to be accurate on their own scale.  Jacobi rotations keep that on a graded matrix, a
    // Householder reduction rounds at the scale of ||F||: eigenvalues down to 1e-9 of the largest of a 300-wide factor whose features
    // span four decades, 3e-6 off at most after sweeps, 7e-3 after a reduction.
    // (Small factors are solved in LDS by Jacobi iteration, with no workspace to speak of: 1000 factors of 128 in 48 KB, where the
    // direct route takes hundreds of MB; a workspace sized for that is served as well.)
    if (tol < DIRECT_TOL_MIN || (opts && opts->fp32_only != 0) || kfac_eig_direct_ws_bytes(batch, d) > ctx->ws_bytes)
        return kfac_launch_eig_jacobi(ctx, batch, F, d, Q, lam, opts, info);
    const int max_sweeps = opts ? opts->max_sweeps : 0;
    std::vector<StartBasis> start(batch);
    std::vector<int> sweep, rest(batch);
    for (int i = 0; i < batch; ++i) rest[i] = i;
    bool decided = false;
    if (opts && opts->warm_start != 0) {
        std::vector<int> which;
        for (int i = 0; i < batch; ++i)
            if (d[i] > KFAC_EIG_SMALL) which.push_back(i);
        if (!which.empty()) KFAC_CHECK(probe_start_bases(ctx, which, F, d, Q, start));
        sweep = choose_sweeps(ctx, batch, d, start, tol, max_sweeps);
        decided = true;
    }
    // from the identity: by the norms that the direct route forms at its beginning
    const std::function<bool()> few_sweeps = [&]() {
        for (int i = 0; i < batch; ++i) {
            const double off2 = ctx->pinned[4 * i], f2 = off2 + ctx->pinned[4 * i + 1];
            start[i].rel = f2 > 0.0 && f2 < 1e300 ? std::sqrt(off2 / f2) : (f2 == 0.0 ? 0.0 : -1.0);
            start[i].lost = start[i].rel > 1e-2 ? 1.0 : 0.0;
        }
        sweep = choose_sweeps(ctx, batch, d, start, tol, max_sweeps);
        return sweep.empty();
    };
    if (!decided) {
        EigPart D(rest, F, d, Q, lam);
        const int rc = run_direct(ctx, D, opts, tol, &few_sweeps);
        if (rc == KFAC_OK || rc == KFAC_ENOCONV) D.report(info);
        if (rc != KFAC_EIG_STOPPED) return rc;
    }
    std::vector<char> done(batch, 0);
    if (!sweep.empty()) {
        EigPart J(sweep, F, d, Q, lam);
        const int rc = kfac_launch_eig_jacobi(ctx, J.size(), J.F.data(), J.d.data(), J.Q.data(), J.lam.data(), opts, J.info.data());
        if (rc != KFAC_OK && rc != KFAC_ENOCONV) return rc;
        J.report(info);
        for (int k = 0; k < J.size(); ++k) done[J.idx[k]] = J.info[k].converged != 0;    // (max_sweeps may be less than it took)
    }
    rest.clear();
    for (int i = 0; i < batch; ++i)
        if (!done[i]) rest.push_back(i);
    if (rest.empty()) return KFAC_OK;
    EigPart D(rest, F, d, Q, lam);
    const int rc = run_direct(ctx, D, opts, tol, nullptr);
    if (rc == KFAC_OK || rc == KFAC_ENOCONV) D.report(info);
    return rc;
}
