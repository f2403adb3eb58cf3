// The explicit-inverse method of Sec. II-C, Eq. (kfac-damped): Finv = (F + gamma I)^-1 for every Kronecker factor,
// then the preconditioned gradient as two plain products Ginv * grad * Ainv (the method Sec. IV-A and Table I
// compare the eigendecomposition with).  The inverse of a symmetric positive definite matrix is formed the
// classical way, in fp32: blocked Cholesky factorisation F + gamma I = L L^T (128-wide block columns: the diagonal
// block is factored, and inverted, by one workgroup in registers; the panel below it is multiplied by that inverse and the
// trailing matrix gets its rank-128 update on the fp32 MFMA tile engine), then the triangular inverse L^-1 by
// doubling (two products per level), then L^-T L^-1 as one symmetric product.  n^3 flops in all, 2 n/128 + 2 log2(n/128) + 1
// launches per factor.
#include <algorithm>
#include <cmath>
#include "kfac_internal.h"
#include "mfma_gemm.h"

using namespace kfac;

namespace {

constexpr int NB = BM;            // block size of the factorisation = tile edge of the engine

struct InvPtr { const float *F; float *out; };   // one factor: the caller's matrix and where its inverse goes

// One group of factors of the same size, advanced together (blockIdx.y: factor).  Per factor the workspace holds
//   L  [npad][npad]  F + gamma I on entry to the factorisation (both triangles), the Cholesky factor after
//   Li [npad][npad]  L^-1 (lower triangular); the blocks above the diagonal are scratch of the triangular inversion
//   D  [nt][NB][NB]  inverses of the diagonal blocks of L
struct InvArgs {
    float *base;          // first factor's buffers; the next factor's are fstride floats further
    int64_t fstride;
    const InvPtr *tab;    // device table of the group's factors
    int64_t ld;           // npad
    int n, nt, k;         // k: block column (factorisation) or blocks of a pair's first half (triangular inversion) of this launch
    __device__ float *L(int f) const { return base + f * fstride; }
    __device__ float *Li(int f) const { return L(f) + ld * ld; }
    __device__ float *D(int f) const { return Li(f) + ld * ld; }
};

// L = F + gamma I inside n x n, the identity on the padded part of the diagonal, zero elsewhere.
__global__ __launch_bounds__(256) void inv_init_kernel(float gamma, InvArgs a) {
    const int f = blockIdx.y, n = a.n;
    const float *F = a.tab[f].F;
    float *L = a.L(f);
    const int64_t total = a.ld * a.ld;
    for (int64_t e = blockIdx.x * 256ll + threadIdx.x; e < total; e += (int64_t)gridDim.x * 256) {
        const int r = (int)(e / a.ld), c = (int)(e - (int64_t)r * a.ld);
        float v = 0.f;
        if (r < n && c < n) v = F[(int64_t)r * n + c] + (r == c ? gamma : 0.f);
        else if (r == c) v = 1.f;
        L[e] = v;
    }
}

// Diagonal block k: Cholesky factor in place (lower triangle; the upper is cleared) and its inverse, written to D[k]
// and to the diagonal block of Li.  One workgroup per factor.  A pivot that is not positive (the input was not positive definite,
// or not finite) yields NaNs from there on.
// A chain of 128 pivots: latency is all there is.  Thread (ty, tx) keeps elements (ty + 16 a, tx + 16 b) of the block and of its
// inverse in registers; per pivot one column and one row of the inverse so far go through LDS (two buffers, one barrier), and both get
// their rank-1 update, the inverse by the same row operations.  (With both matrices in LDS, three barriers per pivot and the
// inverse by substitution afterwards, a launch took 312 us, nearly half of the inverse method on the ResNet-50 set; now about 100 us.  With 512 threads: 104 us.)
constexpr int DT = NB / 16;
// x / d with r = 1 / d at hand: the product alone carries r's rounding into a whole column of L and a whole row of L^-1, which
// doubled the error of the inverse of a 129-wide factor
__device__ inline float quotient(float x, float d, float r) {
    const float q = x * r;
    return fmaf(fmaf(-q, d, x), r, q);
}
struct DiagSmem { float col[2][NB], xrow[2][NB]; };
__device__ inline void inv_diag_block(const InvArgs &a, int f, int k, DiagSmem &sm) {
    float (&col)[2][NB] = sm.col, (&xrow)[2][NB] = sm.xrow;
    const int tid = threadIdx.x, ty = tid >> 4, tx = tid & 15;
    const global_ptr<float> blk = as_global(a.L(f)) + ((int64_t)k * NB) * a.ld + (int64_t)k * NB;
    float S[DT][DT], X[DT][DT];
#pragma unroll
    for (int p = 0; p < DT; ++p)
#pragma unroll
        for (int q = 0; q < DT; ++q) {
            const int r = ty + 16 * p, c = tx + 16 * q;
            X[p][q] = r == c ? 1.f : 0.f;
            S[p][q] = q > p ? 0.f : (r >= c ? blk[(int64_t)r * a.ld + c] : blk[(int64_t)c * a.ld + r]);   // the lower triangle is the valid one
        }
#pragma unroll
    for (int jb = 0; jb < DT; ++jb)
        for (int jj = 0; jj < 16; ++jj) {
            const int j = 16 * jb + jj, h = jj & 1;
            if (tx == jj)
#pragma unroll
                for (int p = jb; p < DT; ++p) col[h][ty + 16 * p] = S[p][jb];
            if (ty == jj)
#pragma unroll
                for (int q = 0; q <= jb; ++q) xrow[h][tx + 16 * q] = X[jb][q];
            __syncthreads();
            const float sq = sqrtf(col[h][j]), rs = 1.f / sq;
            float lr[DT], lc[DT], xs[DT];
#pragma unroll
            for (int p = jb; p < DT; ++p) {
                const float vr = quotient(col[h][ty + 16 * p], sq, rs), vc = quotient(col[h][tx + 16 * p], sq, rs);
                lr[p] = p > jb || ty > jj ? vr : 0.f;
                lc[p] = p > jb || tx > jj ? vc : 0.f;
            }
#pragma unroll
            for (int q = 0; q <= jb; ++q) xs[q] = quotient(xrow[h][tx + 16 * q], sq, rs);
#pragma unroll
            for (int p = jb; p < DT; ++p) {
#pragma unroll
                for (int q = jb; q <= p; ++q) S[p][q] = fmaf(-lr[p], lc[q], S[p][q]);
                if (tx == jj) S[p][jb] = p == jb && ty == jj ? sq : (p > jb || ty > jj ? lr[p] : S[p][jb]);
#pragma unroll
                for (int q = 0; q <= jb; ++q) X[p][q] = fmaf(-lr[p], xs[q], X[p][q]);
            }
            if (ty == jj)
#pragma unroll
                for (int q = 0; q <= jb; ++q) X[jb][q] = xs[q];
        }
    const global_ptr<float> Dk = as_global(a.D(f)) + (int64_t)k * NB * NB;
    const global_ptr<float> Lik = as_global(a.Li(f)) + ((int64_t)k * NB) * a.ld + (int64_t)k * NB;
#pragma unroll
    for (int p = 0; p < DT; ++p)
#pragma unroll
        for (int q = 0; q < DT; ++q) {
            const int r = ty + 16 * p, c = tx + 16 * q;
            const float x = r >= c ? X[p][q] : 0.f;
            blk[(int64_t)r * a.ld + c] = r >= c ? S[p][q] : 0.f;
            Dk[r * NB + c] = x;
            Lik[(int64_t)r * a.ld + c] = x;
        }
}
__global__ __launch_bounds__(256) void inv_diag_kernel(InvArgs a) {
    __shared__ DiagSmem sm;
    inv_diag_block(a, blockIdx.x, a.k, sm);
}

__device__ inline void inv_tri_decode(int idx, int &ti, int &tj) {   // idx = ti (ti + 1) / 2 + tj, tj <= ti
    int t = (int)((sqrtf(8.f * (float)idx + 1.f) - 1.f) * 0.5f);
    while ((t + 1) * (t + 2) / 2 <= idx) ++t;
    while (t * (t + 1) / 2 > idx) --t;
    ti = t;
    tj = idx - t * (t + 1) / 2;
}

// The five products, one 128 x 128 output tile per workgroup (all operands are padded to whole tiles):
//   PANEL   L[i,k] <- L[i,k] D_k^T                                      i > k              (grid: nt-k-1)
//   UPDATE  L[i,j] <- L[i,j] - L[i,k] L[j,k]^T                          i >= j > k         (grid: lower tiles)
//           and then, by the workgroup of the first of them, the diagonal block k + 1: the others' tiles hide its chain of pivots
//   HALF    Li[j,i] <- sum_{c = j}^{m-1} L[i,c] Li[c,j]    scratch: block (i, j) of L21 Li11, kept above the diagonal
//   JOIN    Li[i,j] <- -sum_{c = m}^{i} Li[i,c] Li[j,c]    (block (c, j) of the scratch is at (j, c))
//           for every pair of neighbouring index ranges [m - s, m), [m, m + s) of s = a.k blocks whose inverses are there:
//           j in the first, i in the second                                               (grid: pairs * s^2)
//   GRAM    out[i,j] <- sum_{c >= i} Li[c,i]^T Li[c,j], and its mirror  i >= j             (grid: lower tiles)
enum { INV_PANEL = 0, INV_UPDATE, INV_HALF, INV_JOIN, INV_GRAM };
template <int MODE>
__global__ __launch_bounds__(NTHREADS) __attribute__((amdgpu_waves_per_eu(2))) void inv_gemm_kernel(InvArgs a) {
    __shared__ union { TileSmem tile; DiagSmem diag; } shared;
    TileSmem &sm = shared.tile;
    floatx16 acc[2][2];
    const int64_t ld = a.ld;
    // UPDATE goes round the factors first, so that every factor's first tile, which has the pivots behind it, starts at once
    const int npad = a.nt * NB, f = MODE == INV_UPDATE ? blockIdx.x : blockIdx.y, tile = MODE == INV_UPDATE ? blockIdx.y : blockIdx.x;
    float *const L = a.L(f), *const Li = a.Li(f), *const D = a.D(f);
    if (MODE == INV_PANEL) {
        const int i = a.k + 1 + blockIdx.x;
        float *Lik = L + ((int64_t)i * NB) * ld + (int64_t)a.k * NB;
        OpStrided<float, true> A{Lik, ld, 1, NB, NB, -1};                                     // elem(m,c) = L[i,k][m][c]
        OpStrided<float, true> B{D + (int64_t)a.k * NB * NB, NB, 1, NB, NB, -1};              // elem(n,c) = D_k[n][c]
        gemm_tile(A, B, 0, 0, 0, NB, sm, acc);
        for_each_acc(acc, [&](int r, int c, float v) { Lik[(int64_t)r * ld + c] = v; });
    } else if (MODE == INV_UPDATE) {
        int ti, tj;
        inv_tri_decode(tile, ti, tj);
        const int i = a.k + 1 + ti, j = a.k + 1 + tj;
        OpStrided<float, true> A{L + ((int64_t)i * NB) * ld + (int64_t)a.k * NB, ld, 1, NB, NB, -1};
        OpStrided<float, true> B{L + ((int64_t)j * NB) * ld + (int64_t)a.k * NB, ld, 1, NB, NB, -1};
        gemm_tile(A, B, 0, 0, 0, NB, sm, acc);
        float *Lij = L + ((int64_t)i * NB) * ld + (int64_t)j * NB;
        for_each_acc(acc, [&](int r, int c, float v) { Lij[(int64_t)r * ld + c] -= v; });
        if (tile == 0) {
            __syncthreads();       // the tile is written
            inv_diag_block(a, f, a.k + 1, shared.diag);
        }
    } else if (MODE == INV_HALF || MODE == INV_JOIN) {
        const int s = a.k, idx = blockIdx.x, pair = idx / (s * s), m = (2 * pair + 1) * s;
        const int i = m + (idx / s) % s, j = m - s + idx % s;
        if (i >= a.nt) return;
        if (MODE == INV_HALF) {
            OpStrided<float, true> A{L + ((int64_t)i * NB) * ld, ld, 1, NB, m * NB, -1};           // elem(r,c) = L[i*NB+r][c]
            OpStrided<float, false> B{Li + (int64_t)j * NB, 1, ld, NB, m * NB, -1};                // elem(n,c) = Li[c][j*NB+n]
            gemm_tile(A, B, 0, 0, j * NB, m * NB, sm, acc);
            float *H = Li + ((int64_t)j * NB) * ld + (int64_t)i * NB;
            for_each_acc_transposed(acc, reinterpret_cast<float *>(&sm), [&](int r, int c, float v) { H[(int64_t)r * ld + c] = v; });
        } else {
            // the scratch is the block's transpose, so that the blocks of one column j are one row of the matrix: elem(n,c) = H[j*NB+n][c]
            OpStrided<float, true> A{Li + ((int64_t)i * NB) * ld, ld, 1, NB, (i + 1) * NB, -1};     // elem(r,c) = Li[i*NB+r][c]
            OpStrided<float, true> B{Li + ((int64_t)j * NB) * ld, ld, 1, NB, (i + 1) * NB, -1};
            gemm_tile(A, B, 0, 0, m * NB, (i + 1) * NB, sm, acc);
            float *Lij = Li + ((int64_t)i * NB) * ld + (int64_t)j * NB;
            for_each_acc(acc, [&](int r, int c, float v) { Lij[(int64_t)r * ld + c] = -v; });
        }
    } else {
        int i, j;
        inv_tri_decode(blockIdx.x, i, j);
        OpStrided<float, false> A{Li + (int64_t)i * NB, 1, ld, NB, npad, -1};                  // elem(m,c) = Li[c][i*NB+m]
        OpStrided<float, false> B{Li + (int64_t)j * NB, 1, ld, NB, npad, -1};                  // elem(n,c) = Li[c][j*NB+n]
        gemm_tile(A, B, 0, 0, i * NB, npad, sm, acc);                                          // Li[c, i] = 0 for c < i
        const int n = a.n;
        float *out = a.tab[f].out;
        for_each_acc(acc, [&](int r, int c, float v) {
            const int gr = i * NB + r, gc = j * NB + c;
            if (gr < n && gc < n) out[(int64_t)gr * n + gc] = v;
        });
        if (i != j)
            for_each_acc_transposed(acc, reinterpret_cast<float *>(&sm), [&](int r, int c, float v) {
                const int gr = j * NB + r, gc = i * NB + c;
                if (gr < n && gc < n) out[(int64_t)gr * n + gc] = v;
            });
    }
}

inline int inv_npad(int n) { return (n + NB - 1) / NB * NB; }
inline size_t inv_bytes_one(int n) {
    const size_t np = inv_npad(n), nt = np / NB;
    return kfac_align_up((2 * np * np + nt * NB * NB) * sizeof(float), 256);
}

// grad <- Ginv grad Ainv: T = grad Ainv into the workspace, then grad = Ginv T.
struct EpiStoreBf16 {
    unsigned short *C;
    int64_t ld;
    __device__ void operator()(int r, int c, float v) const {
        unsigned u = __float_as_uint(v);
        if ((u & 0x7fffffffu) > 0x7f800000u) { C[(int64_t)r * ld + c] = (unsigned short)((u >> 16) | 0x40u); return; }
        u += 0x7fffu + ((u >> 16) & 1u);    // round to nearest even
        C[(int64_t)r * ld + c] = (unsigned short)(u >> 16);
    }
};

}  // namespace

// Workspace: the table of pointers, then room for the largest group of equal-sized factors (a group too large for
// the workspace at hand is cut into several).  With room for more, up to four groups are in flight at once.
static size_t inv_table_bytes(int batch) { return kfac_align_up((size_t)batch * sizeof(InvPtr), 256); }
size_t kfac_invert_ws_bytes_impl(int batch, const int *d) {
    size_t m = 0;
    for (int b = 0; b < batch; ++b) m = std::max(m, inv_bytes_one(d[b]));
    return inv_table_bytes(batch) + m;
}

namespace {
struct InvGroup { int n, first, count; };   // `count` factors of size n, entries first.. of the sorted table

// The whole chain of one group on one stream.
int inv_enqueue_group(kfac_ctx *ctx, hipStream_t st, const InvGroup &g, const InvPtr *tab_dev, float *slot, float damping) {
    const int n = g.n, np = inv_npad(n), nt = np / NB, nm = g.count;
    InvArgs a;
    a.base = slot;
    a.fstride = (int64_t)(inv_bytes_one(n) / sizeof(float));
    a.tab = tab_dev + g.first;
    a.ld = np; a.n = n; a.nt = nt; a.k = 0;
    const double n3 = (double)nm * n * n * n;
    {
        KfacProfScope prof(ctx, KC_INVERSE, n3 / 3.0, 0.0, st);
        hipLaunchKernelGGL(inv_init_kernel, dim3((unsigned)std::min<int64_t>(((int64_t)np * np + 255) / 256, 2048), nm), dim3(256), 0, st,
                           damping, a);
        hipLaunchKernelGGL(inv_diag_kernel, dim3(nm), dim3(256), 0, st, a);
        for (int k = 0; k + 1 < nt; ++k) {
            a.k = k;
            const int rest = nt - k - 1;
            hipLaunchKernelGGL(inv_gemm_kernel<INV_PANEL>, dim3(rest, nm), dim3(NTHREADS), 0, st, a);
            hipLaunchKernelGGL(inv_gemm_kernel<INV_UPDATE>, dim3(nm, rest * (rest + 1) / 2), dim3(NTHREADS), 0, st, a);
        }
    }
    {
        KfacProfScope prof(ctx, KC_INVERSE, n3 / 3.0, 0.0, st);
        // by doubling: a block row after the other is nt - 1 dependent pairs of launches of at most nt tiles each (119 + 17 us per
        // pair on the ResNet-50 set)
        for (int s = 1; s < nt; s *= 2) {
            a.k = s;
            const int pairs = (nt - s + 2 * s - 1) / (2 * s);      // with a second half that is not empty
            hipLaunchKernelGGL(inv_gemm_kernel<INV_HALF>, dim3(pairs * s * s, nm), dim3(NTHREADS), 0, st, a);
            hipLaunchKernelGGL(inv_gemm_kernel<INV_JOIN>, dim3(pairs * s * s, nm), dim3(NTHREADS), 0, st, a);
        }
    }
    KfacProfScope prof(ctx, KC_INVERSE, n3 / 3.0, 0.0, st);
    hipLaunchKernelGGL(inv_gemm_kernel<INV_GRAM>, dim3(nt * (nt + 1) / 2, nm), dim3(NTHREADS), 0, st, a);
    KFAC_HIP_CHECK(hipGetLastError());
    return KFAC_OK;
}
}  // namespace

int kfac_launch_invert_factors(kfac_ctx *ctx, int batch, const float *const *F, const int *d, float damping, float *const *Finv) {
    if (kfac_invert_ws_bytes_impl(batch, d) > ctx->ws_bytes) return KFAC_EWORKSPACE;
    // factors sorted by size (largest first); equal sizes form groups
    std::vector<int> order(batch);
    for (int b = 0; b < batch; ++b) order[b] = b;
    std::stable_sort(order.begin(), order.end(), [&](int p, int q) { return d[p] > d[q]; });
    std::vector<InvPtr> tab(batch);
    for (int t = 0; t < batch; ++t) tab[t] = InvPtr{F[order[t]], Finv[order[t]]};
    InvPtr *tab_dev = (InvPtr *)ctx->ws;
    KFAC_CHECK(kfac_upload(ctx, tab_dev, tab.data(), (size_t)batch * sizeof(InvPtr)));
    char *pool = ctx->ws + inv_table_bytes(batch);
    const size_t pool_bytes = ctx->ws_bytes - inv_table_bytes(batch);
    // four equal regions, one per internal stream, if each then still holds the largest factor; else one region
    const size_t largest = inv_bytes_one(d[order[0]]);
    const int nstreams = pool_bytes / KFAC_NUM_AUX_STREAMS >= largest ? KFAC_NUM_AUX_STREAMS : 1;
    const size_t region = kfac_align_up(pool_bytes / nstreams - 255, 256) ;
    std::vector<InvGroup> groups;
    for (int t = 0; t < batch;) {
        int e = t;
        const size_t one = inv_bytes_one(d[order[t]]);
        const int cap = (int)std::max<size_t>(1, region / one);
        while (e < batch && d[order[e]] == d[order[t]] && e - t < cap) ++e;
        groups.push_back(InvGroup{d[order[t]], t, e - t});
        t = e;
    }
    // the internal streams start after everything already queued on the caller's stream (the table upload included) ...
    KFAC_HIP_CHECK(hipEventRecord(ctx->ev_fork, ctx->stream));
    for (int i = 0; i < nstreams; ++i) KFAC_HIP_CHECK(hipStreamWaitEvent(ctx->aux[i], ctx->ev_fork, 0));
    // groups dealt to the stream with the least work so far (largest first); a stream's groups use its region in turn
    double load[KFAC_NUM_AUX_STREAMS] = {0, 0, 0, 0};
    int rc = KFAC_OK;
    for (const InvGroup &g : groups) {
        int best = 0;
        for (int i = 1; i < nstreams; ++i) if (load[i] < load[best]) best = i;
        const double nt = inv_npad(g.n) / NB;
        load[best] += nt * 145e-6 + (double)g.count * g.n * (double)g.n * g.n / 60e12;   // a block column's serial launches + products
        rc = inv_enqueue_group(ctx, ctx->aux[best], g, tab_dev, (float *)(pool + (size_t)best * region), damping);
        if (rc != KFAC_OK) break;
    }
    // ... and the caller's stream continues after all of them
    for (int i = 0; i < nstreams; ++i) {
        if (hipEventRecord(ctx->ev_join[i], ctx->aux[i]) != hipSuccess) return KFAC_EHIP;
        if (hipStreamWaitEvent(ctx->stream, ctx->ev_join[i], 0) != hipSuccess) return KFAC_EHIP;
    }
    return rc;
}

// ---- grad <- Ginv grad Ainv for a batch of layers: two launches, each over the output tiles of every layer ----
namespace {
struct InvLayer {
    const float *Ainv, *Ginv;
    void *grad;
    float *T;          // [dG][dA] intermediate grad * Ainv
    int dA, dG, bf16;
    int tile0, tn;     // first tile of the layer in the launch, tiles per tile row
};

// STAGE 0: T = grad Ainv.  STAGE 1: grad = Ginv T.
template <int STAGE>
__global__ __launch_bounds__(NTHREADS) __attribute__((amdgpu_waves_per_eu(2))) void inv_precond_kernel(const InvLayer *layers, int nlayers) {
    __shared__ TileSmem sm;
    // the layer whose tile range holds this workgroup: the last one that starts at or before it
    int l = 0;
    for (int base = 0; base < nlayers; base += 64) {
        const int idx = base + (int)(threadIdx.x & 63);
        const bool le = idx < nlayers && layers[idx].tile0 <= (int)blockIdx.x;
        const unsigned long long m = __ballot(le);
        if (m == 0) break;
        l = base + 63 - __builtin_clzll(m);
    }
    l = __builtin_amdgcn_readfirstlane(l);
    const InvLayer L = layers[l];
    const int t = blockIdx.x - L.tile0;
    const int i0 = (t / L.tn) * BM, j0 = (t % L.tn) * BM;
    if (STAGE == 0) {
        OpStrided<float, false> b{L.Ainv, 1, L.dA, L.dA, L.dA, -1};            // elem(c,k) = Ainv[k][c]
        float *T = L.T;
        const int dA = L.dA;
        auto epi = [=](int r, int c, float v) { T[(int64_t)r * dA + c] = v; };
        if (L.bf16) {
            OpStrided<unsigned short, true> a{(const unsigned short *)L.grad, L.dA, 1, L.dG, L.dA, -1};
            gemm_tile_ragged(a, b, i0, j0, L.dA, L.dG, L.dA, sm, epi);
        } else {
            OpStrided<float, true> a{(const float *)L.grad, L.dA, 1, L.dG, L.dA, -1};
            gemm_tile_ragged(a, b, i0, j0, L.dA, L.dG, L.dA, sm, epi);
        }
    } else {
        OpStrided<float, true> a{L.Ginv, L.dG, 1, L.dG, L.dG, -1};
        OpStrided<float, false> b{L.T, 1, L.dA, L.dA, L.dG, -1};               // elem(c,k) = T[k][c]
        if (L.bf16) {
            const EpiStoreBf16 e{(unsigned short *)L.grad, L.dA};
            gemm_tile_ragged(a, b, i0, j0, L.dG, L.dG, L.dA, sm, [=](int r, int c, float v) { e(r, c, v); });
        } else {
            float *g = (float *)L.grad;
            const int dA = L.dA;
            gemm_tile_ragged(a, b, i0, j0, L.dG, L.dG, L.dA, sm, [=](int r, int c, float v) { g[(int64_t)r * dA + c] = v; });
        }
    }
}
}  // namespace

size_t kfac_precondition_inverse_ws_bytes_impl(int n, const kfac_precond_inv_item *items) {
    size_t b = kfac_align_up((size_t)n * sizeof(InvLayer), 256);
    for (int i = 0; i < n; ++i) b += kfac_align_up((size_t)items[i].dA * items[i].dG * sizeof(float), 256);
    return b;
}

int kfac_launch_precondition_inverse_batched(kfac_ctx *ctx, int n, const kfac_precond_inv_item *items) {
    if (kfac_precondition_inverse_ws_bytes_impl(n, items) > ctx->ws_bytes) return KFAC_EWORKSPACE;
    std::vector<InvLayer> layers(n);
    char *p = ctx->ws + kfac_align_up((size_t)n * sizeof(InvLayer), 256);
    int tiles = 0;
    double fl0 = 0.0, fl1 = 0.0;
    for (int i = 0; i < n; ++i) {
        const kfac_precond_inv_item &it = items[i];
        const int tm = (it.dG + BM - 1) / BM, tn = (it.dA + BM - 1) / BM;
        layers[i] = InvLayer{it.Ainv, it.Ginv, it.grad, (float *)p, it.dA, it.dG, it.grad_dtype == KFAC_BF16 ? 1 : 0, tiles, tn};
        p += kfac_align_up((size_t)it.dA * it.dG * sizeof(float), 256);
        tiles += tm * tn;
        fl0 += 2.0 * it.dG * (double)it.dA * it.dA;
        fl1 += 2.0 * it.dG * (double)it.dG * it.dA;
    }
    InvLayer *d_layers = (InvLayer *)ctx->ws;
    KFAC_CHECK(kfac_upload(ctx, d_layers, layers.data(), (size_t)n * sizeof(InvLayer)));
    {
        KfacProfScope prof(ctx, KC_PRECOND_GEMM, fl0, 0.0);
        hipLaunchKernelGGL(inv_precond_kernel<0>, dim3(tiles), dim3(NTHREADS), 0, ctx->stream, (const InvLayer *)d_layers, n);
    }
    KfacProfScope prof(ctx, KC_PRECOND_GEMM, fl1, 0.0);
    hipLaunchKernelGGL(inv_precond_kernel<1>, dim3(tiles), dim3(NTHREADS), 0, ctx->stream, (const InvLayer *)d_layers, n);
    KFAC_HIP_CHECK(hipGetLastError());
    return KFAC_OK;
}
