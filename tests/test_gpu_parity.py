"""GPU parity: every C-ABI call against the fp64 CPU oracle on the same seeded inputs.

Tolerances (the benchmark spec): factors and preconditioned gradients relative Frobenius error
<= 1e-4 in fp32 (<= 2e-2 with bf16 inputs); eigenpairs: ||F - Q diag(lam) Q^T||_F <= 1e-5 ||F||_F and
eigenvalues within 1e-5 * lam_max of the oracle's; unfold is bit-exact (data movement only).
"""
import os
import subprocess
import sys
import threading
import time

import numpy as np
import pytest
import torch

import oracle
from paper_2007_00784_amd import kfac as K
from paper_2007_00784_amd import synthetic as S
from gpu_util import Ctx, relfro, ndt_to_rows

pytestmark = pytest.mark.gpu

TOL_F32 = 1e-4
TOL_BF16 = 2e-2
TOL_RES = 1e-5
TOL_LAM = 1e-5


@pytest.fixture(scope="module")
def ctx():
    c = Ctx(1 << 30)
    yield c
    c.close()


# ------------------------------------------------------------------ unfold
UNFOLD_CASES = [
    # N, C, H, k, stride, pad
    (2, 3, 5, 3, 1, 1),
    (1, 1, 5, 7, 1, 3),
    (2, 2, 7, 3, 2, 1),
    (3, 4, 8, 1, 2, 0),
    (2, 3, 37, 7, 2, 3),       # several row chunks per plane after staging limits
    (4, 16, 8, 3, 1, 1),       # config-1 layer
    (2, 64, 14, 3, 1, 1),
    (2, 130, 7, 3, 2, 1),      # many channels per workgroup, ragged channel tail
    (1, 3, 224, 7, 2, 3),      # stem geometry: chunked rows
    (2, 8, 56, 3, 1, 1),
    (2, 5, 28, 3, 2, 1),       # stride 2 onto a 14 x 14 map: the tile holds the output
    (1, 2, 14, 5, 2, 2),
    (3, 20, 7, 3, 1, 1),       # 7 x 7 map, several channels per workgroup with a ragged tail
    (2, 4, 56, 3, 2, 1),       # stride 2 onto 28 x 28: one channel per workgroup
]


@pytest.mark.parametrize("case", UNFOLD_CASES)
@pytest.mark.parametrize("bf16", [False, True])
def test_unfold_bit_exact(ctx, case, bf16):
    N, C, H, k, s, p = case
    x = np.random.default_rng(1).standard_normal((N, C, H, H)).astype(np.float32)
    if bf16:
        x = S.bf16_bits_to_f32(S.to_bf16_bits(x)).reshape(x.shape)
    out = ctx.unfold(x, k, k, s, p, bf16=bf16).float().cpu().numpy()
    ref = oracle.unfold(x, k, k, s, s, p, p)
    assert np.array_equal(ndt_to_rows(out), ref)


# ------------------------------------------------------------------ factors
FACTOR_CASES = [
    # layout, N, d, T, ones
    ("RD", 64, 10, 1, 0),
    ("RD", 300, 65, 1, 1),
    ("RD", 2048, 144, 1, 1),
    ("NDT", 32, 144, 64, 1),       # config-1 A factor
    ("NDT", 32, 16, 64, 0),        # config-1 G factor
    ("NDT", 7, 130, 49, 1),        # T = 49, ragged tiles
    ("NDT", 3, 257, 196, 0),
    ("NDT", 5, 300, 5, 1),         # T < K slab
    ("RD", 5000, 33, 1, 1),        # split-K on a single tile
    ("NDT", 64, 64, 784, 1),       # deep split-K
    ("NDT", 9, 200, 9, 1),         # bf16 engine: every example ends in a group that overlaps the one before by 7
    ("NDT", 4, 130, 8, 0),         # bf16 engine: exactly one group per example
    ("NDT", 40, 257, 100, 1),      # bf16 engine: T = 12.5 groups, three tiles per side, contraction ends mid-slab
    ("NDT", 6, 70, 4, 1),          # grouped engine, fp32: one group per example (bf16: element-wise engine, T < 8)
    ("NDT", 6, 70, 7, 1),          # grouped engine, fp32: second group overlaps the first by one position
    ("NDT", 3, 20, 15, 0),         # grouped engine: bf16 second group overlaps by one, fp32 fourth by one
    ("NDT", 600, 129, 49, 1),      # T = 49 with split-K: several jobs per tile, column sums across splits, ragged tile
]


def test_unfold_batched_bit_exact(ctx):
    """Every unfold case, fp32 and bf16 mixed, in one batched call (one launch per element type; a workgroup finds
    its layer by binary search over the layers' first workgroup indices), bit-exact against the oracle; an empty
    batch is a no-op and two layers writing the same output are rejected."""
    rng = np.random.default_rng(3)
    K.kfac_unfold_batched(ctx.h, [], [], [])
    xs, convs, outs, refs = [], [], [], []
    for (N, C, H, k, s, p) in UNFOLD_CASES:
        for bf16 in (False, True):
            x = rng.standard_normal((N, C, H, H)).astype(np.float32)
            if bf16:
                x = S.bf16_bits_to_f32(S.to_bf16_bits(x)).reshape(x.shape)
            Ho = (H + 2 * p - k) // s + 1
            xd = ctx.to_dev(x, bf16)
            xs.append(xd); convs.append((k, k, s, p))
            outs.append(torch.full((N, C * k * k, Ho * Ho), float("nan"), dtype=xd.dtype, device=ctx.dev))
            refs.append(oracle.unfold(x, k, k, s, s, p, p))
    assert K.kfac_unfold_workspace_bytes(len(xs)) <= ctx.ws.numel()
    K.kfac_unfold_batched(ctx.h, xs, convs, outs)
    torch.cuda.synchronize()
    for o, ref in zip(outs, refs):
        assert np.array_equal(ndt_to_rows(o.float().cpu().numpy()), ref)
    with pytest.raises(K.KfacError):
        K.kfac_unfold_batched(ctx.h, xs[:2], convs[:2], [outs[0], outs[0]])


@pytest.mark.parametrize("case", FACTOR_CASES)
@pytest.mark.parametrize("bf16", [False, True])
def test_update_factors_matches_oracle(ctx, case, bf16):
    layout, N, d, T, ones = case
    rng = np.random.default_rng(2)
    D = d + ones
    F = None
    Fd = torch.full((D, D), float("nan"), dtype=torch.float32, device=ctx.dev)
    for upd, decay in enumerate([0.0, 0.95, 0.95]):
        X = np.maximum(rng.standard_normal((N, d, T)), 0).astype(np.float32) if layout == "NDT" else \
            np.maximum(rng.standard_normal((N * T, d)), 0).astype(np.float32)
        if bf16:
            X = S.bf16_bits_to_f32(S.to_bf16_bits(X)).reshape(X.shape)
        rows = ndt_to_rows(X) if layout == "NDT" else X.astype(np.float64)
        R = rows.shape[0]
        Fb = oracle.gram(rows, ones, 1.0 / R)
        F = Fb if upd == 0 else oracle.ema(F, Fb, decay)
        Xd = ctx.to_dev(X, bf16)
        ctx.update_factors(Xd, K.KFAC_LAYOUT_NDT if layout == "NDT" else K.KFAC_LAYOUT_RD, N, d, T, ones,
                           1.0 / R, decay, Fd)
        torch.cuda.synchronize()
        got = Fd.cpu().numpy()
        assert np.isfinite(got).all()
        assert np.array_equal(got, got.T)
        assert relfro(got, F) <= TOL_F32
    if ones:
        assert abs(got[D - 1, D - 1] - 1.0) < 1e-6


def test_update_factors_batched_matches_oracle(ctx):
    """Every case above, fp32 and bf16 operands mixed, in ONE batched call per update (all four operand forms
    in the same call; job tables, per-factor partial buffers, the shared reducer), two updates so the
    running average of each factor is exercised, plus an empty batch."""
    rng = np.random.default_rng(5)
    K.kfac_update_factors_batched(ctx.h, [])
    F = [None] * (2 * len(FACTOR_CASES))
    Fd = [torch.full((d + ones, d + ones), float("nan"), dtype=torch.float32, device=ctx.dev)
          for (_, _, d, _, ones) in FACTOR_CASES for _ in range(2)]
    for upd, decay in enumerate([0.0, 0.9]):
        items = []
        for ci, (layout, N, d, T, ones) in enumerate(FACTOR_CASES):
            for bf16 in (False, True):
                j = 2 * ci + int(bf16)
                X = np.maximum(rng.standard_normal((N, d, T)), 0).astype(np.float32) if layout == "NDT" else \
                    np.maximum(rng.standard_normal((N * T, d)), 0).astype(np.float32)
                if bf16:
                    X = S.bf16_bits_to_f32(S.to_bf16_bits(X)).reshape(X.shape)
                rows = ndt_to_rows(X) if layout == "NDT" else X.astype(np.float64)
                R = rows.shape[0]
                Fb = oracle.gram(rows, ones, 1.0 / R)
                F[j] = Fb if upd == 0 else oracle.ema(F[j], Fb, decay)
                items.append(dict(X=ctx.to_dev(X, bf16), layout=K.KFAC_LAYOUT_NDT if layout == "NDT" else K.KFAC_LAYOUT_RD,
                                  N=N, d=d, T=T, append_ones=ones, scale=1.0 / R, decay=decay, F=Fd[j]))
        assert K.kfac_update_factors_workspace_bytes(items) <= ctx.ws.numel()
        K.kfac_update_factors_batched(ctx.h, items)
        torch.cuda.synchronize()
        for j in range(len(F)):
            got = Fd[j].cpu().numpy()
            assert np.isfinite(got).all(), j
            assert np.array_equal(got, got.T), j
            assert relfro(got, F[j]) <= TOL_F32, (j, relfro(got, F[j]))
    # the same factor twice in one batch is rejected
    with pytest.raises(K.KfacError):
        K.kfac_update_factors_batched(ctx.h, [items[0], items[0]])


def test_update_factors_deterministic(ctx):
    rng = np.random.default_rng(3)
    X = ctx.to_dev(rng.standard_normal((20000, 70)).astype(np.float32))
    outs = []
    for _ in range(2):
        Fd = torch.zeros((71, 71), dtype=torch.float32, device=ctx.dev)
        ctx.update_factors(X, K.KFAC_LAYOUT_RD, 20000, 70, 1, 1, 1.0 / 20000, 0.0, Fd)
        torch.cuda.synchronize()
        outs.append(Fd.cpu().numpy())
    assert np.array_equal(outs[0], outs[1])


# ------------------------------------------------------------------ eig
def gram_factor(n, rows, seed, ones=True):
    rng = np.random.default_rng(seed)
    X = np.maximum(rng.standard_normal((rows, n - (1 if ones else 0))), 0)
    return oracle.gram(X, 1 if ones else 0, 1.0 / rows).astype(np.float32)


def check_eigpairs(F32, lam, Q, label=""):
    F = F32.astype(np.float64)
    lam = lam.astype(np.float64)
    Q = Q.astype(np.float64)
    n = F.shape[0]
    nf = np.linalg.norm(F)
    assert np.isfinite(lam).all() and np.isfinite(Q).all(), label
    assert np.all(np.diff(lam) >= 0), label
    res = np.linalg.norm(F - (Q * lam) @ Q.T) / nf
    orth = np.linalg.norm(Q.T @ Q - np.eye(n), 2)
    ref, _ = oracle.eigh(F)
    lerr = np.abs(lam - ref).max() / max(abs(ref).max(), 1e-300)
    print("%s n=%d residual=%.2e orth2=%.2e lam_err=%.2e" % (label, n, res, orth, lerr))
    assert res <= TOL_RES, label
    assert lerr <= TOL_LAM, label
    assert orth <= 1e-4, label


EIG_SIZES = [(1, 1), (2, 5), (16, 40), (17, 9), (65, 200), (128, 64), (129, 300), (145, 2048), (257, 100),
             (289, 600), (577, 300), (640, 2000)]


@pytest.mark.parametrize("n,rows", EIG_SIZES)
def test_eig_single(ctx, n, rows):
    F = gram_factor(n, rows, seed=n)
    Ld, Qd, info = ctx.eig([F])
    assert info[0][2], info
    check_eigpairs(F, Ld[0].cpu().numpy(), Qd[0].cpu().numpy(), "single")


def test_eig_batch_mixed_sizes(ctx):
    sizes = [(16, 50), (145, 500), (10, 3), (145, 700), (289, 100), (64, 64), (300, 1000), (33, 100), (289, 900)]
    mats = [gram_factor(n, r, seed=100 + i, ones=(i % 2 == 0)) for i, (n, r) in enumerate(sizes)]
    Ld, Qd, info = ctx.eig(mats)
    for i, F in enumerate(mats):
        assert info[i][2]
        check_eigpairs(F, Ld[i].cpu().numpy(), Qd[i].cpu().numpy(), "batch[%d]" % i)


def test_eig_known_spectrum_and_diagonal(ctx):
    n = 200
    u = np.random.default_rng(5).standard_normal(n); u /= np.linalg.norm(u)
    H = np.eye(n) - 2 * np.outer(u, u)
    D = np.concatenate([np.zeros(50), np.full(60, 0.5), np.linspace(1, 9, 89), [100.0]])
    F = (H @ np.diag(D) @ H).astype(np.float32)
    Dg = np.diag(np.random.default_rng(6).random(150)).astype(np.float32)
    Ld, Qd, info = ctx.eig([F, Dg])
    lam = Ld[0].cpu().numpy()
    assert np.abs(lam - np.sort(D)).max() <= TOL_LAM * 100
    check_eigpairs(F, lam, Qd[0].cpu().numpy(), "householder")
    assert np.array_equal(Ld[1].cpu().numpy(), np.sort(np.diag(Dg)))
    assert info[1][0] == 0


def test_eig_warm_start(ctx):
    """A slowly moving factor (running average with 5 % of a new batch, Sec. IV-B) decomposed again from the
    previous eigenvectors: the same invariants hold, and by Jacobi sweeps (which is what a tolerance below 1e-6 asks for) it
    takes fewer of them than from the identity; a flat-path factor and a two-level one, plus a small one (which ignores the
    option) in the same batch.  Starting from the exact eigenvectors of the same matrix converges at once.  A decomposition
    reports what it did: never none for a factor that moved."""
    sizes = [(577, 1500), (2100, 3000), (65, 200)]
    F0 = [gram_factor(n, r, seed=40 + i) for i, (n, r) in enumerate(sizes)]
    F1 = [(0.95 * a.astype(np.float64) + 0.05 * gram_factor(n, r, seed=50 + i)).astype(np.float32)
          for i, (a, (n, r)) in enumerate(zip(F0, sizes))]
    Fd0 = [ctx.to_dev(f) for f in F0]
    Fd1 = [ctx.to_dev(f) for f in F1]
    Q = [torch.zeros_like(f) for f in Fd0]
    lam = [torch.zeros(f.shape[0], dtype=torch.float32, device=ctx.dev) for f in Fd0]
    info0 = K.kfac_eig(ctx.h, Fd0, Q, lam)
    again = K.kfac_eig(ctx.h, Fd0, Q, lam, warm_start=True)          # Q holds the eigenvectors of the same matrices
    torch.cuda.synchronize()
    assert all(c for (_, _, c) in again) and again[0][0] <= 1 and again[1][0] <= 1, again
    for i, F in enumerate(F0):
        check_eigpairs(F, lam[i].cpu().numpy(), Q[i].cpu().numpy(), "warm-same[%d]" % i)
    warm = K.kfac_eig(ctx.h, Fd1, Q, lam, warm_start=True)
    torch.cuda.synchronize()
    for i, F in enumerate(F1):
        check_eigpairs(F, lam[i].cpu().numpy(), Q[i].cpu().numpy(), "warm[%d]" % i)
    assert all(c for (_, _, c) in warm) and all(s >= 1 for (s, _, _) in warm), warm
    K.kfac_eig(ctx.h, Fd0, Q, lam)
    swept = K.kfac_eig(ctx.h, Fd1, Q, lam, warm_start=True, tol=5e-7)
    torch.cuda.synchronize()
    for i, F in enumerate(F1):
        check_eigpairs(F, lam[i].cpu().numpy(), Q[i].cpu().numpy(), "warm sweeps[%d]" % i)
    cold = K.kfac_eig(ctx.h, Fd1, Q, lam, tol=5e-7)
    torch.cuda.synchronize()
    print("sweeps cold", [x[0] for x in cold], "warm", [x[0] for x in swept], "first", [x[0] for x in info0])
    assert all(c for (_, _, c) in swept) and all(c for (_, _, c) in cold)
    assert 1 <= swept[0][0] < cold[0][0] and 1 <= swept[1][0] < cold[1][0]


def test_eig_warm_start_from_eigenvectors_that_still_hold(ctx):
    """Factors that have not moved, or hardly, since their eigenvectors were formed need no sweep or one; a factor of the same
    call that is another matrix altogether is decomposed anew, and so is one whose basis is of no use.  Every result is as good
    as without a start."""
    sizes = [130, 256, 257, 577, 2100, 577, 64, 300, 300]
    F0 = [gram_factor(n, 3 * n, seed=60 + i) for i, n in enumerate(sizes)]
    Fd = [ctx.to_dev(f) for f in F0]
    Q, lam = [torch.zeros_like(f) for f in Fd], [torch.zeros(f.shape[0], device=ctx.dev) for f in Fd]
    K.kfac_eig(ctx.h, Fd, Q, lam)
    same = K.kfac_eig(ctx.h, Fd[:5], Q[:5], lam[:5], warm_start=True)
    torch.cuda.synchronize()
    assert all(c and s == 0 for (s, _, c) in same), same
    for i in range(5):
        check_eigpairs(F0[i], lam[i].cpu().numpy(), Q[i].cpu().numpy(), "unmoved[%d]" % i)
    F1 = list(F0)
    F1[3] = (0.9999 * F0[3].astype(np.float64) + 1e-4 * gram_factor(577, 1731, seed=80)).astype(np.float32)
    F1[5] = gram_factor(577, 1200, seed=81)
    F1[7] = np.zeros((300, 300), np.float32)
    Q[8].fill_(float("nan"))
    for i in (3, 5, 7):
        Fd[i].copy_(torch.from_numpy(F1[i]))
    info = K.kfac_eig(ctx.h, Fd, Q, lam, warm_start=True)
    torch.cuda.synchronize()
    print("sweeps", [s for (s, _, _) in info])
    assert all(c for (_, _, c) in info) and all(info[i][0] == 0 for i in range(3)), info
    assert info[8][0] == 1, info
    for i, F in enumerate(F1):
        if i != 7:
            check_eigpairs(F, lam[i].cpu().numpy(), Q[i].cpu().numpy(), "moved or not[%d]" % i)
    assert torch.equal(lam[7], torch.zeros_like(lam[7]))
    q = Q[7].double()
    assert float((q.T.contiguous() @ q - torch.eye(300, device=ctx.dev, dtype=torch.float64)).norm()) <= 300 * 2.0 ** -22


@pytest.mark.parametrize("what", ["zeros", "nan", "scaled", "one column"])
def test_eig_warm_start_from_what_is_no_basis(ctx, what):
    """A first call with the option on, before there are eigenvectors: decomposed as without it."""
    mats = [gram_factor(n, 2 * n, seed=90 + i) for i, n in enumerate([130, 300, 577])] + [np.zeros((200, 200), np.float32)]
    Fd = [ctx.to_dev(f) for f in mats]
    Q, lam = [torch.zeros_like(f) for f in Fd], [torch.zeros(f.shape[0], device=ctx.dev) for f in Fd]
    if what != "zeros":
        K.kfac_eig(ctx.h, Fd, Q, lam)
    for q in Q:
        if what == "nan":
            q.fill_(float("nan"))
        elif what == "scaled":
            q.mul_(1.01)
        elif what == "one column":
            q[:, -1] = 0.0
    info = K.kfac_eig(ctx.h, Fd, Q, lam, warm_start=True)
    torch.cuda.synchronize()
    assert all(c and s <= 1 for (s, _, c) in info), info
    for i in range(3):
        check_eigpairs(mats[i], lam[i].cpu().numpy(), Q[i].cpu().numpy(), what)
    q = Q[3].double()
    assert float((q.T.contiguous() @ q - torch.eye(200, device=ctx.dev, dtype=torch.float64)).norm()) <= 200 * 2.0 ** -22


def _eig_seconds(ctx, mats, **kw):
    Fd = [ctx.to_dev(f) for f in mats]
    Q, lam = [torch.empty_like(f) for f in Fd], [torch.empty(f.shape[0], device=ctx.dev) for f in Fd]
    best = 1e9
    for _ in range(6):
        torch.cuda.synchronize()
        t = time.perf_counter()
        info = K.kfac_eig(ctx.h, Fd, Q, lam, **kw)
        best = min(best, time.perf_counter() - t)
    return best, info, Q, lam


@pytest.mark.parametrize("n", [64, 129, 256, 257, 577, 2100])
@pytest.mark.parametrize("off", [0.0, 1e-7])
def test_eig_diagonal_factor_costs_no_decomposition(ctx, n, off):
    """A factor that is diagonal as it stands (to the tolerance): no sweep, sorted, and a fraction of the time that a dense one of
    that size takes (an eighth to a half)."""
    rng = np.random.default_rng(n)
    dg = rng.permutation(np.linspace(0.1, 2.0, n))
    E = rng.standard_normal((n, n))
    F = (np.diag(dg) + off * np.linalg.norm(dg) / np.linalg.norm(E) * (E + E.T) / 2.0).astype(np.float32)
    t, info, Q, lam = _eig_seconds(ctx, [F])
    assert info[0][2] and info[0][0] == 0, info
    check_eigpairs(F, lam[0].cpu().numpy(), Q[0].cpu().numpy(), "diagonal")
    if off == 0.0:
        assert np.array_equal(lam[0].cpu().numpy(), np.sort(np.diag(F)))
    dense, _, _, _ = _eig_seconds(ctx, [gram_factor(n, 2 * n, seed=1)])
    print("diagonal %.0f us, dense %.0f us" % (t * 1e6, dense * 1e6))
    assert t < 0.65 * dense, (t, dense)


def test_eig_diagonal_beside_dense_factors(ctx):
    mats = [np.eye(n, dtype=np.float32) * 0.5 if i % 2 == 0 else gram_factor(n, 2 * n, seed=i) for i, n in enumerate([577, 300, 64, 64, 200, 200, 1, 130])]
    Ld, Qd, info = ctx.eig(mats)
    assert all(c for (_, _, c) in info), info
    for i, F in enumerate(mats):
        check_eigpairs(F, Ld[i].cpu().numpy(), Qd[i].cpu().numpy(), "beside[%d]" % i)


@pytest.mark.parametrize("n,count", [(260, 65), (300, 50), (257, 130)])
def test_eig_crowd_of_diagonal_factors_costs_no_decomposition(n, count):
    """More narrow factors than the first launch on the chip takes: what a decomposition of all of them costs is more than the widest's columns (65 of 260
    2.6 ms, by sweeps 1.6), so diagonal ones are left to the sweeps, of which they need none."""
    F = [torch.diag(torch.rand(n, device="cuda") + 0.5) for _ in range(count)]
    Q, lam, info = decompose_on_device(F)
    for f, q, l, i in zip(F, Q, lam, info):
        assert i[2] and i[0] == 0, i
        assert torch.equal(l, torch.diagonal(f).sort().values) and torch.equal(f @ q, q * l)


@pytest.mark.parametrize("n,moved,sweeps", [(577, 1e-2, 2), (577, 5e-2, 1), (1153, 1e-2, 2), (1153, 5e-2, 1)])
def test_eig_start_basis_moved_a_little_and_more(ctx, n, moved, sweeps):
    """Two sweeps from the eigenvectors of a factor that moved by 1 % are cheaper than a decomposition (which reports one), four after 5 % are not."""
    F0, F1 = gram_factor(n, 2 * n, seed=n), gram_factor(n, 2 * n, seed=n + 1)
    _, Q, _ = ctx.eig([F0])
    F = ((1.0 - moved) * F0 + moved * F1).astype(np.float32)
    lam = [torch.empty(n, device="cuda")]
    info = K.kfac_eig(ctx.h, [torch.from_numpy(F).cuda()], Q, lam, warm_start=True)
    assert info[0][2] and info[0][0] == sweeps, info
    check_eigpairs(F, lam[0].cpu().numpy(), Q[0].cpu().numpy(), "moved")


def test_eig_start_basis_where_columns_go_by_the_chain():
    """Where the chain of launches reduces a factor (a device without cooperative launches, columns past what fits the chip), four sweeps from
    the eigenvectors of a factor that moved by 5 % are cheaper than a decomposition: 7.6 ms, 11.7."""
    n = 1153
    F0, F1 = gram_factor(n, 2 * n, seed=n), gram_factor(n, 2 * n, seed=n + 1)
    F = (0.95 * F0 + 0.05 * F1).astype(np.float32)
    for workgroups, sweeps in ((256, 1), (0, 4)):
        c = Ctx(K.kfac_eig_workspace_bytes([n]) + 4096)
        K.lib().kfac_limit_chip(c.h, workgroups, 1 << 18)
        _, Q, _ = c.eig([F0])
        lam = [torch.empty(n, device="cuda")]
        info = K.kfac_eig(c.h, [torch.from_numpy(F).cuda()], Q, lam, warm_start=True)
        c.close()
        assert info[0][2] and info[0][0] == sweeps, (workgroups, info)
        check_eigpairs(F, lam[0].cpu().numpy(), Q[0].cpu().numpy(), "by the chain")


@pytest.mark.parametrize("n", [577, 1153])
@pytest.mark.parametrize("tol,by_sweeps", [(0.1, True), (1e-2, False), (1e-3, False)])
def test_eig_loose_tolerance_takes_the_cheaper_route(ctx, n, tol, by_sweeps):
    """To 0.1 one sweep is enough and cheaper than a decomposition; to 1e-2 it would take four, which cost more (577 wide 3.6 ms, directly 2.4).  A
    cap on the sweeps that is too low does not stand in the way of the latter."""
    F = gram_factor(n, 2 * n, seed=n)
    exact, _, _, _ = _eig_seconds(ctx, [F])
    t, info, Qd, Ld = _eig_seconds(ctx, [F], tol=tol)
    assert t <= 1.15 * exact, (t, exact)
    lam, Q = Ld[0].cpu().numpy().astype(np.float64), Qd[0].cpu().numpy().astype(np.float64)
    assert info[0][2] and 0 < info[0][0] < 3 and (1e-4 if by_sweeps else 0.0) < info[0][1] <= (tol if by_sweeps else 2e-6), info
    F64 = F.astype(np.float64)
    assert np.linalg.norm(F64 - (Q * lam) @ Q.T) <= 1.1 * tol * np.linalg.norm(F64)
    assert np.linalg.norm(Q.T @ Q - np.eye(n), 2) <= 1e-4
    Ld, Qd, info = ctx.eig([F], tol=1e-2, max_sweeps=1)
    assert info[0][2] and info[0][0] == 1, info
    check_eigpairs(F, Ld[0].cpu().numpy(), Qd[0].cpu().numpy(), "capped")


def test_eig_max_sweeps_reports_noconv(ctx):
    F = gram_factor(300, 500, seed=7)
    with pytest.raises(K.KfacError) as e:
        ctx.eig([F], max_sweeps=1, tol=1e-7)
    assert e.value.code == K.KFAC_ENOCONV
    Ld, Qd, info = ctx.eig([F], max_sweeps=1, tol=1e-7, raise_on_noconv=False)
    assert not info[0][2] and info[0][0] == 1
    assert np.isfinite(Qd[0].cpu().numpy()).all()


def test_eig_many_factors_of_one_size(ctx):
    """200 factors of one blocked size class advance as one group: every one of them gets its own norms,
    flags and eigenpairs (the group's bookkeeping is sized by its member count, not by a fixed launch)."""
    n, count = 160, 200
    mats = [gram_factor(n, 200 + 3 * i, seed=1000 + i, ones=(i % 2 == 0)) for i in range(count)]
    Ld, Qd, info = ctx.eig(mats)
    assert all(c for (_, _, c) in info), [i for i, x in enumerate(info) if not x[2]]
    for i in list(range(0, count, 7)) + [127, 128, 129, count - 1]:
        check_eigpairs(mats[i], Ld[i].cpu().numpy(), Qd[i].cpu().numpy(), "many[%d]" % i)
    for i in range(count):      # the cheap invariants on every member: trace and orthonormal first/last columns
        lam, Q = Ld[i].cpu().numpy().astype(np.float64), Qd[i].cpu().numpy().astype(np.float64)
        assert abs(lam.sum() - np.trace(mats[i].astype(np.float64))) <= 1e-5 * abs(lam).max() * n, i
        assert abs(np.linalg.norm(Q[:, 0]) - 1) < 1e-4 and abs(np.linalg.norm(Q[:, -1]) - 1) < 1e-4, i


def test_eig_is_reproducible(ctx):
    """Same input, same bits: the norms that decide convergence and the Rayleigh quotients are summed in a
    fixed order (small, flat and two-level path)."""
    mats = [gram_factor(n, r, seed=70 + i) for i, (n, r) in enumerate([(100, 300), (577, 900), (2100, 2500)])]
    L1, Q1, i1 = ctx.eig(mats)
    L2, Q2, i2 = ctx.eig(mats)
    assert i1 == i2
    for a, b in zip(L1 + Q1, L2 + Q2):
        assert torch.equal(a, b)


@pytest.mark.parametrize("n", [40, 230, 300, 2100])
def test_eig_non_finite_input(ctx, n):
    """A NaN in the factor: KFAC_ENOCONV, and every element of that factor's outputs is non-finite, while a
    healthy factor of the same call is decomposed as usual."""
    bad = gram_factor(n, 2 * n, seed=3)
    bad[n // 2, n // 3] = np.nan
    bad[n // 3, n // 2] = np.nan
    good = gram_factor(n, 2 * n, seed=4)
    with pytest.raises(K.KfacError) as e:
        ctx.eig([bad, good])
    assert e.value.code == K.KFAC_ENOCONV
    Ld, Qd, info = ctx.eig([bad, good], raise_on_noconv=False)
    assert not info[0][2] and info[1][2], info
    assert not np.isfinite(Ld[0].cpu().numpy()).any() and not np.isfinite(Qd[0].cpu().numpy()).any()
    check_eigpairs(good, Ld[1].cpu().numpy(), Qd[1].cpu().numpy(), "beside NaN")


# edges of the direct route: the register kernels' sizes (64, 128, 192, 256), the first and last sizes of a 128-wide tile,
# panels of 32 columns, back-transformation blocks of 128 reflectors and contraction pieces of 512
DIRECT_SIZES = [(3, 9), (63, 90), (64, 20), (127, 500), (191, 100), (192, 700), (193, 90), (255, 40), (256, 800), (258, 700),
                (288, 100), (383, 900), (384, 60), (385, 500), (512, 1300), (513, 200), (545, 1500), (641, 90)]


@pytest.mark.parametrize("n,rows", DIRECT_SIZES)
def test_eig_direct_at_the_edges_of_its_kernels(ctx, n, rows):
    F = gram_factor(n, rows, seed=n, ones=n % 2 == 0)
    Ld, Qd, info = ctx.eig([F])
    assert info[0][2] and info[0][0] == 1, info
    check_eigpairs(F, Ld[0].cpu().numpy(), Qd[0].cpu().numpy(), "direct")


def _special(kind, n):
    rng = np.random.default_rng(n)
    if kind == "ones":                   # rank one: n - 1 zeros
        return np.ones((n, n))
    if kind == "identity plus":          # n - 1 equal eigenvalues
        return 3.0 * np.eye(n) + np.ones((n, n))
    if kind == "mostly zero":            # decoupled rows
        return np.diag((np.arange(n) < 3) * 1.0)
    if kind == "equal blocks":           # every eigenvalue of a block n / 4 times
        return np.kron(np.eye(n // 4), np.ones((4, 4)))
    if kind == "repeated gram":          # generic spectrum, every eigenvalue four times
        return np.kron(np.eye(4), gram_factor(n // 4, n, seed=n).astype(np.float64))
    if kind == "pairs":                  # eigenvalues in pairs that agree to 1e-14, eigenvectors not local
        m = n // 2 * 2 + 1
        return np.diag(np.abs(np.arange(m) - m // 2).astype(np.float64)) + np.diag(np.ones(m - 1), 1) + np.diag(np.ones(m - 1), -1)
    if kind == "tiny":                   # squares below the range of fp32
        return gram_factor(n, 2 * n, seed=n).astype(np.float64) * 1e-30
    d = 10.0 ** rng.uniform(-4, 0.5, n)  # graded: eigenvalues over nine decades
    return gram_factor(n, 3 * n, seed=n, ones=False).astype(np.float64) * d[:, None] * d[None, :]


@pytest.mark.parametrize("n", [100, 300])
@pytest.mark.parametrize("kind", ["ones", "identity plus", "mostly zero", "equal blocks", "repeated gram", "pairs", "tiny", "graded"])
def test_eig_direct_on_special_spectra(ctx, kind, n):
    """Multiple, zero and nearly equal eigenvalues: the eigenvectors come out orthonormal without the Jacobi route's help
    (which would report several sweeps), within the same bounds as any other factor."""
    F = _special(kind, n).astype(np.float32)
    Ld, Qd, info = ctx.eig([F])
    assert info[0][2] and info[0][0] <= 1, info
    scale = 1e30 if kind == "tiny" else 1.0
    check_eigpairs((F.astype(np.float64) * scale).astype(np.float32), Ld[0].cpu().numpy().astype(np.float64) * scale, Qd[0].cpu().numpy(), kind)


@pytest.mark.parametrize("n,rows,seed", [(4609, 3136, 0), (4609, 3136, 1), (4609, 3136, 2), (4609, 3136, 3), (8192, 2000, 0)])
def test_eig_direct_large_graded_and_rank_deficient(n, rows, seed):
    """Features scaled over four decades, fewer rows than columns: thousands of eigenvalues around 1e-11 of the largest with
    localised eigenvectors, some of which agree to more digits than fp64 has at the largest one.  The direct route has to tell
    them apart (one sweep reported: Jacobi iteration was not needed).  8192: the largest size, past 32 row blocks."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    X = torch.randn((rows, n), generator=gen, device="cuda").relu_() * 10.0 ** (torch.rand(n, generator=gen, device="cuda") * 4.0 - 3.0)
    X[:, -1] = 1.0
    F = (X.double().T.contiguous() @ X.double() / rows).float()
    F = ((F + F.T) * 0.5).contiguous()
    c = Ctx(K.kfac_eig_workspace_bytes([n]) + 4096)
    Q, lam = torch.empty_like(F), torch.empty(n, device="cuda")
    info = K.kfac_eig(c.h, [F], [Q], [lam])
    torch.cuda.synchronize()
    c.close()
    assert info[0][2] and info[0][0] == 1, info
    assert bool((lam[1:] >= lam[:-1]).all())
    Fd, Qd = F.double(), Q.double()
    assert float((Fd @ Qd - Qd * lam.double()).norm() / Fd.norm()) <= TOL_RES
    # n^2 inner products of unit vectors that are rounded to fp32: 2^-24 apiece
    assert float((Qd.T.contiguous() @ Qd - torch.eye(n, device="cuda", dtype=torch.float64)).norm()) <= n * 2.0 ** -24


def two_clusters(n, seed):
    """Eigenvalues around 1 and around -1, each half within 1e-4, and a dense basis: what the direct route has the largest residual for, since
    the rounding inside a cluster is not corrected."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    B = torch.linalg.qr(torch.randn((n, n), generator=gen, device="cuda", dtype=torch.float64))[0].contiguous()
    lam = 1.0 + 1e-4 * torch.rand(n, generator=gen, device="cuda", dtype=torch.float64)
    lam[::2] *= -1.0
    F = (B * lam) @ B.T.contiguous()
    return ((F + F.T) * 0.5).float().cpu().numpy()


@pytest.mark.parametrize("tol", [1e-6, 0.0])
def test_eig_converged_means_within_the_callers_tolerance(ctx, tol):
    """Two clusters of 2300 eigenvalues come out of the direct route about 1.3e-6 ||F|| off: within the default tolerance of 2e-6, not
    within 1e-6.  There the factor is decomposed by Jacobi sweeps, between two factors of the same call that are not."""
    mats = [gram_factor(300, 900, seed=1), two_clusters(4600, 2), gram_factor(100, 300, seed=3)]
    Ld, Qd, info = ctx.eig(mats, tol=tol)
    for i, F in enumerate(mats):
        assert info[i][2] and info[i][1] <= (tol or 2e-6), info
        check_eigpairs(F, Ld[i].cpu().numpy(), Qd[i].cpu().numpy(), "tol[%d]" % i)
    assert info[0][0] == 1 and info[2][0] == 1 and (info[1][0] > 1) == (tol == 1e-6), info


@pytest.mark.parametrize("sizes,ws", [([64] * 12 + [17, 100, 128], 1 << 16), ([145, 16], 320 << 10), ([300, 577, 129], 6 << 20)])
def test_eig_in_a_workspace_that_holds_jacobi_sweeps_only(sizes, ws):
    """Less than the direct decomposition takes: iterated instead, not refused."""
    assert K.kfac_eig_workspace_bytes(sizes) > ws
    c = Ctx(ws)
    mats = [gram_factor(n, 2 * n, seed=n + i) for i, n in enumerate(sizes)]
    Ld, Qd, info = c.eig(mats)
    c.close()
    for i, F in enumerate(mats):
        assert info[i][2] and info[i][0] > 1, info
        check_eigpairs(F, Ld[i].cpu().numpy(), Qd[i].cpu().numpy(), "little workspace[%d]" % i)


@pytest.mark.parametrize("n", [300, 577])
def test_eig_fp32_only_keeps_small_eigenvalues_of_a_graded_factor(ctx, n):
    """Features scaled over four decades: with fp32_only, eigenvalues down to 1e-9 of the largest are accurate on their own
    scale (a reduction to tridiagonal form leaves some of them 1e-2 and more off).  Rotations keep that scale; what is left is
    the off-diagonal norm at which the sweeps stop, 2e-6 ||F||: all of it in one entry beside the largest eigenvalue would move one
    of 1e-9 by (2e-6)^2 / 1e-9 of itself.  (Measured: 1.4e-4 at 300.)  An fp64 solver resolves them to 1e-6."""
    rng = np.random.default_rng(n)
    d = 10.0 ** rng.uniform(-4, 0, n)
    F = (gram_factor(n, 3 * n, seed=n, ones=False).astype(np.float64) * d[:, None] * d[None, :]).astype(np.float32)
    Ld, Qd, info = ctx.eig([F], fp32_only=True)
    lam = Ld[0].cpu().numpy().astype(np.float64)
    assert info[0][2], info
    check_eigpairs(F, lam, Qd[0].cpu().numpy(), "graded fp32")
    ref = np.linalg.eigvalsh(F.astype(np.float64))
    sel = ref > 1e-9 * ref.max()
    err = np.abs(lam - ref)[sel] / ref[sel]
    print("%d eigenvalues, largest relative error %.1e" % (sel.sum(), err.max()))
    assert err.max() <= 4e-3


# Jacobi sweeps: what tolerances below 1e-6 and fp32_only ask for.  In LDS (64, 128), flat (129 to 640), two-level (2100).
SWEEPS = [dict(tol=5e-7), dict(fp32_only=True)]


@pytest.mark.parametrize("n,rows", [(2, 5), (64, 20), (128, 300), (129, 100), (145, 2048), (577, 300), (640, 900), (2100, 2500)])
@pytest.mark.parametrize("kw", SWEEPS, ids=["tol", "fp32_only"])
def test_eig_by_sweeps(ctx, n, rows, kw):
    F = gram_factor(n, rows, seed=n + 5)
    Ld, Qd, info = ctx.eig([F], **kw)
    assert info[0][2] and info[0][0] >= min(n - 1, 3) and info[0][1] <= kw.get("tol", 2e-6), info
    check_eigpairs(F, Ld[0].cpu().numpy(), Qd[0].cpu().numpy(), "sweeps")


def test_eig_by_sweeps_mixed_sizes_repeatable_and_beside_nan(ctx):
    """A batch over all three forms: every member's eigenpairs, the same bits again, and a factor with a NaN or an infinity only
    spoils its own outputs, and says so."""
    sizes = [(16, 50), (145, 500), (2100, 2600), (10, 3), (289, 100), (128, 64), (2300, 900), (289, 900), (577, 1500)]
    mats = [gram_factor(n, r, seed=300 + i, ones=(i % 2 == 0)) for i, (n, r) in enumerate(sizes)]
    L1, Q1, i1 = ctx.eig(mats, tol=5e-7)
    L2, Q2, i2 = ctx.eig(mats, tol=5e-7)
    assert i1 == i2 and all(c and s > 1 for (s, _, c) in i1), i1
    for i, F in enumerate(mats):
        assert torch.equal(L1[i], L2[i]) and torch.equal(Q1[i], Q2[i]), i
        check_eigpairs(F, L1[i].cpu().numpy(), Q1[i].cpu().numpy(), "sweeps[%d]" % i)
    bad = {0: np.nan, 1: np.nan, 2: np.inf, 4: np.inf, 5: np.inf, 6: np.nan}
    for b, x in bad.items():
        mats[b] = mats[b].copy()
        mats[b][3, 5] = mats[b][5, 3] = x
    for kw in (dict(tol=5e-7), dict()):        # by sweeps; directly
        with pytest.raises(K.KfacError) as e:
            ctx.eig(mats, **kw)
        assert e.value.code == K.KFAC_ENOCONV
        L3, Q3, i3 = ctx.eig(mats, raise_on_noconv=False, **kw)
        for i in range(len(mats)):
            if i in bad:
                assert not i3[i][2] and not torch.isfinite(L3[i]).any() and not torch.isfinite(Q3[i]).any(), i
            else:
                assert i3[i][2] and float((L3[i] - L1[i]).abs().max()) <= TOL_LAM * float(L1[i].max()), i
                check_eigpairs(mats[i], L3[i].cpu().numpy(), Q3[i].cpu().numpy(), "beside nan[%d]" % i)


def test_eig_direct_many_large_factors(ctx):
    """Large and small factors in one call, more than the chip holds at once, so that some wait until others have shrunk: every result as
    good as a single factor's, and complete when the call returns."""
    dims = [2900, 1300, 2900, 100, 2900, 20, 2900, 2900, 300, 2900]
    gen = torch.Generator(device="cuda").manual_seed(5)
    F = []
    for n in dims:
        X = torch.randn((2 * n, n), generator=gen, device="cuda")
        G = X.T.contiguous() @ X / (2 * n)
        F.append(((G + G.T) * 0.5).contiguous())
    c = Ctx(K.kfac_eig_workspace_bytes(dims) + 4096)
    Q, lam = [torch.empty_like(f) for f in F], [torch.empty(n, device="cuda") for n in dims]
    info = K.kfac_eig(c.h, F, Q, lam)
    for f, q, l, n, i in zip(F, Q, lam, dims, info):     # on the caller's stream, without a synchronisation in between
        assert i[2] and i[0] == 1, (n, i)
        fd, qd = f.double(), q.double()
        assert float((fd @ qd - qd * l.double()).norm() / fd.norm()) <= TOL_RES, n
        assert float((qd.T.contiguous() @ qd - torch.eye(n, device="cuda", dtype=torch.float64)).norm()) <= max(n, 16) * 2.0 ** -22, n
    c.close()


def gram_on_device(dims, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    F = []
    for n in dims:
        X = torch.randn((2 * n, n), generator=gen, device="cuda")
        G = X.T.contiguous() @ X / (2 * n)
        F.append(((G + G.T) * 0.5).contiguous())
    torch.cuda.synchronize()
    return F


def decompose_on_device(F):
    """One call on the current stream: eigenvectors, eigenvalues, info."""
    dims = [f.shape[0] for f in F]
    c = Ctx(K.kfac_eig_workspace_bytes(dims) + 4096)
    Q, lam = [torch.empty_like(f) for f in F], [torch.empty(n, device="cuda") for n in dims]
    info = K.kfac_eig(c.h, F, Q, lam)
    c.close()
    return Q, lam, info


# the reduction on the chip: first and last matrix of every number of column slots (512 k wide, without the first column), the widest one, the
# narrowest that begins with columns by the chain of launches, more factors than fit at once; then the same edges of the narrow workgroups (256 k),
# in calls that crowd the chip from the first launch on (a factor counts for a sixteenth of its columns; 256 and more are a crowd)
@pytest.mark.parametrize("dims", [[257, 513], [514, 258], [1025, 1026], [1537, 1538], [2049, 2050], [2561, 2562], [3073, 3074], [3585, 3586], [4097, 4098],
                                  [4609], [4610, 300], [1025] * 14 + [300] * 60,
                                  [257, 258] * 10, [513, 514] * 5, [769, 770] * 3, [1025, 1026] * 3, [1281, 1282] * 2, [1537, 1538] * 2, [1793, 1794] * 2,
                                  [2049] * 3 + [1000], [2050, 2049, 2049]])
def test_eig_reduction_at_the_edges_of_its_column_slots(dims):
    F = gram_on_device(dims, 11)
    Q, lam, info = decompose_on_device(F)
    for f, q, l, n, i in zip(F, Q, lam, dims, info):
        assert i[2] and i[0] == 1, (n, i)          # one sweep: the direct route's own result
        fd, qd = f.double(), q.double()
        assert float((fd @ qd - qd * l.double()).norm() / fd.norm()) <= TOL_RES, n
        assert float((qd.T.contiguous() @ qd - torch.eye(n, device="cuda", dtype=torch.float64)).norm()) <= max(n, 16) * 2.0 ** -22, n


def spectrum(n, kind, gen):
    """Eigenvalues, and a dense orthogonal basis for them, in fp64."""
    u = torch.rand(n, generator=gen, device="cuda", dtype=torch.float64)
    lam = {"spread": 1.0 + u, "narrow": 1.0 + 0.02 * u, "clusters": 1.0 + torch.floor(4 * u) + 1e-9 * u, "repeated": 1.0 + torch.floor(8 * u),
           "indefinite": 2.0 * u - 1.0, "one large": torch.where(torch.arange(n, device="cuda") == 0, 1e4, 1.0 + u)}[kind]
    return lam, torch.linalg.qr(torch.randn((n, n), generator=gen, device="cuda", dtype=torch.float64))[0].contiguous()


# what the reduction on the chip rounds more than once per panel is taken out again: residuals as they were with a rounding per panel (4 to
# 6.5e-7 for Gram matrices, up to 1.03e-6 for random symmetric ones at 4609), so that a tol of 1e-6 is still met directly
@pytest.mark.parametrize("n,samples", [(577, 30), (1153, 30), (1153, 2), (2305, 2), (2305, 30), (4609, 2)])
def test_eig_direct_residual_of_wide_gram_factors(n, samples):
    gen = torch.Generator(device="cuda").manual_seed(n)
    X = torch.randn((samples * n, n), generator=gen, device="cuda")
    G = X.T.contiguous() @ X / (samples * n)
    F = ((G + G.T) * 0.5).contiguous()
    c = Ctx(K.kfac_eig_workspace_bytes([n]) + 4096)
    Q, lam = torch.empty_like(F), torch.empty(n, device="cuda")
    info = K.kfac_eig(c.h, [F], [Q], [lam], tol=1e-6)
    c.close()
    assert info[0][2] and info[0][0] == 1, info
    fd, qd = F.double(), Q.double()
    assert float((fd @ qd - qd * lam.double()).norm() / fd.norm()) <= 7e-7
    assert float((qd.T.contiguous() @ qd - torch.eye(n, device="cuda", dtype=torch.float64)).norm()) <= n * 2.0 ** -22


# the correction of the eigenvectors: edges of its tiles and of the split-fp16 products' slabs, spectra whose gaps are all small, partly none at
# all or of both signs, factors of any scale
@pytest.mark.parametrize("kind", ["spread", "narrow", "clusters", "repeated", "indefinite", "one large"])
@pytest.mark.parametrize("n,scale", [(257, 1.0), (383, 1e-12), (384, 1.0), (641, 1e9), (2049, 1.0)])
def test_eig_corrected_eigenvectors(n, scale, kind):
    lam64, B = spectrum(n, kind, torch.Generator(device="cuda").manual_seed(n))
    F = (scale * ((B * lam64) @ B.T.contiguous())).float()
    F = ((F + F.T) * 0.5).contiguous()
    Q, lam, info = decompose_on_device([F])
    assert info[0][2] and info[0][0] == 1, info
    fd, qd = F.double(), Q[0].double()
    assert float((fd @ qd - qd * lam[0].double()).norm() / fd.norm()) <= 7e-7
    assert float((qd.T.contiguous() @ qd - torch.eye(n, device="cuda", dtype=torch.float64)).norm()) <= n * 2.0 ** -22
    assert float((lam[0].double() - scale * lam64.sort().values).abs().max()) <= 1e-6 * scale * float(lam64.abs().max())


def decompose_with(F, workgroups, polls):
    """As decompose_on_device(), the reduction on the chip limited to so many workgroups and looks at the others' words."""
    dims = [f.shape[0] for f in F]
    c = Ctx(K.kfac_eig_workspace_bytes(dims) + 4096)
    K.lib().kfac_limit_chip(c.h, workgroups, polls)
    Q, lam = [torch.empty_like(f) for f in F], [torch.empty(n, device="cuda") for n in dims]
    info = K.kfac_eig(c.h, F, Q, lam)
    c.close()
    for f, q, l, n, i in zip(F, Q, lam, dims, info):
        assert i[2] and i[0] == 1, (n, i)
        fd, qd = f.double(), q.double()
        assert float((fd @ qd - qd * l.double()).norm() / fd.norm()) <= 7e-7, n
        assert float((qd.T.contiguous() @ qd - torch.eye(n, device="cuda", dtype=torch.float64)).norm()) <= max(n, 16) * 2.0 ** -22, n
    return Q + lam


# compute units held by other kernels: a workgroup that does not find the others' words gives up (here: at its first look).  The factor is then
# decomposed with the chain of launches, to the last bit as if there were nothing else
@pytest.mark.parametrize("dims", [[1025], [4611], [2050, 300, 100, 700, 257]])
def test_eig_reduction_on_the_chip_given_up(dims):
    F = gram_on_device(dims, 31)
    got, chain = decompose_with(F, 256, 0), decompose_with(F, 0, 0)
    assert len(dims) > 1 or all(torch.equal(a, b) for a, b in zip(got, chain))


# a stream that may use few compute units (columns by the chain of launches until the rest fits), a device without launches of that kind, and
# more workgroups than can be resident: the launch is refused, and the chain serves the call
@pytest.mark.parametrize("workgroups", [0, 1, 5, 40, 64, 4096])
def test_eig_reduction_on_part_of_the_chip(workgroups):
    decompose_with(gram_on_device([1300, 700] + [1025] * (14 if workgroups > 256 else 1) + [90], 41), workgroups, 1 << 18)


def test_eig_columns_by_the_chain_do_not_wait_on_the_chip():
    """6145 wide, a quarter of the columns go by the chain of launches and the rest on the chip: less than all of them by the chain (72 ms and 99;
    with the chip's launches already queued behind the chain it was 122)."""
    F = gram_on_device([6145], 71)
    Q, lam, c = [torch.empty_like(F[0])], [torch.empty(6145, device="cuda")], Ctx(K.kfac_eig_workspace_bytes([6145]) + 4096)
    took = []
    for workgroups in (256, 0):
        K.lib().kfac_limit_chip(c.h, workgroups, 1 << 18)
        best = 1e9
        for _ in range(3):
            torch.cuda.synchronize()
            t = time.perf_counter()
            info = K.kfac_eig(c.h, F, Q, lam)
            best = min(best, time.perf_counter() - t)
            assert info[0][2] and info[0][0] == 1, info
        took.append(best)
    c.close()
    assert took[0] < 0.9 * took[1], took


OTHER_PROCESS = """
import sys
sys.path[:0] = [{root!r}, {tests!r}]
import torch
from test_gpu_parity import decompose_on_device, gram_on_device
F = gram_on_device([1300, 600], 51)
print("ready", flush=True)
for _ in range(40):
    assert all(i[2] and i[0] == 1 for i in decompose_on_device(F)[2])
print("done", flush=True)
"""


def test_eig_of_two_processes_at_once():
    """The device serves launches that need all their workgroups at once to one process at a time and refuses them to others: these calls
    get the chain of launches."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    code = OTHER_PROCESS.format(root=root, tests=os.path.join(root, "tests"))
    other = subprocess.Popen([sys.executable, "-c", code], stdout=subprocess.PIPE, text=True)
    try:
        assert other.stdout.readline() == "ready\n"
        F = gram_on_device([1300, 600], 52)
        while other.poll() is None:
            assert all(i[2] and i[0] == 1 for i in decompose_on_device(F)[2])
        assert other.wait() == 0 and other.stdout.read() == "done\n"
    finally:
        other.kill()
        other.wait()


def test_eig_reductions_of_two_threads_at_once():
    """Two contexts on streams of their own, each of which wants the whole chip: both come out as they do alone, bit by bit."""
    F = [gram_on_device(d, 21) for d in ([2050, 700], [1600, 1600])]
    alone = [decompose_on_device(f) for f in F]
    got = [[], []]

    def work(k):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(3):
                got[k].append(decompose_on_device(F[k]))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for a, results in zip(alone, got):
        assert len(results) == 3
        for g in results:
            assert a[2] == g[2]
            assert all(torch.equal(x, y) for x, y in zip(a[0] + a[1], g[0] + g[1]))


@pytest.mark.parametrize("N,d,T,bf16,layout", [(32, 144, 64, False, K.KFAC_LAYOUT_NDT), (9, 130, 49, False, K.KFAC_LAYOUT_NDT), (40, 257, 64, True, K.KFAC_LAYOUT_NDT),
                                                (1111, 70, 1, False, K.KFAC_LAYOUT_RD), (3, 17, 3, False, K.KFAC_LAYOUT_NDT)])
def test_update_factors_batch_too_small_for_the_machine(N, d, T, bf16, layout):
    """A batch of two factors is cut into shorter jobs than a large one, if its workspace holds their partial sums, and into
    the usual ones if it does not: the same factors either way."""
    gen = torch.Generator(device="cuda").manual_seed(d)
    shapes = [(N, d, T), (N, 16, T)] if layout == K.KFAC_LAYOUT_NDT else [(N, d), (N, 16)]
    X = [torch.randn(s, generator=gen, device="cuda").to(torch.bfloat16 if bf16 else torch.float32) for s in shapes]
    for ws in (64 << 20, 1 << 16):
        c = Ctx(ws)
        F = [torch.zeros((x.shape[1] + 1, x.shape[1] + 1), device="cuda") for x in X]
        K.kfac_update_factors_batched(c.h, [dict(X=x, dtype=K.KFAC_BF16 if bf16 else K.KFAC_F32, layout=layout, N=N, d=x.shape[1], T=T, append_ones=1,
                                                 scale=1.0 / (N * T), decay=0.0, F=f) for x, f in zip(X, F)])
        torch.cuda.synchronize()
        c.close()
        for x, f in zip(X, F):
            rows = (x.double().permute(0, 2, 1).reshape(N * T, -1) if x.dim() == 3 else x.double()).cpu().numpy()
            assert relfro(f.cpu().numpy(), oracle.gram(rows, 1, 1.0 / (N * T))) <= 1e-6, (ws, x.shape)


# 128 m and up to 64 more features: the last row of tiles in slices of 32 columns, its diagonal tile with the contraction shared by the waves
# (one or two 32-wide blocks of it); more than 64: under the map of quadrants
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("d", [31, 33, 64, 129, 144, 160, 161, 192, 193, 320, 321])
def test_update_factors_ragged_last_tiles(d, bf16):
    """Sums of products of integers up to 8, below 2^24: exact in fp32 whatever the order."""
    gen = torch.Generator(device="cuda").manual_seed(d)
    N, T = 6, 49
    X = torch.randint(-8, 9, (N, d, T), generator=gen, device="cuda").to(torch.bfloat16 if bf16 else torch.float32)
    rows = torch.cat([X.double().permute(0, 2, 1).reshape(N * T, d), torch.ones((N * T, 1), device="cuda", dtype=torch.float64)], 1)
    want = (rows.T.contiguous() @ rows).float()
    c = Ctx(64 << 20)
    F = [torch.full((d + 1, d + 1), float("nan"), device="cuda") for _ in range(3)]
    K.kfac_update_factors(c.h, X, K.KFAC_LAYOUT_NDT, N, d, T, 1, 1.0, 0.0, F[0], dtype=K.KFAC_BF16 if bf16 else K.KFAC_F32)
    K.kfac_update_factors_batched(c.h, [dict(X=X, dtype=K.KFAC_BF16 if bf16 else K.KFAC_F32, layout=K.KFAC_LAYOUT_NDT, N=N, d=d, T=T, append_ones=1,
                                             scale=1.0, decay=0.0, F=f) for f in F[1:]])
    torch.cuda.synchronize()
    c.close()
    for f in F:
        assert torch.equal(f, want)


# ------------------------------------------------------------------ precondition
# (230, 100) and (97, 200): edge tiles between 65 and 127 wide and tall (accumulator blocks masked under the full
# wave map); the others: edge tiles at most 64 wide or tall (the waves share them in slices)
PRECOND_CASES = [(10, 4), (145, 16), (65, 10), (289, 32), (577, 64), (130, 257), (230, 100), (97, 200)]


@pytest.mark.parametrize("dA,dG", PRECOND_CASES)
@pytest.mark.parametrize("bf16", [False, True])
def test_precondition_matches_oracle(ctx, dA, dG, bf16):
    rng = np.random.default_rng(8)
    A = gram_factor(dA, 3 * dA, seed=dA).astype(np.float64)
    G = oracle.gram(rng.standard_normal((3 * dG, dG)) * 1e-2, 0, 1.0 / (3 * dG))
    lamA, QA = oracle.eigh(A)
    lamG, QG = oracle.eigh(G)
    gamma = 1e-3 * lamA.mean() * lamG.mean()
    grad = (rng.standard_normal((dG, dA)) * 1e-2).astype(np.float32)
    if bf16:
        grad = S.bf16_bits_to_f32(S.to_bf16_bits(grad)).reshape(grad.shape)
    ref = oracle.precondition(QA, lamA, QG, lamG, gamma, grad)
    gd = ctx.to_dev(grad, bf16)
    K.kfac_precondition(ctx.h, ctx.to_dev(QA.astype(np.float32)), ctx.to_dev(lamA.astype(np.float32)),
                        ctx.to_dev(QG.astype(np.float32)), ctx.to_dev(lamG.astype(np.float32)), gamma, gd)
    torch.cuda.synchronize()
    got = gd.float().cpu().numpy()
    assert relfro(got, ref) <= (TOL_BF16 if bf16 else TOL_F32)


@pytest.mark.parametrize("bf16", [False, True])
def test_precondition_in_small_and_large_tiles(bf16):
    """The same layers in a call of few tiles and beside a layer that fills the machine (tiles of 64 and of 128), against fp64.  Four products of
    up to 600 terms with orthogonal matrices: fp32 sums are off by less than 4 sqrt(600) 2^-24 = 6e-6; a rounding of the result to bf16 by 2^-9."""
    gen = torch.Generator(device="cuda").manual_seed(4)
    sizes = PRECOND_CASES + [(64, 64), (128, 65), (129, 63), (4, 1), (2500, 2500)]
    basis = lambda n: torch.linalg.qr(torch.randn((n, n), generator=gen, device="cuda", dtype=torch.float64))[0].contiguous()
    QA, QG = [basis(a) for a, _ in sizes], [basis(g) for _, g in sizes]
    lamA, lamG = [torch.rand(a, generator=gen, device="cuda") for a, _ in sizes], [torch.rand(g, generator=gen, device="cuda") for _, g in sizes]
    grads = [torch.randn((g, a), generator=gen, device="cuda").to(torch.bfloat16 if bf16 else torch.float32) for a, g in sizes]
    c = Ctx(256 << 20)
    for count in (len(sizes) - 1, len(sizes)):
        got = [g.clone() for g in grads[:count]]
        nu = torch.empty(1, device="cuda")
        K.kfac_precondition_batched_scaled(c.h, [q.float() for q in QA[:count]], lamA[:count], [q.float() for q in QG[:count]], lamG[:count], 0.1, got,
                                           kappa=1e30, lr=0.1, nu=nu)
        torch.cuda.synchronize()
        assert float(nu) == 1.0
        for qa, qg, la, lg, g, x in zip(QA, QG, lamA, lamG, grads, got):
            v = (qg.T.contiguous() @ g.double() @ qa) / (lg.double()[:, None] * la.double()[None, :] + 0.1)
            want = qg @ v @ qa.T.contiguous()
            assert float((x.double() - want).norm() / want.norm()) <= (2.0 ** -8 if bf16 else 1.5e-5), (count, x.shape)
    c.close()


@pytest.mark.parametrize("dA,dG", PRECOND_CASES + [(1000, 300), (4, 1)])
@pytest.mark.parametrize("bf16", [False, True])
def test_precondition_split_f16_matches_oracle(ctx, dA, dG, bf16):
    """The same step with the GEMM chain on the split-fp16 engine (operands of any extent and alignment, per-layer
    power-of-two scales from the gradient's and V2's Frobenius norms), to the same bar as the fp32 chain; a
    gradient scaled far outside fp16's range (1e-9, 1e+6) must come out the same, and a zero gradient stays zero."""
    rng = np.random.default_rng(8)
    A = gram_factor(dA, 3 * dA, seed=dA).astype(np.float64)
    G = oracle.gram(rng.standard_normal((3 * dG, dG)) * 1e-2, 0, 1.0 / (3 * dG))
    lamA, QA = oracle.eigh(A)
    lamG, QG = oracle.eigh(G)
    gamma = 1e-3 * lamA.mean() * lamG.mean()
    dev = [ctx.to_dev(QA.astype(np.float32)), ctx.to_dev(lamA.astype(np.float32)),
           ctx.to_dev(QG.astype(np.float32)), ctx.to_dev(lamG.astype(np.float32))]
    for mag in (1e-2, 1e-9, 1e6, 0.0):
        grad = (rng.standard_normal((dG, dA)) * mag).astype(np.float32)
        if bf16:
            grad = S.bf16_bits_to_f32(S.to_bf16_bits(grad)).reshape(grad.shape)
        ref = oracle.precondition(QA, lamA, QG, lamG, gamma, grad)
        gd = ctx.to_dev(grad, bf16)
        K.kfac_precondition_batched(ctx.h, [dev[0]], [dev[1]], [dev[2]], [dev[3]], gamma, [gd], split_f16=True)
        torch.cuda.synchronize()
        got = gd.float().cpu().numpy()
        assert np.isfinite(got).all()
        if mag == 0.0:
            assert not got.any()
        else:
            assert relfro(got, ref) <= (TOL_BF16 if bf16 else TOL_F32), (mag, relfro(got, ref))


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("split", [False, True])
def test_precondition_batched_with_gradient_scaling(ctx, bf16, split):
    """Sec. V-C: the batched preconditioner followed by nu = min(1, sqrt(kappa / (lr^2 sum_l |<P_l, g_l>|))).
    Three layers of different tile counts (one tile, ragged tiles, several tiles) in one call, against the oracle
    end to end, against the oracle's nu on the library's own unscaled output, and with a kappa that does not clip."""
    rng = np.random.default_rng(11)
    dims = [(65, 16), (300, 130), (145, 257)]
    QAs, lAs, QGs, lGs, grads, refs = [], [], [], [], [], []
    gamma = None
    for dA, dG in dims:
        A = gram_factor(dA, 3 * dA, seed=dA).astype(np.float64)
        G = oracle.gram(rng.standard_normal((3 * dG, dG)), 0, 1.0 / (3 * dG))
        lamA, QA = oracle.eigh(A)
        lamG, QG = oracle.eigh(G)
        gamma = 1e-2
        grad = (rng.standard_normal((dG, dA)) * 1e-2).astype(np.float32)
        if bf16:
            grad = S.bf16_bits_to_f32(S.to_bf16_bits(grad)).reshape(grad.shape)
        refs.append(oracle.precondition(QA, lamA, QG, lamG, gamma, grad))
        QAs.append(ctx.to_dev(QA.astype(np.float32))); lAs.append(ctx.to_dev(lamA.astype(np.float32)))
        QGs.append(ctx.to_dev(QG.astype(np.float32))); lGs.append(ctx.to_dev(lamG.astype(np.float32)))
        grads.append(grad)
    tol = TOL_BF16 if bf16 else TOL_F32
    # unscaled output of the library, for the same inputs
    plain = [ctx.to_dev(g, bf16) for g in grads]
    K.kfac_precondition_batched(ctx.h, QAs, lAs, QGs, lGs, gamma, plain, split_f16=split)
    torch.cuda.synchronize()
    plain = [p.float().cpu().numpy().astype(np.float64) for p in plain]
    lr = 0.1
    s_sum = sum(abs(float((p * g).sum())) for p, g in zip(plain, grads))
    for kappa, clipped in [(1e-3 * lr * lr * s_sum, True), (10.0 * lr * lr * s_sum, False)]:
        gd = [ctx.to_dev(g, bf16) for g in grads]
        nu_d = torch.full((1,), float("nan"), dtype=torch.float32, device=ctx.dev)
        K.kfac_precondition_batched_scaled(ctx.h, QAs, lAs, QGs, lGs, gamma, gd, kappa, lr, nu_d, split_f16=split)
        torch.cuda.synchronize()
        nu = float(nu_d.item())
        nu_own = oracle.grad_scale(plain, grads, kappa, lr)          # oracle formula on the library's own P_l
        nu_ref = oracle.grad_scale(refs, grads, kappa, lr)           # oracle end to end
        assert (nu < 1.0) == clipped
        assert abs(nu - nu_own) <= 2e-6 * nu_own
        assert abs(nu - nu_ref) <= tol * nu_ref
        if clipped:
            assert nu == pytest.approx(np.sqrt(1e-3), rel=1e-5)
        for j in range(len(dims)):
            got = gd[j].float().cpu().numpy()
            assert relfro(got, nu_ref * refs[j]) <= tol
            assert relfro(got, nu * plain[j]) <= (4e-3 if bf16 else 1e-6)   # bf16: one more rounding of the product
    with pytest.raises(K.KfacError):
        K.kfac_precondition_batched_scaled(ctx.h, QAs, lAs, QGs, lGs, gamma, gd, 0.0, lr, nu_d)


def test_gradient_scaling_of_many_layers_and_tiles():
    """More layers and tiles than one round of the sum's waves and lanes: nu against the fp64 sum over the unscaled results (own rounding 2^-24, that of
    the results' storage averages out below it), the same in every call.  The sum must not take long beside the products: one tile
    after another it took 47 us for the twenty layers here."""
    gen = torch.Generator(device="cuda").manual_seed(6)
    R = lambda *s: torch.randn(s, generator=gen, device="cuda")
    for sizes in ([(1, 1)], [(65 + 9 * i, 40 + 7 * i) for i in range(33)] + [(1100, 1000)], [(496, 280)] * 20, [(2049, 2048)]):
        args = [R(a, a) / a ** 0.5 for a, _ in sizes], [R(a).abs() for a, _ in sizes], [R(g, g) / g ** 0.5 for _, g in sizes], [R(g).abs() for _, g in sizes], 0.1
        grads = [R(g, a) for a, g in sizes]
        c = Ctx(K.kfac_precondition_workspace_bytes(sizes))
        plain, nu = [g.clone() for g in grads], torch.empty(1, device="cuda")
        K.kfac_precondition_batched(c.h, *args, plain)
        total = sum(abs(float((p.double() * g.double()).sum())) for p, g in zip(plain, grads))
        for _ in range(2):
            got = [g.clone() for g in grads]
            K.kfac_precondition_batched_scaled(c.h, *args, got, kappa=1e-4 * total, lr=0.1, nu=nu)
            assert abs(float(nu) - 0.1) <= 2e-7, (len(sizes), float(nu))
            assert all(torch.equal(x, p * nu) for x, p in zip(got, plain))

        def us(scaled):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(10):
                if scaled:
                    K.kfac_precondition_batched_scaled(c.h, *args, plain, kappa=1e30, lr=0.1, nu=nu)
                else:
                    K.kfac_precondition_batched(c.h, *args, plain)
            e1.record()
            torch.cuda.synchronize()
            return e0.elapsed_time(e1) * 100
        if len(sizes) == 20:
            with_nu, without = min(us(True) for _ in range(5)), min(us(False) for _ in range(5))
            assert with_nu <= without + 30, (sizes[0], with_nu, without)
        c.close()


@pytest.mark.parametrize("dA,dG", [(145, 16), (300, 130), (577, 64), (230, 100)])
def test_explicit_inverse_method_matches_cholesky_oracle(ctx, dA, dG):
    """Sec. II-C, Eq. (kfac-damped): (G + gamma I)^-1 grad (A + gamma I)^-1.  The library forms it in the eigenbasis
    of its own eigendecompositions (factored denominator); the oracle by two Cholesky solves with no
    eigendecomposition at all, so this checks factors -> eig -> precondition against an independent route."""
    rng = np.random.default_rng(dA)
    # zero-mean unit-variance samples on both sides: spectra within [0.1, 3], so that one damping value means the same
    # for both factors and the damped inverses are well conditioned (the sensitivity to the eigensolver's 1e-6 ||F||
    # stays below the 1e-4 bar; ill-conditioned cases are exercised in test_gpu_configs.py)
    X = rng.standard_normal((3 * dA, dA - 1)).astype(np.float32)
    Gr = rng.standard_normal((4 * dG, dG)).astype(np.float32)
    Ad = torch.zeros((dA, dA), dtype=torch.float32, device=ctx.dev)
    Gd = torch.zeros((dG, dG), dtype=torch.float32, device=ctx.dev)
    ctx.update_factors(ctx.to_dev(X), K.KFAC_LAYOUT_RD, X.shape[0], dA - 1, 1, 1, 1.0 / X.shape[0], 0.0, Ad)
    ctx.update_factors(ctx.to_dev(Gr), K.KFAC_LAYOUT_RD, Gr.shape[0], dG, 1, 0, 1.0 / Gr.shape[0], 0.0, Gd)
    Ld, Qd, info = ctx.eig([Ad, Gd])
    assert all(c for (_, _, c) in info)
    A = oracle.gram(X, 1, 1.0 / X.shape[0])
    G = oracle.gram(Gr, 0, 1.0 / Gr.shape[0])
    grad = (rng.standard_normal((dG, dA)) * 1e-2).astype(np.float32)
    for gamma in (0.3, 1.0):
        ref = oracle.precondition_inverse(G, A, gamma, grad)
        gd = ctx.to_dev(grad)
        K.kfac_precondition_batched(ctx.h, [Qd[0]], [Ld[0]], [Qd[1]], [Ld[1]], gamma, [gd], factored_damping=True)
        torch.cuda.synchronize()
        got = gd.cpu().numpy()
        assert relfro(got, ref) <= TOL_F32, (gamma, relfro(got, ref))
        # and it is not the hot path's damping
        g2 = ctx.to_dev(grad)
        K.kfac_precondition_batched(ctx.h, [Qd[0]], [Ld[0]], [Qd[1]], [Ld[1]], gamma, [g2])
        torch.cuda.synchronize()
        assert relfro(g2.cpu().numpy(), ref) > 1e-3


def _spd_factor(rng, n, rows, relu=True):
    X = rng.standard_normal((rows, n - 1))
    if relu:
        X = np.maximum(X, 0)
    X = X.astype(np.float32)
    return oracle.gram(X, 1, 1.0 / rows)


@pytest.mark.parametrize("n,rows", [(1, 8), (5, 40), (64, 256), (128, 300), (129, 300), (300, 200), (577, 1200), (1153, 1500)])
def test_invert_factors_matches_cholesky_oracle(ctx, n, rows):
    """Sec. II-C, Eq. (kfac-damped): (F + gamma I)^-1 by the library's blocked Cholesky inverse against the oracle's
    Cholesky solve of (F + gamma I) X = I in fp64.  Sizes straddle the 128-wide blocks; (300, 200) is rank deficient
    (only the damping makes it definite).  An fp32 inverse carries a relative error of the order of
    cond(F + gamma I) * 6e-8, so the bound is max(2e-6, 2e-7 * cond) with cond from the fp64 spectrum (measured:
    0.02 .. 0.1 of it)."""
    rng = np.random.default_rng(31 * n + rows)
    F = _spd_factor(rng, n, rows)
    lam = np.linalg.eigvalsh(F)
    Fd = ctx.to_dev(F.astype(np.float32))
    F32 = Fd.cpu().numpy().astype(np.float64)
    for gamma in (1e-1, 1e-3):
        ref = oracle.spd_solve(F32 + gamma * np.eye(n), np.eye(n))
        out = torch.full((n, n), float("nan"), dtype=torch.float32, device=ctx.dev)
        K.kfac_invert_factors(ctx.h, [Fd], gamma, [out])
        torch.cuda.synchronize()
        got = out.cpu().numpy().astype(np.float64)
        cond = (max(lam[-1], 0) + gamma) / (max(lam[0], 0) + gamma)
        err = relfro(got, ref)
        assert err <= max(2e-6, 2e-7 * cond), (n, gamma, err, cond)
        # the defining property, in fp64 on the fp32 result
        res = np.linalg.norm(got @ (F32 + gamma * np.eye(n)) - np.eye(n)) / np.sqrt(n)
        assert res <= max(2e-6, 2e-7 * cond), (n, gamma, res, cond)


@pytest.mark.parametrize("n", [129, 257, 385, 513, 641, 897, 1100])
def test_invert_factors_every_shape_of_the_doubling(ctx, n):
    """2 to 9 blocks of 128: whole pairs, a short second half, none.  Well conditioned, so the bound is fp32's."""
    gen = torch.Generator(device="cuda").manual_seed(n)
    X = torch.randn((4 * n, n), generator=gen, device="cuda", dtype=torch.float64)
    F = (X.T.contiguous() @ X / (4 * n)).float()
    F = ((F + F.T) * 0.5).contiguous()
    out = torch.full_like(F, float("nan"))
    K.kfac_invert_factors(ctx.h, [F], 0.1, [out])
    torch.cuda.synchronize()
    A = F.cpu().double() + 0.1 * torch.eye(n, dtype=torch.float64)
    ref = torch.linalg.inv(A)
    cond = float(torch.linalg.matrix_norm(A, 2) * torch.linalg.matrix_norm(ref, 2))
    assert float((out.cpu().double() - ref).norm() / ref.norm()) <= max(2e-6, 2e-7 * cond)


def test_invert_factors_batch_of_mixed_sizes(ctx):
    """Several factors in one call share the workspace one after another; every inverse is checked."""
    rng = np.random.default_rng(77)
    dims = [257, 16, 130, 257, 400]
    Fs = [_spd_factor(rng, n, 3 * n, relu=False) for n in dims]
    Fd = [ctx.to_dev(F.astype(np.float32)) for F in Fs]
    outs = [torch.zeros((n, n), dtype=torch.float32, device=ctx.dev) for n in dims]
    assert 0 < K.kfac_invert_workspace_bytes(dims) <= K.kfac_workspace_bytes(max(dims), 1, 1)
    K.kfac_invert_factors(ctx.h, Fd, 0.05, outs)
    torch.cuda.synchronize()
    for F, o, n in zip(Fd, outs, dims):
        ref = oracle.spd_solve(F.cpu().numpy().astype(np.float64) + 0.05 * np.eye(n), np.eye(n))
        assert relfro(o.cpu().numpy(), ref) <= 1e-5, n
    with pytest.raises(K.KfacError):
        K.kfac_invert_factors(ctx.h, Fd, 0.0, outs)
    with pytest.raises(K.KfacError):
        K.kfac_invert_factors(ctx.h, Fd, 0.05, Fd)


@pytest.mark.parametrize("dA,dG", [(145, 16), (300, 130), (577, 64), (230, 100)])
@pytest.mark.parametrize("bf16", [False, True])
def test_precondition_inverse_matches_oracle(ctx, dA, dG, bf16):
    """The whole inverse method, factors -> Cholesky inverses -> Ginv grad Ainv, against the oracle's two Cholesky
    solves (Sec. II-C, Eq. (kfac-damped)); well-conditioned factors as in
    test_explicit_inverse_method_matches_cholesky_oracle, fp32 and bf16 gradients."""
    rng = np.random.default_rng(dA + 5)
    X = rng.standard_normal((3 * dA, dA - 1)).astype(np.float32)
    Gr = rng.standard_normal((4 * dG, dG)).astype(np.float32)
    Ad = torch.zeros((dA, dA), dtype=torch.float32, device=ctx.dev)
    Gd = torch.zeros((dG, dG), dtype=torch.float32, device=ctx.dev)
    ctx.update_factors(ctx.to_dev(X), K.KFAC_LAYOUT_RD, X.shape[0], dA - 1, 1, 1, 1.0 / X.shape[0], 0.0, Ad)
    ctx.update_factors(ctx.to_dev(Gr), K.KFAC_LAYOUT_RD, Gr.shape[0], dG, 1, 0, 1.0 / Gr.shape[0], 0.0, Gd)
    A = oracle.gram(X, 1, 1.0 / X.shape[0])
    G = oracle.gram(Gr, 0, 1.0 / Gr.shape[0])
    grad = (rng.standard_normal((dG, dA)) * 1e-2).astype(np.float32)
    if bf16:
        grad = S.bf16_bits_to_f32(S.to_bf16_bits(grad)).reshape(grad.shape)
    Ai, Gi = torch.empty_like(Ad), torch.empty_like(Gd)
    for gamma in (0.3, 1.0):
        ref = oracle.precondition_inverse(G, A, gamma, grad)
        K.kfac_invert_factors(ctx.h, [Ad, Gd], gamma, [Ai, Gi])
        gd = ctx.to_dev(grad, bf16)
        K.kfac_precondition_inverse(ctx.h, Ai, Gi, gd)
        torch.cuda.synchronize()
        got = gd.float().cpu().numpy()
        assert relfro(got, ref) <= (TOL_BF16 if bf16 else TOL_F32), (gamma, relfro(got, ref))


def test_precondition_inverse_batched_equals_per_layer(ctx):
    """One batched call over layers of different shapes and gradient types gives, bit for bit, what the per-layer call
    gives (same tiles, same order of operations)."""
    rng = np.random.default_rng(9)
    shapes = [(145, 16, False), (300, 130, True), (64, 257, False), (129, 128, True)]
    Ai, Gi, g1, g2 = [], [], [], []
    for dA, dG, bf16 in shapes:
        A = _spd_factor(rng, dA, 2 * dA, relu=False)
        G = _spd_factor(rng, dG, 2 * dG, relu=False)
        Ai.append(ctx.to_dev(np.linalg.inv(A + 0.5 * np.eye(dA)).astype(np.float32)))
        Gi.append(ctx.to_dev(np.linalg.inv(G + 0.5 * np.eye(dG)).astype(np.float32)))
        g = rng.standard_normal((dG, dA)).astype(np.float32)
        g1.append(ctx.to_dev(g, bf16))
        g2.append(ctx.to_dev(g, bf16))
    K.kfac_precondition_inverse_batched(ctx.h, Ai, Gi, g1)
    for a, g, x in zip(Ai, Gi, g2):
        K.kfac_precondition_inverse(ctx.h, a, g, x)
    torch.cuda.synchronize()
    for x, y in zip(g1, g2):
        assert torch.equal(x, y)


@pytest.mark.parametrize("dA,dG,rows", [(145, 16, 2048), (577, 64, 1500), (289, 32, 200)])
def test_explicit_inverse_method_at_the_papers_damping(ctx, dA, dG, rows):
    """The explicit-inverse method where it is hard: ReLU-activation A factors (one eigenvalue ~ 0.16 d_A over a bulk
    of ~0.3; rank deficient in the last case), gradient factors of size 1e-6, damping 1e-3 (the paper's ImageNet
    value, Sec. VI) -- against the oracle's two Cholesky solves.  The inverse of F + gamma I amplifies a perturbation
    of F by cond(F + gamma I) = (lam_max + gamma) / (lam_min + gamma), and an fp32 eigendecomposition is a
    perturbation of F of the order of fp32's unit roundoff, so the bound is
    max(1e-4, 6e-8 * (cond_A + cond_G)), from the oracle's spectra (measured: 2e-9 .. 5e-9 times that sum)."""
    rng = np.random.default_rng(1000 + dA)
    X = np.maximum(rng.standard_normal((rows, dA - 1)), 0).astype(np.float32)
    Gr = (rng.standard_normal((rows, dG)) * 1e-3).astype(np.float32)
    Ad = torch.zeros((dA, dA), dtype=torch.float32, device=ctx.dev)
    Gd = torch.zeros((dG, dG), dtype=torch.float32, device=ctx.dev)
    ctx.update_factors(ctx.to_dev(X), K.KFAC_LAYOUT_RD, rows, dA - 1, 1, 1, 1.0 / rows, 0.0, Ad)
    ctx.update_factors(ctx.to_dev(Gr), K.KFAC_LAYOUT_RD, rows, dG, 1, 0, 1.0 / rows, 0.0, Gd)
    Ld, Qd, info = ctx.eig([Ad, Gd])
    assert all(c for (_, _, c) in info)
    A = oracle.gram(X, 1, 1.0 / rows)
    G = oracle.gram(Gr, 0, 1.0 / rows)
    gamma = 1e-3
    la, lg = np.linalg.eigvalsh(A), np.linalg.eigvalsh(G)
    cond = (la.max() + gamma) / (max(la.min(), 0.0) + gamma) + (lg.max() + gamma) / (max(lg.min(), 0.0) + gamma)
    bound = max(TOL_F32, 6e-8 * cond)
    grad = (rng.standard_normal((dG, dA)) * 1e-2).astype(np.float32)
    ref = oracle.precondition_inverse(G, A, gamma, grad)
    gd = ctx.to_dev(grad)
    K.kfac_precondition_batched(ctx.h, [Qd[0]], [Ld[0]], [Qd[1]], [Ld[1]], gamma, [gd], factored_damping=True)
    torch.cuda.synchronize()
    err = relfro(gd.cpu().numpy(), ref)
    print("explicit inverse dA=%d dG=%d rows=%d: cond %.1e, error %.2e (bound %.1e)" % (dA, dG, rows, cond, err, bound))
    assert err <= bound


# ------------------------------------------------------------------ whole path, config 1
def test_single_conv_layer_end_to_end(ctx):
    """3x3 conv 16->16 on 8x8, batch 32: three factor updates, eig, precondition, against the oracle and
    against brute-force inversion of the damped Kronecker product."""
    wl = S.workload("single_conv")
    lay = wl.layers[0]
    A = G = None
    Ad = torch.full((145, 145), float("nan"), dtype=torch.float32, device=ctx.dev)
    Gd = torch.full((16, 16), float("nan"), dtype=torch.float32, device=ctx.dev)
    for upd in range(3):
        t = S.layer_inputs(wl, 0, update=upd)
        P = oracle.unfold(t["x"], 3, 3, 1, 1, 1, 1)
        gr = t["g"].transpose(0, 2, 3, 1).reshape(-1, lay.c_out)
        R = P.shape[0]
        Ab, Gb = oracle.gram(P, 1, 1.0 / R), oracle.gram(gr, 0, 1.0 / R)
        A = Ab if A is None else oracle.ema(A, Ab, wl.decay)
        G = Gb if G is None else oracle.ema(G, Gb, wl.decay)
        decay = 0.0 if upd == 0 else wl.decay
        Pd = ctx.unfold(t["x"], 3, 3, 1, 1)
        ctx.update_factors(Pd, K.KFAC_LAYOUT_NDT, wl.batch, 144, lay.T, 1, 1.0 / R, decay, Ad)
        gd = ctx.to_dev(t["g"].reshape(wl.batch, lay.c_out, lay.T))
        ctx.update_factors(gd, K.KFAC_LAYOUT_NDT, wl.batch, 16, lay.T, 0, 1.0 / R, decay, Gd)
    torch.cuda.synchronize()
    assert relfro(Ad.cpu().numpy(), A) <= TOL_F32
    assert relfro(Gd.cpu().numpy(), G) <= TOL_F32
    Ld, Qd, info = ctx.eig([Ad, Gd])
    check_eigpairs(Ad.cpu().numpy(), Ld[0].cpu().numpy(), Qd[0].cpu().numpy(), "A")
    check_eigpairs(Gd.cpu().numpy(), Ld[1].cpu().numpy(), Qd[1].cpu().numpy(), "G")
    lamA, QA = oracle.eigh(A)
    lamG, QG = oracle.eigh(G)
    for gamma in (wl.damping, 1e-3 * lamA.mean() * lamG.mean()):
        ref = oracle.precondition(QA, lamA, QG, lamG, gamma, t["gradw"])
        gd = ctx.to_dev(t["gradw"])
        K.kfac_precondition(ctx.h, Qd[0], Ld[0], Qd[1], Ld[1], gamma, gd)
        torch.cuda.synchronize()
        got = gd.cpu().numpy()
        assert relfro(got, ref) <= TOL_F32
        assert relfro(got, oracle.bruteforce(G, A, gamma, t["gradw"])) <= TOL_F32


# ------------------------------------------------------------------ error paths (host-side validation)
def test_invalid_arguments_are_rejected(ctx):
    F = torch.zeros((4, 4), device=ctx.dev)
    X = torch.zeros((8, 4), device=ctx.dev)
    L = K.lib()
    assert L.kfac_update_factors(ctx.h, None, 0, 0, 8, 4, 1, 0, 1.0, 0.0, F.data_ptr()) == K.KFAC_EINVAL
    assert L.kfac_update_factors(ctx.h, X.data_ptr(), 7, 0, 8, 4, 1, 0, 1.0, 0.0, F.data_ptr()) == K.KFAC_EINVAL
    assert L.kfac_update_factors(ctx.h, X.data_ptr(), 0, 0, 8, 4, 1, 0, 1.0, 1.5, F.data_ptr()) == K.KFAC_EINVAL
    assert L.kfac_update_factors(ctx.h, X.data_ptr(), 0, 0, 0, 4, 1, 0, 1.0, 0.5, F.data_ptr()) == K.KFAC_EINVAL
    assert L.kfac_precondition(ctx.h, F.data_ptr(), F.data_ptr(), 4, F.data_ptr(), F.data_ptr(), 4, 0.0,
                               F.data_ptr(), 0) == K.KFAC_EINVAL
    d = K.kfac_conv_desc(1, 1, 4, 4, 3, 3, 0, 1, 1, 1, 0)
    import ctypes
    assert L.kfac_unfold(ctx.h, ctypes.byref(d), X.data_ptr(), F.data_ptr()) == K.KFAC_EINVAL
    small = Ctx(1 << 16)
    big = torch.zeros((300, 300), device=ctx.dev)
    with pytest.raises(K.KfacError) as e:
        K.kfac_eig(small.h, [big], [torch.empty_like(big)], [torch.empty(300, device=ctx.dev)])
    assert e.value.code == K.KFAC_EWORKSPACE
    small.close()


# ------------------------------------------------------------------ per-kernel timing
def test_profile_reports_every_kernel_class(ctx):
    """One stretch of calls that launches more kernel classes than sixteen: all of them come back."""
    F = [ctx.to_dev(gram_factor(n, 2 * n, seed=n)) for n in (2100, 577, 100)]
    Q, lam = [torch.empty_like(f) for f in F], [torch.empty(f.shape[0], device=ctx.dev) for f in F]
    X = torch.randn((8, 20, 6, 6), device=ctx.dev)
    P = torch.empty((8, 180, 36), device=ctx.dev)
    grads = [torch.randn((100, 577), device=ctx.dev) for _ in range(2)]
    inv = torch.empty_like(F[2])
    K.kfac_profile_begin(ctx.h)
    K.kfac_unfold(ctx.h, X, 3, 3, 1, 1, P)
    for dt in (torch.float32, torch.bfloat16):
        A = torch.empty((180, 180), device=ctx.dev)
        K.kfac_update_factors(ctx.h, P.to(dt), K.KFAC_LAYOUT_NDT, 8, 180, 36, 0, 1.0 / 288, 0.0, A)
    K.kfac_eig(ctx.h, F, Q, lam)
    K.kfac_eig(ctx.h, F, Q, lam, tol=5e-7)
    args = ([Q[1]] * 2, [lam[1]] * 2, [Q[2]] * 2, [lam[2]] * 2, 1e-2, grads)
    K.kfac_precondition_batched_scaled(ctx.h, *args, kappa=1e-3, lr=0.1, nu=torch.empty(1, device=ctx.dev))
    K.kfac_precondition_batched(ctx.h, *args, split_f16=True)
    K.kfac_invert_factors(ctx.h, [F[2]], 0.1, [inv])
    stats = K.kfac_profile_end(ctx.h)
    want = {"unfold", "syrk", "syrk_bf16", "precond_gemm", "precond_gemm_split", "precond_scale", "factor_inverse", "eig_small", "eig_pivot_solve",
            "eig_apply", "eig_outer_cols", "eig_outer_rows", "eig_post_gemm", "eig_misc", "eig_reduce_mv", "eig_reduce_vec", "eig_reduce_update",
            "eig_tridiag_solve", "eig_back"}
    assert want <= set(stats), want - set(stats)
    for name, st in stats.items():
        assert st["launches"] > 0 and st["ms"] > 0.0, (name, st)
    assert stats["eig_reduce_vec"]["bytes"] > 0.0 and stats["eig_reduce_mv"]["bytes"] > 0.0
    assert all(stats[k]["flops"] > 0.0 for k in ("eig_tridiag_solve", "eig_reduce_update", "eig_back"))
