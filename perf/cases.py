"""Performance cases of the K-FAC preconditioner library: what they are, how their inputs are made, one pass of each.

A case is a layer set (the shapes of a network's layers at a batch size) and the calls a training program makes on it:

  step          one whole K-FAC step: unfold, both factors of every layer folded into their running averages,
                eigendecomposition of every factor, every gradient preconditioned
  factors       only the factor update (what runs every f_fac iterations)
  eig           only the decomposition and the preconditioning with its result, from the identity or (warm) from the
                eigenvectors of the factors before they moved
  precondition  only the preconditioning (what runs every iteration), plain or with the gradient scaling nu
  inverse       the explicit-inverse method: damped factors inverted, gradients preconditioned by two products
  layer         one layer through the single-layer calls: unfold, two factor updates, preconditioning

Eigenvectors are defined up to sign, and up to a rotation inside a cluster of eigenvalues (thousands of equal ones in a
rank-deficient factor), so they cannot be compared element by element: a pass that decomposes returns the eigenvalues
and the preconditioned gradients, which every column of every eigenvector matrix enters.  The gradient factors have the
size of per-sample gradients (sigma_g = 0.05), so that the products of eigenvalues lie on both sides of the damping and
the eigenpairs matter to the result.

A step updates its running averages and its gradients in place.  So that a pass can be repeated, it begins with what
a training iteration has by then: the running averages as they were before this batch and fresh gradients, one device
copy each.
"""
import math

import torch

from paper_2007_00784_amd import kfac as K
from paper_2007_00784_amd.synthetic import Layer

DECAY = 0.95
SIGMA_G = 0.05
SIGMA_W = 1e-2


# ---------------------------------------------------------------- layer sets
def bottleneck_layers(width, blocks, image, classes):
    """Convs + FC of a bottleneck ResNet (width 64, blocks 3,4,6,3, image 224, 1000 classes: ResNet-50)."""
    out = [Layer("stem", 3, width, 7, 2, 3, image)]
    h = ((image + 6 - 7) // 2 + 1 + 1) // 2          # stem, then a 3x3 stride-2 pooling
    c_prev = width
    for si, nb in enumerate(blocks):
        w = width << si
        for b in range(nb):
            s = 2 if (b == 0 and si > 0) else 1
            pre = "s%db%d" % (si + 1, b)
            out.append(Layer(pre + ".reduce", c_prev, w, 1, 1, 0, h))
            out.append(Layer(pre + ".conv3", w, w, 3, s, 1, h))
            ho = out[-1].h_out
            out.append(Layer(pre + ".expand", w, 4 * w, 1, 1, 0, ho))
            if b == 0:
                out.append(Layer(pre + ".proj", c_prev, 4 * w, 1, s, 0, h))
            h, c_prev = ho, 4 * w
    out.append(Layer("fc", c_prev, classes, 1, 1, 0, 1, fc=True))
    return out


def basic_layers(width, nblocks, image, classes):
    """CIFAR-style ResNet: three stages of nblocks blocks of two 3x3 convs (width 16, 5 blocks, image 32: ResNet-32)."""
    out = [Layer("stem", 3, width, 3, 1, 1, image)]
    h, c_prev = image, width
    for si in range(3):
        w = width << si
        for b in range(nblocks):
            s = 2 if (b == 0 and si > 0) else 1
            pre = "s%db%d" % (si + 1, b)
            out.append(Layer(pre + ".conv1", c_prev, w, 3, s, 1, h))
            if s == 2:
                out.append(Layer(pre + ".short", c_prev, w, 1, 2, 0, h))
            h = out[-1].h_out
            out.append(Layer(pre + ".conv2", w, w, 3, 1, 1, h))
            c_prev = w
    out.append(Layer("fc", c_prev, classes, 1, 1, 0, 1, fc=True))
    return out


def linear_layers(widths):
    return [Layer("fc%d" % i, a, b, 1, 1, 0, 1, fc=True) for i, (a, b) in enumerate(zip(widths, widths[1:]))]


def layers_of(case):
    ints = [int(v) for v in case["sizes"].split(",")]
    if case["net"] == "bottleneck":                      # width, four block counts, image, classes
        return bottleneck_layers(ints[0], ints[1:5], ints[5], ints[6])
    if case["net"] == "basic":                           # width, blocks per stage, image, classes
        return basic_layers(*ints)
    if case["net"] == "linear":                          # widths
        return linear_layers(ints)
    return [Layer("conv", *ints)]                        # one conv: c_in, c_out, kernel, stride, pad, image


# ---------------------------------------------------------------- the cases
def case_of(name, kind, net, sizes, batch, damping=1e-3, bf16=False, warm=False, scaled=False, graded=False):
    c = dict(kind=kind, net=net, sizes=sizes, batch=batch, damping=damping, bf16=bf16, warm=warm, scaled=scaled, graded=graded)
    if name:
        c["name"] = name
    return c


RESNET50 = "64,3,4,6,3,224,1000"


def listed():
    return [
        # the smallest whole step: one 3x3 conv, factors 145 and 16 wide; launches and latency are all there is
        case_of("step_single_conv", "step", "conv", "16,16,3,1,1,8", 32),
        # one mid-size layer through the single-layer calls, as a per-layer hook of a training program makes them
        case_of("layer_conv_128", "layer", "conv", "128,128,3,1,1,28", 32),
        # a small network: 68 factors 10 to 577 wide, all of them too small to fill the machine alone
        case_of("step_resnet32_cifar", "step", "basic", "16,5,32,10", 128, damping=3e-3),
        # Linear layers only: [R][d] operands, no unfold, factors of rank far below their width
        case_of("step_linear", "step", "linear", "2048,2048,2048,1000", 256),
        # the largest single factor (4609 wide, rank deficient, spectrum graded over eight decades) and its 512-wide partner
        case_of("eig_largest_factor", "eig", "conv", "512,512,3,1,1,7", 64, graded=True),
        # what a training loop does from its second decomposition on: factors moved by one running-average update,
        # started from their previous eigenvectors (one block per stage of ResNet-50, factors 64 to 4609)
        case_of("eig_warm_start", "eig", "bottleneck", "64,1,1,1,1,224,1000", 32, warm=True),
        # the factor update of ResNet-50, fp32 at batch 32 and bf16 at batch 64 (every 10th iteration in training)
        case_of("factors_resnet50", "factors", "bottleneck", RESNET50, 32),
        case_of("factors_resnet50_bf16", "factors", "bottleneck", RESNET50, 64, bf16=True),
        # the preconditioning of ResNet-50 (every iteration): fp32 with the gradient scaling nu, bf16 gradients on the
        # split-fp16 products
        case_of("precondition_resnet50", "precondition", "bottleneck", RESNET50, 32, scaled=True),
        case_of("precondition_resnet50_bf16", "precondition", "bottleneck", RESNET50, 64, bf16=True),
        # the explicit-inverse method on the same set
        case_of("inverse_resnet50", "inverse", "bottleneck", RESNET50, 32, damping=1e-2),
        # the benchmark's step: all 54 layers, 108 factors 64 to 4609 wide
        case_of("step_resnet50", "step", "bottleneck", RESNET50, 32),
    ]


def log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same kinds: layer counts, widths, image sizes and batches drawn over the whole range, odd ones
    among them (never more than the full ResNet-50 set)."""
    kind = rng.choice(["step", "step", "factors", "eig", "eig", "precondition", "inverse", "layer"])
    damping = rng.choice([1e-3, 3e-3, 1e-2])
    if kind == "inverse":
        damping = rng.choice([1e-2, 3e-2])
    if kind == "layer":
        k = rng.choice([1, 3, 3, 5])
        image = log_int(rng, 7, 56)
        c = case_of(None, kind, "conv", "%d,%d,%d,%d,%d,%d" % (log_int(rng, 3, 300), log_int(rng, 8, 512), k, rng.choice([1, 1, 2]), k // 2, image),
                    log_int(rng, 8, 64), damping, bf16=rng.random() < 0.3)
        return c
    net = rng.choice(["conv", "basic", "linear", "bottleneck", "bottleneck"])
    bf16 = kind in ("factors", "precondition") and rng.random() < 0.5
    if net == "conv":
        sizes = "%d,%d,3,%d,1,%d" % (log_int(rng, 8, 512), log_int(rng, 8, 512), rng.choice([1, 2]), log_int(rng, 7, 28))
        batch = log_int(rng, 16, 64)
    elif net == "basic":
        sizes = "%d,%d,%d,%d" % (log_int(rng, 8, 64), rng.randint(1, 5), rng.randint(16, 40), rng.choice([10, 100]))
        batch = log_int(rng, 16, 128)
    elif net == "linear":
        sizes = ",".join(str(log_int(rng, 64, 3000)) for _ in range(rng.randint(2, 5)))
        batch = log_int(rng, 32, 512)
    else:
        sizes = "%d,%d,%d,%d,%d,%d,%d" % (log_int(rng, 12, 64), rng.randint(1, 3), rng.randint(1, 3), rng.randint(1, 3), rng.randint(1, 2),
                                          rng.randint(64, 224), rng.choice([10, 100, 1000]))
        batch = log_int(rng, 8, 48)
    return case_of(None, kind, net, sizes, batch, damping, bf16=bf16, warm=kind == "eig" and rng.random() < 0.4,
                   scaled=kind == "precondition" and rng.random() < 0.5, graded=kind == "eig" and net == "conv" and rng.random() < 0.5)


# ---------------------------------------------------------------- inputs
class State:
    """Buffers of one case, and the library context a training program keeps beside them."""

    def __init__(self, case, seed):
        self.case = case
        self.dev = torch.device("cuda:0")
        self.gen = torch.Generator(device=self.dev).manual_seed(seed)
        self.layers = layers_of(case)
        self.N = case["batch"]
        self.dt = torch.bfloat16 if case["bf16"] else torch.float32
        self.ctx = None
        dims = [l.d_a for l in self.layers] + [l.d_g for l in self.layers]
        self.dims = dims
        need = max(K.kfac_eig_workspace_bytes(dims), K.kfac_update_factors_workspace_bytes(self.factor_items(None)),
                   K.kfac_precondition_workspace_bytes([(l.d_a, l.d_g) for l in self.layers]),
                   K.kfac_invert_workspace_bytes(dims), K.kfac_workspace_bytes(max(dims), 1, max(l.rows(self.N) for l in self.layers)))
        self.ws = torch.empty(need + 4096, dtype=torch.uint8, device=self.dev)
        self.ctx = K.kfac_create(0, torch.cuda.current_stream(self.dev).cuda_stream, self.ws)

    def __del__(self):
        if self.ctx is not None and torch is not None:      # (None: the interpreter is going down)
            torch.cuda.synchronize()
            K.kfac_destroy(self.ctx)
            self.ctx = None

    def normal(self, shape, sigma=1.0):
        return torch.randn(shape, generator=self.gen, device=self.dev).mul_(sigma)

    def flat(self, shapes, dtype=torch.float32):
        """One buffer for a list of tensors (each starts on a 256-byte boundary), and the views of it."""
        sizes = [(math.prod(s) + 127) // 128 * 128 for s in shapes]
        buf = torch.zeros(sum(sizes), dtype=dtype, device=self.dev)
        views, at = [], 0
        for s, z in zip(shapes, sizes):
            views.append(buf[at:at + math.prod(s)].view(s))
            at += z
        return buf, views

    def draw_batch(self):
        """Activations ReLU(N(0,1)) (graded: channels scaled over 1e-3..1e1) and output gradients of one batch."""
        self.x, self.g = [], []
        for l in self.layers:
            x = self.normal((self.N, l.c_in) if l.fc else (self.N, l.c_in, l.h_in, l.h_in)).relu_()
            if self.case["graded"]:
                s = 10.0 ** (torch.rand(l.c_in, generator=self.gen, device=self.dev) * 4.0 - 3.0)
                x *= s.view((1, -1) if l.fc else (1, -1, 1, 1))
            self.x.append(x.to(self.dt))
            self.g.append(self.normal((self.N, l.c_out) if l.fc else (self.N, l.c_out, l.T), SIGMA_G).to(self.dt))

    def factor_items(self, decay):
        """Arguments of the batched factor update (decay None: sizes only)."""
        items = []
        code = K.KFAC_BF16 if self.dt is torch.bfloat16 else K.KFAC_F32
        for i, l in enumerate(self.layers):
            lay, T = (K.KFAC_LAYOUT_RD, 1) if l.fc else (K.KFAC_LAYOUT_NDT, l.T)
            for d, ones in ((l.d_a - 1, 1), (l.d_g, 0)):
                it = dict(X=None, dtype=code, layout=lay, N=self.N, d=d, T=T, append_ones=ones, F=None)
                if decay is not None:
                    X = self.g[i] if not ones else (self.patches[i] if l.needs_unfold else self.x[i])
                    it.update(X=X, scale=1.0 / (self.N * T), decay=decay, F=self.F[2 * i + (0 if ones else 1)])
                items.append(it)
        return items

    def alloc_factors(self):
        self.patches = [torch.empty(self.N * (l.d_a - 1) * l.T, dtype=self.dt, device=self.dev) if l.needs_unfold else None for l in self.layers]
        self.F_flat, self.F = self.flat([(d, d) for l in self.layers for d in (l.d_a, l.d_g)])

    def alloc_eig(self):
        self.lam_flat, self.lam = self.flat([(d,) for l in self.layers for d in (l.d_a, l.d_g)])
        self.Q_flat, self.Q = self.flat([(d, d) for l in self.layers for d in (l.d_a, l.d_g)])

    def alloc_grads(self):
        self.grad_flat, self.grad = self.flat([(l.d_g, l.d_a) for l in self.layers], self.dt)
        self.grad0 = torch.zeros_like(self.grad_flat)
        self.grad0.copy_(self.normal(self.grad_flat.shape, SIGMA_W))

    # ---- the calls of a pass ----
    def update_factors(self, decay):
        idx = [i for i, l in enumerate(self.layers) if l.needs_unfold]
        if idx:
            K.kfac_unfold_batched(self.ctx, [self.x[i] for i in idx],
                                  [(self.layers[i].k, self.layers[i].k, self.layers[i].stride, self.layers[i].pad) for i in idx],
                                  [self.patches[i] for i in idx])
        K.kfac_update_factors_batched(self.ctx, self.items if decay == DECAY else self.factor_items(decay))

    def eig(self, warm=False):
        K.kfac_eig(self.ctx, self.F, self.Q, self.lam, warm_start=warm)

    def precondition(self):
        self.grad_flat.copy_(self.grad0)
        if self.case["scaled"]:
            K.kfac_precondition_batched_scaled(self.ctx, kappa=1e-3, lr=0.1, nu=self.nu, items=self.pitems)
        else:
            K.kfac_precondition_batched(self.ctx, items=self.pitems)

    def marshal_precondition(self):
        self.nu = torch.zeros(1, device=self.dev)
        self.pitems = K.precond_items(self.Q[0::2], self.lam[0::2], self.Q[1::2], self.lam[1::2], self.case["damping"], self.grad,
                                      split_f16=self.case["bf16"])


def orthogonal(n, gen, dev):
    """A dense orthogonal matrix without a factorisation: the cosine basis with its rows and columns in random order and
    of random sign."""
    i = torch.arange(n, device=dev, dtype=torch.float64)
    c = torch.cos(math.pi / n * (i[None, :] + 0.5) * i[:, None]) * math.sqrt(2.0 / n)
    c[0] *= math.sqrt(0.5)
    c = c[torch.randperm(n, generator=gen, device=dev)][:, torch.randperm(n, generator=gen, device=dev)]
    sign = torch.randint(0, 2, (2, n), generator=gen, device=dev).double() * 2 - 1
    return (c * sign[0][:, None] * sign[1][None, :]).float()


def prepare(case, seed):
    s = State(case, seed)
    kind = case["kind"]
    if kind in ("step", "factors", "layer"):
        s.alloc_factors()
        s.draw_batch()
        s.update_factors(0.0)               # the running averages: one earlier batch, then the batch of this pass
        s.F0_flat = s.F_flat.clone()
        s.draw_batch()
        s.items = K.factor_items(s.factor_items(DECAY))
    if kind in ("eig", "inverse"):
        s.alloc_factors()
        s.draw_batch()
        s.update_factors(0.0)
        if case["warm"]:
            s.alloc_eig()
            s.eig()
            s.Q0_flat = s.Q_flat.clone()
        if not case["graded"]:
            s.draw_batch()
            s.items = K.factor_items(s.factor_items(DECAY))
            s.update_factors(DECAY)
        s.x = s.g = s.patches = None        # a decomposition has the factors only
    if kind != "factors":
        s.alloc_grads()
    if kind in ("step", "layer", "precondition") or (kind == "eig" and not case["warm"]):
        s.alloc_eig()
    if kind in ("layer", "precondition"):   # eigenpairs of the decomposition in force
        for q, lam in zip(s.Q, s.lam):
            q.copy_(orthogonal(q.shape[0], s.gen, s.dev))
            lam.copy_(torch.rand(lam.shape, generator=s.gen, device=s.dev).mul_(0.7))
        for i, l in enumerate(s.layers):
            s.lam[2 * i][-1] = 0.16 * l.d_a
            s.lam[2 * i + 1].mul_(2 * SIGMA_G ** 2)
        for lam in s.lam:
            lam.copy_(lam.sort().values)
    if kind == "inverse":
        s.Finv_flat, s.Finv = s.flat([(d, d) for l in s.layers for d in (l.d_a, l.d_g)])
        s.inv_items = K.precond_inv_items(s.Finv[0::2], s.Finv[1::2], s.grad)
    elif kind != "factors":
        s.marshal_precondition()
    torch.cuda.synchronize()
    return s


# ---------------------------------------------------------------- one pass
def run(s):
    kind = s.case["kind"]
    if kind in ("step", "factors", "layer"):
        s.F_flat.copy_(s.F0_flat)
    if kind == "layer":
        l = s.layers[0]
        X = s.x[0]
        if l.needs_unfold:
            K.kfac_unfold(s.ctx, s.x[0], l.k, l.k, l.stride, l.pad, s.patches[0])
            X = s.patches[0]
        scale = 1.0 / (s.N * l.T)
        K.kfac_update_factors(s.ctx, X, K.KFAC_LAYOUT_NDT, s.N, l.d_a - 1, l.T, 1, scale, DECAY, s.F[0])
        K.kfac_update_factors(s.ctx, s.g[0], K.KFAC_LAYOUT_NDT, s.N, l.d_g, l.T, 0, scale, DECAY, s.F[1])
        s.grad_flat.copy_(s.grad0)
        K.kfac_precondition(s.ctx, s.Q[0], s.lam[0], s.Q[1], s.lam[1], s.case["damping"], s.grad[0])
        return [s.F_flat, s.grad_flat]
    if kind == "factors":
        s.update_factors(DECAY)
        return [s.F_flat]
    if kind == "precondition":
        s.precondition()
        return [s.grad_flat, s.nu] if s.case["scaled"] else [s.grad_flat]
    if kind == "inverse":
        s.grad_flat.copy_(s.grad0)
        K.kfac_invert_factors(s.ctx, s.F, s.case["damping"], s.Finv)
        K.kfac_precondition_inverse_batched(s.ctx, items=s.inv_items)
        return [s.Finv_flat, s.grad_flat]
    if kind == "eig":
        if s.case["warm"]:
            s.Q_flat.copy_(s.Q0_flat)
        s.eig(s.case["warm"])
        s.precondition()
        return [s.lam_flat, s.grad_flat]
    s.update_factors(DECAY)
    s.eig()
    s.precondition()
    return [s.F_flat, s.lam_flat, s.grad_flat]


# ---------------------------------------------------------------- work and tolerance
def work(case):
    """Factors: every sample and gradient read once, every factor read and written, the symmetric half of the products.
    Decomposition: reduction to tridiagonal form (4/3 n^3) and back-transformation of all eigenvectors (2 n^3).
    Inverse: Cholesky inverse (n^3), two products.  Preconditioning: four products."""
    e = 2 if case["bf16"] else 4
    kind = case["kind"]
    b = f = 0.0
    for l in layers_of(case):
        R = case["batch"] * l.T
        x = case["batch"] * l.c_in * (1 if l.fc else l.h_in * l.h_in)
        sq = float(l.d_a) ** 2 + float(l.d_g) ** 2
        cube = float(l.d_a) ** 3 + float(l.d_g) ** 3
        grad = float(l.d_a) * l.d_g
        if kind in ("step", "factors", "layer"):
            b += e * (x + R * l.d_g) + 8.0 * sq
            f += float(R) * (l.d_a * (l.d_a + 1.0) + l.d_g * (l.d_g + 1.0))
        if kind in ("step", "eig"):
            b += 8.0 * sq                    # factor in, eigenvectors out
            f += 10.0 / 3.0 * cube
        if kind == "inverse":
            b += 8.0 * sq + 2.0 * e * grad
            f += cube + 2.0 * grad * (l.d_a + l.d_g)
        if kind in ("step", "eig", "precondition", "layer"):
            b += 4.0 * sq + 2.0 * e * grad
            f += 4.0 * grad * (l.d_a + l.d_g)
    return {"bytes": b, "flops": f}


def tolerance(case):
    """About four times the distance from the same pass in 64 bits, measured on the listed cases: factors 3e-8 (sums of up to
    4e5 fp32 products, each entry within 4e-7), preconditioned fp32 gradients 1.5e-6, bf16 ones 1.7e-3 (one rounding of
    the result), the inverse method 2e-4 (fp32 inverses of matrices of
    condition up to 7e4), gradients through a decomposition
    5e-5 at 4609 (rounding errors of the size of fp32's unit times the norm of a factor, against the damping)."""
    kind = case["kind"]
    if kind == "factors":
        return {"rel": 1e-6}
    if kind in ("precondition", "layer"):
        return {"rel": 7e-3, "max": 0.02} if case["bf16"] else {"rel": 6e-6}
    if kind == "inverse":
        return {"rel": 1e-3}
    return {"rel": 3e-4}
