"""The work that programs have this library do, as measurable cases.

Every case is a call of a public entry point on matrices already in HBM:

* ``sqrtm``     one or a batch of principal square roots (forward only);
* ``grad``      ``sqrtm_autograd`` forward and backward (matrix square root
                layers in training);
* ``refine``    approximate-Newton refinement of a root from a factor kept
                over a sequence of nearby matrices (no factorisation);
* ``rootm``     a principal cube root.

The matrix families are those of ``workloads``: symmetric positive definite
and complex Hermitian positive definite with a prescribed condition number
(Alg. 3), real nonsymmetric A = 2 I + G / sqrt(n) (real Schur route), complex
A = B B (complex Schur route).  They are drawn with torch on the device.
"""

from __future__ import annotations

import math

import torch

import paper_2607_12430_amd as msq

DEV = "cuda"
F64, C128 = torch.float64, torch.complex128

# Sizes per (entry point, family): batch range, order range and precisions.
RANGES = {
    ("sqrtm", "spd"): ((1, 1), (48, 4096), ("fp32", "fp64", "bf16split", "auto")),
    ("sqrtm", "spd_batch"): ((2, 64), (24, 512), ("fp32", "fp64")),
    ("sqrtm", "hpd"): ((1, 1), (32, 1024), ("fp32", "fp64")),
    ("sqrtm", "nonsym"): ((1, 1), (32, 2048), ("fp32", "fp64")),
    ("sqrtm", "square"): ((1, 1), (32, 1024), ("fp32",)),
    ("grad", "spd_batch"): ((2, 64), (24, 512), ("fp32", "fp64")),
    ("grad", "nonsym"): ((1, 1), (32, 768), ("fp32",)),
    ("refine", "spd"): ((1, 1), (64, 2048), ("fp32",)),
    ("rootm", "cube"): ((1, 1), (32, 512), ("fp32",)),
}


def _case(name, call, kind, n, batch=1, prec="fp32", kappa=1e4):
    return {"name": name, "call": call, "kind": kind, "n": n, "batch": batch, "prec": prec,
            "kappa": kappa}


def listed():
    return [
        # a covariance of a few dozen features, root wanted now: launches and
        # host time count
        _case("spd_64", "sqrtm", "spd", 64, kappa=1e2),
        # small FP64 solve, lam in [1e-2, 1e2] (whitening, preconditioning)
        _case("spd_fp64_256", "sqrtm", "spd", 256, prec="fp64"),
        # ragged order, learned choice of the factor's precision
        _case("spd_auto_1531", "sqrtm", "spd", 1531, prec="auto", kappa=1e3),
        # the benchmark's solve: dense SPD, kappa 1e4
        _case("spd_4096", "sqrtm", "spd", 4096),
        # covariance pooling layer of a training step: 64 roots of order 512
        # and their gradients
        _case("spd_batch_64x512_grad", "grad", "spd_batch", 512, batch=64),
        # complex Hermitian (density matrix, array covariance), ragged order
        _case("hpd_500", "sqrtm", "hpd", 500),
        # tracking a slowly changing matrix with the factor kept
        _case("refine_1000", "refine", "spd", 1000),
        # small nonsymmetric root (matrix function of a transition matrix)
        _case("nonsym_100", "sqrtm", "nonsym", 100),
        # nonsymmetric root as a differentiable operation
        _case("nonsym_333_grad", "grad", "nonsym", 333),
        # real nonsymmetric solve of order 2048, real Schur route
        _case("nonsym_2048", "sqrtm", "nonsym", 2048),
        # complex non-Hermitian A = B^2, complex Schur route
        _case("square_1024", "sqrtm", "square", 1024),
        # principal cube root of a real matrix
        _case("cube_256", "rootm", "cube", 256),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call, kind = rng.choice(sorted(RANGES))
    (b0, b1), (n0, n1), precs = RANGES[call, kind]
    n = _log_int(rng, n0, n1)
    batch = _log_int(rng, b0, b1)
    kappa = float("%.3g" % 10.0 ** rng.uniform(1.0, 5.0))
    prec = rng.choice(precs)
    if kind == "nonsym" and prec == "fp64":
        n = min(n, 1280)  # a float64 real Schur form costs twice the float one
    return {"call": call, "kind": kind, "n": n, "batch": batch, "prec": prec, "kappa": kappa}


# ------------------------------------------------------------------ inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _randn(shape, g, dtype=F64):
    return torch.randn(*shape, generator=g, device=DEV, dtype=dtype)


def _haar(n, g, dtype=F64):
    """Haar-distributed orthogonal (unitary) matrix: QR of a Gaussian matrix
    with the phases of diag(R) folded in."""
    q, r = torch.linalg.qr(_randn((n, n), g, dtype))
    d = torch.diagonal(r)
    return q * torch.where(d == 0, torch.ones_like(d), d / d.abs())[None, :]


def _eigs(n, kappa, g):
    s = math.sqrt(kappa)
    u = torch.rand(n, generator=g, device=DEV, dtype=F64)
    lam = torch.exp((2.0 * u - 1.0) * math.log(s))
    lam[0], lam[-1] = 1.0 / s, s
    return lam


def _spd(n, kappa, g, dtype=F64):
    """(A, Q, lam): A = Q diag(lam) Q^H, exactly symmetric (Hermitian)."""
    q, lam = _haar(n, g, dtype), _eigs(n, kappa, g)
    a = (q * lam.to(dtype)[None, :]) @ q.mH.contiguous()
    return (0.5 * (a + a.mH)).contiguous(), q, lam


def _nonsym(n, g):
    return 2.0 * torch.eye(n, device=DEV, dtype=F64) + _randn((n, n), g) / math.sqrt(n)


def _square_root_matrix(n, g):
    """B = Q (D + N) Q^H, D uniform in |z - 2| < 1.5, N strictly upper with
    standard deviation 0.1 / sqrt(n): the principal root of B B."""
    q = _haar(n, g, C128)
    rad = 1.5 * torch.sqrt(torch.rand(n, generator=g, device=DEV, dtype=F64))
    ang = 2.0 * math.pi * torch.rand(n, generator=g, device=DEV, dtype=F64)
    t = torch.diag(2.0 + torch.polar(rad, ang))
    t = t + torch.triu(_randn((n, n), g, C128), 1) * (0.1 / math.sqrt(n))
    return q @ t @ q.mH.contiguous()


def _cube_root_matrix(n, g):
    """B = 2 I + G / sqrt(n): its spectrum lies in |z - 2| <= 1, inside
    |arg z| < pi / 3, so B is the principal cube root of B B B."""
    return _nonsym(n, g)


def _inputs(case, seed):
    """The call's input tensors and, per matrix, what its construction knows
    about the answer."""
    g, n = _gen(seed), case["n"]
    kind, kappa = case["kind"], case["kappa"]
    known = None
    if kind == "spd":
        a, q, lam = _spd(n, kappa, g)
        known = [(q, lam)]
    elif kind == "spd_batch":
        parts = [_spd(n, kappa, g) for _ in range(case["batch"])]
        a = torch.stack([p[0] for p in parts])
        known = [(p[1], p[2]) for p in parts]
    elif kind == "hpd":
        a, q, lam = _spd(n, kappa, g, C128)
        known = [(q, lam)]
    elif kind == "nonsym":
        a = _nonsym(n, g)
    elif kind == "square":
        b = _square_root_matrix(n, g)
        a, known = b @ b, b
    else:
        b = _cube_root_matrix(n, g)
        a, known = b @ b @ b, b
    extra = {}
    if case["call"] == "grad":
        extra["gbar"] = torch.randn(a.shape, generator=g, device=DEV, dtype=a.dtype)
        if kind == "spd_batch":  # a loss of a symmetric root has a symmetric gradient
            extra["gbar"] = 0.5 * (extra["gbar"] + extra["gbar"].mT)
    elif case["call"] == "refine":
        # the next matrix of the sequence: the same eigenvectors turned a
        # little, eigenvalues moved by up to 0.1 %
        q, lam = known[0]
        lam1 = lam * (1.0 + 1e-3 * (2.0 * torch.rand(n, generator=g, device=DEV, dtype=F64) - 1.0))
        k = _randn((n, n), g) * (1e-5 / math.sqrt(n))
        k = k - k.mT
        eye = torch.eye(n, device=DEV, dtype=F64)
        q1 = torch.linalg.solve(eye + 0.5 * k, (eye - 0.5 * k) @ q)
        a1 = (q1 * lam1[None, :]) @ q1.mT.contiguous()
        extra["a1"] = (0.5 * (a1 + a1.mT)).contiguous()
        known = [(q1, lam1)]
    return a.contiguous(), known, extra


def prepare(case, seed):
    a, known, extra = _inputs(case, seed)
    state = {"call": case["call"], "prec": case["prec"], "a": a, **extra}
    if case["call"] == "grad":
        state["a"] = a.requires_grad_(True)
    elif case["call"] == "refine":
        state["x0"], _, state["factor"] = msq.sqrtm(a, prec=case["prec"], structure="hpd",
                                                    keep_factor=True)
    return state


# -------------------------------------------------------------------- a pass

def run(state):
    call = state["call"]
    if call == "sqrtm":
        x, _ = msq.sqrtm(state["a"], prec=state["prec"])
        return {"x": x}
    if call == "grad":
        x = msq.sqrtm_autograd(state["a"], prec=state["prec"])
        (g,) = torch.autograd.grad(x, state["a"], state["gbar"])
        return {"x": x, "g": g}
    if call == "refine":
        x = state["x0"].clone()  # the last root is where the next one starts
        msq.refine(state["factor"], state["a1"], x, init_from_factor=False)
        return {"x": x}
    x, _ = msq.rootm(state["a"], p=3, prec=state["prec"])
    return {"x": x}


# ------------------------------------------------------------- required work

def work(case):
    """Bytes: the matrices in and out once.  Flops: a Schur (spectral)
    factorisation, the first iterate and two corrections with their residuals
    by the textbook counts, symmetric outputs counted once; complex
    arithmetic as real operations."""
    n, b, call, kind = case["n"], case["batch"], case["call"], case["kind"]
    n3 = float(n) ** 3
    item = 16 if kind in ("hpd", "square") else 8
    if kind in ("spd", "spd_batch", "hpd"):
        factor = (4 / 3 + 4 / 3 + 2 + 1) * n3  # reduction, eigenvectors, back-transformation, X_0
        sweep, resid = 6 * n3, n3
    else:
        factor = (25 + 4) * n3  # real Schur form with vectors, Q S Q^T
        sweep, resid = (8 + 2) * n3, 2 * n3
    if call == "refine":
        flops = 2 * sweep + 3 * resid
    elif case["prec"] == "fp64":
        flops = factor + resid
    else:
        flops = factor + 2 * sweep + 3 * resid
    tensors = 2
    if call == "grad":
        flops += 2 * (sweep + resid)
        tensors = 4  # A, Gbar, X, G
    elif call == "refine":
        tensors = 3
    elif call == "rootm":
        flops += 2 * 2 * n3 * 2
    if item == 16:
        flops *= 4
    return {"bytes": float(tensors * b * n * n * item), "flops": b * flops}


# ------------------------------------------------------------ 64-bit answers

def _db_sqrt(a):
    """Principal square root by the product form of the Denman-Beavers
    iteration in float64."""
    eye = torch.eye(a.shape[-1], device=a.device, dtype=a.dtype)
    m, x = a.clone(), a.clone()
    for _ in range(40):
        mi = torch.linalg.inv(m)
        x = 0.5 * x @ (eye + mi)
        m = 0.5 * (eye + 0.5 * (m + mi))
        if float(torch.linalg.matrix_norm(m - eye)) < 1e-14 * a.shape[-1]:
            break
    return x


def _adjoint(x, gbar):
    """G with X^T G + G X^T = Gbar from the eigendecomposition of X^T."""
    w, v = torch.linalg.eig(x.mT.cpu())
    vi = torch.linalg.inv(v)
    c = vi @ gbar.cpu().to(C128) @ v
    return (v @ (c / (w[:, None] + w[None, :])) @ vi).real


def exact(case, seed):
    a, known, extra = _inputs(case, seed)
    kind = case["kind"]
    if kind in ("square", "cube"):
        return {"x": known}
    if kind == "nonsym":
        x = _db_sqrt(a)
        if case["call"] != "grad":
            return {"x": x}
        return {"x": x, "g": _adjoint(x, extra["gbar"]) if case["n"] <= 768 else None}
    xs, gs = [], []
    for i, (q, lam) in enumerate(known):
        s, qh = torch.sqrt(lam), q.mH.contiguous()
        xs.append((q * s.to(q.dtype)[None, :]) @ qh)
        if case["call"] == "grad":
            c = qh @ extra["gbar"][i] @ q
            gs.append(q @ (c / (s[:, None] + s[None, :])) @ qh)
    if case["call"] == "grad":
        return {"x": torch.stack(xs), "g": torch.stack(gs)}
    return {"x": torch.stack(xs) if kind == "spd_batch" else xs[0]}
