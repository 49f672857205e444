"""Performance cases of the eigensolver library: its steps and its whole calls
through the public Python entry points, over the sizes a user runs them at.

A case is a dict of plain values with a "kind":

  filter    chase_filter on a start block (FP64, or FP64 products on INT8)
  ritz      chase_filter_ritz, the defect-correction form of the mixed modes
  lanczos   chase_lanczos, the spectral bounds
  qr        chase_qr, the orthonormalisation of a filtered block
  rr        chase_rayleigh_ritz on a nearly converged block
  solve     chase_solve, Algorithm 1 from library-drawn start blocks
  filter_grad   chase_filter with a recorded tape, then chase_filter_adjoint
  eigvec_grad   chase_eigval_adjoint and chase_eigvec_adjoint of the lowest pairs

A program keeps its handle (the library's workspace) from call to call, so
prepare() makes it; H, the blocks and everything else are drawn from the
seed on the GPU.  Eigenvectors are returned with their free phase fixed
against a reference vector, as programs that compare or continue them do.
"""
import math

import numpy as np
import torch

import paper_2205_02491_amd as pk

DEV = "cuda"
# filter interval of the cases whose H is a scaled Gaussian Hermitian matrix
# (spectrum on [-1, 1]): the lowest ~10% are wanted
B_SUP, MU_1, MU_NE = 1.02, -1.01, -0.7


def listed():
    return [
        # the smallest calls a program makes: a small dense problem stepped by
        # hand, where launches and latency are all there is
        dict(name="filter_c128_256x16", kind="filter", n=256, k=16, cplx=True, deg_lo=20,
             deg_hi=20, emu=0),
        # first filter of the small workload (n=1000, nev 100, nex 40, degree 20)
        dict(name="filter_c128_1000x140", kind="filter", n=1000, k=140, cplx=True, deg_lo=20,
             deg_hi=20, emu=0),
        # a later iteration of a real problem: ragged sizes, optimised degrees
        dict(name="filter_f64_5003x173", kind="filter", n=5003, k=173, cplx=False, deg_lo=4,
             deg_hi=26, emu=0),
        # the flagship workload's block (n=20000, nev 1000, nex 300), optimised degrees
        dict(name="filter_c128_20000x1300", kind="filter", n=20000, k=1300, cplx=True, deg_lo=2,
             deg_hi=10, emu=0),
        # FP64 products on the INT8 matrix cores (14 moduli)
        dict(name="filter_int8_c128_4000x260", kind="filter", n=4000, k=260, cplx=True, deg_lo=10,
             deg_hi=20, emu=14),
        # a defect-form pass of the two-term split-BF16 mode
        dict(name="ritz_bf16x2_c128_8000x260", kind="ritz", n=8000, k=260, cplx=True, deg_lo=8,
             deg_hi=24, prec=pk.PREC_BF16X2),
        # spectral bounds at the differentiation workload's size (n=8000)
        dict(name="lanczos_c128_8000", kind="lanczos", n=8000, k=260, cplx=True, nvec=4,
             steps=25),
        # QR of the flagship workload's block
        dict(name="qr_c128_20000x1300", kind="qr", n=20000, k=1300, cplx=True, locked=0),
        # Rayleigh-Ritz of a nearly converged block (n=8000, nev 200, nex 60)
        dict(name="rr_c128_8000x260", kind="rr", n=8000, k=260, cplx=True),
        # the small workload end to end
        dict(name="solve_c128_1000", kind="solve", n=1000, nev=100, nex=40, cplx=True),
        # forward and backward of a differentiable filtered block
        dict(name="filter_grad_c128_3000x96", kind="filter_grad", n=3000, k=96, cplx=True,
             deg_lo=10, deg_hi=10),
        # backward of eigenvalues and eigenvectors, real symmetric
        dict(name="eigvec_grad_f64_2000x100", kind="eigvec_grad", n=2000, k=100, cplx=False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Sizes from the smallest listed to a few thousand rows (blocks of up to
    a tenth of them), so that a drawn case stays below the largest listed."""
    kind = rng.choice(["filter", "filter", "filter", "filter", "ritz", "lanczos", "qr", "rr",
                       "solve", "filter_grad", "eigvec_grad"])
    cplx = rng.random() < 0.6
    if kind == "filter":
        emu = 14 if rng.random() < 0.2 else 0
        n = _log_int(rng, 200, 4500 if emu else 9000)
        lo = 2 * rng.randint(1, 10)
        return dict(kind=kind, n=n, k=_log_int(rng, 8, max(12, n // 10)), cplx=cplx, deg_lo=lo,
                    deg_hi=lo + 2 * rng.randint(0, 8), emu=emu)
    if kind == "ritz":
        n = _log_int(rng, 500, 9000)
        lo = 2 * rng.randint(2, 8)
        return dict(kind=kind, n=n, k=_log_int(rng, 8, max(12, n // 10)), cplx=cplx, deg_lo=lo,
                    deg_hi=lo + 2 * rng.randint(0, 8),
                    prec=rng.choice([pk.PREC_FP32, pk.PREC_BF16X3, pk.PREC_BF16X2]))
    if kind == "lanczos":
        n = _log_int(rng, 300, 12000)
        return dict(kind=kind, n=n, k=max(10, n // 20), cplx=cplx, nvec=rng.choice([4, 4, 8, 1]),
                    steps=rng.choice([25, 25, 15]))
    if kind == "qr":
        n = _log_int(rng, 300, 15000)
        k = _log_int(rng, 12, min(1000, max(16, n // 8)))
        return dict(kind=kind, n=n, k=k, cplx=cplx,
                    locked=0 if rng.random() < 0.6 else rng.randint(1, k // 2))
    if kind == "rr":
        n = _log_int(rng, 300, 8000)
        return dict(kind=kind, n=n, k=_log_int(rng, 12, max(16, n // 20)), cplx=cplx)
    if kind == "solve":
        n = _log_int(rng, 300, 1800)
        nev = rng.randint(max(8, n // 25), n // 9)
        return dict(kind=kind, n=n, nev=nev, nex=max(6, int(nev * rng.uniform(0.3, 0.5))),
                    cplx=cplx)
    if kind == "filter_grad":
        n = _log_int(rng, 200, 4000)
        lo = 2 * rng.randint(2, 6)
        return dict(kind=kind, n=n, k=_log_int(rng, 8, max(12, n // 20)), cplx=cplx, deg_lo=lo,
                    deg_hi=lo + 2 * rng.randint(0, 3))
    n = _log_int(rng, 200, 2000)
    return dict(kind="eigvec_grad", n=n, k=_log_int(rng, 6, max(8, n // 15)), cplx=cplx)


# ------------------------------------------------------------------ inputs
def _dtype(case):
    return torch.complex128 if case["cplx"] else torch.float64


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _randn(g, shape, dt):
    return torch.randn(shape, generator=g, dtype=dt, device=DEV)


def _gaussian_hermitian(n, dt, g):
    """Gaussian Hermitian (symmetric) matrix scaled to the spectrum [-1, 1]."""
    z = _randn(g, (n, n), dt)
    h = z + z.mH
    del z
    # entries of z + z^H have variance 2: semicircle radius 2 sqrt(2 n)
    h /= 2.0 * math.sqrt(2.0 * n)
    return h


def _jittered(n, g, lo=-1.0, hi=1.0):
    """Ascending values on [lo, hi], evenly spaced up to a random shift of at
    most 0.3 spacings each."""
    u = torch.rand(n, generator=g, dtype=torch.float64, device=DEV)
    return lo + (hi - lo) * (torch.arange(n, dtype=torch.float64, device=DEV) + 0.5
                             + 0.6 * (u - 0.5)) / n


def _haar(n, dt, g):
    q, r = torch.linalg.qr(_randn(g, (n, n), dt))
    d = torch.diagonal(r)
    return q * (d / d.abs())[None, :]


def _planted(q, lam):
    h = torch.matmul(q * lam[None, :].to(q.dtype), q.mH.contiguous())
    return ((h + h.mH) / 2).contiguous()


def _reflected(n, dt, g, lam, k):
    """(H, V): H = R diag(lam) R with R = I - 2 U U^H a block reflector, and
    the eigenvectors V = R[:, :k] of the k lowest values."""
    u, _ = torch.linalg.qr(_randn(g, (n, 32), dt))
    du = lam[:, None].to(dt) * u
    t = 2.0 * torch.matmul(u, torch.matmul(u.mH, du)) - du
    # R D R = D + 2 (2 U U^H D U - D U) U^H - 2 U (D U)^H
    h = 2.0 * torch.matmul(t, u.mH.contiguous())
    h -= 2.0 * torch.matmul(u, du.mH.contiguous())
    idx = torch.arange(n, device=DEV)
    h[idx, idx] += lam.to(dt)
    h = ((h + h.mH) / 2).contiguous()
    v = -2.0 * torch.matmul(u, u[:k].mH.contiguous())
    v[torch.arange(k, device=DEV), torch.arange(k, device=DEV)] += 1.0
    return h, v


def _degrees(case):
    k, lo, hi = case["k"], case["deg_lo"], case["deg_hi"]
    d = lo + (hi - lo) * (np.arange(k) + 1) / k
    return (2 * np.ceil(d / 2)).astype(np.int32)


def _inputs(case, seed):
    """The tensors of a case, from the seed alone."""
    kind, n, dt = case["kind"], case["n"], _dtype(case)
    g = _gen(seed)
    if kind in ("filter", "filter_grad"):
        s = dict(H=_gaussian_hermitian(n, dt, g), X=_randn(g, (n, case["k"]), dt))
        if kind == "filter_grad":
            s["gY"] = _randn(g, (n, case["k"]), dt)
        return s
    if kind == "ritz":
        # residuals of a few correct digits around shifts at the wanted end
        v, _ = torch.linalg.qr(_randn(g, (n, case["k"]), dt))
        theta = torch.linspace(-1.0, MU_NE - 0.02, case["k"], dtype=torch.float64)
        r = _randn(g, (n, case["k"]), dt) * (1e-4 / math.sqrt(n))
        return dict(H=_gaussian_hermitian(n, dt, g), V=v.contiguous(), R=r, theta=theta.numpy())
    if kind == "lanczos":
        return dict(H=_gaussian_hermitian(n, dt, g), S=_randn(g, (n, case["nvec"]), dt))
    if kind == "qr":
        # a filtered block: columns of very different lengths, condition ~1e3
        k = case["k"]
        x = _randn(g, (n, k), dt)
        x += 30.0 * x[:, :1] * torch.rand(k, generator=g, dtype=torch.float64, device=DEV)[None]
        x *= torch.logspace(0, 3, k, dtype=torch.float64, device=DEV)[None]
        if case["locked"]:
            x[:, :case["locked"]] = torch.linalg.qr(x[:, :case["locked"]])[0]
        return dict(X=x.contiguous())
    if kind == "rr":
        lam = _jittered(n, g)
        h, v = _reflected(n, dt, g, lam, case["k"])
        v = v + _randn(g, v.shape, dt) * (1e-3 / math.sqrt(n))
        return dict(H=h, Q=torch.linalg.qr(v)[0].contiguous(), ref=_randn(g, (1, n), dt))
    if kind == "solve":
        return dict(H=_planted(_haar(n, dt, g), _jittered(n, g)), ref=_randn(g, (1, n), dt))
    # eigvec_grad: k wanted pairs on [-1, -0.8], the others on [-0.5, 1]
    k = case["k"]
    lam = torch.cat([_jittered(k, g, -1.0, -0.8), _jittered(n - k, g, -0.5, 1.0)])
    q = _haar(n, dt, g)
    return dict(H=_planted(q, lam), q=q, lam=lam, V=q[:, :k].contiguous(),
                G=_randn(g, (n, k), dt), gl=np.random.RandomState(seed % (1 << 31)).randn(k))


def prepare(case, seed):
    s = _inputs(case, seed)
    kind, n, dt = case["kind"], case["n"], _dtype(case)
    if kind == "eigvec_grad":
        s["lam"] = s["lam"][:case["k"]].cpu().numpy()
        del s["q"]
    kw = {}
    if case.get("emu"):
        kw["fp64_emulation"] = case["emu"]
    if kind == "ritz":
        kw["filter_prec"] = case["prec"]
    if kind == "filter_grad":
        kw["adjoint_reserve"] = case["deg_hi"]
    if kind == "eigvec_grad":
        kw["adjoint_reserve"] = 2
    if kind == "lanczos":
        kw.update(lanczos_vecs=case["nvec"], lanczos_steps=case["steps"])
    if kind == "solve":
        nev, nex = case["nev"], case["nex"]
    else:
        nev, nex = case["k"] - 1, 1
    s["handle"] = pk.Handle(n, nev, nex, dt, pk.default_opts(**kw))
    s["case"] = case
    if "deg_lo" in case:
        s["degrees"] = _degrees(case)
    return s


def _fix_phase(V, ref):
    """V's columns with ref^H v real and positive."""
    t = torch.matmul(ref.conj(), V)
    return V * (t.conj() / t.abs())


# ------------------------------------------------------------------ one pass
def run(s):
    case, h = s["case"], s["handle"]
    kind = case["kind"]
    if kind == "filter":
        return pk.chase_filter(s["H"], s["X"], s["degrees"], B_SUP, MU_1, MU_NE, handle=h)
    if kind == "ritz":
        return pk.chase_filter_ritz(s["H"], s["V"], s["R"], s["theta"], s["degrees"], B_SUP, MU_1,
                                    MU_NE, prec=case["prec"], handle=h)
    if kind == "lanczos":
        return pk.chase_lanczos(s["H"], s["S"], handle=h)
    if kind == "qr":
        return pk.chase_qr(s["X"], case["locked"], handle=h)
    if kind == "rr":
        ritz, V, res = pk.chase_rayleigh_ritz(s["H"], s["Q"], handle=h)
        return ritz, _fix_phase(V, s["ref"]), res
    if kind == "solve":
        ev, V, _, _ = pk.chase_solve(s["H"], case["nev"], case["nex"], 1e-12, 20, handle=h)
        return ev, _fix_phase(V, s["ref"])
    if kind == "filter_grad":
        Y, _ = pk.chase_filter(s["H"], s["X"], s["degrees"], B_SUP, MU_1, MU_NE,
                               record_tape=True, handle=h)
        dH = torch.zeros_like(s["H"])
        gX = pk.chase_filter_adjoint(s["H"], s["gY"], dH, h, want_gX=True)
        return Y, dH, gX
    dH = torch.zeros_like(s["H"])
    pk.chase_eigval_adjoint(s["V"], s["gl"], dH, handle=h)
    pk.chase_eigvec_adjoint(s["H"], s["V"], s["lam"], s["G"], dH, handle=h, tol=1e-11)
    return dH


# ------------------------------------------------------------------ work
def work(case):
    n = case["n"]
    cplx = case["cplx"]
    esz, f = (16, 8.0) if cplx else (8, 2.0)
    kind = case["kind"]
    h_bytes = float(n) * n * esz
    if kind == "solve":
        # one filter of degree 20 and Rayleigh-Ritz of the whole block at least
        k = case["nev"] + case["nex"]
        return dict(bytes=h_bytes + n * k * esz,
                    flops=f * n * n * k * 21 + f * n * k * k * 3.0)
    k = case["k"]
    blk = float(n) * k * esz
    if kind in ("filter", "ritz", "filter_grad"):
        mv = float(_degrees(case).sum())
        if kind == "ritz":
            return dict(bytes=h_bytes + 3 * blk, flops=f * n * n * (mv - k))
        if kind == "filter":
            return dict(bytes=h_bytes + 2 * blk, flops=f * n * n * mv)
        return dict(bytes=2 * h_bytes + 4 * blk, flops=3.0 * f * n * n * mv)
    if kind == "lanczos":
        # every step needs the whole of H after the step before it
        return dict(bytes=case["steps"] * h_bytes, flops=f * n * n * case["steps"] * case["nvec"])
    if kind == "qr":
        # Gram matrix (half of it), factor, triangular product
        return dict(bytes=2 * blk, flops=f * n * k * k)
    if kind == "rr":
        return dict(bytes=h_bytes + 2 * blk, flops=f * n * n * k + f * n * k * k * 2.5)
    # eigvec_grad: three rank-k updates and at least one product with H
    return dict(bytes=2 * h_bytes + 2 * blk, flops=f * n * n * k * 4)


# ------------------------------------------------------------------ 64-bit reference
def _coefs(m):
    c, e = 0.5 * (B_SUP + MU_NE), 0.5 * (B_SUP - MU_NE)
    s1 = e / (MU_1 - c)
    out, s = [(s1 / e, c, 0.0)], s1
    for _ in range(2, m + 1):
        sn = 1.0 / (2.0 / s1 - s)
        out.append((2.0 * sn / e, c, -s * sn))
        s = sn
    return out


def _filter_torch(H, X, deg):
    """p_{m_a}(H) x_a of Eq. (3)."""
    deg = torch.as_tensor(deg, device=X.device)
    prev, cur, out = torch.zeros_like(X), X, torch.zeros_like(X)
    for s, (a, c, b) in enumerate(_coefs(int(deg.max())), 1):
        prev, cur = cur, a * (torch.matmul(H, cur) - c * cur) + b * prev
        out = torch.where((deg == s)[None, :], cur, out)
    return out


def _ritz_torch(H, V, R, theta, deg):
    """p(H) V from H V = V diag(theta) + R (the relation the call is given)."""
    deg = torch.as_tensor(deg, device=V.device)
    th = torch.as_tensor(theta, device=V.device)[None, :].to(V.dtype)
    tp, t = torch.zeros_like(th), torch.ones_like(th)
    prev, cur, out = torch.zeros_like(V), torch.zeros_like(V), torch.zeros_like(V)
    for s, (a, c, b) in enumerate(_coefs(int(deg.max())), 1):
        nxt = a * (torch.matmul(H, cur) - c * cur) + b * prev + a * t * R
        prev, cur = cur, nxt
        tp, t = t, a * (th - c) * t + b * tp
        out = torch.where((deg == s)[None, :], t * V + cur, out)
    return out


def _tridiag_bounds(alpha, beta, n, n_e):
    b_sup, mu_1, nodes = -np.inf, np.inf, []
    nvec = alpha.shape[0]
    for a, b in zip(alpha, beta):
        th, y = np.linalg.eigh(np.diag(a) + np.diag(b[:-1], 1) + np.diag(b[:-1], -1))
        b_sup, mu_1 = max(b_sup, th[-1] + abs(b[-1])), min(mu_1, th[0])
        nodes += [(t, w * w / nvec) for t, w in zip(th, y[0])]
    cum = 0.0
    for t, w in sorted(nodes):
        cum += w
        if cum * n >= n_e * (1 - 1e-9):
            return b_sup, mu_1, min(max(t, mu_1), b_sup)
    return b_sup, mu_1, b_sup


def exact(case, seed):
    s = _inputs(case, seed)
    kind, n = case["kind"], case["n"]
    if kind == "filter":
        return _filter_torch(s["H"], s["X"], _degrees(case)), None
    if kind == "ritz":
        return _ritz_torch(s["H"], s["V"], s["R"], s["theta"], _degrees(case)), None
    if kind == "lanczos":
        H, w = s["H"], s["S"]
        q0, bt = torch.zeros_like(w), torch.zeros(w.shape[1], dtype=torch.float64, device=DEV)
        q = w / torch.linalg.vector_norm(w, dim=0)
        al, be = [], []
        for _ in range(case["steps"]):
            w = torch.matmul(H, q) - q0 * bt
            a = (q.conj() * w).sum(0).real
            w = w - q * a
            bt = torch.linalg.vector_norm(w, dim=0)
            q0, q = q, w / bt
            al.append(a)
            be.append(bt)
        al, be = torch.stack(al, 1).cpu().numpy(), torch.stack(be, 1).cpu().numpy()
        return (*_tridiag_bounds(al, be, n, case["k"]), al, be, None)
    if kind == "qr":
        X, L = s["X"], case["locked"]
        q, r = torch.linalg.qr(X)
        d = torch.diagonal(r)
        q = q * (d / d.abs())[None, :]
        if L:
            q[:, :L] = X[:, :L]
        return q
    if kind == "rr":
        P = torch.matmul(s["H"], s["Q"])
        G = torch.matmul(s["Q"].mH, P)
        th, W = torch.linalg.eigh(((G + G.mH) / 2).cpu())
        W, thd = W.to(DEV), th.to(DEV)
        V = torch.matmul(s["Q"], W)
        res = torch.linalg.vector_norm(torch.matmul(P, W) - V * thd[None, :], dim=0)
        return th.numpy(), _fix_phase(V, s["ref"]), res.cpu().numpy()
    if kind == "solve":
        th, U = torch.linalg.eigh(s["H"].cpu())
        m = case["nev"]
        return th[:m].numpy(), _fix_phase(U[:, :m].to(DEV), s["ref"])
    if kind == "filter_grad":
        H = s["H"].clone().requires_grad_(True)
        X = s["X"].clone().requires_grad_(True)
        Y = _filter_torch(H, X, _degrees(case))
        gH, gX = torch.autograd.grad(Y, (H, X), s["gY"])
        return Y.detach(), (gH + gH.mH) / 2, gX
    # eigvec_grad: first-order perturbation on the planted eigenvectors
    k, q, lam, V, G = case["k"], s["q"], s["lam"], s["V"], s["G"]
    C = torch.matmul(q.mH, G)                       # components of the gradient
    den = lam[:k][None, :] - lam[:, None]           # lambda_j - mu_i
    den[:k, :] += torch.eye(k, dtype=torch.float64, device=DEV)
    F = C / den.to(C.dtype)
    F[torch.arange(k), torch.arange(k)] = torch.as_tensor(s["gl"], device=DEV).to(C.dtype)
    A = torch.matmul(torch.matmul(q, F), V.mH.contiguous())
    return (A + A.mH) / 2
