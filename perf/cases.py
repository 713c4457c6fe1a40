"""Performance cases of the library: what a program that uses it calls, over the sizes it is used at.

A case is a dict of plain values.  ``kind`` names the entry point:

* ``apply``         api.laplacian_apply: y = Delta x for n link fields (FP64 or FP32);
* ``spectrum``      api.power_spectrum: Chebyshev moments and window powers of n sources;
* ``filter``        api.cheb_filter: the window projections of n fields;
* ``solve``         api.rational_apply: R(Delta) x, every shift to its FP64 residual (mode 0: FP64, 1: mixed);
* ``kinetic_force`` api.kinetic_force: K and dK/d omega (two solves and the link derivative);
* ``spectrum_bwd``  api.power_spectrum_bwd: gradients of the window powers for the source and the links;
* ``gauge_force``   api.wilson_gauge_force: the Wilson force and action;
* ``leapfrog``      api.leapfrog_step: one implicit leapfrog step.

The launch configuration is the library's default (no autotuning), as in a program that only calls
these functions.  Links are 1 + i eps H projected onto SU(3) (H Gaussian in the generators) or Haar;
fields are Gaussian.  ``exact`` computes the outputs from their definitions in FP64 with torch alone.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2112_04556_amd import api, inputs

ITERS = {0.9: 31, 0.5: 26}     # multi-shift iterations of the kappa pole sets at tol 1e-10
TOL = 1e-10
BETA = 5.5


def _case(name, kind, L, n=1, dtype="f64", links="eps", **kw):
    c = {"kind": kind, "L0": L[0], "L1": L[1], "L2": L[2], "L3": L[3], "n": n, "dtype": dtype, "links": links,
         "eps": 0.5}
    if name:
        c["name"] = name
    c.update(kw)
    return c


def listed():
    return [
        # the smallest lattice of the tests and of quick checks: one launch, latency only
        _case("apply_f64_4x4x4x4", "apply", (4, 4, 4, 4), eps=0.3),
        # the largest single-GPU lattice: one link field in HBM
        _case("apply_f64_32x32x32x64", "apply", (32, 32, 32, 64), eps=0.4),
        # a small FP32 batch on the paper's intermediate lattice
        _case("apply_f32_24x24x24x24_n4", "apply", (24, 24, 24, 24), n=4, dtype="f32", links="haar"),
        # stochastic spectra: a batch of FP32 sources on Haar links
        _case("spectrum_f32_24x24x24x24_n8", "spectrum", (24, 24, 24, 24), n=8, dtype="f32", links="haar",
              degree=64, windows=64),
        # a ragged lattice (rows that do not divide a wavefront), FP64, odd degree
        _case("spectrum_f64_12x10x14x9_n2", "spectrum", (12, 10, 14, 9), n=2, degree=33, windows=16),
        # projecting a momentum field onto a few windows
        _case("filter_f64_16x16x16x16", "filter", (16, 16, 16, 16), degree=32, windows=4),
        # the rational mass term at the paper's 16^4, one field in FP64 and a batch in mixed precision
        _case("solve_f64_16x16x16x16", "solve", (16, 16, 16, 16), kappa=0.9, poles=12, mode=0),
        _case("solve_mixed_16x16x16x16_n8", "solve", (16, 16, 16, 16), n=8, kappa=0.9, poles=12, mode=1),
        # the force of a molecular-dynamics step
        _case("kinetic_force_mixed_16x16x16x16", "kinetic_force", (16, 16, 16, 16), kappa=0.9, poles=8, mode=1,
              eps=0.4),
        # gradients of a spectrum (training or tuning a window)
        _case("spectrum_bwd_16x16x16x16", "spectrum_bwd", (16, 16, 16, 16), degree=64, windows=16),
        # the force whose spectrum is measured, on the largest lattice
        _case("gauge_force_32x32x32x64", "gauge_force", (32, 32, 32, 64), eps=0.4),
        # a whole integrator step on a small lattice: long chains of small launches
        _case("leapfrog_12x12x12x12", "leapfrog", (12, 12, 12, 12), kappa=0.9, poles=12, mode=0, step=0.02),
    ]


def _volume(c):
    return c["L0"] * c["L1"] * c["L2"] * c["L3"]


def _cost(c):
    """Site-fields moved by all stencil sweeps and vector passes of a case, FP32 counted half."""
    k = c["kind"]
    sweeps = {"apply": 1, "gauge_force": 4, "spectrum": (c.get("degree", 0) + 1) // 2, "filter": c.get("degree", 0),
              "spectrum_bwd": 8 * c.get("degree", 0)}.get(k)
    if sweeps is None:
        sweeps = 3 * ITERS[c["kappa"]] * {"solve": 1, "kinetic_force": 2, "leapfrog": 16}[k] + 8 * c["poles"]
    return _volume(c) * c["n"] * sweeps * (0.5 if c["dtype"] == "f32" else 1.0)


def _extents(rng, lo, hi):
    """Four extents whose product is spread over [lo, hi] on a log scale; half of the lattices are made of
    multiples of 4 (production shapes), the others of any extents, odd ones among them."""
    while True:
        side = math.exp(rng.uniform(math.log(lo), math.log(hi))) ** 0.25
        L = [max(2, int(round(side * math.exp(rng.uniform(-0.35, 0.35))))) for _ in range(4)]
        if rng.random() < 0.5 and side >= 6:
            L = [max(4, 4 * int(round(v / 4))) for v in L]
        if lo <= L[0] * L[1] * L[2] * L[3] <= hi:
            return tuple(L)


def draw(rng):
    limit = max(_cost(c) for c in listed())
    while True:
        kind = rng.choice(["apply", "apply", "spectrum", "filter", "solve", "kinetic_force", "spectrum_bwd",
                           "gauge_force", "leapfrog"])
        hi = {"apply": 2097152, "gauge_force": 2097152, "spectrum": 331776, "filter": 331776, "solve": 331776,
              "kinetic_force": 131072, "spectrum_bwd": 131072, "leapfrog": 20736}[kind]
        L = _extents(rng, 256, hi)
        links = rng.choice(["eps", "haar"])
        c = _case(None, kind, L, links=links, eps=rng.choice([0.3, 0.4, 0.5]))
        if kind in ("apply", "spectrum"):
            c["dtype"] = rng.choice(["f64", "f32"])
        if kind in ("apply", "spectrum", "filter", "solve"):
            c["n"] = rng.choice([1, 1, 2, 3, 4, 5, 8])
        if kind in ("spectrum", "filter", "spectrum_bwd"):
            c["degree"] = int(round(math.exp(rng.uniform(math.log(8), math.log(128)))))
            c["windows"] = rng.choice([2, 4, 7, 16] if kind == "filter" else [4, 16, 33, 64])
        if kind in ("solve", "kinetic_force", "leapfrog"):
            c["links"] = "eps"
            c["kappa"] = rng.choice([0.9, 0.5])
            c["poles"] = rng.choice([8, 12, 16])
            c["mode"] = rng.choice([0, 1])
        if kind == "leapfrog":
            c["step"] = 0.02
        if _cost(c) <= limit:
            return c


# ------------------------------------------------------------------------------------------
# inputs

def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _generator(seed, stream, device):
    g = torch.Generator(device=device)
    g.manual_seed((int(seed) * 1_000_003 + stream * 7919 + 17) % (2 ** 62))
    return g


def _links(c, seed, device):
    """Complex SU(3) links (4, V, 3, 3)."""
    V = _volume(c)
    g = _generator(seed, 0, device)
    out = torch.empty((4, V, 3, 3), dtype=torch.complex128, device=device)
    T = inputs.gell_mann_half().to(device)
    for mu in range(4):
        if c["links"] == "haar":
            z = torch.randn(2, V, 3, 3, generator=g, dtype=torch.float64, device=device)
            out[mu] = inputs.reunitarize(torch.complex(z[0], z[1]))
        else:
            h = torch.randn(V, 8, generator=g, dtype=torch.float64, device=device).to(torch.complex128)
            m = (1j * c["eps"] * (h @ T.reshape(8, 9))).reshape(V, 3, 3)
            out[mu] = inputs.reunitarize(m + torch.eye(3, dtype=torch.complex128, device=device))
    return out


def _fields(c, seed, device):
    g = _generator(seed, 1, device)
    x = torch.randn(c["n"], 4, 8, _volume(c), generator=g, dtype=torch.float64, device=device)
    return x if c["dtype"] == "f64" else x.float()


def _gamma(c, seed):
    return np.random.default_rng(int(seed) % (2 ** 32)).standard_normal((c["n"], c["windows"]))


def prepare(case, seed):
    c = case
    dev = torch.device("cuda")
    dt = torch.float64 if c["dtype"] == "f64" else torch.float32
    L = (c["L0"], c["L1"], c["L2"], c["L3"])
    st = {"c": c, "L": L, "U": api.pack_links(L, _links(c, seed, dev), dt)}
    if c["kind"] != "gauge_force":
        st["x"] = _fields(c, seed, dev)
    if "kappa" in c:
        st["rat"] = api.rational_kappa(c["kappa"], c["poles"])
        st["solver"] = api.Solver(tol=TOL, mode=c["mode"])
    if c["kind"] == "spectrum_bwd":
        st["gamma"] = _gamma(c, seed)
    return st


def run(state):
    c, L, U = state["c"], state["L"], state["U"]
    k = c["kind"]
    if k == "apply":
        return api.laplacian_apply(L, U, state["x"])
    if k == "spectrum":
        return api.power_spectrum(L, U, state["x"], c["degree"], c["windows"])
    if k == "filter":
        return api.cheb_filter(L, U, state["x"], c["degree"], c["windows"])
    if k == "solve":
        out = api.rational_apply(L, U, state["x"], state["rat"], state["solver"])
        return out["y"], out["K"]
    if k == "kinetic_force":
        out = api.kinetic_force(L, U, state["x"], state["rat"], state["solver"])
        return out["K"], out["dK"]
    if k == "spectrum_bwd":
        return api.power_spectrum_bwd(L, U, state["x"], state["gamma"], c["degree"], c["windows"])
    if k == "gauge_force":
        return api.wilson_gauge_force(L, U, BETA)
    U1, P1, _ = api.leapfrog_step(L, U, state["x"], state["rat"], c["step"], BETA, state["solver"], fp_tol=TOL)
    return U1, P1


# ------------------------------------------------------------------------------------------
# the work of one pass

def work(case):
    """Bytes and flops of one pass.  Per site a stencil sweep reads the 48 link reals that determine four
    SU(3) matrices and 32 reals per input field, and writes 32 per output field; it needs the four 8x8
    adjoint matrices (about 500 flops each) and eight 8x8 by 8x4 products per field.  A recursion or CG
    iteration depends on the whole of the one before, so each counts its own sweep."""
    c = case
    V, n, k = _volume(c), c["n"], c["kind"]
    ts = 8 if c["dtype"] == "f64" else 4
    lap_flops = V * (4 * 500 + n * 8 * 4 * 64 * 2)
    link_deriv = V * 4 * n * (4 * 64 * 4 + 1500)

    def solve():
        # per iteration: links, the residual and the direction read and written; the shifts' solutions
        # are sums over the residuals, written once
        it, p = ITERS[c["kappa"]], c["poles"]
        return (V * ts * (it * (48 + 128 * n) + 32 * n * (2 + 2 * p)),
                it * (lap_flops + V * n * 32 * (8 + 4 * p)))

    if k == "apply":
        by, fl = V * ts * (48 + 64 * n), lap_flops
    elif k == "spectrum":
        K = (c["degree"] + 1) // 2
        by, fl = V * ts * (48 * K + 32 * n * (3 * K - 2)), K * (lap_flops + V * n * 32 * 6)
    elif k == "filter":
        D, w = c["degree"], c["windows"]
        by, fl = V * ts * (48 * D + 32 * n * (3 * D - 1 + w)), D * (lap_flops + V * n * 32 * 2 * w)
    elif k == "solve":
        by, fl = solve()
    elif k == "kinetic_force":
        sb, sf = solve()
        by, fl = 2 * sb + V * ts * (48 + 32 + 64 * n * c["poles"]), 2 * sf + c["poles"] * link_deriv
    elif k == "spectrum_bwd":
        D = c["degree"]
        by = V * ts * (48 * 2 * D + 32 * n * (3 * 3 * D) + 64 * D)
        fl = D * (3 * lap_flops + link_deriv)
    elif k == "gauge_force":
        by, fl = V * ts * (48 + 32), V * 4 * 13 * 216
    else:
        sb, sf = solve()
        by, fl = 16 * sb, 16 * sf
    return {"bytes": by, "flops": fl}


# ------------------------------------------------------------------------------------------
# the outputs in FP64 from their definitions

class _Operator:
    """Delta on component fields (..., 4, 8, V): the adjoint matrices R^{ab} = 2 Re Tr(T^a U T^b U^dag)
    of all 18 stored link reals, periodic shifts by torch.roll."""

    def __init__(self, c, U):
        self.shape = (c["L3"], c["L2"], c["L1"], c["L0"])
        self.V = _volume(c)
        T = inputs.gell_mann_half().to(U.device)
        self.R = torch.empty((4, 8, 8, self.V), dtype=torch.float64, device=U.device)
        for mu in range(4):
            Uc = U[mu].conj()
            for b in range(8):
                W = U[mu] @ T[b]
                Y = (W[:, :, None, :] * Uc[:, None, :, :]).sum(-1)
                for a in range(8):
                    self.R[mu, a, b] = 2.0 * (T[a].T * Y).sum((-1, -2)).real

    def at(self, x, mu, sign):
        """x(s + sign mu)."""
        y = x.reshape(x.shape[:-1] + self.shape)
        return torch.roll(y, -sign, dims=y.dim() - 1 - mu).reshape(x.shape)

    def lap(self, x):
        out = 8.0 * x
        for mu in range(4):
            f, R = self.at(x, mu, +1), self.R[mu]
            back = torch.zeros_like(x)
            for a in range(8):
                out -= R[:, a] * f[..., a:a + 1, :]
                back += R[a] * x[..., a:a + 1, :]          # R^T x at the link's own site
            out -= self.at(back, mu, -1)
        return out

    def cheb(self, x, degree):
        """T_k(Delta/8 - 1) x for k = 0..degree."""
        t0 = x
        yield t0
        t1 = self.lap(x) / 8.0 - x
        yield t1
        for _ in range(2, degree + 1):
            t0, t1 = t1, 2.0 * (self.lap(t1) / 8.0 - t1) - t0
            yield t1

    def cg(self, b, sigma):
        """(Delta + sigma)^{-1} b for every leading field, to rounding."""
        def dot(u, v):
            return (u * v).sum((-1, -2, -3), keepdim=True)
        x, r, p = torch.zeros_like(b), b.clone(), b.clone()
        rr = bb = dot(b, b)
        for _ in range(2000):
            Ap = self.lap(p) + sigma * p
            al = rr / dot(p, Ap)
            x += al * p
            r -= al * Ap
            rn = dot(r, r)
            if bool((rn <= 1e-30 * bb).all()):
                break
            p = r + (rn / rr) * p
            rr = rn
        return x

    def link_derivative(self, A, B, weight, C):
        """C[mu][b][e] += weight sum (B(x+mu)^b A(x)^e + A(x+mu)^b B(x)^e), summed over the fields and nu."""
        A, B = A.reshape(-1, 8, self.V), B.reshape(-1, 8, self.V)
        for mu in range(4):
            Af, Bf = self.at(A, mu, +1), self.at(B, mu, +1)
            for b in range(8):
                C[mu, b] += weight * (Bf[:, b:b + 1] * A + Af[:, b:b + 1] * B).sum(0)

    def contract(self, C):
        """G^c = sum_{d,e} f^{dec} (R C)^{de}: the derivative for U -> exp(i omega^c T^c) U."""
        T = inputs.gell_mann_half()
        out = torch.zeros((4, 8, self.V), dtype=torch.float64, device=C.device)
        f = torch.zeros(8, 8, 8, dtype=torch.float64)
        for d in range(8):
            for e in range(8):
                com = T[d] @ T[e] - T[e] @ T[d]
                for k in range(8):
                    f[d, e, k] = (-2j * torch.trace(com @ T[k])).real
        for mu in range(4):
            RC = torch.zeros_like(C[mu])
            for b in range(8):
                RC += self.R[mu][:, b:b + 1] * C[mu][b:b + 1]
            for d in range(8):
                for e in range(8):
                    for k in range(8):
                        if abs(f[d, e, k]) > 1e-12:
                            out[mu, k] += float(f[d, e, k]) * RC[d, e]
        return out


def _window_coefficients(degree, windows):
    """Jackson-damped Chebyshev coefficients of equal windows on [0, 16]."""
    th = np.arccos(np.clip(np.linspace(0.0, 16.0, windows + 1) / 8.0 - 1.0, -1.0, 1.0))
    k = np.arange(1, degree + 1)
    co = np.empty((windows, degree + 1))
    co[:, 0] = (th[:-1] - th[1:]) / np.pi
    co[:, 1:] = 2.0 * (np.sin(np.outer(th[:-1], k)) - np.sin(np.outer(th[1:], k))) / (k * np.pi)
    N = degree + 1
    q = np.pi / (N + 1)
    j = np.arange(N)
    return co * (((N - j + 1) * np.cos(q * j) + np.sin(q * j) / np.tan(q)) / (N + 1))


def _poles(c):
    n, kappa = c["poles"], c["kappa"]
    s = math.sqrt((1.0 - kappa) * (1.0 + 15.0 * kappa))
    th = (2.0 * np.arange(1, n + 1) - 1.0) * np.pi / (4.0 * n)
    return np.sqrt(s) / (n * kappa * np.cos(th) ** 2), (1.0 - kappa + s * np.tan(th) ** 2) / kappa


def _gauge_exact(c, U):
    shape = (c["L3"], c["L2"], c["L1"], c["L0"])
    T = inputs.gell_mann_half().to(U.device)

    def at(m, mu, sign):
        y = m.reshape(shape + (3, 3))
        return torch.roll(y, -sign, dims=3 - mu).reshape(m.shape)

    def mul(a, b):
        return (a[:, :, :, None] * b[:, None, :, :]).sum(-2)

    def dag(a):
        return a.conj().transpose(-1, -2)

    F = torch.empty((4, 8, U.shape[1]), dtype=torch.float64, device=U.device)
    plaq = 0.0
    for mu in range(4):
        A = torch.zeros_like(U[mu])
        for nu in range(4):
            if nu != mu:
                corner = mul(at(U[nu], mu, +1), dag(at(U[mu], nu, +1)))
                A += mul(corner, dag(U[nu]))
                low = mul(dag(at(U[nu], mu, +1)), mul(dag(U[mu]), U[nu]))
                A += at(low, nu, -1)
        M = mul(U[mu], A)
        for a in range(8):
            F[mu, a] = -(BETA / 3.0) * (T[a].T * M).sum((-1, -2)).imag
        plaq += float(M.diagonal(dim1=-2, dim2=-1).real.sum())
    return F, BETA * (6.0 * U.shape[1] - plaq / 12.0)


def exact(case, seed):
    c = case
    k = c["kind"]
    if k == "leapfrog" or _cost(c) * c["n"] > 4e9:
        return None
    dev = _device()
    U = _links(c, seed, dev)
    if c["dtype"] == "f32":
        U = U.to(torch.complex64).to(torch.complex128)
    if k == "gauge_force":
        return _gauge_exact(c, U)
    op = _Operator(c, U)
    del U
    x = _fields(c, seed, dev).double()
    if k == "apply":
        return op.lap(x)
    if k in ("solve", "kinetic_force"):
        r, s = _poles(c)
        xs = [op.cg(x, float(sj)) for sj in s]
        y = sum(float(rj) * xj for rj, xj in zip(r, xs))
        K = 0.5 * (y * y).sum((-1, -2, -3)).cpu().numpy()
        if k == "solve":
            return y, K
        C = torch.zeros((4, 8, 8, op.V), dtype=torch.float64, device=dev)
        for rj, sj, xj in zip(r, s, xs):
            op.link_derivative(op.cg(y, float(sj)), xj, -float(rj), C)
        return K, op.contract(C)[None]
    D = c["degree"]
    co = _window_coefficients(D, c["windows"])
    if k == "spectrum":
        mom = np.stack([(x * t).sum((-1, -2, -3)).cpu().numpy() for t in op.cheb(x, D)], axis=1)
        return mom, mom @ co.T
    if k == "filter":
        y = torch.zeros((c["windows"],) + tuple(x.shape), dtype=torch.float64, device=dev)
        for j, t in enumerate(op.cheb(x, D)):
            for w in range(c["windows"]):
                y[w] += float(co[w, j]) * t
        return y
    # spectrum_bwd: with beta_k = sum_w gamma_w co[w, k], the adjoint vectors of t_k obey
    # tb_k = beta_k F + 2 A tb_{k+1} - tb_{k+2}; grad_F = 2 p(A) F
    beta = torch.as_tensor(_gamma(c, seed) @ co, device=dev)
    t = list(op.cheb(x, D))
    gF = sum(2.0 * beta[:, j, None, None, None] * tj for j, tj in enumerate(t))
    C = torch.zeros((4, 8, 8, op.V), dtype=torch.float64, device=dev)
    b1, b2 = torch.zeros_like(x), torch.zeros_like(x)
    for j in range(D, 0, -1):
        b1, b2 = beta[:, j, None, None, None] * x + 2.0 * (op.lap(b1) / 8.0 - b1) - b2, b1
        op.link_derivative(b1, t[j - 1], 0.125 if j == 1 else 0.25, C)
    return gF, op.contract(C)[None]
