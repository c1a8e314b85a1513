"""The work a user of this library has it do, as measurable cases.

A case is a dict of plain values: the kind of call, the box of nx * ny * nz hexahedra, lx
Gauss-Lobatto-Legendre points per direction, the mesh deformation and the coefficients.
`prepare` builds what a program holds before the call (mesh, gather-scatter and coefficient
handles, operands on the GPU), `run` makes one pass through the public entry points, `work`
states the bytes and operations that pass cannot do without, and `exact` evaluates the same
outputs from the definitions in 64-bit torch, sharing no code with the library.
"""
import math

import numpy as np
import torch

# Poisson (pressure) operator; velocity Helmholtz operator of the Re = 5000, dt = 5e-4 run;
# Helmholtz operator with a variable diffusivity h1 = exp(Gaussian random field), dt = 1e-3.
COEFS = {"poisson": (1.0, 0.0), "velocity": (1.0 / 5000.0, 1.0 / 5e-4), "variable": (None, 1000.0)}


def _case(name, kind, nx, ny, nz, lx, eps=0.05, coef="poisson", dtype="f64", nf=1, **more):
    c = dict(kind=kind, nx=nx, ny=ny, nz=nz, lx=lx, eps=eps, coef=coef, dtype=dtype, nf=nf, **more)
    return dict(c, name=name) if name else c


def listed():
    return [
        # The smallest call: operator, gather-scatter and mask on 64 affine elements, as a
        # verification run or one subdomain of a strongly scaled run makes it (launch latency).
        _case("apply_64el_lx6", "apply", 4, 4, 4, 6, eps=0.0),
        # 50 Jacobi-CG steps on the same mesh: the latency of a small solve's iteration.
        _case("pcg50_64el_lx6", "pcg", 4, 4, 4, 6, eps=0.0, iters=50),
        # The operator benchmark of the method's literature: lx = 10, up to 8192 elements.
        _case("ax_8192el_lx10", "ax", 16, 16, 32, 10),
        # The headline operator: 32^3 curved elements, lx = 8.
        _case("ax_32768el_lx8", "ax", 32, 32, 32, 8),
        # Ragged box, odd lx, FP32, every coefficient a field or non-zero.
        _case("ax_f32_7429el_lx7", "ax", 19, 23, 17, 7, coef="variable", dtype="f32"),
        # Three velocity components at high order sharing one read of the geometry.
        _case("ax3_32768el_lx12", "ax", 32, 32, 32, 12, coef="velocity", nf=3),
        # Assembly of a load vector (gather-scatter and mask) at the headline size.
        _case("assemble_32768el_lx8", "assemble", 32, 32, 32, 8),
        # A large FP64 Jacobi-CG solve, a fixed number of steps.
        _case("pcg200_32768el_lx8", "pcg", 32, 32, 32, 8, iters=200),
        # The velocity solve of a time step: three components at once, high order, FP32
        # iteration with FP64 reliable updates to 1e-10.
        _case("velocity_8000el_lx12", "velocity", 20, 20, 20, 12, coef="velocity", nf=3, rtol=1e-10),
        # The pressure solve of a time step: GMRES(10), two-level Schwarz with overlap.
        _case("pressure_32768el_lx8", "pressure", 32, 32, 32, 8, precond="schwarz_overlap", restart=10, rtol=1e-10),
        # A small ragged pressure solve with the defaults: GMRES(30), element-only Schwarz.
        _case("pressure_960el_lx6", "pressure", 12, 10, 8, 6, precond="schwarz", restart=30, rtol=1e-10),
        # Differentiated variable-coefficient solve: forward, adjoint solve and h1 gradient.
        _case("gradient_4096el_lx8", "gradient", 16, 16, 16, 8, coef="variable", rtol=1e-12),
    ]


def _box(rng, lx, most, least):
    """A box of elements with between about least and most local points, spread over the logarithm."""
    n = math.exp(rng.uniform(math.log(least), math.log(most))) / lx ** 3
    side = max(1.0, n) ** (1.0 / 3.0)
    a, b = rng.uniform(0.7, 1.4), rng.uniform(0.7, 1.4)
    d = [max(1, round(side * f)) for f in (a, b, 1.0 / (a * b))]
    while d[0] * d[1] * d[2] * lx ** 3 > most:
        d[d.index(max(d))] -= 1
    return d


def draw(rng):
    kind = rng.choice(["ax", "ax", "ax", "adjoint", "apply", "assemble", "pcg", "pcg", "velocity", "pressure",
                       "pressure", "gradient"])
    eps = rng.choice([0.0, 0.03, 0.05])
    if kind in ("ax", "adjoint", "apply", "assemble"):
        lx = rng.choice([4, 5, 6, 7, 8, 8, 9, 10, 10, 11, 12, 14, 16])
        dtype = rng.choice(["f64", "f64", "f32"])
        coef = "poisson" if kind in ("adjoint", "assemble") else rng.choice(["poisson", "poisson", "velocity", "variable"])
        nf = 1 if kind == "adjoint" else rng.choice([1, 1, 3])
        nx, ny, nz = _box(rng, lx, 17e6 if nf == 3 else 34e6, 13e3)
        return _case(None, kind, nx, ny, nz, lx, eps=eps, coef=coef, dtype=dtype, nf=nf)
    lx = rng.choice([5, 6, 7, 8, 8, 9, 10, 12])
    if kind == "pcg":
        nx, ny, nz = _box(rng, lx, 17e6, 13e3)
        return _case(None, kind, nx, ny, nz, lx, eps=eps, coef=rng.choice(["poisson", "velocity"]), iters=rng.randrange(40, 201))
    if kind == "velocity":
        nx, ny, nz = _box(rng, lx, 14e6, 13e3)
        return _case(None, kind, nx, ny, nz, lx, eps=eps, coef="velocity", nf=3, rtol=1e-10)
    if kind == "pressure":
        nx, ny, nz = _box(rng, lx, 17e6, 50e3)
        return _case(None, kind, nx, ny, nz, lx, eps=eps, precond=rng.choice(["schwarz", "schwarz_overlap"]),
                     restart=rng.choice([10, 20, 30]), rtol=1e-10)
    nx, ny, nz = _box(rng, lx, 4e6, 30e3)
    return _case(None, kind, nx, ny, nz, lx, eps=eps, coef="variable", rtol=1e-12)


def _points(c):
    return c["nx"] * c["ny"] * c["nz"] * c["lx"] ** 3


def _uniform(n, seed, dtype=torch.float64):
    """n draws of U[-1, 1) on the GPU."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.rand(n, generator=g, device="cuda", dtype=torch.float64).mul_(2.0).sub_(1.0).to(dtype)


def _random_field(xyz, seed, sigma=0.5, ell=0.2, modes=64):
    """h1 = exp(g), g a smooth Gaussian random field (random Fourier features) at the points xyz (3, n)."""
    r = np.random.default_rng(seed)
    omega, phi = r.normal(0.0, 1.0 / ell, (modes, 3)), r.uniform(0.0, 2.0 * math.pi, modes)
    g = torch.zeros_like(xyz[0])
    for m in range(modes):
        g += torch.cos(xyz[0] * omega[m, 0] + xyz[1] * omega[m, 1] + xyz[2] * omega[m, 2] + phi[m])
    return torch.exp(g.mul_(sigma * math.sqrt(2.0 / modes)))


def _dtype(c):
    return torch.float32 if c["dtype"] == "f32" else torch.float64


def prepare(c, seed):
    from paper_2107_01243_amd import sem

    P = sem.BoxProblem.build(c["nx"], c["lx"], c["eps"], fp32=c["dtype"] == "f32" or c["kind"] == "velocity",
                             ny=c["ny"], nz=c["nz"])
    h1, h2 = COEFS[c["coef"]]
    s = {"case": c, "P": P, "h2": h2}
    if h1 is None:
        h1 = s["h1"] = _random_field(P.xyz.view(3, -1), seed + 1)
    if c["kind"] != "gradient" and c["coef"] != "poisson":
        P.coef.set_helmholtz(h1, h2)
    u = s["u"] = _uniform(P.n * c["nf"], seed, _dtype(c))
    if c["kind"] == "ax":
        s["w"] = torch.empty_like(u)
    elif c["kind"] == "adjoint":
        s["v"] = _uniform(P.n, seed + 2, _dtype(c))
    elif c["kind"] in ("pcg", "velocity", "pressure"):
        s["b"] = P.assemble(u, c["nf"])
    elif c["kind"] == "gradient":
        s["b"], s["target"] = P.assemble(u), _uniform(P.n, seed + 2).mul_(1e-6)
    if c["kind"] == "pressure":  # a program that steps in time has the preconditioner in hand
        sem.schwarz_apply(torch.empty_like(u), s["b"], P.coef, P.msh, P.Xh, P.gs, overlap=c["precond"] == "schwarz_overlap")
    return s


def run(s):
    c, P = s["case"], s["P"]
    kind, nf = c["kind"], c["nf"]
    if kind == "ax":
        return P.ax(s["u"], nf, out=s["w"])
    if kind == "apply":
        return P.apply(s["u"], nf)
    if kind == "assemble":
        return P.assemble(s["u"], nf)
    if kind == "adjoint":
        return P.adjoint(s["u"], s["v"])
    if kind == "pcg":
        return P.solve(s["b"], rtol=0.0, max_iter=c["iters"])[0]
    if kind == "velocity":
        return P.solve(s["b"], nfields=3, rtol=c["rtol"], mixed=True)[0]
    if kind == "pressure":
        return P.gmres(s["b"], rtol=c["rtol"], restart=c["restart"], precond=c["precond"])[0]
    from paper_2107_01243_amd.autograd import HelmholtzSolve

    h1, b = s["h1"].clone().requires_grad_(True), s["b"].clone().requires_grad_(True)
    u = HelmholtzSolve.apply(h1, b, P, s["h2"], c["rtol"])
    loss = 0.5 * (u - s["target"]).square().sum()
    loss.backward()
    return {"u": u.detach(), "grad_h1": h1.grad, "grad_b": b.grad}


def work(c):
    n, nf, lx = _points(c), c["nf"], c["lx"]
    word = 4 if c["dtype"] == "f32" else 8
    # words of G, B and h1 per point, and operations per point and field, of one operator application
    geo = 6 + (c["coef"] != "poisson") + (c["coef"] == "variable")
    ax = 12 * lx + 15 + 3 * (c["coef"] != "poisson")
    kind = c["kind"]
    if kind in ("ax", "apply"):
        return {"bytes": n * word * (geo + 2 * nf), "flops": n * nf * ax}
    if kind == "adjoint":
        return {"bytes": n * word * 9, "flops": n * (12 * lx + 20)}
    shared = 1.0 - ((lx - 2) / lx) ** 3
    if kind == "assemble":
        return {"bytes": n * nf * word * 2 + 4 * n * shared, "flops": n * nf}
    # one CG step: r, dinv, p, G in and p, w out; the shared values in and out; x, p, r, dinv, w in and x, r out
    def cg(w):
        return n * ((geo + 1 + 4 * nf) * w + 2 * shared * w * nf + (1 + 6 * nf) * w)

    if kind == "pcg":
        return {"bytes": c["iters"] * cg(8), "flops": c["iters"] * n * (ax + 16)}
    if kind == "velocity":  # about 13 FP32 steps and 6 FP64 residuals
        return {"bytes": 13 * cg(4) + 6 * n * 8 * (geo + 5 * nf), "flops": n * nf * (13 * (ax + 16) + 6 * ax)}
    if kind == "pressure":  # per step an operator, a preconditioner (r in, z out, box factors) and the basis twice
        steps, box = 30, lx + 2 if c["precond"] == "schwarz_overlap" else lx
        words = 8 + 2 * shared + 2 + 3 * (box * box + box) / lx ** 3 + 2 * (c["restart"] / 2 + 2)
        return {"bytes": steps * n * 8 * words, "flops": steps * n * (ax + 12 * box ** 4 / lx ** 3 + 4 * c["restart"])}
    steps = 2 * 330  # forward and adjoint solve, about 330 steps each at lx = 8
    return {"bytes": steps * cg(8), "flops": steps * n * (ax + 16)}


# ------------------------------------------------------------------ the definitions in 64 bits
def _gll(lx):
    """Points, weights and derivative matrix D[i, l] = l_l'(xi_i) of the Lagrange basis on the GLL points."""
    N = lx - 1
    P = np.polynomial.legendre.Legendre.basis(N)
    x = np.concatenate([[-1.0], np.sort(P.deriv().roots().real) if N > 1 else [], [1.0]])
    for _ in range(3):  # Newton steps on P_N'
        x[1:-1] -= P.deriv()(x[1:-1]) / P.deriv(2)(x[1:-1]) if N > 1 else 0.0
    x = 0.5 * (x - x[::-1])
    w = 2.0 / (N * (N + 1) * P(x) ** 2)
    L = P(x)
    D = np.zeros((lx, lx))
    for i in range(lx):
        for l in range(lx):
            if i != l:
                D[i, l] = L[i] / (L[l] * (x[i] - x[l]))
    D[0, 0], D[N, N] = -N * (N + 1) / 4.0, N * (N + 1) / 4.0
    return x, w, torch.from_numpy(D).cuda()


class _Exact:
    def __init__(self, c):
        lx = self.lx = c["lx"]
        N, ne = lx - 1, (c["nx"], c["ny"], c["nz"])
        xi, w, self.D = _gll(lx)
        self.E = ne[0] * ne[1] * ne[2]
        shape = (ne[2], ne[1], ne[0], lx, lx, lx)  # element z, y, x; point k, j, i
        X, I = [], []
        for d in range(3):  # x, y, z
            sh = [1] * 6
            sh[2 - d], sh[5 - d] = ne[d], lx
            el = np.arange(ne[d])[:, None]
            co = (el + (xi[None, :] + 1.0) / 2.0) / ne[d]
            ids = el * N + np.arange(lx)[None, :]
            X.append(torch.from_numpy(co).cuda().reshape(sh).expand(shape).reshape(-1))
            I.append(torch.from_numpy(ids).cuda().reshape(sh).expand(shape).reshape(-1))
        M = [m * N + 1 for m in ne]
        self.glb, self.nglb = I[0] + M[0] * (I[1] + M[1] * I[2]), M[0] * M[1] * M[2]
        wall = torch.zeros_like(self.glb, dtype=torch.bool)
        for d in range(3):
            wall |= (I[d] == 0) | (I[d] == M[d] - 1)
        del I
        self.free = (~wall).double()
        s = [torch.sin(2.0 * math.pi * x) for x in X]
        self.xyz = torch.stack([X[0] + c["eps"] * s[1] * s[2], X[1] + c["eps"] * s[2] * s[0], X[2] + c["eps"] * s[0] * s[1]])
        del X, s
        m = [self.grad(self.xyz[q]) for q in range(3)]  # m[c][d] = d x_c / d r_d
        C = [[m[(q + 1) % 3][(d + 1) % 3] * m[(q + 2) % 3][(d + 2) % 3] - m[(q + 1) % 3][(d + 2) % 3] * m[(q + 2) % 3][(d + 1) % 3]
              for d in range(3)] for q in range(3)]
        J = sum(m[0][d] * C[0][d] for d in range(3))
        del m
        W = torch.from_numpy(w).cuda()
        rho = (W[:, None, None] * W[None, :, None] * W[None, None, :]).reshape(1, -1).expand(self.E, -1).reshape(-1)
        self.B = rho * J
        self.G = {(p, q): rho / J * sum(C[t][p] * C[t][q] for t in range(3)) for p, q in ((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))}
        self.h1, self.h2 = COEFS[c["coef"]]

    def _d(self, u, M, axis):
        """M applied along direction axis (0: i, 1: j, 2: k) of every element."""
        lx = self.lx
        if axis == 0:
            return torch.matmul(u.view(-1, lx), M.T.contiguous()).view(-1)
        return torch.matmul(M, u.view(-1, lx, lx ** axis)).reshape(-1)

    def grad(self, u):
        return [self._d(u, self.D, a) for a in range(3)]

    def flux(self, u):
        g = self.grad(u)
        return [sum(self.G[min(p, q), max(p, q)] * g[q] for q in range(3)) for p in range(3)]

    def ax(self, u):
        Dt = self.D.T.contiguous()
        w = sum(self._d(self.h1 * f, Dt, a) for a, f in enumerate(self.flux(u)))
        return w + self.h2 * self.B * u if self.h2 else w

    def gs(self, u):
        return torch.zeros(self.nglb, dtype=u.dtype, device=u.device).index_add_(0, self.glb, u)[self.glb]

    def apply(self, u):
        return self.gs(self.ax(u)) * self.free

    def solve(self, b, iters, tol=0.0):
        """Jacobi-preconditioned conjugate gradients from zero."""
        lx = self.lx
        Sq = (self.D * self.D).T.contiguous()
        dg = torch.diagonal(self.D)
        dd = [dg.view(1, *[lx if 3 - a == q else 1 for q in (1, 2, 3)]).expand(self.E, lx, lx, lx).reshape(-1) for a in range(3)]
        diag = sum(self._d(self.h1 * self.G[a, a], Sq, a) for a in range(3))
        for p, q in ((0, 1), (0, 2), (1, 2)):
            diag = diag + 2.0 * self.h1 * self.G[p, q] * dd[p] * dd[q]
        diag = self.gs(diag + self.h2 * self.B)
        mult = self.gs(torch.ones_like(b))
        dinv = self.free / diag
        x, r, p, rz = torch.zeros_like(b), b.clone(), torch.zeros_like(b), None
        b2 = torch.sum(b * b / mult)
        for k in range(iters):
            z = dinv * r
            new = torch.sum(r * z / mult)
            p = z + (new / rz) * p if rz is not None else z
            rz = new
            q = self.apply(p)
            a = rz / torch.sum(p * q / mult)
            x += a * p
            r -= a * q
            if tol and k % 10 == 9 and float(torch.sum(r * r / mult) / b2) <= tol * tol:
                break
        return x, mult


def exact(c, seed):
    kind, n, nf = c["kind"], _points(c), c["nf"]
    if kind in ("velocity", "pressure", "gradient") and n > 1.5e6 or kind == "pcg" and n * c["iters"] > 1e9:
        return None
    X = _Exact(c)
    if X.h1 is None:
        X.h1 = _random_field(X.xyz, seed + 1)
    u = _uniform(n * nf, seed, _dtype(c)).double()
    fields = u.view(nf, n)
    if kind in ("ax", "apply"):
        op = X.ax if kind == "ax" else X.apply
        return torch.cat([op(f) for f in fields])
    if kind == "assemble":
        return torch.cat([X.gs(f) * X.free for f in fields])
    if kind == "adjoint":
        v = _uniform(n, seed + 2, _dtype(c)).double()
        return sum(g * f for g, f in zip(X.grad(v), X.flux(u)))
    b = [X.gs(f) * X.free for f in fields]
    if kind == "pcg":
        return X.solve(b[0], c["iters"])[0]
    if kind in ("velocity", "pressure"):
        return torch.cat([X.solve(f, 4000, 1e-14)[0] for f in b])
    target = _uniform(n, seed + 2).mul_(1e-6)
    x, mult = X.solve(b[0], 4000, 1e-14)
    lam = X.solve(X.gs(x - target) * X.free, 4000, 1e-14)[0]
    return {"u": x, "grad_h1": -sum(g * f for g, f in zip(X.grad(lam), X.flux(x))), "grad_b": lam / mult}
