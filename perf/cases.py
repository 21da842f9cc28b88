"""What a program that uses this library has it do, as cases that can be timed.

Five kinds of work, each through the entry points of
``paper_2201_00241_amd.rh`` and on the synthetic grids of ``gridgen``:

* ``hvp``      k reduced-Hessian-vector products of one solved network;
* ``hessian``  its full dense reduced Hessian, in blocks of directions;
* ``batch``    one launch over several networks (eager, or recorded once and
               replayed);
* ``tracking`` one update of the real-time tracking loop: new loads, power
               flow and gradient on the device, Hessian, dense solve,
               projected parameters;
* ``cholesky`` a dense SPD solve on the device.

A case holds plain values; the seed given to ``prepare`` draws its loads and
directions.  ``exact`` evaluates the same results with plain torch in 64 bits
from the complex-power branch formulas and dense linear algebra.
"""
from __future__ import annotations

import functools
import math
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import torch

import gridgen
from paper_2201_00241_amd import rh


def listed():
    return [
        # the smallest call there is: the full Hessian of a textbook grid,
        # where launch and call overhead are everything
        dict(name="hessian-9bus", kind="hessian", n_bus=9, grid_seed=0, prec="fp64", k_block=5),
        # one direction, as a conjugate-gradient step asks for
        dict(name="hvp-1k-k1", kind="hvp", n_bus=1000, grid_seed=1000, k=1, prec="fp64"),
        # a block of directions in the refined FP32 mode on a small grid
        dict(name="hvp-1k-k128-refined", kind="hvp", n_bus=1000, grid_seed=1000, k=128, prec="refined"),
        # a serving request of medium size on the 10k grid
        dict(name="hvp-10k-k16", kind="hvp", n_bus=10000, grid_seed=2000, k=16, prec="fp64"),
        # the benchmark's block in the refined mode
        dict(name="hvp-10k-k256-refined", kind="hvp", n_bus=10000, grid_seed=2000, k=256, prec="refined"),
        # the headline: the full Hessian at 10k buses in k = 256 blocks
        dict(name="hessian-10k", kind="hessian", n_bus=10000, grid_seed=2000, prec="fp64", k_block=256),
        # a serving launch: requests over grids of several sizes at once
        dict(name="batch-mixed", kind="batch", sizes="1000,10000,9,1000,10000", grid_seed=1000,
             ks="128,16,5,1,128", prec="fp64", recorded=False),
        # many operating points of the largest grid, recorded and replayed
        dict(name="batch-70k", kind="batch", sizes="70000,70000,70000,70000", grid_seed=3000, ks="128,128,128,128",
             prec="fp64", recorded=True),
        # one request on the largest grid in the refined mode
        dict(name="hvp-70k-k128-refined", kind="hvp", n_bus=70000, grid_seed=3000, k=128, prec="refined"),
        # one minute of the tracking loop at the two benchmark sizes
        dict(name="tracking-1k", kind="tracking", n_bus=1000, grid_seed=1000),
        dict(name="tracking-10k", kind="tracking", n_bus=10000, grid_seed=2000),
        # the dense system of the largest network of the paper (n_p = 4,555)
        dict(name="cholesky-4555", kind="cholesky", n=4555, nrhs=1, pad=0),
    ]


def draw(rng):
    kind = rng.choice(["hvp", "hvp", "hvp", "hessian", "batch", "tracking", "cholesky"])

    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    seed = rng.randrange(1 << 20)
    prec = rng.choice(["fp64", "fp64", "refined"])
    if kind == "hvp":
        n = log_int(60, 40000)
        return dict(kind=kind, n_bus=n, grid_seed=seed, k=log_int(1, max(2, min(1024, 4_000_000 // n))), prec=prec)
    if kind == "hessian":
        n = log_int(60, 9000)
        return dict(kind=kind, n_bus=n, grid_seed=seed, prec=prec if n < 4000 else "fp64",
                    k_block=rng.choice([64, 100, 256, 512]))
    if kind == "batch":
        m = rng.randint(2, 6)
        sizes = [log_int(100, 20000) for _ in range(m)]
        ks = [log_int(1, 200) for _ in range(m)]
        return dict(kind=kind, sizes=",".join(map(str, sizes)), grid_seed=seed, ks=",".join(map(str, ks)),
                    prec=prec, recorded=rng.random() < 0.5)
    if kind == "tracking":
        return dict(kind=kind, n_bus=log_int(100, 9000), grid_seed=seed)
    return dict(kind=kind, n=log_int(30, 4500), nrhs=rng.choice([1, 1, 2, 5, 16]), pad=rng.choice([0, 0, 1, 13]))


# ---- inputs -----------------------------------------------------------------


@functools.lru_cache(maxsize=8)
def _base_grid(n_bus, grid_seed):
    """The network itself: topology, line data, generators and base loads."""
    if n_bus < 60:
        return gridgen.ring9(grid_seed)
    for name, c in gridgen.CONFIGS.items():
        if c["n_bus"] == n_bus and grid_seed == 1000 * gridgen.CONFIG_INDEX[name]:
            return gridgen.config_grid(name, 0)
    # other sizes: branch and generator ratios of the configurations, loaded
    # lightly enough (about half the limit) that every topology is solvable
    alpha = min(0.15, 0.12 * (10000 / n_bus) ** 0.85)
    n_gen = max(3, n_bus // 10 if n_bus <= 15000 else n_bus // 14)
    return gridgen.geometric(n_bus, int(1.35 * n_bus), n_gen, grid_seed, alpha, kappa=0.085 * alpha)


def _loaded(case_n, grid_seed, seed, frac):
    return gridgen.perturb_loads(_base_grid(case_n, grid_seed), seed, frac)


def _seed(*parts):
    return np.random.default_rng([int(p) for p in parts])


def _directions(n_p, k, seed, i=0):
    """A (k, n_p) block of Gaussian directions, row j = direction j."""
    return _seed(seed, 7, i).standard_normal((k, n_p))


def _sizes(case):
    return [int(v) for v in case["sizes"].split(",")], [int(v) for v in case["ks"].split(",")]


def _batch_grids(case, seed):
    sizes, _ = _sizes(case)
    out = []
    for i, n in enumerate(sizes):
        # grids of a configuration's size are that configuration's
        own = {1000: 1000, 10000: 2000, 70000: 3000, 9: 0}.get(n, case["grid_seed"] + n)
        out.append(_loaded(n, own, seed * 64 + i, 0.1))
    return out


def _tracking_inputs(case, seed):
    base = _base_grid(case["n_bus"], case["grid_seed"])
    now = gridgen.perturb_loads(base, seed, 0.02)
    n_pv = base.n_gen - 1
    vg = np.zeros(base.n_bus)
    vg[base.gen_bus] = base.Vg
    pg = np.zeros(base.n_bus)
    pg[base.gen_bus] = base.Pg
    pv = np.flatnonzero(base.bus_type == gridgen.PV)
    p = np.concatenate([pg[pv], [vg[base.ref_bus]], vg[pv]])
    lo = np.concatenate([np.zeros(n_pv), np.full(n_pv + 1, 0.94)])
    hi = np.concatenate([2.0 * np.maximum(pg[pv], 0.1), np.full(n_pv + 1, 1.06)])
    ramp = np.concatenate([np.full(n_pv, 0.01), np.full(n_pv + 1, 0.002)])
    return base, now, p, lo, hi, ramp


def _spd(case, seed, dev):
    """A reduced Hessian's like: a strong diagonal and smooth low-rank coupling."""
    n = case["n"]
    r = _seed(seed, 11)
    d = r.uniform(1.0, 4.0, n)
    U = r.standard_normal((n, 24)) / math.sqrt(24)
    b = r.standard_normal((case["nrhs"], n))
    U = torch.from_numpy(U).to(dev)
    A = U @ U.T
    A = (A + A.T) * 0.5
    A.diagonal().add_(torch.from_numpy(d).to(dev))
    return A, torch.from_numpy(b).to(dev)


class _State:
    pass


def _prec(case):
    return rh.RH_FP64 if case["prec"] == "fp64" else rh.RH_FP32_REFINED


def _solved(ctx, grid):
    net = rh.Network(ctx, grid)
    net.solve()
    return net


def prepare(case, seed):
    s = _State()
    s.case = case
    s.ctx = rh.Context(0)
    kind = case["kind"]
    if kind in ("hvp", "hessian"):
        s.net = _solved(s.ctx, _loaded(case["n_bus"], case["grid_seed"], seed, 0.1))
        n_p = s.net.n_p
        if kind == "hvp":
            s.W = torch.from_numpy(_directions(n_p, case["k"], seed)).cuda()
            s.out = torch.zeros_like(s.W)
        else:
            s.out = torch.zeros((n_p, n_p), dtype=torch.float64, device="cuda")
    elif kind == "batch":
        _, ks = _sizes(case)
        # distinct networks may be set up from different threads
        with ThreadPoolExecutor(4) as pool:
            s.nets = list(pool.map(lambda g: _solved(s.ctx, g), _batch_grids(case, seed)))
        s.W = [torch.from_numpy(_directions(n.n_p, k, seed, i)).cuda() for i, (n, k) in enumerate(zip(s.nets, ks))]
        s.out = [torch.zeros_like(w) for w in s.W]
        torch.cuda.synchronize()
        if case["recorded"]:
            s.batch = s.ctx.batch(s.nets, s.W, s.out, prec=_prec(case))
    elif kind == "tracking":
        base, now, s.p, s.lo, s.hi, s.ramp = _tracking_inputs(case, seed)
        s.Pd, s.Qd = now.Pd, now.Qd
        s.net = rh.Network(s.ctx, base)
        s.net.solve_device()
        s.x_prev = s.net.state()  # the operating point of the minute before
        s.grad = torch.zeros(s.net.n_p, dtype=torch.float64, device="cuda")
        s.d = torch.zeros_like(s.grad)
    else:
        s.A0, s.B0 = _spd(case, seed, "cuda")
        n, ld = case["n"], case["n"] + case["pad"]
        s.A = torch.zeros((n, ld), dtype=torch.float64, device="cuda")
        s.B = torch.zeros((case["nrhs"], ld), dtype=torch.float64, device="cuda")
    return s


def run(s):
    case, kind = s.case, s.case["kind"]
    stream = torch.cuda.current_stream().cuda_stream
    if kind == "hvp":
        s.net.hvp_device(s.W, s.out, stream=stream, prec=_prec(case))
        return s.out
    if kind == "hessian":
        s.net.reduced_hessian_device(s.out, k_block=case["k_block"], stream=stream, prec=_prec(case))
        return s.out
    if kind == "batch":
        if case["recorded"]:
            s.batch.launch(stream)
        else:
            s.ctx.hvp_batch_device(s.nets, s.W, s.out, stream=stream, prec=_prec(case))
        return s.out
    if kind == "tracking":
        net = s.net
        net.set_parameters(s.p)
        net.set_initial_state(s.x_prev)
        net.set_loads(s.Pd, s.Qd)
        net.solve_device()
        x = net.state()
        net.reduced_gradient_device(s.grad, stream=stream)
        net.tracking_step_device(k_block=256, lo=s.lo, hi=s.hi, ramp=s.ramp, d=s.d, stream=stream)
        return {"x": x, "grad": s.grad, "d": s.d, "p": net.get_parameters()}
    n = case["n"]
    s.A[:, :n].copy_(s.A0)  # the factorisation works in place
    s.B[:, :n].copy_(s.B0)
    s.ctx.cholesky_solve_device(s.A, s.B, stream=stream)
    return {"L": s.A, "X": s.B}


# ---- the work a pass cannot do without --------------------------------------


def _dims(n_bus):
    if n_bus < 60:
        return 14, 5
    for c in gridgen.CONFIGS.values():
        if c["n_bus"] == n_bus:
            return 2 * n_bus - 1 - c["n_gen"], 2 * c["n_gen"] - 1
    n_gen = max(3, n_bus // 10 if n_bus <= 15000 else n_bus // 14)
    return 2 * n_bus - 1 - n_gen, 2 * n_gen - 1


def _hvp_work(n_bus, k, reads_w=True):
    """The factors (about 16 entries of L and U per state, value and column),
    the branch coefficients (2.7 incidences of 6 values per bus) and G_p once;
    every direction read and every product written once.  Two solves of 2
    operations per factor entry, and 14 per incidence, for each direction."""
    n_x, n_p = _dims(n_bus)
    data = 12 * 16 * n_x + 48 * 2.7 * n_bus + 12 * 8 * n_p
    return data + 8 * k * n_p * (2 if reads_w else 1), k * (64 * n_x + 38 * n_bus + 32 * n_p)


def work(case):
    kind = case["kind"]
    if kind == "hvp":
        b, f = _hvp_work(case["n_bus"], case["k"])
    elif kind == "hessian":
        b, f = _hvp_work(case["n_bus"], _dims(case["n_bus"])[1], reads_w=False)
    elif kind == "batch":
        parts = [_hvp_work(n, k) for n, k in zip(*_sizes(case))]
        b, f = sum(p[0] for p in parts), sum(p[1] for p in parts)
    elif kind == "tracking":
        # four Newton steps (the factorisation about 20 operations per factor
        # entry), the full Hessian, and its Cholesky factor
        n_x, n_p = _dims(case["n_bus"])
        b, f = _hvp_work(case["n_bus"], n_p, reads_w=False)
        b += 4 * 2 * 8 * 16 * n_x + 8 * n_p * n_p
        f += 4 * 20 * 16 * n_x + n_p ** 3 / 3
    else:
        n, q = case["n"], case["nrhs"]
        b, f = 8 * n * n + 16 * n * q, n ** 3 / 3 + 2.0 * n * n * q  # each triangle once, B twice
    return {"bytes": b, "flops": f}


# ---- the same results in plain 64-bit torch ---------------------------------


class _Exact:
    """One operating point with dense G_x: g, f and their derivatives from the
    branch flows as functions of the angles and magnitudes at both ends."""

    def __init__(self, g, dev, p=None):
        t = lambda a: torch.as_tensor(np.asarray(a), device=dev)  # noqa: E731
        n = self.n = g.n_bus
        y = 1.0 / (g.br_r + 1j * g.br_x)
        self.par = torch.stack([t(y.real.copy()), t(y.imag.copy()), t(0.5 * g.br_b)], 1)
        f, o = t(g.br_from.astype(np.int64)), t(g.br_to.astype(np.int64))
        self.var = torch.stack([f, o, n + f, n + o], 1)  # (theta_f, theta_t, v_f, v_t) in z
        self.inj = torch.stack([f, n + f, o, n + o], 1)  # (P_f, Q_f, P_t, Q_t) in the injections
        bt = np.asarray(g.bus_type)
        pv, pq = np.flatnonzero(bt == gridgen.PV), np.flatnonzero(bt == gridgen.PQ)
        ref = g.ref_bus
        self.ref, self.n_pv = ref, pv.size
        self.xi = t(np.concatenate([pv, pq, n + pq]))  # place of x in z, and of g's rows in the injections
        self.vi = t(np.concatenate([[n + ref], n + pv]))  # place of the voltage parameters in z
        gi = np.full(n, -1)
        gi[g.gen_bus] = np.arange(g.n_gen)
        self.c2, self.c1 = t(g.c2[gi[pv]]), t(g.c1[gi[pv]])
        self.c2r, self.c1r = float(g.c2[gi[ref]]), float(g.c1[gi[ref]])
        self.load = torch.cat([t(g.Pd), t(g.Qd)])
        self.p = t(np.concatenate([g.Pg[gi[pv]], [g.Vg[gi[ref]]], g.Vg[gi[pv]]]) if p is None else p)
        v0 = np.ones(n) if g.v0 is None else g.v0
        z = torch.zeros(2 * n, dtype=torch.float64, device=dev)
        z[n:] = t(v0)
        z[self.vi] = self.p[self.n_pv:]
        for _ in range(20):
            r = self.mismatch(z)
            if float(r.abs().max()) <= 2e-14 * n ** 0.5:
                break
            z[self.xi] -= torch.linalg.solve(self.gx(z), r)
        self.z = z
        self.lu = torch.linalg.lu_factor(self.gx(z))
        J = self.jac(z)
        e = torch.zeros((2 * n, 1), dtype=torch.float64, device=dev)
        e[ref] = 1.0
        self.dPref = self.jt(J, e)[:, 0]
        slope = 2.0 * self.c2r * float(self.inject(z)[ref] + self.load[ref]) + self.c1r
        self.lam = -self.solve(slope * self.dPref[self.xi][:, None], True)
        mu = torch.zeros(2 * n, dtype=torch.float64, device=dev)
        mu[self.xi] = self.lam[:, 0]
        mu[ref] = slope
        hess = torch.func.hessian(lambda zb, par, m: (self.flows(zb, par) * m).sum())
        self.H = torch.func.vmap(hess)(z[self.var], self.par, mu[self.inj])
        self.J = J
        self.slope = slope

    @staticmethod
    def flows(zb, par):
        thf, tht, vf, vt = zb.unbind(-1)
        g, b, h = par.unbind(-1)
        c, s, k = torch.cos(thf - tht), torch.sin(thf - tht), vf * vt
        return torch.stack([g * vf * vf - k * (g * c + b * s), -(b + h) * vf * vf - k * (g * s - b * c),
                            g * vt * vt - k * (g * c - b * s), -(b + h) * vt * vt + k * (g * s + b * c)], -1)

    def inject(self, z):
        out = torch.zeros(2 * self.n, dtype=torch.float64, device=z.device)
        return out.index_add_(0, self.inj.reshape(-1), self.flows(z[self.var], self.par).reshape(-1))

    def mismatch(self, z):
        r = (self.inject(z) + self.load)[self.xi]
        r[:self.n_pv] -= self.p[:self.n_pv]
        return r

    def jac(self, z):
        return torch.func.vmap(torch.func.jacfwd(self.flows))(z[self.var], self.par)

    def gx(self, z):
        J, n = self.jac(z), self.n
        at = torch.full((2 * n,), -1, dtype=torch.int64, device=z.device)
        at[self.xi] = torch.arange(self.xi.numel(), device=z.device)
        r, c = at[self.inj][:, :, None].expand(-1, 4, 4), at[self.var][:, None, :].expand(-1, 4, 4)
        ok = (r >= 0) & (c >= 0)
        G = torch.zeros((self.xi.numel(),) * 2, dtype=torch.float64, device=z.device)
        return G.index_put_((r[ok], c[ok]), J[ok], accumulate=True)

    def scatter(self, to, v):
        """Per-branch (m, 4, k) values summed into 2n rows."""
        out = torch.zeros((2 * self.n, v.shape[-1]), dtype=torch.float64, device=v.device)
        return out.index_add_(0, to.reshape(-1), v.reshape(-1, v.shape[-1]))

    def jz(self, dz):
        return self.scatter(self.inj, self.J @ dz[self.var])

    def jt(self, J, y):
        return self.scatter(self.var, J.transpose(1, 2) @ y[self.inj])

    def solve(self, b, transposed=False):
        lu, piv = self.lu
        # a few columns at a time: the triangular solves' workspace grows with them
        return torch.cat([torch.linalg.lu_solve(lu, piv, c.contiguous(), adjoint=transposed)
                          for c in b.split(256, dim=1)], 1)

    def gpt(self, psi):
        """G_p^T psi for the rows psi of g."""
        y = torch.zeros((2 * self.n, psi.shape[1]), dtype=torch.float64, device=psi.device)
        y[self.xi] = psi
        return torch.cat([-psi[:self.n_pv], self.jt(self.J, y)[self.vi]])

    def gradient(self):
        pg = self.p[:self.n_pv]
        f = torch.cat([2.0 * self.c2 * pg + self.c1, self.slope * self.dPref[self.vi]])
        return f + self.gpt(self.lam)[:, 0]

    def hvp(self, W):
        """(n_p, k) directions to (n_p, k) products."""
        dz = torch.zeros((2 * self.n, W.shape[1]), dtype=torch.float64, device=W.device)
        dz[self.vi] = W[self.n_pv:]
        b = self.jz(dz)[self.xi]
        b[:self.n_pv] -= W[:self.n_pv]
        dz[self.xi] = -self.solve(b)
        y = self.scatter(self.var, self.H @ dz[self.var])
        y += 2.0 * self.c2r * self.dPref[:, None] * (self.dPref @ dz)[None, :]
        psi = -self.solve(y[self.xi], True)
        yp = torch.cat([2.0 * self.c2[:, None] * W[:self.n_pv], y[self.vi]])
        return yp + self.gpt(psi)


def _step(H, g):
    """(H + tau I) d = -g with the smallest tau of the library's sequence."""
    diag = H.diagonal()
    beta = 1e-3 * float(diag.abs().max()) or 1e-3
    tau = 0.0 if float(diag.min()) > 0.0 else -float(diag.min()) + beta
    eye = torch.eye(H.shape[0], dtype=H.dtype, device=H.device)
    while True:
        L, info = torch.linalg.cholesky_ex(H + tau * eye)
        if int(info) == 0:
            return torch.cholesky_solve(-g[:, None], L)[:, 0]
        tau = max(2.0 * tau, beta)


# dense factorisations beyond this many states take too long
_MOST_STATES = 20000


def exact(case, seed):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    kind = case["kind"]
    if kind == "cholesky":
        A, B = _spd(case, seed, dev)
        n, ld = case["n"], case["n"] + case["pad"]
        L = torch.linalg.cholesky(A)
        full = torch.zeros((n, ld), dtype=torch.float64, device=dev)
        # row j of the buffer is column j of the matrix: L^T on and above the
        # diagonal, the input left as it was below it
        full[:, :n] = torch.triu(L.T) + torch.tril(A, -1)
        X = torch.zeros((case["nrhs"], ld), dtype=torch.float64, device=dev)
        X[:, :n] = torch.cholesky_solve(B.T, L).T
        return {"L": full, "X": X}
    if kind == "batch":
        sizes, ks = _sizes(case)
        sizes_ok = [_dims(n)[0] <= 6000 for n in sizes]  # several instances: the smaller ones
        if not any(sizes_ok):
            return None
        out = []
        for i, (g, k, ok) in enumerate(zip(_batch_grids(case, seed), ks, sizes_ok)):
            W = torch.from_numpy(_directions(g.n_p, k, seed, i)).to(dev)
            out.append(_Exact(g, dev).hvp(W.T).T.contiguous() if ok else None)
        return out
    if _dims(case["n_bus"])[0] > _MOST_STATES:
        return None
    if kind == "tracking":
        _, now, p, lo, hi, ramp = _tracking_inputs(case, seed)
        e = _Exact(now, dev, p)
        g = e.gradient()
        d = _step(e.hvp(torch.eye(p.size, dtype=torch.float64, device=dev)), g)
        pn = p + d.cpu().numpy()
        pn = np.minimum(np.maximum(pn, p - ramp), p + ramp)
        return {"x": e.z[e.xi].cpu(), "grad": g, "d": d, "p": np.minimum(np.maximum(pn, lo), hi)}
    g = _loaded(case["n_bus"], case["grid_seed"], seed, 0.1)
    e = _Exact(g, dev)
    if kind == "hvp":
        return e.hvp(torch.from_numpy(_directions(g.n_p, case["k"], seed)).to(dev).T).T.contiguous()
    return e.hvp(torch.eye(g.n_p, dtype=torch.float64, device=dev)).T.contiguous()
