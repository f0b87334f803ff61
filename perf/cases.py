"""Performance cases: the work a program has this framework do, through its public entry points.

A case names a kind of call and its sizes; ``prepare`` makes what the program
holds before the call (seeded inputs, workspaces, contexts), ``run`` makes one
pass, ``exact`` evaluates the same pass in 64 bits with plain torch and numpy,
and ``work`` states the bytes and operations the pass cannot do without.

Kinds:

* ``dyson``    Green's function with the filling found by bisection, then both bubbles
* ``remap``    kernel functions of the reducible vertices, then the channel remap
* ``sigma``    the regulated Schwinger-Dyson self-energy
* ``bse``      the Bethe-Salpeter equation of one channel for every transfer
* ``iterate``  a context continued from a saved state: one whole parquet iteration
* ``solve``    a context started from the bare vertex and iterated (parameter scans)
* ``batch``    rounds of the batched solver over many instances of one box
* ``mlp``      one training step of the warm-start network
"""
import math

import numpy as np
import torch

from paper_1510_03330_amd.ops import Batch, Solver, Stage
from paper_1510_03330_amd.warmstart import MLP
from workloads import ModelParams

DEV = "cuda:0"
SIGN = (1.0, 1.0, -1.0, 1.0)          # channels d, m, s, t


def listed():
    box44 = dict(Lx=4, Ly=4, f=2, level=2)
    box88 = dict(Lx=8, Ly=8, f=2, level=2)
    return [
        # the smallest stage calls: launch latency and serial chains (the 4x4 instances of a parameter scan)
        dict(name="dyson_4x4_nv8", kind="dyson", Nv=8, prec="fp64", **box44),
        # self-energy of a small complex128 box (the 4x4 training solves of the warm start run it every iteration)
        dict(name="sigma_4x4_nv16_fp64", kind="sigma", Nv=16, prec="fp64", **box44),
        # one step of the 3000 that train the 4x4 warm-start network (144 solutions, three fields)
        dict(name="mlp_4x4_step", kind="mlp", inputs=4, hidden=512, layers=3, out=432, batch=64),
        # the momentum-independent problem, Nv = 32, from the bare vertex
        dict(name="solve_local_nv32_fp64", kind="solve", Lx=1, Ly=1, Nv=32, f=2, level=2, prec="fp64", iters=8),
        # an ordinary lattice: 4x4, Nv = 16, complex64 (n = 256, 240 blocks per channel)
        dict(name="iterate_4x4_nv16_fp32", kind="iterate", Nv=16, prec="fp32", **box44),
        # the batched solver: eight 4x4, Nv = 8 instances, four rounds between readouts
        dict(name="batch_4x4_nv8_fp64", kind="batch", Nv=8, prec="fp64", count=8, rounds=4, **box44),
        # a whole iteration of an 8x8 lattice on the headline path
        dict(name="iterate_8x8_nv8_bf16x3", kind="iterate", Nv=8, prec="bf16x3", **box88),
        # odd lattice, complex128: nothing is a power of two
        dict(name="remap_5x7_nv10_fp64", kind="remap", Lx=5, Ly=7, Nv=10, f=2, level=2, prec="fp64"),
        # the benchmark's full size, stage by stage
        dict(name="remap_8x8_nv16_fp32", kind="remap", Nv=16, prec="fp32", **box88),
        dict(name="bse_8x8_nv16_bf16x3", kind="bse", Nv=16, prec="bf16x3", channel=1, **box88),
        # the largest box of the batched workload (n = 512, 496 blocks), FP32 products
        dict(name="bse_4x4_nv32_fp32", kind="bse", Nv=32, prec="fp32", channel=2, **box44),
        # complex128 with a ragged last panel (n = 336)
        dict(name="bse_6x4_nv14_fp64", kind="bse", Lx=6, Ly=4, Nv=14, f=2, level=2, prec="fp64", channel=0),
    ]


def _sizes(c):
    nk = c["Lx"] * c["Ly"]
    n, nq = nk * c["Nv"], nk * (c["Nv"] - 1)
    el = 16 if c["prec"] == "fp64" else 8
    return nk, n, nq, el


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["dyson", "remap", "sigma", "bse", "bse", "iterate", "solve", "batch", "mlp"])
    if kind == "mlp":
        out = 3 * _log_int(rng, 8, 200)                      # three fields, 8 .. 200 solutions
        return dict(kind=kind, inputs=rng.randint(1, 4), hidden=_log_int(rng, 64, 512), layers=rng.randint(2, 3),
                    out=out, batch=min(64, out // 3))
    prec = rng.choice(["fp64", "fp32", "bf16x3"])
    lim = dict(remap=4.1e9, sigma=4.1e9, iterate=4.8e8, batch=3e7, dyson=1e12, bse=1.1e9, solve=6e6)[kind]
    if kind == "solve":
        prec, lattices, nvs = "fp64", [(1, 1), (1, 1), (2, 2), (1, 2)], (8, 32)
    elif kind == "batch":
        prec, lattices, nvs = "fp64", [(2, 2), (2, 3), (3, 3), (4, 4)], (4, 10)
    else:
        lattices, nvs = [(2, 2), (3, 3), (2, 5), (4, 4), (4, 5), (6, 4), (5, 7), (6, 6), (8, 4), (7, 7), (8, 8)], (4, 32)
    if kind == "dyson":
        prec = "fp64"
    while True:
        lx, ly = rng.choice(lattices)
        nv = 2 * _log_int(rng, nvs[0] / 2, nvs[1] / 2)
        c = dict(kind=kind, Lx=lx, Ly=ly, Nv=nv, f=rng.choice([2, 2, 2, 1, 3]), level=rng.choice([2, 2, 2, 1]),
                 prec=prec)
        nk, n, nq, el = _sizes(c)
        vol = nq * n * n * (1 if kind == "bse" else 4) * el / 8
        if kind == "bse":                                    # complex128 products cost about three times as much
            vol *= 3.0 if prec == "fp64" else (1.5 if prec == "fp32" else 1.0)
            vol *= n / 1024
        if kind == "iterate":
            vol *= max(1.0, n / 512)
        if kind == "batch":
            c.update(count=_log_int(rng, 2, 16), rounds=4)
            vol *= c["count"]
        if kind == "solve":
            c["iters"] = rng.randint(4, 8)
        if kind == "bse":
            c["channel"] = rng.randint(0, 3)
        if n <= 1024 and vol <= lim:
            return c


# ------------------------------------------------------------------ inputs
def _params(c, seed, i=0):
    """Model parameters of instance i: moderate coupling, so that the iteration contracts and no block of the
    first Bethe-Salpeter equations (bare vertex, small self-energy) lies near its instability."""
    r = np.random.default_rng([int(seed), 7, i])
    kw = dict(Lx=c["Lx"], Ly=c["Ly"], Nv=c["Nv"], f_ext=c["f"], kernel_level=c["level"])
    if c["Lx"] * c["Ly"] == 1:
        return ModelParams(U=float(r.uniform(0.6, 1.0)), beta=float(r.uniform(3.0, 5.0)), D=2.0, **kw)
    if c["kind"] in ("solve", "batch"):
        return ModelParams(U=float(r.uniform(0.5, 1.2)), beta=float(r.uniform(2.0, 3.0)),
                           filling=float(r.uniform(0.85, 0.98)), mu_mode=1, **kw)
    return ModelParams(U=float(r.uniform(0.9, 1.2)), beta=float(r.uniform(3.0, 4.0)), tp=float(r.uniform(-0.25, -0.15)),
                       filling=float(r.uniform(0.85, 0.95)), mu_mode=1, **kw)


def _sigma(p, seed):
    """A self-energy with the analytic structure of one: a pole per momentum, Sigma(-nu) = conj Sigma(nu)."""
    g = torch.Generator(device=DEV).manual_seed(int(seed) * 4 + 1)
    nk, nve = p.Nk, p.f_ext * p.Nv
    a = 0.1 + 0.3 * torch.rand(nk, generator=g, device=DEV, dtype=torch.float64)
    b = torch.rand(nk, generator=g, device=DEV, dtype=torch.float64) - 0.5
    nu = (2 * torch.arange(-nve // 2, nve // 2, device=DEV, dtype=torch.float64) + 1) * math.pi / p.beta
    return (a[None, :] / (1j * nu[:, None] - b[None, :])).contiguous()


def _envelope(p):
    nu = torch.arange(p.Nk * p.Nv, device=DEV) // p.Nk - p.Nv // 2 + 0.5
    return 1.0 / (1.0 + nu.abs() / 4.0)


def _vertex(p, dtype, seed, channels, scale, offset=None):
    """Seeded complex normal vertices [channels][Nq][n][n], decaying with both fermionic frequencies."""
    n, nq = p.Nk * p.Nv, p.Nk * (p.Nv - 1)
    g = torch.Generator(device=DEV).manual_seed(int(seed) * 4 + 2)
    out = torch.empty((channels, nq, n, n), dtype=dtype, device=DEV)
    e = _envelope(p).to(torch.float32)
    env = scale * e[:, None] * e[None, :]
    for r in range(channels):
        for q0 in range(0, nq, 64):
            q1 = min(nq, q0 + 64)
            z = torch.randn((q1 - q0, n, n), generator=g, device=DEV, dtype=torch.complex64) * env
            out[r, q0:q1] = z if offset is None else z + offset[r]
    return out


def _lam(p):
    return (p.U, -p.U, 2.0 * p.U, 0.0)


def _phi(p, dtype, seed, channels=(0, 1, 2, 3), mean=0.3):
    """Reducible vertices as an iteration meets them: a part that does not decay (the first-level kernel) of the
    sign and order of the bare vertex, and a decaying rest."""
    return _vertex(p, dtype, seed, len(channels), 0.3, [mean * _lam(p)[r] for r in channels])


def _green(st, p, seed):
    g = torch.empty(st.g_shape, dtype=torch.complex128, device=DEV)
    mu = torch.empty(1, dtype=torch.float64, device=DEV)
    st.dyson_update(_sigma(p, seed), g, mu)
    return g, mu


def prepare(c, seed):
    if c["kind"] == "mlp":
        net = MLP([c["inputs"], *[c["hidden"]] * c["layers"], c["out"]], DEV, seed=int(seed))
        g = torch.Generator(device=DEV).manual_seed(int(seed))
        x = 2.0 * torch.rand((c["batch"], c["inputs"]), generator=g, device=DEV) - 1.0
        t = torch.randn((c["batch"], c["out"]), generator=g, device=DEV)
        return dict(c=c, net=net, x=x, t=t)
    p = _params(c, seed)
    s = dict(c=c, p=p)
    kind = c["kind"]
    if kind == "batch":
        s["b"] = Batch([_params(c, seed, i) for i in range(c["count"])], c["prec"])
        return s
    if kind == "solve":
        s["solver"] = Solver(p, c["prec"])
        return s
    if kind == "iterate":
        s["solver"] = Solver(p, c["prec"])
        s["sigma"] = _sigma(p, seed)
        s["phi"] = _phi(p, s["solver"].stage.vdtype, seed)
        return s
    st = s["st"] = Stage(p, c["prec"])
    c128 = dict(dtype=torch.complex128, device=DEV)
    if kind == "dyson":
        s["sigma"] = _sigma(p, seed)
        s["out"] = (torch.empty(st.g_shape, **c128), torch.empty(1, dtype=torch.float64, device=DEV),
                    torch.empty(st.x_shape, **c128), torch.empty(st.x_shape, **c128))
        return s
    s["k1"], s["k2"] = torch.empty(st.k1_shape, **c128), torch.empty(st.k2_shape, **c128)
    if kind == "bse":
        g, _ = _green(st, p, seed)
        x = (torch.empty(st.x_shape, **c128), torch.empty(st.x_shape, **c128))
        st.bubble_build(g, *x)
        s["chi"] = x[0 if c["channel"] < 2 else 1]
        s["gamma"] = _vertex(p, st.vdtype, seed, 1, 0.5, [_lam(p)[c["channel"]]])[0]
        s["phi"] = _phi(p, st.vdtype, seed + 1, (c["channel"],), 1.0)[0]
        s["ws"] = torch.empty(st.bse_workspace_bytes(), dtype=torch.uint8, device=DEV)
        s["stats"] = torch.empty((st.d.Nq, 4), dtype=torch.int32, device=DEV)
        return s
    s["phi"] = _phi(p, st.vdtype, seed)
    if kind == "remap":
        s["gamma"] = torch.empty_like(s["phi"])
    else:
        s["g"], s["mu"] = _green(st, p, seed)
        st.kernel_extract(s["phi"], s["k1"], s["k2"])
        s["sigma"] = torch.empty(st.sigma_shape, **c128)
        s["ws"] = torch.empty(st.sigma_workspace_bytes(), dtype=torch.uint8, device=DEV)
    return s


# --------------------------------------------------------------------- run
def run(s):
    c = s["c"]
    kind = c["kind"]
    if kind == "dyson":
        g, mu, xph, xpp = s["out"]
        s["st"].dyson_update(s["sigma"], g, mu)
        s["st"].bubble_build(g, xph, xpp)
        return dict(g=g, mu=mu, xph=xph, xpp=xpp)
    if kind == "remap":
        s["st"].kernel_extract(s["phi"], s["k1"], s["k2"])
        s["st"].channel_remap(_lam(s["p"]), s["phi"], s["k1"], s["k2"], s["gamma"])
        return dict(k1=s["k1"], k2=s["k2"], gamma=list(s["gamma"]))
    if kind == "sigma":
        s["st"].sigma_sde(s["phi"], s["k1"], s["k2"], s["g"], s["mu"], s["sigma"], ws=s["ws"])
        return dict(sigma=s["sigma"])
    if kind == "bse":
        s["st"].bse_solve(c["channel"], s["gamma"], s["chi"], s["phi"], alpha=0.5, stats=s["stats"], ws=s["ws"])
        return dict(phi=s["phi"], flags=s["stats"][:, 2])
    if kind == "iterate":
        v = s["solver"]
        v.set("phi", s["phi"])
        v.set("sigma", s["sigma"])
        v.iterate(1)
        return dict(sigma=v.get("sigma"), phi=list(v.get("phi")))
    if kind == "solve":
        v = s["solver"]
        v.reinit()
        v.iterate(c["iters"])
        return dict(sigma=v.get("sigma"), phi=v.get("phi"))
    if kind == "batch":
        s["b"].iterate(c["rounds"], tol=0.0)
        s["b"].status()
        return [dict(sigma=s["b"].get(i, "sigma"), k2=s["b"].get(i, "k2")) for i in range(c["count"])]
    net = s["net"]
    acts, _ = net.forward(s["x"])
    loss = net.backward(s["x"], acts, s["t"])
    net.adam(1e-3)
    return dict(acts=acts, loss=loss, grad=net.g, p=net.p, m=net.m, v=net.v)


def work(c):
    if c["kind"] == "mlp":
        w = [c["inputs"], *[c["hidden"]] * c["layers"], c["out"]]
        cnt = sum(w[i + 1] * (w[i] + 1) for i in range(len(w) - 1))
        mm = sum(w[i + 1] * w[i] for i in range(len(w) - 1))
        # parameters, moments and gradient in and out, bf16 weights, activations
        return dict(bytes=4 * cnt * 7 + 2 * cnt * 2 + 8 * c["batch"] * sum(w), flops=6.0 * c["batch"] * mm)
    nk, n, nq, el = _sizes(c)
    vol = float(nq) * n * n
    ng, nve = 2 * c["f"] * c["Nv"], c["f"] * c["Nv"]
    dyson = dict(bytes=16.0 * nk * (nve + ng) + 32.0 * nq * n, flops=50 * 10.0 * ng * nk + 16.0 * nq * n)
    remap = dict(bytes=8 * vol * el + 64.0 * nq * n, flops=64 * vol)
    sigma = dict(bytes=4 * vol * el + 64.0 * nq * n, flops=46 * vol)
    bse = dict(bytes=3 * vol * el, flops=32.0 / 3.0 * vol * n)
    one = {"dyson": [dyson], "remap": [remap], "sigma": [sigma], "bse": [bse]}.get(
        c["kind"], [dyson, remap, sigma, bse, bse, bse, bse])
    times = {"solve": c.get("iters", 1), "batch": c.get("rounds", 1) * c.get("count", 1)}.get(c["kind"], 1)
    return {k: times * sum(o[k] for o in one) for k in ("bytes", "flops")}


# ------------------------------------------------------- the same in 64 bits
class _Ref:
    """The parquet equations of one box with plain torch operations in complex128."""

    def __init__(self, p):
        self.p = p
        self.nk, self.nv, self.nw = p.Nk, p.Nv, p.Nv - 1
        self.n, self.nq = p.Nk * p.Nv, p.Nk * (p.Nv - 1)
        self.nve, self.ng = p.f_ext * p.Nv, 2 * p.f_ext * p.Nv
        k = torch.arange(self.nk, device=DEV)
        self.kx, self.ky = k // p.Ly, k % p.Ly
        self.row_n = torch.arange(self.n, device=DEV) // self.nk - self.nv // 2      # frequency of a box index
        self.row_K = torch.arange(self.n, device=DEV) % self.nk
        cx, cy = torch.cos(2 * math.pi * self.kx.double() / p.Lx), torch.cos(2 * math.pi * self.ky.double() / p.Ly)
        self.eps = -2 * p.t * (cx + cy) - 4 * p.tp * cx * cy

    def add(self, a, b, sb=1):
        p = self.p
        return (a // p.Ly + sb * (b // p.Ly)) % p.Lx * p.Ly + (a % p.Ly + sb * (b % p.Ly)) % p.Ly

    def nu(self, count):
        return (2 * torch.arange(-(count // 2), count // 2, device=DEV, dtype=torch.float64) + 1) * math.pi / self.p.beta

    def dyson(self, sigma):
        p = self.p
        sg = torch.zeros((self.ng, self.nk), dtype=torch.complex128, device=DEV)
        sg[self.ng // 2 - self.nve // 2:self.ng // 2 + self.nve // 2] = sigma
        nu = self.nu(self.ng)[:, None]
        if self.nk == 1:
            g0 = (2 / p.D ** 2) * 1j * (nu - torch.sign(nu) * torch.sqrt(nu * nu + p.D ** 2))
            return 1 / (1 / g0 - sg), 0.0
        mu = p.mu_fixed
        if p.mu_mode == 1:
            sn, nun, en = sg.cpu().numpy(), nu.cpu().numpy(), self.eps.cpu().numpy()
            pos = nun[self.ng // 2:, 0]
            lo, hi = en.min() - 10 - abs(p.U), en.max() + 10 + abs(p.U)
            while hi - lo >= 1e-14:
                mu = 0.5 * (lo + hi)
                if mu in (lo, hi):
                    break
                g = 1 / (1j * nun + mu - en - sn)
                x = en - mu
                part = (1 / (pos[:, None] ** 2 + x * x)).sum(0)
                safe = np.where(x == 0, 1.0, x)
                full = np.where(x == 0, p.beta ** 2 / 8, p.beta * np.tanh(p.beta * x / 2) / (4 * safe))
                dens = 0.5 + (g.real.sum() + 2 * (-x * (full - part)).sum()) / (p.beta * self.nk)
                lo, hi = (lo, mu) if 2 * dens > p.filling else (mu, hi)
            mu = 0.5 * (lo + hi)
        return 1 / (1j * nu + mu - self.eps - sg), float(mu)

    def gat(self, g, n, K):
        return g[n + self.ng // 2, K]

    def bubbles(self, g):
        p = self.p
        q = torch.arange(self.nq, device=DEV)[:, None]
        m, Q = q // self.nk - (self.nv // 2 - 1), q % self.nk
        n, K = self.row_n[None], self.row_K[None]
        gk = self.gat(g, n, K)
        xph = gk * self.gat(g, n + m, self.add(K, Q)) / (p.beta * self.nk)
        xpp = gk * self.gat(g, m - n - 1, self.add(Q, K, -1)) / (2 * p.beta * self.nk)
        return xph, xpp

    def kernels(self, phi):
        k1 = torch.zeros((4, self.nq), dtype=torch.complex128, device=DEV)
        k2 = torch.zeros((4, self.nq, self.n), dtype=torch.complex128, device=DEV)
        top, bot = self.nv - 1, 0
        for r in range(4):
            for jm in range(self.nw):
                m = jm - (self.nv // 2 - 1)
                edges = [top, bot] if m == 0 else [top if (m > 0) == (r < 2) else bot]
                q = slice(jm * self.nk, (jm + 1) * self.nk)
                for e in edges:
                    cols = slice(e * self.nk, (e + 1) * self.nk)
                    row = phi[r, q, :, cols].to(torch.complex128).mean(-1)
                    k2[r, q] += row / len(edges)
                    k1[r, q] += row[:, cols].mean(-1) / len(edges)
        k2 -= k1[:, :, None]
        if self.p.kernel_level == 1:
            k2.zero_()
        return k1, k2

    def remap(self, phi, k1, k2):
        n, nk, hb = self.n, self.nk, self.nv // 2 - 1
        nn, K = self.row_n[:, None], self.row_K[:, None]
        n2, K2 = self.row_n[None], self.row_K[None]
        row = torch.arange(n, device=DEV)[:, None]
        flat = [f.reshape(-1) for f in phi]
        out = [torch.empty((self.nq, n, n), dtype=torch.complex128, device=DEV) for _ in range(4)]

        def at(mp, P, nb, B):
            """Both channels' accessor at (k, b; p): stored, kernel-filled, or zero."""
            ok_p = mp.abs() <= hb
            ok = ok_p & (nb >= -self.nv // 2) & (nb < self.nv // 2)
            pi = torch.where(ok_p, (mp + hb) * nk + P, 0)
            idx = (pi * n + row) * n + torch.where(ok, (nb + self.nv // 2) * nk + B, 0)

            def get(r):
                fill = torch.where(ok_p, k1[r][pi] + k2[r].reshape(-1)[pi * n + row], 0)
                return torch.where(ok, flat[r][idx].to(torch.complex128), fill)
            return get

        for qi in range(self.nq):
            m, Q = qi // nk - hb, torch.tensor(qi % nk, device=DEV)
            full = torch.zeros((n, n), dtype=torch.int64, device=DEV)
            kq, dk = self.add(K, Q), self.add(K2, K, -1)
            bar = at(n2 - nn, dk + full, nn + m + full, kq + full)
            pp = at(nn + n2 + m + 1, self.add(self.add(K, K2), Q), n2 + full, K2 + full)
            st1 = at(n2 - nn, dk + full, m - n2 - 1 + full, self.add(Q, K2, -1) + full)
            st2 = at(m - nn - n2 - 1, self.add(self.add(Q, K, -1), K2, -1), n2 + full, K2 + full)
            d, mm, s, t = bar(0), bar(1), pp(2), pp(3)
            lam = _lam(self.p)
            out[0][qi] = lam[0] - 0.5 * d - 1.5 * mm + 0.5 * s + 1.5 * t
            out[1][qi] = lam[1] - 0.5 * d + 0.5 * mm - 0.5 * s + 0.5 * t
            d1, m1, d2, m2 = st1(0), st1(1), st2(0), st2(1)
            out[2][qi] = lam[2] + 0.5 * d1 - 1.5 * m1 + 0.5 * d2 - 1.5 * m2
            out[3][qi] = lam[3] - 0.5 * d1 - 0.5 * m1 + 0.5 * d2 + 0.5 * m2
        return out

    def sigma1(self, g, mu):
        """Second-order diagram over all frequencies: imaginary time, two Gauss-Legendre panels."""
        p, nk = self.p, self.nk
        nu = self.nu(self.nve)
        emax = p.D if nk == 1 else float((self.eps - mu).abs().max())
        x, w = np.polynomial.legendre.leggauss(6 * self.nve + 48 + 3 * int(math.ceil(p.beta * emax)))
        h = 0.25 * p.beta
        tau = torch.tensor(np.concatenate([h * (x + 1), 2 * h + h * (x + 1)]), device=DEV)
        wt = torch.tensor(np.concatenate([h * w, h * w]), device=DEV)
        if nk == 1:
            th = torch.arange(1, 201, device=DEV, dtype=torch.float64) * math.pi / 201
            e, cw = p.D * torch.cos(th), 2 * torch.sin(th) ** 2 / 201
        else:
            e, cw = self.eps - mu, None
        pole_w = 1 / (1j * nu[:, None] - e[None])
        pole_t = torch.where(e >= 0, -torch.exp(-tau[:, None] * e.clamp(min=0)) / (1 + torch.exp(-p.beta * e.clamp(min=0))),
                             -torch.exp((p.beta - tau)[:, None] * e.clamp(max=0)) / (torch.exp(p.beta * e.clamp(max=0)) + 1))
        if cw is not None:
            pole_w, pole_t = (pole_w * cw).sum(1, keepdim=True), (pole_t * cw).sum(1, keepdim=True)
        dg = g[self.ng // 2 - self.nve // 2:self.ng // 2 + self.nve // 2] - pole_w
        gkt = pole_t + torch.exp(-1j * tau[:, None] * nu[None]) @ dg / p.beta
        kx, ky = self.kx.double(), self.ky.double()
        ph = torch.exp(2j * math.pi * (kx[:, None] * kx[None] / p.Lx + ky[:, None] * ky[None] / p.Ly))
        grt = gkt @ ph.T / nk
        neg = self.add(torch.zeros_like(self.kx), torch.arange(nk, device=DEV), -1)
        srt = p.U ** 2 * grt ** 2 * grt.flip(0)[:, neg]
        return ((torch.exp(1j * nu[:, None] * tau[None]) * wt) @ srt) @ ph.conj()

    def sigma(self, phi, k1, k2, g, mu):
        """Sigma~_1 + the kernel vertex over the extended box + (Phi - kernels) over the box, in native arguments."""
        p, nk, n = self.p, self.nk, self.n
        K = torch.arange(nk, device=DEV)
        kp, pk = self.add(K[:, None], K[None]), self.add(K[None], K[:, None], -1)      # [K][P]: K + P, P - K
        hF, hB, fb, hb = self.nve // 2, self.nve // 2 - 1, self.nv // 2, self.nv // 2 - 1
        nke, nb = torch.arange(-hF, hF, device=DEV), torch.arange(-self.ng // 2, self.ng // 2, device=DEV)
        ext = torch.zeros((self.nve, nk), dtype=torch.complex128, device=DEV)
        box = slice(hF - fb, hF + fb)

        def row(i):                                           # G at a frequency, zero outside its grid
            ok = (i >= -self.ng // 2) & (i < self.ng // 2)
            return torch.where(ok[:, None], g[i.clamp(-self.ng // 2, self.ng // 2 - 1) + self.ng // 2], 0)

        for jm in range(self.nw):
            mp = jm - hb
            q = slice(jm * nk, (jm + 1) * nk)
            gk = row(nke + mp)[:, kp]                         # [k freq][K][P]: G(k + p)
            gp = row(mp - nke - 1)[:, pk]                     # G(p - k)
            u1 = row(nb)[:, :, None] * row(nb + mp)[:, kp]    # [b freq][B][P]
            u3 = row(nb)[:, :, None] * row(mp - nb - 1)[:, pk]

            def weights(a, b, hf, hbos):
                a, b = a[:, None], b[None]
                i1, i2 = ((mp + a + b + 1).abs() <= hbos), ((b - a).abs() <= hbos)
                i3 = (mp - a - b - 1).abs() <= hbos
                bin_, kin = (b >= -hf) & (b < hf), (a + mp >= -hf) & (a + mp < hf)
                return ((bin_ * (1 + i1.double())).to(torch.complex128), (kin * (i2.double() + i1.double())).to(torch.complex128),
                        (bin_ * (1 + i3.double())).to(torch.complex128))

            w16, w25, w34 = weights(nke, nb, hF, hB)
            s16, s25, s34 = (w @ u.sum(1) for w, u in ((w16, u1), (w25, u1), (w34, u3)))      # [k freq][P]
            c = k1[:, q][:, None, None, :].expand(4, self.nve, nk, nk).clone()
            kk2 = k2[:, q].reshape(4, nk, self.nv, nk).permute(0, 2, 3, 1)                    # [r][freq][K][P]
            c[:, box] += kk2
            inb = slice(self.ng // 2 - fb, self.ng // 2 + fb)
            v1 = [(u1[inb] * kk2[r]).sum(1) for r in (0, 1)]                                  # [b freq in box][P]
            v3 = (u3[inb] * (kk2[2] + kk2[3])).sum(1)
            kern = gk * (c[0] * s16[:, None] - c[1] * (s16 + 2 * s25)[:, None]) + gp * (c[2] + c[3]) * s34[:, None]
            kern = kern + gk * (w16[:, inb] @ v1[0] - (w16 + 2 * w25)[:, inb] @ v1[1])[:, None] \
                + gp * (w34[:, inb] @ v3)[:, None]
            ext += kern.sum(-1)
            # the box: Phi minus its kernel value
            b16, b25, b34 = weights(nke[box], nb[inb], fb, hb)
            big = [w.repeat_interleave(nk, 0).repeat_interleave(nk, 1) for w in (b16, b16 + 2 * b25, b34)]
            for P in range(nk):
                qi = jm * nk + P

                def diff(r):
                    return phi[r][qi].to(torch.complex128) - (k1[r, qi] + k2[r, qi][:, None] + k2[r, qi][None])
                f1, f3 = u1[inb][:, :, P].reshape(-1), u3[inb][:, :, P].reshape(-1)
                t1 = (big[0] * diff(0) - big[1] * diff(1)) @ f1
                t3 = (big[2] * (diff(2) + diff(3))) @ f3
                ext[box] += gk[box][:, :, P] * t1.view(self.nv, nk) + gp[box][:, :, P] * t3.view(self.nv, nk)
        return self.sigma1(g, mu) - p.U / (4 * p.beta ** 2 * nk ** 2) * ext

    def inverse(self, a):
        """Batched inverse by recursive block elimination (a is the identity plus a small-norm kernel)."""
        n = a.shape[-1]
        if n == 1:
            return 1 / a
        h = (n + 1) // 2
        p = self.inverse(a[:, :h, :h].contiguous())
        b, c = a[:, :h, h:].contiguous(), a[:, h:, :h].contiguous()
        pb, cp = p @ b, c @ p
        s = self.inverse(a[:, h:, h:] - c @ pb)
        top = torch.cat([p + pb @ (s @ cp), -(pb @ s)], 2)
        return torch.cat([top, torch.cat([-(s @ cp), s], 2)], 1)

    def bse(self, r, gamma, x, phi, alpha):
        out = torch.empty((self.nq, self.n, self.n), dtype=torch.complex128, device=DEV)
        eye = torch.eye(self.n, dtype=torch.complex128, device=DEV)
        step = max(1, (1 << 27) // (self.n * self.n))
        for q0 in range(0, self.nq, step):
            gm = gamma[q0:q0 + step].to(torch.complex128)
            a = eye - SIGN[r] * gm * x[q0:q0 + step, None, :]
            inv = self.inverse(a)
            f = inv @ gm
            f = f + inv @ (gm - a @ f)
            out[q0:q0 + step] = alpha * (f - gm) + (1 - alpha) * phi[q0:q0 + step].to(torch.complex128)
        return out

    def iterate(self, sigma, phi):
        g, mu = self.dyson(sigma)
        xph, xpp = self.bubbles(g)
        k1, k2 = self.kernels(phi)
        gamma = self.remap(phi, k1, k2)
        new = self.sigma(phi, k1, k2, g, mu)
        a = self.p.alpha
        phi = [self.bse(r, gamma[r], xph if r < 2 else xpp, phi[r], a) for r in range(4)]
        return a * new + (1 - a) * sigma, torch.stack(phi), k2

    def start(self):
        g, mu = self.dyson(torch.zeros((self.nve, self.nk), dtype=torch.complex128, device=DEV))
        return self.sigma1(g, mu), torch.zeros((4, self.nq, self.n, self.n), dtype=torch.complex128, device=DEV)


def _exact_mlp(c, seed):
    s = prepare(c, seed)
    net, x, t = s["net"], s["x"].double(), s["t"].double()
    w = net.widths
    p0 = net.p.double()
    layers, off = [], 0
    for i in range(len(w) - 1):
        k = w[i] * w[i + 1]
        wt = net.p[off:off + k].to(torch.bfloat16).double().view(w[i + 1], w[i])
        layers.append((wt, p0[off + k:off + k + w[i + 1]]))
        off += k + w[i + 1]
    acts, h = [], x
    for i, (wt, b) in enumerate(layers):
        h = h @ wt.T + b
        h = torch.tanh(h) if i < len(layers) - 1 else h
        acts.append(h)
    d = 2 * (acts[-1] - t) / t.numel()
    grads = []
    for i in reversed(range(len(layers))):
        hin = acts[i - 1] if i else x
        grads.append(torch.cat([(d.T @ hin).reshape(-1), d.sum(0)]))
        if i:
            d = (d @ layers[i][0]) * (1 - hin * hin)
    g = torch.cat(grads[::-1])
    m, v = 0.1 * g, 0.001 * g * g
    p = p0 - 1e-3 * (m / 0.1) / (torch.sqrt(v / 0.001) + 1e-8)
    return dict(acts=torch.cat([a.reshape(-1) for a in acts]), loss=((acts[-1] - t) ** 2).mean().view(1), grad=g, p=p,
                m=m, v=v)


def exact(c, seed):
    kind = c["kind"]
    if kind == "mlp":
        return _exact_mlp(c, seed)
    if kind == "batch":
        out = []
        for i in range(c["count"]):
            ref = _Ref(_params(c, seed, i))
            sg, phi = ref.start()
            for _ in range(c["rounds"]):
                sg, phi, k2 = ref.iterate(sg, phi)
            out.append(dict(sigma=sg, k2=k2))
        return out
    p = _params(c, seed)
    ref = _Ref(p)
    if kind == "solve":
        sg, phi = ref.start()
        for _ in range(c["iters"]):
            sg, phi, _ = ref.iterate(sg, phi)
        return dict(sigma=sg, phi=phi)
    if kind == "dyson":
        g, mu = ref.dyson(_sigma(p, seed))
        xph, xpp = ref.bubbles(g)
        return dict(g=g, mu=torch.tensor([mu], dtype=torch.float64), xph=xph, xpp=xpp)
    dtype = torch.complex128 if c["prec"] == "fp64" else torch.complex64
    if kind == "bse":
        g, _ = ref.dyson(_sigma(p, seed))
        x = ref.bubbles(g)[0 if c["channel"] < 2 else 1]
        gamma = _vertex(p, dtype, seed, 1, 0.5, [_lam(p)[c["channel"]]])[0]
        phi = _phi(p, dtype, seed + 1, (c["channel"],), 1.0)[0]
        return dict(phi=ref.bse(c["channel"], gamma, x, phi, 0.5), flags=None)
    phi = _phi(p, dtype, seed)
    if kind == "iterate":
        sg, new, _ = ref.iterate(_sigma(p, seed), phi)
        return dict(sigma=sg, phi=list(new))
    k1, k2 = ref.kernels(phi)
    if kind == "remap":
        return dict(k1=k1, k2=k2, gamma=ref.remap(phi, k1, k2))
    g, mu = ref.dyson(_sigma(p, seed))
    return dict(sigma=ref.sigma(phi, k1, k2, g, mu))
