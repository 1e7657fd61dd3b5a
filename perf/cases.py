"""The workloads that this package's speed is measured on, and what they have to return.

Every case is one pass of a user's program through the package's public entry
points: field evaluations of small lattices, runs of string iterations (with
the options of the reparametrisation and of step 1), batched sweeps, the
autograd form.  A case is a dict:

  op      "eval"     StringMethod.eval of a given string: energies, field, terms
          "noalloc"  the same through ssm_eval_noalloc (fixed scratch, no context)
          "string"   set_string, iterate, then string, energies and barrier
          "sweep"    the same for a batch of uneven lattices with a tolerance,
                     plus tangents and force norms (the convergence report)
          "rk"       string iterations whose step 1 is the adaptive integrator
          "llg"      time integration of every image
          "grad"     autograd: energies, gradients in spins and parameters
  nx, ny, nz, K      lattice and images; np > 1: a batch of np problems (op
                     "sweep": square monolayers of nx..ny sites a side)
  prec    "fp64" or "fp32" (the mixed form)
  iters, tau, graph  iterations, step (or interval), iterations per replayed graph
  spline, climb      options of the reparametrisation
  J, d, ku, D        parameters (a batch spreads d and ku around them)
  kind, R            initial string: "bloch" or "boundary", skyrmion radius
"""
import math

import torch

from paper_1804_07135_amd import ssm


def _case(name=None, **kw):
    c = dict(op="string", nx=32, ny=32, nz=1, K=10, np=1, prec="fp64", iters=0, tau=0.1, graph=0, spline=False,
             climb=False, J=1.0, d=0.3, ku=0.1, D=0.01, kind="bloch", R=5.0)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one evaluation of the smallest production lattice: latency and launches
        _case("eval_32x32x1_k10_fp64", op="eval"),
        # the allocation-free evaluation of a small ragged bilayer
        _case("noalloc_60x44x2_k12_fp32", op="noalloc", nx=60, ny=44, nz=2, K=12, prec="fp32"),
        # a Bloch-point barrier of a small monolayer, iterations replayed as graphs
        _case("string_32x32x1_k10_fp64", iters=40, graph=20),
        # the boundary process on a small monolayer in the mixed form
        _case("string_64x64x1_k20_fp32", nx=64, ny=64, K=20, prec="fp32", iters=40, graph=20, kind="boundary"),
        # the paper's production shape: 112 x 112 monolayer, 60 images, its material
        _case("string_112x112x1_k60_fp32", nx=112, ny=112, K=60, prec="fp32", iters=20, graph=20, R=10.0,
              d=0.1, ku=0.02, D=2.787e-4),
        # a ragged multilayer stepped without graph replay
        _case("string_200x180x5_k20_fp32", nx=200, ny=180, nz=5, K=20, prec="fp32", iters=5, d=0.25, ku=0.08,
              D=0.02, R=12.0),
        # the headline lattice: skyrmion tube, 48 images, mixed form
        _case("string_256x256x8_k48_fp32", nx=256, ny=256, nz=8, K=48, prec="fp32", iters=10, graph=10, D=0.02,
              R=20.0),
        # the same in double precision, as a check run would do it
        _case("string_256x256x8_k48_fp64", nx=256, ny=256, nz=8, K=48, iters=2, D=0.02, R=20.0),
        # the (k_u, d) sweep: 64 uneven monolayers in one context, spline and climbing image, force tolerance
        _case("sweep_64pts_k16_fp32", op="sweep", nx=48, ny=96, K=16, np=64, prec="fp32", iters=20, graph=10,
              spline=True, climb=True, d=0.25, ku=0.125),
        # a phase diagram's iteration: four points of the paper's shape, adaptive integrator over its interval
        _case("rk_112x112x1_k60_4pts_fp32", op="rk", nx=112, ny=112, K=60, np=4, prec="fp32", iters=1, tau=1.737,
              R=10.0, d=0.1, ku=0.02, D=2.787e-4),
        # spin dynamics of a ragged trilayer
        _case("llg_100x75x3_k24_fp64", op="llg", nx=100, ny=75, nz=3, K=24, tau=0.5, D=0.02, R=8.0),
        # training through the energy: value and gradients
        _case("grad_128x128x4_k32_fp64", op="grad", nx=128, ny=128, nz=4, K=32, d=0.25, ku=0.08, D=0.02, R=12.0),
    ]


# site-images evaluated in 32 bits (those in 64 count twice) that a drawn case
# may take: under those of the largest listed one, whatever its padding
_MOST = 1.0e8


def draw(rng):
    def logint(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    op = rng.choice(["eval", "noalloc", "string", "string", "string", "sweep", "rk", "llg", "grad"])
    prec = rng.choice(["fp64", "fp32"])
    nz = rng.choice([1, 1, 1, 1, 2, 3, 4, 5, 8, 12])
    d, ku, D = rng.uniform(0.1, 0.4), rng.uniform(0.05, 0.2), rng.choice([2.787e-4, 0.01, 0.02])
    kw = dict(op=op, prec=prec, d=round(d, 4), ku=round(ku, 4), D=D, kind=rng.choice(["bloch", "boundary"]))
    if op == "sweep":
        lo = logint(24, 72)
        kw.update(nx=lo, ny=lo + logint(8, 64), K=rng.choice([8, 12, 16, 20, 32]), np=logint(4, 64),
                  iters=20, graph=10, spline=rng.random() < 0.6, climb=rng.random() < 0.6)
        mean = ((kw["nx"] + kw["ny"]) / 2) ** 2 * kw["K"] * 23 * (2 if prec == "fp64" else 1)
        kw["np"] = max(2, min(kw["np"], int(_MOST / mean)))
    else:
        nx, ny, K = logint(10, 300), logint(10, 300), logint(4, 64)
        if op == "rk":
            kw.update(iters=1, tau=round(rng.uniform(0.4, 1.8), 3), np=rng.choice([1, 1, 2, 4]))
        elif op == "llg":
            kw.update(tau=round(rng.uniform(0.2, 0.8), 3))
        elif op == "string":
            kw.update(graph=rng.choice([0, 10]), spline=rng.random() < 0.25, climb=rng.random() < 0.25)
            kw["iters"] = 10 if kw["graph"] else rng.choice([3, 5, 8])
        if op == "noalloc":  # what its fixed scratch holds
            nz, nx, ny, K = min(nz, 2), min(nx, 64), min(ny, 64), min(K, 16)
        evals = {"rk": 40, "llg": 40}.get(op, kw.get("iters", 0) + 1) * kw.get("np", 1) * (2 if prec == "fp64" else 1)
        # the padded lattice sets the cost: fewer images, layers and rows until the case is small enough
        while nx * ny * max(nz, 1) * K * evals > _MOST:
            if K > 8:
                K = K * 3 // 4
            elif nz > 2:
                nz //= 2
            else:
                nx, ny = max(10, nx * 4 // 5), max(10, ny * 4 // 5)
        kw.update(nx=nx, ny=ny, nz=nz, K=K)
    kw["R"] = round(max(2.0, min(kw["nx"], kw["ny"]) / rng.uniform(6.0, 12.0)), 2)
    return _case(**kw)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _problems(c):
    """Problem dicts of a case; the points of a batch differ in d and k_u (and size, for a sweep)."""
    out = []
    n = c["np"]
    for i in range(n):
        f = (i + 0.5) / n - 0.5 if n > 1 else 0.0
        g = ((i * 7) % n + 0.5) / n - 0.5 if n > 1 else 0.0
        nx, ny = c["nx"], c["ny"]
        if c["op"] == "sweep":
            nx = ny = c["nx"] + (i * 37) % (c["ny"] - c["nx"] + 1)
        out.append(dict(nx=nx, ny=ny, nz=c["nz"], K=c["K"], J=c["J"], d=c["d"] * (1 + 0.8 * f),
                        ku=c["ku"] * (1 + 0.8 * g), D=c["D"]))
    return out


def _string(c, p, gen, dev):
    """Initial string [K,3,nz,ny,nx] of one problem: the skyrmion's closed-form path
    (Bloch point: the angle shrinks; boundary: the centre moves out past an edge),
    every spin perturbed by 1e-3 and renormalised; FP64."""
    nx, ny, nz, K, R = p["nx"], p["ny"], p["nz"], p["K"], c["R"]
    x = torch.arange(nx, dtype=torch.float64, device=dev)[None, None, None, :]
    y = torch.arange(ny, dtype=torch.float64, device=dev)[None, None, :, None]
    t = (torch.arange(K, dtype=torch.float64, device=dev) / (K - 1))[:, None, None, None]
    cx, cy = (nx - 1) / 2.0, (ny - 1) / 2.0
    if c["kind"] == "boundary":
        rx = x - (cx + t * (nx - 1 + 2.0 * R - cx))
        ry = (y - cy).expand(K, 1, ny, nx)
        rx = rx.expand(K, 1, ny, nx)
        th = 2.0 * torch.atan2(torch.full_like(rx, R), torch.hypot(rx, ry))
        th[K - 1] = 0.0
    else:
        rx = (x - cx).expand(K, 1, ny, nx)
        ry = (y - cy).expand(K, 1, ny, nx)
        th = (1.0 - t) * 2.0 * torch.atan2(torch.full_like(rx, R), torch.hypot(rx, ry))
    ph = torch.atan2(ry, rx)
    s = torch.stack([-torch.sin(th) * torch.cos(ph), -torch.sin(th) * torch.sin(ph), torch.cos(th)], dim=1)
    s = s.expand(K, 3, nz, ny, nx).contiguous()
    s = s + 1e-3 * torch.randn(s.shape, dtype=torch.float64, device=dev, generator=gen)
    return s / torch.linalg.vector_norm(s, dim=1, keepdim=True)


def _inputs(c, seed):
    """(problems, their strings in the case's type)."""
    dev = _device()
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    probs = _problems(c)
    dt = torch.float64 if c["prec"] == "fp64" else torch.float32
    return probs, [_string(c, p, gen, dev).to(dt) for p in probs]


def prepare(case, seed):
    c = case
    probs, strings = _inputs(c, seed)
    spins = strings[0] if len(strings) == 1 else torch.cat([s.reshape(-1) for s in strings])
    st = dict(case=c, probs=probs, spins=spins)
    prec = ssm.SSM_FP64 if c["prec"] == "fp64" else ssm.SSM_FP32_MIXED
    if c["op"] == "noalloc":
        st["prec"] = prec
        return st
    sm = ssm.StringMethod(probs, prec, with_rk=c["op"] in ("rk", "llg"))
    if c["op"] in ("string", "sweep"):
        sm.set_options(check_every=10, graph_chunk=c["graph"])
        if c["spline"] or c["climb"]:
            sm.set_reparam(ssm.SSM_INTERP_SPLINE if c["spline"] else ssm.SSM_INTERP_LINEAR, c["climb"])
    st["sm"] = sm
    if c["op"] == "grad":
        p = probs[0]
        st["theta"] = torch.tensor([p["J"], p["d"], p["ku"], p["D"]], dtype=torch.float64, requires_grad=True)
        st["spins"] = spins.requires_grad_(True)
        gen = torch.Generator(device=spins.device)
        gen.manual_seed(seed + 1)
        st["g"] = torch.rand(c["K"], dtype=torch.float64, device=spins.device, generator=gen) + 0.5
    return st


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
_RK_TOL = 1e-5
_SWEEP_TOL = 1e-4


def run(state):
    c, s = state["case"], state["spins"]
    op = c["op"]
    if op == "noalloc":
        E = torch.empty(c["K"], dtype=torch.float64, device=s.device)
        T = torch.empty((c["K"], 4), dtype=torch.float64, device=s.device)
        h = torch.empty_like(s)
        ssm.ssm_eval_noalloc(state["probs"], state["prec"], s, h, E, T)
        return dict(E=E, field=h, terms=T)
    sm = state["sm"]
    if op == "eval":
        E, h, T = sm.eval(s)
        return dict(E=E, field=h, terms=T)
    if op == "grad":
        E = ssm.spin_energy(s, state["theta"], sm)
        gs, gt = torch.autograd.grad(E, (s, state["theta"]), state["g"])
        return dict(E=E.detach(), gs=gs, gt=gt)
    sm.set_string(s)
    if op == "llg":
        sm.set_integrator(ssm.SSM_STEP_DOPRI54, _RK_TOL, _RK_TOL, c["tau"] / 10)
        sm.llg(c["tau"], 0.5)
        return dict(string=sm.get_string(), E=sm.energies())
    if op == "rk":
        sm.set_integrator(ssm.SSM_STEP_DOPRI54, _RK_TOL, _RK_TOL, c["tau"] / 10)
    it = sm.iterate(c["iters"], c["tau"], _SWEEP_TOL if op == "sweep" else 0.0)
    out = dict(iters=it, string=sm.get_string(), E=sm.energies(), barrier=sm.barrier())
    if op == "sweep":
        out["tangent"], out["force"] = sm.tangents()
    return out


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
# field evaluations of one interval of the adaptive integrator: the first
# slope and six per attempted step, five attempts (the usual count of an
# interval started at a tenth of its length)
_RK_EVALS = 31


def work(case):
    c = case
    b = 8 if c["prec"] == "fp64" else 4
    nb = flops = 0.0
    for p in _problems(c):
        N, K = p["nx"] * p["ny"] * p["nz"], p["K"]
        string = 3.0 * N * K * b
        pad = 4 * p["nx"] * p["ny"] * (2 * p["nz"] if p["nz"] > 1 else 1)
        # six real transforms of the padded lattice, the 3x3 product, about 100 operations a site
        field = K * (6 * 2.5 * pad * math.log2(max(2, pad)) + 15.0 * pad + 100.0 * N)
        if c["op"] in ("eval", "noalloc", "grad"):
            nb += 2 * string  # spins in, field (gradient) out
            flops += field
        else:
            it = max(1, c["iters"])
            ev = _RK_EVALS if c["op"] in ("rk", "llg") else 1
            # an iteration reads the string and writes it stepped, then reads
            # that and writes the reparametrised one; an evaluation of a stage
            # reads the string and writes the slope
            nb += it * (2 * string * ev + (0 if c["op"] == "llg" else 2 * string)) + 2 * string
            flops += (it * ev + 1) * field
    return {"bytes": nb, "flops": flops}


# ---------------------------------------------------------------------------
# the same results in 64 bits, from the paper's equations in plain torch
# ---------------------------------------------------------------------------
_COMP = [(0, 0), (0, 1), (0, 2), (1, 1), (1, 2), (2, 2)]


class _Lattice:
    """Field, energies and string steps of one problem in FP64."""

    def __init__(self, p, dev):
        self.p, self.dev = p, dev
        n = (p["nz"], p["ny"], p["nx"])
        self.n = n
        self.P = tuple(2 * k if k > 1 else 1 for k in n)
        ax = []
        for k, P in zip(n, self.P):
            a = torch.arange(P, dtype=torch.float64, device=dev)
            a = torch.where(a >= k, a - P, a)
            ax.append((a, a.abs() < k))  # the offset -k never pairs two sites
        z, y, x = torch.meshgrid(ax[0][0], ax[1][0], ax[2][0], indexing="ij")
        ok = ax[0][1][:, None, None] & ax[1][1][None, :, None] & ax[2][1][None, None, :]
        r2 = x * x + y * y + z * z
        ok = ok & (r2 > 0)
        ri = torch.where(ok, r2, torch.ones_like(r2)).rsqrt()
        v = (x, y, z)
        self.k = [torch.fft.rfftn(torch.where(ok, 3 * v[a] * v[b] * ri ** 5 - (ri ** 3 if a == b else 0.0),
                                              torch.zeros_like(r2))) for a, b in _COMP]

    def dipolar(self, s):
        out = torch.empty_like(s)
        step = max(1, int(4e7 // (3 * self.P[0] * self.P[1] * self.P[2])))
        idx = {}
        for i, (a, b) in enumerate(_COMP):
            idx[a, b] = idx[b, a] = i
        nz, ny, nx = self.n
        for k in range(0, s.shape[0], step):
            f = torch.fft.rfftn(s[k:k + step], s=self.P, dim=(-3, -2, -1))
            for a in range(3):
                g = sum(self.k[idx[a, b]] * f[:, b] for b in range(3))
                out[k:k + step, a] = torch.fft.irfftn(g, s=self.P, dim=(-3, -2, -1))[:, :nz, :ny, :nx]
        return out

    def field(self, s):
        """h and the unit-parameter term energies [K,4]."""
        p = self.p

        def shift(dim, by):
            r = torch.zeros_like(s)
            n = s.shape[dim]
            if n > 1:
                if by > 0:
                    r.narrow(dim, 0, n - 1).copy_(s.narrow(dim, 1, n - 1))
                else:
                    r.narrow(dim, 1, n - 1).copy_(s.narrow(dim, 0, n - 1))
            return r

        xp, xm, yp, ym = shift(-1, 1), shift(-1, -1), shift(-2, 1), shift(-2, -1)
        nb = xp + xm + yp + ym
        dm = torch.stack([-(xp[:, 2] - xm[:, 2]), -(yp[:, 2] - ym[:, 2]),
                          xp[:, 0] - xm[:, 0] + yp[:, 1] - ym[:, 1]], dim=1)
        del xp, xm, yp, ym
        nb += shift(-3, 1)
        nb += shift(-3, -1)
        hd = self.dipolar(s)
        dims = (1, 2, 3, 4)
        T = torch.stack([-0.5 * (s * nb).sum(dims), -0.5 * (s * dm).sum(dims), -(s[:, 2] ** 2).sum((1, 2, 3)),
                         -0.5 * (s * hd).sum(dims)], dim=1)
        h = p["J"] * nb + p["d"] * dm + p["D"] * hd
        h[:, 2] += 2.0 * p["ku"] * s[:, 2]
        return h, T

    def theta(self):
        p = self.p
        return torch.tensor([p["J"], p["d"], p["ku"], p["D"]], dtype=torch.float64, device=self.dev)

    def energies(self, T):
        return T @ self.theta()

    @staticmethod
    def unit(s):
        return s / torch.linalg.vector_norm(s, dim=1, keepdim=True)

    @staticmethod
    def perp(s, v):
        return v - (s * v).sum(1, keepdim=True) * s

    def rhs(self, s, cp, cd):
        h, _ = self.field(s)
        r = cd * ((s * s).sum(1, keepdim=True) * h - (s * h).sum(1, keepdim=True) * s)
        return r - cp * torch.cross(s, h, dim=1) if cp else r

    def iterate(self, s, iters, tau, spline, climb):
        for _ in range(iters):
            h, T = self.field(s)
            F = self.perp(s, h)
            kci = None
            if climb:
                k = int(torch.argmax(self.energies(T)))
                if 0 < k < s.shape[0] - 1:
                    kci = k
                    t = self.perp(s[k:k + 1], s[k + 1:k + 2] - s[k - 1:k])
                    n2 = (t * t).sum()
                    F[k:k + 1] -= 2.0 * ((F[k:k + 1] * t).sum() / n2 if n2 > 0 else 0.0) * t
            s = self.reparam(self.unit(s + tau * F), spline, kci)
        return s

    def reparam(self, ss, spline, kci):
        K = ss.shape[0]
        seg = torch.stack([torch.linalg.vector_norm(ss[k] - ss[k - 1]) for k in range(1, K)]).cpu()
        al = torch.cat([torch.zeros(1, dtype=torch.float64), torch.cumsum(seg, 0)])
        if not al[-1] > 0:
            return ss
        al = (al / al[-1]).tolist()
        W = torch.zeros(K, K, dtype=torch.float64)
        if spline and K > 2 and all(al[j + 1] > al[j] for j in range(K - 1)):
            # second derivatives of the natural cubic spline: A M = B f
            A = torch.eye(K, dtype=torch.float64)
            B = torch.zeros(K, K, dtype=torch.float64)
            for i in range(1, K - 1):
                hl, hr = al[i] - al[i - 1], al[i + 1] - al[i]
                A[i, i - 1], A[i, i], A[i, i + 1] = hl / 6, (hl + hr) / 3, hr / 6
                B[i, i - 1], B[i, i], B[i, i + 1] = 1 / hl, -1 / hl - 1 / hr, 1 / hr
            M = torch.linalg.solve(A, B)
        else:
            M = None
        copied = [0, K - 1] + ([kci] if kci is not None else [])
        for k in range(K):
            if k in copied:
                W[k, k] = 1.0
                continue
            if kci is None:
                t = k / (K - 1)
            elif k <= kci:
                t = al[kci] * k / kci
            else:
                t = al[kci] + (1 - al[kci]) * (k - kci) / (K - 1 - kci)
            j = max(i for i in range(K - 1) if al[i] <= t)
            w = al[j + 1] - al[j]
            if M is None:
                f = (t - al[j]) / w if w > 0 else 0.0
                W[k, j], W[k, j + 1] = 1 - f, f
            else:
                a = (al[j + 1] - t) / w
                b = 1 - a
                W[k, j] += a
                W[k, j + 1] += b
                W[k] += ((a ** 3 - a) * M[j] + (b ** 3 - b) * M[j + 1]) * w * w / 6
        out = (W.to(self.dev) @ ss.reshape(K, -1)).reshape(ss.shape)
        out = self.unit(out)
        for k in copied:
            out[k] = ss[k]
        return out

    def dopri(self, s, Tint, dt0, cp, cd):
        """Adaptive Dormand-Prince 5(4) of every image over Tint, renormalised at the end."""
        a = [[], [1 / 5], [3 / 40, 9 / 40], [44 / 45, -56 / 15, 32 / 9],
             [19372 / 6561, -25360 / 2187, 64448 / 6561, -212 / 729],
             [9017 / 3168, -355 / 33, 46732 / 5247, 49 / 176, -5103 / 18656],
             [35 / 384, 0, 500 / 1113, 125 / 192, -2187 / 6784, 11 / 84]]
        e = [35 / 384 - 5179 / 57600, 0, 500 / 1113 - 7571 / 16695, 125 / 192 - 393 / 640,
             -2187 / 6784 + 92097 / 339200, 11 / 84 - 187 / 2100, -1 / 40]
        K = s.shape[0]
        t, dtp, act = [0.0] * K, [dt0] * K, list(range(K))
        k0 = self.rhs(s, cp, cd)
        s = s.clone()
        while act:
            cap = [dtp[i] >= Tint - t[i] for i in act]
            hs = [Tint - t[i] if q else dtp[i] for i, q in zip(act, cap)]
            hv = torch.tensor(hs, dtype=torch.float64, device=self.dev)[:, None, None, None, None]
            y0 = s[act]
            ks = [k0[act]]
            for st in range(1, 7):
                y = y0 + hv * sum(c * k for c, k in zip(a[st], ks) if c)
                ks.append(self.rhs(y, cp, cd))
            err = hv * sum(c * k for c, k in zip(e, ks) if c)
            sc = _RK_TOL + _RK_TOL * torch.maximum(y0.abs(), y.abs())
            en = (err / sc).square().mean(dim=(1, 2, 3, 4)).sqrt().tolist()
            left = []
            for m, i in enumerate(act):
                fac = min(5.0, max(0.2, 0.9 * max(en[m], 1e-10) ** -0.2))
                if en[m] <= 1.0:
                    s[i], k0[i] = y[m], ks[6][m]
                    t[i] += hs[m]
                    if not cap[m]:
                        left.append(i)
                else:
                    fac = min(fac, 1.0)
                    left.append(i)
                dtp[i] = hs[m] * fac
            act = left
        return self.unit(s)

    def tangents(self, s, h):
        K = s.shape[0]
        d = torch.stack([s[min(k + 1, K - 1)] - s[max(k - 1, 0)] for k in range(K)])
        t = self.perp(s, d)
        n2 = (t * t).sum((1, 2, 3, 4), keepdim=True)
        inv = torch.where(n2 > 0, n2.rsqrt(), torch.zeros_like(n2))
        F = self.perp(s, h)
        cf = (F * t).sum((1, 2, 3, 4), keepdim=True) * inv * inv
        cf[0] = cf[K - 1] = 0.0
        return t * inv, torch.linalg.vector_norm(F - cf * t, dim=1).max()


def _join(parts):
    return parts[0] if len(parts) == 1 else torch.cat([x.reshape(-1) for x in parts])


def exact(case, seed):
    c = case
    op = c["op"]
    probs, strings = _inputs(c, seed)
    dev = strings[0].device
    out = dict(string=[], E=[], barrier=[], tangent=[], force=[], field=[], terms=[])
    for p, s in zip(probs, strings):
        L = _Lattice(p, dev)
        s = s.to(torch.float64)
        if op == "grad":
            gen = torch.Generator(device=dev)
            gen.manual_seed(seed + 1)
            g = torch.rand(c["K"], dtype=torch.float64, device=dev, generator=gen) + 0.5
            h, T = L.field(s)
            return dict(E=L.energies(T), gs=-g.view(-1, 1, 1, 1, 1) * h, gt=(g[:, None] * T).sum(0).cpu())
        if op == "llg":
            s = L.dopri(s, c["tau"], c["tau"] / 10, 1 / 1.25, 0.5 / 1.25)
        elif op == "rk":
            s = L.reparam(L.dopri(s, c["tau"], c["tau"] / 10, 0.0, 1.0), c["spline"], None)
        elif op in ("string", "sweep"):
            s = L.iterate(s, c["iters"], c["tau"], c["spline"], c["climb"])
        h, T = L.field(s)
        E = L.energies(T)
        out["string"].append(s)
        out["E"].append(E)
        if op in ("eval", "noalloc"):
            out["field"].append(h)
            out["terms"].append(T)
            continue
        k = int(torch.argmax(E))
        out["barrier"].append(torch.cat([torch.stack([E[k] - E[0], torch.tensor(float(k), device=dev,
                                                                                dtype=torch.float64)]), T[k] - T[0]]))
        if op == "sweep":
            t, f = L.tangents(s, h)
            out["tangent"].append(t)
            out["force"].append(f)
    E = torch.cat(out["E"])
    if op in ("eval", "noalloc"):
        return dict(E=E, field=_join(out["field"]), terms=torch.cat(out["terms"]))
    if op == "llg":
        return dict(string=_join(out["string"]), E=E)
    r = dict(iters=None, string=_join(out["string"]), E=E, barrier=torch.stack(out["barrier"]))
    if op == "sweep":
        r["tangent"], r["force"] = _join(out["tangent"]), torch.stack(out["force"])
    return r
