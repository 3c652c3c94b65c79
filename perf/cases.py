"""The work that programs have this library do, as measurable cases.

A case is a dict of plain values.  ``prepare`` builds what a program holds
before the call (fields made from a seed, a handle, a checkpoint), ``run``
makes one pass through the public entry points, ``exact`` gives the same
outputs in 64 bits from plain torch, and ``work`` the bytes and operations
of one pass.

Kinds of cases
  operator  one spectral operator applied to fields (diagnostics, tests)
  fields    every output field of a solved batch (what a run writes to disk)
  step      one load step from a checkpoint, to the default tolerances
  sequence  a few queued load steps of a batch from a checkpoint
  static    one load step of a caller-held state, no allocation
  evolve    device-driven iterations of Algorithm 3 or 4
  crack     an iteration-capped load step of grids with a running crack
  serve     two load-step requests of every problem of a server

Steps restart from a checkpoint, as a program that retries an increment
does, so every pass does the same work.
"""

import math

import numpy as np
import torch

from paper_2203_16467_amd import autotune, spff

NU = 0.2
DEVICE = "cuda:0"
OPS = {"project": spff.OP_PROJECT, "laplacian": spff.OP_NEG_LAPLACIAN, "displacement": spff.OP_DISPLACEMENT}
SPLITS = {"none": spff.SPLIT_NONE, "spectral": spff.SPLIT_SPECTRAL, "voldev": spff.SPLIT_VOLDEV}
ALL_FIELDS = 0x7F


def _case(kind, nx, ny, batch=1, **kw):
    c = dict(kind=kind, nx=nx, ny=ny, batch=batch, fp64=False, at=1, split="spectral", contact="same", ell=2.0,
             damage=False, amp=0.1, load=0.45, ticks=1, graph=False, tuned=False, steps=1)
    c.update(kw)
    return c


def listed():
    return [
        # a projection on the smallest grid in use: launch and call latency
        _case("operator", 64, 64, op="project", name="project-64"),
        # a double-precision operator on a few rectangular grids
        _case("operator", 1024, 256, 3, op="laplacian", fp64=True, name="laplacian-3x1024x256-f64"),
        # writing out a batch: strain, stress, energy, displacement, state
        _case("fields", 512, 512, 8, amp=0.2, graph=True, ticks=32, name="fields-8x512"),
        # one elastic load step of the CPU-sized problem, default options
        _case("step", 64, 64, name="step-64"),
        # the plain single-problem path: AT2, so mechanics and phase field
        # alternate, one host check per tick
        _case("step", 256, 256, at=2, load=0.4, name="step-256-at2"),
        # double precision, as parity checks and tight tolerances need it
        _case("step", 512, 512, fp64=True, amp=0.2, name="step-512-f64"),
        # a caller-held state, rectangular grid, AT2 with the isotropic energy
        _case("static", 256, 128, at=2, split="none", load=0.4, ticks=8, name="static-256x128-at2"),
        # viscous evolution of an odd batch driven on the device
        _case("evolve", 256, 256, 13, alg=3, at=2, split="voldev", amp=0.2, load=0.3, steps=4, graph=True, ticks=16,
              name="evolve-13x256"),
        # few problems with a crack, the production model, capped iterations:
        # the launches of a nucleation tail
        _case("crack", 512, 512, 3, split="spectral", contact="none", damage=True, ell=5.0, amp=0.2, load=0.3,
              graph=True, ticks=32, name="crack-3x512"),
        # the batched workload at full occupancy: two queued load steps
        _case("sequence", 512, 512, 64, amp=0.2, load=0.3, steps=2, graph=True, ticks=32, tuned=True,
              name="batch-64x512"),
        # the largest single grid, high contrast, short length scale
        _case("step", 2048, 2048, ell=1.0, amp=0.3, load=0.4, graph=True, ticks=16, tuned=True, name="step-2048"),
        # a serving mix: grids of 128^2 .. 1024^2, AT1 and AT2 alternating
        _case("serve", 1024, 1024, 12, load=0.35, graph=True, ticks=8, name="serve-12"),
    ]


def _grid(rng, lo, hi, most):
    """A rectangular power-of-two grid, a third of them square."""
    while True:
        a, b = rng.randint(lo, hi), rng.randint(lo, hi)
        if rng.random() < 1 / 3:
            b = a
        if a + b <= most:
            return 1 << a, 1 << b


def _batch(rng, nx, ny, px=1 << 22, most=64):
    """A batch size spread over its logarithm, at most px pixels in all."""
    return max(1, int(round(math.exp(rng.uniform(0, math.log(max(1, min(most, px // (nx * ny)))))))))


def draw(rng):
    kind = rng.choice(["operator", "fields", "step", "step", "step", "sequence", "sequence", "static", "evolve",
                       "crack", "serve"])
    amp, load = round(rng.uniform(0.05, 0.25), 3), round(rng.uniform(0.2, 0.45), 3)
    f64 = rng.random() < 0.25
    at = rng.choice([1, 1, 2])
    split = rng.choice(["none", "spectral", "spectral", "voldev"])
    graph = rng.random() < 0.5
    ticks = rng.choice([8, 16, 32]) if graph else rng.choice([1, 4])
    common = dict(amp=amp, load=load if at == 1 else min(load, 0.4), fp64=f64, at=at, split=split, graph=graph,
                  ticks=ticks)
    if kind == "operator":
        nx, ny = _grid(rng, 3, 11, 22)
        return _case(kind, nx, ny, _batch(rng, nx, ny), op=rng.choice(sorted(OPS)), fp64=f64)
    if kind == "fields":
        nx, ny = _grid(rng, 6, 11, 20)
        return _case(kind, nx, ny, _batch(rng, nx, ny, 1 << 21), **dict(common, at=1))
    if kind == "static":
        nx, ny = _grid(rng, 5, 10, 18)
        return _case(kind, nx, ny, **dict(common, graph=False))
    if kind == "evolve":
        nx, ny = _grid(rng, 6, 9, 18)
        return _case(kind, nx, ny, _batch(rng, nx, ny, 1 << 20, 16), alg=rng.choice([3, 4]), steps=rng.randint(2, 5),
                     **dict(common, at=rng.choice([1, 2])))
    if kind == "crack":
        nx, ny = _grid(rng, 7, 10, 19)
        return _case(kind, nx, ny, _batch(rng, nx, ny, 1 << 20, 8), contact=rng.choice(["none", "same"]),
                     damage=rng.random() < 0.5, ell=float(rng.choice([2, 4, 5])),
                     **dict(common, load=min(load, 0.3)))
    if kind == "serve":
        return _case(kind, 512, 512, rng.randint(3, 12), **dict(common, at=1, fp64=False, graph=True, ticks=8,
                                                                load=min(load, 0.35)))
    if kind == "sequence":
        nx, ny = _grid(rng, 6, 10, 18)
        px = 1 << (21 if f64 or at == 2 else 22)
        return _case(kind, nx, ny, _batch(rng, nx, ny, px), steps=rng.randint(1, 3), **common)
    nx, ny = _grid(rng, 5, 11, 21)
    return _case(kind, nx, ny, ell=float(rng.choice([1, 2, 3])), **common)


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _real(case):
    return torch.float64 if case["fp64"] else torch.float32


def _modulus(case, seed, nx=None, ny=None, index=0):
    """E = max(1 + amp z, 1/2), z a unit-variance Gaussian random field with
    a correlation length of 1/32 of the grid; float32 values."""
    nx, ny = nx or case["nx"], ny or case["ny"]
    g = torch.Generator().manual_seed((seed * 1009 + index) & 0x7FFFFFFF)
    w = torch.randn(ny, nx, generator=g, dtype=torch.float64)
    corr = max(2.0, min(nx, ny) / 32.0)
    ky = torch.fft.fftfreq(ny, dtype=torch.float64)[:, None] * 2 * math.pi
    kx = torch.fft.rfftfreq(nx, dtype=torch.float64)[None, :] * 2 * math.pi
    z = torch.fft.irfft2(torch.fft.rfft2(w) * torch.exp(-(kx * kx + ky * ky) * corr * corr / 4), s=(ny, nx))
    z = z - z.mean()
    return torch.clamp(1 + case["amp"] * z / z.std(), min=0.5).float()


def _moduli(case, seed):
    return torch.stack([_modulus(case, seed, index=b) for b in range(case["batch"])]).to(_real(case))


def _strain(case, factor=1.0):
    """Uniaxial macroscopic strain at `factor` of the case's load, which is
    in units of the homogeneous AT1 strength."""
    lam, mu = NU / (1 - NU - 2 * NU * NU), 1 / (2 + 2 * NU)
    em = math.sqrt(3 / (8 * case["ell"] * (lam + 2 * mu)))
    return np.array([0.0, case["load"] * factor * em, 0.0])


def _crack(case):
    """Phase field of a centred straight crack over a third of the grid."""
    nx, ny, ell = case["nx"], case["ny"], case["ell"]
    y = (torch.arange(ny, dtype=torch.float64) - ny // 2)[:, None]
    x = (torch.arange(nx, dtype=torch.float64) - nx // 2)[None, :]
    r = torch.sqrt(torch.clamp(x.abs() - nx / 6, min=0) ** 2 + y * y)
    phi = torch.where(r <= 2 * ell, (1 - r / (2 * ell)) ** 2, torch.zeros_like(r))
    return phi.expand(case["batch"], ny, nx).to(_real(case)).contiguous()


def _operand(case, seed):
    """Smooth-plus-noise fields, as stresses and phase fields are."""
    g = torch.Generator().manual_seed(seed & 0x7FFFFFFF)
    planes = () if case["op"] == "laplacian" else (3,)
    x = torch.randn((case["batch"],) + planes + (case["ny"], case["nx"]), generator=g, dtype=torch.float64)
    return (0.2 * x + torch.cumsum(x, -1) / math.sqrt(case["nx"])).to(_real(case))


def _serve_problems(case, seed):
    """(config case, E) of the served problems: four grids, AT1 and AT2."""
    out = []
    for i in range(case["batch"]):
        n = min(128 << (i % 4), case["nx"])
        out.append((dict(case, nx=n, ny=n, batch=1, at=1 + (i // 4) % 2), _modulus(case, seed, n, n, i)))
    return out


def _config(case):
    kw = dict(nx=case["nx"], ny=case["ny"], at=case["at"], split=SPLITS[case["split"]], ell=case["ell"], nu=NU,
              contact=spff.CONTACT_SAME if case["contact"] == "same" else SPLITS[case["contact"]],
              irreversibility=spff.IRR_DAMAGE if case["damage"] else spff.IRR_CRACK_SET,
              precision=spff.FP64 if case["fp64"] else spff.FP32, ticks_per_sync=case["ticks"],
              use_graph=1 if case["graph"] else 0)
    if case["kind"] == "crack":
        kw.update(max_am=2, max_newton=1, max_cg=CRACK_CG, max_bccg=CRACK_BCCG)
    if case["kind"] == "evolve":
        # the load advances every iteration; Algorithm 4 stays below its bound
        kw.update(evolution=spff.EVOL_TIME if case["alg"] == 3 else spff.EVOL_NEAR_EQ, eta=0.5, dt_max=1.0, dt_min=1e-3,
                  dphi_max=1e30, dphi_min=1e30, fphi_max=1e6, drive_threshold=1e6, deps_max=1e-3)
    return spff.default_config(**kw)


CRACK_CG, CRACK_BCCG = 20, 12
#: the load of the checkpoint that a step starts from
BEFORE = 0.97


def prepare(case, seed):
    kind = case["kind"]
    if kind == "serve":
        probs = _serve_problems(case, seed)
        px = sum(E.numel() for _, E in probs)
        sv = spff.Server(px * 4 * 6 + (160 << 20) + px * 4 * 14, ticks_per_sync=case["ticks"], use_graph=1,
                         device=DEVICE)
        ids = [sv.register(_config(c), E.to(DEVICE)) for c, E in probs]
        return dict(case=case, server=sv, ids=ids, loads=[_strain(case, BEFORE), _strain(case)])
    if kind == "operator":
        E = torch.ones((case["batch"], case["ny"], case["nx"]), dtype=_real(case), device=DEVICE)
        return dict(case=case, problem=spff.Problem(E, _config(case)), x=_operand(case, seed).to(DEVICE))
    E = _moduli(case, seed).to(DEVICE)
    cfg = _config(case)
    if kind == "static":
        return dict(case=case, cfg=cfg, E=E[0].contiguous(), eps=_strain(case),
                    state=torch.zeros((5, case["ny"], case["nx"]), dtype=_real(case), device=DEVICE))
    p = spff.Problem(E, cfg)
    if case["tuned"]:
        plans, _, _ = autotune.tune(case["nx"], case["ny"], case["batch"])
        autotune.apply(p, plans)
    s = dict(case=case, problem=p)
    if kind == "crack":
        st = torch.zeros((case["batch"], 5, case["ny"], case["nx"]), dtype=_real(case), device=DEVICE)
        st[:, 3] = st[:, 4] = _crack(case).to(DEVICE)
        return dict(s, state=st, eps0=np.zeros(3), eps=_strain(case))
    if kind == "evolve":
        st = torch.zeros((case["batch"], 5, case["ny"], case["nx"]), dtype=_real(case), device=DEVICE)
        return dict(s, state=st, eps0=_strain(case), deps=_strain(case, 0.05))
    p.load_step(_strain(case, BEFORE))
    if kind == "fields":
        return s
    st, eps0 = p.get_state()
    ramp = np.stack([_strain(case, 1 + 0.03 * k) for k in range(case["steps"])])
    return dict(s, state=st, eps0=eps0, eps=_strain(case), ramp=ramp)


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------
STEP_FIELDS = spff.FIELD_PHI | spff.FIELD_STRAIN | spff.FIELD_STRESS


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "serve":
        sv = state["server"]
        tickets = [sv.submit(i, eps) for i in state["ids"] for eps in state["loads"]]
        while sv.progress(1)[1]:
            pass
        for t in tickets:
            sv.poll(t)
        return [sv.get_fields(i, spff.FIELD_PHI | spff.FIELD_EPS_STAR) for i in state["ids"]]
    if kind == "static":
        st = state["state"].clone()
        spff.load_step_static(state["cfg"], state["E"], st, state["eps"])
        return {"state": st}
    p = state["problem"]
    if kind == "operator":
        return {"out": p.apply_operator(OPS[case["op"]], state["x"])}
    if kind == "fields":
        return p.get_fields(ALL_FIELDS)
    p.set_state(state["state"], state["eps0"])
    if kind == "evolve":
        p.run_evolution(state["deps"], nsteps=case["steps"])
    elif kind == "sequence":
        p.run_sequence(state["ramp"])
    else:
        p.load_step(state["eps"])
    return p.get_fields(STEP_FIELDS)


# ---------------------------------------------------------------------------
# Bytes and operations of one pass
# ---------------------------------------------------------------------------
def _iterations(case):
    """(CG, BCCG) iterations of a pass over one problem, as such cases take
    them at the default tolerances."""
    if case["kind"] == "crack":
        return 2 * CRACK_CG, 2 * CRACK_BCCG
    cg = (4 if case["split"] == "none" else 6) + int(40 * case["amp"])
    cg, bccg = (cg, 0) if case["at"] == 1 else (2 * cg, 15)
    if case["kind"] in ("evolve", "sequence"):
        return cg * case["steps"], bccg * case["steps"]
    return (2 * cg, 2 * bccg) if case["kind"] == "serve" else (cg, bccg)


def work(case):
    r = 8 if case["fp64"] else 4
    if case["kind"] == "serve":
        px = sum(min(128 << (i % 4), case["nx"]) ** 2 for i in range(case["batch"]))
    else:
        px = case["nx"] * case["ny"] * case["batch"]
    fft = 2.5 * math.log2(case["nx"] * case["ny"])  # operations of one real transform, per pixel
    if case["kind"] == "operator":
        pin, pout = {"project": (3, 3), "laplacian": (1, 1), "displacement": (3, 2)}[case["op"]]
        return {"bytes": float(px * r * (pin + pout)), "flops": px * (fft * (pin + pout) + 10)}
    if case["kind"] == "fields":
        # E, phi, phi_ref and eps* in; 14 planes out; a transform for u*
        return {"bytes": float(px * r * (6 + 14)), "flops": px * (fft * 5 + 60)}
    cg, bccg = _iterations(case)
    # a CG iteration: E, phi, the strain, r, p and theta in, r, p and theta
    # out, three transforms each way; a BCCG iteration: phi, phi_ref, r, p, d
    # and b in, phi, r and p out, two transforms forward and one back
    return {"bytes": float(px * r * (23 * cg + 9 * bccg + 20)),
            "flops": px * (cg * (6 * fft + 100) + bccg * (3 * fft + 30) + 100)}


# ---------------------------------------------------------------------------
# The same outputs in 64 bits, from plain torch
# ---------------------------------------------------------------------------
class _Exact:
    """The published method on one grid, in 64 bits: Newton-CG on the
    projected equilibrium and bound-constrained CG for the phase field."""

    def __init__(self, case, E, tol=1e-11):
        dev = DEVICE if torch.cuda.is_available() else "cpu"
        self.E = E.to(dev, torch.float64)
        self.case, self.tol = case, tol
        ny, nx = self.E.shape
        self.shape = (ny, nx)
        qy = torch.fft.fftfreq(ny, dtype=torch.float64, device=dev)[:, None]
        qx = torch.fft.rfftfreq(nx, dtype=torch.float64, device=dev)[None, :]
        self.lap = (2 * math.pi) ** 2 * (qx * qx + qy * qy)
        gy, gx = qy.expand(ny, nx // 2 + 1).clone(), qx.expand(ny, nx // 2 + 1).clone()
        gy[ny // 2] = 0
        gx[:, nx // 2] = 0
        self.gx, self.gy, self.g2 = gx, gy, gx * gx + gy * gy
        self.inv = torch.where(self.g2 > 0, 1 / torch.where(self.g2 > 0, self.g2, torch.ones_like(self.g2)),
                               torch.zeros_like(self.g2))
        self.lam = NU / (1 - NU - 2 * NU * NU) * self.E
        self.mu = self.E / (2 + 2 * NU)
        self.contact = case["split"] if case["contact"] == "same" else case["contact"]
        cw = 8 / 3 if case["at"] == 1 else 2.0
        self.cwl, self.kappa = 1 / (cw * case["ell"]), 2 * case["ell"] / cw

    def project(self, s):
        h = torch.fft.rfft2(s)
        txx, tyy, txy = self.gy ** 2 * self.inv, self.gx ** 2 * self.inv, -self.gx * self.gy * self.inv
        d = txx * h[0] + tyy * h[1] + 2 * txy * h[2]
        live = (self.g2 > 0).to(torch.float64)
        out = torch.stack([live * (h[0] - d * txx), live * (h[1] - d * tyy), live * (h[2] - d * txy)])
        return torch.fft.irfft2(out, s=self.shape)

    def neg_lap(self, x):
        return torch.fft.irfft2(self.lap * torch.fft.rfft2(x), s=self.shape)

    def displacement(self, e):
        h = torch.fft.rfft2(e)
        gx, gy = self.gx, self.gy
        ex, ey = h[0] * gx + h[2] * gy, h[2] * gx + h[1] * gy
        s = (gx * ex + gy * ey) * self.inv
        u = torch.stack([(2 * ex - gx * s), (2 * ey - gy * s)]) * self.inv * (-1j / (2 * math.pi))
        return torch.fft.irfft2(u, s=self.shape)

    # -- constitutive law: (xx, yy, xy) planes ---------------------------
    def _parts(self, e, split):
        """psi+ and sigma+, sigma- of the undamaged material."""
        lam, mu = self.lam, self.mu
        tr = e[0] + e[1]
        one = torch.stack([torch.ones_like(tr), torch.ones_like(tr), torch.zeros_like(tr)])
        dd = e[0] ** 2 + e[1] ** 2 + 2 * e[2] ** 2
        if split == "none":
            return 0.5 * lam * tr * tr + mu * dd, lam * tr * one + 2 * mu * e, torch.zeros_like(e)
        tp, tm = tr.clamp(min=0), tr.clamp(max=0)
        if split == "voldev":
            K = lam + 2 * mu / 3
            return (0.5 * K * tp * tp + mu * (dd - tr * tr / 3), (K * tp - 2 * mu * tr / 3) * one + 2 * mu * e,
                    K * tm * one)
        e1, e2, n = self._eigen(e)
        p1, p2, m1, m2 = e1.clamp(min=0), e2.clamp(min=0), e1.clamp(max=0), e2.clamp(max=0)
        D = torch.stack([n[0], -n[0], n[1]])
        part = lambda t, a, b: lam * t * one + mu * ((a + b) * one + (a - b) * D)  # noqa: E731
        return 0.5 * lam * tp * tp + mu * (p1 * p1 + p2 * p2), part(tp, p1, p2), part(tm, m1, m2)

    @staticmethod
    def _eigen(e):
        """Eigenvalues and the unit deviator (D / r) of a symmetric 2 x 2."""
        m, d = 0.5 * (e[0] + e[1]), 0.5 * (e[0] - e[1])
        r = torch.sqrt(d * d + e[2] * e[2])
        safe = torch.where(r > 0, r, torch.ones_like(r))
        return m + r, m - r, torch.stack([torch.where(r > 0, d / safe, torch.ones_like(r)), e[2] / safe])

    def stress(self, e, phi):
        _, sp, sm = self._parts(e, self.contact)
        return (1 - phi) ** 2 * sp + sm

    def tangent(self, e, p, phi):
        """d stress(e, phi) along p."""
        hk, lam, mu = (1 - phi) ** 2, self.lam, self.mu
        tr, dtr = e[0] + e[1], p[0] + p[1]
        one = torch.stack([torch.ones_like(tr), torch.ones_like(tr), torch.zeros_like(tr)])
        if self.contact == "none":
            return hk * (lam * dtr * one + 2 * mu * p)
        ramp = torch.where(tr > 0, hk, (tr < 0).to(hk))  # ramps have no slope at 0
        if self.contact == "voldev":
            K = lam + 2 * mu / 3
            return (ramp * K * dtr - hk * 2 * mu * dtr / 3) * one + hk * 2 * mu * p
        # in the eigenbasis: each eigenvalue carries hk if it is positive,
        # and the shear between the two the divided difference
        e1, e2, n = self._eigen(e)
        w1, w2 = (torch.where(v > 0, hk, (v < 0).to(hk)) for v in (e1, e2))
        gap = e1 - e2
        w12 = torch.where(gap > 1e-300, (w1 * e1 - w2 * e2) / torch.where(gap > 1e-300, gap, torch.ones_like(gap)),
                          0.5 * (w1 + w2))
        dd = 0.5 * (p[0] - p[1])
        along, across = n[0] * dd + n[1] * p[2], n[0] * p[2] - n[1] * dd
        d1, d2 = w1 * (0.5 * dtr + along), w2 * (0.5 * dtr - along)
        s, q = d1 + d2, d1 - d2
        D, T = torch.stack([n[0], -n[0], n[1]]), torch.stack([-n[1], n[1], n[0]])
        return lam * ramp * dtr * one + mu * (s * one + q * D + 2 * w12 * across * T)

    # -- sub-problems ------------------------------------------------------
    @staticmethod
    def dot(a, b):
        return float((a[0] * b[0]).sum() + (a[1] * b[1]).sum() + 2 * (a[2] * b[2]).sum())

    def mechanics(self, eps, eb, phi, max_newton=60, max_cg=100000):
        bar = torch.tensor(eb, dtype=torch.float64, device=eps.device)[:, None, None]
        target = None
        for it in range(max_newton + 1):
            R = self.project(self.stress(bar + eps, phi))
            res = math.sqrt(self.dot(R, R))
            if target is None:
                h = self.stress(bar + torch.zeros_like(eps), phi)
                target = self.tol * max(math.sqrt(self.dot(h, h)), res)
            if res <= target or it == max_newton:
                break
            inner = target if self.contact == "none" else max(0.1 * res, target)
            th, r = torch.zeros_like(eps), -R
            p, rr = r, self.dot(r, r)
            for _ in range(max_cg):
                q = self.project(self.tangent(bar + eps, p, phi))
                pq = self.dot(p, q)
                if pq <= 0:
                    break
                a = rr / pq
                th, r = th + a * p, r - a * q
                new = self.dot(r, r)
                p, rr = r + (new / rr) * p, new
                if math.sqrt(rr) <= inner:
                    break
            eps = eps + th
        return eps

    def phase(self, eps, eb, phi, ref, eta_dt=0.0, max_it=100000):
        bar = torch.tensor(eb, dtype=torch.float64, device=eps.device)[:, None, None]
        pp = self._parts(bar + eps, self.case["split"])[0]
        d = 2 * pp + (2 * self.cwl if self.case["at"] == 2 else 0.0) + eta_dt
        b = 2 * pp - (self.cwl if self.case["at"] == 1 else 0.0) + eta_dt * ref
        lo = ref if self.case["damage"] else torch.where(ref >= 0.9, ref, torch.zeros_like(ref))
        J = lambda x: d * x + self.kappa * self.neg_lap(x)  # noqa: E731

        def residual(x):
            r = J(x) - b
            act = ((x <= lo) & (r > 0)) | ((x >= 1) & (r < 0))
            return torch.where(act, torch.zeros_like(r), r), act

        x = torch.minimum(torch.maximum(phi, lo), torch.ones_like(phi))
        r, act = residual(x)
        target = self.tol * max(float(b.norm()), float(r.norm()))
        p, best, since = -r, float("inf"), 0
        for _ in range(max_it):
            n = float(r.norm())
            best, since = (n, 0) if n < best else (best, since + 1)
            if n <= target or since > 50:
                break
            p = torch.where(act, torch.zeros_like(p), p)
            pq = float((p * J(p)).sum())
            if pq <= 0:
                break
            a = -float((r * p).sum()) / pq
            x = torch.minimum(torch.maximum(x + a * p, lo), torch.ones_like(x))
            old = r
            r, act = residual(x)
            p = -r + (float((r * (r - old)).sum()) / (a * pq)) * p
        return x

    def step(self, eps, phi, eb, max_am=1000, **caps):
        ref = phi
        mech = {k: v for k, v in caps.items() if k in ("max_newton", "max_cg")}
        pf = {k: v for k, v in caps.items() if k == "max_it"}
        for _ in range(max_am):
            eps = self.mechanics(eps, eb, phi, **mech)
            new = self.phase(eps, eb, phi, ref, **pf)
            moved, phi = float((new - phi).abs().sum()), new
            if moved <= 1e-3 * self.case["ell"] ** 2:
                break
        return eps, phi, ref


def exact(case, seed):
    kind = case["kind"]
    zero = lambda s: torch.zeros((3,) + s.shape, dtype=torch.float64, device=s.E.device)  # noqa: E731
    if kind == "operator":
        s = _Exact(case, torch.ones(case["ny"], case["nx"]))
        f = {"project": s.project, "laplacian": s.neg_lap, "displacement": s.displacement}[case["op"]]
        return {"out": torch.stack([f(x.to(s.E)) for x in _operand(case, seed)])}
    if kind == "serve":
        out = []
        for c, E in _serve_problems(case, seed):
            s = _Exact(c, E)
            eps, phi, ref = s.step(zero(s), torch.zeros_like(s.E), _strain(case, BEFORE))
            eps, phi, ref = s.step(eps, phi, _strain(case))
            out.append({"phi": phi[None], "eps_star": eps})
        return out
    outs = []
    for b, E in enumerate(_moduli(case, seed)):
        s = _Exact(case, E, tol=1e-6 if kind == "crack" else 1e-11)
        eps, phi, eb = zero(s), torch.zeros_like(s.E), _strain(case)
        if kind == "crack":
            eps, phi, ref = s.step(eps, _crack(case)[b].to(s.E), eb, max_am=2, max_newton=1, max_cg=CRACK_CG,
                                   max_it=CRACK_BCCG)
        elif kind == "evolve":
            for _ in range(case["steps"]):
                eb = eb + _strain(case, 0.05)
                eps = s.mechanics(eps, eb, phi)
                phi = s.phase(eps, eb, phi, phi, eta_dt=0.5)
        else:
            ramp = [_strain(case)]
            if kind == "fields":
                ramp = [_strain(case, BEFORE)]
            elif kind == "sequence":
                ramp = [_strain(case, 1 + 0.03 * k) for k in range(case["steps"])]
            # from zero to the checkpoint's load, then the steps of the pass
            if kind in ("step", "sequence") and case["at"] == 2:
                eps, phi, _ = s.step(eps, phi, _strain(case, BEFORE))
            for eb in ramp if case["at"] == 2 else ramp[-1:]:
                eps, phi, ref = s.step(eps, phi, eb)
        bar = torch.tensor(eb, dtype=torch.float64, device=eps.device)[:, None, None]
        if kind == "static":
            return {"state": torch.cat([eps, phi[None], ref[None]])}
        o = {"phi": phi[None], "strain": bar + eps, "stress": s.stress(bar + eps, phi)}
        if kind == "fields":
            o.update(phi_ref=ref[None], eps_star=eps, psi_plus=s._parts(bar + eps, case["split"])[0][None],
                     disp=s.displacement(eps))
        outs.append(o)
    return {k: torch.stack([o[k] for o in outs]) for k in outs[0]}
