"""What a user of the solver has it do, as cases that can be timed: Euler
steps from the smallest mesh to 4096 x 4096 and 192^3 nodes, in FP64 and the
mixed precisions, stepped one call at a time, asynchronously, as a pack and
through the server, with slip and non-reflecting walls, and the
Navier-Stokes steps with both preconditioners.

A pass sets a state, steps it and reads the new state back, on device
buffers where the interface takes them (packs and the server take host
arrays).  `exact` is the same scheme written down once more in plain torch
FP64, slot by slot over whole arrays.
"""
import math
import time

import numpy as np
import torch

from paper_2106_02159_amd import abi
from paper_2106_02159_amd.workloads import Mesh

GAMMA = 1.4
CFL = 0.5
PREC = {"fp64": abi.PREC_FP64, "mixed": abi.PREC_MIXED, "mixed_fp32": abi.PREC_MIXED_FP32}


# ---------------------------------------------------------------------------
# The cases.
# ---------------------------------------------------------------------------
def listed():
    return [
        # one step of the smallest mesh of the serving workload: launches and
        # their latency are all there is
        dict(name="euler2d_64_vortex", kind="step", flow="vortex", nx=64, ny=64, prec="fp64",
             steps=1),
        # the vortex leaving through non-reflecting faces (80 x 80 in the
        # tests), a short run of single steps on a small odd mesh
        dict(name="euler2d_97x83_open", kind="open", flow="stream", nx=97, ny=83, prec="fp64",
             steps=3),
        # a small mesh stepped asynchronously, as a program that looks at the
        # state now and then does
        dict(name="euler2d_256_async", kind="async", flow="quadrants", nx=256, ny=256,
             prec="fp64", steps=8),
        # an ordinary mesh of ragged size (rows that are no multiple of the
        # wavefront), slip walls
        dict(name="euler2d_1001x1003", kind="step", flow="quadrants", nx=1001, ny=1003,
             prec="fp64", steps=2),
        # the headline workload of the benchmark
        dict(name="euler2d_4096", kind="step", flow="quadrants", nx=4096, ny=4096, prec="fp64",
             steps=2),
        # FP32 storage and FP32 evaluation of the viscosity, periodic in x
        dict(name="euler2d_2048_fp32eval", kind="step", flow="quadrants", nx=2048, ny=2048,
             prec="mixed_fp32", steps=2, perx=True),
        # the 3D shock tube, the large 3D workload
        dict(name="euler3d_192", kind="step", flow="tube", nx=192, ny=192, nz=192, prec="fp64",
             steps=1),
        # the same flow on an odd mesh with FP32 storage
        dict(name="euler3d_101x67x83_mixed", kind="step", flow="tube", nx=101, ny=67, nz=83,
             prec="mixed", steps=2),
        # Navier-Stokes: a Strang step of the viscous shock tube
        dict(name="strang3d_128", kind="strang", flow="tube", nx=128, ny=128, nz=128,
             prec="fp64", steps=1, mu=1e-4, pc="jacobi"),
        # a viscous-dominated parabolic step: multigrid-preconditioned solves
        dict(name="parabolic2d_501x400_gmg", kind="parabolic", flow="smooth", nx=501, ny=400,
             prec="fp64", steps=1, mu=1.0, dt=5e-3, pc="gmg"),
        # many small simulations advanced by shared launches
        dict(name="pack2d_24", kind="pack", flow="quadrants", count=24, nmin=48, nmax=200,
             prec="fp64", steps=4),
        # the server: a burst of independent requests, packed and streamed
        dict(name="serve2d_12", kind="serve", flow="quadrants", count=12, nmin=64, nmax=400,
             prec="fp64", steps=12),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step3", "step3", "open", "async", "strang",
                       "parabolic", "pack", "serve"])
    prec = rng.choice(["fp64", "fp64", "mixed", "mixed_fp32"])
    if kind in ("step", "async"):
        nx, ny = _log_int(rng, 33, 3000), _log_int(rng, 33, 3000)
        flow = rng.choice(["quadrants", "quadrants", "vortex"])
        c = dict(kind=kind, flow=flow, nx=nx, ny=ny, prec=prec, steps=rng.randint(1, 3))
        if flow == "quadrants":
            c["perx"] = rng.random() < 0.25
        if kind == "async":
            c.update(prec=rng.choice(["fp64", "mixed"]), steps=rng.randint(2, 10),
                     nx=min(nx, 700), ny=min(ny, 700))
        return c
    if kind == "step3":
        n = [_log_int(rng, 17, 150) for _ in range(3)]
        return dict(kind="step", flow="tube", nx=n[0], ny=n[1], nz=n[2], prec=prec,
                    steps=rng.randint(1, 2))
    if kind == "open":
        return dict(kind="open", flow="stream", nx=_log_int(rng, 40, 700),
                    ny=_log_int(rng, 40, 700), prec=rng.choice(["fp64", "mixed"]),
                    steps=rng.randint(1, 3))
    if kind == "strang":
        n = [_log_int(rng, 17, 110) for _ in range(3)]
        return dict(kind="strang", flow="tube", nx=n[0], ny=n[1], nz=n[2], prec="fp64", steps=1,
                    mu=rng.choice([1e-4, 1e-3]), pc="jacobi")
    if kind == "parabolic":
        pc = rng.choice(["gmg", "jacobi"])
        return dict(kind="parabolic", flow="smooth", nx=_log_int(rng, 65, 700),
                    ny=_log_int(rng, 65, 700), prec="fp64", steps=1,
                    mu=1.0 if pc == "gmg" else 1e-3, dt=5e-3, pc=pc)
    if kind == "pack":
        return dict(kind="pack", flow="quadrants", count=rng.randint(6, 30),
                    nmin=rng.randint(33, 64), nmax=rng.randint(90, 220),
                    prec=rng.choice(["fp64", "mixed"]), steps=rng.randint(1, 5))
    return dict(kind="serve", flow="quadrants", count=rng.randint(4, 14),
                nmin=rng.randint(40, 90), nmax=rng.randint(150, 420),
                prec=rng.choice(["fp64", "mixed"]), steps=rng.randint(4, 12))


# ---------------------------------------------------------------------------
# Meshes and initial data, from the case and the seed alone.
# ---------------------------------------------------------------------------
def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _mesh(case, nx=None, ny=None):
    nx, ny = nx or case["nx"], ny or case["ny"]
    if case["flow"] == "tube":
        return Mesh(3, (nx, ny, case["nz"]), (0.0,) * 3, (1.0,) * 3, (False,) * 3)
    if case["flow"] == "vortex":
        return Mesh(2, (nx, ny), (-5.0, -5.0), (5.0, 5.0), (True, True))
    if case["flow"] == "stream":
        return Mesh(2, (nx, ny), (-1.0, -1.0), (1.0, 1.0), (False, False))
    return Mesh(2, (nx, ny), (0.0, 0.0), (1.0, 1.0), (bool(case.get("perx")), False))


def _member_sizes(case):
    """Sizes spread evenly over their logarithm, in a shuffled order."""
    lo, hi = math.log(case["nmin"]), math.log(case["nmax"])
    n = [int(round(math.exp(lo + (hi - lo) * (k + 0.5) / case["count"])))
         for k in range(case["count"])]
    return [n[k] for k in np.random.default_rng(case["count"]).permutation(case["count"])]


FAR = (1.0, 1.0, 0.0, 4.0 / 1.4)  # rho, u, v, p of the stream (Mach 1/2)


def _conserved(rho, vel, p):
    ke = sum(v * v for v in vel) * 0.5 * rho
    return torch.stack([rho] + [rho * v for v in vel] + [p / (GAMMA - 1.0) + ke])


def _state(flow, mesh, seed):
    """(nc, nz, ny, nx) FP64 initial state on the device."""
    r = np.random.default_rng(seed)
    dev = _device()
    h = mesh.spacing()
    ax = [torch.arange(mesh.n[d], dtype=torch.float64, device=dev) * h[d] + mesh.lo[d]
          for d in range(mesh.dim)]
    X = list(torch.meshgrid(*ax[::-1], indexing="ij"))[::-1]

    def waves(amp, count=3):
        """A sum of smooth waves that fit the box, |.| <= amp."""
        s = torch.zeros_like(X[0])
        for _ in range(count):
            t = torch.ones_like(X[0])
            for d in range(mesh.dim):
                k = int(r.integers(1, 4))
                w = 2.0 * math.pi * k / (mesh.hi[d] - mesh.lo[d])
                t = t * torch.sin(w * (X[d] - mesh.lo[d]) + float(r.uniform(0, 2 * math.pi)))
            s = s + t
        return s * (amp / count)

    if flow == "vortex":  # a travelling isentropic vortex
        beta, x0, y0 = r.uniform(3, 5), r.uniform(-2, 2), r.uniform(-2, 2)
        dx = torch.remainder(X[0] - x0 + 5.0, 10.0) - 5.0
        dy = torch.remainder(X[1] - y0 + 5.0, 10.0) - 5.0
        e = torch.exp(0.5 * (1.0 - dx * dx - dy * dy))
        f = beta / (2 * math.pi) * e
        T = 1.0 - (GAMMA - 1.0) * beta ** 2 / (8 * GAMMA * math.pi ** 2) * e * e
        rho = T ** (1.0 / (GAMMA - 1.0))
        return _conserved(rho, (1.0 - f * dy, 1.0 + f * dx), rho ** GAMMA)
    if flow == "stream":  # a vortex in a uniform stream, near the outflow
        r0, vb = 0.25, float(r.uniform(0.25, 0.75))
        x, y = X[0] - float(r.uniform(0.3, 0.7)), X[1] - float(r.uniform(-0.3, 0.3))
        psi = torch.exp(0.5 * (1.0 - (x * x + y * y) / r0 ** 2))
        one = torch.ones_like(x)
        return _conserved(one, (FAR[1] - vb / r0 * psi * y, vb / r0 * psi * x),
                          FAR[3] - 0.5 * (vb * psi) ** 2)
    if flow == "smooth":
        return _conserved(1.0 + waves(0.3), (waves(0.3), waves(0.3)), 1.0 + waves(0.3))
    if flow == "quadrants":  # four constant states and smooth waves on them
        q = []
        for _ in range(4):
            q.append((math.exp(r.uniform(math.log(0.1), math.log(2.0))), r.uniform(-1, 1),
                      r.uniform(-1, 1), r.uniform(0.05, 1.0)))
        at = (X[0] >= 0.5).long() + 2 * (X[1] >= 0.5).long()
        st = torch.tensor(q, dtype=torch.float64, device=dev)
        v = [st[:, k][at] for k in range(4)]
        return _conserved(v[0] * (1.0 + waves(0.05)), (v[1] + waves(0.02), v[2] + waves(0.02)),
                          v[3] * (1.0 + waves(0.05)))
    # Mach-3 shock tube along x, 1% density noise
    g, m2 = GAMMA, 9.0
    rho2, p2 = 1.4 * (g + 1) * m2 / ((g - 1) * m2 + 2), (2 * g * m2 - (g - 1)) / (g + 1)
    post = X[0] < 0.25
    full = lambda a, b: torch.where(post, torch.full_like(X[0], a), torch.full_like(X[0], b))
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed))
    noise = torch.rand(X[0].shape, dtype=torch.float64, device=dev, generator=gen) * 2.0 - 1.0
    zero = torch.zeros_like(X[0])
    return _conserved(full(rho2, 1.4) * (1.0 + 0.01 * noise),
                      (full(3.0 * (1.0 - 1.4 / rho2), 0.0), zero, zero), full(p2, 1.0))


def _far_state():
    return [FAR[0], FAR[0] * FAR[1], FAR[0] * FAR[2],
            FAR[3] / (GAMMA - 1.0) + 0.5 * FAR[0] * (FAR[1] ** 2 + FAR[2] ** 2)]


def _viscous(case):
    return dict(mu=case["mu"], lam=0.0, kappa=1.4 * case["mu"], cv=2.5, cg_rtol=1e-10,
                cg_maxit=2000,
                precond=abi.PC_GMG if case["pc"] == "gmg" else abi.PC_JACOBI)


# ---------------------------------------------------------------------------
def prepare(case, seed):
    prec = PREC[case["prec"]]
    if case["kind"] in ("pack", "serve"):
        meshes = [_mesh(case, n, n) for n in _member_sizes(case)]
        U = [_state(case["flow"], m, seed + 7 * k).reshape(4, -1).cpu().numpy()
             for k, m in enumerate(meshes)]
        if case["kind"] == "pack":
            pack = abi.Pack([abi.Graph(m) for m in meshes], cfl=CFL, precision=prec)
            return dict(case=case, pack=pack, U=U)
        server = abi.Server(64 << 30, max_running=8, cfl=CFL, precision=prec, chunk=2, depth=2,
                            pack_nodes=1 << 17, pack_max=64)
        return dict(case=case, server=server, meshes=meshes, U=U)
    mesh = _mesh(case)
    solver = abi.Solver(abi.Graph(mesh), cfl=CFL, precision=prec)
    if case["kind"] == "open":
        solver.set_boundary([abi.BC_NONREFLECTING] * 4, abi.NR_CHARACTERISTIC,
                            [_far_state()] * 4)
    if case["kind"] in ("strang", "parabolic"):
        solver.set_viscous(**_viscous(case))
    U = _state(case["flow"], mesh, seed).reshape(mesh.dim + 2, -1).contiguous()
    out = torch.empty_like(U)
    if U.is_cuda:
        torch.cuda.synchronize()
    return dict(case=case, solver=solver, U=U, out=out)


def run(state):
    case = state["case"]
    kind, steps = case["kind"], case["steps"]
    if kind == "pack":
        pack, n = state["pack"], len(state["U"])
        for k in range(n):
            pack.set_state(k, state["U"][k])
        pack.step_cfl_async(steps)
        status, t = pack.finish()
        return dict(U=[pack.get_state(k) for k in range(n)], t=t, status=status)
    if kind == "serve":
        sv = state["server"]
        ids = [sv.submit(m, U, steps) for m, U in zip(state["meshes"], state["U"])]
        done = 0
        while done < len(ids):
            done += sv.progress()
            if done < len(ids):
                time.sleep(2e-4)
        t = [sv.request(i).t_sim for i in ids]
        res = [sv.result(i) for i in ids]
        return dict(U=[u for u, _ in res], t=t, status=[s for _, s in res])
    s, out = state["solver"], state["out"]
    s.set_state_device(state["U"].data_ptr())
    if kind == "async":
        s.step_cfl_async(steps)
        status, t = s.async_finish()
        s.get_state_device(out.data_ptr())
        return dict(U=out, t=t, status=status)
    t = []
    for _ in range(steps):
        if kind == "strang":
            t.append(s.step_strang_cfl())
        elif kind == "parabolic":
            s.step_parabolic(case["dt"])
        else:
            t.append(s.step_cfl())
    s.get_state_device(out.data_ptr())
    return dict(U=out, t=t)


def work(case):
    """Per stage the state in and out, U^n in two of three stages, and the
    arithmetic of the 3^d-point scheme; a parabolic step: its vectors once
    per solve."""
    dim = 3 if case["flow"] == "tube" else 2
    if case["kind"] in ("pack", "serve"):
        N = sum(n * n for n in _member_sizes(case))
    else:
        N = case["nx"] * case["ny"] * case.get("nz", 1)
    nc, W = dim + 2, 3 ** dim
    steps = case["steps"]
    hyp = {"strang": 2, "parabolic": 0}.get(case["kind"], 1) * steps
    par = steps if case["kind"] in ("strang", "parabolic") else 0
    stage_b, stage_f = nc * 8 * (2 + 2.0 / 3.0), W * (60 + 40 * nc)
    par_b, par_f = 8 * (2 * nc + 8 * dim + 8), 4 * W * (dim * dim + 1)
    return {"bytes": float(N) * (3 * hyp * stage_b + par * par_b),
            "flops": float(N) * (3 * hyp * stage_f + par * par_f)}


# ---------------------------------------------------------------------------
# The scheme in plain torch FP64.  Fields are (..., nz, ny, nx); slot o =
# (dx, dy, dz) of node i is the node at that offset.
# ---------------------------------------------------------------------------
class _Scheme:
    def __init__(self, mesh, open_far=None):
        self.dim, self.n, self.per, self.h = mesh.dim, mesh.n, mesh.periodic, mesh.spacing()
        self.nc, self.far = self.dim + 2, open_far
        dev, dim = _device(), self.dim
        self.offs = [tuple((k // 3 ** d) % 3 - 1 for d in range(dim)) for k in range(3 ** dim)]

        def along(d, v):  # a 1D array along direction d, broadcastable
            shape = [1] * dim
            shape[dim - 1 - d] = self.n[d]
            return torch.as_tensor(v, dtype=torch.float64, device=dev).reshape(shape)

        f1, c1, ok1, ml = [], [], [], []
        for d in range(dim):
            n, h = self.n[d], self.h[d]
            f, c, ok = {}, {}, {}
            for o in (-1, 0, 1):
                F = np.full(n, 2 * h / 3 if o == 0 else h / 6)
                G = np.full(n, 0.5 * o)
                K = np.ones(n)
                if not self.per[d]:
                    if o == 0:
                        F[0] = F[-1] = h / 3
                        G[0], G[-1] = -0.5, 0.5
                    else:
                        K[0 if o < 0 else -1] = 0
                f[o], c[o], ok[o] = along(d, F), along(d, G), along(d, K)
            f1.append(f), c1.append(c), ok1.append(ok)
            m = np.full(n, h)
            if not self.per[d]:
                m[0] = m[-1] = h / 2
            ml.append(along(d, m))
        prod = lambda v: math.prod(v[1:], start=v[0])
        shape = tuple(self.n[::-1])
        self.m = prod(ml).expand(shape).contiguous()
        self.mij = [prod([f1[d][o[d]] for d in range(dim)]) for o in self.offs]
        self.cij = [[prod([c1[e][o[e]] if d == e else f1[d][o[d]] for d in range(dim)])
                     for e in range(dim)] for o in self.offs]
        self.ok = [(prod([ok1[d][o[d]] for d in range(dim)]) > 0).expand(shape)
                   for o in self.offs]
        self.deg = sum(k.double() for k in self.ok) - 1.0
        self.rel = (self.m / self.m.sum()) ** (1.5 / dim)
        nrm = []  # int_{dOmega} phi_i n
        for d in range(dim):
            if self.per[d]:
                nrm.append(torch.zeros(shape, dtype=torch.float64, device=dev))
                continue
            s = np.zeros(self.n[d])
            s[0], s[-1] = -1.0, 1.0
            nrm.append((along(d, s) * prod([ml[e] for e in range(dim) if e != d])).expand(shape))
        nrm = torch.stack(nrm)
        ln = nrm.square().sum(0).sqrt()
        self.wall = ln > 0
        self.nrm = nrm / torch.where(self.wall, ln, torch.ones_like(ln))

    def sh(self, f, o):
        return torch.roll(f, [-o[d] for d in range(self.dim)], [-1 - d for d in range(self.dim)])

    def prim(self, U):
        v = U[1:-1] / U[0]
        e = U[-1] - 0.5 * U[0] * v.square().sum(0)
        return v, (GAMMA - 1.0) * e, e

    def flux(self, U, v, p, c):
        vc = sum(v[d] * c[d] for d in range(self.dim))
        return torch.stack([U[0] * vc] + [U[1 + d] * vc + p * c[d] for d in range(self.dim)] +
                           [(U[-1] + p) * vc])

    @staticmethod
    def lam(uL, pL, aL, uR, pR, aR):
        g, ex = GAMMA, (GAMMA - 1.0) / (2.0 * GAMMA)
        num = (aL + aR - 0.5 * (g - 1.0) * (uR - uL)).clamp_min(0.0)
        ps = (num / (aL * pL ** -ex + aR * pR ** -ex)) ** (1.0 / ex)
        cg = (g + 1.0) / (2.0 * g)
        l1 = uL - aL * torch.sqrt(1.0 + cg * (ps / pL - 1.0).clamp_min(0.0))
        l3 = uR + aR * torch.sqrt(1.0 + cg * (ps / pR - 1.0).clamp_min(0.0))
        return torch.maximum(-l1, l3).clamp_min(0.0)

    def viscosity(self, U):
        v, p, _ = self.prim(U)
        a = torch.sqrt(GAMMA * p / U[0])
        out = []
        for k, o in enumerate(self.offs):
            if not any(o):
                out.append(None)
                continue
            vj, pj, aj = self.sh(v, o), self.sh(p, o), self.sh(a, o)
            c = self.cij[k]
            # c_ji has the moved components reversed
            ct = [-c[d] if o[d] else c[d] for d in range(self.dim)]
            d = torch.zeros_like(p)
            for cc, L, R in ((c, (v, p, a), (vj, pj, aj)), (ct, (vj, pj, aj), (v, p, a))):
                cn = sum(x * x for x in cc).sqrt()
                un = [sum(s[0][e] * cc[e] for e in range(self.dim)) / cn for s in (L, R)]
                d = torch.maximum(d, self.lam(un[0], L[1], L[2], un[1], R[1], R[2]) * cn)
            out.append(torch.where(self.ok[k], d, torch.zeros_like(d)))
        return out

    def dt(self, U):
        d = sum(x for x in self.viscosity(U) if x is not None)
        return CFL * float((self.m / (2.0 * d)).min())

    def psi(self, u, P, l, pmin):
        w = u + l * P
        return w[-1] - 0.5 * w[1:-1].square().sum(0) / w[0] - pmin * w[0].clamp_min(0) ** GAMMA

    def search(self, u, P, rmin, rmax, pmin):
        Pr = P[0]
        one = torch.ones_like(Pr)
        l = torch.where(Pr > 0, (rmax - u[0]) / torch.where(Pr > 0, Pr, one),
                        torch.where(Pr < 0, (rmin - u[0]) / torch.where(Pr < 0, Pr, one), one))
        l = l.clamp(0.0, 1.0)
        bad = self.psi(u, P, l, pmin) < 0
        if bool(bad.any()):
            ub, Pb, pb, lb = u[:, bad], P[:, bad], pmin[bad], l[bad]
            lo, hi = torch.zeros_like(lb), lb.clone()
            for _ in range(60):
                mid = 0.5 * (lo + hi)
                f = self.psi(ub, Pb, mid, pb) >= 0
                lo, hi = torch.where(f, mid, lo), torch.where(f, hi, mid)
            l[bad] = torch.where(self.psi(ub, Pb, 0.0, pb) < 0, torch.zeros_like(lo), lo)
        return l

    def stage(self, U, tau):
        v, p, e = self.prim(U)
        rho = U[0]
        a = torch.sqrt(GAMMA * p / rho)
        s = torch.log(e) - GAMMA * torch.log(rho)
        eta, Phi = -rho * s, torch.exp(s)
        etap = torch.stack([GAMMA - s - U[1:-1].square().sum(0) / (2.0 * rho * e)] +
                           [U[1 + k] / e for k in range(self.dim)] + [-rho / e])
        num, den, scl = (torch.zeros_like(p) for _ in range(3))
        for k, o in enumerate(self.offs):
            c = self.cij[k]
            Uj, vj, pj = self.sh(U, o), self.sh(v, o), self.sh(p, o)
            t = self.sh(eta, o) * sum(vj[x] * c[x] for x in range(self.dim)) - \
                (etap * self.flux(Uj, vj, pj, c)).sum(0)
            t = torch.where(self.ok[k], t, torch.zeros_like(t))
            cn = sum(x * x for x in c).sqrt() * self.ok[k]
            num, den = num + t, den + t.abs()
            scl = scl + cn * self.sh(a, o) * (Uj[0] + self.sh(eta, o).abs())
        alpha = num.abs() / (den + 1e-2 * scl)
        d = self.viscosity(U)
        FH, UL = torch.zeros_like(U), U.clone()
        rmin, rmax, pmin = rho.clone(), rho.clone(), Phi.clone()
        for k, o in enumerate(self.offs):
            c, ok = self.cij[k], self.ok[k]
            Uj = self.sh(U, o)
            fj, fi = self.flux(Uj, self.sh(v, o), self.sh(p, o), c), self.flux(U, v, p, c)
            FH = FH - torch.where(ok, fj, torch.zeros_like(fj))
            if d[k] is None:
                continue
            dH = 0.5 * (alpha + self.sh(alpha, o)) * d[k]
            FH = FH + torch.where(ok, dH * (Uj - U), torch.zeros_like(fj))
            UL = UL + tau / self.m * torch.where(ok, d[k] * (Uj - U) - (fj - fi),
                                                 torch.zeros_like(fj))
            rb = 0.5 * (rho + Uj[0]) - (fj[0] - fi[0]) / (2.0 * torch.where(ok, d[k], d[k] + 1))
            rmin = torch.where(ok, torch.minimum(rmin, rb), rmin)
            rmax = torch.where(ok, torch.maximum(rmax, rb), rmax)
            pmin = torch.where(ok, torch.minimum(pmin, self.sh(Phi, o)), pmin)
        rmin, rmax, pmin = (1 - self.rel) * rmin, (1 + self.rel) * rmax, (1 - self.rel) * pmin
        Fm = FH / self.m

        def P(k):
            o = self.offs[k]
            dH = 0.5 * (alpha + self.sh(alpha, o)) * d[k]
            return tau * self.deg / self.m * (self.mij[k] * (Fm - self.sh(Fm, o)) +
                                              (dH - d[k]) * (self.sh(U, o) - U))

        W = len(self.offs)
        sym = lambda l, k: torch.minimum(l[k], self.sh(l[W - 1 - k], self.offs[k]))
        slots = [k for k in range(W) if d[k] is not None]
        l1 = {k: self.search(UL, P(k), rmin, rmax, pmin) for k in slots}
        V = UL.clone()
        for k in slots:
            V = V + torch.where(self.ok[k], sym(l1, k) * P(k) / self.deg, torch.zeros_like(V))
        l2 = {}
        for k in slots:
            r = 1.0 - sym(l1, k)
            l2[k] = self.search(V, r * P(k), rmin, rmax, pmin) * r
        out = V.clone()
        for k in slots:
            out = out + torch.where(self.ok[k], sym(l2, k) * P(k) / self.deg,
                                    torch.zeros_like(V))
        return out

    def post(self, U):
        """Slip projection, or the characteristic far-field post-processing."""
        if self.far is None:
            mn = (U[1:-1] * self.nrm).sum(0)
            return torch.cat([U[:1], U[1:-1] - mn * self.nrm, U[-1:]])
        g = GAMMA
        n = self.nrm
        D = torch.tensor(self.far, dtype=U.dtype, device=U.device).reshape(-1, 1, 1) + 0 * U

        def parts(X):
            v, p, _ = self.prim(X)
            vn = (v * n).sum(0)
            return X[0], vn, v - vn * n, p, torch.sqrt(g * p / X[0])

        (r, vn, vt, p, a), (rd, vnd, vtd, pd, ad) = parts(U), parts(D)
        inflow = vn < 0
        C1, C3 = vnd - 2 * ad / (g - 1), vn + 2 * a / (g - 1)
        S = torch.where(inflow, pd * rd ** -g, p * r ** -g)
        un, ap = 0.5 * (C1 + C3), 0.25 * (g - 1) * (C3 - C1)
        rr = (ap * ap / (g * S)) ** (1 / (g - 1))
        vv = torch.where(inflow, vtd, vt) + un * n
        X = _conserved(rr, [vv[k] for k in range(self.dim)], S * rr ** g)
        sup = a <= vn.abs()
        X = torch.where(sup & inflow, D, torch.where(sup & ~inflow, U, X))
        return torch.where(self.wall, X, U)

    def step(self, U, tau):
        w = self.post(self.stage(U, tau))
        w = self.post(0.75 * U + 0.25 * self.stage(w, tau))
        return self.post(U / 3.0 + 2.0 / 3.0 * self.stage(w, tau))

    # -- parabolic step ------------------------------------------------------
    def cells(self):
        """Gauss points of the reference cell: (weight, phi_a, grad phi_a),
        and the mask of the nodes that are the lowest corner of a cell."""
        dim, L = self.dim, 1 << self.dim
        pts = [0.5 - 0.5 / math.sqrt(3.0), 0.5 + 0.5 / math.sqrt(3.0)]
        q = []
        for k in range(L):
            x = [pts[(k >> d) & 1] for d in range(dim)]
            N1 = [(1 - x[d], x[d]) for d in range(dim)]
            phi = [math.prod(N1[d][(a >> d) & 1] for d in range(dim)) for a in range(L)]
            grad = [[(1 if (a >> e) & 1 else -1) / self.h[e] *
                     math.prod(N1[d][(a >> d) & 1] for d in range(dim) if d != e)
                     for e in range(dim)] for a in range(L)]
            q.append((math.prod(self.h) / L, phi, grad))
        has = self.ok[self.offs.index((1,) * dim)].double()
        corner = [tuple((a >> d) & 1 for d in range(dim)) for a in range(L)]
        return q, has, corner

    def parabolic(self, U, dt, mu, kappa, cv):
        dim = self.dim
        q, has, corner = self.cells()
        rho, m = U[0], self.m
        V0 = U[1:-1] / rho
        e0 = U[-1] / rho - 0.5 * V0.square().sum(0)
        free = (~self.wall).double()

        def gather(f):
            return [self.sh(f, c) * has for c in corner]

        def scatter(parts):
            return sum(self.sh(x * has, tuple(-t for t in c)) for x, c in zip(parts, corner))

        def stress(G):
            tr = sum(G[k][k] for k in range(dim))
            return [[mu * (G[k][j] + G[j][k]) - (2.0 / 3.0 * mu * tr if k == j else 0.0)
                     for j in range(dim)] for k in range(dim)]

        def grads(Vc, g):
            return [[sum(Vc[a][k] * g[a][j] for a in range(len(g))) for j in range(dim)]
                    for k in range(dim)]

        def A(V):
            Vc = gather(V)
            parts = [0.0] * len(corner)
            for w, _, g in q:
                S = stress(grads(Vc, g))
                for a in range(len(corner)):
                    parts[a] = parts[a] + w * torch.stack(
                        [sum(S[k][j] * g[a][j] for j in range(dim)) for k in range(dim)])
            return scatter(parts)

        def B(e):
            ec = gather(e)
            parts = [0.0] * len(corner)
            for w, _, g in q:
                ge = [sum(ec[a] * g[a][j] for a in range(len(g))) for j in range(dim)]
                for a in range(len(corner)):
                    parts[a] = parts[a] + (w * kappa / cv) * sum(ge[j] * g[a][j]
                                                                for j in range(dim))
            return scatter(parts)

        def solve(op, b, x, diag):
            r = b - op(x)
            z = r / diag
            p, rz, bb = z.clone(), float((r * z).sum()), float((b * b).sum())
            for _ in range(4000):
                if float((r * r).sum()) <= 1e-28 * bb:
                    break
                y = op(p)
                al = rz / float((p * y).sum())
                x, r = x + al * p, r - al * y
                z = r / diag
                new = float((r * z).sum())
                p, rz = z + (new / rz) * p, new
            return x

        hh = sum(1.0 / x ** 2 for x in self.h)  # about the operators' diagonal
        V = solve(lambda x: free * (rho * m * x + 0.5 * dt * A(x)) + (1 - free) * x,
                  free * m * U[1:-1], free * V0, rho * m + 2.0 * dt * mu * hh * m)
        K = 0.0
        Vc = gather(V)
        parts = [0.0] * len(corner)
        for w, phi, g in q:
            G = grads(Vc, g)
            S = stress(G)
            se = sum(S[k][j] * G[k][j] for k in range(dim) for j in range(dim))
            parts = [x + w * phi[a] * se for a, x in enumerate(parts)]
        K = scatter(parts) / m
        e = solve(lambda x: rho * m * x + 0.5 * dt * B(x), rho * m * e0 + 0.5 * dt * m * K, e0,
                  rho * m + 2.0 * dt * kappa / cv * hh * m)
        e, V = 2.0 * e - e0, free * (2.0 * V - V0)
        if float(e.min()) <= 0.0:
            return None  # the scheme limits such a step
        return torch.cat([U[:1], rho * V, (rho * e + 0.5 * rho * V.square().sum(0))[None]])


def _exact_run(case, mesh, U):
    """(state, times) of the case's steps, or None."""
    S = _Scheme(mesh, _far_state() if case["kind"] == "open" else None)
    if case["kind"] != "open":
        U = S.post(U)  # the state call projects the wall nodes
    visc = dict(mu=case.get("mu"), kappa=1.4 * case.get("mu", 0.0), cv=2.5)
    t = []
    for _ in range(case["steps"]):
        if case["kind"] == "parabolic":
            U = S.parabolic(U, case["dt"], **visc)
            if U is None:
                return None
            continue
        tau = S.dt(U)
        t.append(tau)
        U = S.step(U, tau)
        if case["kind"] == "strang":
            U = S.parabolic(U, 2.0 * tau, **visc)
            if U is None:
                return None
            U = S.step(U, tau)
    return U.reshape(mesh.dim + 2, -1), t


def exact(case, seed):
    if case["kind"] in ("pack", "serve"):
        sizes = _member_sizes(case)
        if sum(n * n for n in sizes) * case["steps"] > 4e6 * 3 or \
                case["count"] * case["steps"] > 150:
            return None
        U, T = [], []
        for k, n in enumerate(sizes):
            mesh = _mesh(case, n, n)
            u, t = _exact_run(case, mesh, _state(case["flow"], mesh, seed + 7 * k))
            U.append(u.cpu().numpy())
            T.append(sum(t))
        t = np.array(T) if case["kind"] == "pack" else T
        return dict(U=U, t=t, status=[0] * len(U))
    mesh = _mesh(case)
    got = _exact_run(case, mesh, _state(case["flow"], mesh, seed))
    if got is None:
        return None
    U, t = got
    if case["kind"] == "async":
        return dict(U=U, t=sum(t), status=0)
    return dict(U=U, t=t)
