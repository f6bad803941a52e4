"""Timed workloads of the split-form DGSEM operator, each through the Python
binding's public entry points (paper_2306_12891_amd.dg).

The listed cases are the workloads of bench.py and the two reverse-mode paths:

* Runge-Kutta steps (``rk_step``) of the box operator -- Euler, Navier-Stokes
  in FP64 and in mixed precision, with the Smagorinsky model, with
  wall-modelled faces, with the DG/FV blending -- and of the curved operator;
* the checkpointed reverse rollout (gradient of a trajectory with respect to
  its start state), and the operator with its vector-Jacobian product through
  autograd.

``draw`` spreads over the same families: every degree from 2 to 7, meshes from
a few elements to a few million nodes with odd and ragged sizes, and the
volume / surface flux pairs of each family.

A case is a dict: ``flow`` (which start state and options), ``N``, ``nx``,
``ny``, ``nz``, ``vf`` / ``sf`` (flux names), ``call`` (rk_step, rollout or
operator).  Start states are closed-form flows plus a smooth seeded
perturbation (and, where a developed solution would have them, small jumps
between elements).

``exact`` evaluates the same definitions with plain torch tensor operations in
64 bits: the split-form flux differencing node pair by node pair, BR1 with a
full gradient on every element, the subcell scheme, curl-form metrics; reverse
mode by torch.autograd.
"""
import math

import numpy as np
import torch

from paper_2306_12891_amd import dg

GAMMA, PR, PRT = 1.4, 0.72, 0.9
TWO_PI = 2.0 * math.pi
RK_A = [0.0, -567301805773.0 / 1357537059087.0, -2404267990393.0 / 2016746695238.0,
        -3550918686646.0 / 2091501179385.0, -1275806237668.0 / 842570457699.0]
RK_B = [1432997174477.0 / 9575080441755.0, 5161836677717.0 / 13612068292357.0,
        1720146321549.0 / 2090206949498.0, 3134564353537.0 / 4481467310338.0,
        2277821191437.0 / 14882151754819.0]
VOL = {"kg": dg.KG, "pi": dg.PI, "std": dg.STD}
SURF = {"llf": dg.LLF, "roe": dg.ROE}

# per flow: box, viscosity, CFL, further options
FLOWS = {
    "wave": dict(hi=(TWO_PI,) * 3, mu=0.0, cfl=0.5),
    "tgv": dict(hi=(TWO_PI,) * 3, mu=1.0 / 1600, cfl=0.5),
    "tgv_mixed": dict(hi=(TWO_PI,) * 3, mu=1.0 / 1600, cfl=0.5, precision=dg.MIXED),
    "tgv_les": dict(hi=(TWO_PI,) * 3, mu=1.0 / 1600, cfl=0.5, Cs=0.17),
    "tgv_curved": dict(hi=(TWO_PI,) * 3, mu=1.0 / 1600, cfl=0.35, warp=0.04),
    "channel": dict(hi=(TWO_PI, 2.0, math.pi), mu=2e-5, cfl=0.5, Cs=0.17, wall=1),
    "sod": dict(hi=(1.0, 0.125, 0.125), mu=0.0, cfl=0.4, blending=1),
    "sod_ns": dict(hi=(1.0, 0.125, 0.125), mu=2e-6, cfl=0.4, blending=1),
}
U_INF, MA_INF = 1.0, 0.7  # van Driest transformation of the wall model


def _case(name, flow, N, n, vf, sf, call="rk_step", **more):
    c = {"flow": flow, "N": N, "nx": n[0], "ny": n[1], "nz": n[2], "vf": vf, "sf": sf, "call": call}
    c.update(more)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: a density wave on 4^3 elements, a test-sized run bound by launches
        _case("wave_n3_4", "wave", 3, (4, 4, 4), "kg", "llf"),
        # inviscid production run, the smallest mesh of the size sweep
        _case("wave_n7_32", "wave", 7, (32, 32, 32), "kg", "llf"),
        # the headline workload of the benchmark: Taylor-Green vortex, 134 M nodes
        _case("tgv_n7_64", "tgv", 7, (64, 64, 64), "pi", "roe"),
        # the same flow at the resolution and degree of the paper's LES meshes
        _case("tgv_n5_32", "tgv", 5, (32, 32, 32), "pi", "roe"),
        # mixed-precision operator
        _case("tgv_mixed_n7_32", "tgv_mixed", 7, (32, 32, 32), "pi", "roe"),
        # Smagorinsky LES
        _case("tgv_les_n5_32", "tgv_les", 5, (32, 32, 32), "pi", "roe"),
        # curved elements
        _case("tgv_curved_n5_32", "tgv_curved", 5, (32, 32, 32), "pi", "roe"),
        # wall-modelled LES of a channel
        _case("channel_n5_32", "channel", 5, (32, 32, 32), "pi", "roe"),
        # shock tube: DG/FV blending, inviscid, a small launch-bound mesh
        _case("sod_n5_64x8x8", "sod", 5, (64, 8, 8), "kg", "llf"),
        # shock tube: DG/FV blending with the viscous terms, the degree of the paper's cascade LES
        _case("sod_ns_n4_256x16x16", "sod_ns", 4, (256, 16, 16), "kg", "llf"),
        # gradient of a trajectory: checkpointed rollout, forward and backward
        _case("rollout_n5_16", "tgv", 5, (16, 16, 16), "pi", "roe", "rollout", steps=6, every=3),
        # operator and its reverse product on a small ragged mesh
        _case("operator_n4_9x7x5", "tgv", 4, (9, 7, 5), "kg", "llf", "operator"),
    ]


def draw(rng):
    flow = rng.choice(["wave", "tgv", "tgv", "tgv_mixed", "tgv_les", "tgv_curved", "channel", "sod", "sod_ns",
                       "rollout", "operator"])
    call = "rk_step"
    most = 6e6
    more = {}
    if flow == "rollout":
        call, most = "rollout", 6e5
        flow = rng.choice(["tgv", "wave"])
        more = {"steps": rng.randint(2, 6), "every": rng.randint(1, 4)}
    elif flow == "operator":
        call, most = "operator", 2e6
        flow = rng.choice(["tgv", "tgv", "tgv_les", "tgv_curved", "wave"])
    N = rng.choice([2, 3, 4, 5, 6, 7])
    if flow in ("sod", "sod_ns"):
        vf, sf = "kg", "llf"
        most = min(most, 4e6)
    elif flow == "tgv_mixed":
        vf, sf = rng.choice([("pi", "roe"), ("pi", "llf"), ("std", "llf")])
    else:
        vf, sf = rng.choice([("pi", "roe"), ("pi", "llf"), ("kg", "llf"), ("kg", "roe"), ("std", "llf")])
    nodes = math.exp(rng.uniform(math.log(2e4), math.log(most)))
    elems = max(8.0, nodes / (N + 1) ** 3)
    if flow in ("sod", "sod_ns"):  # long tubes
        nt = max(2, round((elems / rng.uniform(8.0, 24.0)) ** (1 / 3)))
        n = (max(8, round(elems / nt ** 2)), nt, max(2, nt + rng.randint(-1, 1)))
    else:
        e = elems ** (1 / 3)
        a, b = rng.uniform(0.7, 1.4), rng.uniform(0.7, 1.4)
        n = (max(2, round(e * a)), max(2, round(e * b)), max(2, round(e / (a * b))))
    return _case(None, flow, N, n, vf, sf, call, **more)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _device():
    return "cuda:0" if torch.cuda.is_available() else "cpu"


def _basis(N):
    """LGL nodes and weights, derivative matrix, inverse orthonormal Vandermonde (numpy, float64)."""
    leg = np.polynomial.legendre
    c = np.zeros(N + 1)
    c[N] = 1.0
    inner = np.sort(np.real(leg.legroots(leg.legder(c)))) if N > 1 else np.zeros(0)
    for _ in range(3):  # Newton polish of the interior nodes
        if N > 1:
            d1, d2 = leg.legder(c), leg.legder(c, 2)
            inner = inner - leg.legval(inner, d1) / leg.legval(inner, d2)
    x = np.concatenate([[-1.0], inner, [1.0]])
    x = 0.5 * (x - x[::-1])
    LN = leg.legval(x, c)
    w = 2.0 / (N * (N + 1) * LN * LN)
    D = np.zeros((N + 1, N + 1))
    for i in range(N + 1):
        for j in range(N + 1):
            if i != j:
                D[i, j] = LN[i] / (LN[j] * (x[i] - x[j]))
    D[0, 0], D[N, N] = -N * (N + 1) / 4.0, N * (N + 1) / 4.0
    V = np.stack([np.sqrt(j + 0.5) * leg.legval(x, np.eye(N + 1)[j]) for j in range(N + 1)], axis=1)
    return x, w, D, np.linalg.inv(V)


def _coordinates(case):
    """Node coordinates x, y, z, each broadcastable to (nz, ny, nx, N+1, N+1, N+1)."""
    N, n, hi = case["N"], (case["nx"], case["ny"], case["nz"]), FLOWS[case["flow"]]["hi"]
    xi = torch.from_numpy(0.5 * (_basis(N)[0] + 1.0))
    out = []
    for d in range(3):
        line = (torch.arange(n[d], dtype=torch.float64)[:, None] + xi[None, :]) * (hi[d] / n[d])
        shape = [1] * 6
        shape[2 - d], shape[5 - d] = n[d], N + 1
        out.append(line.reshape(shape).to(_device()))
    return out


def _warped(case):
    """Curved mesh: every box node displaced by a smooth periodic field."""
    X = _coordinates(case)
    f = FLOWS[case["flow"]]
    t = [X[d] / f["hi"][d] for d in range(3)]
    ph = [(0.0, 0.1, 0.2), (0.3, 0.0, 0.4), (0.5, 0.6, 0.0)]
    A = f["warp"] * min(f["hi"])
    return [X[d] + A * torch.sin(TWO_PI * (t[0] + ph[d][0])) * torch.sin(TWO_PI * (t[1] + ph[d][1]))
            * torch.sin(TWO_PI * (t[2] + ph[d][2])) for d in range(3)]


def _state(case, seed):
    """Start state, shape (nElems, 5, N+1, N+1, N+1)."""
    f = FLOWS[case["flow"]]
    rng = np.random.default_rng(seed)
    x, y, z = _warped(case) if "warp" in f else _coordinates(case)
    L = f["hi"]

    def smooth(amp, modes=3):
        s = 0.0
        for _ in range(modes):
            k = rng.integers(1, 3, size=3)
            p = rng.uniform(0.0, TWO_PI, size=3)
            s = s + rng.uniform(-1.0, 1.0) * torch.sin(TWO_PI / L[0] * int(k[0]) * x + p[0]) \
                * torch.cos(TWO_PI / L[1] * int(k[1]) * y + p[1]) * torch.sin(TWO_PI / L[2] * int(k[2]) * z + p[2])
        return amp / modes * s

    if case["flow"].startswith("tgv"):
        p0 = 1.0 / (GAMMA * 0.01)
        u = torch.sin(x) * torch.cos(y) * torch.cos(z) + smooth(0.05)
        v = -torch.cos(x) * torch.sin(y) * torch.cos(z) + smooth(0.05)
        w = smooth(0.05)
        p = p0 + (torch.cos(2 * x) + torch.cos(2 * y)) * (torch.cos(2 * z) + 2.0) / 16.0
        rho = p / p0
    elif case["flow"] == "channel":
        eta = y - 1.0
        env = 1.0 - eta * eta
        u = 1.0 - eta ** 8 + env * smooth(0.1)
        v, w = env * smooth(0.1), env * smooth(0.1)
        rho = 1.0 + 0.0 * u
        p = rho / (GAMMA * MA_INF * MA_INF)
    elif case["flow"].startswith("sod"):
        xc = (torch.arange(case["nx"], dtype=torch.float64, device=x.device) + 0.5) * (L[0] / case["nx"])
        left = (xc < 0.5).reshape(1, 1, -1, 1, 1, 1)
        one = 1.0 + smooth(0.01)
        rho = torch.where(left, 1.0, 0.125) * one
        p = torch.where(left, 1.0, 0.1) * one
        u = v = w = smooth(0.01)
    else:
        rho = 1.0 + 0.2 * torch.sin(x + y + z) + smooth(0.05)
        u, v, w = 1.0 + smooth(0.05), 1.0 + smooth(0.05), 1.0 + smooth(0.05)
        p = 1.0 + smooth(0.05)
    ne, n1 = case["nx"] * case["ny"] * case["nz"], case["N"] + 1
    U = torch.empty((case["nz"], case["ny"], case["nx"], 5, n1, n1, n1), dtype=torch.float64, device=x.device)
    U[:, :, :, 0] = rho
    U[:, :, :, 1] = rho * u
    U[:, :, :, 2] = rho * v
    U[:, :, :, 3] = rho * w
    U[:, :, :, 4] = p / (GAMMA - 1.0) + 0.5 * rho * (u * u + v * v + w * w)
    if case["call"] != "rk_step" or not case["flow"].startswith("sod"):
        # element-wise constant jumps of the size a discrete solution has
        j = torch.from_numpy(1e-4 * rng.standard_normal((case["nz"], case["ny"], case["nx"], 5))).to(U.device)
        U *= 1.0 + j[..., None, None, None]
    return U.reshape(ne, 5, n1, n1, n1)


def _cotangent(case, seed):
    g = torch.Generator().manual_seed(seed + 1)
    ne, n1 = case["nx"] * case["ny"] * case["nz"], case["N"] + 1
    return torch.randn((ne, 5, n1, n1, n1), generator=g, dtype=torch.float64).to(_device())


def _operator(case):
    f = FLOWS[case["flow"]]
    more = {k: f[k] for k in ("precision", "Cs", "blending") if k in f}
    op = dg.DG((case["nx"], case["ny"], case["nz"]), case["N"], gamma=GAMMA, mu=f["mu"], hi=f["hi"],
               equations=dg.NS if f["mu"] > 0 else dg.EULER, vol_flux=VOL[case["vf"]], surf_flux=SURF[case["sf"]],
               **more)
    if "warp" in f:
        ne, n1 = op.n_elems, case["N"] + 1
        X = torch.stack(_warped(case), dim=3).reshape(ne, 3, n1, n1, n1).contiguous()
        op.set_geometry(X)
    if "wall" in f:
        op.set_wall_model(f["wall"], U_INF, MA_INF)
    return op


def _dt(case):
    """Time step from closed-form bounds of the flow, the same for every seed."""
    f = FLOWS[case["flow"]]
    speed = {"tgv": 1.1 + 2 * 10.3, "cha": 1.2 + 3 * 1.45, "sod": 1.0 + 3 * 1.25, "wav": 3 * 1.1 + 3 * 1.5}
    dx = [f["hi"][d] / case[k] for d, k in enumerate(("nx", "ny", "nz"))]
    rate = (speed[case["flow"][:3]] + (10.3 if case["flow"][:3] == "tgv" else 0.0)) / min(dx)
    return f["cfl"] / ((case["N"] + 1) * rate)


def prepare(case, seed):
    s = {"call": case["call"], "op": _operator(case), "U": _state(case, seed), "dt": _dt(case)}
    if case["call"] != "rk_step":
        s["cot"] = _cotangent(case, seed)
        s["U"].requires_grad_(True)
        s["steps"], s["every"] = case.get("steps"), case.get("every")
    return s


def run(s):
    if s["call"] == "rk_step":
        return s["op"].rk_step(s["U"], s["dt"])
    if s["call"] == "rollout":
        V = dg.rollout(s["op"], s["U"], s["dt"], s["steps"], checkpoint_every=s["every"])
    else:
        V = dg.DGOperator.apply(s["U"], s["op"])
    (grad,) = torch.autograd.grad(V, s["U"], s["cot"])
    return {"out": V.detach(), "grad": grad}


def work(case):
    """One operator evaluation with its stage update reads the state and the
    register and writes both (the first stage reads no register, the last
    writes none: 720 B per node and step); a curved mesh adds its ten metric
    values per node.  A reverse product reads the state and the cotangent and
    writes one.  Operations: the two-point fluxes of the three lines of each
    node, and for the viscous terms gradient and divergence along them."""
    n1 = case["N"] + 1
    nodes = case["nx"] * case["ny"] * case["nz"] * n1 ** 3
    f = FLOWS[case["flow"]]
    metric = 80 if "warp" in f else 0
    per = 3 * n1 * 17 + (3 * n1 * 16 if f["mu"] > 0 else 0)
    step = 720 + 5 * metric
    if case["call"] == "rk_step":
        return {"bytes": nodes * step, "flops": nodes * 5 * per}
    if case["call"] == "rollout":
        return {"bytes": nodes * case["steps"] * (step + 5 * (120 + metric)), "flops": nodes * case["steps"] * 15 * per}
    return {"bytes": nodes * (80 + 120 + 2 * metric), "flops": nodes * 3 * per}


# ---------------------------------------------------------------------------
# the definitions in plain torch, 64 bits
# ---------------------------------------------------------------------------
class _Plain:
    """U_t = L(U) on tensors of shape (nz, ny, nx, 5, N+1, N+1, N+1)."""

    def __init__(self, case):
        self.c, self.f = case, FLOWS[case["flow"]]
        self.N, self.n = case["N"], (case["nx"], case["ny"], case["nz"])
        N, dev = self.N, _device()
        self.xi, self.w, D, Vinv = _basis(N)
        Dh = 2.0 * D
        Dh[0, 0] = Dh[N, N] = 0.0
        Dw = D.copy()
        Dw[0, 0] += 1.0 / self.w[0]
        Dw[N, N] -= 1.0 / self.w[N]
        t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
        self.D, self.Dh, self.Dw, self.Vinv = t(D), t(Dh), t(Dw), t(Vinv)
        self.dx = [self.f["hi"][d] / self.n[d] for d in range(3)]
        self.wall = self.f.get("wall", -1)
        self.mu = self.f["mu"]
        self.kappa = self.mu * GAMMA / ((GAMMA - 1.0) * PR)
        if "warp" in self.f:
            self.metrics(_warped(case))
        else:
            self.J = self.dx[0] * self.dx[1] * self.dx[2] / 8.0
            self.Ja = [[self.J * 2.0 / self.dx[i] if i == m else 0.0 for m in range(3)] for i in range(3)]
            self.delta2 = ((self.dx[0] * self.dx[1] * self.dx[2]) ** (1 / 3) / (N + 1)) ** 2

    # -- lines and faces: direction d is node axis -1-d and element axis 2-d
    def along(self, M, a, d):
        return torch.movedim(torch.matmul(torch.movedim(a, -1 - d, -1), M.T), -1, -1 - d)

    @staticmethod
    def at(a, d, l):
        return a if isinstance(a, float) else a.select(-1 - d, l)

    def line(self, v, d):
        """A vector along direction d, broadcastable over scalar fields."""
        shape = [1, 1, 1]
        shape[2 - d] = -1
        return torch.as_tensor(np.ascontiguousarray(v), dtype=torch.float64, device=_device()).reshape(shape)

    def metrics(self, X):
        X = [x + 0.0 * sum(X) for x in X]
        mid = [0.5 * (x[..., :1, :1, :1] + x[..., -1:, -1:, -1:]) for x in X]
        X = [x - m for x, m in zip(X, mid)]
        dX = [[self.along(self.D, X[m], i) for i in range(3)] for m in range(3)]
        self.Ja = [[None] * 3 for _ in range(3)]
        for i in range(3):
            j, k = (i + 1) % 3, (i + 2) % 3
            for n in range(3):
                m, l = (n + 1) % 3, (n + 2) % 3
                self.Ja[i][n] = -(self.along(self.D, X[l] * dX[m][k], j) - self.along(self.D, X[l] * dX[m][j], k))
        self.J = sum(dX[0][i] * (dX[1][(i + 1) % 3] * dX[2][(i + 2) % 3] - dX[1][(i + 2) % 3] * dX[2][(i + 1) % 3])
                     for i in range(3))
        wt = self.line(self.w, 0) * self.line(self.w, 1) * self.line(self.w, 2)
        vol = (wt * self.J).sum(dim=(-1, -2, -3), keepdim=True)
        self.delta2 = (vol ** (1 / 3) / (self.N + 1)) ** 2

    # -- pointwise
    @staticmethod
    def prim(U):
        rho = U[0]
        u = [U[1] / rho, U[2] / rho, U[3] / rho]
        p = (GAMMA - 1.0) * (U[4] - 0.5 * (U[1] * u[0] + U[2] * u[1] + U[3] * u[2]))
        return {"r": rho, "u": u, "p": p, "E": U[4], "h": (U[4] + p) / rho, "e": U[4] / rho, "th": p / rho}

    @staticmethod
    def dot(n, u):
        return sum(n[m] * u[m] for m in range(3) if not (isinstance(n[m], float) and n[m] == 0.0))

    def twopoint(self, a, b, n):
        """F#(a, b) . n for a vector n."""
        add = lambda f, m, p: f if isinstance(n[m], float) and n[m] == 0.0 else f + p * n[m]  # noqa: E731
        if self.c["vf"] == "std":
            fa, fb = a["r"] * self.dot(n, a["u"]), b["r"] * self.dot(n, b["u"])
            pm = 0.5 * (a["p"] + b["p"])
            return [0.5 * (fa + fb)] + [add(0.5 * (fa * a["u"][m] + fb * b["u"][m]), m, pm) for m in range(3)] \
                + [0.5 * (fa * a["h"] + fb * b["h"])]
        um = [0.5 * (a["u"][m] + b["u"][m]) for m in range(3)]
        un, pm = self.dot(n, um), 0.5 * (a["p"] + b["p"])
        fr = 0.5 * (a["r"] + b["r"]) * un
        if self.c["vf"] == "kg":
            fE = fr * 0.5 * (a["e"] + b["e"]) + pm * un
        else:
            fE = fr * 0.5 * (a["h"] + b["h"])
        return [fr] + [add(fr * um[m], m, pm) for m in range(3)] + [fE]

    def riemann(self, a, b, n):
        """f*(a, b; n) with a on the minus side, n a unit vector."""
        f = self.twopoint(a, b, n)
        dr, dE = b["r"] - a["r"], b["E"] - a["E"]
        ua, ub = self.dot(n, a["u"]), self.dot(n, b["u"])
        if self.c["sf"] == "llf":
            lam = torch.maximum(ua.abs() + torch.sqrt(GAMMA * a["th"]), ub.abs() + torch.sqrt(GAMMA * b["th"]))
            dm = [b["r"] * b["u"][m] - a["r"] * a["u"][m] for m in range(3)]
            D = [lam * dr] + [lam * x for x in dm] + [lam * dE]
        else:
            sa, sb = torch.sqrt(a["r"]), torch.sqrt(b["r"])
            av = lambda x, y: (sa * x + sb * y) / (sa + sb)  # noqa: E731
            u = [av(a["u"][m], b["u"][m]) for m in range(3)]
            H, un, rt = av(a["h"], b["h"]), av(ua, ub), sa * sb
            q2 = u[0] * u[0] + u[1] * u[1] + u[2] * u[2]
            c2 = (GAMMA - 1.0) * (H - 0.5 * q2)
            c = torch.sqrt(c2)
            dp, dun = b["p"] - a["p"], ub - ua
            du = [b["u"][m] - a["u"][m] for m in range(3)]
            w1 = (un - c).abs() * 0.5 * (dp - rt * c * dun) / c2
            w5 = (un + c).abs() * 0.5 * (dp + rt * c * dun) / c2
            l2, a2 = un.abs(), dr - dp / c2
            D = [w1 + w5 + l2 * a2]
            for m in range(3):
                D.append(w1 * (u[m] - c * n[m]) + w5 * (u[m] + c * n[m]) + l2 * (a2 * u[m] + rt * (du[m] - dun * n[m])))
            D.append(w1 * (H - c * un) + w5 * (H + c * un)
                     + l2 * (a2 * 0.5 * q2 + rt * (self.dot(u, du) - un * dun)))
        return [f[v] - 0.5 * D[v] for v in range(5)]

    # -- interfaces: fields at the + face (l = N) of every element and at the - face of its + neighbour
    def sides(self, a, d):
        """(minus, plus) values at the + faces: own l = N, the + neighbour's l = 0."""
        return self.at(a, d, self.N), (a if isinstance(a, float) else torch.roll(self.at(a, d, 0), -1, 2 - d))

    @staticmethod
    def pick(P, g):
        return {k: [g(x) for x in v] if isinstance(v, list) else g(v) for k, v in P.items()}

    @staticmethod
    def mirror(P, d):
        return {k: [-x if m == d else x for m, x in enumerate(v)] if isinstance(v, list) else v for k, v in P.items()}

    def face_pairs(self, P, d):
        """[(minus, plus, keep)] for all faces of direction d: the values belong to the + face (first) and the
        - face (second) of the elements; walls see the mirrored own state."""
        L, R = self.pick(P, lambda a: self.sides(a, d)[0]), self.pick(P, lambda a: self.sides(a, d)[1])
        return L, R

    def put(self, x, d, faces_plus, faces_minus):
        """Adds (1/w)(delta_N f+ - delta_0 f-) along direction d to the nodal field x."""
        e = torch.zeros_like(x)
        e.select(-1 - d, self.N).add_(faces_plus / self.w[self.N])
        e.select(-1 - d, 0).sub_(faces_minus / self.w[0])
        return x + e

    def wall_slab(self, a, d, side):
        return a.select(2 - d, self.n[d] - 1 if side else 0)

    def both_faces(self, fun, P, d, n):
        """fun(minus, plus, n) at every + face and - face of the elements (lists of fields)."""
        L, R = self.face_pairs(P, d)
        plus = fun(L, R, n)
        minus = [torch.roll(x, 1, 2 - d) for x in plus]
        if d == self.wall:
            for side in (0, 1):
                own = self.pick(P, lambda a: self.wall_slab(self.at(a, d, self.N if side else 0), d, side))
                oth = self.mirror(own, d)
                v = fun(own, oth, n) if side else fun(oth, own, n)
                tgt = plus if side else minus
                for k in range(len(tgt)):
                    x = tgt[k].clone()
                    self.wall_slab(x, d, side).copy_(v[k])
                    tgt[k] = x
        return plus, minus

    # -- wall model
    @staticmethod
    def law(x):
        k = 0.4 * x
        ek = torch.exp(k)
        b = 1.0 + k * (1.0 + k * (0.5 + k / 6.0))
        return x + 0.1108 * (ek - b - k ** 4 / 24.0), 1.0 + 0.1108 * 0.4 * (ek - b)

    def wall_flux(self, P, d, side):
        """Viscous flux through the wall faces (momentum x, y, z; energy)."""
        no, nx = (self.N, 0) if side else (0, self.N)
        own = self.pick(P, lambda a: self.wall_slab(self.at(a, d, no), d, side))
        far = self.pick(P, lambda a: self.wall_slab(self.at(a, d, nx), d, side))
        tang = [m for m in range(3) if m != d]
        sp = torch.sqrt(far["u"][tang[0]] ** 2 + far["u"][tang[1]] ** 2)
        r = 0.5 * (GAMMA - 1.0) * MA_INF * MA_INF * PR ** (1 / 3)
        b = math.sqrt(r / (1.0 + r))
        u = (U_INF / b) * torch.asin(torch.clamp(b * sp / U_INF, max=1.0))
        h = self.dx[d]
        lre = torch.log(h * u * own["r"] / self.mu)
        s = torch.clamp(0.5 * lre, max=math.log(1700.0))
        for _ in range(60):
            x = torch.exp(s)
            y, dy = self.law(x)
            s = s - (s + torch.log(y) - lre) / (1.0 + x * dy / y)
        ut = u / torch.exp(s)
        c = (-1.0 if side else 1.0) * own["r"] * ut * ut / sp
        zero = torch.zeros_like(c)
        return [c * far["u"][m] if m in tang else zero for m in range(3)] + [zero]

    # -- blending
    def alpha(self, P):
        N = self.N
        m = P["r"] * P["p"]
        for d in range(3):
            m = self.along(self.Vinv, m, d)
        e = m * m
        k = torch.arange(N + 1, device=e.device)
        mx = torch.maximum(k[:, None, None], torch.maximum(k[None, :, None], k[None, None, :]))
        tot = e.sum(dim=(-1, -2, -3))
        top = (e * (mx == N)).sum(dim=(-1, -2, -3))
        nxt = (e * (mx == N - 1)).sum(dim=(-1, -2, -3))
        E = torch.maximum(top / tot, nxt / (tot - top))
        T = 0.5 * 10.0 ** (-1.8 * (N + 1) ** 0.25)
        a = 1.0 / (1.0 + torch.exp(-(math.log(9999.0) / T) * (E - T)))
        a = torch.clamp(a, max=0.7)
        a = torch.where(a < 0.01, torch.zeros_like(a), a)
        nb = a
        for d in range(3):
            nb = torch.maximum(nb, 0.5 * torch.maximum(torch.roll(a, 1, 2 - d), torch.roll(a, -1, 2 - d)))
        return torch.where(nb < 0.01, torch.zeros_like(nb), nb)

    def subcells(self, P, faces):
        """U_t of the finite-volume subcells (minmod in the inner ones)."""
        N = self.N
        edge = np.concatenate([[-1.0], -1.0 + np.cumsum(self.w)])
        W = [P["r"], P["u"][0], P["u"][1], P["u"][2], P["p"]]
        out = [0.0] * 5
        for d in range(3):
            A = [torch.movedim(x, -1 - d, -1) for x in W]
            t = lambda v: torch.as_tensor(v, dtype=torch.float64, device=A[0].device)  # noqa: E731
            right, left = [x.clone() for x in A], [x.clone() for x in A]
            if N >= 2:
                hl, hr = t(1.0 / np.diff(self.xi)[:-1]), t(1.0 / np.diff(self.xi)[1:])
                dp, dm = t((edge[1:] - self.xi)[1:N]), t((edge[:-1] - self.xi)[1:N])
                R, L = [], []
                for x in A:
                    a, b = (x[..., 1:N] - x[..., :N - 1]) * hl, (x[..., 2:] - x[..., 1:N]) * hr
                    s = torch.where(a * b <= 0, torch.zeros_like(a), torch.where(a > 0, torch.minimum(a, b),
                                                                                 torch.maximum(a, b)))
                    R.append(x[..., 1:N] + s * dp)
                    L.append(x[..., 1:N] + s * dm)
                ok = (R[0] > 0) & (R[4] > 0) & (L[0] > 0) & (L[4] > 0)
                for v in range(5):
                    right[v][..., 1:N] = torch.where(ok, R[v], A[v][..., 1:N])
                    left[v][..., 1:N] = torch.where(ok, L[v], A[v][..., 1:N])

            def full(w):
                E = w[4] / (GAMMA - 1.0) + 0.5 * w[0] * (w[1] ** 2 + w[2] ** 2 + w[3] ** 2)
                return self.prim([w[0], w[0] * w[1], w[0] * w[2], w[0] * w[3], E])

            n = [1.0 if m == d else 0.0 for m in range(3)]
            f = self.riemann(full([x[..., :N] for x in right]), full([x[..., 1:] for x in left]), n)
            for v in range(5):
                F = torch.cat([faces[d][1][v][..., None], f[v], faces[d][0][v][..., None]], dim=-1)
                g = (F[..., 1:] - F[..., :-1]) * t(2.0 / (self.dx[d] * self.w))
                out[v] = out[v] - torch.movedim(g, -1, -1 - d)
        return out

    # -- the operator
    def __call__(self, U):
        N = self.N
        P = self.prim([U.select(3, v) for v in range(5)])
        curved = "warp" in self.f
        acc = [torch.zeros_like(P["r"]) for _ in range(5)]
        faces, normals = [], []
        for i in range(3):
            if curved:
                Nf = [0.5 * sum(self.sides(self.Ja[i][m], i)) for m in range(3)]
                size = torch.sqrt(Nf[0] ** 2 + Nf[1] ** 2 + Nf[2] ** 2)
                nrm = [x / size for x in Nf]
            else:
                Nf, size = self.Ja[i], self.Ja[i][i]
                nrm = [1.0 if m == i else 0.0 for m in range(3)]
            normals.append(Nf)
            fp, fm = self.both_faces(lambda a, b, n: [size * x for x in self.riemann(a, b, n)], P, i, nrm)
            faces.append((fp, fm))
            s = [torch.zeros_like(P["r"]) for _ in range(5)]
            for l in range(N + 1):
                Pl = self.pick(P, lambda a: self.at(a, i, l).unsqueeze(-1 - i))
                if curved:
                    n = [0.5 * (x + self.at(x, i, l).unsqueeze(-1 - i)) for x in self.Ja[i]]
                else:
                    n = self.Ja[i]
                col = self.line(self.Dh[:, l].cpu().numpy(), i)
                F = self.twopoint(P, Pl, n)
                s = [s[v] + col * F[v] for v in range(5)]
            for v in range(5):
                acc[v] = acc[v] - self.put(s[v], i, fp[v], fm[v])
        acc = [a / self.J for a in acc]
        if self.f.get("blending"):
            al = self.alpha(P)[..., None, None, None]
            scaled = [([x / self.Ja[d][d] for x in faces[d][0]], [x / self.Ja[d][d] for x in faces[d][1]])
                      for d in range(3)]
            fv = self.subcells(P, scaled)
            acc = [(1.0 - al) * acc[v] + al * fv[v] for v in range(5)]
        if self.mu > 0:
            visc = self.viscous(P, normals)
            acc = [acc[0]] + [acc[1 + k] + visc[k] for k in range(4)]
        return torch.stack(acc, dim=3)

    def viscous(self, P, normals):
        q = P["u"] + [P["th"]]
        g = [[0.0] * 4 for _ in range(3)]
        for i in range(3):
            fun = lambda a, b, n: [0.5 * (x + y) for x, y in zip(a["u"] + [a["th"]], b["u"] + [b["th"]])]  # noqa: E731
            qp, qm = self.both_faces(fun, P, i, None)
            for c in range(4):
                s = self.put(self.along(self.Dw, q[c], i), i, qp[c], qm[c])
                for m in range(3):
                    Ja = self.Ja[i][m]
                    if not (isinstance(Ja, float) and Ja == 0.0):
                        g[m][c] = g[m][c] + Ja * s / self.J
        mu, kap = self.mu, self.kappa
        if "Cs" in self.f:
            S2 = sum(2.0 * g[a][a] ** 2 for a in range(3)) + sum((g[a][b] + g[b][a]) ** 2
                                                                 for a, b in ((0, 1), (0, 2), (1, 2)))
            mut = P["r"] * (self.f["Cs"] ** 2 * self.delta2) * torch.sqrt(S2)
            mu, kap = mu + mut, kap + mut * (GAMMA / ((GAMMA - 1.0) * PRT))
        div = (2.0 / 3.0) * (g[0][0] + g[1][1] + g[2][2])
        Fv = []  # Fv[d][component]
        for d in range(3):
            F = [mu * (g[d][j] + g[j][d]) - (mu * div if j == d else 0.0) for j in range(3)]
            Fv.append(F + [self.dot(P["u"], F) + kap * g[d][3]])
        out = [0.0] * 4
        for i in range(3):
            wf = [self.wall_flux(P, i, side) for side in (0, 1)] if i == self.wall else None
            for c in range(4):
                vec = [Fv[m][c] for m in range(3)]
                con = self.dot(self.Ja[i], vec)
                s = [self.sides(x, i) for x in vec]
                plus = self.dot(normals[i], [0.5 * (a + b) for a, b in s])
                minus = torch.roll(plus, 1, 2 - i)
                if wf is not None:
                    plus, minus = plus.clone(), minus.clone()
                    self.wall_slab(minus, i, 0).copy_(self.Ja[i][i] * wf[0][c])
                    self.wall_slab(plus, i, 1).copy_(self.Ja[i][i] * wf[1][c])
                out[c] = out[c] + self.put(self.along(self.Dw, con, i), i, plus, minus) / self.J
        return out


def _stage(L, U, G, k, dt):
    G = RK_A[k] * G + L(U) if k else L(U)
    return U + (RK_B[k] * dt) * G, G


def exact(case, seed):
    L, dt = _Plain(case), _dt(case)
    n1 = case["N"] + 1
    shape = (case["nz"], case["ny"], case["nx"], 5, n1, n1, n1)
    U = _state(case, seed)
    flat = U.shape
    U = U.reshape(shape)
    if case["call"] == "rk_step":
        with torch.no_grad():
            G = None
            for k in range(5):
                U, G = _stage(L, U, G, k, dt)
        return U.reshape(flat)
    cot = _cotangent(case, seed).reshape(shape)
    if case["call"] == "operator":
        U.requires_grad_(True)
        V = L(U)
        (g,) = torch.autograd.grad(V, U, cot)
        return {"out": V.detach().reshape(flat), "grad": g.reshape(flat)}
    with torch.no_grad():
        trace, G = [], torch.zeros_like(U)
        for _ in range(case["steps"]):
            for k in range(5):
                trace.append((U, G))
                U, G = _stage(L, U, G, k, dt)
    out, Ub, Gb = U, cot, torch.zeros_like(cot)
    for j in reversed(range(len(trace))):
        u, G = (x.detach().requires_grad_(True) for x in trace[j])
        V, H = _stage(L, u, G, j % 5, dt)
        Ub, Gn = torch.autograd.grad((V, H), (u, G), (Ub, Gb), allow_unused=True)
        Gb = torch.zeros_like(cot) if Gn is None else Gn
    return {"out": out.reshape(flat), "grad": Ub.reshape(flat)}
