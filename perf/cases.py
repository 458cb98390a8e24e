"""The work that a user of this library has it do, as cases that can be timed.

A case is one pass through the public entry points of
``paper_2207_11571_amd.binding``:

advance   Runge-Kutta steps of one solve, plain, with the forcing network at
          every stage, or with the correction after each step
residual  one evaluation of the operator p(q)
frame     what the accuracy studies do between two recorded times: steps, the
          filter to the low order, the error against a reference, diagnostics
pairs     training pairs from a high-order state, Eq. (5) or Algorithm 1
train     one Adam step of the forcing network on a minibatch
serve     a mixed set of Taylor-Green requests through the solve server

``listed`` holds the cases that stand for the range, ``draw`` gives others of
the same range, ``exact`` what plain float64 torch computes for the same
inputs (a separate implementation of the method, on whole arrays).
"""
import math

import numpy as np
import torch

from paper_2207_11571_amd import binding as B

GAMMA, PRANDTL, PRANDTL_T, MACH = 1.4, 0.72, 0.6, 0.1
P0 = 1.0 / (GAMMA * MACH * MACH)
ENERGY = P0 / (GAMMA - 1.0) + 0.125          # level of rho e in these flows
HIDDEN = (256, 256, 256)
RK_A, RK_B = (0.0, -5.0 / 9.0, -153.0 / 128.0), (1.0 / 3.0, 15.0 / 16.0, 8.0 / 15.0)
LARGEST = 32 ** 3 * 7 ** 3                   # nodes of the largest listed mesh


def listed():
    return [
        # the smallest mesh of the served stream, one step per call, as a
        # loop that records something after every step makes it
        dict(name="step_4_p3", kind="advance", N=4, P=3, Re=200.0, Cs=0.0, steps=1, net="", form=""),
        # the corrected low order on the paper's 8^3 mesh: the online use of
        # the trained network in the accuracy studies
        dict(name="steps_8_p3_net", kind="advance", N=8, P=3, Re=1600.0, Cs=0.0, steps=2, net="stage", form="all"),
        # the corrected throughput workload
        dict(name="step_16_p3_net", kind="advance", N=16, P=3, Re=200.0, Cs=0.0, steps=1, net="stage", form="all"),
        # the headline throughput workload
        dict(name="step_16_p6", kind="advance", N=16, P=6, Re=1600.0, Cs=0.0, steps=1, net="", form=""),
        # the high-order scheme with the Smagorinsky closure (Table 1 case 3)
        dict(name="step_16_p8_les", kind="advance", N=16, P=8, Re=1600.0, Cs=0.1, steps=1, net="", form=""),
        # a larger solve than the chip's caches hold
        dict(name="step_32_p6", kind="advance", N=32, P=6, Re=1600.0, Cs=0.0, steps=1, net="", form=""),
        # the bare operator on an odd mesh and order
        dict(name="residual_11_p5", kind="residual", N=11, P=5, Re=200.0, Cs=0.0, viscous=True),
        # a plain higher order of the accuracy study, between two records
        dict(name="frame_8_p6", kind="frame", N=8, P=6, P_lo=3, Re=200.0, Cs=0.0, steps=2),
        # one low-order step of the training window on the paper's mesh:
        # the high-order evolution and its pairs
        dict(name="pairs_8_p8_p3", kind="pairs", form="alg1", N=8, P=8, P_lo=3, Re=200.0, Cs=0.0, m_sub=3),
        # minibatches of the accuracy studies (the paper's network) and of
        # the throughput workload
        dict(name="train_512_momenta", kind="train", batch=512, P=3, form="momenta", shuffled=True),
        dict(name="train_4096_all", kind="train", batch=4096, P=3, form="all", shuffled=True),
        # the mixed request stream, a short piece of it
        dict(name="serve_mixed", kind="serve", t_end=0.008, small=2, medium=1, large=1),
    ]


def _spread(rng, lo, hi):
    """An integer of [lo, hi], spread over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo - 0.49), math.log(hi + 0.49)))))))


def draw(rng):
    kind = rng.choice(["advance", "advance", "advance", "corrected", "corrected", "residual", "frame", "pairs",
                       "train", "train", "serve"])
    Re = float(rng.choice([30, 200, 1600]))
    Cs = rng.choice([0.0, 0.0, 0.1])
    if kind in ("advance", "residual"):
        P = rng.randint(1, 8)
        N = _spread(rng, 2, min(40, int((LARGEST / (P + 1) ** 3) ** (1.0 / 3.0) + 1e-9)))
        if kind == "residual":
            return dict(kind=kind, N=N, P=P, Re=Re, Cs=Cs, viscous=rng.random() < 0.8)
        steps = rng.randint(1, max(1, min(3, LARGEST // (N ** 3 * (P + 1) ** 3))))
        return dict(kind=kind, N=N, P=P, Re=Re, Cs=Cs, steps=steps, net="", form="")
    if kind == "corrected":
        return dict(kind="advance", N=_spread(rng, 2, 20), P=rng.choice([2, 3, 3, 3]), Re=Re, Cs=Cs,
                    steps=rng.randint(1, 3), net=rng.choice(["stage", "stage", "post"]),
                    form=rng.choice(["all", "momenta"]))
    if kind == "frame":
        return dict(kind=kind, N=_spread(rng, 3, 16), P=rng.randint(4, 8), P_lo=rng.choice([2, 3]), Re=Re, Cs=Cs,
                    steps=rng.randint(1, 2))
    if kind == "pairs":
        return dict(kind=kind, form=rng.choice(["eq5", "alg1"]), N=_spread(rng, 3, 12), P=rng.randint(5, 8),
                    P_lo=rng.choice([2, 3]), Re=Re, Cs=Cs, m_sub=rng.randint(1, 4))
    if kind == "train":
        return dict(kind=kind, batch=_spread(rng, 40, 8192), P=rng.choice([2, 3, 3]),
                    form=rng.choice(["all", "momenta"]), shuffled=rng.random() < 0.8)
    return dict(kind="serve", t_end=round(rng.uniform(0.003, 0.008), 4), small=rng.randint(1, 3),
                medium=rng.randint(0, 2), large=0)


# ------------------------------------------------------------------- inputs

def _dt(N, P, Re):
    """A step inside the CFL limit at speed |v| + c = 11.5."""
    h, n = 2.0 * math.pi / N, P + 1
    return min(0.4 * h / (n * n * 11.5), 0.4 * h * h * Re * PRANDTL / (n ** 4 * GAMMA * 1.05))


def _random(seed):
    return np.random.default_rng(np.random.SeedSequence([int(seed) & 0xFFFFFFFF, 2207]))


def _coordinates(N, P, device):
    x = np.polynomial.legendre.leggauss(P + 1)[0]
    x1 = ((np.arange(N)[:, None] + 0.5 * (x[None, :] + 1.0)) * (2.0 * math.pi / N))
    x1 = torch.from_numpy(x1).to(device)
    return x1[None, None, :, None, None, :], x1[None, :, None, None, :, None], x1[:, None, None, :, None, None]


def _state(N, P, seed, device="cuda"):
    """A Taylor-Green vortex some time after its start: the vortex shifted
    and with modes of higher wavenumbers on top, density and pressure varying
    as at Mach 0.1; [5][E][n_p]."""
    r = _random(seed)
    n = P + 1
    X, Y, Z = _coordinates(N, P, device)
    sx, sy, sz = (float(r.uniform(0.0, 6.0)) for _ in range(3))
    one = torch.ones((N, N, N, n, n, n), dtype=torch.float64, device=device)
    v = [torch.sin(X + sx) * torch.cos(Y + sy) * torch.cos(Z + sz) * one,
         -torch.cos(X + sx) * torch.sin(Y + sy) * torch.cos(Z + sz) * one, 0.0 * one]
    p = P0 + (torch.cos(2 * (X + sx)) + torch.cos(2 * (Y + sy))) * (torch.cos(2 * (Z + sz)) + 2.0) / 16.0
    rho = 1.0 + 0.004 * torch.sin(X + sy) * torch.cos(Y - sz) * one
    for _ in range(4):
        a = [int(k) for k in r.integers(1, 1 + max(2, min(6, N // 2)), 3)]
        f = [float(t) for t in r.uniform(0.0, 6.28, 3)]
        mode = torch.sin(a[0] * X + f[0]) * torch.sin(a[1] * Y + f[1]) * torch.sin(a[2] * Z + f[2])
        for d in range(3):
            v[d] = v[d] + float(r.uniform(-0.12, 0.12)) * mode
        p = p + float(r.uniform(-0.02, 0.02)) * mode
    q = torch.stack([rho, rho * v[0], rho * v[1], rho * v[2],
                     p / (GAMMA - 1.0) + 0.5 * rho * (v[0] ** 2 + v[1] ** 2 + v[2] ** 2)])
    return q.reshape(5, N ** 3, n ** 3).contiguous()


def _net(P, form, seed):
    """(dims, [(W, b), ...] float32, norm, options) of a forcing network of
    the documented shapes: tanh on all variables, or relu on the momenta."""
    r = _random(seed + 77)
    n_io = 3 if form == "momenta" else 5
    dims = [n_io * (P + 1) ** 3, *HIDDEN, n_io * (P + 1) ** 3]
    layers = [((r.standard_normal((o, i)) / math.sqrt(i)).astype(np.float32),
               (0.02 * r.standard_normal(o)).astype(np.float32)) for i, o in zip(dims[:-1], dims[1:])]
    norm = [1.0, 0.0, 0.0, 0.0, ENERGY, 0.01, 0.5, 0.5, 0.5, 1.0] + [0.0] * 5 + [1e-3, 1e-2, 1e-2, 1e-2, 1e-1]
    opt = dict(activation="relu", in_vars=(1, 2, 3), out_vars=(1, 2, 3)) if form == "momenta" else {}
    return dims, layers, norm, opt


def _model(P, form, seed, train):
    dims, layers, norm, opt = _net(P, form, seed)
    return B.Model(dims, B.pack_params(layers), norm, train=train, **opt)


def _rows(case, seed, device="cuda"):
    """A dataset of sixteen minibatches: element rows around the levels of
    the flow, forcings of the size that the network is scaled for, and a
    shuffle of it."""
    width, rows = 5 * (case["P"] + 1) ** 3, 16 * case["batch"]
    g = torch.Generator(device=device).manual_seed(int(seed) & 0x7FFFFFFF)
    norm = _net(case["P"], case["form"], 0)[2]

    def field(mu, sigma):
        n_p = width // 5
        mu = torch.tensor(mu, dtype=torch.float32, device=device).repeat_interleave(n_p)
        sigma = torch.tensor(sigma, dtype=torch.float32, device=device).repeat_interleave(n_p)
        smooth = torch.randn((rows, 5), generator=g, device=device).repeat_interleave(n_p, dim=1)
        return mu + sigma * (0.8 * smooth + 0.6 * torch.randn((rows, width), generator=g, device=device))

    x, y = field(norm[0:5], norm[5:10]), field(norm[10:15], norm[15:20])
    perm = torch.randperm(rows, generator=g, device=device).to(torch.int32)
    return x.contiguous(), y.contiguous(), perm


def _requests(case, seed):
    """The request mix: orders and meshes of the served stream, in turn."""
    r = _random(seed + 5)
    kinds = []
    for N, count in ((4, case["small"]), (8, case["medium"]), (16, case["large"])):
        for i in range(count):
            kinds += [(3, N, "post" if i % 2 else "stage"), (6, N, "")] + ([(8, N, "")] if N < 16 else [])
    return [dict(P=P, N=N, net=net, Re=float(r.choice([30.0, 200.0, 1600.0]))) for P, N, net in kinds]


# ------------------------------------------------------------ prepare and run

def prepare(case, seed):
    kind = case["kind"]
    if kind == "train":
        x, y, perm = _rows(case, seed)
        return dict(case=case, model=_model(case["P"], case["form"], seed, True), x=x, y=y, perm=perm, at=0,
                    loss=torch.zeros(1, dtype=torch.float32, device="cuda"))
    if kind == "serve":
        reqs = _requests(case, seed)
        room = sum(B.solve_footprint(q["P"], q["N"], bool(q["net"])) for q in reqs) + (1 << 20)
        return dict(case=case, server=B.Server(room, max_slots=64), model=_model(3, "all", seed, False), reqs=reqs)
    s = dict(case=case, mesh=B.Mesh(case["N"], case["P"], case["Re"], Cs=case["Cs"],
                                    viscous=case.get("viscous", True)),
             q=_state(case["N"], case["P"], seed), dt=_dt(case["N"], case["P"], case["Re"]))
    s["k"] = s["mesh"].field(0.0)
    if kind == "advance" and case["net"]:
        s["model"] = _model(case["P"], case["form"], seed, False)
    if kind in ("frame", "pairs"):
        s["lo"] = B.Mesh(case["N"], case["P_lo"], case["Re"], Cs=case["Cs"])
    if kind == "frame":
        s["q_lo"], s["ref"] = s["lo"].field(), _state(case["N"], case["P_lo"], seed + 1)
        s["err"] = torch.zeros(3, dtype=torch.float64, device="cuda")
        s["diag"] = torch.zeros(8, dtype=torch.float64, device="cuda")
    if kind == "pairs":
        width = 5 * (case["P_lo"] + 1) ** 3
        s["x"], s["y"] = (torch.empty((case["N"] ** 3, width), dtype=torch.float32, device="cuda") for _ in range(2))
        s["ws"] = None
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "advance":
        step = B.dg_rk_step_post if case["net"] == "post" else B.dg_rk_step
        step(s["mesh"], s["q"], s["k"], s["dt"], case["steps"], model=s.get("model"))
        return s["q"]
    if kind == "residual":
        B.dg_residual(s["mesh"], s["q"], s["k"])
        return s["k"]
    if kind == "frame":
        B.dg_rk_step(s["mesh"], s["q"], s["k"], s["dt"], case["steps"])
        B.dg_project(s["mesh"], s["lo"], s["q"], s["q_lo"])
        B.dg_error_inf(s["lo"], s["q_lo"], s["ref"], s["err"])
        B.dg_diagnostics(s["mesh"], s["q"], out=s["diag"])
        return dict(q=s["q"], q_lo=s["q_lo"], err=s["err"], diag=s["diag"])
    if kind == "pairs":
        if case["form"] == "eq5":
            s["ws"] = B.dg_forcing_target(s["mesh"], s["lo"], s["q"], s["x"], s["y"], ws=s["ws"])
        else:
            s["ws"] = B.dg_increment_target(s["mesh"], s["lo"], s["q"], s["k"], s["dt"] * case["m_sub"],
                                            case["m_sub"], s["x"], s["y"], ws=s["ws"])
        return dict(q=s["q"], x=s["x"], y=s["y"])
    if kind == "train":
        m, b = s["model"], case["batch"]
        if case["shuffled"]:
            B.nn_train_step(m, s["x"], s["y"], lr=1e-3, loss=s["loss"], idx=s["perm"][s["at"] * b:(s["at"] + 1) * b])
        else:
            B.nn_train_step(m, s["x"][s["at"] * b:(s["at"] + 1) * b], s["y"][s["at"] * b:(s["at"] + 1) * b], lr=1e-3,
                            loss=s["loss"])
        s["at"] = (s["at"] + 1) % 16
        return dict(loss=s["loss"], params=m.params, grad=m.grad, m=m.m, v=m.v)
    srv = s["server"]
    ids = [srv.submit(r["Re"], r["P"], r["N"], case["t_end"], use_nn=bool(r["net"]),
                      model=s["model"] if r["net"] else None, ke_every=8, ke_capacity=64,
                      want_state=r["N"] <= 8, after_step=r["net"] == "post") for r in s["reqs"]]
    srv.drain()
    return [srv.results(i) if r["N"] <= 8 else srv.results(i)[0] for i, r in zip(ids, s["reqs"])]


# ----------------------------------------------------------------------- work

def _dg_work(N, P, stages, viscous=True):
    """Operations of `stages` evaluations of the operator: the line
    contractions (gradient of four variables, divergence of five fluxes),
    the node fluxes, the face values and fluxes."""
    n, E = P + 1, N ** 3
    node = 3 * 2 * n * (5 + (4 if viscous else 0)) + (190 if viscous else 70)
    face = 2 * n * (5 + (12 if viscous else 0)) + (330 if viscous else 200)
    return stages * E * (n ** 3 * node + 6 * n * n * face)


def _step_bytes(N, P):
    """One Runge-Kutta step: every stage needs the whole field of the stage
    before it, so state and register go through memory once a stage (the
    first stage reads no register)."""
    return N ** 3 * (P + 1) ** 3 * 5 * 8 * (3 + 4 + 4)


def work(case):
    kind = case["kind"]
    if kind in ("train", "serve") or case.get("net"):
        P = case.get("P", 3)
        io = (3 if case.get("form") == "momenta" else 5) * (P + 1) ** 3
        weights = io * 256 + 2 * 256 * 256 + 256 * io
    if kind == "train":
        # rows read; weights, moments read and written, the gradient and the
        # two 16-bit copies written; forward, data and weight gradients
        return dict(bytes=case["batch"] * 4.0 * 2 * io + weights * (6 * 4.0 + 4 + 4), flops=6.0 * case["batch"] * weights)
    if kind == "serve":
        total = dict(bytes=0.0, flops=0.0)
        for r in _requests(case, 0):
            steps = math.ceil(case["t_end"] / _dt(r["N"], r["P"], r["Re"]))
            sub = dict(kind="advance", N=r["N"], P=r["P"], steps=steps, net=r["net"], form="all" if r["net"] else "")
            w = work(sub)
            total = {k: total[k] + w[k] for k in total}
        return total
    N, P, field = case["N"], case["P"], case["N"] ** 3 * (case["P"] + 1) ** 3 * 40.0
    if kind == "residual":
        return dict(bytes=2.0 * field, flops=_dg_work(N, P, 1, case["viscous"]))
    if kind == "advance":
        w = dict(bytes=float(case["steps"] * _step_bytes(N, P)), flops=float(_dg_work(N, P, 3 * case["steps"])))
        if case["net"]:
            evals = case["steps"] * (3 if case["net"] == "stage" else 1)
            w["bytes"] += evals * weights * 2.0
            w["flops"] += evals * 2.0 * N ** 3 * weights
        return w
    n_lo = case["P_lo"] + 1
    low = N ** 3 * n_lo ** 3 * 40.0
    filt = 2.0 * 5 * N ** 3 * ((P + 1) ** 3 * n_lo + (P + 1) ** 2 * n_lo ** 2 + (P + 1) * n_lo ** 3)
    if kind == "frame":
        # steps, then the state read once more, the low-order field written, the reference read
        return dict(bytes=case["steps"] * _step_bytes(N, P) + field + 2 * low,
                    flops=float(_dg_work(N, P, 3 * case["steps"]) + filt + 25 * N ** 3 * (P + 1) ** 3))
    if case["form"] == "eq5":
        return dict(bytes=field + low, flops=float(_dg_work(N, P, 1) + _dg_work(N, case["P_lo"], 1) + 2 * filt))
    return dict(bytes=case["m_sub"] * _step_bytes(N, P) + field + low,
                flops=float(_dg_work(N, P, 3 * case["m_sub"]) + _dg_work(N, case["P_lo"], 3) + 2 * filt))


# --------------------------------------------------------------- float64 torch

class _Basis:
    def __init__(self, P, device):
        x, w = np.polynomial.legendre.leggauss(P + 1)
        x, w = x.astype(np.longdouble), w.astype(np.longdouble)
        n = P + 1
        lam = np.array([1.0 / np.prod([x[j] - x[k] for k in range(n) if k != j]) for j in range(n)], np.longdouble)
        D = np.zeros((n, n), np.longdouble)
        for i in range(n):
            for j in range(n):
                if i != j:
                    D[i, j] = lam[j] / lam[i] / (x[i] - x[j])
            D[i, i] = -D[i].sum()

        def ends(t):
            b = lam / (t - x)
            return b / b.sum()

        def put(a):
            return torch.from_numpy(np.ascontiguousarray(a).astype(np.float64)).to(device)

        self.x, self.w = put(x), put(w)
        self.hat = put((D * w[:, None]).T / w[:, None])
        self.end = (put(ends(np.longdouble(-1.0))), put(ends(np.longdouble(1.0))))
        self.lift = tuple(put(ends(np.longdouble(t)) / w) for t in (-1.0, 1.0))


def _line(A, M, d):
    """M along the node axis of direction d."""
    return (A.movedim(-1 - d, -1) @ M.T).movedim(-1, -1 - d)


def _shift(A, d, by):
    return torch.roll(A, by, dims=A.dim() - 4 - d)


class _Flow:
    """The operator p(q) on arrays [v, ez, ey, ex, k, j, i]."""

    def __init__(self, N, P, Re, Cs, viscous=True, device="cuda"):
        self.N, self.P, self.n, self.b, self.viscous = N, P, P + 1, _Basis(P, device), viscous
        self.h = 2.0 * math.pi / N
        self.mu = 1.0 / Re
        self.kappa = self.mu * GAMMA / ((GAMMA - 1.0) * PRANDTL)
        self.les = (Cs * self.h / (P + 1)) ** 2

    def blocks(self, q):
        return q.reshape(5, self.N, self.N, self.N, self.n, self.n, self.n)

    @staticmethod
    def pressure(q):
        return (GAMMA - 1.0) * (q[4] - 0.5 * (q[1] ** 2 + q[2] ** 2 + q[3] ** 2) / q[0])

    def prim(self, q):
        return torch.stack([q[1] / q[0], q[2] / q[0], q[3] / q[0], self.pressure(q) / q[0]])

    def trace(self, A, side, d):
        return _line(A, self.b.end[side][None, :], d)

    def weak(self, F, up, low, d):
        shape = (-1,) + (1,) * d
        return (2.0 / self.h) * (self.b.lift[1].reshape(shape) * up - self.b.lift[0].reshape(shape) * low
                                 - _line(F, self.b.hat, d))

    def euler(self, q, d):
        v, p = q[1 + d] / q[0], self.pressure(q)
        F = q * v
        F[1 + d] += p - P0
        F[4] += p * v
        return F

    def stress(self, q, g, d):
        mu, kappa = self.mu, self.kappa
        if self.les > 0.0:
            SS = sum((0.5 * (g[a][b] + g[b][a])) ** 2 for a in range(3) for b in range(3))
            mut = q[0] * self.les * torch.sqrt(2.0 * SS)
            mu, kappa = mu + mut, kappa + mut * GAMMA / ((GAMMA - 1.0) * PRANDTL_T)
        F = torch.zeros_like(q)
        for a in range(3):
            tau = mu * (g[a][d] + g[d][a])
            if a == d:
                tau = tau - (2.0 / 3.0) * mu * (g[0][0] + g[1][1] + g[2][2])
            F[1 + a] = tau
            F[4] += q[1 + a] / q[0] * tau
        F[4] += kappa * g[d][3]
        return F

    def roe(self, L, R, d):
        pL, pR = self.pressure(L), self.pressure(R)
        a, b = torch.sqrt(L[0]), torch.sqrt(R[0])
        rt = a * b
        vt = [(a * L[1 + i] / L[0] + b * R[1 + i] / R[0]) / (a + b) for i in range(3)]
        H = (a * (L[4] + pL) / L[0] + b * (R[4] + pR) / R[0]) / (a + b)
        v2 = vt[0] ** 2 + vt[1] ** 2 + vt[2] ** 2
        c = torch.sqrt((GAMMA - 1.0) * (H - 0.5 * v2))
        dv = [R[1 + i] / R[0] - L[1 + i] / L[0] for i in range(3)]
        dp, drho = pR - pL, R[0] - L[0]
        F = 0.5 * (self.euler(L, d) + self.euler(R, d))
        for lam, amp, sgn, hh in ((vt[d] - c, (dp - rt * c * dv[d]) / (2 * c * c), -1.0, H - c * vt[d]),
                                  (vt[d], drho - dp / (c * c), 0.0, 0.5 * v2),
                                  (vt[d] + c, (dp + rt * c * dv[d]) / (2 * c * c), 1.0, H + c * vt[d])):
            s = 0.5 * lam.abs() * amp
            F[0] -= s
            for i in range(3):
                F[1 + i] -= s * (vt[i] + sgn * c if i == d else vt[i])
            F[4] -= s * hh
        for i in range(3):
            if i != d:
                s = 0.5 * vt[d].abs() * rt * dv[i]
                F[1 + i] -= s
                F[4] -= s * vt[i]
        return F

    def rhs(self, q):
        W = self.prim(q)
        g = []
        if self.viscous:
            for d in range(3):
                up = 0.5 * (self.prim(self.trace(q, 1, d)) + self.prim(_shift(self.trace(q, 0, d), d, -1)))
                g.append(self.weak(W, up, _shift(up, d, 1), d))
        out = torch.zeros_like(q)
        for d in range(3):
            G = self.euler(q, d)
            L, R = self.trace(q, 1, d), _shift(self.trace(q, 0, d), d, -1)
            hat = self.roe(L, R, d)
            if self.viscous:
                G -= self.stress(q, g, d)
                hat -= 0.5 * (self.stress(L, [self.trace(x, 1, d) for x in g], d)
                              + self.stress(R, [_shift(self.trace(x, 0, d), d, -1) for x in g], d))
            out -= self.weak(G, hat, _shift(hat, d, 1), d)
        return out

    def steps(self, q, dt, n, net=None, post=False, each=None):
        """n low-storage Runge-Kutta steps of q in blocks form."""
        for i in range(n):
            s0 = net(q) if net is not None and post else None
            k = 0.0
            for a, b in zip(RK_A, RK_B):
                R = self.rhs(q)
                if net is not None and not post:
                    R = R + net(q)
                k = a * k + dt * R
                q = q + b * k
            if s0 is not None:
                q = q + dt * s0
            if each is not None:
                each(i + 1, q)
        return q

    def quadrature(self):
        w = self.b.w
        return w[:, None, None] * w[None, :, None] * w[None, None, :]

    def kinetic(self, q):
        return float((self.quadrature() * 0.5 * (q[1] ** 2 + q[2] ** 2 + q[3] ** 2) / q[0]).sum()
                     * (0.5 * self.h) ** 3 / (2.0 * math.pi) ** 3)

    def speed(self, q):
        return float((torch.sqrt((q[1] ** 2 + q[2] ** 2 + q[3] ** 2)) / q[0]
                      + torch.sqrt(GAMMA * self.pressure(q) / q[0])).max())


def _forcing(P, form, seed, device="cuda"):
    """s(q) of the network in float64, on blocks."""
    dims, layers, norm, _ = _net(P, form, seed)
    use = [1, 2, 3] if form == "momenta" else [0, 1, 2, 3, 4]
    Ws = [(torch.from_numpy(W).double().to(device), torch.from_numpy(b).double().to(device)) for W, b in layers]

    def s(q):
        shape = q.shape
        f = q.reshape(5, -1, (P + 1) ** 3)
        h = torch.cat([(f[v] - norm[v]) / norm[5 + v] for v in use], dim=1)
        for i, (W, b) in enumerate(Ws):
            h = h @ W.T + b
            if i + 1 < len(Ws):
                h = torch.relu(h) if form == "momenta" else torch.tanh(h)
        out = torch.zeros_like(f)
        for j, v in enumerate(use):
            out[v] = norm[15 + v] * h[:, j * f.shape[2]:(j + 1) * f.shape[2]] + norm[10 + v]
        return out.reshape(shape)

    return s


def _filter(hi, lo, f):
    """Nodal -> Legendre modes -> truncated -> nodal, per direction."""
    k = np.arange(lo.n)
    Vh = np.polynomial.legendre.legvander(hi.b.x.cpu().numpy(), lo.P)
    Vl = np.polynomial.legendre.legvander(lo.b.x.cpu().numpy(), lo.P)
    G = torch.from_numpy(Vl @ (((2 * k + 1) / 2.0)[:, None] * Vh.T * hi.b.w.cpu().numpy()[None, :])).to(f.device)
    for d in range(3):
        f = _line(f, G, d)
    return f


def _exact_train(case, seed, device):
    x, y, perm = _rows(case, seed, device)
    at = perm[:case["batch"]].long() if case["shuffled"] else slice(0, case["batch"])
    x, y = x[at].double(), y[at].double()
    dims, layers, norm, _ = _net(case["P"], case["form"], seed)
    n_p = (case["P"] + 1) ** 3
    use = [1, 2, 3] if case["form"] == "momenta" else [0, 1, 2, 3, 4]
    h = torch.cat([(x[:, v * n_p:(v + 1) * n_p] - norm[v]) / norm[5 + v] for v in use], dim=1)
    t = torch.cat([(y[:, v * n_p:(v + 1) * n_p] - norm[10 + v]) / norm[15 + v] for v in use], dim=1)
    Ws = [(torch.from_numpy(W).double().to(device).requires_grad_(), torch.from_numpy(b).double().to(device).requires_grad_())
          for W, b in layers]
    for i, (W, b) in enumerate(Ws):
        h = h @ W.T + b
        if i + 1 < len(Ws):
            h = torch.relu(h) if case["form"] == "momenta" else torch.tanh(h)
    loss = ((h - t) ** 2).mean()
    flat = [p for pair in Ws for p in pair]
    g = torch.cat([a.reshape(-1) for a in torch.autograd.grad(loss, flat)])
    p = torch.cat([a.detach().reshape(-1) for a in flat])
    m, v = 0.1 * g, 0.001 * g * g
    return dict(loss=loss.detach().reshape(1), params=p - 1e-3 * g / (g.abs() + 1e-7), grad=g, m=m, v=v)


def _exact_serve(case, seed, device):
    out = []
    for r in _requests(case, seed):
        flow = _Flow(r["N"], r["P"], r["Re"], 0.0, device=device)
        X, Y, Z = _coordinates(r["N"], r["P"], device)
        one = torch.ones((r["N"],) * 3 + (flow.n,) * 3, dtype=torch.float64, device=device)
        u, v = torch.sin(X) * torch.cos(Y) * torch.cos(Z) * one, -torch.cos(X) * torch.sin(Y) * torch.cos(Z) * one
        p = P0 + (torch.cos(2 * X) + torch.cos(2 * Y)) * (torch.cos(2 * Z) + 2.0) / 16.0
        q = torch.stack([one, u, v, 0.0 * one, p / (GAMMA - 1.0) + 0.5 * (u * u + v * v)])
        nn_ = flow.n
        dt = min(0.4 * flow.h / (nn_ ** 2 * flow.speed(q)), 0.4 * flow.h ** 2 * r["Re"] * PRANDTL / (nn_ ** 4 * GAMMA))
        n = max(1, math.ceil(case["t_end"] / dt - 1e-12))
        dt = case["t_end"] / n
        ke = [0.0, flow.kinetic(q)]

        def each(i, s):
            if i % 8 == 0 or i == n:
                ke.extend([i * dt, flow.kinetic(s)])

        net = _forcing(3, "all", seed, device) if r["net"] else None
        q = flow.steps(q, dt, n, net, r["net"] == "post", each)
        ke = np.array((ke + [0.0] * 128)[:128])
        out.append((ke, q.reshape(-1)) if r["N"] <= 8 else ke)
    return out


def exact(case, seed):
    device = "cuda" if torch.cuda.is_available() else "cpu"
    kind = case["kind"]
    if kind == "train":
        return _exact_train(case, seed, device)
    if kind == "serve":
        return _exact_serve(case, seed, device)
    N, P = case["N"], case["P"]
    flow = _Flow(N, P, case["Re"], case["Cs"], case.get("viscous", True), device)
    q0 = _state(N, P, seed, device)
    shape, q = q0.shape, flow.blocks(q0)
    dt = _dt(N, P, case["Re"])
    if kind == "advance":
        net = _forcing(P, case["form"], seed, device) if case["net"] else None
        return flow.steps(q, dt, case["steps"], net, case["net"] == "post").reshape(shape)
    if kind == "residual":
        return flow.rhs(q).reshape(shape)
    lo = _Flow(N, case["P_lo"], case["Re"], case["Cs"], True, device)
    rows = lambda f: f.reshape(5, N ** 3, lo.n ** 3).permute(1, 0, 2).reshape(N ** 3, -1)  # noqa: E731
    if kind == "frame":
        q = flow.steps(q, dt, case["steps"])
        q_lo = _filter(flow, lo, q)
        ref = lo.blocks(_state(N, case["P_lo"], seed + 1, device))
        w = flow.quadrature() * (0.5 * flow.h) ** 3
        diag = [flow.kinetic(q), flow.speed(q), float(q[0].min())] + [float((w * q[v]).sum()) for v in range(5)]
        return dict(q=q.reshape(shape), q_lo=q_lo.reshape(5, N ** 3, -1),
                    err=torch.stack([(q_lo[v] - ref[v]).abs().max() for v in (1, 2, 3)]),
                    diag=np.array(diag))
    q_nn = _filter(flow, lo, q)
    if case["form"] == "eq5":
        return dict(q=q0, x=rows(q_nn), y=rows(_filter(flow, lo, flow.rhs(q)) - lo.rhs(q_nn)))
    dt_lo = dt * case["m_sub"]
    after = lo.steps(q_nn, dt_lo, 1)
    q = flow.steps(q, dt_lo / case["m_sub"], case["m_sub"])
    return dict(q=q.reshape(shape), x=rows(q_nn), y=rows((_filter(flow, lo, q) - after) / dt_lo))
