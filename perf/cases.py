"""Performance cases of the GP-MPPI library: the calls its users make, over the range they make them in.

The kinds of work:
  step    one control iteration of one problem (`Controller.step`): rollout of K samples over T
          steps, weights, control update; every precision form, with or without `gpmppi_tune`
          (a program that runs one problem size for hours tunes it once, a script does not),
          with the terrain ensemble and Step-2 tightening as options
  loop    a stretch of the closed loop on the device (`gpmppi_closed_loop`, HIP graph)
  batch   one iteration of many problems of uneven sizes (`gpmppi_batch_step`, tuned)
  grad    the gradient of the smoothed expected cost (`gpmppi_grad`)
  fit     two iterations of fitting controls and GP hyperparameters by the gradient
          (`expected_cost` and `backward`: every iteration rebuilds the GPs)
  update  new GP data (`gpmppi_set_gp`) and its predictions at n queries (`gpmppi_gp_predict`)

Inputs are the repository's seeded workloads.  The start states are those of a run's beginning: the
robot near its track's start and heading along it, no obstacle within reach of it, a small warm
start.  There the indicator terms of the stage cost are constant over the samples' whole spread, so
two correct evaluations differ by rounding only and not by a cost jump of a sample that grazes a
threshold.
"""
import copy
import math

import numpy as np
import torch

from paper_2411_03289_amd import gpmppi as B
from paper_2411_03289_amd import workloads as W

PRECISION = {"fp32": B.FP32, "bf16": B.BF16, "bf16x3": B.BF16X3}
AMPLITUDE = W.RESIDUAL_AMPLITUDE
TAU, CHECKPOINT = 0.05, 10
CLEARANCE = 2.5   # metres around the start kept free of obstacles


def listed():
    return [
        # the smallest instance of the repository (256 samples, 50 training points), as a script
        # calls it: launches and per-step latency
        dict(name="step_small", kind="step", form="fp32", K=256, T=20, M=50, n_obs=5, path="circle", tune=False),
        # the paper's GP of 300 training points, sizes that are no multiple of a tile, untuned
        dict(name="step_paper_300", kind="step", form="fp32", K=2500, T=40, M=300, n_obs=12, path="eight", tune=False),
        # the mid-size controller of the tests and the closed loop, untuned, in the accurate BF16 form
        dict(name="step_mid_bf16x3", kind="step", form="bf16x3", K=4096, T=50, M=256, n_obs=20, path="eight", tune=False),
        # terrain ensemble and tightening along the nominal sequence (the paper's Step 2)
        dict(name="step_tighten_terrain", kind="step", form="fp32", K=2048, T=30, M=256, n_obs=20, path="eight",
             tune=False, tighten=1, terrains=3),
        # the headline workload, each form at its tuned shape
        dict(name="step_large_bf16", kind="step", form="bf16", K=16384, T=100, M=1024, n_obs=50, path="eight", tune=True),
        dict(name="step_large_bf16x3", kind="step", form="bf16x3", K=16384, T=100, M=1024, n_obs=50, path="eight",
             tune=True),
        dict(name="step_large_fp32", kind="step", form="fp32", K=16384, T=100, M=1024, n_obs=50, path="eight", tune=True),
        # half a second of driving at 20 Hz, on the device, from a standing start of the run
        dict(name="loop_mid", kind="loop", form="fp32", K=4096, T=50, M=256, n_obs=20, path="eight", tune=True, n=10),
        # a fleet: problems of uneven K, T, M, obstacle count and track in one call
        dict(name="batch_16", kind="batch", form="fp32", n=16, first=0),
        # the gradient's own workload
        dict(name="grad_mid", kind="grad", K=4096, T=50, M=512, n_obs=20, path="eight"),
        # hyperparameter and control fitting: GP rebuild, gradient, autograd, twice per pass
        dict(name="fit_small", kind="fit", K=256, T=20, M=200, n_obs=5, path="circle"),
        # online learning: a new GP from 1024 points, then predictions at a ragged number of queries
        dict(name="update_1024", kind="update", form="fp32", M=1024, n=1000),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step"] * 5 + ["loop", "batch", "grad", "fit", "update"])
    path = rng.choice(["circle", "eight"])
    form = rng.choice(["fp32", "bf16", "bf16x3"])
    if kind == "step":
        while True:
            K, T, M = _log(rng, 64, 16384), _log(rng, 10, 100), _log(rng, 16, 1024)
            if rng.random() < 0.3:
                M = rng.choice([64, 256, 512, 1024])
            case = dict(kind=kind, form=form, K=K, T=T, M=M, n_obs=rng.randint(0, 50), path=path,
                        tune=rng.random() < 0.5)
            if rng.random() < 0.2:
                case["tighten"] = 1
            if rng.random() < 0.2:
                case["terrains"] = rng.randint(2, 3)
            return case
    if kind == "loop":
        return dict(kind=kind, form=form, K=_log(rng, 256, 8192), T=_log(rng, 15, 60), M=_log(rng, 50, 512),
                    n_obs=rng.randint(0, 30), path=path, tune=rng.random() < 0.7, n=rng.randint(3, 8))
    if kind == "batch":
        case = dict(kind=kind, form=form, n=rng.randint(3, 16), first=rng.randint(0, 48))
        most = work(listed()[6])["flops"]
        while work(case)["flops"] > most:
            case["n"] -= 1
        return case
    if kind == "grad":
        return dict(kind=kind, K=_log(rng, 64, 4096), T=_log(rng, 10, 50), M=_log(rng, 40, 512),
                    n_obs=rng.randint(0, 20), path=path)
    if kind == "fit":
        return dict(kind=kind, K=_log(rng, 64, 1024), T=_log(rng, 10, 40), M=_log(rng, 40, 512),
                    n_obs=rng.randint(0, 20), path=path)
    return dict(kind=kind, form=form, M=_log(rng, 50, 1024), n=_log(rng, 100, 20000))


# ---------------------------------------------------------------- inputs
def _start(pr, rng):
    """Start state and warm start near the beginning of the run; obstacles out of its reach."""
    o = pr.obstacles
    if len(o):
        clear = np.hypot(o[:, 0] - pr.x0[0], o[:, 1] - pr.x0[1]) - o[:, 2] > CLEARANCE
        pr.obstacles = np.ascontiguousarray(o[clear])
    x0 = (pr.x0 + rng.uniform(-1.0, 1.0, 5) * np.array([0.05, 0.05, 0.1, 0.2, 0.1])).astype(np.float32)
    U = (0.2 * rng.uniform(-1.0, 1.0, (pr.T, 2))).astype(np.float32)
    return x0, U


def _problem(case, seed):
    """One problem, its start state, its warm start and the noise seed, all from the seed alone."""
    rng = np.random.Generator(np.random.PCG64([seed, 11]))
    path = case.get("path", "eight")
    small = path == "circle"
    over = dict(K=case.get("K", 64), T=case.get("T", 10), M=case["M"], n_obs=case.get("n_obs", 5), path=path,
                seed_data=50_000 + seed)
    if small and case["M"] <= 50:
        over["N"] = case["M"]
    pr = W.make_config(0 if small else 1, **over)
    pr.params = dict(pr.params)
    if case.get("tighten"):
        pr.params["tighten"] = 1
    if case.get("terrains"):
        n = case["terrains"]
        W.add_terrains(pr, 60_000 + seed, weights=np.array((0.5, 0.3, 0.2)[:n]) / sum((0.5, 0.3, 0.2)[:n]), n_terr=n)
    x0, U = _start(pr, rng)
    return pr, x0, U, int(rng.integers(1, 2 ** 40))


def _batch(case, seed):
    prs, x0s, Us = [], [], []
    rng = np.random.Generator(np.random.PCG64([seed, 12]))
    for pid in range(case["first"], case["first"] + case["n"]):
        pr = W.make_batch_problem(pid)   # the sizes are the fleet's own, whatever the seed
        M, n_obs = pr.M, len(pr.obstacles)
        data = W.make_config(1, K=pr.K, T=pr.T, M=M, n_obs=n_obs, seed_data=70_000 + 100 * seed + pid)
        pr.Z, pr.y, pr.obstacles = data.Z, data.y, data.obstacles
        x0, U = _start(pr, rng)
        prs.append(pr)
        x0s.append(x0)
        Us.append(U)
    return prs, x0s, Us, int(rng.integers(1, 2 ** 40))


def _hyper(pr, seed):
    """Two hyperparameter settings a fit passes through."""
    rng = np.random.Generator(np.random.PCG64([seed, 13]))
    return [(pr.log_ell + 0.1 * rng.uniform(-1, 1, (2, 4)), pr.log_sf + 0.1 * rng.uniform(-1, 1, 2)) for _ in range(2)]


def _dev(a):
    return torch.as_tensor(np.asarray(a), dtype=torch.float32, device="cuda").contiguous()


def prepare(case, seed):
    kind, s = case["kind"], dict(kind=case["kind"])
    if kind == "batch":
        prs, x0s, Us, s["seed"] = _batch(case, seed)
        s["b"] = B.gpmppi_batch_init(prs, PRECISION[case["form"]])
        s["x0"] = _dev(np.concatenate(x0s))
        s["U"] = _dev(np.concatenate([u.reshape(-1) for u in Us]))
        B.gpmppi_batch_tune(s["b"], s["x0"], s["U"], s["seed"], 1)
        nK = s["b"].K_off[-1]
        s["out"] = [torch.empty_like(s["U"])] + [torch.empty(nK, device="cuda") for _ in range(2)]
        return s
    pr, x0, U, s["seed"] = _problem(case, seed)
    s["pr"], s["x0"], s["U"] = pr, _dev(x0), _dev(U)
    if kind == "step":
        s["ctrl"] = B.Controller(pr, PRECISION[case["form"]])
        if case["tune"]:
            B.gpmppi_tune(s["ctrl"].ctx, s["x0"], s["U"], s["seed"], 3)
    elif kind == "loop":
        s["n"] = case["n"]
        s["ctx"] = B.gpmppi_init(pr, PRECISION[case["form"]])
        if case["tune"]:
            B.gpmppi_tune(s["ctx"], s["x0"], s["U"], s["seed"], 3)
        s["hist"] = torch.empty(case["n"] + 1, 5, device="cuda")
        s["U0"] = torch.empty(case["n"], 2, device="cuda")
    elif kind == "grad":
        s["ctx"] = B.gpmppi_init(pr, B.FP32)
        s["every"] = min(CHECKPOINT, pr.T)
        s["out"] = [torch.empty(n, device="cuda") for n in (1, 2 * pr.T, 8, 2, pr.K)]
    elif kind == "fit":
        s["gp"] = B.GradProblem(pr, seed=s["seed"], tau=TAU, checkpoint_every=CHECKPOINT, x0=x0)
        s["hyper"] = [(torch.tensor(le, dtype=torch.float64, requires_grad=True),
                       torch.tensor(ls, dtype=torch.float64, requires_grad=True)) for le, ls in _hyper(pr, seed)]
        s["U"].requires_grad_(True)
    else:
        s["ctx"] = B.gpmppi_init(pr, PRECISION[case["form"]])
        s["q"] = _dev(W.random_queries(case["n"], 80_000 + seed))
        s["new"] = copy.copy(_problem(case, seed + 500_000)[0])
        s["out"] = [torch.empty(2, case["n"], device="cuda") for _ in range(2)]
    return s


def run(s):
    kind = s["kind"]
    if kind == "step":
        U, costs, weights = s["ctrl"].step(s["x0"], s["U"], s["seed"])
        return {"U": U, "costs": costs, "weights": weights}
    if kind == "loop":
        x, U = s["x0"].clone(), s["U"].clone()   # an episode begins at its start state
        B.gpmppi_closed_loop(s["ctx"], x, U, s["seed"], s["n"], AMPLITUDE, s["hist"], s["U0"], use_graph=True)
        return {"x": x, "U": U, "hist": s["hist"], "U0": s["U0"]}
    if kind == "batch":
        U, costs, weights = s["out"]
        B.gpmppi_batch_step(s["b"], s["x0"], s["U"], s["seed"], U, costs, weights)
        return {"U": U, "costs": costs, "weights": weights}
    if kind == "grad":
        J, dU, dle, dls, costs = s["out"]
        B.gpmppi_grad(s["ctx"], s["x0"], s["U"], s["seed"], TAU, s["every"], J, dU, dle, dls, costs)
        return {"J": J, "dU": dU, "dlog_ell": dle, "dlog_sf": dls, "costs": costs}
    if kind == "fit":
        out = []
        for le, ls in s["hyper"]:
            s["U"].grad = le.grad = ls.grad = None
            J = B.expected_cost(s["gp"], s["U"], le, ls)
            J.backward()
            out.append({"J": J.detach(), "dU": s["U"].grad, "dlog_ell": le.grad.float(), "dlog_sf": ls.grad.float()})
        return out
    mean, var = s["out"]
    B.gpmppi_set_gp(s["ctx"], s["new"])
    B.gpmppi_gp_predict(s["ctx"], s["q"], mean, var)
    return {"mean": mean, "var": var}


# ---------------------------------------------------------------- work
def _rollout_flops(K, T, M, n_obs, P):
    # both outputs: triangular variance contraction, kernel vectors and means; dynamics and world
    return float(K) * T * (2 * M * (M + 1) + 2 * M * (3 * 4 + 1) + 4 * M + 150 + 25 * n_obs + 12 * P)


def _build_flops(M):
    return 2 * (M ** 3 / 3 + M ** 3 / 3 + 2.0 * M * M)   # Cholesky, triangular inverse, alpha, both outputs


def work(case):
    kind = case["kind"]
    if kind == "batch":
        flops = bytes_ = 0.0
        for pid in range(case["first"], case["first"] + case["n"]):
            p = W.make_batch_problem(pid)
            flops += _rollout_flops(p.K, p.T, p.M, len(p.obstacles), len(p.path_pts))
            bytes_ += 2 * 20 * p.M + 8 * p.K + 16 * p.T + 4 * p.M * (p.M + 1)
        return {"bytes": bytes_, "flops": flops}
    M = case["M"]
    gp_bytes = 2 * 20 * M + 4 * M * (M + 1)   # scaled inputs, alpha and triangular factor of both outputs
    if kind == "update":
        return {"bytes": 2 * 40 * M + 32 * case["n"],
                "flops": _build_flops(M) + case["n"] * (2.0 * M * (M + 1) + 30 * M)}
    K, T = case["K"], case["T"]
    roll = _rollout_flops(K, T, M, case["n_obs"], 256 if case["path"] == "eight" else 0)
    if kind == "step":
        return {"bytes": gp_bytes + 8 * K + 16 * T, "flops": roll}
    if kind == "loop":
        return {"bytes": case["n"] * (gp_bytes + 28) + 16 * T, "flops": roll * case["n"]}
    # forward, r = (K + sn^2 I)^-1 k of every sample-step, and the symmetric sum of r r^T, both outputs
    grad = roll + float(K) * T * (2 * 2 * M * M + 2 * M * M)
    if kind == "grad":
        return {"bytes": gp_bytes + 4 * K + 16 * T, "flops": grad}
    return {"bytes": 2 * (2 * 40 * M + 16 * T), "flops": 2 * (grad + _build_flops(M))}


# ---------------------------------------------------------------- 64-bit reference
# The method in plain float64 torch: Philox4x32-10 noise, GP regression by Cholesky, Euler unicycle,
# covariance, tightened constraints, costs, weights; gradients by autograd.
def _philox(c, key):
    mask = 0xFFFFFFFF
    k0, k1 = key & mask, (key >> 32) & mask
    x0, x1, x2, x3 = c

    def mul(m, x):   # m x over 32-bit words, in 64-bit integers
        lo, hi = m * (x & 0xFFFF), m * (x >> 16)
        s = (lo >> 16) + hi
        return (s >> 16) & mask, ((s & 0xFFFF) << 16) | (lo & 0xFFFF)

    for r in range(10):
        if r:
            k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
        h0, l0 = mul(0xD2511F53, x0)
        h1, l1 = mul(0xCD9E8D57, x2)
        x0, x1, x2, x3 = h1 ^ x1 ^ k0, l1, h0 ^ x3 ^ k1, l0
    return x0, x1


def _noise(pr, K, seed, dev):
    k = torch.arange(pr.T, device=dev, dtype=torch.int64)[:, None].expand(pr.T, K)
    s = torch.arange(K, device=dev, dtype=torch.int64)[None, :].expand(pr.T, K)
    w0, w1 = _philox((k, s, torch.full_like(k, pr.pid), torch.zeros_like(k)), seed)
    u1, u2 = (((w >> 9).double() + 0.5) * 2.0 ** -23 for w in (w0, w1))
    r = torch.sqrt(-2.0 * torch.log(u1))
    return torch.stack([pr.params["sig_v"] * r * torch.cos(2 * math.pi * u2),
                        pr.params["sig_w"] * r * torch.sin(2 * math.pi * u2)], -1)


class _Gp64:
    """Both outputs' GPs in float64 on `dev`; hyperparameters may be tensors that need gradients."""

    def __init__(self, pr, dev, log_ell=None, log_sf=None):
        d = dict(dtype=torch.float64, device=dev)
        le = torch.as_tensor(pr.log_ell, **d) if log_ell is None else log_ell
        self.sf2 = torch.exp(2 * (torch.as_tensor(pr.log_sf, **d) if log_sf is None else log_sf))
        self.sn2 = torch.exp(2 * torch.as_tensor(pr.log_sn, **d))
        self.iell = torch.exp(-le)
        Z = torch.as_tensor(pr.Z, **d)
        w = None if pr.terrain_y is None else torch.as_tensor(pr.terrain_w, **d)
        y = torch.as_tensor(pr.y, **d) if w is None else torch.einsum("i,iom->om", w, torch.as_tensor(pr.terrain_y, **d))
        self.vs = 1.0 if w is None else float((w * w).sum())
        self.z, self.inv, self.alpha = [], [], []
        for o in range(2):
            z = Z[o] * self.iell[o]
            A = self.kernel(o, z, z) + self.sn2[o] * torch.eye(len(z), **d)
            L = torch.linalg.cholesky(A)
            self.z.append(z)
            self.inv.append(torch.cholesky_inverse(L))
            self.alpha.append(torch.cholesky_solve(y[o][:, None], L)[:, 0])

    def kernel(self, o, a, b):
        r2 = sum((a[:, None, d] - b[None, :, d]) ** 2 for d in range(4))
        return self.sf2[o] * torch.exp(-0.5 * r2)

    def __call__(self, q):
        m, s2 = [], []
        for o in range(2):
            k = self.kernel(o, q * self.iell[o], self.z[o])
            m.append(k @ self.alpha[o])
            lat = self.sf2[o] - ((k @ self.inv[o]) * k).sum(1)
            s2.append(self.vs * (self.sn2[o] + torch.clamp(lat, min=0.0)))
        return m, s2


def _world(pr, p, S, dev):
    """Distance to the centreline, tightened half-width and least tightened obstacle distance."""
    a, b, c = S[0][0], S[0][1], S[1][1]
    h = 0.5 * (a - c)
    e2 = h * h + b * b   # the derivative of sqrt at 0 is taken as 0
    lmax = 0.5 * (a + c) + torch.where(e2 > 0, torch.sqrt(torch.where(e2 > 0, e2, 1.0)), 0.0)
    pos = torch.where(lmax > 0, torch.sqrt(torch.where(lmax > 0, lmax, 1.0)), 0.0)
    rbar = pr.params["half_width"] - math.sqrt(-2.0 * math.log1p(-pr.params["p_x"])) * pos
    d = dict(dtype=torch.float64, device=dev)
    if pr.path_kind == 0:
        dl = torch.abs(torch.sqrt((p[0] - pr.circle[0]) ** 2 + (p[1] - pr.circle[1]) ** 2) - pr.circle[2])
    else:
        v = torch.as_tensor(pr.path_pts, **d)
        e = torch.roll(v, -1, 0) - v
        rx, ry = p[0][:, None] - v[:, 0], p[1][:, None] - v[:, 1]
        t = torch.clamp((rx * e[:, 0] + ry * e[:, 1]) / (e * e).sum(1), 0.0, 1.0)
        d2 = ((rx - t * e[:, 0]) ** 2 + (ry - t * e[:, 1]) ** 2).min(1).values
        dl = torch.where(d2 > 0, torch.sqrt(torch.where(d2 > 0, d2, 1.0)), 0.0)
    if not len(pr.obstacles):
        return dl, rbar, torch.full_like(dl, math.inf)
    ob = torch.as_tensor(pr.obstacles, **d)
    dx, dy = p[0][:, None] - ob[:, 0], p[1][:, None] - ob[:, 1]
    rho2 = dx * dx + dy * dy
    rho = torch.sqrt(rho2)
    a, b, c = (x.reshape(-1, 1) for x in (a, b, c))
    var = (a * dx * dx + 2 * b * dx * dy + c * dy * dy) / rho2
    sd = torch.where(var > 0, torch.sqrt(torch.where(var > 0, var, 1.0)), 0.0)
    z = math.sqrt(2.0) * float(torch.erfinv(torch.tensor(2.0 * pr.params["p_x"] - 1.0, dtype=torch.float64)))
    return dl, rbar, ((rho - ob[:, 2]) - z * sd).min(1).values


def _rollout64(pr, gp, x0, U, seed, dev, K=None, smooth=None, noise=True):
    """Costs [K], sampled controls [T][K][2] and Sigma_XY per step; smooth: the indicators' temperature."""
    P, K = pr.params, K or pr.K
    dt, it, iw = P["dt"], P["dt"] / P["tau_v"], P["dt"] / P["tau_w"]
    lo, hi = (torch.tensor(P[n], dtype=torch.float64, device=dev) for n in ("u_min", "u_max"))
    eps = _noise(pr, K, seed, dev) if noise else 0.0
    u = torch.clamp(U[:, None, :] + eps, lo, hi)
    if not noise:
        u = u.expand(pr.T, K, 2)
    tight = _rollout64(pr, gp, x0, U, 0, dev, K=1, noise=False)[2] if noise and P.get("tighten") else None
    x = [x0[i].expand(K).clone() for i in range(5)]
    S = [[torch.zeros(K, dtype=torch.float64, device=dev) for _ in range(5)] for _ in range(5)]
    cost, pos = torch.zeros(K, dtype=torch.float64, device=dev), []
    for k in range(pr.T):
        m, s2 = gp(torch.stack([x[3], x[4], u[k, :, 0], u[k, :, 1]], 1))
        sn, cs = torch.sin(x[2]), torch.cos(x[2])
        one = torch.ones(K, dtype=torch.float64, device=dev)
        A = {(0, 2): -dt * x[3] * sn, (0, 3): dt * cs, (1, 2): dt * x[3] * cs, (1, 3): dt * sn, (2, 4): dt * one,
             (0, 0): one, (1, 1): one, (2, 2): one, (3, 3): (1 - it) * one, (4, 4): (1 - iw) * one}
        AS = [[sum(A[i, n] * S[n][j] for n in range(5) if (i, n) in A) for j in range(5)] for i in range(5)]
        S = [[sum(AS[i][n] * A[j, n] for n in range(5) if (j, n) in A) for j in range(5)] for i in range(5)]
        S[3][3] = S[3][3] + dt * dt * s2[0]
        S[4][4] = S[4][4] + dt * dt * s2[1]
        x = [x[0] + dt * x[3] * cs, x[1] + dt * x[3] * sn, x[2] + dt * x[4],
             x[3] + it * (u[k, :, 0] - x[3]) + dt * m[0], x[4] + iw * (u[k, :, 1] - x[4]) + dt * m[1]]
        pos.append([S[0][0], S[0][1], S[1][1]])
        C = S
        if tight is not None:
            C = [[tight[k][0], tight[k][1]], [None, tight[k][2]]]
        dl, rbar, om = _world(pr, x, C, dev)
        lane = (dl > rbar).double() if smooth is None else torch.sigmoid((dl - rbar) / smooth)
        hit = (om <= 0).double() if smooth is None else torch.sigmoid(-om / smooth)
        cost = cost + (P["w_var"] * (s2[0] + s2[1]) + P["w_dev"] * dl / P["half_width"]
                       + P["w_lane"] * P["discount"] ** k * lane + P["w_speed"] * (P["v_des"] - x[3]) ** 2
                       + P["w_obs"] * hit)
    return cost, u, pos


def _step64(pr, gp, x0, U, seed, dev):
    cost, u, _ = _rollout64(pr, gp, x0, U, seed, dev)
    w = torch.softmax(-(cost - cost.min()) / pr.params["lam"], 0)
    return torch.einsum("s,tsc->tc", w, u), cost, w


def _grad64(pr, x0, U, le, ls, seed, dev):
    U, le, ls = (torch.as_tensor(np.asarray(a), dtype=torch.float64, device=dev).requires_grad_(True)
                 for a in (U, le, ls))
    costs = _rollout64(pr, _Gp64(pr, dev, le, ls), x0, U, seed, dev, smooth=TAU)[0]
    J = costs.mean()
    dU, dle, dls = torch.autograd.grad(J, (U, le, ls))
    return J.detach(), dU, dle, dls, costs.detach()


def exact(case, seed):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    d = dict(dtype=torch.float64, device=dev)
    kind = case["kind"]
    if kind == "batch":
        prs, x0s, Us, noise = _batch(case, seed)
        got = []
        for pr, x0, U in zip(prs, x0s, Us):
            got.append(_step64(pr, _Gp64(pr, dev), torch.as_tensor(x0, **d), torch.as_tensor(U, **d), noise, dev))
        U, costs, w = (torch.cat([g[i].reshape(-1) for g in got]) for i in range(3))
        return {"U": U, "costs": costs, "weights": w}
    pr, x0, U, noise = _problem(case, seed)
    if kind == "update":
        new = _problem(case, seed + 500_000)[0]
        q = torch.as_tensor(W.random_queries(case["n"], 80_000 + seed).astype(np.float32), **d)
        m, s2 = _Gp64(new, dev)(q)
        return {"mean": torch.stack(m), "var": torch.stack(s2)}
    x, U64 = torch.as_tensor(x0, **d), torch.as_tensor(U, **d)
    if kind == "grad":
        J, dU, dle, dls, costs = _grad64(pr, x, U, pr.log_ell, pr.log_sf, noise, dev)
        return {"J": J.reshape(1), "dU": dU.reshape(-1), "dlog_ell": dle.reshape(-1), "dlog_sf": dls, "costs": costs}
    if kind == "fit":
        out = []
        for le, ls in _hyper(pr, seed):
            J, dU, dle, dls, _ = _grad64(pr, x, U, le, ls, noise, dev)
            out.append({"J": J, "dU": dU, "dlog_ell": dle, "dlog_sf": dls})
        return out
    gp = _Gp64(pr, dev)
    if kind == "step":
        U1, cost, w = _step64(pr, gp, x, U64, noise, dev)
        return {"U": U1, "costs": cost, "weights": w}
    P, hist, U0 = pr.params, [x], []
    for t in range(case["n"]):
        U1 = _step64(pr, gp, x, U64, noise + t, dev)[0]
        u, res = U1[0], AMPLITUDE * torch.sin(x[3] * x[4])
        x = torch.stack([x[0] + P["dt"] * x[3] * torch.cos(x[2]), x[1] + P["dt"] * x[3] * torch.sin(x[2]),
                         x[2] + P["dt"] * x[4], x[3] + P["dt"] / P["tau_v"] * (u[0] - x[3]) + P["dt"] * res,
                         x[4] + P["dt"] / P["tau_w"] * (u[1] - x[4]) + P["dt"] * res])
        U64 = torch.cat([U1[1:], U1[-1:]])
        hist.append(x)
        U0.append(u)
    return {"x": x, "U": U64, "hist": torch.stack(hist), "U0": torch.stack(U0)}
