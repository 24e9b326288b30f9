"""Workloads of the library as a caller runs them, for timing and comparing outputs.

Every case is one call (or the few calls that belong together) of the public
binding: a chief near the Earth-Moon L1/L2 region, a deputy a small offset
away, evenly spaced azimuth/elevation observations with Gaussian noise, and
candidate states from a box around the chief. Sizes are those of the small,
single-large-swarm, uneven-batch and refinement workloads and what lies
between them; ``draw`` spreads over the same ranges.

  eval       fitness of m particles of one problem
  propagate  states of m particles at K sample times (the close-approach screen)
  predict    angles of m particles at the observation times
  grad       differentiable cost: forward and backward
  normal     Gauss-Newton normal equations
  solve      a whole swarm solve on the library's own storage
  swarm      a swarm in the caller's arrays: initialise, iterate, read the best
  batch      FP64 swarms of many uneven problems
  eval32     FP32 fitness of many uneven problems
  mixed      mixed-precision swarms of many uneven problems
  refine     mixed-precision swarms, then Gauss-Newton refinement
"""
import numpy as np
import torch

import paper_2207_13175_amd as iod

MU = 0.012150585
L1_X, L2_X = 0.8369151288, 1.1556821631
SIGMA, SIGMA_RANGE = 1e-5, 1e-7
BATCHED = ("batch", "eval32", "mixed", "refine")

# flop-equivalents (square root, division and arctangent count one each)
STEP, OBS, UPDATE = 186, 27, 50
# tangent of one RK4 step: four products of the 6x6 stage Jacobian with the
# state transition matrix, and their combination (6 columns)
TANGENT = 6 * (4 * 20 + 3 * 12 + 12)
# transposed tangent of one RK4 step applied to one vector
COTANGENT = 4 * 20 + 6 * 9


def listed():
    return [
        # the smallest useful call: one small swarm's fitness (256 particles, 500 steps)
        dict(name="eval_small", kind="eval", m=256, K=10, per=50, h=1e-3, chi2=False, ranged=False,
             offgrid=False),
        # an odd-sized swarm with ranges and off-grid observation times, least-squares cost
        dict(name="eval_ragged", kind="eval", m=5001, K=37, per=61, h=1e-3, chi2=True, ranged=True,
             offgrid=True),
        # the close-approach screen of a workload generator: many sample times, states out
        dict(name="propagate_screen", kind="propagate", m=2048, K=620, per=5, h=1e-3, chi2=False,
             ranged=False, offgrid=False),
        # gradient-based use: differentiable cost, forward and backward
        dict(name="grad_medium", kind="grad", m=1000, K=40, per=50, h=1e-3, chi2=True, ranged=False,
             offgrid=False),
        # normal equations of a handful of candidates
        dict(name="normal_few", kind="normal", m=96, K=60, per=42, h=1e-3, chi2=True, ranged=False,
             offgrid=False),
        # the small workload solved whole
        dict(name="solve_small", kind="solve", m=256, K=10, per=50, h=1e-3, n_iter=100, chi2=False,
             ranged=False, offgrid=False),
        # a medium swarm over the long arc, solved whole
        dict(name="solve_medium", kind="solve", m=12000, K=40, per=100, h=5e-4, n_iter=4,
             chi2=False, ranged=False, offgrid=False),
        # the single large swarm, a few iterations in the caller's arrays
        dict(name="swarm_large", kind="swarm", m=65536, K=40, per=100, h=5e-4, n_iter=3, chi2=False,
             ranged=False, offgrid=False),
        # uneven problems in FP64
        dict(name="batch_uneven", kind="batch", P=256, m_lo=512, m_hi=8192, K_lo=5, K_hi=80,
             T_lo=0.2, T_hi=3.0, n_iter=4),
        # their FP32 fitness alone, absolute state
        dict(name="eval32_uneven", kind="eval32", P=256, m_lo=512, m_hi=8192, K_lo=5, K_hi=80,
             T_lo=0.2, T_hi=3.0, offset=False),
        # and their mixed-precision solve, offset from the chief
        dict(name="mixed_uneven", kind="mixed", P=256, m_lo=512, m_hi=8192, K_lo=5, K_hi=80,
             T_lo=0.2, T_hi=3.0, n_iter=4, offset=True),
        # a short mixed-precision swarm and the refinement of its best particles
        dict(name="refine_short", kind="refine", P=384, m_lo=2048, m_hi=2048, K_lo=10, K_hi=60,
             T_lo=0.5, T_hi=2.5, n_iter=5, n_cand=16, n_gn=40, offset=False),
    ]


def _log(rng, lo, hi):
    return int(round(np.exp(rng.uniform(np.log(lo), np.log(hi)))))


def draw(rng):
    kind = rng.choice(["eval", "eval", "propagate", "predict", "grad", "normal", "solve", "swarm",
                       "batch", "eval32", "mixed", "refine"])
    if kind in BATCHED:
        c = dict(kind=kind, P=_log(rng, 16, 256), m_lo=512, m_hi=_log(rng, 1024, 8192), K_lo=5,
                 K_hi=rng.randint(20, 80), T_lo=0.2, T_hi=rng.uniform(1.0, 3.0))
        if kind != "eval32":
            c["n_iter"] = rng.randint(1, 4)
        if kind != "batch":
            c["offset"] = rng.random() < 0.5
        if kind == "refine":
            c.update(n_cand=rng.choice([4, 8, 16, 32]), n_gn=rng.randint(5, 40))
        return c
    top = {"eval": 65536, "propagate": 4096, "predict": 20000, "grad": 8192, "normal": 8192,
           "solve": 32768, "swarm": 65536}[kind]
    K = rng.randint(3, 80)
    fine = rng.random() < 0.4
    c = dict(kind=kind, m=_log(rng, 40, top), K=K, per=max(2, _log(rng, 200, 4000 if fine else 2500) // K),
             h=5e-4 if fine else 1e-3, chi2=rng.random() < 0.5, ranged=rng.random() < 0.3,
             offgrid=rng.random() < 0.3)
    if kind in ("solve", "swarm"):
        c["n_iter"] = rng.randint(1, 20 if c["m"] < 2048 else 4)
    return c


# --------------------------------------------------------------------------
# Inputs: numpy draws and the simulated measurements (host)
# --------------------------------------------------------------------------

def _deriv(s):
    x, y, z, vx, vy, vz = s
    d1, d2, q = x + MU, x - (1 - MU), y * y + z * z
    c1 = (1 - MU) / (d1 * d1 + q) ** 1.5
    c2 = MU / (d2 * d2 + q) ** 1.5
    return np.array([vx, vy, vz, 2 * vy + x - c1 * d1 - c2 * d2, -2 * vx + y - (c1 + c2) * y,
                     -(c1 + c2) * z])


def _paths(s0, t):
    """Trajectories of s0 [6, n] (numpy RK4, steps of at most 0.004 TU) at each
    one's own times t [n][K_n]: list of [K_n, 6]."""
    n = s0.shape[1]
    sub = np.array([int(np.ceil((tk[1] - tk[0] if len(tk) > 1 else tk[0]) / 0.004)) for tk in t])
    out = [np.empty((len(tk), 6)) for tk in t]
    ends = np.array([len(tk) for tk in t]) * sub
    first = np.array([tk[0] for tk in t])
    step = np.array([tk[1] - tk[0] if len(tk) > 1 else tk[0] for tk in t])
    s = s0.copy()
    for j in range(int(ends.max())):
        dt = np.where(j < sub, first, step) / sub
        k1 = _deriv(s)
        k2 = _deriv(s + dt / 2 * k1)
        k3 = _deriv(s + dt / 2 * k2)
        k4 = _deriv(s + dt * k3)
        s = s + dt / 6 * (k1 + 2 * k2 + 2 * k3 + k4)
        for p in np.flatnonzero(((j + 1) % sub == 0) & (j < ends)):
            out[p][(j + 1) // sub[p] - 1] = s[:, p]
    return out


def _problem(rng, box):
    base = L1_X if rng.random() < 0.5 else L2_X
    chief = np.zeros(6)
    chief[0] = base + rng.uniform(-0.02, 0.02)
    chief[2] = rng.uniform(-0.1, 0.1)
    d = rng.standard_normal(3)
    chief[3:] = d / np.linalg.norm(d) * 0.3 * rng.random() ** (1 / 3)
    d = rng.standard_normal(3)
    truth = chief + np.concatenate([d / np.linalg.norm(d) * box / 2 * rng.random() ** (1 / 3),
                                    rng.uniform(-box / 2, box / 2, 3)])
    return chief, truth


def _near(path):
    """Whether a path passes within 0.05 LU of the Moon or 0.1 LU of the Earth."""
    moon = np.linalg.norm(path[:, :3] - [1 - MU, 0, 0], axis=1).min()
    earth = np.linalg.norm(path[:, :3] - [-MU, 0, 0], axis=1).min()
    return not (moon > 0.05 and earth > 0.1)


def _inputs(case, seed):
    """Problems of a case: chief, truth, times, observed angles and ranges.
    The sizes of a batch's problems belong to the case, the rest to the seed."""
    P = case.get("P", 1)
    rngs = [np.random.default_rng([seed, p]) for p in range(P)]
    sizes = np.random.default_rng([P, case.get("m_hi", 0), case.get("K_hi", 0)])
    box = 2e-3 if "P" in case or case["per"] * case["K"] < 1000 else 1e-2
    chief, truth, t, m = np.zeros((P, 6)), np.zeros((P, 6)), [None] * P, np.zeros(P, dtype=np.int64)
    paths = [None] * (2 * P)
    for p in range(P):
        if "P" in case:
            K = int(sizes.integers(case["K_lo"], case["K_hi"] + 1))
            per = max(1, int(round(sizes.uniform(case["T_lo"], case["T_hi"]) / (K * 1e-3))))
            t[p] = np.arange(1, K + 1) * (per * 1e-3)
            m[p] = int(round(np.exp(sizes.uniform(np.log(case["m_lo"]), np.log(case["m_hi"])))))
        else:
            t[p] = np.arange(1, case["K"] + 1) * (case["per"] * case["h"])
            if case["offgrid"]:
                t[p] = t[p] - 0.37 * case["h"]
            m[p] = case["m"]
    todo = list(range(P))
    for _ in range(200):
        for p in todo:
            chief[p], truth[p] = _problem(rngs[p], box)
        s0 = np.concatenate([chief[todo], truth[todo]]).T.copy()
        got = _paths(s0, [t[p] for p in todo] * 2)
        for i, p in enumerate(todo):
            paths[p], paths[P + p] = got[i], got[len(todo) + i]
        todo = [p for p in todo if _near(paths[p]) or _near(paths[P + p])]
        if not todo:
            break
    angles, ranges = [], []
    for p in range(P):
        rho = paths[P + p][:, :3] - paths[p][:, :3]
        r = np.linalg.norm(rho, axis=1)
        n = rngs[p].standard_normal((len(t[p]), 3))
        angles.append(np.stack([np.arctan2(rho[:, 1], rho[:, 0]), np.arcsin(rho[:, 2] / r)], 1)
                      + SIGMA * n[:, :2])
        ranges.append(np.abs(r + SIGMA_RANGE * n[:, 2]))
    return dict(chief=chief, truth=truth, t=t, angles=angles, ranges=ranges, m=m, box=box,
                lo=chief - box, hi=chief + box)


def _states(case, I, seed, ld, off):
    """Candidate states [6, ld] on the GPU: uniform in each problem's box."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    x = torch.rand((6, ld), generator=g, dtype=torch.float64, device="cuda")
    lo = torch.from_numpy(I["lo"]).cuda()
    if case["kind"] in BATCHED:
        col = torch.zeros(ld, dtype=torch.int64, device="cuda")
        for p in range(len(off) - 1):
            col[off[p]:off[p + 1]] = p
        return lo.t()[:, col] + 2 * I["box"] * x
    return lo[0][:, None] + 2 * I["box"] * x


# --------------------------------------------------------------------------

def prepare(case, seed):
    I = _inputs(case, seed)
    s = dict(case=case, m=I["m"])
    if case["kind"] in BATCHED:
        P = case["P"]
        b = iod.iod_create_batch([MU] * P, I["chief"], I["t"], I["angles"], [SIGMA] * P, h=1e-3)
        s["b"] = b
        if case["kind"] == "eval32":
            off = iod.iod_batch_offsets(b, I["m"])
            s["x"] = _states(case, I, seed, int(off[-1]), off)
            s["cost"] = torch.zeros(int(off[-1]), dtype=torch.float64, device="cuda")
        else:
            iod.iod_batch_set_config(b, block=64)
            s["params"] = [iod.pso_params(0.7, 1.5, 1.5, seed, I["lo"][p], I["hi"][p], problem=p)
                           for p in range(P)]
        if "offset" in case:
            iod.iod_batch_set_fp32_mode(b, iod.IOD_FP32_RELATIVE if case["offset"]
                                        else iod.IOD_FP32_ABSOLUTE)
            # the chief tables of the offset formulation are built by a batch's first FP32 call
            if case["kind"] == "eval32":
                iod.iod_batch_eval_f32(b, s["x"], s["m"], s["cost"])
        return s
    mode = iod.IOD_COST_CHI2 if case["chi2"] else iod.IOD_COST_PAPER
    common = dict(h=case["h"], cost_mode=mode)
    if case["ranged"]:
        h = iod.iod_create_ranged(MU, I["chief"][0], I["t"][0], I["angles"][0], I["ranges"][0],
                                  SIGMA, SIGMA_RANGE, **common)
    else:
        h = iod.iod_create(MU, I["chief"][0], I["t"][0], I["angles"][0], SIGMA, **common)
    s["h"] = h
    m, K, kind = case["m"], case["K"], case["kind"]
    ld = (m + 63) // 64 * 64
    kw = dict(dtype=torch.float64, device="cuda")
    if kind in ("solve", "swarm"):
        s["params"] = iod.pso_params(0.7, 1.5, 1.5, seed, I["lo"][0], I["hi"][0])
        if kind == "swarm":
            s["swarm"] = iod.Swarm(m, hist_len=case["n_iter"] + 1)
        return s
    x = _states(case, I, seed, ld, None)
    if kind == "grad":
        s["x"] = x[:, :m].t().contiguous().requires_grad_()
        return s
    s["x"] = x
    if kind == "eval":
        s["cost"] = torch.zeros(ld, **kw)
    elif kind == "propagate":
        s["states"] = torch.zeros((K, 6, ld), **kw)
    elif kind == "predict":
        s["angles"] = torch.zeros((K, 2, ld), **kw)
    else:
        s["chi2"], s["jtj"], s["jtr"] = (torch.zeros(n, **kw) for n in (ld, (21, ld), (6, ld)))
    return s


def run(s):
    c = s["case"]
    kind, m = c["kind"], s["m"]
    if kind == "eval":
        iod.iod_eval_swarm(s["h"], s["x"], c["m"], s["cost"])
        return s["cost"][:c["m"]]
    if kind == "propagate":
        iod.iod_propagate(s["h"], s["x"], c["m"], s["states"])
        return s["states"][:, :, :c["m"]]
    if kind == "predict":
        iod.iod_predict(s["h"], s["x"], c["m"], s["angles"])
        return s["angles"][:, :, :c["m"]]
    if kind == "grad":
        cost = iod.iod_cost(s["x"], s["h"])
        g, = torch.autograd.grad(cost.sum(), s["x"])
        return {"cost": cost, "grad": g}
    if kind == "normal":
        iod.iod_normal_eq(s["h"], s["x"], c["m"], s["chi2"], s["jtj"], s["jtr"])
        return {k: s[k][..., :c["m"]] for k in ("chi2", "jtj", "jtr")}
    if kind == "solve":
        return iod.iod_solve(s["h"], s["params"], c["m"], c["n_iter"])
    if kind == "swarm":
        w = s["swarm"]
        iod.iod_swarm_init(s["h"], w, s["params"])
        iod.iod_step(s["h"], w, s["params"], c["n_iter"])
        best = iod.iod_swarm_best(s["h"], w)
        n = c["m"]
        return dict(x=w.x[:, :n], v=w.v[:, :n], p=w.p[:, :n], jp=w.jp[:n], cost=w.cost[:n], best=best)
    if kind == "eval32":
        iod.iod_batch_eval_f32(s["b"], s["x"], m, s["cost"])
        return s["cost"]
    if kind == "batch":
        return iod.iod_batch_solve(s["b"], s["params"], m, c["n_iter"])
    if kind == "mixed":
        return iod.iod_batch_solve_mixed(s["b"], s["params"], m, c["n_iter"], top_k=64)
    return iod.iod_batch_solve_polished(s["b"], s["params"], m, c["n_iter"], top_k=64,
                                        n_cand=c["n_cand"], n_gn=c["n_gn"])


def work(case):
    """Flop-equivalents of the propagations and residuals (the tangent or
    cotangent sweeps where sensitivities are asked for), and the bytes of the
    inputs and outputs. Batches: expected values of the drawn sizes."""
    kind = case["kind"]
    if kind in BATCHED:
        lo, hi = case["m_lo"], case["m_hi"]
        m = case["P"] * ((hi - lo) / np.log(hi / lo) if hi > lo else lo)
        steps, K = 500 * (case["T_lo"] + case["T_hi"]), (case["K_lo"] + case["K_hi"]) / 2
        one = steps * STEP + K * OBS
        if kind == "eval32":
            return {"flops": m * one, "bytes": 56 * m}
        n = case["n_iter"]
        f, b = n * m * (one + UPDATE), 8 * case["P"] * (n + 8)
        if kind == "refine":
            # one pass of the normal equations over the candidates at the least
            f += case["P"] * case["n_cand"] * steps * (STEP + TANGENT)
        return {"flops": f, "bytes": b}
    m, K, S = case["m"], case["K"], case["K"] * case["per"]
    one = S * STEP + K * (OBS + (10 if case["ranged"] else 0))
    if kind == "solve":
        return {"flops": case["n_iter"] * m * (one + UPDATE), "bytes": 8 * (case["n_iter"] + 8)}
    if kind == "swarm":
        return {"flops": case["n_iter"] * m * (one + UPDATE), "bytes": 160 * m}
    if kind == "grad":
        return {"flops": m * (one + S * COTANGENT), "bytes": 104 * m}
    if kind == "normal":
        return {"flops": m * (one + S * TANGENT), "bytes": 272 * m}
    out = {"eval": 8, "propagate": 48 * K, "predict": 16 * K}[kind]
    return {"flops": m * one, "bytes": (48 + out) * m}


# --------------------------------------------------------------------------
# The values themselves: plain torch in float64
# --------------------------------------------------------------------------

def _f(s, jac):
    """Right-hand side of s [6, ...] and, if asked, the gravity block [3][3]."""
    x, y, z, vx, vy, vz = s
    d1, d2, q = x + MU, x - (1 - MU), y * y + z * z
    r1, r2 = torch.rsqrt(d1 * d1 + q), torch.rsqrt(d2 * d2 + q)
    c1, c2 = (1 - MU) * r1 ** 3, MU * r2 ** 3
    cs = c1 + c2
    f = torch.stack([vx, vy, vz, 2 * vy + x - c1 * d1 - c2 * d2, y - 2 * vx - cs * y, -cs * z])
    if not jac:
        return f, None
    e1, e2 = 3 * c1 * r1 * r1, 3 * c2 * r2 * r2
    p1, p2 = torch.stack([d1, y, z]), torch.stack([d2, y, z])
    G = e1 * p1[:, None] * p1[None] + e2 * p2[:, None] * p2[None]
    i = torch.arange(3, device=s.device)
    G[i, i] -= cs
    G[0, 0] += 1
    G[1, 1] += 1
    return f, G


def _ft(G, U):
    """Tangent of the right-hand side: U [6, c, n] through the block G [3, 3, n]."""
    a = (G[:, :, None] * U[None, :3]).sum(1)
    a[0] += 2 * U[4]
    a[1] -= 2 * U[3]
    return torch.cat([U[3:], a])


def _step(s, U, h):
    jac = U is not None
    sk, uk, fs, us = s, U, 0, 0
    for w, c in ((1, h / 2), (2, h / 2), (2, h), (1, None)):
        f, G = _f(sk, jac)
        fs = fs + w * f
        if jac:
            d = _ft(G, uk)
            us = us + w * d
        if c is not None:
            sk = s + c * f
            uk = U + c * d if jac else None
    return s + h / 6 * fs, U + h / 6 * us if jac else None


def _walk(x, t, h, jac, see):
    """RK4 on the grid t = j h with a partial step to each off-grid time;
    see(k, state, tangent) at each observation."""
    s, n = x, 0
    U = torch.eye(6, dtype=x.dtype, device=x.device)[:, :, None].expand(6, 6, x.shape[1]) if jac else None
    for k, tk in enumerate(t):
        near = int(np.floor(tk / h + 0.5))
        on = abs(tk - near * h) <= 1e-9 * h
        for _ in range(n, near if on else int(np.floor(tk / h))):
            s, U = _step(s, U, h)
            n += 1
        a, b = (s, U) if on else _step(s, U, tk - n * h)
        see(k, a, b)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("solve", "swarm", "batch", "mixed", "refine"):
        return None   # each iteration follows the comparisons of the one before
    I = _inputs(case, seed)
    if kind == "eval32":
        off = np.concatenate([[0], np.cumsum((I["m"] + 63) // 64 * 64)])
        return _exact_batch(case, I, _states(case, I, seed, int(off[-1]), off), off)
    m, h, t = case["m"], case["h"], I["t"][0]
    ld = (m + 63) // 64 * 64
    x = _states(case, I, seed, ld, None)[:, :m]
    chief = torch.from_numpy(I["chief"][0]).cuda()[:, None]
    rc = []
    _walk(chief, t, h, False, lambda k, s, U: rc.append(s[:3]))
    got = []
    if kind == "propagate":
        _walk(x, t, h, False, lambda k, s, U: got.append(s))
        return torch.stack(got)
    if kind == "predict":
        def angles(k, s, U):
            rho = s[:3] - rc[k]
            got.append(torch.stack([torch.atan2(rho[1], rho[0]), torch.asin(rho[2] / rho.norm(dim=0))]))
        _walk(x, t, h, False, angles)
        return torch.stack(got)
    jac = kind != "eval"
    R = 3 if case["ranged"] else 2
    z = dict(cost=0, grad=0, chi2=0, jtr=0, N=0)

    def residuals(k, s, U):
        r, dr = _residual(s[:3] - rc[k], I["angles"][0][k], I["ranges"][0][k] if R == 3 else None)
        e = (r * r).sum(0)
        z["cost"] = z["cost"] + (e if case["chi2"] else e * e)
        if jac:
            J = (dr[:, :, None] * U[None, :3]).sum(1)
            g = (J * r[:, None]).sum(0)
            z["grad"] = z["grad"] + (2 if case["chi2"] else 4 * e) * g
            z["chi2"], z["jtr"] = z["chi2"] + e, z["jtr"] + g
            z["N"] = z["N"] + (J[:, :, None] * J[:, None]).sum(0)
    _walk(x, t, h, jac, residuals)
    if kind == "eval":
        return z["cost"]
    if kind == "grad":
        return {"cost": z["cost"], "grad": z["grad"].t().contiguous()}
    i, j = np.triu_indices(6)
    return {"chi2": z["chi2"], "jtj": z["N"][i, j], "jtr": z["jtr"]}


def _residual(rho, ang, rng):
    """Whitened residuals [R, n] at rho [3, n] and their gradient [R, 3, n]."""
    sa, ca, sb, cb = np.sin(ang[0]), np.cos(ang[0]), np.sin(ang[1]), np.cos(ang[1])
    x, y, z = rho
    q2 = x * x + y * y
    q, r2 = q2.sqrt(), q2 + z * z
    r = [torch.atan2(sa * x - ca * y, ca * x + sa * y) / SIGMA,
         torch.atan2(sb * q - cb * z, cb * q + sb * z) / SIGMA]
    d = [torch.stack([y / q2, -x / q2, torch.zeros_like(x)]) / SIGMA,
         torch.stack([z * x / q / r2, z * y / q / r2, -q / r2]) / SIGMA]
    if rng is not None:
        n = r2.sqrt()
        r.append((rng - n) / SIGMA_RANGE)
        d.append(-rho / n / SIGMA_RANGE)
    return torch.stack(r), torch.stack(d)


def _exact_batch(case, I, x, off):
    """FP64 costs of every problem's columns, all problems stepped together;
    columns past a problem's particles keep the zeros they had."""
    P, dev = case["P"], x.device
    col = torch.zeros(x.shape[1], dtype=torch.int64, device=dev)
    live = torch.zeros(x.shape[1], dtype=torch.bool, device=dev)
    for p in range(P):
        col[off[p]:off[p + 1]] = p
        live[off[p]:off[p] + int(I["m"][p])] = True
    at = {}
    for p in range(P):
        for k, tk in enumerate(I["t"][p]):
            at.setdefault(int(round(tk / 1e-3)), []).append((p, k))
    chief = torch.from_numpy(I["chief"]).to(dev).t().contiguous()
    J = torch.zeros(x.shape[1], dtype=torch.float64, device=dev)
    s = x
    for n in range(1, max(at) + 1):
        s, _ = _step(s, None, 1e-3)
        chief, _ = _step(chief, None, 1e-3)
        for p, k in at.get(n, ()):
            c = slice(int(off[p]), int(off[p] + I["m"][p]))
            r, _ = _residual(s[:3, c] - chief[:3, p:p + 1], I["angles"][p][k], None)
            J[c] += (r * r).sum(0) ** 2
    return torch.where(live, J, torch.zeros_like(J))
