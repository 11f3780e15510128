"""What a user of the framework has it do, as measurable cases: the minimum-norm estimate, the
set-up from it, the filter and fixed-interval smoother in both precisions, checkpointed, with
several data sets, with a transition matrix, the mean-only smoother, and the serving loop.

Sizes follow the framework's own workloads (``synth.py``, ``bench.py``, the tests): N = 500 sources
with 60 sensors, N = 5124 with 306, the free-orientation N = 15372, serving jobs of N near 2000.
Inputs are made on the GPU from the seed with the distributions of those workloads: a dipole lead
field of unit Frobenius norm, sources in a ball (small sizes) or on a shell, a Gaussian-kernel (or
scaled identity) process covariance, sinusoidal source patches seen at 5 dB. Horizons are shorter
than the workloads' (a pass is a chain of equal time steps), so that a pass stays well under 2 s.
"""
import math

import torch

from paper_1107_4192_amd import kfmeg

DEV = "cuda"
F64 = torch.float64


def listed():
    return [
        # The smallest call: one minimum-norm estimate in a tight loop that cannot allocate.
        {"name": "mne_noalloc_500", "kind": "mne", "N": 500, "m": 60, "T": 50, "noalloc": True},
        # The paper's static estimate of a whole recording at the paper's size.
        {"name": "mne_5124", "kind": "mne", "N": 5124, "m": 306, "T": 200, "noalloc": False},
        # Parameter set-up before a filter run: x0 and Q from the static estimates.
        {"name": "init_5124", "kind": "init", "N": 5124, "m": 306, "T": 200},
        # The small workload: filter and smoother, bound by launches and latency.
        {"name": "run_500", "kind": "run", "N": 500, "m": 60, "T": 50, "ball": True},
        # A mid-size job whose covariances do not all fit: every 7th kept, the rest recomputed.
        {"name": "run_2000_ckpt", "kind": "run", "N": 2000, "m": 204, "T": 48, "stride": 7},
        # The headline workload's time steps: filter and smoother in float64 at the paper's size.
        {"name": "run_5124", "kind": "run", "N": 5124, "m": 306, "T": 16},
        # The same in mixed precision with a float32 store.
        {"name": "run_5124_mixed", "kind": "run", "N": 5124, "m": 306, "T": 12, "mixed": True, "store32": True},
        # Filter and smoothed means only, over a longer recording.
        {"name": "means_5124", "kind": "means", "N": 5124, "m": 306, "T": 64},
        # Eight data sets (trials) of one subject through one covariance pass, a ragged size.
        {"name": "batch8_1999", "kind": "run", "N": 1999, "m": 203, "T": 24, "B": 8},
        # The six-neighbour transition of the source model (denser sites make P_{t+1|t} so ill-conditioned
        # that the smoothed variances are not determined to the digits that float64 outputs are held to).
        {"name": "neighbour_1500", "kind": "run", "N": 1500, "m": 204, "T": 24, "neigh": True},
        # Free orientation, three columns a site: the largest state.
        {"name": "free_15372_mixed", "kind": "run", "N": 15372, "m": 306, "T": 3, "mixed": True, "store32": True,
         "free": True},
        # Six jobs of different sizes through the serving loop, four at a time.
        {"name": "serve_2000_mixed", "kind": "serve", "N": 2000, "m": 204, "T": 30, "jobs": 6, "mixed": True,
         "store32": True},
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["mne", "mne", "init", "run", "run", "run", "run", "run", "means", "serve"])
    m = rng.randint(30, 306)
    if kind in ("mne", "init"):
        case = {"kind": kind, "N": _logint(rng, 300, 6000), "m": m, "T": _logint(rng, 5, 400)}
        if kind == "mne":
            case["noalloc"] = rng.random() < 0.5
        return case
    if kind == "serve":
        return {"kind": kind, "N": _logint(rng, 500, 2000), "m": m, "T": rng.randint(10, 40),
                "jobs": rng.randint(2, 6), "mixed": rng.random() < 0.5, "store32": rng.random() < 0.5}
    N = _logint(rng, 300, 5124)
    m = min(m, N // 3)
    # about the same work whatever N, and never more than the largest listed case
    T = max(3, min(120, int(rng.uniform(0.3, 1.0) * 12 * (5124 / N) ** 2)))
    if kind == "means":
        return {"kind": kind, "N": N, "m": m, "T": T}
    case = {"kind": kind, "N": N, "m": m, "T": T}
    option = rng.choice(["plain", "plain", "mixed", "stride", "batch", "neigh", "ball"])
    if option == "mixed":
        case["mixed"] = True
        case["store32"] = rng.random() < 0.7
    elif option == "stride":
        case["stride"] = rng.randint(2, 9)
    elif option == "batch":
        case["B"] = rng.randint(2, 9)
    elif option == "neigh":
        N = _logint(rng, 300, 1600)
        case.update(N=N, m=min(m, N // 4), T=rng.randint(8, 40), neigh=True)
    elif option == "ball":
        case["ball"] = True
    return case


# ---------------------------------------------------------------- inputs
def _unit(g, n):
    v = torch.randn((n, 3), generator=g, dtype=F64, device=DEV)
    return v / v.norm(dim=1, keepdim=True)


def _model(N, m, T, seed, B=1, ball=False, free=False, neigh=False):
    """X, Q, R, x0, P0, Y (B x T x m) and the sites' transition (CSR) or None, on the GPU."""
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1009 + 17)
    n = N // 3 if free else N
    u = torch.rand((n, 1), generator=g, dtype=F64, device=DEV)
    sites = _unit(g, n) * (0.07 * u ** (1.0 / 3.0) if ball else 0.06 + 0.01 * u)
    sensors = _unit(g, m)
    sensors[:, 2].abs_()
    sensors *= 0.11
    if free:
        pos = sites.repeat_interleave(3, dim=0)
        normals = torch.eye(3, dtype=F64, device=DEV).repeat(n, 1)
    else:
        pos, normals = sites, _unit(g, n)
    diff = sensors[:, None, :] - pos[None, :, :]
    X = (diff * normals[None]).sum(2) / diff.norm(dim=2) ** 3
    X = (X / X.norm()).contiguous()
    d2 = torch.empty((n, n), dtype=F64, device=DEV)
    for a in range(0, n, 1024):
        d = sites[a:a + 1024, None, :] - sites[None, :, :]
        d2[a:a + 1024] = (d * d).sum(2)
    t = torch.arange(1, T + 1, dtype=F64, device=DEV)
    truth = torch.zeros((T, N), dtype=F64, device=DEV)
    if ball:
        Q = 1e-2 * torch.eye(N, dtype=F64, device=DEV)
        active = torch.randperm(N, generator=g, device=DEV)[:5]
        truth[:, active] = 0.1 * torch.randn((T, active.numel()), generator=g, dtype=F64, device=DEV).cumsum(0)
        sigma2 = 1e-4
    else:
        K = 1e-2 * torch.exp(-d2 / (2.0 * 0.01 ** 2))
        if free:
            Q = torch.zeros((N, N), dtype=F64, device=DEV)
            for a in range(3):
                Q[a::3, a::3] = K
        else:
            Q = K
        centres = torch.randperm(n, generator=g, device=DEV)[:3]
        wave = torch.rand((3, 2), generator=g, dtype=F64, device=DEV)
        for k in range(centres.numel()):
            near = d2[centres[k]].topk(min(42, n), largest=False).indices
            course = torch.sin(2.0 * math.pi * (10.0 + 30.0 * wave[k, 0]) * t / 600.0 + 2.0 * math.pi * wave[k, 1])
            for a in range(3 if free else 1):
                truth[:, (3 * near + a) if free else near] = course[:, None]
        sigma2 = float((truth @ X.T).square().mean()) / 10.0 ** 0.5
    R = sigma2 * torch.eye(m, dtype=F64, device=DEV)
    Y = (truth @ X.T)[None] + math.sqrt(sigma2) * torch.randn((B, T, m), generator=g, dtype=F64, device=DEV)
    F = None
    if neigh:
        d2.fill_diagonal_(math.inf)
        near = d2.topk(6, largest=False).indices
        own = torch.arange(n, device=DEV)[:, None]
        cols = torch.cat([own, near], dim=1)
        vals = torch.full((n, 7), 0.5 / 6, dtype=F64, device=DEV)
        vals[:, 0] = 0.5
        cols, order = cols.sort(dim=1)
        vals = vals.gather(1, order)
        F = (torch.arange(0, 7 * n + 1, 7, dtype=torch.int32, device=DEV), cols.reshape(-1).to(torch.int32),
             vals.reshape(-1).contiguous())
    x0 = torch.zeros(N, dtype=F64, device=DEV)
    P0 = torch.eye(N, dtype=F64, device=DEV)
    return {"X": X, "Q": Q, "R": R, "x0": x0, "P0": P0, "Y": Y.contiguous(), "F": F}


def _case_model(case, seed):
    return _model(case["N"], case["m"], case["T"], seed, case.get("B", 1), case.get("ball", False),
                  case.get("free", False), case.get("neigh", False))


def _jobs(case):
    """Sizes of the serving loop's jobs: like its seeded stream, of different N and T."""
    return [(max(90, case["N"] // (1 + j % 3)), max(30, case["m"] // (1 + j % 3)), case["T"] + 3 * j)
            for j in range(case["jobs"])]


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("mne", "init"):
        p = _case_model(case, seed)
        st = {"case": case, "X": p["X"], "R": p["R"], "Y": p["Y"][0].contiguous()}
        if kind == "mne":      # a source prior with spatial correlation
            st["C"] = p["Q"] + p["P0"]
            st["J"] = torch.empty((case["T"], case["N"]), dtype=F64, device=DEV)
        else:
            st["C"] = p["P0"]
        return st
    precision = kfmeg.KF_MIXED if case.get("mixed") else kfmeg.KF_FP64
    if kind == "serve":
        jobs = [_model(N, m, T, seed * 16 + j) for j, (N, m, T) in enumerate(_jobs(case))]
        srv = kfmeg.Server(hbm_budget_bytes=16 << 30, max_active=4, precision=precision,
                           store_fp32=case.get("store32", False))
        return {"case": case, "jobs": jobs, "srv": srv}
    p = _case_model(case, seed)
    ks = kfmeg.KalmanSmoother(p["X"], p["Q"], p["R"], p["x0"], p["P0"], T_max=case["T"], precision=precision,
                              store_fp32=case.get("store32", False), checkpoint_stride=case.get("stride", 0),
                              keep_gain_factors=kind == "means", F=p["F"])
    Y = p["Y"] if case.get("B", 1) > 1 else p["Y"][0].contiguous()
    return {"case": case, "ks": ks, "Y": Y}


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "mne":
        if case["noalloc"]:
            return {"J": kfmeg.mne_solve_noalloc(state["X"], state["C"], state["R"], state["Y"], state["J"])}
        return {"J": kfmeg.mne_solve(state["X"], state["C"], state["R"], state["Y"])}
    if kind == "init":
        x0, Q = kfmeg.kf_init_from_mne(state["X"], state["C"], state["R"], state["Y"], 1e-3)
        return {"x0": x0, "Q": Q}
    if kind == "serve":
        srv = state["srv"]
        ids = [srv.submit(p["X"], p["Q"], p["R"], p["x0"], p["P0"], p["Y"][0]) for p in state["jobs"]]
        got = [srv.wait(i) for i in ids]
        return {"x_smooth": [r[0] for r in got], "Pdiag_smooth": [r[1] for r in got]}
    ks, Y = state["ks"], state["Y"]
    if kind == "means":
        res = ks.smooth_means(ks.filter(Y))
        return {"x_filt": res.x_filt, "Pdiag_filt": res.Pdiag_filt, "x_smooth": res.x_smooth}
    res = ks.run_batch(Y) if case.get("B", 1) > 1 else ks.run(Y)
    return {"x_filt": res.x_filt, "Pdiag_filt": res.Pdiag_filt, "x_smooth": res.x_smooth,
            "Pdiag_smooth": res.Pdiag_smooth}


# ---------------------------------------------------------------- what the path cannot do without
def _run_work(N, m, T, B=1, means=False):
    """Filter: the factor of S, C = L^-1 X P, its next X P by rank-m updates, a symmetric rank-m downdate.
    Smoother: a factorisation of every P_{t+1|t} (its failure is an error), the diagonal of one symmetric
    N x N congruence (a triangular product) and symmetric rank-2m updates; means only: matrix-vector."""
    filt = m ** 3 / 3.0 + 5.0 * N * m * m + 1.0 * N * N * m + 6.0 * B * m * N
    smooth = 2.0 * B * N * N + 4.0 * B * m * N
    if not means:
        smooth += N ** 3 / 3.0 + 1.0 * N ** 3 + 4.0 * N * N * m
    nbytes = 8.0 * (m * N + 2 * N * N + m * m + N + B * T * m + 2 * B * T * N + (1 if means else 2) * T * N)
    return nbytes, T * filt + (T - 1) * smooth


def work(case):
    kind, N, m, T = case["kind"], case["N"], case["m"], case["T"]
    if kind in ("mne", "init"):
        nbytes = 8.0 * (N * N + m * N + m * m + T * m + (T * N if kind == "mne" else N * N + N))
        flops = 2.0 * N * N * m + 1.0 * N * m * m + m ** 3 / 3.0 + 2.0 * m * m * T + 2.0 * N * m * T
        if kind == "init":
            flops += 1.0 * N * N * (T - 1)
        return {"bytes": nbytes, "flops": flops}
    if kind == "serve":
        both = [_run_work(*j) for j in _jobs(case)]
        return {"bytes": sum(b for b, _ in both), "flops": sum(f for _, f in both)}
    b, f = _run_work(N, m, T, case.get("B", 1), kind == "means")
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------- the same in plain torch, 64 bits
def _exact_mne(X, C, R, Y):
    G = C @ X.T
    L = torch.linalg.cholesky(X @ G + R)
    return (G @ torch.cholesky_solve(Y.T.contiguous(), L)).T.contiguous()


def _exact_run(p, T, means=False):
    X, Q, R = p["X"], p["Q"], p["R"]
    N, m = X.shape[1], X.shape[0]
    B = p["Y"].shape[0]
    F = None
    if p["F"] is not None:
        rows = torch.arange(N, device=DEV).repeat_interleave(7)
        F = torch.zeros((N, N), dtype=F64, device=DEV)
        F[rows, p["F"][1].long()] = p["F"][2]
    mul = (lambda v: v) if F is None else (lambda v: F @ v)
    x = p["x0"][:, None].expand(N, B).contiguous()
    P = p["P0"].clone()
    xs, Ps = [], []
    for t in range(T):
        x = mul(x)
        P = P + Q if F is None else F @ P @ F.T + Q
        Bm = X @ P
        S = Bm @ X.T + R
        L = torch.linalg.cholesky((S + S.T) / 2)
        C = torch.linalg.solve_triangular(L, Bm, upper=False)
        e = p["Y"][:, t].T - X @ x
        x = x + C.T @ torch.linalg.solve_triangular(L, e.contiguous(), upper=False)
        P = P - C.T @ C
        P = (P + P.T) / 2
        xs.append(x)
        Ps.append(P)
    sx, sd = [None] * T, [None] * T
    sx[T - 1], sP = xs[T - 1], Ps[T - 1]
    sd[T - 1] = sP.diagonal().clone()
    for t in range(T - 2, -1, -1):
        FP = mul(Ps[t])
        Pn = Ps[t] + Q if F is None else FP @ F.T + Q
        L = torch.linalg.cholesky((Pn + Pn.T) / 2)
        A = torch.cholesky_solve(FP, L).T
        sx[t] = xs[t] + A @ (sx[t + 1] - mul(xs[t]))
        if not means:
            sP = Ps[t] + A @ (sP - Pn) @ A.T
            sP = (sP + sP.T) / 2
            sd[t] = sP.diagonal().clone()
    one = (lambda v: torch.stack(v).permute(2, 0, 1)) if B > 1 else (lambda v: torch.stack(v)[:, :, 0])
    out = {"x_filt": one(xs).contiguous(), "Pdiag_filt": torch.stack([P.diagonal() for P in Ps]),
           "x_smooth": one(sx).contiguous()}
    if not means:
        out["Pdiag_smooth"] = torch.stack(sd)
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind == "run" and case["N"] > 8000:
        return None                # factorisations of this order take too long in plain torch
    if kind == "serve":
        got = [_exact_run(_model(N, m, T, seed * 16 + j), T) for j, (N, m, T) in enumerate(_jobs(case))]
        return {"x_smooth": [r["x_smooth"] for r in got], "Pdiag_smooth": [r["Pdiag_smooth"] for r in got]}
    p = _case_model(case, seed)
    if kind == "mne":
        return {"J": _exact_mne(p["X"], p["Q"] + p["P0"], p["R"], p["Y"][0])}
    if kind == "init":
        J = _exact_mne(p["X"], p["P0"], p["R"], p["Y"][0])
        D = J[1:] - J[:-1]
        D = D - D.mean(0, keepdim=True)
        Q = D.T @ D / (D.shape[0] - 1)
        Q += 1e-3 * torch.eye(case["N"], dtype=F64, device=DEV)
        return {"x0": J[0].clone(), "Q": (Q + Q.T) / 2}
    return _exact_run(p, case["T"], kind == "means")
