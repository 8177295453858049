"""Planning workloads whose speed is measured, each through the package's public entry points.

A case is one call that a robot's program makes: a plan (Alg. 1) of one scene, a batch of plans,
a projection of given samples, a plan with several Gaussians, or a set of requests through the
continuous-batching server.  Sizes are those of ``paper_2309_08235_amd.workloads`` and of the
tests, with odd ones among them; scenes follow the same recipes (random discs or spheres between
a start and a goal at rest, some of them moving).

``exact`` evaluates the projection in 64 bits with plain torch.  A plan of several CEM iterations
has no such value: its selections turn on differences that rounding decides.
"""
from __future__ import annotations

import math
from dataclasses import replace

import numpy as np
import torch

from paper_2309_08235_amd import priest as P
from paper_2309_08235_amd.serve import Server

DEV = "cuda"

# What a case holds where it does not say otherwise.
DEFAULTS = dict(dims=2, n_coeff=11, n_steps=100, horizon=15.0, n_obs=50, n_samples=1000,
                n_problems=1, n_proj_iters=100, n_cem=20, n_elite=0, rest=False, moving=True,
                mixed=False, bounds=False, weighted=False, cma=False, paths=False)


def _case(name, kind, **kw):
    c = dict(DEFAULTS, kind=kind, **kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: a 64-sample plan of one CEM iteration, where latency and launches count
        _case("plan_2d_small", "plan", n_steps=50, horizon=10.0, n_obs=4, n_samples=64,
              n_proj_iters=50, n_cem=1, rest=True, moving=False),
        # one robot planning one scene at the paper's scale (2D, 20 of 50 obstacles moving)
        _case("plan_2d", "plan", n_elite=100),
        # the same with the options of navigation in earnest, at odd sizes and a long horizon:
        # workspace bounds, curvature / path / steering cost, CMA-ES-style covariance
        _case("plan_2d_options", "plan", n_coeff=9, n_steps=149, horizon=18.0, n_obs=37,
              n_samples=733, n_proj_iters=50, n_cem=13, bounds=True, weighted=True, cma=True),
        # one aerial robot among 128 spheres
        _case("plan_3d", "plan", dims=3, n_obs=128, n_samples=2000, n_elite=200, moving=False),
        # a fleet of 64 ground robots, every CEM step batched, the loop replayed as a graph
        _case("plan_batch_2d", "plan_batch", n_problems=64, n_elite=100),
        # the largest: 64 aerial scenes of 2000 samples each in one graph-replayed batch
        _case("plan_batch_3d", "plan_batch", dims=3, n_obs=128, n_samples=2000, n_problems=64,
              n_elite=200, moving=False),
        # the projection optimizer as an operator on given samples (any other sampler around it)
        _case("project_2d", "project"),
        # the same in mixed precision (BF16 right-hand side, last 10 iterations in FP32)
        _case("project_2d_mixed", "project", mixed=True),
        # one large projection: 64000 samples of one scene
        _case("project_2d_large", "project", n_samples=64000),
        # predicted obstacle paths (positions at every time stamp) in 3D, an odd sample count
        _case("project_3d_paths", "project", dims=3, n_samples=613, paths=True),
        # D-PRIEST: four Gaussians of 250 samples on one scene
        _case("dpriest_2d", "dpriest", n_problems=4, n_samples=250, n_elite=25),
        # 64 requests of mixed sizes through the continuous-batching server, host buffers in and
        # out (256..2048 samples, 8..128 obstacles, 50 or 100 steps, 20 x 5 iterations each)
        _case("serve_2d", "serve", n_problems=64, n_samples=2048, n_obs=128, n_proj_iters=20, n_cem=5),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    top = max(_flops(c) for c in listed())
    kind = rng.choice(["plan", "plan", "plan_batch", "project", "project_batch", "dpriest", "serve"])
    while True:
        if kind == "serve":
            return _case(None, kind, n_problems=_log_int(rng, 4, 96), n_samples=2048, n_obs=128,
                         n_proj_iters=rng.randint(10, 30), n_cem=rng.randint(2, 6))
        c = _case(None, kind, dims=rng.choice([2, 2, 3]), n_coeff=rng.randint(7, 13),
                  n_steps=_log_int(rng, 20, 200), horizon=round(rng.uniform(10.0, 20.0), 2),
                  n_obs=_log_int(rng, 4, 140), n_samples=_log_int(rng, 64, 2400),
                  n_proj_iters=_log_int(rng, 15, 110), n_cem=_log_int(rng, 1, 20),
                  rest=rng.random() < 0.3, moving=rng.random() < 0.6,
                  bounds=rng.random() < 0.25, mixed=rng.random() < 0.15)
        if kind == "project":
            c.update(n_samples=_log_int(rng, 64, 64000))
        if kind in ("plan_batch", "project_batch"):
            c.update(n_problems=_log_int(rng, 2, 64))
        if kind == "dpriest":
            c.update(n_problems=rng.randint(2, 8), n_samples=_log_int(rng, 64, 600))
        if kind in ("plan", "plan_batch", "dpriest"):
            c.update(weighted=rng.random() < 0.25, cma=rng.random() < 0.25)
        elif not c["moving"]:
            c.update(paths=rng.random() < 0.4)
        if _flops(c) <= top and _path_bytes(c) < 1 << 28:
            return c


def _flops(c):
    """The dense part of the alternating minimisation (forward rows, norm bounds, right-hand side,
    multiplier and QP step) over every sample and iteration; obstacle pairs are not counted, since
    most of them can be shown not to touch."""
    d, nv, K = c["dims"], c["n_coeff"], c["n_steps"]
    N, P_ = c["n_samples"], c["n_problems"]
    if c["kind"] == "serve":
        N, K = 960, 75  # means of the requests' sizes
    per = 12 * d * nv * K + 2 * K * (2 * d + 2) + d * (5 * nv + 2 * nv * nv)
    loops = 1 if c["kind"].startswith("project") else c["n_cem"]
    return float(per) * N * P_ * c["n_proj_iters"] * loops


def _path_bytes(c):
    return 4 * c["n_problems"] * c["n_obs"] * (c["n_steps"] * c["dims"] + 2) if c["paths"] else 0


def work(case):
    c = case
    D, N, P_ = c["dims"] * c["n_coeff"], c["n_samples"], c["n_problems"]
    scenes = P_ * (c["dims"] * 24 + c["n_obs"] * 32) + _path_bytes(c)
    if c["kind"].startswith("project"):
        nbytes = scenes + P_ * N * (2 * D + 2) * 4
    elif c["kind"] == "serve":
        nbytes = scenes + P_ * (D + 1) * 4
    else:
        nbytes = scenes + P_ * (4 * (D + D * D) * 2 + N * (2 * D + 2) * 4)
    return {"bytes": float(nbytes), "flops": _flops(c)}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _scene(rng, dims, n_obs, rest_box, radii, start, goal, moving):
    """bc [dims, 6] and obs [n_obs, 8]; obstacles keep 1 m clear of start and goal."""
    bc = np.zeros((dims, 6))
    bc[:, 0], bc[:, 3] = start, goal
    obs = np.zeros((n_obs, 8))
    got = 0
    while got < n_obs:
        c = rng.uniform(rest_box[0], rest_box[1], size=(2 * n_obs, dims))
        r = rng.uniform(radii[0], radii[1], size=2 * n_obs)
        ok = np.minimum(np.linalg.norm(c - start, axis=1), np.linalg.norm(c - goal, axis=1)) >= r + 1.0
        k = min(n_obs - got, int(ok.sum()))
        obs[got:got + k, :dims] = c[ok][:k]
        obs[got:got + k, 6] = obs[got:got + k, 7] = r[ok][:k]
        got += k
    if moving:  # the last 40% of them, in the plane
        m = int(round(0.4 * n_obs))
        head, speed = rng.uniform(0, 2 * np.pi, m), rng.uniform(0.0, 1.0, m)
        obs[n_obs - m:, 3], obs[n_obs - m:, 4] = speed * np.cos(head), speed * np.sin(head)
    return bc, obs


def _inputs(case, seed):
    """Everything made from the seed, as float64 arrays."""
    c = case
    rng = np.random.Generator(np.random.PCG64(seed))
    d, nv, K = c["dims"], c["n_coeff"], c["n_steps"]
    start, goal = (np.zeros(2), np.full(2, 10.0)) if d == 2 else (np.full(3, 4.0), np.full(3, 16.0))
    box, radii = ((0.5, 9.5), (0.2, 0.5)) if d == 2 else ((0.0, 20.0), (0.2, 0.8))
    if c["n_obs"] <= 8:
        box, radii = ((2.0, 8.0), (0.3, 0.6)) if d == 2 else ((5.0, 15.0), (0.4, 0.8))
    n_scenes = 1 if c["kind"] == "dpriest" else c["n_problems"]
    scenes = [_scene(rng, d, c["n_obs"], box, radii, start, goal, c["moving"]) for _ in range(n_scenes)]
    bc = np.stack([s[0] for s in scenes])
    obs = np.stack([s[1] for s in scenes])
    if c["paths"]:  # circling obstacles, given by their positions at every time stamp
        t = np.arange(K) * (c["horizon"] / (K - 1))
        ph = rng.uniform(0, 2 * np.pi, obs.shape[:2])
        om = rng.uniform(-1.0, 1.0, obs.shape[:2])
        pos = np.repeat(obs[:, :, None, :d], K, axis=2)
        ang = ph[:, :, None] + om[:, :, None] * t
        pos[..., 0] += 0.5 * (np.cos(ang) - np.cos(ph)[:, :, None])
        pos[..., 1] += 0.5 * (np.sin(ang) - np.sin(ph)[:, :, None])
        obs = np.concatenate([pos.reshape(n_scenes, c["n_obs"], K * d), obs[:, :, 6:8]], axis=2)
    mean = np.concatenate([np.linspace(start[x], goal[x], nv) for x in range(d)])
    return dict(bc=bc, obs=obs, mean=mean, rng=rng, start=start, goal=goal)


def _samples(case, seed, mean):
    """Projection inputs: the straight line plus unit normals, float32 [P, N, D], made on the GPU."""
    g = torch.Generator(device=DEV).manual_seed(int(seed))
    z = torch.randn((case["n_problems"], case["n_samples"], mean.size), generator=g, device=DEV)
    return z + torch.as_tensor(mean, dtype=torch.float32, device=DEV)


def _limits(case):
    return (1.5, 2.0) if case["dims"] == 2 else (2.0, 3.0)


def _bounds(case):
    if not case["bounds"]:
        return None, None
    return ((-0.3,) * 2, (10.3,) * 2) if case["dims"] == 2 else ((3.5,) * 3, (16.5,) * 3)


def _cem(case):
    N = case["n_samples"]
    n_proj = max(1, int(math.floor(N * 80 / 110 + 0.5)))
    n_elite = case["n_elite"] or max(1, int(math.floor(N * 20 / 110 + 0.5)))
    cost = P.Cost(P.COST_WEIGHTED, 1.0, 0.5, 0.2, 0.3 if case["dims"] == 2 else 0.0) if case["weighted"] else None
    return P.Cem(N, case["n_cem"], case["n_proj_iters"], n_proj, min(n_elite, n_proj), cost=cost,
                 update=P.UPDATE_CMA if case["cma"] else P.UPDATE_MPPI)


_STREAM = None


def _stream():
    """The program's planning stream (graph replay needs one that is not the default)."""
    global _STREAM
    if _STREAM is None:
        _STREAM = torch.cuda.Stream()
    return _STREAM


def _t(x):
    return torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float32).to(DEV)


def prepare(case, seed):
    if case["kind"] == "serve":
        return _prepare_server(case, seed)
    inp = _inputs(case, seed)
    v_max, a_max = _limits(case)
    s_min, s_max = _bounds(case)
    prob = P.Problem(case["dims"], case["n_coeff"], case["n_steps"], case["horizon"], case["n_obs"],
                     v_max=v_max, a_max=a_max, bc_mask=P.BC_REST if case["rest"] else P.BC_DEFAULT,
                     precision=P.BF16_MIXED if case["mixed"] else P.FP32, s_min=s_min, s_max=s_max,
                     obs_model=P.OBS_PATH if case["paths"] else P.OBS_VELOCITY)
    st = dict(case=case, prob=prob, bc=_t(inp["bc"]), obs=_t(inp["obs"]))
    if case["kind"].startswith("project"):
        st["xi"] = _samples(case, seed, inp["mean"])
    else:
        G, D = case["n_problems"], prob.D
        cem = _cem(case)
        mean = np.tile(inp["mean"], (G, 1))
        if case["kind"] == "dpriest":  # means fanned out sideways, as distinct Gaussians start
            taper = np.sin(np.pi * np.arange(case["n_coeff"]) / (case["n_coeff"] - 1))
            off = 1.5 * (np.arange(G) - (G - 1) / 2.0) / math.sqrt(2.0)
            mean[:, :case["n_coeff"]] -= off[:, None] * taper
            mean[:, case["n_coeff"]:2 * case["n_coeff"]] += off[:, None] * taper
        st.update(cem=cem, mu0=_t(mean), cov0=torch.eye(D, device=DEV).repeat(G, 1, 1), seed=int(seed),
                  mu=torch.empty((G, D), device=DEV), cov=torch.empty((G, D, D), device=DEV),
                  out=prob.plan_outputs(cem, G, full=True), ws=prob.workspace(cem, G))
    _settle(st)
    torch.cuda.synchronize()
    return st


def _settle(st):
    """The handle's first call of this shape, in which it picks its tile shape: a program makes it
    once, then plans scene after scene with the same handle."""
    case, prob = st["case"], st["prob"]
    if case["kind"] == "project":
        prob.project(st["bc"][0], st["obs"][0], st["xi"][0], 8)
    elif case["kind"] == "project_batch":
        prob.project_batch(st["bc"], st["obs"], st["xi"], 8)
    else:
        once = replace(st["cem"], n_cem=1)
        mu, cov = st["mu0"].clone(), st["cov0"].clone()
        if case["kind"] == "plan":
            prob.plan(st["bc"], st["obs"], once, mu, cov, out=st["out"], workspace=st["ws"])
        elif case["kind"] == "plan_batch":
            prob.plan_batch(case["n_problems"], st["bc"], st["obs"], once, mu, cov, out=st["out"],
                            workspace=st["ws"])
        else:
            prob.plan_dpriest(case["n_problems"], st["bc"], st["obs"], once, mu, cov, out=st["out"],
                              workspace=st["ws"])


def _prepare_server(case, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    srv = Server(max_robots=256, v_max=1.5, a_max=2.0, seed=int(seed), memory_budget=1 << 28)
    reqs = []
    for i in range(case["n_problems"]):
        K, T, span = ((50, 10.0, 7.0), (100, 15.0, 10.0))[i % 2]
        start = rng.uniform(0.0, 2.0, 2)
        n = int(rng.choice([256, 512, 1024, 2048]))
        bc, obs = _scene(rng, 2, int(rng.integers(8, 129)), (start - 0.5, start + span + 0.5),
                         (0.2, 0.5), start, start + span, True)
        reqs.append(dict(robot=i, bc=bc.astype(np.float32), obs=obs.astype(np.float32), n_samples=n,
                         n_steps=K, horizon=T, n_cem=case["n_cem"], n_proj_iters=case["n_proj_iters"],
                         n_proj=int(math.floor(n * 80 / 110 + 0.5)),
                         n_elite=int(math.floor(n * 20 / 110 + 0.5)),
                         warm_start=P.WARM_RESET, stream_id=i))
    for key in sorted({(q["n_steps"], q["obs"].shape[0], q["horizon"]) for q in reqs}):
        srv.prepare(*key)
    torch.cuda.synchronize()
    return dict(case=case, server=srv, reqs=reqs)


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(state):
    kind = state["case"]["kind"]
    if kind == "serve":
        srv = state["server"]
        ids = [srv.submit(**q) for q in state["reqs"]]
        done = {c.request_id: c for c in srv.drain()}
        return {"best_xi": np.stack([done[i].best_xi for i in ids]),
                "best_cost": np.array([done[i].best_cost for i in ids], np.float32),
                "status": np.array([done[i].status for i in ids], np.int32)}
    prob, bc, obs = state["prob"], state["bc"], state["obs"]
    iters = state["case"]["n_proj_iters"]
    if kind == "project":
        xo, r, c1 = prob.project(bc[0], obs[0], state["xi"][0], iters)
        return {"xi_bar": xo, "resid": r, "c1": c1}
    if kind == "project_batch":
        xo, r, c1 = prob.project_batch(bc, obs, state["xi"], iters)
        return {"xi_bar": xo, "resid": r, "c1": c1}
    with torch.cuda.stream(_stream()):
        # every plan starts from its own initial distribution
        mu, cov, out = state["mu"].copy_(state["mu0"]), state["cov"].copy_(state["cov0"]), state["out"]
        more = {}
        if kind == "plan":
            prob.plan(bc, obs, state["cem"], mu, cov, seed=state["seed"], out=out, workspace=state["ws"])
        elif kind == "plan_batch":
            prob.plan_batch(state["case"]["n_problems"], bc, obs, state["cem"], mu, cov,
                            seed=state["seed"], out=out, workspace=state["ws"], use_graph=True)
        else:
            xi, cost, group, _ = prob.plan_dpriest(state["case"]["n_problems"], bc, obs, state["cem"], mu,
                                                   cov, seed=state["seed"], out=out, workspace=state["ws"])
            more = {"pick_xi": xi, "pick_cost": cost, "pick_group": group}
    return dict(out, mu=mu, cov=cov, **more)


# ---------------------------------------------------------------------------
# 64-bit values
# ---------------------------------------------------------------------------
def _basis(nv, K, T):
    n = nv - 1
    tau = np.arange(K) / (K - 1)

    def bern(m):
        return np.stack([math.comb(m, i) * tau ** i * (1 - tau) ** (m - i) for i in range(m + 1)], 1)

    def diff(m):  # coefficients of a degree-m polynomial -> those of its derivative
        return m * (np.eye(m + 1)[1:] - np.eye(m + 1)[:-1]) / T

    return bern(n), bern(n - 1) @ diff(n), bern(n - 2) @ diff(n - 1) @ diff(n)


def _project64(case, bc, obs, xi):
    """The projection of one problem's samples xi [N, D] (Appendix, eqs. (14)-(15)), in 64 bits."""
    c, dev = case, xi.device
    d, nv, K, M = c["dims"], c["n_coeff"], c["n_steps"], c["n_obs"]
    rows = _basis(nv, K, c["horizon"])
    Pm, Pd, Pdd = (torch.as_tensor(x, dtype=torch.float64, device=dev) for x in rows)
    FtF = (M + (2 if c["bounds"] else 0)) * Pm.T @ Pm + Pd.T @ Pd + Pdd.T @ Pdd
    A = torch.stack([Pm[0], Pd[0], Pdd[0], Pm[-1], Pd[-1], Pdd[-1]][:6])
    use = list(range(6)) if c["rest"] else [0, 1, 2, 3]
    A, E = A[use], len(use)
    kkt = torch.zeros((nv + E, nv + E), dtype=torch.float64, device=dev)
    kkt[:nv, :nv] = torch.eye(nv, device=dev) + FtF
    kkt[:nv, nv:], kkt[nv:, :nv] = A.T, A
    inv = torch.linalg.inv(kkt)[:nv]
    b = bc[:, use]  # [d, E]
    v_max, a_max = _limits(c)
    s_min, s_max = _bounds(c)
    t = torch.arange(K, dtype=torch.float64, device=dev) * (c["horizon"] / (K - 1))
    if c["paths"]:
        opos, axes = obs[:, :K * d].reshape(M, K, d), obs[:, K * d:]
    else:
        opos, axes = obs[:, None, :d] + obs[:, None, 3:3 + d] * t[:, None], obs[:, 6:8]
    semi = axes[:, [0, 0, 1][:d]]  # [M, d]

    def pushes(x):
        """Push-outs of the position, velocity and acceleration rows, and the squared residual."""
        p, v, a = (torch.einsum("ndc,kc->ndk", x, W) for W in (Pm, Pd, Pdd))
        S, r2 = torch.zeros_like(p), torch.zeros((x.shape[0], K), dtype=torch.float64, device=dev)
        for j in range(M):
            delta = p - opos[j].T
            n = ((delta / semi[j][:, None]) ** 2).sum(1).sqrt()
            e = delta * torch.clamp(1 / torch.clamp(n, min=1e-12) - 1, min=0)[:, None]
            S += e
            r2 += (e * e).sum(1)
        out = []
        for w, top in ((v, v_max), (a, a_max)):
            e = w * torch.clamp(top / torch.clamp(w.norm(dim=1), min=1e-30) - 1, max=0)[:, None]
            r2 += (e * e).sum(1)
            out.append(e)
        if s_min is not None:
            for x_ in range(d):
                e = p[:, x_].clamp(s_min[x_], s_max[x_]) - p[:, x_]
                S[:, x_] += e
                r2 += e * e
        return S, out[0], out[1], r2, (p, v, a)

    x0 = xi.reshape(-1, d, nv)
    x, lam = x0.clone(), torch.zeros_like(x0)
    for _ in range(c["n_proj_iters"]):
        S, dv, da, _, _ = pushes(x)
        g = S @ Pm + dv @ Pd + da @ Pdd
        lam = lam + g
        eta = x0 + lam + g + x @ FtF
        x = torch.einsum("ndc,ec->nde", torch.cat([eta, b.expand(len(x), d, E)], 2), inv)
    _, _, _, r2, pva = pushes(x)
    return x.reshape(-1, d * nv), r2.sum(1).sqrt(), _cost64(c, bc, pva)


def _cost64(case, bc, pva):
    p, v, a = pva
    acc = (a * a).sum(1)
    if not case["weighted"]:
        return acc.sum(1)
    den = ((v * v).sum(1) + 1e-2) ** 1.5
    if case["dims"] == 2:
        cross = v[:, 0] * a[:, 1] - v[:, 1] * a[:, 0]
        kappa2, steer2 = (cross / den) ** 2, torch.atan(cross / den) ** 2
    else:
        kappa2 = (torch.linalg.cross(v, a, dim=1) ** 2).sum(1) / den ** 2
        steer2 = 0.0
    u = (bc[:, 3] - bc[:, 0])[:, None]
    rel = p - bc[:, 0][:, None]
    lam = ((rel * u).sum(1) / (u * u).sum()).clamp(0, 1)
    dist = (rel - lam[:, None] * u).norm(dim=1)
    return (acc + 0.5 * kappa2 + 0.2 * dist + 0.3 * steer2).sum(1)


def exact(case, seed):
    c = case
    one_draw = c["kind"] in ("plan", "plan_batch") and c["n_cem"] == 1
    if c["kind"] not in ("project", "project_batch") and not one_draw:
        return None
    pairs = float(c["n_samples"]) * c["n_problems"] * c["n_steps"] * (c["n_obs"] + 4) * c["n_proj_iters"]
    if pairs > 1e11:
        return None
    inp = _inputs(c, seed)
    bc, obs = (_t(inp[k]).double() for k in ("bc", "obs"))
    if one_draw:
        xi = torch.stack([_normals(int(seed), q, c["n_samples"], inp["mean"].size)
                          for q in range(c["n_problems"])])
        D = inp["mean"].size  # Sigma = I, factored with its jitter: 1e-5 tr(Sigma) / D = 1e-5
        xi = xi * math.sqrt(1.0 + 1e-5) + _t(inp["mean"]).double()
    else:
        xi = _samples(c, seed, inp["mean"]).double()
    step = max(1, int(4e7 // (c["dims"] * c["n_steps"])))
    res = []
    for q in range(c["n_problems"]):
        parts = [_project64(c, bc[q], obs[q], x) for x in xi[q].split(step)]
        res.append([torch.cat(x) for x in zip(*parts)])
    xo, r, c1 = (torch.stack(x) for x in zip(*res))
    if one_draw:  # the selections and what rests on them turn on ties of rounding
        rest = dict.fromkeys(["best_xi", "best_cost", "elite_idx", "proj_idx", "status", "mu", "cov"])
        return dict(rest, xi=xi, xi_bar=xo, resid=r, c1=c1)
    if c["kind"] == "project":
        xo, r, c1 = xo[0], r[0], c1[0]
    return {"xi_bar": xo, "resid": r, "c1": c1}


def _normals(seed, stream, n, D):
    """The first draw's standard normals: Philox4x32-10 with counter (sample, d / 4, 0, stream)
    and key `seed` (Salmon et al., SC'11), then Box-Muller in 64 bits."""
    nq = (D + 3) // 4
    full = 0xFFFFFFFF
    w = [np.repeat(np.arange(n, dtype=np.uint64), nq), np.tile(np.arange(nq, dtype=np.uint64), n),
         np.zeros(n * nq, np.uint64), np.full(n * nq, stream, np.uint64)]
    k0, k1 = seed & full, (seed >> 32) & full
    for _ in range(10):
        lo, hi = w[0] * np.uint64(0xD2511F53), w[2] * np.uint64(0xCD9E8D57)
        w = [(hi >> np.uint64(32)) ^ w[1] ^ np.uint64(k0), hi & np.uint64(full),
             (lo >> np.uint64(32)) ^ w[3] ^ np.uint64(k1), lo & np.uint64(full)]
        k0, k1 = (k0 + 0x9E3779B9) & full, (k1 + 0xBB67AE85) & full
    u = [((x >> np.uint64(9)).astype(np.float64) + 0.5) * 2.0 ** -23 for x in w]
    z = np.stack([f(u[2 * h], u[2 * h + 1]) for h in (0, 1) for f in (
        lambda a, b: np.sqrt(-2 * np.log(a)) * np.cos(2 * np.pi * b),
        lambda a, b: np.sqrt(-2 * np.log(a)) * np.sin(2 * np.pi * b))], 1)
    return torch.as_tensor(z.reshape(n, 4 * nq)[:, :D].copy(), device=DEV)
