"""Batched plans captured as two chains of half the problems (launches of one
to three times the waves that the device holds), replayed several times with
eager work in between: the same outputs, bit for bit, as the eager loop."""
import numpy as np
import pytest
import torch

from paper_2309_08235_amd import workloads as W
from tests.test_gpu_parity import _cem
from tests.test_gpu_refit_paths import t32

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2309_08235_amd.priest")

CASES = [
    # (base, shape, problems, samples, given noise, CMA rule); K = 100: 7 waves
    # a time-split block; one wave per 16 / slots samples otherwise
    (W.C2, (2, 1, 0), 9, 1000, False, False),    # 7875 waves
    (W.C2, (2, 0, 1), 63, 600, False, True),     # 4725
    (W.C2, (2, 0, 0), 13, 2048, True, False),    # 3328: one chain
    (W.C2, (4, 0, 0), 11, 2000, True, True),     # 5500
    (W.C3, (4, 0, 1), 17, 1001, True, False),    # 4267
]


@pytest.mark.parametrize("base,shape,n_problems,n,given,cma", CASES,
                         ids=[f"{c[0].dims}d {c[1]} {c[2]}x{c[3]}" for c in CASES])
def test_captured_batch_equals_eager(base, shape, n_problems, n, given, cma):
    print(f"halves: {base.dims}d {shape} P={n_problems} N={n}", flush=True)
    wl = W.with_changes(base, n_obs=min(base.n_obs, 20), n_samples=n, n_proj=W.default_n_proj(n),
                        n_elite=W.default_n_elite(n), n_proj_iters=10)
    gp = P.Problem.from_workload(wl)
    gp.set_tiling(shape)
    scenes = [W.scene(wl, 3 + i) for i in range(n_problems)]
    bc = t32(np.stack([s[0] for s in scenes]))
    obs = t32(np.stack([s[1] for s in scenes]))
    cem = _cem(wl, n_cem=3, **({"update": 1} if cma else {}))
    noise = None
    if given:
        g = torch.Generator(device="cuda").manual_seed(3)
        noise = torch.randn((n_problems, 3, n, wl.D), generator=g, device="cuda")
    mu0 = t32(np.stack([W.initial_mean(wl)] * n_problems))
    cov0 = t32(np.stack([W.initial_cov(wl)] * n_problems))
    stream = torch.cuda.Stream()
    ws = gp.workspace(cem, n_problems)
    out_g, mu_g, cov_g = gp.plan_outputs(cem, n_problems), mu0.clone(), cov0.clone()
    for seed in (5, 5, 5):
        mu_e, cov_e = mu0.clone(), cov0.clone()
        out_e = gp.plan_batch(n_problems, bc, obs, cem, mu_e, cov_e, seed=seed, noise=noise)
        mu_g.copy_(mu0)
        cov_g.copy_(cov0)
        for v in out_g.values():
            v.zero_()
        torch.cuda.synchronize()
        gp.plan_batch(n_problems, bc, obs, cem, mu_g, cov_g, seed=seed, noise=noise, out=out_g,
                      workspace=ws, use_graph=True, stream=stream)
        torch.cuda.synchronize()
        for k, v in out_e.items():
            assert torch.equal(v, out_g[k]), k
        assert torch.equal(mu_e, mu_g) and torch.equal(cov_e, cov_g)
    gp.close()


@pytest.mark.parametrize("base,shape,n_problems,n,cma", [
    (W.C2, (2, 1, 0), 7, 901, False),    # 5537 waves
    (W.C2, (2, 0, 1), 63, 600, True),    # 4725
    (W.C3, (4, 0, 1), 21, 850, False),   # 4473
], ids=["2d time-split", "2d counter", "3d counter"])
def test_longer_captured_batch_equals_eager(base, shape, n_problems, n, cma):
    """As above, with the iterations that earn the second chain, and no given noise."""
    print(f"halves: {base.dims}d {shape} P={n_problems} N={n}, 30 iterations", flush=True)
    wl = W.with_changes(base, n_obs=min(base.n_obs, 20), n_samples=n, n_proj=W.default_n_proj(n),
                        n_elite=W.default_n_elite(n), n_proj_iters=30)
    gp = P.Problem.from_workload(wl)
    gp.set_tiling(shape)
    scenes = [W.scene(wl, 3 + i) for i in range(n_problems)]
    bc, obs = t32(np.stack([s[0] for s in scenes])), t32(np.stack([s[1] for s in scenes]))
    cem = _cem(wl, n_cem=3, **({"update": 1} if cma else {}))
    mu0 = t32(np.stack([W.initial_mean(wl)] * n_problems))
    cov0 = t32(np.stack([W.initial_cov(wl)] * n_problems))
    stream, ws = torch.cuda.Stream(), gp.workspace(cem, n_problems)
    out, mu, cov = gp.plan_outputs(cem, n_problems, full=True), mu0.clone(), cov0.clone()
    for _ in range(3):
        mu_e, cov_e = mu0.clone(), cov0.clone()
        want = gp.plan_batch(n_problems, bc, obs, cem, mu_e, cov_e, seed=5)
        mu.copy_(mu0), cov.copy_(cov0)
        for v in out.values():
            v.zero_()
        torch.cuda.synchronize()
        gp.plan_batch(n_problems, bc, obs, cem, mu, cov, seed=5, out=out, workspace=ws, use_graph=True,
                      stream=stream)
        torch.cuda.synchronize()
        for k, v in want.items():
            assert torch.equal(v, out[k]), k
        assert torch.equal(mu_e, mu) and torch.equal(cov_e, cov)
    gp.close()
