"""The refit kernel where its branches change: selections whose keys fall into
one bin of the value histogram, sit at both ends of it or are not finite, and
refits of as many elites as are staged at once, or one more."""
import numpy as np
import pytest
import torch

from paper_2309_08235_amd import workloads as W
from tests.parity import oracle_problem
from tests.test_gpu_parity import _cem, _check_cem_step
from tests.test_gpu_refit_paths import np64, t32
from tests.test_gpu_select import reference

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2309_08235_amd.priest")


def keys(kind, n, rng):
    if kind == "one_bin":       # values a few ulps apart, and one far away
        v = (np.float32(1.0) + rng.integers(0, 5 * n, n).astype(np.float32) * np.float32(2.0**-22))
        v[n // 2] = 1e30
    elif kind == "two_ends":    # at most two values in the histogram
        v = np.where(rng.random(n) < 0.5, 0.0, 3.0e38).astype(np.float32)
    elif kind == "not_finite":
        v = rng.random(n, dtype=np.float32)
        v[::4] = np.inf
        v[1::7] = np.nan
    else:                       # "denormal": no spread that a quotient could use
        v = (rng.integers(0, n, n).astype(np.float32) * np.float32(1e-45))
    return v


@pytest.mark.parametrize("kind", ["one_bin", "two_ends", "not_finite", "denormal"])
@pytest.mark.parametrize("n", [1, 64, 513, 1024, 1025, 2048])
def test_selection_of_crafted_keys(kind, n):
    print(f"select {kind} N={n}", flush=True)
    rng = np.random.default_rng(n + len(kind))
    r = keys(kind, n, rng)
    c1 = (rng.integers(0, 3, n) * 0.5).astype(np.float32)
    for n_proj, n_elite in {(n, n if n <= 512 else 512), (max(1, n // 2), max(1, n // 5)), (max(1, n // 3), 1)}:
        with np.errstate(over="ignore", invalid="ignore"):
            # NaN ranks as +inf
            _, want = reference(np.where(np.isnan(r), np.float32(np.inf), r), c1, n_proj, n_elite)
        e = torch.full((n_elite,), -1, dtype=torch.int32, device="cuda")
        P.priest_debug_select(n_proj, n_elite, torch.tensor(r, device="cuda"), torch.tensor(c1, device="cuda"), e)
        np.testing.assert_array_equal(e.cpu().numpy(), want)


@pytest.mark.parametrize("n_coeff,n_elite", [(12, 170), (12, 171), (16, 128), (16, 256), (16, 384), (16, 385)])
def test_refit_of_all_staged_elites_or_one_more(n_coeff, n_elite):
    """2D, D = 24 and 32: rows of 4080, 4104, 4096, 8192, 12288 and 12320 values."""
    print(f"refit n_coeff={n_coeff} n_elite={n_elite}", flush=True)
    n = 560
    wl = W.with_changes(W.C1, n_coeff=n_coeff, n_samples=n, n_proj=W.default_n_proj(n), n_elite=n_elite,
                        n_proj_iters=10)
    gp = P.Problem.from_workload(wl)
    bc, obs = W.boundary_values(wl), W.obstacles(wl, 5)
    cem = _cem(wl)
    mu0, cov0 = W.initial_mean(wl), W.initial_cov(wl)
    noise = W.standard_normals(7, (1, wl.n_samples, wl.D))
    mu, cov = t32(mu0), t32(cov0)
    out = gp.plan(t32(bc), t32(obs), cem, mu, cov, noise=t32(noise))
    torch.cuda.synchronize()
    _check_cem_step(oracle_problem(wl), bc, obs, wl, cem, mu0, cov0, noise[0], out, np64(mu), np64(cov),
                    f"n_coeff={n_coeff} n_elite={n_elite}")
    gp.close()


def test_served_refits_of_mixed_sizes():
    """Requests of one server step share a refit launch: the largest number of
    elites of the largest problems (D = 48) beside few, and beside as many as
    have all rows staged, with the results of each request alone."""
    from paper_2309_08235_amd import serve as S
    sw = W.ServingWorkload(dims=3, n_coeff=16, n_proj_iters=4, n_cem=2, n_robots=3)
    bc = np.zeros((3, 6))
    bc[:, 3] = 7.0
    obs = np.zeros((3, 8))
    obs[:, :3] = np.array([[2, 2, 3], [4, 5, 4], [5, 4, 6]])
    obs[:, 6] = obs[:, 7] = 0.5
    reqs = [W.ServingRequest(index=i, robot=i, arrival=0.0, n_samples=n, n_obs=3, n_steps=50, horizon=10.0,
                             n_proj=n_proj, n_elite=n_elite, bc=bc, obs=obs)
            for i, (n, n_proj, n_elite) in enumerate([(2048, 2048, 2048), (1000, 700, 256), (64, 40, 5)])]

    def serve(rs):
        s = S.Server.for_workload(sw, max_active=8, max_robots=3, memory_budget=64 << 20, seed=9)
        for q in rs:
            s.submit_request(q, sw, warm_start=1)
        done = s.drain()
        s.close()
        return {c.request_id: c for c in done}

    print("served refits: 2048, 256 and 5 elites, D = 48", flush=True)
    mixed = serve(reqs)
    assert len(mixed) == 3
    for k, q in enumerate(reqs):
        alone = serve([q])[1]
        assert alone.status == 0 and mixed[k + 1].status == 0
        assert alone.best_cost == mixed[k + 1].best_cost
        np.testing.assert_array_equal(alone.best_xi, mixed[k + 1].best_xi)
