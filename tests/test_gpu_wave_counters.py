"""The whole-horizon projection shapes inside batched plans, where the waves
draw sample groups from the problems' counters (at most 64 are used) and stage
the factor's rows a few at a time: the same plans, bit for bit, as the
time-split shape gives."""
import numpy as np
import pytest
import torch

from paper_2309_08235_amd import workloads as W
from tests.test_gpu_parity import _cem
from tests.test_gpu_refit_paths import t32

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2309_08235_amd.priest")

CASES = [
    # (base, problems, samples, coefficients)
    (W.C1, 1, 70, 11), (W.C1, 2, 9, 16), (W.C1, 63, 33, 11), (W.C1, 64, 17, 7), (W.C1, 65, 64, 13),
    (W.C1, 130, 12, 11), (W.C3, 1, 30, 16), (W.C3, 3, 130, 11), (W.C3, 70, 6, 12),
]


@pytest.mark.parametrize("base,n_problems,n,n_coeff", CASES,
                         ids=[f"{c[0].dims}d {c[1]}x{c[2]} nv{c[3]}" for c in CASES])
def test_batched_plans_identical_in_every_shape(base, n_problems, n, n_coeff):
    print(f"counters: {base.dims}d P={n_problems} N={n} nv={n_coeff}", flush=True)
    wl = W.with_changes(base, n_obs=min(base.n_obs, 20), n_coeff=n_coeff, n_samples=n,
                        n_proj=max(1, (3 * n) // 4), n_elite=max(1, n // 4), n_proj_iters=12)
    gp = P.Problem.from_workload(wl)
    scenes = [W.scene(wl, 3 + i) for i in range(n_problems)]
    bc = t32(np.stack([s[0] for s in scenes]))
    obs = t32(np.stack([s[1] for s in scenes]))
    cem = _cem(wl, n_cem=3)
    want = None
    for shape in [(4, 1, 0)] + [c for c in gp.tiling_candidates() if c[1] == 0]:
        gp.set_tiling(shape)
        mu = t32(np.stack([W.initial_mean(wl)] * n_problems))
        cov = t32(np.stack([W.initial_cov(wl)] * n_problems))
        out = gp.plan_batch(n_problems, bc, obs, cem, mu, cov, seed=5)
        torch.cuda.synchronize()
        got = [out[k] for k in ("best_xi", "best_cost", "xi", "xi_bar", "resid", "c1", "status")] + [mu, cov]
        if want is None:
            want = [g.clone() for g in got]
        else:
            for a, b in zip(want, got):
                assert torch.equal(a, b), shape
    gp.close()
