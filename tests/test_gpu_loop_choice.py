"""The time-split shapes run a loop without obstacle searches in the first
iterations and in crowded tiles, and a searching loop in between; the whole-horizon
shape has neither and the same bits.  Cases: iteration counts on both sides of
every point where the loop may change (after 4, 12, 28 iterations; 8 and 24
searching ones later), scenes in which no, some and all tiles are crowded, more
than the two groups of 64 obstacles whose masks a wave keeps in registers, every
obstacle and radius kind."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2309_08235_amd import workloads as W
from tests.parity import check_projection, oracle_problem
from tests.test_gpu_near_obstacles import _scene, t32

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P(gpu_lib):
    from paper_2309_08235_amd import priest
    return priest


def _project(P, wl, bc, obs, xi, n_iters, **options):
    """Results of every tile shape: {shape: [tensors of each iteration count]}."""
    prob = P.Problem.from_workload(wl, **options)
    out = {}
    for c in prob.tiling_candidates():
        prob.set_tiling(c)
        out[c] = [x.cpu().numpy() for n in n_iters for x in prob.project(t32(bc), t32(obs), xi, n)]
    prob.close()
    return out


def _same(out, label):
    want = out[(4, 0, 0)]
    for c, got in out.items():
        for g, w in zip(got, want):
            np.testing.assert_array_equal(g, w, err_msg=f"{label} tiling {c}")


EDGES = [1, 3, 4, 5, 7, 8, 9, 11, 12, 13, 15, 16, 17, 19, 20, 24, 27, 28, 29, 36, 37, 52, 61]
SCENES = [  # dims, obstacles, of them in one place, steps, samples
    (2, 3, 0, 33, 9), (2, 40, 6, 100, 21), (2, 129, 0, 64, 13), (2, 260, 70, 100, 9), (2, 400, 0, 40, 30),
    (3, 5, 4, 33, 6), (3, 129, 66, 100, 9), (3, 300, 0, 64, 10),
]


@pytest.mark.parametrize("dims,M,crowd,K,N", SCENES)
def test_every_iteration_count_has_the_same_bits(P, dims, M, crowd, K, N):
    print(f"[gpu-case] loop choice: {dims}D M={M} crowd={crowd} K={K} N={N}", flush=True)
    wl, bc, obs = _scene(dims, M, crowd, 11)
    wl = W.with_changes(wl, n_steps=K)
    _same(_project(P, wl, bc, obs, t32(W.samples(wl, 3, n=N)), EDGES), f"{dims}D M={M}")


@pytest.mark.parametrize("M,crowd", [(5, 4), (129, 66), (300, 0)])
def test_every_iteration_count_in_space(P, M, crowd):
    """In 3D the loop may change after 1, 3, 7, 15 and 31 iterations, with 4 left."""
    print(f"[gpu-case] loop choice: 3D edges M={M} crowd={crowd}", flush=True)
    wl, bc, obs = _scene(3, M, crowd, 12)
    counts = [1, 2, 4, 5, 6, 7, 8, 11, 12, 14, 15, 18, 19, 20, 31, 34, 35, 36]
    _same(_project(P, wl, bc, obs, t32(W.samples(wl, 3, n=10)), counts), f"3D M={M}")


@pytest.mark.parametrize("dims", [2, 3])
@pytest.mark.parametrize("kind", ["radii", "bounds", "bf16"])
@pytest.mark.parametrize("M,crowd", [(12, 0), (150, 40)])
def test_every_kind_has_the_same_bits(P, dims, kind, M, crowd):
    print(f"[gpu-case] loop choice: {dims}D {kind} M={M}", flush=True)
    wl, bc, obs = _scene(dims, M, crowd, 13)
    options = {}
    if kind == "radii":
        obs[::3, 6:8] *= 1.25
    elif kind == "bounds":
        lo, hi = np.minimum(bc[:, 0], bc[:, 3]) - 1.0, np.maximum(bc[:, 0], bc[:, 3]) + 1.0
        options = dict(s_min=lo.tolist(), s_max=hi.tolist())
    else:
        options = dict(precision=1, n_refine_fp32=4)
    xi = t32(W.samples(wl, 3, n=11))
    _same(_project(P, wl, bc, obs, xi, [5, 12, 13, 28, 40], **options), f"{dims}D {kind}")


@pytest.mark.parametrize("dims", [2, 3])
@pytest.mark.parametrize("M,crowd", [(12, 0), (150, 40)])
def test_paths_match_oracle(P, dims, M, crowd):
    """Obstacle paths have one tile shape only: against the oracle."""
    print(f"[gpu-case] loop choice: {dims}D paths M={M}", flush=True)
    wl, bc, obs = _scene(dims, M, crowd, 13)
    prob, op = P.Problem.from_workload(wl, obs_model=P.OBS_PATH), oracle_problem(wl, obs_model=1)
    path = W.trajectory_obstacles(wl, obs, swirl=0.5, seed=5)
    xi = W.samples(wl, 3, n=11).astype(np.float32)
    for n in (5, 13, 28):
        want = O.project(op, bc, path, xi.astype(np.float64), n).xi_bar
        got = prob.project(t32(bc), t32(path), t32(xi), n)[0].cpu().numpy()
        check_projection(op, bc, path, xi, got, want, n, label=f"{dims}D paths, {n} iterations")
    prob.close()


@pytest.mark.parametrize("n_iter,most", [(6, 0.185), (40, 0.16)])
def test_crowded_scene_keeps_its_lead(P, n_iter, most):
    """500 obstacles in the plane, 1000 samples: every tile is crowded.  A search
    in each iteration costs more there than it saves: the split shape then took
    0.255 (6 iterations) and 0.206 (40) of the whole-horizon shape's kernel time,
    without searches 0.134 and 0.123; the bounds are the geometric means."""
    print(f"[gpu-case] loop choice: kernel times, {n_iter} iterations", flush=True)
    wl = W.with_changes(W.C2, n_obs=500)
    bc, obs = W.scene(wl, 0)
    prob = P.Problem.from_workload(wl)
    bc, obs, xi = t32(bc), t32(obs), t32(W.samples(wl, 7, n=1000))
    ms = {}
    for c in ((4, 1, 0), (4, 0, 0)):
        prob.set_tiling(c)
        prob.project(bc, obs, xi, n_iter)
        times = []
        for _ in range(6):
            torch.cuda.synchronize()
            P.priest_profile_read()
            P.priest_profile_enable(True)
            for _ in range(8):
                prob.project(bc, obs, xi, n_iter)
            P.priest_profile_enable(False)
            n, t = P.priest_profile_read()
            times.append(t / n)
        ms[c] = min(times)
    prob.close()
    assert ms[(4, 1, 0)] <= most * ms[(4, 0, 0)], ms
