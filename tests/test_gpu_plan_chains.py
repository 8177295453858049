"""How many chains a captured batch takes, and that it falls back to one, with the
same outputs, where the second stream cannot be had.  A library loaded ahead of
the HIP runtime counts the streams that the plan call creates and can refuse
them, leaving an error behind as a failed creation does; so each case runs in a
process of its own."""
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

SHIM = """
typedef int (*create_t)(void**, unsigned);
typedef int (*device_t)(int);
static create_t create;
static device_t device;
int created, refuse;
void set_real(void* c, void* d) { create = (create_t)c; device = (device_t)d; }
int hipStreamCreateWithFlags(void** s, unsigned flags) {
  ++created;
  return refuse ? device(1 << 20) : create(s, flags);  // (no such device: an error, and it sticks)
}
"""

CHILD = """
import ctypes, os, sys
shim = ctypes.CDLL(sys.argv[1], mode=os.RTLD_GLOBAL | os.RTLD_NOW)
import numpy as np
import torch
sys.path.insert(0, sys.argv[2])
from paper_2309_08235_amd import priest as P, workloads as W
from tests.test_gpu_parity import _cem
hip = P.lib()
shim.set_real(ctypes.cast(hip.hipStreamCreateWithFlags, ctypes.c_void_p),
              ctypes.cast(hip.hipSetDevice, ctypes.c_void_p))
created, refuse = (ctypes.c_int.in_dll(shim, n) for n in ("created", "refuse"))
chains, refused, n_cem = (int(v) for v in sys.argv[3:6])
cus = torch.cuda.get_device_properties(0).multi_processor_count
# K = 100, 2 axis slots: 7 waves for 8 samples; 1.5 times the 16 waves that each CU holds
n_problems = 9
n = 8 * ((24 * cus) // (7 * n_problems))
wl = W.with_changes(W.C2, n_obs=10, n_samples=n, n_proj=W.default_n_proj(n),
                    n_elite=W.default_n_elite(n), n_proj_iters=30)
gp = P.Problem.from_workload(wl)
gp.set_tiling((2, 1, 0))
t32 = lambda x: torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float32).cuda()
scenes = [W.scene(wl, 3 + i) for i in range(n_problems)]
bc, obs = t32(np.stack([s[0] for s in scenes])), t32(np.stack([s[1] for s in scenes]))
cem = _cem(wl, n_cem=n_cem)
g = torch.Generator(device="cuda").manual_seed(3)
noise = torch.randn((n_problems, n_cem, n, wl.D), generator=g, device="cuda")
mu0 = t32(np.stack([W.initial_mean(wl)] * n_problems))
cov0 = t32(np.stack([W.initial_cov(wl)] * n_problems))
stream, ws = torch.cuda.Stream(), gp.workspace(cem, n_problems)
out, mu, cov = gp.plan_outputs(cem, n_problems, full=True), mu0.clone(), cov0.clone()
refuse.value = refused
if sys.argv[6] == "pending":  # an error that someone else left is reported, not swallowed
    hip.hipSetDevice(1 << 20)
    try:
        gp.plan_batch(n_problems, bc, obs, cem, mu, cov, seed=5, noise=noise, out=out, workspace=ws,
                      use_graph=True, stream=stream)
    except P.PriestError as e:
        print("reported:", e, flush=True)
        sys.exit(0)
    sys.exit("not reported")
for replay in range(3):
    mu_e, cov_e = mu0.clone(), cov0.clone()
    want = gp.plan_batch(n_problems, bc, obs, cem, mu_e, cov_e, seed=5, noise=noise,
                         out=gp.plan_outputs(cem, n_problems, full=True))
    mu.copy_(mu0), cov.copy_(cov0)
    for v in out.values():
        v.zero_()
    torch.cuda.synchronize()
    before = created.value
    gp.plan_batch(n_problems, bc, obs, cem, mu, cov, seed=5, noise=noise, out=out, workspace=ws,
                  use_graph=True, stream=stream)
    torch.cuda.synchronize()
    assert created.value - before == (chains == 2 and replay == 0), created.value - before
    for k, v in want.items():
        assert torch.equal(v, out[k]), k
    assert torch.equal(mu_e, mu) and torch.equal(cov_e, cov)
gp.close()
print("same outputs", flush=True)
"""


@pytest.mark.parametrize("chains,refused,n_cem", [(2, 0, 3), (2, 1, 3), (1, 0, 1)])
def test_chains_of_a_captured_batch(tmp_path, gpu_lib, chains, refused, n_cem):
    print(f"[gpu-case] plan chains: {chains} refused={refused} n_cem={n_cem}", flush=True)
    from tests.conftest import ROOT
    src, shim, child = tmp_path / "shim.c", str(tmp_path / "shim.so"), tmp_path / "child.py"
    src.write_text(SHIM)
    child.write_text(CHILD)
    subprocess.run(["gcc", "-shared", "-fPIC", str(src), "-o", shim], check=True)
    r = subprocess.run([sys.executable, str(child), shim, ROOT, str(chains), str(refused), str(n_cem), ""],
                       capture_output=True, text=True, timeout=110)
    assert r.returncode == 0 and "same outputs" in r.stdout, r.stdout + r.stderr


def test_an_error_from_before_a_captured_batch_is_reported(tmp_path, gpu_lib):
    """One chain creates no stream, so there is no error of its own to take back."""
    print("[gpu-case] plan chains: an error pending before the call", flush=True)
    from tests.conftest import ROOT
    src, shim, child = tmp_path / "shim.c", str(tmp_path / "shim.so"), tmp_path / "child.py"
    src.write_text(SHIM)
    child.write_text(CHILD)
    subprocess.run(["gcc", "-shared", "-fPIC", str(src), "-o", shim], check=True)
    r = subprocess.run([sys.executable, str(child), shim, ROOT, "1", "0", "1", "pending"],
                       capture_output=True, text=True, timeout=110)
    assert r.returncode == 0 and "reported:" in r.stdout, r.stdout + r.stderr
