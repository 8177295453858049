"""The shape picked in one call serves calls of every iteration count, so the
launches that the tuner times are alike whichever call comes first."""
import subprocess

from paper_2309_08235_amd import build

PROGRAM = """
#include <cstdio>
#include "priest_internal.h"
int main() {
  int bad = 0;
  for (int bf = 0; bf <= 1; ++bf) {
    priest::ProjArgs want{};
    for (int n : {1, 2, 8, 10, 11, 23, 24, 25, 60, 100, 500}) {
      priest::ProjArgs a{};
      a.n_iter = n;
      a.bf16_iters = bf ? (n > 10 ? n - 10 : 1) : 0;
      const priest::ProjArgs t = priest::trial_args(a);
      if (n == 1) want = t;
      if (t.n_iter < 1 || t.n_iter != want.n_iter || t.bf16_iters != want.bf16_iters ||
          t.trial_of != want.trial_of || (t.bf16_iters > 0) != (bf > 0) || t.bf16_iters > t.n_iter) {
        ++bad;
        std::printf("%d iterations, %d: trial of %d (%d, %d)\\n", n, bf, t.n_iter, t.bf16_iters, t.trial_of);
      }
    }
  }
  return bad != 0;
}
"""


def test_trials_do_not_depend_on_the_first_call(tmp_path):
    src, exe = tmp_path / "trial.hip", str(tmp_path / "trial")
    src.write_text(PROGRAM)
    subprocess.run([build.HIPCC, *build.FLAGS, "-I", build.CSRC, str(src), "-L" + build.PKG,
                    "-l:libpriest.so", "-Wl,-rpath," + build.PKG, "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
