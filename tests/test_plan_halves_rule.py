"""Which captured plan loops run as two chains of half the problems each: those
of more waves than the device holds and under three times as many (two, where
the whole-horizon shape draws its groups from a counter), and of enough CEM
iterations for one half's refits to overlap the other's projections."""
import subprocess

from paper_2309_08235_amd import build

PROGRAM = """
#include <cstdio>
#include "priest_internal.h"
using namespace priest;
int bad = 0;
void want(bool two, int P, int n_cem, int dims, int K, int N, TileCfg t) {
  ProjArgs a{};
  a.dims = dims, a.nv = 11, a.K = K, a.N = N, a.n_iter = 50;
  apply_tiling(a, t);
  if (halves_pay(a, P, n_cem, 256) != two) {
    ++bad;
    std::printf("P=%d cem=%d %dD K=%d N=%d %d%d%d: %d\\n", P, n_cem, dims, K, N, t.axis_slots,
                t.row_tiles, t.persistent, !two);
  }
}
int main() {
  for (int P : {5, 6, 8, 10, 14}) {
    want(false, P, 1, 2, 100, 1000, TileCfg{2, 1, 0});  // nothing to overlap
    for (int cem : {2, 3, 20}) want(true, P, cem, 2, 100, 1000, TileCfg{2, 1, 0});
  }
  want(false, 4, 20, 2, 100, 1000, TileCfg{2, 1, 0});   // 0.85
  want(false, 15, 20, 2, 100, 1000, TileCfg{2, 1, 0});  // 3.2
  want(false, 1, 20, 2, 100, 8000, TileCfg{2, 1, 0});   // one problem
  // whole horizon: one wave per group, up to three rounds
  for (int N : {1000, 1300, 1700, 2000}) {
    want(true, 22, 2, 3, 100, N, TileCfg{4, 0, 0});
    want(false, 22, 1, 3, 100, N, TileCfg{4, 0, 0});
  }
  // groups drawn from a counter: three CEM iterations, under two rounds
  for (int N : {757, 1000, 1350}) {
    for (int cem : {1, 2}) want(false, 22, cem, 3, 108, N, TileCfg{4, 0, 1});
    want(true, 22, 3, 3, 108, N, TileCfg{4, 0, 1});
  }
  for (int N : {1500, 1750, 2000})
    for (int cem : {1, 3, 20}) want(false, 22, cem, 3, 108, N, TileCfg{4, 0, 1});
  return bad != 0;
}
"""


def test_two_chains_only_where_they_pay(tmp_path):
    src, exe = tmp_path / "halves.hip", str(tmp_path / "halves")
    src.write_text(PROGRAM)
    subprocess.run([build.HIPCC, *build.FLAGS, "-I", build.CSRC, str(src), "-L" + build.PKG,
                    "-l:libpriest.so", "-Wl,-rpath," + build.PKG, "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr


def test_loops_of_little_work_take_one_chain(tmp_path):
    """The fork and join have to be earned back: by n_cem (n_iter + 10) = 120, or
    60 with one wave a group, and with a counter by 20 problems."""
    program = PROGRAM[:PROGRAM.index("int main")].replace("a.n_iter = 50", "a.n_iter = iters")
    program = program.replace("int bad = 0;", "int bad = 0, iters;") + """
int main() {
  iters = 5;
  for (int cem : {2, 4, 7}) want(false, 9, cem, 2, 100, 1000, TileCfg{2, 1, 0});
  want(true, 9, 8, 2, 100, 1000, TileCfg{2, 1, 0});
  want(false, 22, 3, 3, 100, 1000, TileCfg{4, 0, 0});
  want(true, 22, 4, 3, 100, 1000, TileCfg{4, 0, 0});
  iters = 30;
  want(false, 9, 2, 2, 100, 1000, TileCfg{2, 1, 0});
  want(true, 9, 3, 2, 100, 1000, TileCfg{2, 1, 0});
  want(false, 19, 20, 3, 100, 1200, TileCfg{4, 0, 1});
  want(true, 20, 20, 3, 100, 1200, TileCfg{4, 0, 1});
  want(true, 24, 3, 3, 100, 1200, TileCfg{4, 0, 1});   // 1.76
  want(false, 26, 20, 3, 100, 1200, TileCfg{4, 0, 1});  // 1.90
  return bad != 0;
}
"""
    src, exe = tmp_path / "little.hip", str(tmp_path / "little")
    src.write_text(program)
    subprocess.run([build.HIPCC, *build.FLAGS, "-I", build.CSRC, str(src), "-L" + build.PKG,
                    "-l:libpriest.so", "-Wl,-rpath," + build.PKG, "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
