"""Which elite row an element of the refit's staged rows belongs to: the
division by the number of coefficients (one for the selection hook, up to 48
for a problem) must be exact over every index that is staged, or the refit
reads outside its samples."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2309_08235_amd", "csrc")

PROGRAM = """
#include <cstdio>
#include "quotient.h"
int main() {
  int bad = 0;
  for (uint32_t d = 1; d <= 48; ++d) {
    const uint32_t inv = priest::inverse_of(d);
    for (uint32_t i = 0; i <= 12288; ++i)
      if (priest::quotient(i, inv) != i / d) {
        if (bad++ < 5) std::printf("%u / %u: %u\\n", i, d, priest::quotient(i, inv));
      }
  }
  return bad != 0;
}
"""


def test_row_of_every_staged_element(tmp_path):
    src, exe = tmp_path / "rows.cpp", str(tmp_path / "rows")
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(src), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
