"""The rules that pick a launch while nobody set its shape: compiled here from
the library's header and asked on the CPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2411_15001_amd", "csrc")

# reads "precision limiters bnd n nx ny [nx ny ...]", prints "rows height groups"
PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "vlbm_internal.h"
int main() {
  int prec, lims, bnd, n;
  while (scanf("%d %d %d %d", &prec, &lims, &bnd, &n) == 4) {
    vlbm::Scheme sc{};
    sc.limiters = lims;
    sc.order = 2;
    std::vector<int> nx(n), ny(n);
    vlbm::Extent x;
    for (int i = 0; i < n; ++i) {
      if (scanf("%d %d", &nx[i], &ny[i]) != 2) return 1;
      x.add(nx[i], ny[i]);
    }
    auto strips = [&](int h) {
      long long k = 0;
      for (int i = 0; i < n; ++i) k += (nx[i] + 63ll) / 64 * ((ny[i] + h - 1ll) / h);
      return k;
    };
    const bool rows = vlbm::use_rows(x, bnd != 0, prec, sc);
    const int h = rows ? vlbm::kRowsPerGroup : MARCH_ROWS;
    const long long groups = rows ? strips(h) : (strips(h) + 3) / 4;
    printf("%d %d %lld\n", rows ? 1 : 0, h, (groups + 7) / 8 * 8);
  }
}
""".replace("MARCH_ROWS", "vlbm::march_rows(prec, (lims & 6) != 0, strips)")

PP, LMP, RLMP = 9, 11, 13


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, exe = str(d / "rules.cpp"), str(d / "rules")
    with open(src, "w") as f:
        f.write(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC,
                    "-I" + os.path.join(ROOT, "include"), src, "-o", exe], check=True)

    def run(queries):
        """[(precision, limiters, bnd, [(nx, ny), ...])] -> [(rows, height, groups)]"""
        text = "\n".join(" ".join(str(v) for v in (p, l, int(b), len(s), *[k for xy in s for k in xy]))
                         for p, l, b, s in queries)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(int(v) for v in line.split()) for line in out.splitlines()]

    return run


def test_every_accepted_grid_fits_a_launch(ask):
    """A launch holds fewer than 2^32 threads.  Strips of 64 rows stay below for
    every grid of fewer than 2^32 cells with sides below 2^30; the choice must
    not exceed them on grids of a few columns and many rows."""
    queries = []
    for nx in (1, 2, 3, 4, 5, 8, 16, 63, 64, 65, 128, 130, 1000, 65536, 1 << 26, (1 << 30) - 1):
        top = min((1 << 30) - 1, ((1 << 32) - 1) // nx)
        for ny in sorted({1, 4, top // 64, top // 16, top // 8, top // 4, top // 2, top - 3, top,
                          min(top, (1 << 26) - 32), min(top, 1 << 26), min(top, (1 << 26) + 1)} - {0}):
            for prec in (0, 1):
                for lims in (0, PP, LMP, RLMP):
                    queries += [(prec, lims, bnd, [(nx, ny)]) for bnd in (False, True)]
    queries += [(prec, LMP, True, [(1, 1 << 25)] * 3) for prec in (0, 1)]
    for q, (rows, h, groups) in zip(queries, ask(queries)):
        assert 0 < groups * 256 < 1 << 32, q
        assert h in (4, 8, 12, 16, 24, 32, 48, 64), q
