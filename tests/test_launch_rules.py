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
""".replace("MARCH_ROWS", "vlbm::march_rows(x, bnd != 0, prec, (lims & 6) != 0, strips)")

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


# us a step on an MI355X at strips of 4 .. 64 rows: (precision, limiters, sizes)
HEIGHTS = (4, 8, 12, 16, 24, 32, 48, 64)
MEASURED = [
    ((0, PP, [(1, 1000000)]), (3914.0, 3049.3, 2760.5, 2622.1, 2472.1, 2409.6, 2368.1, 2362.1)),
    ((1, PP, [(1, 1000000)]), (2369.2, 1880.6, 1718.8, 1640.3, 1559.2, 1532.3, 1518.6, 1527.7)),
    ((1, LMP, [(1, 1000000)]), (3259.3, 2385.0, 2099.0, 1969.5, 1821.5, 1769.1, 1736.0, 1737.1)),
    ((1, PP, [(4, 1000000)]), (2420.8, 1880.6, 1751.9, 1681.3, 1590.2, 1561.9, 1550.6, 1558.4)),
    ((1, PP, [(20, 200000)]), (508.9, 413.2, 386.9, 374.9, 371.9, 378.3, 403.2, 418.1)),
    ((1, PP, [(40, 200000)]), (538.9, 456.7, 430.8, 421.5, 424.6, 433.3, 460.1, 462.0)),
    ((0, LMP, [(70, 100000)]), (1446.1, 1073.8, 966.6, 905.2, 851.8, 830.7, 839.7, 863.8)),
    ((0, PP, [(100000, 20)]), (194.1, 186.1, 192.3, 229.1, 163.3, 162.8, 162.9, 163.1)),
    ((1, LMP, [(100000, 20)]), (123.7, 115.8, 118.6, 143.9, 93.7, 93.8, 93.7, 93.7)),
    ((1, PP, [(32, 32)] * 3000), (261.9, 217.4, 215.5, 194.4, 222.0, 200.0, 201.8, 202.2)),
    ((1, PP, [(16, 16)] * 5000), (219.7, 177.5, 202.3, 160.8, 161.0, 160.6, 160.3, 160.3)),
    ((1, PP, [(1, 2048)] * 64), (316.0, 252.5, 238.4, 224.1, 238.2, 215.5, 251.4, 214.5)),
    ((1, LMP, [(2000, 20)] * 60), (151.6, 133.1, 128.2, 139.7, 105.1, 105.2, 105.0, 104.7)),
    ((0, PP, [(256, 256)] * 200), (971.5, 849.1, 830.0, 840.9, 855.4, 882.1, 840.5, 926.5)),
    ((1, LMP, [(256, 256)] * 200), (699.3, 550.8, 521.7, 493.1, 480.3, 489.8, 505.5, 517.1)),
]


@pytest.mark.parametrize("case", MEASURED, ids=lambda c: "p%d_l%d_%dx%dx%d" % (c[0][0], c[0][1], len(c[0][2]), *c[0][2][0]))
def test_strip_height_of_narrow_and_short_instances(case, ask):
    """Narrow instances, whose strips leave lanes idle, and instances lower than
    a strip: the height picked is within 8% of the best that was measured (the
    tallest strips that fill one round, the shape that lbm_get_launch reports,
    are up to 54% slower than the best on these)."""
    (prec, lims, sizes), times = case
    rows, h, _ = ask([(prec, lims, False, sizes)])[0]
    assert rows == 0
    assert times[HEIGHTS.index(h)] <= 1.08 * min(times), h


# us a step on an MI355X with descriptions on four sides (walls and zero
# gradient): (precision, limiters, sizes), the row kernel, marches by strip height
DESCRIBED = [
    ((0, LMP, [(1000, 750)]), 73.7, {8: 161.6, 12: 113.7, 16: 134.4, 24: 178.8, 32: 224.2, 48: 317.4, 64: 414.9}),
    ((1, LMP, [(1000, 750)]), 58.7, {8: 97.4, 12: 105.3, 16: 124.2, 24: 164.5, 32: 206.7, 48: 290.5, 64: 391.6}),
    ((0, LMP, [(1800, 1800)]), 347.4, {8: 501.4, 12: 485.5, 16: 489.9, 24: 514.2, 32: 447.3, 48: 628.8, 64: 427.4}),
    ((1, LMP, [(2500, 2500)]), 423.5, {8: 477.9, 12: 457.7, 16: 460.1, 24: 476.2, 32: 481.7, 48: 581.7, 64: 516.9}),
    ((0, LMP, [(4096, 4096)]), 1697.1, {8: 2321.9, 12: 2150.5, 16: 2012.1, 24: 1985.9, 32: 1854.1, 48: 1975.2, 64: 1774.1}),
    ((1, LMP, [(4096, 4096)]), 1004.3, {8: 1114.0, 12: 1035.7, 16: 962.5, 24: 945.9, 32: 890.9, 48: 957.9, 64: 857.7}),
    ((0, LMP, [(8192, 8192)]), 6583.6, {8: 9173.8, 12: 8293.3, 16: 7869.0, 24: 7448.3, 32: 7227.7, 48: 7289.7, 64: 6872.9}),
    ((1, LMP, [(8192, 8192)]), 3824.6, {8: 4338.0, 12: 3979.6, 16: 3805.1, 24: 3604.7, 32: 3550.4, 48: 3459.2, 64: 3433.7}),
    ((0, PP, [(8192, 8192)]), 5380.6, {8: 6869.0, 12: 6281.3, 16: 6179.6, 24: 5855.0, 32: 5845.2, 48: 5748.5, 64: 5659.8}),
    ((1, PP, [(6000, 6000)]), 1930.5, {8: 1989.9, 12: 1852.2, 16: 1777.2, 24: 1724.8, 32: 1718.8, 48: 1704.9, 64: 1739.1}),
    ((1, PP, [(130, 66666)]), 605.9, {8: 764.0, 12: 729.9, 16: 724.1, 24: 737.6, 32: 761.6, 48: 826.5, 64: 824.0}),
    ((0, LMP, [(64, 4000)]), 44.2, {4: 61.4, 8: 77.6, 12: 97.0, 16: 118.4, 24: 165.5, 32: 211.5, 48: 299.8, 64: 387.6}),
    ((1, LMP, [(64, 4000)]), 32.7, {4: 52.6, 8: 64.7, 12: 81.2, 16: 99.4, 24: 143.3, 32: 182.9, 48: 259.9, 64: 337.7}),
    ((1, LMP, [(64, 12000)]), 74.4, {8: 82.8, 12: 86.8, 16: 102.3, 24: 134.2, 32: 167.6, 48: 248.6, 64: 339.8}),
    ((0, LMP, [(64, 25000)]), 266.0, {8: 298.7, 12: 300.8, 16: 258.7, 24: 349.0, 32: 236.8, 48: 324.2, 64: 411.3}),
    ((1, LMP, [(64, 25000)]), 148.3, {8: 148.7, 12: 166.5, 16: 127.0, 24: 171.9, 32: 172.5, 48: 238.9, 64: 318.4}),
    ((0, LMP, [(128, 50000)]), 1021.3, {8: 936.8, 12: 893.4, 16: 874.0, 24: 870.9, 32: 887.8, 48: 957.4, 64: 845.3}),
    ((1, LMP, [(128, 50000)]), 597.7, {8: 479.1, 12: 451.1, 16: 452.7, 24: 477.3, 32: 450.6, 48: 573.1, 64: 426.7}),
    ((0, LMP, [(130, 8333)]), 228.0, {8: 304.5, 12: 302.2, 16: 254.2, 24: 349.3, 32: 236.6, 48: 331.1, 64: 424.8}),
    ((0, LMP, [(130, 66666)]), 1808.6, {8: 1859.9, 12: 1666.9, 16: 1580.6, 24: 1520.0, 32: 1514.8, 48: 1556.0, 64: 1627.1}),
    ((1, LMP, [(260, 5000)]), 119.6, {8: 162.4, 12: 178.8, 16: 149.2, 24: 196.5, 32: 210.6, 48: 296.0, 64: 389.1}),
    ((0, LMP, [(64, 64)] * 256), 175.5, {8: 163.2, 12: 202.6, 16: 143.6, 24: 182.9, 32: 224.2, 48: 297.3, 64: 404.1}),
    ((1, LMP, [(64, 64)] * 256), 106.6, {8: 86.8, 12: 105.6, 16: 109.0, 24: 141.2, 32: 173.6, 48: 242.0, 64: 310.2}),
    ((0, LMP, [(128, 128)] * 128), 320.7, {4: 397.1, 8: 310.5, 12: 306.9, 16: 270.2, 24: 348.0, 32: 245.8, 48: 328.2, 64: 411.7}),
    ((1, LMP, [(128, 128)] * 128), 196.8, {4: 210.4, 8: 171.6, 12: 183.6, 16: 145.6, 24: 191.0, 32: 191.4, 48: 259.0, 64: 330.2}),
    ((0, LMP, [(64, 64)] * 64), 42.0, {4: 61.4, 8: 77.4, 12: 95.7, 16: 116.4, 24: 157.8, 32: 202.8, 48: 276.5, 64: 389.2}),
]


@pytest.mark.parametrize("case", DESCRIBED, ids=lambda c: "p%d_l%d_%dx%dx%d" % (c[0][0], c[0][1], len(c[0][2]), *c[0][2][0]))
def test_kernel_of_described_boundaries(case, ask):
    """With boundary descriptions: the kernel and strip height picked are within
    5% of the fastest that was measured."""
    (prec, lims, sizes), row_kernel, marches = case
    rows, h, _ = ask([(prec, lims, True, sizes)])[0]
    took = row_kernel if rows else marches[h]
    assert took <= 1.05 * min(row_kernel, *marches.values()), (rows, h)
