"""Where the several-workgroup one-sided SVD keeps the columns that its workgroups exchange
(csrc/svd_columns.h), on the CPU: simulated workgroups perform the same rotations, and between
two exchanges they run in any order, one of them to its end before another begins.  Every
workgroup has to see the columns that rotations one after another give, bit for bit."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2607_23187_amd", "csrc")

PROGRAM = r"""
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>
#include "svd_columns.h"

struct Wg { unsigned ver[64] = {}; };

int main(int argc, char** argv) {
  const int n = atoi(argv[1]), m = atoi(argv[2]), G = atoi(argv[3]), rots = atoi(argv[4]);
  const bool one_copy = atoi(argv[5]);  // the planted mistake: both copies at one address
  const int ldc = (m + 1) & ~1, c = (n + G - 1) / G;
  std::mt19937_64 rng(1000 * n + G);
  std::uniform_real_distribution<double> u(-1.0, 1.0);
  std::vector<double> Y(je::svd_column_doubles(n, ldc), 0.0), ref((size_t)n * ldc, 0.0);
  for (int k = 0; k < n; ++k)
    for (int i = 0; i < m; ++i) ref[(size_t)k * ldc + i] = Y[je::svd_column_at(0, k, n, ldc) + i] = u(rng);
  std::vector<Wg> wg(G);
  long long wrong = 0;
  for (int r = 0; r < rots; ++r) {
    // columns that repeat from rotation to rotation as well as any others
    int p = (int)(rng() % n), q = (int)(rng() % n);
    if (r % 3 == 0) p = r % 2 ? 0 : n - 1;
    if (p == q) q = (p + 1) % n;
    const double cs = std::cos(u(rng)), sn = std::sqrt(1.0 - cs * cs);
    std::vector<int> order(G);
    for (int g = 0; g < G; ++g) order[g] = g;
    std::shuffle(order.begin(), order.end(), rng);
    const std::vector<double> rp(&ref[(size_t)p * ldc], &ref[(size_t)p * ldc] + m);
    const std::vector<double> rq(&ref[(size_t)q * ldc], &ref[(size_t)q * ldc] + m);
    for (int g : order) {
      unsigned* ver = wg[g].ver;
      auto version = [&](int k) { return ver[je::svd_version_lane(k)] & je::svd_version_bit(k); };
      const unsigned pv = version(p), qv = version(q);
      auto at = [&](unsigned v, int k) { return je::svd_column_at(one_copy ? 0u : v, k, n, ldc); };
      const double *gp = &Y[at(pv, p)], *gq = &Y[at(qv, q)];
      double *newp = &Y[at(!pv, p)], *newq = &Y[at(!qv, q)];
      ver[je::svd_version_lane(p)] ^= je::svd_version_bit(p);
      ver[je::svd_version_lane(q)] ^= je::svd_version_bit(q);
      std::vector<double> np(m), nq(m);
      for (int i = 0; i < m; ++i) {
        wrong += gp[i] != rp[i];
        wrong += gq[i] != rq[i];
        np[i] = cs * gp[i] + sn * gq[i];
        nq[i] = cs * gq[i] - sn * gp[i];
      }
      if (p / c == g) std::copy(np.begin(), np.end(), newp);
      if (q / c == g) std::copy(nq.begin(), nq.end(), newq);
    }
    for (int i = 0; i < m; ++i) {
      ref[(size_t)p * ldc + i] = cs * rp[i] + sn * rq[i];
      ref[(size_t)q * ldc + i] = cs * rq[i] - sn * rp[i];
    }
  }
  printf("%lld\n", wrong);
  return 0;
}
"""


@pytest.fixture(scope="module")
def simulate(tmp_path_factory):
    d = tmp_path_factory.mktemp("svd_columns")
    src, exe = str(d / "columns.cpp"), str(d / "columns")
    with open(src, "w") as f:
        f.write("#include <cmath>\n" + PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-ffp-contract=off", "-Wall", "-Werror",
                    "-I", CSRC, "-o", exe, src], check=True)

    def run(n, m, groups, rotations, one_copy=False):
        out = subprocess.run([exe, *map(str, (n, m, groups, rotations, int(one_copy)))],
                             check=True, capture_output=True, text=True)
        return int(out.stdout)

    return run


# 64 and more columns use a second bit of a word; two columns: every rotation takes both
@pytest.mark.parametrize("n,m,groups", [(2, 3, 1), (2, 7, 2), (64, 5, 16), (65, 5, 17),
                                        (129, 9, 32), (768, 2, 32), (2048, 1, 32)])
def test_no_workgroup_sees_a_later_column(simulate, n, m, groups):
    assert simulate(n, m, groups, 2000) == 0


def test_one_copy_is_seen(simulate):
    assert simulate(65, 5, 17, 2000, one_copy=True) > 0
