"""The QR steps whose rotations the PCA fit sends to the GPU (csrc/host_linalg.hpp: tridiag_eigen), built
with g++ alone: the rotations of each step are consecutive within the step's bounds, and applied in
order to the rows of the identity they give LAPACK's eigenpairs."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
DRIVER = r"""
#include <stdio.h>
#include "host_linalg.hpp"
int main() {
  int n, steps;
  if (scanf("%d %d", &n, &steps) != 2) return 1;
  std::vector<double> d(n), e(n, 0.0), V((size_t)n * n, 0.0);
  for (double& x : d) if (scanf("%lf", &x) != 1) return 1;
  for (int i = 0; i + 1 < n; ++i) if (scanf("%lf", &e[i]) != 1) return 1;
  for (int i = 0; i < n; ++i) V[(size_t)i * n + i] = 1.0;
  int next = 0, end = 0;
  bool in_order = true;
  const bool ok = hmoe::tridiag_eigen(
      d, e, n, [&](int lo, int hi) { in_order &= next == end; next = lo; end = hi; },
      [&](int k, double c, double s) {
        in_order &= k == next++ && k < end && k + 1 < n;
        for (int j = 0; j < n; ++j) {
          const double a = V[(size_t)k * n + j], b = V[(size_t)(k + 1) * n + j];
          V[(size_t)k * n + j] = c * a - s * b;
          V[(size_t)(k + 1) * n + j] = s * a + c * b;
        }
      }, steps);
  printf("%d %d\n", (int)ok, (int)in_order);
  for (double x : d) printf("%.17g ", x);
  for (double x : V) printf("%.17g ", x);
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("tri")
    (d / "driver.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-O2", "-std=c++17", "-pthread", "-I", os.path.join(ROOT, "paper_1704_06363_amd", "csrc"),
                    str(d / "driver.cpp"), "-o", str(d / "driver")], check=True)
    return str(d / "driver")


def _run(exe, d, e, steps=-1):
    text = "%d %d\n" % (len(d), steps) + " ".join("%.17g" % x for x in [*d, *e])
    out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split()
    n = len(d)
    v = np.array(out[2:], dtype=np.float64)
    return out[0] == "1", out[1] == "1", v[:n], v[n:].reshape(n, n)


@pytest.mark.parametrize("n", [1, 2, 3, 17, 256])
@pytest.mark.parametrize("kind", ["random", "diagonal", "clustered", "split"])
def test_matches_lapack(driver, n, kind):
    rs = np.random.default_rng(n)
    d, e = rs.standard_normal(n) * 5, rs.standard_normal(max(n - 1, 0))
    if kind == "diagonal":
        e[:] = 0.0
    elif kind == "clustered":
        d, e = 1.0 + 1e-9 * np.arange(n), e * 1e-9
    elif kind == "split" and n > 2:
        e[n // 2] = 0.0
    ok, in_order, w, V = _run(driver, d, e)
    A = np.diag(d) + np.diag(e, 1) + np.diag(e, -1) if n > 1 else np.diag(d)
    scale = np.abs(A).max()
    assert ok and in_order
    assert np.abs(np.sort(w) - np.linalg.eigvalsh(A)).max() <= 1e-12 * scale
    assert np.abs(V @ V.T - np.eye(n)).max() <= 1e-12
    assert np.abs(A @ V.T - V.T * w).max() <= 1e-12 * scale


def test_reports_non_convergence(driver):
    rs = np.random.default_rng(1)
    ok, _, _, _ = _run(driver, rs.standard_normal(64), rs.standard_normal(63), steps=1)
    assert not ok
