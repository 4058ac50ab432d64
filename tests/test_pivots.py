"""The elimination that counts eigenvalues (csrc/pivots.h), on the host: exact zero pivots among others of ordinary size.  The compiled program
takes four pivots at a time and the rest as products of rank four, as the kernel does."""
import os
import subprocess

import numpy as np
import pytest

from paper_2605_02218_amd import build as B

PROGRAM = r"""
#include <stdio.h>
#include <vector>
#include "pivots.h"
int main() {
  int n;
  double x;
  while (fread(&n, sizeof n, 1, stdin) == 1 && fread(&x, sizeof x, 1, stdin) == 1) {
    std::vector<double> t((size_t)n * n);
    if (fread(t.data(), 8, t.size(), stdin) != t.size()) return 1;
    for (int i = 0; i < n; ++i) t[i * n + i] -= x;
    int negative = 0;
    for (int s = 0; s < n; s += 4) {
      auto at = [&](int i, int j) { return t[(s + i) * n + s + j]; };
      const covspec::CountedBlock f = covspec::count_block(at(0, 0), at(1, 0), at(1, 1), at(2, 0), at(2, 1), at(2, 2), at(3, 0), at(3, 1), at(3, 2), at(3, 3),
                                                           [](double p) { return 1.0 / p; }, negative);
      const double inv[4][4] = {{1, 0, 0, 0}, {f.n10, 1, 0, 0}, {f.n20, f.n21, 1, 0}, {f.n30, f.n31, f.n32, 1}}, r[4] = {f.r0, f.r1, f.r2, f.r3};
      std::vector<double> u(4 * n, 0.0);
      for (int k = 0; k < 4; ++k)
        for (int j = s + 4; j < n; ++j)
          for (int i = 0; i <= k; ++i) u[k * n + j] = fma(inv[k][i], t[(s + i) * n + j], u[k * n + j]);
      for (int i = s + 4; i < n; ++i)
        for (int j = s + 4; j < n; ++j)
          for (int k = 0; k < 4; ++k) t[i * n + j] = fma(-r[k] * u[k * n + i], u[k * n + j], t[i * n + j]);
    }
    printf("%d\n", n - negative);
  }
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("pivots")
    (d / "count.hip").write_text(PROGRAM)
    subprocess.run([B._hipcc(), "--offload-arch=gfx950", "-O2", "-std=c++17", "-ffp-contract=off", "-I", B.CSRC, str(d / "count.hip"), "-o", str(d / "count")],
                   check=True, capture_output=True)
    return str(d / "count")


def counts(program, matrices):
    data = b"".join(np.int32(len(a)).tobytes() + np.float64(x).tobytes() + np.ascontiguousarray(a, np.float64).tobytes() for a, x in matrices)
    return [int(v) for v in subprocess.run([program], input=data, check=True, capture_output=True, timeout=60).stdout.split()]


def gram(n, rank, seed):
    """Positive semidefinite, the largest diagonal entry 1, so that no entry exceeds it."""
    z = np.random.default_rng(seed).standard_normal((n, rank))
    a = z @ z.T
    return a / a.diagonal().max()


def cases():
    out = {}
    for n, rank in ((64, 80), (64, 20), (128, 160), (128, 40)):
        a = gram(n, rank, n + rank)
        out["ordinary-%d-%d" % (n, rank)] = (a, 0.1)
        out["first-%d-%d" % (n, rank)] = (a, a[0, 0])
        c = a / np.sqrt(np.outer(a.diagonal(), a.diagonal()))
        np.fill_diagonal(c, 1.0)
        out["all-diagonals-%d-%d" % (n, rank)] = (c, 1.0)            # the first pivot is zero, the others are not
    for k in (1, 2, 3, 4, 5, 31, 62):                                # a zero pivot at place k, strongly coupled to those behind it
        a = np.zeros((64, 64))
        np.fill_diagonal(a, np.linspace(0.9, 0.2, 64))
        a[k:, k:] = gram(64 - k, 80, k)
        out["place-%d" % k] = (a, a[k, k])
    a = np.kron(np.eye(32), np.array([[0.5, 0.3], [0.3, 0.5]]))      # every other pivot
    out["pairs"] = (a, 0.5)
    return out


@pytest.mark.parametrize("name", list(cases()))
def test_count_with_exact_zero_pivots(program, name):
    a, x = cases()[name]
    assert os.path.exists(program)
    eig = np.linalg.eigvalsh(a)
    got = counts(program, [(a, x)])[0]
    # a pivot that is not there is a matrix 1e-8 away, and the rest is good to 1e-8 behind it
    tol = 4e-8 * len(a) ** 0.5
    assert (eig >= x + tol).sum() <= got <= (eig >= x - tol).sum(), (name, got, (eig >= x).sum())
