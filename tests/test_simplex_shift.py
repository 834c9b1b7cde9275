"""The simplex shift of the maximum-likelihood correction ends after at most one
round per value, also where values lie within the rounding of the shift, and is
the sorted-values definition's."""
import subprocess

import numpy as np

from oracle import mlcorrect as ML
from paper_2303_10788_amd import build as B

# the kernel's sums: 256 strided partial sums, then a tree; the rounds taken (0: they did not end) and the shift
SOURCE = """
#include <cmath>
#include <cstdio>
#include "simplex.hpp"
int main() {
  unsigned long long n;
  while (std::fread(&n, 8, 1, stdin) == 1) {
    double *mu = new double[n], s[256];
    if (std::fread(mu, 8, n, stdin) != n) return 1;
    ccut::SimplexShift S{-INFINITY, n + 1};
    unsigned long long rounds = 0;
    for (bool more = true; more && rounds <= n + 1; ++rounds) {
      unsigned long long c = 0;
      for (int t = 0; t < 256; ++t) s[t] = 0.0;
      for (unsigned long long i = 0; i < n; ++i)
        if (mu[i] > S.tau) s[i % 256] += mu[i], ++c;
      for (int h = 128; h; h /= 2)
        for (int t = 0; t < h; ++t) s[t] += s[t + h];
      more = S.round(s[0], c);
      if (!more) break;
    }
    double r = rounds > n + 1 ? 0.0 : rounds + 1.0;
    std::fwrite(&r, 8, 1, stdout);
    std::fwrite(&S.tau, 8, 1, stdout);
    delete[] mu;
  }
}
"""


def _run(spectra, tmp_path):
    (tmp_path / "s.cpp").write_text(SOURCE)
    subprocess.run([B.hipcc(), "-no-hip-rt", "-x", "c++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", B.CSRC, "-I",
                    "/opt/rocm/include", str(tmp_path / "s.cpp"), "-o", str(tmp_path / "s")], check=True, capture_output=True)
    data = b"".join(np.uint64(len(m)).tobytes() + m.tobytes() for m in spectra)
    out = subprocess.run([str(tmp_path / "s")], input=data, capture_output=True, check=True, timeout=60).stdout
    return np.frombuffer(out).reshape(-1, 2)


def test_it_ends(tmp_path):
    rng = np.random.default_rng(0)
    spectra = []
    for _ in range(2000):  # physical states: a few eigenvalues, zeros to rounding
        n = int(2 ** rng.integers(2, 10))
        k = int(rng.integers(1, max(2, n // 2)))
        v = rng.random(k)
        spectra.append(rng.permutation(np.concatenate([v / v.sum(), rng.normal(size=n - k) * 1e-17])))
    spectra += [rng.normal(size=int(rng.integers(2, 600))) for _ in range(500)]
    spectra += [np.full(64, 1 / 64), np.zeros(16), np.array([np.nan, 0.5, 0.7]), np.full(4, np.nan), np.array([1e300, -1e300])]
    for mu, (rounds, tau) in zip(spectra, _run(spectra, tmp_path)):
        assert 1 <= rounds <= len(mu) + 1
        if np.isfinite(mu).all() and np.abs(mu).max() < 1e6:
            want = ML.simplex_projection(mu)
            assert np.abs(np.maximum(mu - tau, 0.0) - want).max() <= 1e-12 * max(1.0, np.abs(mu).max())
