"""Rounding error of the D3Q19 MRT collision in 32 bits over many steps: the
header compiled for the CPU, periodic waves, against the same steps in 64
bits. The bar is the error of the plain form of the update, the products with
the moment matrix and its inverse, in the same precision: the collision may be
no further from 64 bits than that, after few steps and after many."""
import subprocess
from pathlib import Path

import pytest

CSRC = Path(__file__).resolve().parent.parent / "paper_1206_0389_amd" / "csrc"

MAIN = r"""
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <utility>
#include <vector>
#define __device__
#define __forceinline__ inline
#include "mrt.h"
using namespace lbm;
using std::vector;
constexpr int n = 16, N = n * n * n;

// f - M^-1 S M (f - f_eq) as it stands
template <typename R, int BASIS>
void plain(R (&f)[19], const MrtParams& p) {
  using T = MrtTables<BASIS>;
  R drho = 0, j[3] = {0, 0, 0}, d[19], pi[3][3] = {};
  for (int i = 0; i < 19; ++i) {
    drho += f[i];
    for (int c = 0; c < 3; ++c) j[c] += R(c_axis(i, c)) * f[i];
  }
  const R uu = j[0] * j[0] + j[1] * j[1] + j[2] * j[2];
  for (int i = 0; i < 19; ++i) {
    const R eu = R(cx(i)) * j[0] + R(cy(i)) * j[1] + R(cz(i)) * j[2];
    d[i] = f[i] - R(weight<19>(i)) * (drho + R(3) * eu + R(4.5) * eu * eu - R(1.5) * uu);
    for (int a = 0; a < 3; ++a)
      for (int b = 0; b < 3; ++b) pi[a][b] += R(c_axis(i, a) * c_axis(i, b)) * d[i];
  }
  R pi2 = 0;
  for (int a = 0; a < 3; ++a)
    for (int b = 0; b < 3; ++b) pi2 += pi[a][b] * pi[a][b];
  const R tau0 = R(p.tau0);
  const R tau = R(0.5) * (tau0 + std::sqrt(tau0 * tau0 + R(p.cs18) * std::sqrt(R(2) * pi2)));
  R dm[19];
  for (int k = 0; k < 19; ++k) {
    const int g = row_group(BASIS, k);
    dm[k] = 0;
    for (int i = 0; i < 19; ++i) dm[k] += R(T::M.a[k][i]) * d[i];
    dm[k] *= g == 0 ? R(0) : (g == 1 ? R(1) / tau : R(p.rates[g - 2]));
  }
  for (int i = 0; i < 19; ++i) {
    R c = 0;
    for (int k = 0; k < 19; ++k)
      if (row_group(BASIS, k) != 0 && is_nonzero(T::Minv.a[i][k])) c += R(T::Minv.a[i][k]) * dm[k];
    f[i] -= c;
  }
}

template <typename R, typename C>
void steps(vector<R>& f, int m, C collide) {
  vector<R> h(f.size());
  for (int t = 0; t < m; ++t) {
    for (int z = 0; z < n; ++z)
      for (int y = 0; y < n; ++y)
        for (int x = 0; x < n; ++x) {
          R g[19];
          for (int i = 0; i < 19; ++i)
            g[i] = f[i * N + (((z - cz(i) + n) % n) * n + (y - cy(i) + n) % n) * n + (x - cx(i) + n) % n];
          collide(g);
          for (int i = 0; i < 19; ++i) h[i * N + (z * n + y) * n + x] = g[i];
        }
    std::swap(f, h);
  }
}

// rms errors of populations and momentum
void error(const vector<float>& f, const vector<double>& r, double e[2]) {
  e[0] = e[1] = 0;
  for (int s = 0; s < N; ++s) {
    double j[3] = {0, 0, 0};
    for (int i = 0; i < 19; ++i) {
      const double d = f[i * N + s] - r[i * N + s];
      e[0] += d * d;
      for (int c = 0; c < 3; ++c) j[c] += c_axis(i, c) * d;
    }
    for (int c = 0; c < 3; ++c) e[1] += j[c] * j[c];
  }
  for (int k = 0; k < 2; ++k) e[k] = std::sqrt(e[k] / N);
}

template <int BASIS>
void run(const MrtParams& p, double drho, unsigned seed) {
  std::mt19937 gen(seed);
  double ph[9];
  for (double& v : ph) v = 6.283185307179586 * gen() / 4294967296.0;
  const double k = 6.283185307179586 / n, U = 0.02;
  vector<float> a(19 * N);
  for (int s = 0; s < N; ++s) {
    const int x = s % n, y = s / n % n, z = s / n / n;
    const double u[3] = {0.002 + U * std::sin(k * y + ph[0]) * std::cos(2 * k * z + ph[1]),
                         0.001 + U * std::sin(k * z + ph[2]) * std::cos(2 * k * x + ph[3]),
                         U * std::sin(k * x + ph[4]) * std::cos(2 * k * y + ph[5])};
    const double d = drho * (std::cos(k * x + ph[6]) + std::cos(2 * k * y + ph[7]) * std::cos(k * z + ph[8]));
    for (int i = 0; i < 19; ++i) {
      const double eu = cx(i) * u[0] + cy(i) * u[1] + cz(i) * u[2];
      a[i * N + s] = float(weight<19>(i) * (d + 3 * eu + 4.5 * eu * eu -
                                            1.5 * (u[0] * u[0] + u[1] * u[1] + u[2] * u[2])));
    }
  }
  vector<float> b = a;
  vector<double> r(a.begin(), a.end());
  int t = 0;
  for (int next : {6, 50, 300}) {
    const int m = next - t;
    t = next;
    steps(a, m, [&](float(&g)[19]) { mrt_collide<float, BASIS>(g, p); });
    steps(b, m, [&](float(&g)[19]) { plain<float, BASIS>(g, p); });
    steps(r, m, [&](double(&g)[19]) { plain<double, BASIS>(g, p); });
    double ea[2], eb[2];
    error(a, r, ea);
    error(b, r, eb);
    std::printf("%d %.17g %.17g %.17g %.17g\n", t, ea[0], eb[0], ea[1], eb[1]);
  }
}

int main(int, char** v) {
  MrtParams p{};
  p.tau0 = 3 * std::atof(v[2]) + 0.5;
  const double cs = std::atof(v[3]);
  p.cs18 = 18 * cs * cs;
  for (int k = 0; k < 5; ++k) p.rates[k] = std::atof(v[6 + k]);
  if (std::atoi(v[1]) == 0) run<0>(p, std::atof(v[4]), std::atoi(v[5]));
  else run<1>(p, std::atof(v[4]), std::atoi(v[5]));
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("rounding")
    (d / "r.cpp").write_text(MAIN)
    subprocess.run(["g++", "-O2", "-march=native", "-ffp-contract=fast", "-std=c++20", "-w",
                    "-I", str(CSRC), "-o", str(d / "r"), str(d / "r.cpp")], check=True)
    return d / "r"


@pytest.mark.parametrize("basis,nu,cs,drho,rates", [
    (0, 1e-3, 0.1, 0.0005, (1, 1, 1, 1, 1)),
    (0, 1e-3, 0.0, 0.02, (1.1, 0.9, 1.3, 0.7, 1)),
    (0, 2e-2, 0.1, 0.0005, (1, 1, 1, 1, 1)),
    (0, 1.0, 0.1, 0.0005, (1, 1, 1, 1, 1)),
    (1, 1e-3, 0.1, 0.0005, (1.19, 1.4, 1.2, 1.4, 1.98)),
    (1, 1e-3, 0.1, 0.02, (1.19, 1.4, 1.2, 1.4, 1.98)),
])
def test_error_no_larger_than_the_plain_form(program, basis, nu, cs, drho, rates):
    args = [basis, nu, cs, drho, 1, *rates]
    out = subprocess.run([str(program)] + [str(a) for a in args], check=True,
                         capture_output=True, text=True).stdout
    for line in out.splitlines():
        t, f, f_plain, j, j_plain = (float(v) for v in line.split())
        assert f <= f_plain, (t, "populations", f / f_plain)
        assert j <= j_plain, (t, "momentum", j / j_plain)
