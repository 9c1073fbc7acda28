"""The scalar parts of the direct eigensolver (eig.hip) on matrices whose
couplings lie far below the others: the reflector, the deflation and the
secular roots are taken from the source, compiled for the host, and run through
a whole tridiagonalisation and divide and conquer.

A Gram of unit trace may hold entries of any size down to the smallest double.
Their squares underflow (a norm of zero over a vector that isn't, or one with a
few bits left), and differences of eigenvalues near 1e-308 have no reciprocal.
Either made the unitary not a number, or not unitary; the ranks that follow are
then no permutation, so memory past a work array could be written."""
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

import workloads as W
from paper_1703_00387_amd import build as B

STUB = r"""
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <vector>
#define __device__
#define __forceinline__ inline
struct double2 { double x, y; };
static double2 make_double2(double x, double y) { return {x, y}; }
static double2 cmul(double2 a, double2 b) { return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x}; }
static double __builtin_amdgcn_sqrt(double x) { return std::sqrt(x); }
static double rsqrt_nr(double x) {   // an estimate and two steps, as on the device
  double y = 1.0 / std::sqrt(x);
  const double h = 0.5 * x;
  for (int i = 0; i < 2; ++i) y = std::fma(y, std::fma(-h * y, y, 0.5), y);
  return y;
}
static double rcp_nr(double x) {
  double y = 1.0 / x;
  for (int i = 0; i < 2; ++i) y = std::fma(y, std::fma(-x, y, 1.0), y);
  return y;
}
template <int NL> double lanes_sum(double a) { return a; }
constexpr double kEps = 2.220446049250313e-16;
using namespace std;
"""

MAIN = r"""
int main(int argc, char** argv) {   // m, then m x m complex entries of the lower triangle's Hermitian matrix on stdin
  const int m = atoi(argv[1]);
  vector<double2> A(m * m), Q(m * m);
  for (auto& a : A) if (scanf("%lf %lf", &a.x, &a.y) != 2) return 1;
  for (int i = 0; i < m; ++i) for (int j = 0; j < m; ++j) Q[i * m + j] = {i == j ? 1.0 : 0.0, 0.0};
  vector<double> d(m), e(m, 0.0);
  for (int k = 0; k + 1 < m; ++k) {
    double xn2 = 0.0;
    for (int i = k + 2; i < m; ++i) xn2 += A[i * m + k].x * A[i * m + k].x + A[i * m + k].y * A[i * m + k].y;
    double beta;
    double2 tau, scl;
    reflector(A[(k + 1) * m + k], xn2, beta, tau, scl);
    d[k] = A[k * m + k].x;
    e[k] = beta;
    vector<double2> v(m, double2{0.0, 0.0}), y(m, double2{0.0, 0.0});
    v[k + 1] = {1.0, 0.0};
    for (int i = k + 2; i < m; ++i) v[i] = cmul(A[i * m + k], scl);
    // A <- H^dag A H and Q <- Q H on the rows and columns past k, H = I - tau v v^dag
    for (int i = k + 1; i < m; ++i)
      for (int j = k + 1; j < m; ++j) { const double2 t = cmul(A[i * m + j], v[j]); y[i].x += t.x; y[i].y += t.y; }
    double dot = 0.0;
    for (int i = k + 1; i < m; ++i) dot += v[i].x * y[i].x + v[i].y * y[i].y;
    const double hv = 0.5 * (tau.x * tau.x + tau.y * tau.y) * dot;
    vector<double2> w(m, double2{0.0, 0.0});
    for (int i = k + 1; i < m; ++i) { w[i] = cmul(tau, y[i]); w[i].x -= hv * v[i].x; w[i].y -= hv * v[i].y; }
    for (int i = k + 1; i < m; ++i)
      for (int j = k + 1; j < m; ++j) {
        const double2 p = cmul(v[i], {w[j].x, -w[j].y}), r = cmul(w[i], {v[j].x, -v[j].y});
        A[i * m + j].x -= p.x + r.x;
        A[i * m + j].y -= p.y + r.y;
      }
    for (int i = 0; i < m; ++i) {
      double2 s = {0.0, 0.0};
      for (int j = k + 1; j < m; ++j) { const double2 t = cmul(Q[i * m + j], v[j]); s.x += t.x; s.y += t.y; }
      s = cmul(s, tau);
      for (int j = k + 1; j < m; ++j) { const double2 t = cmul(s, {v[j].x, -v[j].y}); Q[i * m + j].x -= t.x; Q[i * m + j].y -= t.y; }
    }
  }
  d[m - 1] = A[(m - 1) * m + m - 1].x;
  // divide and conquer, torn at every index, merges of 1 + 1, 2 + 2, ...
  vector<double> D(m), Z(m * m, 0.0);
  for (int i = 0; i < m; ++i) {
    D[i] = in_range(d[i]) - (i > 0 ? fabs(e[i - 1]) : 0.0) - (i + 1 < m ? fabs(e[i]) : 0.0);
    Z[i * m + i] = 1.0;
  }
  for (int h = 1; h < m; h *= 2)
    for (int base = 0; base + h < m; base += 2 * h) {
      const int mid = base + h, s = min(base + 2 * h, m) - base;
      const double rho = 2.0 * fabs(e[mid - 1]), sg = e[mid - 1] < 0.0 ? -1.0 : 1.0;
      vector<int> pm(s);
      for (int i = 0; i < s; ++i) pm[i] = base + i;
      stable_sort(pm.begin(), pm.end(), [&](int a, int b) { return D[a] < D[b]; });
      vector<double> ds(s), zs(s), dv(s), rc(s), rs(s);
      vector<int32_t> kr(s), dr(s), ra(s), rb(s);
      for (int i = 0; i < s; ++i) {
        ds[i] = D[pm[i]];
        zs[i] = (pm[i] < mid ? Z[(mid - 1) * m + pm[i]] : sg * Z[mid * m + pm[i]]) * 0.70710678118654752440;
      }
      const double tol = kEps * fmax(fmax(fabs(ds[0]), fabs(ds[s - 1])), rho);
      int nr;
      const int K = dc_deflate(ds.data(), zs.data(), s, rho, tol, kr.data(), dr.data(), dv.data(), ra.data(), rb.data(),
                               rc.data(), rs.data(), nr);
      vector<double> dk(K), zk(K), et(K), lam(s), U(s * s, 0.0);
      vector<int> og(K);
      for (int i = 0; i < K; ++i) { dk[i] = ds[kr[i]]; zk[i] = zs[kr[i]]; }
      for (int i = 0; i < K; ++i) dc_secular<1, 0>(dk.data(), zk.data(), K, i, rho, 0, og[i], et[i]);
      vector<double> zh(K);
      for (int j = 0; j < K; ++j) {
        double p = 1.0;
        for (int i = 0; i < K; ++i) {
          const double num = (dk[og[i]] - dk[j]) + et[i];
          p *= i == j ? num : num * rcp_nr(dk[i] - dk[j]);
        }
        zh[j] = copysign(sqrt(fabs(p)), zk[j]);
      }
      for (int i = 0; i < K; ++i) {
        double n2 = 0.0;
        for (int t = 0; t < K; ++t) {
          const double x = zh[t] * rcp_nr((dk[t] - dk[og[i]]) - et[i]);
          n2 += x * x;
          U[kr[t] * s + i] = x;
        }
        for (int t = 0; t < K; ++t) U[kr[t] * s + i] *= 1.0 / sqrt(n2);
        lam[i] = dk[og[i]] + et[i];
      }
      for (int i = K; i < s; ++i) { U[dr[i - K] * s + i] = 1.0; lam[i] = dv[i - K]; }
      for (int t = nr - 1; t >= 0; --t)
        for (int i = 0; i < s; ++i) {
          const double x = U[ra[t] * s + i], y = U[rb[t] * s + i];
          U[ra[t] * s + i] = rc[t] * x - rs[t] * y;
          U[rb[t] * s + i] = rs[t] * x + rc[t] * y;
        }
      for (int r = base; r < base + s; ++r) {
        vector<double> row(s, 0.0);
        for (int t = 0; t < s; ++t)
          for (int i = 0; i < s; ++i) row[i] += Z[r * m + pm[t]] * U[t * s + i];
        for (int i = 0; i < s; ++i) Z[r * m + base + i] = row[i];
      }
      for (int i = 0; i < s; ++i) D[base + i] = lam[i];
    }
  for (int i = 0; i < m; ++i)
    for (int j = 0; j < m; ++j) {
      double2 x = {0.0, 0.0};
      for (int t = 0; t < m; ++t) { x.x += Q[i * m + t].x * Z[t * m + j]; x.y += Q[i * m + t].y * Z[t * m + j]; }
      printf("%.17g %.17g\n", x.x, x.y);
    }
  for (int i = 0; i < m; ++i) printf("%.17g 0\n", D[i]);
}
"""


def _function(text, head):
    """The function of `text` whose declaration holds `head`, with its template line."""
    at = text.index(head)
    start = text.rindex("\n\n", 0, at)
    depth, end = 0, text.index("{", at)
    while True:
        depth += {"{": 1, "}": -1}.get(text[end], 0)
        end += 1
        if depth == 0:
            return text[start:end] + "\n"


@pytest.fixture(scope="module")
def solver(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not installed")
    text = open(os.path.join(B.CSRC, "eig.hip")).read()
    const = "".join(re.findall(r"^constexpr double kTiny.*?;.*$\n", text, re.M))
    parts = [_function(text, h) for h in ("void reflector(", "int dc_deflate(", "void dc_secular(")]
    parts.append(_function(text, "double in_range(") if "double in_range(" in text
                 else "static double in_range(double x) { return x; }\n")
    d = tmp_path_factory.mktemp("eig")
    src = d / "s.cpp"
    src.write_text(STUB + const + "".join(parts) + MAIN)
    subprocess.run(["g++", "-O1", "-ffp-contract=off", "-std=c++17", "-o", str(d / "s"), str(src)], check=True)

    def run(G):
        m = len(G)
        inp = "\n".join(f"{float(x.real)!r} {float(x.imag)!r}" for x in G.ravel())
        r = subprocess.run([str(d / "s"), str(m)], input=inp, capture_output=True, text=True, check=True)
        v = np.array([[float(t) for t in line.split()] for line in r.stdout.splitlines()])
        return (v[:m * m, 0] + 1j * v[:m * m, 1]).reshape(m, m), v[m * m:, 0]
    return run


def tiny_cases(m, rng):
    """Rows X whose Gram has entries at, around and under the smallest normal double."""
    c = rng.normal(size=(m, m)) + 1j * rng.normal(size=(m, m))
    s = np.geomspace(1.0, 1e-3, m)
    for e in (1e-60, 1e-100, 1e-110, 1e-140, 1e-155, 1e-158, 1e-162, 1e-170, 1e-250, 1e-308):
        yield f"couplings {e:g}", np.diag(s) + e * c
    yield "rows to 1e-150", c * np.geomspace(1.0, 1e-150, m)[:, None]
    yield "columns to 1e-150", c * np.geomspace(1.0, 1e-150, m)[None, :]
    yield "half of the rows 1e-154", c * np.where(np.arange(m) < m // 2, 1.0, 1e-154)[:, None]
    yield "every other row 1e-158", c * np.where(np.arange(m) % 2 == 0, 1.0, 1e-158)[:, None]
    k = np.where(np.arange(m) % 3 == 0, 1.0, 1e-100)
    yield "thirds at 1e-100 and 1e-120", c * (k * np.where(np.arange(m) % 3 == 2, 1e-20, 1.0))[:, None]


@pytest.mark.parametrize("m", [2, 5, 24, 40])
def test_unitary_whatever_the_range(solver, m):
    """The vectors are unitary and diagonalise G: to 1e-12 of |G|, the sum of some m^2 roundings with room."""
    for name, X in tiny_cases(m, np.random.default_rng(m)):
        X = X / np.linalg.norm(X)
        G = X @ X.conj().T
        G /= np.trace(G).real
        U, lam = solver(G)
        assert np.isfinite(U).all() and np.isfinite(lam).all(), name
        assert np.abs(U.conj().T @ U - np.eye(m)).max() <= 1e-12, name
        assert np.abs(U.conj().T @ G @ U - np.diag(lam)).max() <= 1e-12, name


def equal_cases(m, rng):
    """Rows X whose squared values come in groups that rounding alone tells apart."""
    def unitary(a, b):
        return np.linalg.qr(rng.normal(size=(a, b)) + 1j * rng.normal(size=(a, b)))[0]
    yield "isometry", unitary(m + m // 2, m).T
    yield "unitary", unitary(m, m)
    yield "two values", unitary(m, m) * np.where(np.arange(m) < m // 2, 1.0, 0.5)[None, :] @ unitary(m, m)
    yield "rank 3", unitary(m, 3) @ unitary(m, 3).T
    yield "a few values", unitary(m, m) * (2.0 ** -(np.arange(m) % 5))[None, :] @ unitary(m, m)
    yield "one apart", unitary(m, m) * np.where(np.arange(m) == 0, 3.0, 1.0)[None, :] @ unitary(m, m)


def _check_unitary(solver, X, name):
    X = X / np.linalg.norm(X)
    G = X @ X.conj().T
    G = 0.5 * (G + G.conj().T) / np.trace(G).real
    U, lam = solver(G)
    assert np.isfinite(U).all() and np.isfinite(lam).all(), name
    assert np.abs(U.conj().T @ U - np.eye(len(X))).max() <= 1e-12, name
    assert np.abs(U.conj().T @ G @ U - np.diag(lam)).max() <= 1e-12, name


@pytest.mark.parametrize("m", [6, 33, 70, 100])
def test_unitary_whatever_the_groups(solver, m):
    """Values in groups: the deflating rotations keep the poles in order, so the
    vectors are as good as otherwise."""
    for seed in range(24 if m <= 33 else 8):
        for name, X in equal_cases(m, np.random.default_rng((m, seed))):
            _check_unitary(solver, X, (name, seed))


def test_isometries_of_200_rows(solver):
    """All values equal: a pair's kept value, as a sum of two rounded products,
    fell on the value kept before it in one of eight, and a gap of zero made
    every vector of the merge not a number."""
    for key in range(24):
        q = [np.linalg.qr(W.random_complex((k, 200), (380, 200, 300, key, i)))[0] for k, i in ((200, 1), (300, 2))]
        _check_unitary(solver, q[0] @ q[1].conj().T, key)
