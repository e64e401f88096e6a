// Host construction of the 1D spectral-element tables, in extended precision
// and rounded once (entries of a few FP64 roundings each were most of the FP64
// operator's error).
//
// Sec. 2.2 (eqn FEdiscr): C0 Lagrange basis on the GLL points of degree p.
// Eqn cellIntegrals: n_q-point Gauss-Legendre rule per direction.
// Sec. 3.2 (eqn refact): N^1D[q][i] = l_i(xi_q) and the collocation
// derivative Dtilde^1D[q][r] = d/dxi Ltilde_r(xi_q), Ltilde_r being the
// Lagrange polynomial of degree n_q - 1 on the Gauss points, so that
// D^1D = Dtilde^1D N^1D exactly when n_p <= n_q.
// The even-odd packing (Sec. 4.2, used for the contraction counts of
// eqn flopRealMF) relies on N^1D being centro-symmetric and Dtilde^1D
// centro-antisymmetric, which holds because both point sets are symmetric.
#include <cmath>
#include <stdexcept>

#include "fe_internal.h"

namespace fehx {

namespace {

typedef long double real;

// Legendre P_n(x) and P_n'(x) by the three-term recurrence.
void legendre(int n, real x, real &P, real &dP) {
  real p0 = 1.0L, p1 = x;
  if (n == 0) { P = 1.0L; dP = 0.0L; return; }
  for (int k = 2; k <= n; ++k) {
    real p2 = ((2.0L * k - 1.0L) * x * p1 - (k - 1.0L) * p0) / k;
    p0 = p1;
    p1 = p2;
  }
  P = p1;
  dP = (std::fabs(x) < 1.0L) ? n * (x * p1 - p0) / (x * x - 1.0L) : 0.5L * n * (n + 1) * std::pow(x, n + 1);
}

void gauss_rule(int n, std::vector<real> &x, std::vector<real> &w) {
  x.assign(n, 0.0L);
  w.assign(n, 0.0L);
  for (int i = 0; i < n; ++i) {
    real z = std::cos(std::acos(-1.0L) * (i + 0.75L) / (n + 0.5L));   // Chebyshev-like guess
    for (int it = 0; it < 100; ++it) {
      real P, dP;
      legendre(n, z, P, dP);
      real dz = P / dP;
      z -= dz;
      if (std::fabs(dz) < 1e-20L) break;
    }
    real P, dP;
    legendre(n, z, P, dP);
    x[n - 1 - i] = z;
    w[n - 1 - i] = 2.0L / ((1.0L - z * z) * dP * dP);
  }
}

// GLL: -1, +1 and the roots of P_p'; the roots of P_p' are found by Newton
// on q(x) = P_p'(x), with q'(x) from the Legendre ODE.
void gll_rule(int p, std::vector<real> &x, std::vector<real> &w) {
  x.assign(p + 1, 0.0L);
  w.assign(p + 1, 0.0L);
  x[0] = -1.0L;
  x[p] = 1.0L;
  for (int i = 1; i < p; ++i) {
    // initial guess from the Chebyshev-Gauss-Lobatto points
    real z = -std::cos(std::acos(-1.0L) * i / p);
    for (int it = 0; it < 100; ++it) {
      real P, dP;
      legendre(p, z, P, dP);
      // (1 - x^2) P'' - 2 x P' + p(p+1) P = 0
      real d2P = (2.0L * z * dP - p * (p + 1.0L) * P) / (1.0L - z * z);
      real dz = dP / d2P;
      z -= dz;
      if (std::fabs(dz) < 1e-20L) break;
    }
    x[i] = z;
  }
  for (int i = 0; i <= p; ++i) {
    real P, dP;
    legendre(p, x[i], P, dP);
    w[i] = 2.0L / (p * (p + 1.0L) * P * P);
  }
}

// Barycentric weights of a node set.
std::vector<real> bary(const std::vector<real> &z) {
  int n = (int)z.size();
  std::vector<real> b(n, 1.0L);
  for (int i = 0; i < n; ++i)
    for (int j = 0; j < n; ++j)
      if (j != i) b[i] /= (z[i] - z[j]);
  return b;
}

}  // namespace

Tables1D make_tables(int p, int nq) {
  Tables1D t;
  t.p = p;
  t.np = p + 1;
  t.nq = nq;
  std::vector<real> gll, xq;
  gll_rule(p, gll, t.gllwx);
  gauss_rule(nq, xq, t.wqx);
  // N[q][i] = l_i(xq): barycentric form of the Lagrange basis on GLL nodes
  const std::vector<real> bg = bary(gll);
  t.Nx.assign((size_t)nq * t.np, 0.0L);
  for (int q = 0; q < nq; ++q) {
    const real x = xq[q];
    int hit = -1;
    for (int i = 0; i < t.np; ++i)
      if (std::fabs(x - gll[i]) < 1e-15L) hit = i;   // e.g. xi = 0 in both rules
    if (hit >= 0) {
      for (int i = 0; i < t.np; ++i) t.Nx[q * t.np + i] = (i == hit) ? 1.0L : 0.0L;
      continue;
    }
    real denom = 0.0L;
    std::vector<real> tmp(t.np);
    for (int i = 0; i < t.np; ++i) {
      tmp[i] = bg[i] / (x - gll[i]);
      denom += tmp[i];
    }
    for (int i = 0; i < t.np; ++i) t.Nx[q * t.np + i] = tmp[i] / denom;
  }
  // collocation derivative on the Gauss points
  const std::vector<real> bq = bary(xq);
  t.Dtx.assign((size_t)nq * nq, 0.0L);
  for (int q = 0; q < nq; ++q) {
    real diag = 0.0L;
    for (int r = 0; r < nq; ++r) {
      if (r == q) continue;
      const real v = (bq[r] / bq[q]) / (xq[q] - xq[r]);
      t.Dtx[q * nq + r] = v;
      diag -= v;
    }
    t.Dtx[q * nq + q] = diag;
  }
  auto round = [](const std::vector<real> &v) { return std::vector<double>(v.begin(), v.end()); };
  t.gll = round(gll);
  t.gllw = round(t.gllwx);
  t.xq = round(xq);
  t.wq = round(t.wqx);
  t.N = round(t.Nx);
  t.Dt = round(t.Dtx);
  return t;
}

std::vector<double> eo_pack(const std::vector<long double> &A, int nout, int nin, int sym) {
  const int CO = (nout + 1) / 2, CI = (nin + 1) / 2, HI = nin / 2;
  std::vector<double> out((size_t)CO * (CI + HI), 0.0);
  for (int q = 0; q < nout; ++q)
    for (int i = 0; i < nin; ++i) {
      const long double a = A[q * nin + i], b = A[(nout - 1 - q) * nin + (nin - 1 - i)];
      if (!std::isfinite(a) || !(std::fabs(a - sym * b) <= 1e-11L * (1.0L + std::fabs(a))))
        throw std::runtime_error("1D table lacks the even-odd symmetry");
    }
  for (int q = 0; q < CO; ++q) {
    double *E = &out[(size_t)q * (CI + HI)];
    double *O = E + CI;
    for (int i = 0; i < HI; ++i) {
      E[i] = (double)(0.5L * (A[q * nin + i] + A[q * nin + nin - 1 - i]));
      O[i] = (double)(0.5L * (A[q * nin + i] - A[q * nin + nin - 1 - i]));
    }
    if (nin & 1) E[HI] = (double)A[q * nin + HI];
  }
  return out;
}

}  // namespace fehx
