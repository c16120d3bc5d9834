// Host-side reference-element generator.  See refgen.hpp.
#include "refgen.hpp"

#include <algorithm>
#include <cmath>
#include <stdexcept>
#include <tuple>

namespace dgd {

// Working type: every entry is rounded to FP64 once.  (Generated in FP64 the entries
// were off by up to 2.8e-15 of the largest one; errors of single entries are the same
// in every element and step, and where few entries act, K^e after the projection, they
// do not average out.)
typedef long double real;

const int kPerm3[6][3] = {{0, 1, 2}, {0, 2, 1}, {1, 0, 2}, {1, 2, 0}, {2, 0, 1}, {2, 1, 0}};
const int kFaceVerts[4][3] = {{0, 2, 1}, {0, 1, 3}, {0, 3, 2}, {1, 2, 3}};

int n_modes(int N) { return (N + 1) * (N + 2) * (N + 3) / 6; }

// P_n^(a,b)(x) and its derivative by the three-term recurrence;
// d/dx P_n^(a,b) = (n+a+b+1)/2 P_{n-1}^(a+1,b+1).
static real jacobi(int n, real a, real b, real x) {
  if (n == 0) return 1.0;
  real p0 = 1.0, p1 = 0.5 * ((a - b) + (a + b + 2.0) * x);
  for (int k = 2; k <= n; ++k) {
    real c = 2.0 * k + a + b;
    real a1 = 2.0 * k * (k + a + b) * (c - 2.0);
    real a2 = (c - 1.0) * (c * (c - 2.0) * x + a * a - b * b);
    real a3 = 2.0 * (k + a - 1.0) * (k + b - 1.0) * c;
    real p2 = (a2 * p1 - a3 * p0) / a1;
    p0 = p1;
    p1 = p2;
  }
  return p1;
}

static real djacobi(int n, real a, real b, real x) {
  if (n == 0) return 0.0;
  return 0.5 * (n + a + b + 1.0) * jacobi(n - 1, a + 1.0, b + 1.0, x);
}

static void gauss_jacobi(int n, real alpha, std::vector<real>& t, std::vector<real>& w) {
  t.assign(n, 0.0);
  w.assign(n, 0.0);
  for (int k = 0; k < n; ++k) {
    // Chebyshev-like start, refined by Newton with deflation of found roots
    real x = -std::cos((2.0 * k + 1.0) * M_PI / (2.0 * n));
    if (k > 0 && x <= t[k - 1]) x = 0.5 * (t[k - 1] + 1.0);
    for (int it = 0; it < 200; ++it) {
      real p = jacobi(n, alpha, 0.0, x);
      real dp = djacobi(n, alpha, 0.0, x);
      real defl = 0.0;
      for (int j = 0; j < k; ++j) defl += 1.0 / (x - t[j]);
      real dx = p / (dp - p * defl);
      x -= dx;
      if (std::fabs(dx) < 2e-19L) break;
    }
    t[k] = x;
  }
  std::sort(t.begin(), t.end());
  for (int k = 0; k < n; ++k) {
    real dp = djacobi(n, alpha, 0.0, t[k]);
    w[k] = std::pow(real(2), alpha + 1.0) / ((1.0 - t[k] * t[k]) * dp * dp);
  }
}

struct Mode { int i, j, k; };

static std::vector<Mode> modes(int N) {
  std::vector<Mode> m;
  for (int i = 0; i <= N; ++i)
    for (int j = 0; i + j <= N; ++j)
      for (int k = 0; i + j + k <= N; ++k) m.push_back({i, j, k});
  std::sort(m.begin(), m.end(), [](const Mode& A, const Mode& B) {
    return std::make_tuple(A.i + A.j + A.k, A.i, A.j, A.k) <
           std::make_tuple(B.i + B.j + B.k, B.i, B.j, B.k);
  });
  return m;
}

static real ipow(real x, int n) {
  real r = 1.0;
  for (int k = 0; k < n; ++k) r *= x;
  return r;
}

static void basis_real(int N, const real xi[3], real* phi, real* dphi) {
  const real x = xi[0], y = xi[1], z = xi[2];
  const real omyz = 1.0 - y - z, omz = 1.0 - z;
  const real a = 2.0 * x / omyz - 1.0, b = 2.0 * y / omz - 1.0, c = 2.0 * z - 1.0;
  const real hb = 0.5 * (1.0 - b), hc = 0.5 * (1.0 - c);
  std::vector<Mode> ms = modes(N);
  const int L = (int)ms.size();
  for (int l = 0; l < L; ++l) {
    const int i = ms[l].i, j = ms[l].j, k = ms[l].k;
    const real nrm = std::sqrt((real)((2 * i + 1) * (2 * i + 2 * j + 2) * (2 * i + 2 * j + 2 * k + 3)));
    const real fa = jacobi(i, 0.0, 0.0, a);
    const real gb = jacobi(j, 2.0 * i + 1.0, 0.0, b);
    const real hcv = jacobi(k, 2.0 * i + 2.0 * j + 2.0, 0.0, c);
    const real Bv = ipow(hb, i) * gb;
    const real Cv = ipow(hc, i + j) * hcv;
    phi[l] = nrm * fa * Bv * Cv;
    if (dphi) {
      const real dfa = djacobi(i, 0.0, 0.0, a);
      const real dgb = djacobi(j, 2.0 * i + 1.0, 0.0, b);
      const real dhc = djacobi(k, 2.0 * i + 2.0 * j + 2.0, 0.0, c);
      const real Bp = (i > 0 ? -0.5 * i * ipow(hb, i - 1) * gb : 0.0) + ipow(hb, i) * dgb;
      const real Cp = (i + j > 0 ? -0.5 * (i + j) * ipow(hc, i + j - 1) * hcv : 0.0) +
                        ipow(hc, i + j) * dhc;
      const real pa = dfa * Bv * Cv, pb = fa * Bp * Cv, pc = fa * Bv * Cp;
      // a(x,y,z), b(y,z), c(z): chain rule
      const real dx = pa * 2.0 / omyz;
      const real dy = pa * (1.0 + a) / omyz + pb * 2.0 / omz;
      const real dz = pa * (1.0 + a) / omyz + pb * (1.0 + b) / omz + pc * 2.0;
      dphi[0 * L + l] = nrm * dx;
      dphi[1 * L + l] = nrm * dy;
      dphi[2 * L + l] = nrm * dz;
    }
  }
}

void basis_eval(int N, const double xi[3], double* phi, double* dphi) {
  const int L = n_modes(N);
  const real x[3] = {xi[0], xi[1], xi[2]};
  std::vector<real> p(L), d(3 * (size_t)L);
  basis_real(N, x, p.data(), dphi ? d.data() : nullptr);
  std::copy(p.begin(), p.end(), phi);
  if (dphi) std::copy(d.begin(), d.end(), dphi);
}

static const int kRefVerts[4][3] = {{0, 0, 0}, {1, 0, 0}, {0, 1, 0}, {0, 0, 1}};

RefData build_reference(int N) {
  if (N < 1 || N > 6) throw std::invalid_argument("degree out of range");
  RefData r;
  r.N = N;
  r.L = n_modes(N);
  const int n = N + 1;
  r.Q = n * n * n;
  r.Ns = n * n;
  r.Nt = n;
  std::vector<real> ta, wa, tb, wb, tc, wc, xq, wq, eta, beta, tau;
  gauss_jacobi(n, 0.0, ta, wa);
  gauss_jacobi(n, 1.0, tb, wb);
  gauss_jacobi(n, 2.0, tc, wc);
  for (int ia = 0; ia < n; ++ia)
    for (int ib = 0; ib < n; ++ib)
      for (int ic = 0; ic < n; ++ic) {
        const real A = ta[ia], B = tb[ib], C = tc[ic];
        xq.push_back((1 + A) * (1 - B) * (1 - C) / 8);
        xq.push_back((1 + B) * (1 - C) / 4);
        xq.push_back((1 + C) / 2);
        wq.push_back(wa[ia] * wb[ib] * wc[ic] / 64);
      }
  for (int ia = 0; ia < n; ++ia)
    for (int ib = 0; ib < n; ++ib) {
      eta.push_back((1 + ta[ia]) * (1 - tb[ib]) / 4);
      eta.push_back((1 + tb[ib]) / 2);
      beta.push_back(wa[ia] * wb[ib] / 4);
    }
  for (int z = 0; z < n; ++z) {
    tau.push_back((1 + ta[z]) / 2);
    r.gamma.push_back((double)(wa[z] / 2));
  }
  r.xq.assign(xq.begin(), xq.end());
  r.wq.assign(wq.begin(), wq.end());
  r.eta.assign(eta.begin(), eta.end());
  r.beta.assign(beta.begin(), beta.end());
  r.tau.assign(tau.begin(), tau.end());
  const int L = r.L, Q = r.Q, Ns = r.Ns;
  r.V.assign((size_t)Q * L, 0.0);
  r.Pw.assign((size_t)L * Q, 0.0);
  r.Sw.assign((size_t)3 * L * Q, 0.0);
  std::vector<real> K((size_t)3 * L * L, 0), phi(L), dphi(3 * L);
  for (int q = 0; q < Q; ++q) {
    basis_real(N, &xq[3 * q], phi.data(), dphi.data());
    for (int l = 0; l < L; ++l) {
      r.V[(size_t)q * L + l] = (double)phi[l];
      r.Pw[(size_t)l * Q + q] = (double)(wq[q] * phi[l]);
      for (int e = 0; e < 3; ++e)
        r.Sw[((size_t)e * L + l) * Q + q] = (double)(wq[q] * dphi[e * L + l]);
    }
    for (int e = 0; e < 3; ++e)
      for (int k = 0; k < L; ++k)
        for (int l = 0; l < L; ++l)
          K[((size_t)e * L + k) * L + l] += wq[q] * phi[k] * dphi[e * L + l];
  }
  r.K.assign(K.begin(), K.end());
  // orthonormal polynomials of degree <= N on the face with respect to beta, at its
  // points (modified Gram-Schmidt, twice, on monomials)
  std::vector<std::vector<real>> psi;
  for (int d = 0; d <= N; ++d)
    for (int b = 0; b <= d; ++b) {
      std::vector<real> v(Ns);
      for (int i = 0; i < Ns; ++i)
        v[i] = ipow(eta[2 * i] - real(1) / 3, d - b) * ipow(eta[2 * i + 1] - real(1) / 3, b);
      for (int pass = 0; pass < 2; ++pass) {
        for (const auto& w : psi) {
          real s = 0;
          for (int i = 0; i < Ns; ++i) s += beta[i] * v[i] * w[i];
          for (int i = 0; i < Ns; ++i) v[i] -= s * w[i];
        }
        real s = 0;
        for (int i = 0; i < Ns; ++i) s += beta[i] * v[i] * v[i];
        for (real& x : v) x /= std::sqrt(s);
      }
      psi.push_back(v);
    }
  // (degree 1: the point values)
  const int M = N == 1 ? Ns : (int)psi.size();
  std::vector<real> Psi((size_t)M * Ns, 0), lift((size_t)M * Ns, 0);   // R = lift F
  for (int m = 0; m < M; ++m)
    for (int i = 0; i < Ns; ++i) {
      Psi[m * Ns + i] = N == 1 ? real(m == i) : beta[i] * psi[m][i];
      lift[m * Ns + i] = N == 1 ? (m == i ? beta[i] : 0) : Psi[m * Ns + i];
    }
  r.Psi.assign(Psi.begin(), Psi.end());
  r.F.assign((size_t)4 * 6 * Ns * L, 0.0);
  r.R.assign((size_t)4 * 6 * L * M, 0.0);
  for (int f = 0; f < 4; ++f)
    for (int s = 0; s < 6; ++s) {
      std::vector<real> R((size_t)L * M, 0);
      for (int i = 0; i < Ns; ++i) {
        const real e1 = eta[2 * i], e2 = eta[2 * i + 1];
        const real bary[3] = {1 - e1 - e2, e1, e2};
        real loc[3] = {0, 0, 0};
        for (int j = 0; j < 3; ++j) loc[kPerm3[s][j]] = bary[j];
        real xi[3] = {0, 0, 0};
        for (int j = 0; j < 3; ++j)
          for (int d = 0; d < 3; ++d) xi[d] += loc[j] * kRefVerts[kFaceVerts[f][j]][d];
        basis_real(N, xi, phi.data(), nullptr);
        for (int l = 0; l < L; ++l) {
          r.F[(((size_t)f * 6 + s) * Ns + i) * L + l] = (double)phi[l];
          for (int m = 0; m < M; ++m) R[(size_t)l * M + m] += lift[m * Ns + i] * phi[l];
        }
      }
      std::copy(R.begin(), R.end(), r.R.begin() + ((size_t)f * 6 + s) * L * M);
    }
  // Om[z][j] = int_0^{tau_z} l_j(s) ds for the Lagrange polynomials l_j of the
  // time points (monomial coefficients built factor by factor)
  r.Om.assign((size_t)n * n, 0.0);
  for (int j = 0; j < n; ++j) {
    std::vector<real> c(1, 1);
    for (int k = 0; k < n; ++k) {
      if (k == j) continue;
      const real d = tau[j] - tau[k];
      std::vector<real> nc(c.size() + 1, 0);
      for (size_t i = 0; i < c.size(); ++i) {
        nc[i + 1] += c[i] / d;
        nc[i] -= c[i] * tau[k] / d;
      }
      c.swap(nc);
    }
    for (int z = 0; z < n; ++z) {
      real acc = 0, pw = tau[z];
      for (size_t i = 0; i < c.size(); ++i) {
        acc += c[i] / (i + 1) * pw;
        pw *= tau[z];
      }
      r.Om[(size_t)z * n + j] = (double)acc;
    }
  }
  std::vector<Mode> ms = modes(N);
  for (auto& m : ms) r.deg.push_back(m.i + m.j + m.k);
  return r;
}

}  // namespace dgd
