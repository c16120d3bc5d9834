// Host-side reference-element generator.  See refgen.hpp.
#include "refgen.hpp"

#include <algorithm>
#include <cmath>
#include <mutex>
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
template <class R> static R jacobi(int n, R a, R b, R x) {
  if (n == 0) return 1;
  R p0 = 1, p1 = ((a - b) + (a + b + 2) * x) / 2;
  for (int k = 2; k <= n; ++k) {
    R c = 2 * k + a + b;
    R a1 = 2 * k * (k + a + b) * (c - 2);
    R a2 = (c - 1) * (c * (c - 2) * x + a * a - b * b);
    R a3 = 2 * (k + a - 1) * (k + b - 1) * c;
    R p2 = (a2 * p1 - a3 * p0) / a1;
    p0 = p1;
    p1 = p2;
  }
  return p1;
}

template <class R> static R djacobi(int n, R a, R b, R x) {
  if (n == 0) return 0;
  return (n + a + b + 1) / 2 * jacobi<R>(n - 1, a + 1, b + 1, x);
}

static void gauss_jacobi(int n, real alpha, std::vector<real>& t, std::vector<real>& w) {
  t.assign(n, 0);
  w.assign(n, 0);
  for (int k = 0; k < n; ++k) {
    // Chebyshev-like start, refined by Newton with deflation of found roots
    real x = -std::cos((2.0 * k + 1.0) * M_PI / (2.0 * n));
    if (k > 0 && x <= t[k - 1]) x = (t[k - 1] + 1) / 2;
    for (int it = 0; it < 200; ++it) {
      real p = jacobi<real>(n, alpha, 0, x);
      real dp = djacobi<real>(n, alpha, 0, x);
      real defl = 0;
      for (int j = 0; j < k; ++j) defl += 1 / (x - t[j]);
      real dx = p / (dp - p * defl);
      x -= dx;
      if (std::fabs(dx) < 2e-19L) break;
    }
    t[k] = x;
  }
  std::sort(t.begin(), t.end());
  for (int k = 0; k < n; ++k) {
    real dp = djacobi<real>(n, alpha, 0, t[k]);
    w[k] = std::pow(real(2), alpha + 1) / ((1 - t[k] * t[k]) * dp * dp);
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

template <class R> static R ipow(R x, int n) {
  R r = 1;
  for (int k = 0; k < n; ++k) r *= x;
  return r;
}

// The orthonormal basis phi_ijk = nrm A_i(a) B_ij(b) C_(i+j)k(c) at collapsed
// coordinates (a, b, c), hb = (1 - b)/2, hc = (1 - c)/2: its factors
//   A_i = P_i^(0,0)(a), B_ij = hb^i P_j^(2i+1,0)(b), C_mk = hc^m P_k^(2m+2,0)(c)
// and their derivatives with respect to a, b, c.
template <class R> struct Factors {
  R A[7], B[7][7], C[7][7], dA[7], dB[7][7], dC[7][7];
  void eval_a(int N, R a, bool grad) {
    for (int i = 0; i <= N; ++i) {
      A[i] = jacobi<R>(i, 0, 0, a);
      if (grad) dA[i] = djacobi<R>(i, 0, 0, a);
    }
  }
  void eval_b(int N, R b, R hb, bool grad) { fill(N, 1, b, hb, grad, B, dB); }
  void eval_c(int N, R c, R hc, bool grad) { fill(N, 2, c, hc, grad, C, dC); }

 private:
  static void fill(int N, int add, R x, R h, bool grad, R (*F)[7], R (*dF)[7]) {
    for (int i = 0; i <= N; ++i)
      for (int j = 0; i + j <= N; ++j) {
        const R al = 2 * i + add, p = jacobi<R>(j, al, 0, x), hi = ipow(h, i);
        F[i][j] = hi * p;
        if (grad)
          dF[i][j] = (i > 0 ? -R(i) / 2 * ipow(h, i - 1) * p : R(0)) + hi * djacobi<R>(j, al, 0, x);
      }
  }
};

template <class R>
static void combine(const std::vector<Mode>& ms, const R* nrm, const Factors<R>& f, R a, R b, R hb,
                    R hc, R* phi, R* dphi) {
  const int L = (int)ms.size();
  for (int l = 0; l < L; ++l) {
    const int i = ms[l].i, j = ms[l].j, k = ms[l].k;
    const R Av = f.A[i], Bv = f.B[i][j], Cv = f.C[i + j][k];
    phi[l] = nrm[l] * Av * Bv * Cv;
    if (dphi) {
      // a(x,y,z), b(y,z), c(z): chain rule, 1 - y - z = hb hc, 1 - z = hc
      const R pa = f.dA[i] * Bv * Cv, pb = Av * f.dB[i][j] * Cv, pc = Av * Bv * f.dC[i + j][k];
      const R om = hb * hc;
      dphi[0 * L + l] = nrm[l] * (pa * 2 / om);
      dphi[1 * L + l] = nrm[l] * (pa * (1 + a) / om + pb * 2 / hc);
      dphi[2 * L + l] = nrm[l] * (pa * (1 + a) / om + pb * (1 + b) / hc + pc * 2);
    }
  }
}

template <class R> static std::vector<R> norms(const std::vector<Mode>& ms) {
  std::vector<R> n;
  for (const Mode& m : ms)
    n.push_back(std::sqrt((R)((2 * m.i + 1) * (2 * m.i + 2 * m.j + 2) * (2 * m.i + 2 * m.j + 2 * m.k + 3))));
  return n;
}

// at a point of the reference tetrahedron
template <class R>
static void basis_at(int N, const std::vector<Mode>& ms, const R* nrm, const R xi[3], R* phi, R* dphi) {
  const R x = xi[0], y = xi[1], z = xi[2];
  const R omyz = 1 - y - z, omz = 1 - z;
  const R a = 2 * x / omyz - 1, b = 2 * y / omz - 1, c = 2 * z - 1;
  const R hb = (1 - b) / 2, hc = (1 - c) / 2;
  Factors<R> f;
  f.eval_a(N, a, dphi);
  f.eval_b(N, b, hb, dphi);
  f.eval_c(N, c, hc, dphi);
  combine(ms, nrm, f, a, b, hb, hc, phi, dphi);
}

void basis_eval(int N, const double xi[3], double* phi, double* dphi) {
  const std::vector<Mode> ms = modes(N);
  basis_at<double>(N, ms, norms<double>(ms).data(), xi, phi, dphi);
}

static const int kRefVerts[4][3] = {{0, 0, 0}, {1, 0, 0}, {0, 1, 0}, {0, 0, 1}};

static RefData generate(int N) {
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
  const std::vector<Mode> ms = modes(N);
  const std::vector<real> nrm = norms<real>(ms);
  for (const Mode& m : ms) r.deg.push_back(m.i + m.j + m.k);
  std::vector<real> K((size_t)3 * L * L, 0), phi(L), dphi(3 * L);
  std::vector<Factors<real>> at(n);        // the factors at the points of the one-dimensional rules
  for (int k = 0; k < n; ++k) {
    at[k].eval_a(N, ta[k], true);
    at[k].eval_b(N, tb[k], (1 - tb[k]) / 2, true);
    at[k].eval_c(N, tc[k], (1 - tc[k]) / 2, true);
  }
  for (int q = 0; q < Q; ++q) {
    const int ia = q / (n * n), ib = q / n % n, ic = q % n;
    Factors<real> f;
    for (int i = 0; i <= N; ++i) {
      f.A[i] = at[ia].A[i];
      f.dA[i] = at[ia].dA[i];
      for (int j = 0; i + j <= N; ++j) {
        f.B[i][j] = at[ib].B[i][j];
        f.dB[i][j] = at[ib].dB[i][j];
        f.C[i][j] = at[ic].C[i][j];
        f.dC[i][j] = at[ic].dC[i][j];
      }
    }
    combine<real>(ms, nrm.data(), f, ta[ia], tb[ib], (1 - tb[ib]) / 2, (1 - tc[ic]) / 2, phi.data(), dphi.data());
    for (int l = 0; l < L; ++l) {
      r.V[(size_t)q * L + l] = (double)phi[l];
      r.Pw[(size_t)l * Q + q] = (double)(wq[q] * phi[l]);
      for (int e = 0; e < 3; ++e)
        r.Sw[((size_t)e * L + l) * Q + q] = (double)(wq[q] * dphi[e * L + l]);
    }
    // (a derivative lowers the degree: the other entries are zero)
    for (int e = 0; e < 3; ++e)
      for (int k = 0; k < L; ++k) {
        const real wp = wq[q] * phi[k];
        for (int l = n_modes(r.deg[k]); l < L; ++l) K[((size_t)e * L + k) * L + l] += wp * dphi[e * L + l];
      }
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
        basis_at<real>(N, ms, nrm.data(), xi, phi.data(), nullptr);
        for (int l = 0; l < L; ++l) {
          r.F[(((size_t)f * 6 + s) * Ns + i) * L + l] = (double)phi[l];
          // (psi_m is orthogonal to polynomials of lower degree)
          const int top = N == 1 ? M : (r.deg[l] + 1) * (r.deg[l] + 2) / 2;
          for (int m = 0; m < top; ++m) R[(size_t)l * M + m] += lift[m * Ns + i] * phi[l];
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
  return r;
}

// (constants of the degree: generated by the first handle of a process)
const RefData& build_reference(int N) {
  if (N < 1 || N > 6) throw std::invalid_argument("degree out of range");
  static std::once_flag once[7];
  static RefData data[7];
  std::call_once(once[N], [&] { data[N] = generate(N); });
  return data[N];
}

}  // namespace dgd
