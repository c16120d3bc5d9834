"""Entries of the reference-element data (csrc/refgen.cpp, host code, built here with g++).

Errors of single matrix entries are the same in every element and step, so they do not average out:
each entry has to be the exact value rounded once.  The exact values come from 40-digit arithmetic:
Gauss-Jacobi rules from the roots of the Jacobi polynomial, the basis from its collapsed-coordinate
definition, integrals from monomials (int x^a y^b z^c = a!b!c!/(a+b+c+3)!).
"""
import ctypes
import os
import subprocess

import numpy as np
import pytest

mp = pytest.importorskip("mpmath").mp

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_2502_09714_amd", "csrc")
SHIM = """
#include <cstddef>
#include "refgen.hpp"
static dgd::RefData r;
extern "C" void build(int N) { r = dgd::build_reference(N); }
#define GET(x) extern "C" long get_##x(double* out) { \\
    if (out) for (std::size_t i = 0; i < r.x.size(); ++i) out[i] = r.x[i]; return (long)r.x.size(); }
GET(xq) GET(wq) GET(V) GET(Pw) GET(Sw) GET(K) GET(beta) GET(tau) GET(gamma)
"""


@pytest.fixture(scope="module")
def refgen(tmp_path_factory):
    d = tmp_path_factory.mktemp("refgen")
    (d / "shim.cpp").write_text(SHIM)
    so = str(d / "refgen.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, "-o", so, str(d / "shim.cpp"),
                    os.path.join(CSRC, "refgen.cpp")], check=True)
    return ctypes.CDLL(so)


def _get(lib, name):
    f = getattr(lib, "get_" + name)
    f.restype = ctypes.c_long
    out = np.zeros(f(None))
    f(out.ctypes.data_as(ctypes.c_void_p))
    return out


def _jac(n, a, x):
    """P_n^(a,0)(x) as a sum over powers of (x - 1)/2."""
    return sum(mp.binomial(n, k) * mp.rf(a + n + 1, k) * mp.rf(a + k + 1, n - k) / mp.factorial(n) *
               ((x - 1) / 2) ** k for k in range(n + 1))


def _rule(n, a):
    """n-point rule of weight (1 - t)^a on [-1, 1]: roots, interpolatory weights."""
    g = np.polynomial.legendre.leggauss(64)[0]
    v = [_jac(n, a, mp.mpf(float(x))) for x in np.concatenate([[-1], g, [1]])]
    br = [(float(p), float(q)) for p, q, f, h in zip(np.concatenate([[-1], g]), np.concatenate([g, [1]]), v, v[1:])
          if f * h < 0]
    t = [mp.findroot(lambda x: _jac(n, a, x), (mp.mpf(p), mp.mpf(q)), solver="anderson", tol=mp.mpf(10) ** -70)
         for p, q in br]
    assert len(t) == n
    # int (1-t)^a t^k by substitution s = 1 - t
    mom = [sum(mp.binomial(k, j) * (-1) ** j * mp.mpf(2) ** (a + j + 1) / (a + j + 1) for j in range(k + 1))
           for k in range(n)]
    w = mp.lu_solve(mp.matrix(n, n) + mp.matrix([[x ** k for x in t] for k in range(n)]), mp.matrix(mom))
    return t, [w[i] for i in range(n)]


def _ip(x, n):
    return x ** n if n else mp.mpf(1)


def _phi(m, x):
    i, j, k = m
    om = 1 - x[1] - x[2]
    a, b, c = 2 * x[0] / om - 1, 2 * x[1] / (1 - x[2]) - 1, 2 * x[2] - 1
    return mp.sqrt((2 * i + 1) * (2 * i + 2 * j + 2) * (2 * i + 2 * j + 2 * k + 3)) * _jac(i, 0, a) * \
        _jac(j, 2 * i + 1, b) * _jac(k, 2 * i + 2 * j + 2, c) * _ip((1 - b) / 2, i) * _ip((1 - c) / 2, i + j)


def _exact(N):
    n = N + 1
    (ta, wa), (tb, wb), (tc, wc) = (_rule(n, a) for a in (0, 1, 2))
    pts = [((1 + A) * (1 - B) * (1 - C) / 8, (1 + B) * (1 - C) / 4, (1 + C) / 2) for A in ta for B in tb for C in tc]
    wq = [A * B * C / 64 for A in wa for B in wb for C in wc]
    ms = sorted(((i, j, k) for i in range(n) for j in range(n - i) for k in range(n - i - j)), key=lambda m: (sum(m),) + m)
    L = len(ms)
    # monomial coefficients of the basis from its values at L points of a lattice inside
    lat = [tuple(mp.mpf(4 * m[d] + 1) / (4 * N + 7) for d in range(3)) for m in ms]
    M = mp.matrix([[_ip(x[0], m[0]) * _ip(x[1], m[1]) * _ip(x[2], m[2]) for m in ms] for x in lat])
    coef = M ** -1 * mp.matrix([[_phi(m, x) for m in ms] for x in lat])            # [monomial][mode]
    fac = [mp.factorial(k) for k in range(2 * n + 6)]
    integral = lambda m: fac[m[0]] * fac[m[1]] * fac[m[2]] / fac[sum(m) + 3]       # noqa: E731

    def down(m, e):
        return tuple(v - (d == e) for d, v in enumerate(m)), m[e]

    K, Sw = [], []
    for e in range(3):
        G = mp.matrix(L, L)                      # int mono_a dmono_b/dx_e
        for a, ma in enumerate(ms):
            for b, mb in enumerate(ms):
                lo, f = down(mb, e)
                if f:
                    G[a, b] = f * integral(tuple(x + y for x, y in zip(ma, lo)))
        Ke = coef.T * G * coef
        K += [Ke[k, l] for k in range(L) for l in range(L)]
        D = []
        for x in pts:
            row = []
            for m in ms:
                lo, f = down(m, e)
                row.append(f * _ip(x[0], lo[0]) * _ip(x[1], lo[1]) * _ip(x[2], lo[2]) if f else mp.mpf(0))
            D.append(row)
        dphi = mp.matrix(D) * coef
        Sw += [wq[q] * dphi[q, l] for l in range(L) for q in range(len(pts))]
    V = [[_phi(m, x) for m in ms] for x in pts]
    return dict(xq=[v for x in pts for v in x], wq=wq, V=[v for r in V for v in r],
                Pw=[wq[q] * V[q][l] for l in range(L) for q in range(len(pts))], Sw=Sw, K=K,
                beta=[A * B / 4 for A in wa for B in wb], tau=[(1 + t) / 2 for t in ta], gamma=[w / 2 for w in wa])


@pytest.mark.parametrize("N", [1, 2, 3])
def test_entries_are_the_exact_values_rounded_once(refgen, N):
    with mp.workdps(40):
        want = _exact(N)
        refgen.build(N)
        for name, x in want.items():
            got = _get(refgen, name)
            assert got.size == len(x), name
            top = max(abs(v) for v in x)
            # half a unit in the last place of the entry, and the 64-bit working precision's rounding of
            # sums of at most 4^3 terms
            bound = [abs(v) * mp.mpf(2) ** -53 + top * mp.mpf(2) ** -57 for v in x]
            off = [abs(mp.mpf(float(g)) - v) / b for g, v, b in zip(got, x, bound)]
            assert max(off) <= 1, (name, float(max(off)))
