// Kernels of the Cauchy-Kovalevskaya step (gfx950): prediction, face fluxes,
// corrector.  One 64-lane wavefront per element (k_ck, k_update) or face
// (k_face).
//
// What passes between them is not the states at the time points but the time
// derivatives D^0 .. D^N of the prediction (Eq. CKIter-ref-matrix), one matrix
// per element: rows are modes, columns the NC quantities of all orders.  K^e
// lowers the polynomial degree, so D^i, i >= 1, has only the modes of degree
// <= N - max(i-1, 1) (the damage row of D^1 has all: the projected damage
// source; that of D^i, i >= 2, is zero).  Columns come in the order of falling
// row count, so that the trailing 16-column tiles of every contraction with
// this matrix need fewer matrix-core steps: 17 fragments at degree 4 where the
// five time-point states of ten quantities took 45.  The Taylor sums are
// formed after the contraction, per point, on the vector ALUs.
#pragma once
#include "kernels.hpp"

namespace dgd {

// modes of degree <= d
__host__ __device__ constexpr int modes_upto(int d) {
  return d < 0 ? 0 : (d + 1) * (d + 2) * (d + 3) / 6;
}
// degree of mode l
__host__ __device__ constexpr int mode_degree(int l) {
  int d = 0;
  while (modes_upto(d) <= l) ++d;
  return d;
}

// Wavefronts per SIMD the kernels are compiled for, and how many fragments ahead
// of their use they request the reference matrices.
template <int N, int P> struct StepTune {
  static constexpr int w_ck = P == PREC_F64 ? 2 : 4, w_face = P == PREC_F64 ? 2 : 4,
                       w_update = 2;
  static constexpr int pd_ck = 4, pd_face = 6, pd_update = P == PREC_F64 ? 4 : 10;
};

// Column j of the derivative matrix: 0..9 D^0; 10 the damage row of D^1;
// 11..19 its wave rows; 20 + 9 (i-2) + p: D^i, i >= 2.
// Stored as matrix-core fragments, [element][fragment][lane]: 16-column tile c
// keeps steps(c) k-steps from fragment frag0(c) on; lane (g, n) = (lane / 16,
// lane % 16) holds column 16 c + n at row 4 s + g (rows 16 s + 4 g + 0..3, split
// into BF16 pairs, in the split-BF16 form).
template <int N, int P> struct Deriv {
  static constexpr int KS = Prec<P>::KS;
  static constexpr int NC = 20 + 9 * (N - 1);
  static constexpr int NT = (NC + 15) / 16;
  __host__ __device__ static constexpr int rows(int j) {
    return j <= 10 ? Dims<N>::L : (j < 20 ? modes_upto(N - 1) : modes_upto(N + 1 - (2 + (j - 20) / 9)));
  }
  __host__ __device__ static constexpr int steps(int c) { return (rows(16 * c) + KS - 1) / KS; }
  __host__ __device__ static constexpr int frag0(int c) {
    int f = 0;
    for (int k = 0; k < c; ++k) f += steps(k);
    return f;
  }
  static constexpr int NF = frag0(NT);
  // column of quantity p of order i (p < 9, or i <= 1)
  __host__ __device__ static constexpr int col(int i, int p) {
    return i == 0 ? p : (i == 1 ? (p == 9 ? 10 : 11 + p) : 20 + 9 * (i - 2) + p);
  }
};

// Orders in which lanes and accumulator rows stand for quantities and modes.
// A product's output row r sits in lane group g, register i with r = 4 g + i
// (FP32 accumulators) or g + 4 i (FP64).  Operand rows fed in the order qperm /
// mperm come out with quantity 4 i + g, and mode 16 t + 4 i + g (FP64, FP32) or
// 16 t + 4 g + i (split BF16), in register i of tile t: just the k order of the
// next product's operand, which then needs no data movement.
template <class T> __host__ __device__ constexpr int qperm(int n) {
  return sizeof(T) == 8 ? n : (n & 3) * 4 + (n >> 2);
}
template <int P> __host__ __device__ constexpr int mperm(int n) {
  return P == PREC_F32 ? (n & 3) * 4 + (n >> 2) : n;
}
// mode held by register r (= 4 t + i) of lane group g
template <int P> __device__ inline int reg_mode(int r, int g) {
  return P == PREC_BF16 ? 16 * (r >> 2) + 4 * g + (r & 3) : 4 * r + g;
}
// operand of k-step s from registers in that order
template <int P, class T> __device__ inline typename Prec<P>::AF mode_op(const T* m, int s) {
  if constexpr (P == PREC_BF16)
    return split4(m[4 * s], m[4 * s + 1], m[4 * s + 2], m[4 * s + 3]);
  else
    return m[s];
}

// LDS written by one lane of the wavefront and read by another: the LDS unit
// serves a wavefront's accesses in order, so only the compiler must keep them so.
__device__ inline void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// odd 16-lane rows of a with even rows of b / upper half of a with lower half of b
__device__ inline void swap_rows(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, a),
                                                  __builtin_bit_cast(unsigned, b), false, false);
  const unsigned lo = r[0], hi = r[1];
  a = __builtin_bit_cast(float, lo);
  b = __builtin_bit_cast(float, hi);
}
__device__ inline void swap_halves(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, a),
                                                  __builtin_bit_cast(unsigned, b), false, false);
  const unsigned lo = r[0], hi = r[1];
  a = __builtin_bit_cast(float, lo);
  b = __builtin_bit_cast(float, hi);
}
struct F2 { float x, y; };
__device__ inline void swap_rows(double& a, double& b) {
  F2 p = __builtin_bit_cast(F2, a), q = __builtin_bit_cast(F2, b);
  swap_rows(p.x, q.x);
  swap_rows(p.y, q.y);
  a = __builtin_bit_cast(double, p);
  b = __builtin_bit_cast(double, q);
}
__device__ inline void swap_halves(double& a, double& b) {
  F2 p = __builtin_bit_cast(F2, a), q = __builtin_bit_cast(F2, b);
  swap_halves(p.x, q.x);
  swap_halves(p.y, q.y);
  a = __builtin_bit_cast(double, p);
  b = __builtin_bit_cast(double, q);
}
// 4 x 4 transposition between four registers and the four lane groups:
// afterwards x_k of group g is the former x_g of group k
template <class T> __device__ inline void transpose4(T& x0, T& x1, T& x2, T& x3) {
  swap_rows(x0, x1);
  swap_rows(x2, x3);
  swap_halves(x0, x2);
  swap_halves(x1, x3);
}

template <int R> __device__ inline float ror_add(float v) {
  return v + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
                                           0, __builtin_bit_cast(int, v), 0x120 + R, 0xf, 0xf, true));
}
template <int R> __device__ inline double ror_add(double v) {
  F2 p = __builtin_bit_cast(F2, v), q;
  q.x = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, p.x),
                                                              0x120 + R, 0xf, 0xf, true));
  q.y = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, p.y),
                                                              0x120 + R, 0xf, 0xf, true));
  return v + __builtin_bit_cast(double, q);
}

// sums over the 64 lanes of M values per lane, to out[0..M) in LDS: halving
// exchanges put four sums into the four lane groups, rotations finish them
template <int M, class T> __device__ inline void reduce_to_lds(const T (&x)[M], T* out, int lane) {
  constexpr int M4 = (M + 3) / 4;
  T y[2 * M4];
#pragma unroll
  for (int a = 0; a < 2 * M4; ++a) {
    T u = 2 * a < M ? x[2 * a] : T(0), v = 2 * a + 1 < M ? x[2 * a + 1] : T(0);
    swap_halves(u, v);
    y[a] = u + v;
  }
  const int g = lane >> 4, at = ((g & 1) << 1) | (g >> 1);
#pragma unroll
  for (int b = 0; b < M4; ++b) {
    T u = y[2 * b], v = y[2 * b + 1];
    swap_rows(u, v);
    u = ror_add<8>(u + v);
    u = ror_add<4>(u);
    u = ror_add<2>(u);
    u = ror_add<1>(u);
    if ((lane & 15) == 0) out[4 * b + at] = u;
  }
}

// Products with K^e (mode l' of the result needs modes of higher degree only)
// or its transpose (of lower degree only): the (e, tile, k-step) triples that
// are not zero, in the order they are issued.
template <int NMAX> struct TripleList {
  int n = 0;
  unsigned char e[NMAX] = {}, t[NMAX] = {}, s[NMAX] = {};
};
// K^e: inputs of KIN k-steps, NTO result tiles
template <int N, int P, int KIN, int NTO> constexpr TripleList<3 * KIN * NTO> k_list() {
  TripleList<3 * KIN * NTO> r;
  for (int s = 0; s < KIN; ++s)
    for (int e = 0; e < 3; ++e)
      for (int t = 0; t < NTO; ++t)
        if ((s + 1) * Prec<P>::KS > modes_upto(mode_degree(16 * t))) {
          r.e[r.n] = (unsigned char)e;
          r.t[r.n] = (unsigned char)t;
          r.s[r.n++] = (unsigned char)s;
        }
  return r;
}
// transposed: all MT result tiles, inputs of degree <= (largest of the tile) - 1
template <int N, int P> constexpr TripleList<3 * 16 * 3> kt_list() {
  TripleList<3 * 16 * 3> r;
  constexpr int KS = Prec<P>::KS, L = Dims<N>::L;
  for (int s = 0; KS * s < modes_upto(N - 1); ++s)
    for (int e = 0; e < 3; ++e)
      for (int t = 0; t < Dims<N>::MT; ++t) {
        const int last = 16 * t + 15 < L ? 16 * t + 15 : L - 1;
        if (KS * s < modes_upto(mode_degree(last) - 1)) {
          r.e[r.n] = (unsigned char)e;
          r.t[r.n] = (unsigned char)t;
          r.s[r.n++] = (unsigned char)s;
        }
      }
  return r;
}

// NF fragments ld(0..NF-1) requested PD ahead of their use(k, fragment); the
// scheduling barrier keeps the compiler from sinking the loads to their use
template <int PD, int NF, class AF, class Ld, class Use>
__device__ inline void stream(Ld ld, Use use) {
  AF ring[PD + 1];
#pragma unroll
  for (int k = 0; k < PD && k < NF; ++k) ring[k] = ld(k);
#pragma unroll
  for (int k = 0; k < NF; ++k) {
    if (k + PD < NF) ring[(k + PD) % (PD + 1)] = ld(k + PD);
    __builtin_amdgcn_sched_barrier(0);
    use(k, ring[k % (PD + 1)]);
  }
}

template <int N, int P> struct CkLDS {
  using T = typename Prec<P>::T;
  static constexpr int W = P == PREC_BF16 ? 4 : 1;      // values per fragment entry
  alignas(16) T dz[Deriv<N, P>::NF * 64 * W];
  alignas(16) T r[Dims<N>::NCH * 64];                   // damage rate at the points
  T al[64];                                             // its projection, the damage row of D^1
  T ext[64];                                            // sums of the tangent, then mixing weights
  T tg[48];                                             // cell-averaged tangent / rho, 0, 1/2, 1
};

// Prediction (Appendix A.1, Eqs. CKIter, CKIter-ref-matrix, CKIter-ref-source):
// nodal values at t_n, pointwise tangent and its cell average, damage source,
// recursion D^i = sum_e K^e D^{i-1} (-A*_e)^T; D^0..D^N to HBM.
//
// The recursion stays in registers.  Odd orders contract the modes first (the
// matrix D^T K^eT: D as the row operand, quantities in rows) and then mix the
// quantities (-A*_e from the left); even orders mix first (D as the row operand,
// modes in rows) and contract then (K^e from the left).  Either way the
// accumulators of one product are the operand of the next, and the order of
// D changes from quantities-in-lanes to quantities-in-registers and back.
template <int N, int P, class LW>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(StepTune<N, P>::w_ck))) void k_ck(StepArgs<P> a) {
  using PR = Prec<P>;
  using T = typename PR::T;
  using AF = typename PR::AF;
  using Acc = typename PR::Acc;
  constexpr int PA_ = Accurate<P>::value;
  using PA = Prec<PA_>;
  using DM = Dims<N>;
  using DV = Deriv<N, P>;
  constexpr int L = DM::L, Q = DM::Q, NCH = DM::NCH, MT = DM::MT;
  constexpr int KS = PR::KS, KSL = round_up(L, KS) / KS, NR = P == PREC_BF16 ? 4 * KSL : KSL;
  constexpr int W = CkLDS<N, P>::W, PD = StepTune<N, P>::pd_ck;
  __shared__ CkLDS<N, P> S;

  const int lane = threadIdx.x, n = lane & 15, g = lane >> 4;
  const long long e = elem_index(a);
  if (e < 0) return;
  const int p = qperm<T>(n);

  // D^0 as the row operand: quantity p in lane n, modes in registers
  T d0[NR];
  {
    const T* u = a.U9 + (e * 9 + (p < 9 ? p : 8)) * L;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int l = reg_mode<P>(r, g);
      d0[r] = u[l < L ? l : L - 1];
    }
    if (p == 9) {
      const double* ua = a.Ua + e * L;
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const int l = reg_mode<P>(r, g);
        d0[r] = (T)ua[l < L ? l : L - 1];
      }
    }
#pragma unroll
    for (int r = 0; r < NR; ++r)
      if (p > 9 || reg_mode<P>(r, g) >= L) d0[r] = T(0);
  }
  const Law<T> law{a.amax, a.smin};
  const MatP<T> mt = load_mat<T>(a.mat + e * 8);
  const StepMat<T> m = LW::constants(mt);
  T J[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) J[k] = (T)a.geo[e * 16 + k];
  for (int i = lane; i < DV::NF * 64 * W; i += 64) S.dz[i] = T(0);
  wave_sync();
  // place of quantities-in-lanes register r of order i: its lane's base + roff(r)
  auto roff = [](int r) { return P == PREC_BF16 ? (r >> 2) * 256 + (r & 3) : r * 64; };
  auto lbase = [&](int i) {
    const int j = DV::col(i, p), c = j >> 4;
    const int f0 = c == 0 ? 0 : (c == 1 ? DV::frag0(1) : DV::frag0(DV::NT > 2 ? 2 : 1));
    return (f0 * 64 + g * 16 + (j & 15)) * W;
  };
  if (p < 10) {
    const int b = lbase(0);
#pragma unroll
    for (int r = 0; r < NR; ++r) S.dz[b + roff(r)] = d0[r];
  }

  // nodal values at t_n: the product's rows are quantities, its columns 16
  // points; a transposition over the lane groups gives every lane one point
  T acc[LW::NACC];
#pragma unroll
  for (int k = 0; k < LW::NACC; ++k) acc[k] = T(0);
#pragma unroll 1
  for (int c = 0; c < NCH; ++c) {
    Acc C[4];
    zero_C<P, 4>(C);
    const AF* V = a.Vpk + (size_t)c * 4 * KSL * 64 + lane;
    stream<PD, 4 * KSL, AF>([&](int k) { return V[((k % 4) * KSL + k / 4) * 64]; },
                            [&](int k, const AF& b) {
                              C[k % 4] = PR::mma(mode_op<P>(d0, k / 4), b, C[k % 4]);
                            });
    T u[12];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      T x0 = C[0][i], x1 = C[1][i], x2 = C[2][i], x3 = C[3][i];
      transpose4(x0, x1, x2, x3);
      u[4 * i] = x0;
      u[4 * i + 1] = x1;
      u[4 * i + 2] = x2;
      u[4 * i + 3] = x3;
    }
    const int q = 64 * c + lane;
    const T w = q < Q ? (T)a.wq[q < Q ? q : 0] * a.inv_wsum : T(0);
    const auto v = LW::invariants(u, law);
    LW::tangent_add(v, u, m, law, w, acc);
    S.r[q] = q < Q ? LW::rate(v, m) : T(0);
  }
  reduce_to_lds(acc, S.ext, lane);
  wave_sync();
  if (lane < 48) {
    const T v = lane < 42 ? LW::tangent_entry(S.ext, m, lane / 7, lane % 7) : T(0);
    if (a.Akeep) a.Akeep[e * 48 + lane] = v;
    S.tg[lane] = lane < 42 ? v * m.ir : (lane == 43 ? T(0.5) : (lane == 44 ? T(1) : T(0)));
  }
  // damage source at t_n projected on the modes, one mode per lane
  {
    T s = T(0);
    if (lane < L) {
      typedef T T4 __attribute__((ext_vector_type(4), aligned(16)));
      const T4* pw = (const T4*)a.Psrc + lane;
      const T4* rr = (const T4*)S.r;
#pragma unroll 8
      for (int k = 0; k < (Q + 3) / 4; ++k) {
        const T4 x = pw[k * L], y = rr[k];
        s += x[0] * y[0] + x[1] * y[1] + x[2] * y[2] + x[3] * y[3];
      }
      const int pos = P == PREC_BF16 ? (((lane >> 4) * 64 + ((lane & 15) >> 2) * 16 + 10) << 2) + (lane & 3)
                                     : (lane >> 2) * 64 + (lane & 3) * 16 + 10;
      S.dz[pos] = s;
    }
    S.al[lane] = s;
  }
  wave_sync();
  // -A*_e, rows p (lanes), columns 4 i + g: sum_d Theta^-1_ed W_d
  T As[3][3];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    T w[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) w[d] = S.tg[a.mixP[(i * 3 + d) * 64 + lane]];
#pragma unroll
    for (int ee = 0; ee < 3; ++ee)
      As[ee][i] = J[ee * 3] * w[0] + J[ee * 3 + 1] * w[1] + J[ee * 3 + 2] * w[2];
  }

  const AF* K = a.Kck + lane;
  auto kfrag = [&](int ee, int t, int s) { return K[((ee * MT + t) * KSL + s) * 64]; };
  // contract, then mix: NTO tiles of 16 modes, quantities in rows
  auto contract_mix = [&](const T* in, auto kin, auto nto, Acc* R) {
    constexpr int KIN = decltype(kin)::value, NTO = decltype(nto)::value;
    constexpr auto list = k_list<N, P, KIN, NTO>();
    Acc Z[3][NTO];
#pragma unroll
    for (int ee = 0; ee < 3; ++ee) zero_C<P, NTO>(Z[ee]);
    stream<PD, list.n, AF>([&](int k) { return kfrag(list.e[k], list.t[k], list.s[k]); },
                           [&](int k, const AF& b) {
                             Acc& z = Z[list.e[k]][list.t[k]];
                             z = PR::mma(mode_op<P>(in, list.s[k]), b, z);
                           });
#pragma unroll
    for (int t = 0; t < NTO; ++t) {
#pragma unroll
      for (int k = 0; k < 4; ++k) R[t][k] = 0;
    }
#pragma unroll
    for (int ee = 0; ee < 3; ++ee)
#pragma unroll
      for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int t = 0; t < NTO; ++t) R[t] = PA::mma(As[ee][i], Z[ee][t][i], R[t]);
  };
  // mix, then contract: NTI tiles of 16 modes in, NTO out, modes in rows
  auto mix_contract = [&](const Acc* R, auto kin, auto nto, Acc* C) {
    constexpr int KIN = decltype(kin)::value, NTO = decltype(nto)::value;
    constexpr int NTI = (KIN * KS + 15) / 16;
    constexpr auto list = k_list<N, P, KIN, NTO>();
    T Y[3][NTI * 4];
#pragma unroll
    for (int t = 0; t < NTI; ++t)
#pragma unroll
      for (int ee = 0; ee < 3; ++ee) {
        Acc y;
#pragma unroll
        for (int k = 0; k < 4; ++k) y[k] = 0;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          // tiles past the wave rows of order 1 hold the damage row (i = 2) only
          if (16 * t >= modes_upto(N - 1) && i < 2) continue;
          y = PA::mma(R[t][i], As[ee][i], y);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) Y[ee][4 * t + k] = y[k];
      }
#pragma unroll
    for (int t = 0; t < NTO; ++t) {
#pragma unroll
      for (int k = 0; k < 4; ++k) C[t][k] = 0;
    }
    stream<PD, list.n, AF>([&](int k) { return kfrag(list.e[k], list.t[k], list.s[k]); },
                           [&](int k, const AF& aa) {
                             Acc& z = C[list.t[k]];
                             z = PR::mma(aa, mode_op<P>(Y[list.e[k]], list.s[k]), z);
                           });
  };
  // quantities-in-registers result of order i to the derivative matrix
  auto put_regs = [&](const Acc* R, int i, int rows, int nt) {
    const int mp = mperm<P>(n);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const int pq = 4 * k + g;
      if (pq >= 9) continue;
      const int j = DV::col(i, pq), c = j >> 4;
      const int f0 = c == 0 ? 0 : (c == 1 ? DV::frag0(1) : DV::frag0(DV::NT > 2 ? 2 : 1));
#pragma unroll
      for (int t = 0; t < MT; ++t) {
        if (t >= nt || 16 * t + mp >= rows) continue;
        const int pos = P == PREC_BF16
                            ? (((f0 + t) * 64 + (mp >> 2) * 16 + (j & 15)) << 2) + (mp & 3)
                            : (f0 + 4 * t + (mp >> 2)) * 64 + (mp & 3) * 16 + (j & 15);
        S.dz[pos] = R[t][k];
      }
    }
  };
  // quantities-in-lanes result of order i
  auto put_lanes = [&](const Acc* C, int i, int nsteps) {
    if (p >= 9) return;
    const int b = lbase(i);
#pragma unroll
    for (int r = 0; r < 4 * MT; ++r)
      if (r < (P == PREC_BF16 ? 4 * nsteps : nsteps)) S.dz[b + roff(r)] = C[r >> 2][r & 3];
  };
  constexpr int R1 = modes_upto(N - 1), R3 = modes_upto(N - 2), R4 = modes_upto(N - 3);
  constexpr int NT1 = (R1 + 15) / 16;
  auto ksteps = [](int rows) constexpr { return (rows + KS - 1) / KS; };

  // order 1: all modes in, degree <= N - 1 out; then the damage row
  Acc D1[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int k = 0; k < 4; ++k) D1[t][k] = 0;
  contract_mix(d0, std::integral_constant<int, KSL>{}, std::integral_constant<int, NT1>{}, D1);
  put_regs(D1, 1, R1, NT1);
  if constexpr (N >= 2) {
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      const T v = S.al[16 * t + mperm<P>(n)];
      if (g == 1) D1[t][2] = v;
    }
    // order 2: the damage row brings all modes, degree <= N - 1 out
    Acc D2[NT1];
    mix_contract(D1, std::integral_constant<int, KSL>{}, std::integral_constant<int, NT1>{}, D2);
    put_lanes(D2, 2, ksteps(R1));
    if constexpr (N >= 3) {
      T d2[4 * NT1];
#pragma unroll
      for (int r = 0; r < 4 * NT1; ++r) d2[r] = D2[r >> 2][r & 3];
      Acc D3[1];
      contract_mix(d2, std::integral_constant<int, ksteps(R1)>{}, std::integral_constant<int, 1>{}, D3);
      put_regs(D3, 3, R3, 1);
      if constexpr (N >= 4) {
        Acc D4[1];
        mix_contract(D3, std::integral_constant<int, ksteps(R3)>{}, std::integral_constant<int, 1>{}, D4);
        put_lanes(D4, 4, ksteps(R4));
      }
    }
  }
  wave_sync();
  AF* out = a.Dz + (size_t)e * DV::NF * 64;
  if constexpr (P == PREC_BF16) {
#pragma unroll
    for (int f = 0; f < DV::NF; ++f) {
      const T* v = S.dz + (f * 64 + lane) * 4;
      out[f * 64 + lane] = split4(v[0], v[1], v[2], v[3]);
    }
  } else {
    constexpr int VW = 16 / sizeof(T), NV = DV::NF * 64 / VW;
    typedef T TV __attribute__((ext_vector_type(VW)));
#pragma unroll
    for (int k = 0; k < (NV + 63) / 64; ++k) {
      const int idx = lane + 64 * k;
      if (idx < NV) ((TV*)out)[idx] = ((const TV*)S.dz)[idx];
    }
  }
}

// value of column j (compile time) of a transposed product: C[c][k][i] holds row
// 4 k + i (FP32 accumulators) or k + 4 i (FP64) of tile c
template <class T, class Acc> __device__ inline T column(const Acc (*C)[4], int j) {
  const int m = j & 15;
  return sizeof(T) == 8 ? C[j >> 4][m & 3][m >> 2] : C[j >> 4][m >> 2][m & 3];
}

template <int N, int P> struct UpdLDS {
  using T = typename Prec<P>::T;
  static constexpr int RS = 64 + 16 / sizeof(T);
  alignas(16) T X[10 * RS];       // time integrals at the points of one chunk, [quantity][point]
  T al[2][64];                    // damage row: projected source, lifted flux
};

// Corrector (Appendix A.2, Eqs. 2nd term, 3rd term, rhs term, time-integrated):
// lift of the four face fluxes, volume and source terms, update.
//
// The derivative matrix is evaluated at 64 points at a time (columns in rows of
// the product, transposed so that a lane holds its point's columns); Taylor sums,
// stress and damage rate at every time point are summed in time per point.  The
// flux is linear in velocity and stress and the projection of any point values
// followed by the modal stiffness is the quadrature with S^e, so the ten time
// integrals are projected once (one contraction over the points in place of
// three) and the stiffness, of L x modes of degree < N, and the element's
// Jacobian act on modes.  (Few modes carry what many points did, so the rounding
// of split-BF16 operands would no longer average out there: these two
// contractions take FP32 operands in that form.)
template <int N, int P, class LW>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(StepTune<N, P>::w_update))) void k_update(StepArgs<P> a, const int* fmap,
                                               const typename Prec<P>::T* fflux) {
  using PR = Prec<P>;
  using T = typename PR::T;
  using AF = typename PR::AF;
  using Acc = typename PR::Acc;
  constexpr int PA_ = Accurate<P>::value;
  using PA = Prec<PA_>;
  using DM = Dims<N>;
  using DV = Deriv<N, P>;
  constexpr int L = DM::L, Q = DM::Q, Ns = DM::Ns, Nt = DM::Nt, NCH = DM::NCH, MT = DM::MT;
  constexpr int KS = PR::KS, KSL = round_up(L, KS) / KS, KSN = round_up(Ns, KS) / KS;
  constexpr int NRN = P == PREC_BF16 ? 4 * KSN : KSN, NT = DV::NT, PD = StepTune<N, P>::pd_update;
  using SL = UpdLDS<N, P>;
  __shared__ SL S;

  const int lane = threadIdx.x, n = lane & 15, g = lane >> 4;
  const long long e = elem_index(a);
  if (e < 0) return;
  const int p = qperm<T>(n);

  // lift of the face fluxes (negated where the element is the face's second
  // side; integrals of the finer cluster, cleared, under local time stepping):
  // quantities in rows, modes in columns
  AF dz[DV::NF];
  const AF* dze = a.Dz + (size_t)e * DV::NF * 64 + lane;
#pragma unroll
  for (int f = 0; f < DV::NF; ++f) dz[f] = dze[f * 64];
  T fv[4][NRN], sc[4];
  int sp[4];
#pragma unroll
  for (int f = 0; f < 4; ++f) {
    const int fm = fmap[e * 4 + f];
    sp[f] = conn_perm(a.conn[(e * 4 + f) * 2 + 1]);
    const int nb = a.conn[(e * 4 + f) * 2];
    const bool fine = a.lts_c > 0 && nb >= 0 && a.ecl[nb] == a.lts_c - 1;
    sc[f] = (T)((fm & 1 ? 1.0 : -1.0) * a.fgeo[(e * 4 + f) * 4 + 3] * (fine ? 1.0 : a.dt));
    T* fl = (fine ? a.facc : (T*)fflux) + (size_t)(fm >> 1) * Ns * 10 + (p < 10 ? p : 9);
#pragma unroll
    for (int r = 0; r < NRN; ++r) {
      const int i = reg_mode<P>(r, g);     // face point
      fv[f][r] = fl[(i < Ns ? i : Ns - 1) * 10];
    }
    if (fine) {
      wave_sync();
#pragma unroll
      for (int r = 0; r < NRN; ++r) {
        const int i = reg_mode<P>(r, g);
        if (i < Ns && p < 10) fl[i * 10] = T(0);
      }
    }
  }
  const Law<T> law{a.amax, a.smin};
  const StepMat<T> m = LW::constants(load_mat<T>(a.mat + e * 8));
  Acc U[MT];
  zero_C<P, MT>(U);
#pragma unroll
  for (int f = 0; f < 4; ++f) {
    T v[NRN];
#pragma unroll
    for (int r = 0; r < NRN; ++r)
      v[r] = (reg_mode<P>(r, g) < Ns && p < 10) ? sc[f] * fv[f][r] : T(0);
    const AF* Lf = a.Lpk + (size_t)(f * 6 + sp[f]) * MT * KSN * 64 + lane;
    stream<PD, MT * KSN, AF>([&](int k) { return Lf[((k % MT) * KSN + k / MT) * 64]; },
                             [&](int k, const AF& b) {
                               U[k % MT] = PR::mma(mode_op<P>(v, k / MT), b, U[k % MT]);
                             });
  }

  typename PA::Acc X[MT];
  zero_C<PA_, MT>(X);
#pragma unroll 1
  for (int c = 0; c < NCH; ++c) {
    T x[10];
#pragma unroll
    for (int k = 0; k < 10; ++k) x[k] = T(0);
    {
      Acc C[NT][4];
#pragma unroll
      for (int ct = 0; ct < NT; ++ct) zero_C<P, 4>(C[ct]);
      const AF* V = a.Vpk + (size_t)c * 4 * KSL * 64 + lane;
      stream<PD, 4 * KSL, AF>([&](int k) { return V[((k % 4) * KSL + k / 4) * 64]; },
                              [&](int k, const AF& b) {
                                const int s = k / 4, t = k % 4;
#pragma unroll
                                for (int ct = 0; ct < NT; ++ct)
                                  if (s < DV::steps(ct))
                                    C[ct][t] = PR::mma(dz[DV::frag0(ct) + s], b, C[ct][t]);
                              });
#pragma unroll
      for (int ct = 0; ct < NT; ++ct)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          T x0 = C[ct][0][i], x1 = C[ct][1][i], x2 = C[ct][2][i], x3 = C[ct][3][i];
          transpose4(x0, x1, x2, x3);
          C[ct][0][i] = x0;
          C[ct][1][i] = x1;
          C[ct][2][i] = x2;
          C[ct][3][i] = x3;
        }
#pragma unroll
      for (int z = 0; z < Nt; ++z) {
        const T h = a.hz[z], gz = a.gamma[z];
        T u[10];   // (the velocity is not needed per time point)
#pragma unroll
        for (int k = 0; k < 6; ++k) {
          T v = column<T>(C, DV::col(N, k));
#pragma unroll
          for (int i = N - 1; i >= 0; --i) v = column<T>(C, DV::col(i, k)) + (h * T(1.0 / (i + 1))) * v;
          u[k] = v;
        }
        u[9] = column<T>(C, 9) + h * column<T>(C, 10);
        T sig[6];
        const auto v = LW::invariants(u, law);
        LW::stress(v, u, m, sig);
        x[9] += gz * LW::rate(v, m);
#pragma unroll
        for (int k = 0; k < 6; ++k) x[3 + k] += gz * sig[k];
      }
      // the time integral of the velocity: sum_z gamma_z h_z^i / i! per order
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        x[k] = column<T>(C, 6 + k);
#pragma unroll
        for (int i = 1; i <= N; ++i) x[k] += a.wint[i] * column<T>(C, DV::col(i, 6 + k));
      }
    }
    wave_sync();
#pragma unroll
    for (int k = 0; k < 10; ++k) S.X[k * SL::RS + lane] = x[k];
    wave_sync();
    // projection: X += P_c x, modes in rows, quantities in columns
    typedef T T4 __attribute__((ext_vector_type(4), aligned(16)));
    using PAF = typename PA::AF;
    const T* xs = S.X + (p < 10 ? p : 9) * SL::RS + 4 * g;
    T4 xv[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) xv[k] = *(const T4*)(xs + 16 * k);
    const PAF* Pk = a.PXpk + (size_t)c * MT * 16 * 64 + lane;
    stream<PD, 16 * MT, PAF>([&](int k) { return Pk[((k % MT) * 16 + k / MT) * 64]; },
                             [&](int k, const PAF& aa) {
                               const int s = k / MT;
                               X[k % MT] = PA::mma(aa, xv[s >> 2][s & 3], X[k % MT]);
                             });
  }
  // the projected source (times dt) leaves through LDS, one mode per lane
  if (p == 9) {
#pragma unroll
    for (int r = 0; r < 4 * MT; ++r) S.al[0][reg_mode<PA_>(r, g)] = X[r >> 2][r & 3];
  }
  T u9[3][MT];
  const T* U9 = a.U9 + e * 9 * L;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      const int pq = 4 * i + g, l = 16 * t + n;
      u9[i][t] = U9[(pq < 9 ? pq : 8) * L + (l < L ? l : L - 1)];
    }
  const double ua = a.Ua[e * L + (lane < L ? lane : L - 1)];
  // stiffness on modes, then the Jacobian and the material on quantities
  {
    T xm[4 * MT];
#pragma unroll
    for (int r = 0; r < 4 * MT; ++r) xm[r] = X[r >> 2][r & 3];
    constexpr auto list = kt_list<N, PA_>();
    using PAF = typename PA::AF;
    constexpr int KSA = round_up(L, PA::KS) / PA::KS;
    typename PA::Acc Z[3][MT];
#pragma unroll
    for (int ee = 0; ee < 3; ++ee) zero_C<PA_, MT>(Z[ee]);
    const PAF* Kt = a.Ktl + lane;
    stream<PD, list.n, PAF>(
        [&](int k) { return Kt[((list.e[k] * MT + list.t[k]) * KSA + list.s[k]) * 64]; },
        [&](int k, const PAF& b) {
          auto& z = Z[list.e[k]][list.t[k]];
          z = PA::mma(mode_op<PA_>(xm, list.s[k]), b, z);
        });
    const T rs = (T)a.dt * (p >= 6 ? m.ir : T(1));
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      T w[3];
#pragma unroll
      for (int d = 0; d < 3; ++d) w[d] = rs * a.mixV[(i * 3 + d) * 64 + lane];
#pragma unroll
      for (int ee = 0; ee < 3; ++ee) {
        const T Ag = (T)a.geo[e * 16 + ee * 3] * w[0] + (T)a.geo[e * 16 + ee * 3 + 1] * w[1] +
                     (T)a.geo[e * 16 + ee * 3 + 2] * w[2];
#pragma unroll
        for (int t = 0; t < MT; ++t) U[t] = PA::mma(Ag, Z[ee][t][i], U[t]);
      }
    }
  }
  if (g == 1) {
#pragma unroll
    for (int t = 0; t < MT; ++t) S.al[1][16 * t + n] = U[t][2];
  }
  wave_sync();
  bool bad = false;
  T* O9 = a.W9 + e * 9 * L;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const int pq = 4 * i + g;
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      const int l = 16 * t + n;
      if (pq < 9 && l < L) {
        const T v = u9[i][t] + U[t][i];
        bad |= !isfinite(v);
        O9[pq * L + l] = v;
      }
    }
  }
  if (lane < L) {
    const double v = ua + (double)((T)a.dt * S.al[0][lane]) + (double)S.al[1][lane];
    bad |= !isfinite(v);
    a.Wa[e * L + lane] = v;
  }
  if (bad) a.flag[0] = 1;
}

// Time since each cluster's prediction at the start of the step being corrected
// (all zero in the global step).
struct ClusterOffsets { double v[8]; };

template <int N, int P> struct FaceLDS {
  using T = typename Prec<P>::T;
  static constexpr int JS = 16 * Deriv<N, P>::NT + 16 / sizeof(T);
  alignas(16) T tr[2][Dims<N>::Ns * JS];   // derivative traces of both sides, [point][column]
};

// Face fluxes (Appendix A.2 Eq. 2nd term, A.3), interior faces once: traces of
// both sides' derivative matrices at the shared face points, Taylor sums per
// (time point, face point), local Lax-Friedrichs or boundary flux, time
// quadrature; sum_z gamma_z F* at the face points, [face][Ns][10].
template <int N, int P, class LW>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(StepTune<N, P>::w_face))) void k_face(StepArgs<P> a, const int* faces, long long nfaces,
                                             typename Prec<P>::T* fflux, const int* flist,
                                             ClusterOffsets offs) {
  using PR = Prec<P>;
  using T = typename PR::T;
  using AF = typename PR::AF;
  using Acc = typename PR::Acc;
  using DM = Dims<N>;
  using DV = Deriv<N, P>;
  using SL = FaceLDS<N, P>;
  constexpr int L = DM::L, Ns = DM::Ns, Nt = DM::Nt, NST = DM::NST, NT = DV::NT;
  constexpr int KS = PR::KS, KSL = round_up(L, KS) / KS, JS = SL::JS, PD = StepTune<N, P>::pd_face;
  constexpr int NRD = (Ns * Nt + 63) / 64, FR = 11;
  static_assert(Ns * Nt * FR <= 2 * Ns * JS, "fluxes fit the spent traces");
  __shared__ SL S;

  const int lane = threadIdx.x, n = lane & 15, g = lane >> 4;
  long long fid = elem_of_block(nfaces);
  if (fid >= nfaces) return;
  if (flist) fid = flist[fid];
  const int ef = faces[fid * 2], of = faces[fid * 2 + 1];
  const long long e = ef >> 2;
  const int f = ef & 3;
  const int w = a.conn[ef * 2 + 1];
  const int kind = conn_kind(w), sp = conn_perm(w);
  const bool inner = kind == 0;
  const long long nb = inner ? (long long)(of >> 2) : e;
  const int nf = inner ? (of & 3) : f, sq = inner ? conn_nperm(w) : sp;
  AF dz[2][DV::NF];
#pragma unroll
  for (int side = 0; side < 2; ++side) {
    const AF* d = a.Dz + (size_t)(side ? nb : e) * DV::NF * 64 + lane;
#pragma unroll
    for (int k = 0; k < DV::NF; ++k) dz[side][k] = d[k * 64];
  }
  // (a boundary face evaluates its own side twice and uses the first)
#pragma unroll
  for (int side = 0; side < 2; ++side) {
    const AF* F = a.Fpk + (size_t)((side ? nf : f) * 6 + (side ? sq : sp)) * NST * KSL * 64 + lane;
    Acc C[NT][NST];
#pragma unroll
    for (int ct = 0; ct < NT; ++ct) zero_C<P, NST>(C[ct]);
    stream<PD, NST * KSL, AF>([&](int k) { return F[((k % NST) * KSL + k / NST) * 64]; },
                              [&](int k, const AF& b) {
                                const int s = k / NST, t = k % NST;
#pragma unroll
                                for (int ct = 0; ct < NT; ++ct)
                                  if (s < DV::steps(ct))
                                    C[ct][t] = PR::mma(dz[side][DV::frag0(ct) + s], b, C[ct][t]);
                              });
#pragma unroll
    for (int ct = 0; ct < NT; ++ct)
#pragma unroll
      for (int t = 0; t < NST; ++t) {
        if (16 * t + n < Ns) {
          T* o = S.tr[side] + (16 * t + n) * JS + 16 * ct;
          if constexpr (sizeof(T) == 8) {
#pragma unroll
            for (int i = 0; i < 4; ++i) o[g + 4 * i] = C[ct][t][i];
          } else {
            *(Acc*)(o + 4 * g) = C[ct][t];
          }
        }
      }
  }
  wave_sync();
  const Law<T> law{a.amax, a.smin};
  const MatP<T> mt = load_mat<T>(a.mat + e * 8), mn = load_mat<T>(a.mat + nb * 8);
  const StepMat<T> ma = LW::constants(mt), mb = LW::constants(mn);
  const bool same = same_material(mt, mn);
  T nrm[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) nrm[k] = (T)a.fgeo[(e * 4 + f) * 4 + k];
  T off[2] = {T(0), T(0)};
  if (a.ecl) {
    off[0] = (T)offs.v[a.ecl[e]];
    off[1] = (T)offs.v[a.ecl[nb]];
  }
  T F[NRD][10];
#pragma unroll
  for (int rd = 0; rd < NRD; ++rd) {
    const int idx = lane + 64 * rd;
    if (idx < Ns * Nt) {
      const int z = idx / Ns, i = idx - z * Ns;
      T u[2][10];
#pragma unroll
      for (int side = 0; side < 2; ++side) {
        if (side && !inner) continue;
        const T h = a.hz[z] + off[side];
        const T* d = S.tr[side] + i * JS;
#pragma unroll
        for (int k = 0; k < 9; ++k) {
          T v = d[DV::col(N, k)];
#pragma unroll
          for (int o = N - 1; o >= 0; --o) v = d[DV::col(o, k)] + (h * T(1.0 / (o + 1))) * v;
          u[side][k] = v;
        }
        u[side][9] = d[9] + h * d[10];
      }
      if (inner)
        llf_flux_step<LW>(u[0], u[1], nrm, ma, mb, same, law, F[rd]);
      else
        boundary_flux<typename LW::Plain>(kind, u[0], nrm, mt, law, F[rd]);
    }
  }
  wave_sync();
  T* sF = &S.tr[0][0];
#pragma unroll
  for (int rd = 0; rd < NRD; ++rd) {
    const int idx = lane + 64 * rd;
    if (idx < Ns * Nt) {
#pragma unroll
      for (int k = 0; k < 10; ++k) sF[idx * FR + k] = F[rd][k];
    }
  }
  wave_sync();
  T* out = fflux + (size_t)fid * Ns * 10;
#pragma unroll
  for (int j = 0; j < (Ns * 10 + 63) / 64; ++j) {
    const int idx = lane + 64 * j;
    if (idx < Ns * 10) {
      const int i = idx / 10, k = idx - i * 10;
      T s = T(0);
#pragma unroll
      for (int z = 0; z < Nt; ++z) s += a.gamma[z] * sF[(z * Ns + i) * FR + k];
      out[idx] = s;
    }
  }
}

// Time-point states of the derivatives in Dz (the Taylor sums of Eq.
// taylor_expansion), [E][Nt][10][L] FP64, for dgd_get_time_point_states.
template <int N, int P>
__global__ __launch_bounds__(64) void k_time_points(StepArgs<P> a, double* out) {
  using T = typename Prec<P>::T;
  using DM = Dims<N>;
  using DV = Deriv<N, P>;
  constexpr int L = DM::L, Nt = DM::Nt;
  const long long e = blockIdx.x;
  auto at = [&](int l, int j) -> T {
    const int c = j >> 4, f0 = DV::frag0(c);
    if (l >= DV::rows(j)) return T(0);
    const typename Prec<P>::AF* d = a.Dz + (size_t)e * DV::NF * 64;
    if constexpr (P == PREC_BF16) {
      const bf16s v = d[(f0 + l / 16) * 64 + ((l % 16) / 4) * 16 + (j & 15)];
      auto f = [](short b) { return __builtin_bit_cast(float, (unsigned)(unsigned short)b << 16); };
      return f(v.hi[l & 3]) + f(v.lo[l & 3]);
    } else {
      return d[(f0 + l / 4) * 64 + (l & 3) * 16 + (j & 15)];
    }
  };
  for (int idx = threadIdx.x; idx < 10 * L; idx += 64) {
    const int p = idx / L, l = idx - p * L;
    for (int z = 0; z < Nt; ++z) {
      const T h = a.hz[z];
      T v;
      if (p == 9) {
        v = at(l, 9) + h * at(l, 10);
      } else {
        v = at(l, DV::col(N, p));
        for (int i = N - 1; i >= 0; --i) v = at(l, DV::col(i, p)) + (h * T(1.0 / (i + 1))) * v;
      }
      out[((e * Nt + z) * 10 + p) * L + l] = (double)v;
    }
  }
}

}  // namespace dgd
