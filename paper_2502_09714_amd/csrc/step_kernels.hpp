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

// Form of the reference-matrix contractions of a step.
// FP64 products and FP32 16x16x4 products run on the vector ALUs (measured: a
// stream of them and a stream of vector FMAs on one SIMD take the sum of their
// times); the BF16 matrix cores run beside them.  From degree 3 on the FP32 and
// split-BF16 handles therefore contract on the BF16 matrix cores with three-way
// split operands (Prec<PREC_X3>): x = h + m + l exactly, and the six products of
// weight >= 2^-18, 2^-27 of |a||b| and less left out: not less accurate than FP32
// products (their sums round once per 32 terms).  A 32-term step costs 96 cycles
// of the matrix cores where eight FP32 steps cost 256 cycles of the vector ALUs.
// Below degree 3 a contraction has 4 or 10 terms and FP32 steps are shorter.
template <int N, int P> struct MatForm {
  static constexpr int value = P == PREC_F32 && N >= 3 ? PREC_X3 : P;
};
// The face traces read their matrices (24 of them) from L2, where the split ones
// are half as large again: only from degree 4 on is that the smaller cost.
template <int N, int P> struct FaceForm {
  static constexpr int value = P == PREC_F32 && N >= 4 ? PREC_X3 : P;
};

// Steps of a contraction over R rows: WIDE fragments of Prec<M>::KS rows each,
// and in the three-way form, where 1..4 rows are left over, one FP32 step (TAIL).
// NREG: registers per lane of an operand.
template <int M, int R> struct Steps {
  static constexpr bool TAIL = M == PREC_X3 && R % 32 > 0 && R % 32 <= 4;
  static constexpr int KS = Prec<M>::KS;
  static constexpr int WIDE = TAIL ? R / 32 : (R + KS - 1) / KS;
  static constexpr int NREG = M == PREC_X3 ? 8 * WIDE + TAIL : WIDE;
  // row held by operand register r of lane group g
  __host__ __device__ static constexpr int row(int r, int g) {
    if (M != PREC_X3) return 4 * r + g;
    return r < 8 * WIDE ? 16 * (r >> 2) + 4 * g + (r & 3) : 32 * WIDE + g;
  }
  // wide step s holds rows < hi(s) and >= lo(s)
  __host__ __device__ static constexpr int lo(int s) { return KS * s; }
  __host__ __device__ static constexpr int hi(int s) { return KS * (s + 1); }
};

// Column j of the derivative matrix: 0..9 D^0; 10 the damage row of D^1;
// 11..19 its wave rows; 20 + 9 (i-2) + p: D^i, i >= 2.
// Stored as fragments of four rows, [element][fragment][lane]: 16-column tile c
// keeps steps(c) of them from fragment frag0(c) on; lane (g, n) = (lane / 16,
// lane % 16) holds column 16 c + n at row 4 s + g.
template <int N> struct Deriv {
  static constexpr int NC = 20 + 9 * (N - 1);
  static constexpr int NT = (NC + 15) / 16;
  __host__ __device__ static constexpr int rows(int j) {
    return j <= 10 ? Dims<N>::L : (j < 20 ? modes_upto(N - 1) : modes_upto(N + 1 - (2 + (j - 20) / 9)));
  }
  __host__ __device__ static constexpr int steps(int c) { return (rows(16 * c) + 3) / 4; }
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
  // first fragment of the tile of column j (j not a compile-time constant)
  __device__ static int tile0(int j) {
    const int c = j >> 4;
    return c == 0 ? 0 : (c == 1 ? frag0(1) : frag0(NT > 2 ? 2 : 1));
  }
};

// Launch shapes.  From degree 3 on, k_ck and k_update keep the reference matrices
// in LDS: one workgroup of wpb_* wavefronts per compute unit copies them once and
// walks over elements (read from L2 instead, 67 KB per element at degree 4 missed
// the 32 KB L1 and the wavefronts waited on its pending lines for 60 % of the
// time).  Below degree 3 they fit the L1 and a wavefront takes one element.
// pd_*: how many fragments ahead of their use they are requested.
// (Times here and below: HIP events around warm launches.)
// Update at degree 4: 12 wavefronts 1950 us at 312132 elements, 8 wavefronts 2175;
// at degree 3 16 wavefronts 299 us at 82944 elements, 12 332, 8 379.  FP64 updates
// spill 112 registers when staged or at two wavefronts per SIMD (1465 us for 48000
// elements of degree 4, 990 as it is).
template <int N, int P> struct StepTune {
  static constexpr bool stage_ck = N >= 3, stage_update = N >= 3 && P != PREC_F64;
  static constexpr int wpb_ck = !stage_ck ? 1 : (P == PREC_F64 ? 8 : 16);
  static constexpr int wpb_update = !stage_update ? 1 : (N >= 4 ? 12 : 16);
  static constexpr int w_ck = P == PREC_F64 ? 2 : 4, w_face = P == PREC_F64 ? 2 : 4,
                       w_update = stage_update ? wpb_update / 4 : (P == PREC_F64 && N >= 4 ? 1 : 2);
  static constexpr int pd_ck = 4, pd_face = 6, pd_update = 4;
};

// this wavefront's elements: each XCD (block index mod 8) walks a contiguous range.
// The lane index is made opaque per element: what depends on it alone (table
// addresses, mixing weights) would else be kept in registers over the whole walk
// and spill.
template <int P, class F>
__device__ inline void for_elements(const StepArgs<P>& a, int wpb, F body) {
  const long long n = a.elist ? a.nlist : a.E, per = (n + 7) / 8;
  const long long x = blockIdx.x & 7, b = blockIdx.x >> 3, nb = gridDim.x >> 3;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (long long i = b + nb * wave; i < per; i += nb * wpb) {
    const long long k = x * per + i;
    if (k >= n) break;
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));
    body(a.elist ? (long long)a.elist[k] : k, lane & 63);   // (& 63: offsets fold into the loads)
  }
}

// copy of bytes (a multiple of 16) to LDS by the whole workgroup
__device__ inline void stage(void* dst, const void* src, int bytes) {
  typedef float V4 __attribute__((ext_vector_type(4)));
  for (int i = threadIdx.x; i < bytes / 16; i += blockDim.x) ((V4*)dst)[i] = ((const V4*)src)[i];
}

// Orders in which lanes and accumulator rows stand for quantities and modes.
// A product's output row r sits in lane group g, register i with r = 4 g + i
// (FP32 accumulators) or g + 4 i (FP64).  Operand rows fed in the order qperm /
// mperm come out with quantity 4 i + g, and with the modes of Steps::row, in the
// registers: just the k order of the next product's operand, which then needs no
// data movement.
template <class T> __host__ __device__ constexpr int qperm(int n) {
  return sizeof(T) == 8 ? n : (n & 3) * 4 + (n >> 2);
}
// mode of row (or column) n of 16-mode tile t
template <int N, int M> __host__ __device__ constexpr int mperm(int t, int n) {
  return 16 * t + (M == PREC_F32 || (M == PREC_X3 && t >= 2 * Steps<M, Dims<N>::L>::WIDE)
                       ? (n & 3) * 4 + (n >> 2)
                       : n);
}
// mode in register i of tile t of lane group g
template <int N, int M> __device__ inline int acc_mode(int t, int i, int g) {
  return M == PREC_X3 && t < 2 * Steps<M, Dims<N>::L>::WIDE ? 16 * t + 4 * g + i : 16 * t + 4 * i + g;
}
// operand of wide step s from registers in the order of Steps::row
template <int M, class T> __device__ inline typename Prec<M>::AF wide_op(const T* m, int s) {
  if constexpr (M == PREC_X3)
    return split8(m + 8 * s);
  else
    return m[s];
}
// fragment f of a packed matrix: one value per lane, or the three parts of a
// split fragment one after the other
template <int M>
__device__ inline typename Prec<M>::AF load_frag(const void* tab, int f, int lane) {
  if constexpr (M == PREC_X3) {
    const bf16x8* p = (const bf16x8*)tab + f * 192 + lane;
    return {p[0], p[64], p[128]};
  } else {
    return ((const typename Prec<M>::AF*)tab)[f * 64 + lane];
  }
}
template <int M> struct FragBytes {
  static constexpr int value = M == PREC_X3 ? 3072 : 64 * (int)sizeof(typename Prec<M>::AF);
};
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
// or its transpose (of lower degree only): the (e, tile, wide step) triples that
// are not zero, in the order they are issued.
template <int NMAX> struct TripleList {
  int n = 0;
  unsigned char e[NMAX] = {}, t[NMAX] = {}, s[NMAX] = {};
};
// K^e: inputs of R modes, NTO result tiles
template <int N, int M, int R, int NTO> constexpr auto k_list() {
  using ST = Steps<M, R>;
  TripleList<3 * (ST::WIDE + 1) * NTO> r;
  for (int s = 0; s < ST::WIDE; ++s)
    for (int t = 0; t < NTO; ++t)
      for (int e = 0; e < 3; ++e)
        if (ST::hi(s) > modes_upto(mode_degree(16 * t))) {
          r.e[r.n] = (unsigned char)e;
          r.t[r.n] = (unsigned char)t;
          r.s[r.n++] = (unsigned char)s;
        }
  return r;
}
// transposed: all MT result tiles, inputs of degree <= (largest of the tile) - 1
template <int N, int M> constexpr auto kt_list() {
  using ST = Steps<M, modes_upto(N - 1)>;
  TripleList<3 * (ST::WIDE + 1) * 3> r;
  constexpr int L = Dims<N>::L;
  for (int s = 0; s < ST::WIDE; ++s)
    for (int t = 0; t < Dims<N>::MT; ++t) {
      const int last = 16 * t + 15 < L ? 16 * t + 15 : L - 1;
      for (int e = 0; e < 3; ++e)
        if (ST::lo(s) < modes_upto(mode_degree(last) - 1)) {
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

// state of an element as row operand: quantity p in lane n, modes in registers
template <int N, int P, class T, int NR>
__device__ inline void load_state(const StepArgs<P>& a, long long e, T (&d)[NR], int lane) {
  using SL = Steps<MatForm<N, P>::value, Dims<N>::L>;
  constexpr int L = Dims<N>::L;
  const int g = lane >> 4, p = qperm<T>(lane & 15);
  const T* u = a.U9 + (e * 9 + (p < 9 ? p : 8)) * L;
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int l = SL::row(r, g);
    d[r] = u[l < L ? l : L - 1];
  }
  if (p == 9) {
    const double* ua = a.Ua + e * L;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int l = SL::row(r, g);
      d[r] = (T)ua[l < L ? l : L - 1];
    }
  }
#pragma unroll
  for (int r = 0; r < NR; ++r)
    if (p > 9 || SL::row(r, g) >= L) d[r] = T(0);
}

// values at the 64 points of chunk c: the product's rows are quantities, its
// columns 16 points; a transposition over the lane groups gives every lane one
// point
template <int N, int P, int PD, class T, int NR, class AF>
__device__ inline void nodal(const T (&d)[NR], const AF* dw, const void* Vw, const T* Vt, int c,
                             T (&u)[12], int lane) {
  constexpr int M = MatForm<N, P>::value;
  using PR = Prec<M>;
  using SL = Steps<M, Dims<N>::L>;
  constexpr int WL = SL::WIDE;
  typename PR::Acc C[4];
  zero_C<M, 4>(C);
  stream<PD, 4 * WL, AF>(
      [&](int k) { return load_frag<M>(Vw, (c * 4 + k % 4) * WL + k / 4, lane); },
      [&](int k, const AF& b) { C[k % 4] = PR::mma(dw[k / 4], b, C[k % 4]); });
  if constexpr (SL::TAIL) {
#pragma unroll
    for (int t = 0; t < 4; ++t) C[t] = Prec<P>::mma(d[NR - 1], Vt[(c * 4 + t) * 64 + lane], C[t]);
  }
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    T x0 = C[0][i], x1 = C[1][i], x2 = C[2][i], x3 = C[3][i];
    transpose4(x0, x1, x2, x3);
    u[4 * i] = x0;
    u[4 * i + 1] = x1;
    u[4 * i + 2] = x2;
    u[4 * i + 3] = x3;
  }
}

// mix the quantities of R modes (quantities in registers; As: the matrices of the
// three directions), then contract with K^e: NTO tiles out, modes in rows.  DAM:
// tiles past the modes of degree < N hold the damage row (register 2) only.
template <int N, int P, int R, int NTO, bool DAM, int PD, class Acc, class T>
__device__ inline void mix_contract(const Acc* in, const T (&As)[3][3], const void* Kw, const T* Kt,
                                    Acc* out, int lane) {
  constexpr int M = MatForm<N, P>::value;
  using PR = Prec<M>;
  using PA = Prec<P>;
  using AF = typename PR::AF;
  using ST = Steps<M, R>;
  constexpr int NTI = (R + 15) / 16, R1 = modes_upto(N - 1), NT1 = (R1 + 15) / 16;
  constexpr int WL = Steps<M, Dims<N>::L>::WIDE;
  constexpr auto list = k_list<N, M, R, NTO>();
  constexpr int NY = ST::NREG > 4 * NTI ? ST::NREG : 4 * NTI;
#pragma unroll
  for (int t = 0; t < NTO; ++t) {
#pragma unroll
    for (int k = 0; k < 4; ++k) out[t][k] = 0;
  }
  T Y[3][NY];
  AF Yw[3][ST::WIDE > 0 ? ST::WIDE : 1];
#pragma unroll
  for (int ee = 0; ee < 3; ++ee) {
#pragma unroll
    for (int k = 0; k < NY; ++k) Y[ee][k] = T(0);
#pragma unroll
    for (int t = 0; t < NTI; ++t) {
      Acc y;
#pragma unroll
      for (int k = 0; k < 4; ++k) y[k] = 0;
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        if (DAM && 16 * t >= R1 && i < 2) continue;
        y = PA::mma(in[t][i], As[ee][i], y);
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) Y[ee][4 * t + k] = y[k];
    }
#pragma unroll
    for (int s = 0; s < ST::WIDE; ++s) Yw[ee][s] = wide_op<M>(Y[ee], s);
  }
  stream<PD, list.n, AF>(
      [&](int k) { return load_frag<M>(Kw, (list.e[k] * NT1 + list.t[k]) * WL + list.s[k], lane); },
      [&](int k, const AF& aa) {
        Acc& z = out[list.t[k]];
        z = PR::mma(aa, Yw[list.e[k]][list.s[k]], z);
      });
  if constexpr (ST::TAIL) {
#pragma unroll
    for (int ee = 0; ee < 3; ++ee)
#pragma unroll
      for (int t = 0; t < NTO; ++t)
        out[t] = PA::mma(Kt[(ee * NT1 + t) * 64 + lane], Y[ee][ST::NREG - 1], out[t]);
  }
}

template <int N, int P> struct CkLDS {
  using T = typename Prec<P>::T;
  // fragments of the derivative matrix, padded by 16 bytes each: a column's
  // fragments then start on different banks
  static constexpr int FS = 64 + 16 / sizeof(T);
  alignas(16) T dz[Deriv<N>::NF * FS];
  alignas(16) T r[Dims<N>::NCH * 64];                   // damage rate at the points
  T al[64];                                             // its projection, the damage row of D^1
  T ext[64];                                            // sums of the tangent
  T tg[48];                                             // cell-averaged tangent / rho, 0, 1/2, 1
};

// Prediction (Appendix A.1, Eqs. CKIter, CKIter-ref-matrix, CKIter-ref-source;
// 312132 elements of degree 4: 1340 us, issue of vector ALUs and FP32 products for
// 62 % of it; time-point states from dense FP32 products 4640):
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
__device__ inline void ck_element(const StepArgs<P>& a, long long e, CkLDS<N, P>& S,
                                  const void* Vw, const typename Prec<P>::T* Vt, const void* Kw,
                                  const typename Prec<P>::T* Kt, int lane) {
  constexpr int M = MatForm<N, P>::value;
  using PR = Prec<M>;
  using PA = Prec<P>;
  using T = typename PA::T;
  using AF = typename PR::AF;
  using Acc = typename PR::Acc;
  using DM = Dims<N>;
  using DV = Deriv<N>;
  constexpr int L = DM::L, Q = DM::Q, NCH = DM::NCH, MT = DM::MT;
  using SL = Steps<M, L>;
  constexpr int WL = SL::WIDE, NR = SL::NREG, PD = M == PREC_X3 ? 1 : StepTune<N, P>::pd_ck;
  constexpr int R1 = modes_upto(N - 1), R3 = modes_upto(N - 2), R4 = modes_upto(N - 3);
  constexpr int NT1 = (R1 + 15) / 16;
  const int n = lane & 15, g = lane >> 4;
  const int p = qperm<T>(n);

  T d0[NR];
  load_state<N, P>(a, e, d0, lane);
  const Law<T> law{a.amax, a.smin};
  const StepMat<T> m = LW::constants(load_mat<T>(a.mat + e * 8));
  constexpr int FS = CkLDS<N, P>::FS, VW = 16 / sizeof(T);
  typedef T TV __attribute__((ext_vector_type(VW)));
  for (int i = lane; i < DV::NF * FS / VW; i += 64) ((TV*)S.dz)[i] = TV(T(0));
  wave_sync();
  // tile t of a quantities-in-lanes result of order o, c[0..3] in registers
  typedef T T4 __attribute__((ext_vector_type(4), aligned(16)));
  auto put_tile = [&](int o, int t, const T4& c, int rows) {
    const int j = DV::col(o, p);
    T* d = S.dz + DV::tile0(j) * FS + (j & 15);
    if (M == PREC_X3 && t < 2 * WL) {
      if (16 * t + 4 * g >= rows) return;
#pragma unroll
      for (int i = 0; i < 4; ++i) d[(4 * t + g) * FS + 16 * i] = c[i];
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (16 * t + 4 * i < rows) d[(4 * t + i) * FS + 16 * g] = c[i];
    }
  };
  if (p < 10) {
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      T4 c;
#pragma unroll
      for (int i = 0; i < 4; ++i) c[i] = 4 * t + i < NR ? d0[4 * t + i < NR ? 4 * t + i : 0] : T(0);
      put_tile(0, t, c, L);
    }
  }
  AF d0w[WL > 0 ? WL : 1];
#pragma unroll
  for (int s = 0; s < WL; ++s) d0w[s] = wide_op<M>(d0, s);

  // nodal values at t_n: the product's rows are quantities, its columns 16
  // points; a transposition over the lane groups gives every lane one point
  T acc[LW::NACC];
#pragma unroll
  for (int k = 0; k < LW::NACC; ++k) acc[k] = T(0);
#pragma unroll 1
  for (int c = 0; c < NCH; ++c) {
    T u[12];
    nodal<N, P, PD>(d0, d0w, Vw, Vt, c, u, lane);
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
    S.tg[lane] = lane < 42 ? v * m.ir : (lane == 43 ? T(0.5) : (lane == 44 ? T(1) : T(0)));
  }
  // damage source at t_n projected on the modes, one mode per lane
  {
    T s = T(0);
    if (lane < L) {
      const T4* pw = (const T4*)a.Psrc + lane;
      const T4* rr = (const T4*)S.r;
#pragma unroll 8
      for (int k = 0; k < (Q + 3) / 4; ++k) {
        const T4 x = pw[k * L], y = rr[k];
        s += x[0] * y[0] + x[1] * y[1] + x[2] * y[2] + x[3] * y[3];
      }
      S.dz[(lane >> 2) * FS + 16 * (lane & 3) + 10] = s;          // column 10
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
      As[ee][i] = (T)a.geo[e * 16 + ee * 3] * w[0] + (T)a.geo[e * 16 + ee * 3 + 1] * w[1] +
                  (T)a.geo[e * 16 + ee * 3 + 2] * w[2];
  }

  auto kfrag = [&](int ee, int t, int s) { return load_frag<M>(Kw, (ee * NT1 + t) * WL + s, lane); };
  auto ktail = [&](int ee, int t) { return Kt[(ee * NT1 + t) * 64 + lane]; };
  // contract R modes, then mix: NTO tiles of 16 modes, quantities in rows
  auto contract_mix = [&](const T* in, const AF* inw, auto rows, auto nto, Acc* out) {
    constexpr int R = decltype(rows)::value, NTO = decltype(nto)::value;
    using ST = Steps<M, R>;
    constexpr auto list = k_list<N, M, R, NTO>();
    Acc Z[3][NTO];
#pragma unroll
    for (int ee = 0; ee < 3; ++ee) zero_C<M, NTO>(Z[ee]);
    stream<PD, list.n, AF>([&](int k) { return kfrag(list.e[k], list.t[k], list.s[k]); },
                           [&](int k, const AF& b) {
                             Acc& z = Z[list.e[k]][list.t[k]];
                             z = PR::mma(inw[list.s[k]], b, z);
                           });
    if constexpr (ST::TAIL) {
#pragma unroll
      for (int ee = 0; ee < 3; ++ee)
#pragma unroll
        for (int t = 0; t < NTO; ++t) Z[ee][t] = PA::mma(in[ST::NREG - 1], ktail(ee, t), Z[ee][t]);
    }
#pragma unroll
    for (int t = 0; t < NTO; ++t) {
#pragma unroll
      for (int k = 0; k < 4; ++k) out[t][k] = 0;
    }
#pragma unroll
    for (int ee = 0; ee < 3; ++ee)
#pragma unroll
      for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int t = 0; t < NTO; ++t) out[t] = PA::mma(As[ee][i], Z[ee][t][i], out[t]);
  };
  // quantities-in-registers result of order o to the derivative matrix
  auto put_regs = [&](const Acc* R, int o, int rows, int nt) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const int pq = 4 * k + g;
      if (pq >= 9) continue;
      const int j = DV::col(o, pq), f0 = DV::tile0(j) * FS + (j & 15);
#pragma unroll
      for (int t = 0; t < MT; ++t) {
        if (t >= nt) continue;
        const int l = mperm<N, M>(t, n);
        if (l < rows) S.dz[f0 + (l >> 2) * FS + 16 * (l & 3)] = R[t][k];
      }
    }
  };
  // quantities-in-lanes result of order o
  auto put_lanes = [&](const Acc* C, int o, int rows) {
    if (p >= 9) return;
#pragma unroll
    for (int t = 0; t < MT; ++t)
      if (16 * t < rows) put_tile(o, t, T4{C[t][0], C[t][1], C[t][2], C[t][3]}, (rows + 3) & ~3);
  };

  // order 1: all modes in, degree <= N - 1 out; then the damage row
  Acc D1[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int k = 0; k < 4; ++k) D1[t][k] = 0;
  contract_mix(d0, d0w, std::integral_constant<int, L>{}, std::integral_constant<int, NT1>{}, D1);
  put_regs(D1, 1, R1, NT1);
  if constexpr (N >= 2) {
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      const T v = S.al[mperm<N, M>(t, n)];
      if (g == 1) D1[t][2] = v;
    }
    // order 2: the damage row brings all modes, degree <= N - 1 out
    Acc D2[NT1];
    mix_contract<N, P, L, NT1, true, PD>(D1, As, Kw, Kt, D2, lane);
    put_lanes(D2, 2, R1);
    if constexpr (N >= 3) {
      using S2 = Steps<M, R1>;
      constexpr int N2 = S2::NREG > 4 * NT1 ? S2::NREG : 4 * NT1;
      T d2[N2];
#pragma unroll
      for (int r = 0; r < N2; ++r) d2[r] = r < 4 * NT1 ? D2[r >> 2][r & 3] : T(0);
      AF d2w[S2::WIDE];
#pragma unroll
      for (int s = 0; s < S2::WIDE; ++s) d2w[s] = wide_op<M>(d2, s);
      Acc D3[1];
      contract_mix(d2, d2w, std::integral_constant<int, R1>{}, std::integral_constant<int, 1>{}, D3);
      put_regs(D3, 3, R3, 1);
      if constexpr (N >= 4) {
        Acc D4[1];
        mix_contract<N, P, R3, 1, true, PD>(D3, As, Kw, Kt, D4, lane);
        put_lanes(D4, 4, R4);
      }
    }
  }
  wave_sync();
  T* out = a.Dz + (size_t)e * DV::NF * 64;
  constexpr int NV = DV::NF * 64 / VW;
#pragma unroll
  for (int k = 0; k < (NV + 63) / 64; ++k) {
    const int idx = lane + 64 * k;
    if (idx < NV) ((TV*)out)[idx] = ((const TV*)S.dz)[idx + idx / (64 / VW)];   // (padding skipped)
  }
}

template <int N, int P> struct CkTabs {     // bytes of the matrices in LDS
  static constexpr int M = MatForm<N, P>::value;
  using T = typename Prec<P>::T;
  using SL = Steps<M, Dims<N>::L>;
  static constexpr int NT1 = (modes_upto(N - 1) + 15) / 16;
  static constexpr int vw = Dims<N>::NCH * 4 * SL::WIDE * FragBytes<M>::value;
  static constexpr int vt = SL::TAIL ? Dims<N>::NCH * 4 * 64 * (int)sizeof(T) : 0;
  static constexpr int kw = 3 * NT1 * SL::WIDE * FragBytes<M>::value;
  static constexpr int kt = SL::TAIL ? 3 * NT1 * 64 * (int)sizeof(T) : 0;
  static constexpr int all = StepTune<N, P>::stage_ck ? vw + vt + kw + kt : 0;
  static constexpr int wpb = StepTune<N, P>::wpb_ck;
  static constexpr int bytes = all + wpb * (int)sizeof(CkLDS<N, P>);
  static_assert(bytes <= 163840, "the workgroup's LDS");
};

template <int N, int P, class LW>
__global__ __launch_bounds__((64 * CkTabs<N, P>::wpb))
__attribute__((amdgpu_waves_per_eu(StepTune<N, P>::w_ck))) void k_ck(StepArgs<P> a) {
  using T = typename Prec<P>::T;
  using TB = CkTabs<N, P>;
  __shared__ __attribute__((aligned(64))) char smem[TB::bytes];
  if constexpr (StepTune<N, P>::stage_ck) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    char* tab = smem;
    stage(tab, a.Vw, TB::vw);
    stage(tab + TB::vw, a.Vt, TB::vt);
    stage(tab + TB::vw + TB::vt, a.Kw, TB::kw);
    stage(tab + TB::vw + TB::vt + TB::kw, a.Kt, TB::kt);
    __syncthreads();
    CkLDS<N, P>& S = ((CkLDS<N, P>*)(smem + TB::all))[wave];
    for_elements(a, TB::wpb, [&](long long e, int lane) {
      ck_element<N, P, LW>(a, e, S, tab, (const T*)(tab + TB::vw), tab + TB::vw + TB::vt,
                           (const T*)(tab + TB::vw + TB::vt + TB::kw), lane);
      wave_sync();
    });
  } else {
    CkLDS<N, P>& S = *(CkLDS<N, P>*)smem;
    for_elements(a, 1, [&](long long e, int lane) {
      ck_element<N, P, LW>(a, e, S, a.Vw, a.Vt, a.Kw, a.Kt, lane);
    });
  }
}

// value of column j (compile time) of a transposed product: C[c][k][i] holds row
// 4 k + i (FP32 accumulators) or k + 4 i (FP64) of tile c
template <class T, class Acc> __device__ inline T column(const Acc (*C)[4], int j) {
  const int m = j & 15;
  return sizeof(T) == 8 ? C[j >> 4][m & 3][m >> 2] : C[j >> 4][m >> 2][m & 3];
}

// the derivative matrix of an element as row operand, tile by tile (columns in
// lanes, rows in the order of Steps::row)
template <int N, int M, class T, int NT, int NR>
__device__ inline void load_deriv(const T* dze, T (&d)[NT][NR], int lane) {
  using DV = Deriv<N>;
  const int n = lane & 15, g = lane >> 4;
#pragma unroll
  for (int ct = 0; ct < NT; ++ct) {
    const int rows = DV::rows(16 * ct), steps = DV::steps(ct);
    const T* t = dze + DV::frag0(ct) * 64 + n;
    if constexpr (M == PREC_X3) {
      const bool tail = rows % 32 <= 4;                // one FP32 step more
      const int W = tail ? rows / 32 : 1;
#pragma unroll
      for (int r = 0; r < 8 * W; ++r) {
        const int f = 4 * (r >> 2) + g;
        const T v = t[(f < steps ? f : 0) * 64 + (r & 3) * 16];
        d[ct][r] = f < steps ? v : T(0);
      }
      if (tail) d[ct][8 * W] = t[8 * W * 64 + 16 * g];
    } else {
#pragma unroll
      for (int r = 0; r < NR; ++r)
        if (r < steps) d[ct][r] = t[r * 64 + 16 * g];
    }
  }
}

template <int N, int P> struct UpdLDS {
  using T = typename Prec<P>::T;
  static constexpr int RS = 64 + 16 / sizeof(T);
  // degree 4: 12 registers fewer in the point loop, so that three wavefronts fit a
  // SIMD without spills
  static constexpr bool KEEP = MatForm<N, P>::value == PREC_X3 && N >= 4;
  alignas(16) T X[10 * RS];       // time integrals at the points of one chunk, [quantity][point]
  T al[2][64];                    // damage row: projected source, lifted flux
  alignas(16) T U[KEEP ? Dims<N>::MT * 256 : 4];        // lifted fluxes, during the point loop
};

// Modes of a face flux on its face: orthonormal polynomials of degree <= N in the
// plane.  The basis restricted to a face is such a polynomial, so the lift of
// the (N + 1)^2 point values is the lift of their NM2 projections.  At degree 1 the
// point values themselves (see PointStiffness).
template <int N> struct FaceModes {
  static constexpr int value = N == 1 ? 4 : (N + 1) * (N + 2) / 2;
};
// Degree 1 applies the stiffness to the point values, too, not to the projection.  There
// it acts on one mode and the lift would on three: what FP32 leaves of so few entries
// does not average out, and the waves after four steps were 14 % further from 64 bits
// than with point sums (3.0e-7 against 2.6e-7, rms over 100 states).  The products are as
// many (12 and 4 against 16 and 3, the 8 points being two of a chunk's 16 steps).
template <int N> struct PointStiffness {
  static constexpr bool value = N == 1;
  static constexpr int steps = 4 * ((Dims<N>::Q + 15) / 16);   // of a chunk's 16, those with points
};
// Modes projected one per 16-row tile by matrix products; the few left over
// (3 at degree 4, 4 at degree 3), which only the damage source needs, by a sum
// over the lanes.
template <int N> struct ProjTiles {
  static constexpr int L = Dims<N>::L;
  static constexpr int MTP = L > 16 && L % 16 <= 4 ? L / 16 : Dims<N>::MT;
  static constexpr int LEFT = L > 16 * MTP ? L - 16 * MTP : 0;
};

// Corrector (Appendix A.2, Eqs. 2nd term, 3rd term, rhs term, time-integrated;
// 312132 elements of degree 4: 1950 us, bound by dependency latency at three
// wavefronts per SIMD; volume and lift kernels on time-point states 5940):
// lift of the four face fluxes, volume and source terms, update.
//
// The derivative matrix is evaluated at 64 points at a time (columns in rows of
// the product, transposed so that a lane holds its point's columns); Taylor sums,
// stress and damage rate at every time point are summed in time per point.  The
// flux is linear in velocity and stress and the projection of any point values
// followed by the modal stiffness is the quadrature with S^e, so the ten time
// integrals are projected once (one contraction over the points in place of
// three) and the stiffness, of L x modes of degree < N, and the element's
// Jacobian act on modes.
template <int N, int P, class LW>
__device__ inline void update_element(const StepArgs<P>& a, long long e, const int* fmap,
                                      const typename Prec<P>::T* fflux, UpdLDS<N, P>& S,
                                      const void* Vw, const typename Prec<P>::T* Vt,
                                      const void* Pw, const void* Ktw, int lane) {
  constexpr int M = MatForm<N, P>::value;
  using PR = Prec<M>;
  using PA = Prec<P>;
  using T = typename PA::T;
  using AF = typename PR::AF;
  using Acc = typename PR::Acc;
  using DM = Dims<N>;
  using DV = Deriv<N>;
  constexpr int L = DM::L, Q = DM::Q, Nt = DM::Nt, NCH = DM::NCH, MT = DM::MT;
  constexpr int WL = Steps<M, L>::WIDE, NT = DV::NT;
  constexpr int NM2 = FaceModes<N>::value, MTP = ProjTiles<N>::MTP, LEFT = ProjTiles<N>::LEFT;
  constexpr int PD = M == PREC_X3 ? 1 : StepTune<N, P>::pd_update, PDL = N >= 4 ? 4 : 1;
  using SL = UpdLDS<N, P>;
  const int n = lane & 15, g = lane >> 4;
  const int p = qperm<T>(n);

  // the derivative matrix as row operand: tile ct in dzw[ct], dzt[ct]
  T dzr[NT][Steps<M, L>::NREG];
  load_deriv<N, M>(a.Dz + (size_t)e * DV::NF * 64, dzr, lane);
  // the four face fluxes (integrals of the finer cluster, cleared, under local
  // time stepping), quantity p in lane n, scaled; negated where the element is
  // the face's first side
  constexpr int NF2 = M == PREC_X3 ? 4 : (NM2 + 3) / 4;
  T fv[4][NF2];
  int sp[4];
#pragma unroll
  for (int f = 0; f < 4; ++f) {
    const int fm = fmap[e * 4 + f];
    sp[f] = conn_perm(a.conn[(e * 4 + f) * 2 + 1]);
    const int nb = a.conn[(e * 4 + f) * 2];
    const bool fine = a.lts_c > 0 && nb >= 0 && a.ecl[nb] == a.lts_c - 1;
    const T sc = (T)((fm & 1 ? 1.0 : -1.0) * a.fgeo[(e * 4 + f) * 4 + 3] * (fine ? 1.0 : a.dt));
    T* fl = (fine ? a.facc : (T*)fflux) + (size_t)(fm >> 1) * NM2 * 10 + (p < 10 ? p : 9);
#pragma unroll
    for (int r = 0; r < NF2; ++r) {
      const int i = M == PREC_X3 ? 4 * g + r : 4 * r + g;     // face mode
      fv[f][r] = fl[(i < NM2 ? i : NM2 - 1) * 10];
    }
    if (fine) {
      wave_sync();
#pragma unroll
      for (int r = 0; r < NF2; ++r) {
        const int i = M == PREC_X3 ? 4 * g + r : 4 * r + g;
        if (i < NM2 && p < 10) fl[i * 10] = T(0);
      }
    }
#pragma unroll
    for (int r = 0; r < NF2; ++r) {
      const int i = M == PREC_X3 ? 4 * g + r : 4 * r + g;
      fv[f][r] = (i < NM2 && p < 10) ? sc * fv[f][r] : T(0);
    }
  }
  const Law<T> law{a.amax, a.smin};
  const StepMat<T> m = LW::constants(load_mat<T>(a.mat + e * 8));
  Acc U[MT];
  zero_C<M, MT>(U);
  if constexpr (M == PREC_X3) {
    // two faces per 32-term step: modes of one, then modes of the other
    typedef __bf16 bf16q __attribute__((ext_vector_type(4)));
    const bf16q* Lf[4];
    AF b[2];
#pragma unroll
    for (int f = 0; f < 4; ++f) Lf[f] = (const bf16q*)a.Rw + (size_t)(f * 6 + sp[f]) * MT * 192 + lane;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      T v[8];
#pragma unroll
      for (int r = 0; r < 8; ++r) v[r] = fv[2 * h + (r >> 2)][r & 3];
      b[h] = split8(v);
    }
    stream<PDL, 2 * MT, AF>(
        [&](int k) {
          const bf16q *La = Lf[k / MT * 2] + k % MT * 192, *Lb = Lf[k / MT * 2 + 1] + k % MT * 192;
          AF f;
          f.h = __builtin_shufflevector(La[0], Lb[0], 0, 1, 2, 3, 4, 5, 6, 7);
          f.m = __builtin_shufflevector(La[64], Lb[64], 0, 1, 2, 3, 4, 5, 6, 7);
          f.l = __builtin_shufflevector(La[128], Lb[128], 0, 1, 2, 3, 4, 5, 6, 7);
          return f;
        },
        [&](int k, const AF& f) { U[k % MT] = PR::mma(b[k / MT], f, U[k % MT]); });
  } else {
#pragma unroll
    for (int f = 0; f < 4; ++f) {
      const AF* Lf = (const AF*)a.Rw + (size_t)(f * 6 + sp[f]) * MT * NF2 * 64 + lane;
      stream<PD, MT * NF2, AF>([&](int k) { return Lf[((k % MT) * NF2 + k / MT) * 64]; },
                               [&](int k, const AF& b) {
                                 U[k % MT] = PR::mma(fv[f][k / MT], b, U[k % MT]);
                               });
    }
  }
  if constexpr (SL::KEEP) {
#pragma unroll
    for (int t = 0; t < MT; ++t) ((Acc*)S.U)[64 * t + lane] = U[t];
  }
  AF dzw[NT][WL];
#pragma unroll
  for (int ct = 0; ct < NT; ++ct)
#pragma unroll
    for (int s = 0; s < WL; ++s)
      if (M != PREC_X3 || DV::rows(16 * ct) > 4) dzw[ct][s] = wide_op<M>(dzr[ct], s);

  constexpr bool PS = PointStiffness<N>::value;
  Acc Z[3][MT];
#pragma unroll
  for (int ee = 0; ee < 3; ++ee) zero_C<M, MT>(Z[ee]);
  typename PA::Acc X[MTP];
  zero_C<P, MTP>(X);
  T left[LEFT > 0 ? LEFT : 1];
#pragma unroll
  for (int k = 0; k < (LEFT > 0 ? LEFT : 1); ++k) left[k] = T(0);
#pragma unroll 1
  for (int c = 0; c < NCH; ++c) {
    T x[10];
#pragma unroll
    for (int k = 0; k < 10; ++k) x[k] = T(0);
    {
      Acc C[NT][4];
#pragma unroll
      for (int ct = 0; ct < NT; ++ct) zero_C<M, 4>(C[ct]);
      stream<PD, 4 * WL, AF>(
          [&](int k) { return load_frag<M>(Vw, (c * 4 + k % 4) * WL + k / 4, lane); },
          [&](int k, const AF& b) {
            const int s = k / 4, t = k % 4;
            if constexpr (M == PREC_X3) {
#pragma unroll
              for (int q = 0; q < 6; ++q)
#pragma unroll
                for (int ct = 0; ct < NT; ++ct)
                  if (DV::rows(16 * ct) > 4) C[ct][t] = PR::product(q, dzw[ct][s], b, C[ct][t]);
            } else {
#pragma unroll
              for (int ct = 0; ct < NT; ++ct)
                if (s < DV::steps(ct)) C[ct][t] = PR::mma(dzw[ct][s], b, C[ct][t]);
            }
          });
      if constexpr (M == PREC_X3) {
        // FP32 steps: rows 32..35 of tile 0 at degree 4, the four rows of the
        // last tile at degree 3 (its own first four rows of the matrix)
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) {
          const int rows = DV::rows(16 * ct);
          if (rows % 32 > 4) continue;
#pragma unroll
          for (int t = 0; t < 4; ++t)
            C[ct][t] = PA::mma(dzr[ct][rows / 32 * 8],
                               Vt[((rows > 32 ? 0 : NCH * 4 * Steps<M, L>::TAIL) + c * 4 + t) * 64 + lane],
                               C[ct][t]);
        }
      }
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
        const T gz = a.gamma[z];
        T u[10];   // (the velocity is not needed per time point)
#pragma unroll
        for (int k = 0; k < 6; ++k) {
          T v = column<T>(C, DV::col(N, k));
#pragma unroll
          for (int i = N - 1; i >= 0; --i) v = column<T>(C, DV::col(i, k)) + a.hzi[z][i] * v;
          u[k] = v;
        }
        u[9] = column<T>(C, 9) + a.hzi[z][0] * column<T>(C, 10);
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
    if constexpr (LEFT > 0) {
#pragma unroll
      for (int k = 0; k < LEFT; ++k) left[k] += x[9] * a.PXleft[(c * LEFT + k) * 64 + lane];
    }
    wave_sync();
#pragma unroll
    for (int k = 0; k < 10; ++k) S.X[k * SL::RS + lane] = x[k];
    wave_sync();
    // projection: X += P_c x, modes in rows, quantities in columns
    typedef T T4 __attribute__((ext_vector_type(4), aligned(16)));
    const T* xs = S.X + (p < 10 ? p : 9) * SL::RS;
    if constexpr (M == PREC_X3) {
      AF xw[2];
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const T4 lo = *(const T4*)(xs + 32 * s + 8 * g), hi = *(const T4*)(xs + 32 * s + 8 * g + 4);
        const T v[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        xw[s] = split8(v);
      }
      stream<1, 2 * MTP, AF>(
          [&](int k) { return load_frag<M>(Pw, c * 2 * MTP + k, lane); },
          [&](int k, const AF& aa) { X[k % MTP] = PR::mma(aa, xw[k / MTP], X[k % MTP]); });
    } else {
      T4 xv[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) xv[k] = *(const T4*)(xs + 16 * k + 4 * g);
      constexpr int NS = PS ? PointStiffness<N>::steps : 16;
      stream<PD, NS * MTP, AF>(
          [&](int k) { return load_frag<M>(Pw, c * 16 * MTP + k, lane); },
          [&](int k, const AF& aa) {
            const int s = k / MTP;
            X[k % MTP] = PR::mma(aa, xv[s >> 2][s & 3], X[k % MTP]);
          });
      if constexpr (PS) {
        static_assert(NCH == 1 && MT == 1, "one chunk, one tile");
        stream<PD, 3 * NS, AF>([&](int k) { return load_frag<M>(Ktw, k, lane); },
                               [&](int k, const AF& b) {
                                 const int s = k / 3;
                                 Z[k % 3][0] = PR::mma(xv[s >> 2][s & 3], b, Z[k % 3][0]);
                               });
      }
    }
  }
  // the projected source (times dt) leaves through LDS, one mode per lane
  if (p == 9) {
#pragma unroll
    for (int t = 0; t < MTP; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) S.al[0][acc_mode<N, M>(t, i, g)] = X[t][i];
  }
  if constexpr (LEFT > 0) reduce_to_lds(left, S.al[0] + 16 * MTP, lane);
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
  if constexpr (!PS) {
    using S1 = Steps<M, modes_upto(N - 1)>;
    constexpr int NX = S1::NREG > 4 * MTP ? S1::NREG : 4 * MTP;
    T xm[NX];
#pragma unroll
    for (int r = 0; r < NX; ++r) xm[r] = r < 4 * MTP ? X[r >> 2][r & 3] : T(0);
    AF xw[S1::WIDE];
#pragma unroll
    for (int s = 0; s < S1::WIDE; ++s) xw[s] = wide_op<M>(xm, s);
    constexpr auto list = kt_list<N, M>();
    stream<PD, list.n, AF>([&](int k) { return load_frag<M>(Ktw, k, lane); },
                           [&](int k, const AF& b) {
                             Acc& z = Z[list.e[k]][list.t[k]];
                             z = PR::mma(xw[list.s[k]], b, z);
                           });
  }
  {
    const T rs = (T)a.dt * (p >= 6 ? m.ir : T(1));
    if constexpr (SL::KEEP) {
#pragma unroll
      for (int t = 0; t < MT; ++t) U[t] = ((const Acc*)S.U)[64 * t + lane];
    }
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

template <int N, int P> struct UpdTabs {    // bytes of the matrices in LDS
  static constexpr int M = MatForm<N, P>::value;
  using T = typename Prec<P>::T;
  using SL = Steps<M, Dims<N>::L>;
  // FP32 steps of the evaluation: the leftover rows of tile 0, then the last tile
  static constexpr int ntail =
      M == PREC_X3 ? SL::TAIL + (Deriv<N>::rows(16 * (Deriv<N>::NT - 1)) <= 4) : 0;
  static constexpr int vw = Dims<N>::NCH * 4 * SL::WIDE * FragBytes<M>::value;
  static constexpr int vt = ntail * Dims<N>::NCH * 4 * 64 * (int)sizeof(T);
  static constexpr int pw =
      Dims<N>::NCH * (M == PREC_X3 ? 2 : 16) * ProjTiles<N>::MTP * FragBytes<M>::value;
  static constexpr int kw = kt_list<N, M>().n * FragBytes<M>::value;
  static constexpr int all = StepTune<N, P>::stage_update ? vw + vt + pw + kw : 0;
  static constexpr int wpb = StepTune<N, P>::wpb_update;
  static constexpr int bytes = all + wpb * (int)sizeof(UpdLDS<N, P>);
  static_assert(bytes <= 163840, "the workgroup's LDS");
};

template <int N, int P, class LW>
__global__ __launch_bounds__((64 * UpdTabs<N, P>::wpb))
__attribute__((amdgpu_waves_per_eu(StepTune<N, P>::w_update))) void k_update(
    StepArgs<P> a, const int* fmap, const typename Prec<P>::T* fflux) {
  using T = typename Prec<P>::T;
  using TB = UpdTabs<N, P>;
  __shared__ __attribute__((aligned(64))) char smem[TB::bytes];
  if constexpr (StepTune<N, P>::stage_update) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    char* tab = smem;
    stage(tab, a.Vw, TB::vw);
    stage(tab + TB::vw, a.Vt, TB::vt);
    stage(tab + TB::vw + TB::vt, a.PXw, TB::pw);
    stage(tab + TB::vw + TB::vt + TB::pw, a.Ktw, TB::kw);
    __syncthreads();
    UpdLDS<N, P>& S = ((UpdLDS<N, P>*)(smem + TB::all))[wave];
    for_elements(a, TB::wpb, [&](long long e, int lane) {
      update_element<N, P, LW>(a, e, fmap, fflux, S, tab, (const T*)(tab + TB::vw),
                               tab + TB::vw + TB::vt, tab + TB::vw + TB::vt + TB::pw, lane);
      wave_sync();
    });
  } else {
    UpdLDS<N, P>& S = *(UpdLDS<N, P>*)smem;
    for_elements(a, 1, [&](long long e, int lane) {
      update_element<N, P, LW>(a, e, fmap, fflux, S, a.Vw, a.Vt, a.PXw, a.Ktw, lane);
    });
  }
}

// ---- Picard-iteration predictor --------------------------------------------------
// The alternative to the linearised Cauchy-Kovalevskaya prediction named in the
// paper's Discussion (Section 5.1).  The element-local evolution that the
// recursion differentiates, taken in strong form without linearisation,
//   dU/dt = R(U) = - sum_e K^e P G^e(U) + P r(U),
//   G^e = sum_d Theta^-1_ed F^d(V U) at the volume points, P the projection,
// is solved on the Gauss-Legendre time points by Picard iteration of the
// collocation equations U_z = U^n + dt sum_j Om_zj R(U_j), from U_z = U^n.
template <int P> struct PicardArgs {
  using T = typename Prec<P>::T;
  int iters;
  T om[8][8];
};

template <int N, int P> struct PicardLDS {
  using T = typename Prec<P>::T;
  static constexpr int RS = 64 + 16 / sizeof(T);
  alignas(16) T X[10 * RS];       // velocity, stress and damage rate at the points of one chunk
  T al[64];                       // projected damage rate
};

template <int N, int P> struct PicardTabs {     // bytes of the matrices in LDS, launch shape
  static constexpr int M = MatForm<N, P>::value;
  static constexpr bool staged = M == PREC_X3;
  static constexpr int vw = CkTabs<N, P>::vw, vt = CkTabs<N, P>::vt, kw = CkTabs<N, P>::kw,
                       kt = CkTabs<N, P>::kt;
  static constexpr int pw = Dims<N>::NCH * (M == PREC_X3 ? 2 : 16) * Dims<N>::MT * FragBytes<M>::value;
  static constexpr int all = staged ? vw + vt + kw + kt + pw : 0;
  static constexpr int wpb = !staged ? 1 : (N >= 4 ? 8 : 12);
  static constexpr int waves = staged ? wpb / 4 : (P == PREC_F64 && N >= 4 ? 1 : 2);
  static constexpr int bytes = all + wpb * (int)sizeof(PicardLDS<N, P>);
  static_assert(bytes <= 163840, "the workgroup's LDS");
};

// The iterate and the next one stay in registers as row operands.  The flux is
// linear in velocity and stress, so they and the damage rate are projected once
// per evaluation, mixed as in the corrector and contracted with K^e on modes (as
// even orders of the recursion).  A contraction of the 9 fluxes of each reference
// direction with K^e P over the points, the states in LDS, took 730 us for 10368
// elements of degree 3, against 265 us.
template <int N, int P, class LW>
__device__ inline void picard_element(const StepArgs<P>& a, const PicardArgs<P>& pa, long long e,
                                      PicardLDS<N, P>& S, const void* Vw,
                                      const typename Prec<P>::T* Vt, const void* Kw,
                                      const typename Prec<P>::T* Kt, const void* Pw, int lane) {
  constexpr int M = MatForm<N, P>::value;
  using PR = Prec<M>;
  using PA = Prec<P>;
  using T = typename PA::T;
  using AF = typename PR::AF;
  using Acc = typename PR::Acc;
  using DM = Dims<N>;
  constexpr int L = DM::L, Nt = DM::Nt, NCH = DM::NCH, MT = DM::MT;
  using SL = Steps<M, L>;
  constexpr int WL = SL::WIDE, NR = SL::NREG, PD = M == PREC_X3 ? 1 : 4;
  constexpr int NT1 = (modes_upto(N - 1) + 15) / 16, RS = PicardLDS<N, P>::RS;
  const int n = lane & 15, g = lane >> 4;
  const int p = qperm<T>(n);
  const Law<T> law{a.amax, a.smin};
  const StepMat<T> m = LW::constants(load_mat<T>(a.mat + e * 8));
  T u0[NR], U[Nt][NR], W[Nt][NR];
  load_state<N, P>(a, e, u0, lane);
#pragma unroll
  for (int z = 0; z < Nt; ++z)
#pragma unroll
    for (int r = 0; r < NR; ++r) U[z][r] = u0[r];
  // -sum_d Theta^-1_ed W_d: rows p (lanes), columns 4 i + g of (v, sigma, rate)
  T As[3][3];
  {
    const T rs = p >= 6 ? -m.ir : T(-1);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      T w[3];
#pragma unroll
      for (int d = 0; d < 3; ++d) w[d] = rs * a.mixV[(i * 3 + d) * 64 + lane];
#pragma unroll
      for (int ee = 0; ee < 3; ++ee)
        As[ee][i] = (T)a.geo[e * 16 + ee * 3] * w[0] + (T)a.geo[e * 16 + ee * 3 + 1] * w[1] +
                    (T)a.geo[e * 16 + ee * 3 + 2] * w[2];
    }
  }
  const T dt = (T)a.dt;
#pragma unroll 1
  for (int it = 0; it < pa.iters; ++it) {
#pragma unroll
    for (int z = 0; z < Nt; ++z)
#pragma unroll
      for (int r = 0; r < NR; ++r) W[z][r] = u0[r];
#pragma unroll 1
    for (int jt = 0; jt < Nt; ++jt) {
      // (U[0] is the state at time point jt: the iterate rotates)
      Acc X[MT];
      zero_C<M, MT>(X);
      {
        AF uw[WL > 0 ? WL : 1];
#pragma unroll
        for (int s = 0; s < WL; ++s) uw[s] = wide_op<M>(U[0], s);
#pragma unroll 1
        for (int c = 0; c < NCH; ++c) {
          T u[12], sig[6];
          nodal<N, P, PD>(U[0], uw, Vw, Vt, c, u, lane);
          const auto v = LW::invariants(u, law);
          LW::stress(v, u, m, sig);
          wave_sync();
#pragma unroll
          for (int k = 0; k < 3; ++k) S.X[k * RS + lane] = u[6 + k];
#pragma unroll
          for (int k = 0; k < 6; ++k) S.X[(3 + k) * RS + lane] = sig[k];
          S.X[9 * RS + lane] = LW::rate(v, m);
          wave_sync();
          // projection: quantities in rows, modes in columns
          typedef T T4 __attribute__((ext_vector_type(4), aligned(16)));
          const T* xs = S.X + (p < 10 ? p : 9) * RS;
          if constexpr (M == PREC_X3) {
            AF xw[2];
#pragma unroll
            for (int s = 0; s < 2; ++s) {
              const T4 lo = *(const T4*)(xs + 32 * s + 8 * g), hi = *(const T4*)(xs + 32 * s + 8 * g + 4);
              const T v8[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
              xw[s] = split8(v8);
            }
            stream<1, 2 * MT, AF>(
                [&](int k) { return load_frag<M>(Pw, c * 2 * MT + k, lane); },
                [&](int k, const AF& b) { X[k % MT] = PR::mma(xw[k / MT], b, X[k % MT]); });
          } else {
            T4 xv[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) xv[k] = *(const T4*)(xs + 16 * k + 4 * g);
            stream<PD, 16 * MT, AF>(
                [&](int k) { return load_frag<M>(Pw, c * 16 * MT + k, lane); },
                [&](int k, const AF& b) {
                  const int s = k / MT;
                  X[k % MT] = PR::mma(xv[s >> 2][s & 3], b, X[k % MT]);
                });
          }
        }
      }
      // the damage row changes from modes in lanes to modes in registers in LDS
      if (g == 1) {
#pragma unroll
        for (int t = 0; t < MT; ++t) S.al[mperm<N, M>(t, n)] = X[t][2];
      }
      wave_sync();
      Acc R[NT1];
      mix_contract<N, P, L, NT1, false, PD>(X, As, Kw, Kt, R, lane);
      T k[NR];
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        k[r] = r < 4 * NT1 ? R[r < 4 * NT1 ? r >> 2 : 0][r & 3] : T(0);
        if (p == 9) k[r] = S.al[SL::row(r, g)];
        if (p > 9) k[r] = T(0);
      }
      // the next iterate: U_z += dt Om_z,jt R(U_jt) for every z
#pragma unroll
      for (int z = 0; z < Nt; ++z) {
        const T w = dt * pa.om[z][jt];
#pragma unroll
        for (int r = 0; r < NR; ++r) W[z][r] += w * k[r];
      }
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const T first = U[0][r];
#pragma unroll
        for (int z = 0; z + 1 < Nt; ++z) U[z][r] = U[z + 1][r];
        U[Nt - 1][r] = first;
      }
    }
#pragma unroll
    for (int z = 0; z < Nt; ++z)
#pragma unroll
      for (int r = 0; r < NR; ++r) U[z][r] = W[z][r];
  }
  T* out = a.Uz + (size_t)e * DM::UZE;
  if (p < 10) {
#pragma unroll
    for (int z = 0; z < Nt; ++z)
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const int l = SL::row(r, g);
        if (l < L) out[z * DM::UZT + l * 10 + p] = U[z][r];
      }
  }
}

template <int N, int P, class LW>
__global__ __launch_bounds__((64 * PicardTabs<N, P>::wpb))
__attribute__((amdgpu_waves_per_eu(PicardTabs<N, P>::waves))) void k_picard(StepArgs<P> a,
                                                                            PicardArgs<P> pa) {
  using T = typename Prec<P>::T;
  using TB = PicardTabs<N, P>;
  __shared__ __attribute__((aligned(64))) char smem[TB::bytes];
  if constexpr (TB::staged) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    char *vw = smem, *vt = vw + TB::vw, *kw = vt + TB::vt, *kt = kw + TB::kw, *pw = kt + TB::kt;
    stage(vw, a.Vw, TB::vw);
    stage(vt, a.Vt, TB::vt);
    stage(kw, a.Kw, TB::kw);
    stage(kt, a.Kt, TB::kt);
    stage(pw, a.PXa, TB::pw);
    __syncthreads();
    PicardLDS<N, P>& S = ((PicardLDS<N, P>*)(smem + TB::all))[wave];
    for_elements(a, TB::wpb, [&](long long e, int lane) {
      picard_element<N, P, LW>(a, pa, e, S, vw, (const T*)vt, kw, (const T*)kt, pw, lane);
      wave_sync();
    });
  } else {
    PicardLDS<N, P>& S = *(PicardLDS<N, P>*)smem;
    for_elements(a, 1, [&](long long e, int lane) {
      picard_element<N, P, LW>(a, pa, e, S, a.Vw, a.Vt, a.Kw, a.Kt, a.PXa, lane);
    });
  }
}

// Time since each cluster's prediction at the start of the step being corrected
// (all zero in the global step).
struct ClusterOffsets { double v[8]; };

template <int N, int P> struct FaceLDS {
  using T = typename Prec<P>::T;
  static constexpr int JS = 16 * Deriv<N>::NT + 16 / sizeof(T);
  alignas(16) T tr[2][Dims<N>::Ns * JS];   // derivative traces of both sides, [point][column]
};

// Face fluxes (Appendix A.2 Eq. 2nd term, A.3; 312132 elements of degree 4: 1760 us,
// vector issue for 77 % of it; on time-point states 3430, with the LLF speed by acos and cos), interior faces once: traces of
// both sides' derivative matrices at the shared face points, Taylor sums per
// (time point, face point), local Lax-Friedrichs or boundary flux, time
// quadrature; sum_z gamma_z F* projected on the face modes, [face][NM2][10].
template <int N, int P, class LW>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(StepTune<N, P>::w_face)))
void k_face(StepArgs<P> a, const int* faces, long long nfaces, typename Prec<P>::T* fflux,
            const int* flist, ClusterOffsets offs) {
  constexpr int M = FaceForm<N, P>::value;
  using PR = Prec<M>;
  using PA = Prec<P>;
  using T = typename PA::T;
  using AF = typename PR::AF;
  using Acc = typename PR::Acc;
  using DM = Dims<N>;
  using DV = Deriv<N>;
  using SL = FaceLDS<N, P>;
  using SD = Steps<M, DM::L>;
  constexpr int Ns = DM::Ns, Nt = DM::Nt, NST = DM::NST, NT = DV::NT, WL = SD::WIDE;
  constexpr int JS = SL::JS, PD = M == PREC_X3 ? 2 : StepTune<N, P>::pd_face;
  constexpr int NRD = (Ns * Nt + 63) / 64, FR = 11, NM2 = FaceModes<N>::value;
  static_assert(Ns * Nt * FR + Ns * 10 <= 2 * Ns * JS, "fluxes fit the spent traces");
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
  T dzr[2][NT][SD::NREG];
#pragma unroll
  for (int side = 0; side < 2; ++side)
    load_deriv<N, M>(a.Dz + (size_t)(side ? nb : e) * DV::NF * 64, dzr[side], lane);
  // (a boundary face evaluates its own side twice and uses the first)
#pragma unroll
  for (int side = 0; side < 2; ++side) {
    const int fo = (side ? nf : f) * 6 + (side ? sq : sp);
    Acc C[NT][NST];
#pragma unroll
    for (int ct = 0; ct < NT; ++ct) zero_C<P, NST>(C[ct]);
    AF dzw[NT][WL];
#pragma unroll
    for (int ct = 0; ct < NT; ++ct)
#pragma unroll
      for (int s = 0; s < WL; ++s)
        if (M != PREC_X3 || DV::rows(16 * ct) > 4) dzw[ct][s] = wide_op<M>(dzr[side][ct], s);
    stream<PD, NST * WL, AF>(
        [&](int k) { return load_frag<M>(a.Fst, (fo * NST + k % NST) * WL + k / NST, lane); },
        [&](int k, const AF& b) {
          const int s = k / NST, t = k % NST;
          if constexpr (M == PREC_X3) {
#pragma unroll
            for (int q = 0; q < 6; ++q)
#pragma unroll
              for (int ct = 0; ct < NT; ++ct)
                if (DV::rows(16 * ct) > 4) C[ct][t] = PR::product(q, dzw[ct][s], b, C[ct][t]);
          } else {
#pragma unroll
            for (int ct = 0; ct < NT; ++ct)
              if (s < DV::steps(ct)) C[ct][t] = PR::mma(dzw[ct][s], b, C[ct][t]);
          }
        });
    if constexpr (M == PREC_X3) {
      // FP32 steps, as in the corrector
#pragma unroll
      for (int ct = 0; ct < NT; ++ct) {
        const int rows = DV::rows(16 * ct);
        if (rows % 32 > 4) continue;
#pragma unroll
        for (int t = 0; t < NST; ++t)
          C[ct][t] = PA::mma(dzr[side][ct][rows / 32 * 8],
                             a.Fstt[((rows > 32 ? 0 : 24 * NST * SD::TAIL) + fo * NST + t) * 64 + lane],
                             C[ct][t]);
      }
    }
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
  T* sG = sF + Ns * Nt * FR;
#pragma unroll
  for (int j = 0; j < (Ns * 10 + 63) / 64; ++j) {
    const int idx = lane + 64 * j;
    if (idx < Ns * 10) {
      const int i = idx / 10, k = idx - i * 10;
      T s = T(0);
#pragma unroll
      for (int z = 0; z < Nt; ++z) s += a.gamma[z] * sF[(z * Ns + i) * FR + k];
      sG[idx] = s;
    }
  }
  wave_sync();
  // projection on the face modes: modes in rows, quantities in columns
  Acc C;
#pragma unroll
  for (int i = 0; i < 4; ++i) C[i] = 0;
#pragma unroll
  for (int s = 0; s < (Ns + 3) / 4; ++s) {
    const int i = 4 * s + g;
    C = PA::mma(a.Psi[s * 64 + lane], sG[(i < Ns ? i : Ns - 1) * 10 + (n < 10 ? n : 9)], C);
  }
  T* out = fflux + (size_t)fid * NM2 * 10;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = PA::crow(lane, i);
    if (r < NM2 && n < 10) out[r * 10 + n] = C[i];
  }
}

// Time-point states of the derivatives in Dz (the Taylor sums of Eq.
// taylor_expansion) of the elements from e0 on, [E][Nt][10][L] FP64, for
// dgd_get_time_point_states; with clusters (a.ecl) each element over its own step.
template <int N, int P>
__global__ __launch_bounds__(64) void k_time_points(StepArgs<P> a, long long e0, double* out) {
  using T = typename Prec<P>::T;
  using DM = Dims<N>;
  using DV = Deriv<N>;
  constexpr int L = DM::L, Nt = DM::Nt;
  const long long e = e0 + blockIdx.x;
  out -= (size_t)e0 * Nt * 10 * L;
  const T dt = (T)(a.ecl ? a.dt * (double)(1 << a.ecl[e]) : a.dt);
  auto at = [&](int l, int j) -> T {
    const int c = j >> 4, f0 = DV::frag0(c);
    if (l >= DV::rows(j)) return T(0);
    return a.Dz[((size_t)e * DV::NF + f0 + l / 4) * 64 + 16 * (l & 3) + (j & 15)];
  };
  for (int idx = threadIdx.x; idx < 10 * L; idx += 64) {
    const int p = idx / L, l = idx - p * L;
    for (int z = 0; z < Nt; ++z) {
      const T h = a.tau[z] * dt;
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
