// push.hip -- particle side of the hybrid Yee-FFT PIC step on gfx950:
// field gather + relativistic Boris push + charge-conserving deposit, the
// particle tile sort, the deposit test hook and the charge density.
//
// The push+deposit kernel runs one workgroup per particle tile (particles are
// counting-sorted by tile every few steps).  The workgroup finds the periodic
// bounding box of its particles' cells, stages the six field components of that
// box (plus the stencil halo) in LDS, pushes its particles gathering from LDS,
// accumulates the current of the box in LDS (64-bit integer atomics in the FP32
// form, so the result does not depend on the order), and adds the box to the
// global accumulators with one atomic per node.  Where the two boxes do not fit
// the LDS, it holds the currents alone.
#include <type_traits>

#include "hpic_divide.h"
#include "hpic_internal.h"

namespace hp {

template <class R> struct V2;
template <> struct V2<float> { using T = float2; };
template <> struct V2<double> { using T = double2; };

// ---------------------------------------------------------------- field sources
// Fields as seen by the gather: rows/cols are offsets returned by row()/col()
// for (possibly out-of-range) node indices; pairs share a stencil:
// p0 = (E1, B2) on (i1+1/2, i2), p1 = (E2, B1) on (i1, i2+1/2),
// e3 on (i1, i2), b3 on (i1+1/2, i2+1/2).
template <class R>
struct GlobalFields {
  static constexpr bool local = false;
  gptr<const R> F;
  int n1, n2, cells;
  __device__ int col(int i) const { return wrap_pow2(i, n1); }
  __device__ int row(int j) const { return wrap_small(j, n2) * n1; }
  __device__ typename V2<R>::T p0(int r, int c) const {
    typename V2<R>::T v;
    v.x = F[r + c];
    v.y = F[4 * cells + r + c];
    return v;
  }
  __device__ typename V2<R>::T p1(int r, int c) const {
    typename V2<R>::T v;
    v.x = F[cells + r + c];
    v.y = F[3 * cells + r + c];
    return v;
  }
  __device__ R e3(int r, int c) const { return F[2 * cells + r + c]; }
  __device__ R b3(int r, int c) const { return F[5 * cells + r + c]; }
};

// Field box in LDS with row stride FS, or W where FS is 0.  A literal stride
// makes the nine nodes of a component immediate offsets from one address.
template <class R, int FS>
struct LdsFields {
  static constexpr bool local = true;
  typedef R T2 __attribute__((ext_vector_type(2)));
  lptr<const T2> P0, P1;
  lptr<const R> E3, B3;
  int W;
  __device__ int stride() const { return FS > 0 ? FS : W; }
  __device__ int row(int j) const { return __mul24(j, stride()); }
  __device__ T2 p0(int r, int c) const { return P0[r + c]; }
  __device__ T2 p1(int r, int c) const { return P1[r + c]; }
  __device__ R e3(int r, int c) const { return E3[r + c]; }
  __device__ R b3(int r, int c) const { return B3[r + c]; }
};

// Factor of gather2's result: weights along both axes are doubled in the
// momentum-conserving gather (a field above 1/4 of the largest number is then
// reported as non-finite).
template <class R, bool EC> constexpr R GATHER_SCALE = EC ? R(1) : R(0.25);

// Quadratic gather (Appendix A): momentum-conserving (every component uses the
// quadratic B-spline around its own staggered node) or, with EC, energy-
// conserving (linear weights along the component's staggered directions).
// Returns the fields over GATHER_SCALE.
template <class R, bool EC, class Src>
__device__ __forceinline__ void gather2(const Src &S, int i1, int i2, R f1, R f2, R Ef[3],
                                        R Bf[3]) {
  const int up1 = f1 >= R(0.5), up2 = f2 >= R(0.5);
  R wi1[3], wh1[3], wi2[3], wh2[3];
  if constexpr (EC) {
    spline3<R>(f1 - R(up1), wi1);  // integer nodes along x1
    line3<R>(f1 - R(0.5), wh1);    // half nodes along x1
    spline3<R>(f2 - R(up2), wi2);
    line3<R>(f2 - R(0.5), wh2);
  } else {
    spline3x2<R>(f1 - R(up1), wi1);
    spline3x2<R>(f1 - R(0.5), wh1);
    spline3x2<R>(f2 - R(up2), wi2);
    spline3x2<R>(f2 - R(0.5), wh2);
  }
  int ci[3], ch[3], ri[3], rh[3];
  if constexpr (Src::local) {
    // one origin per axis and stencil, the other nodes at fixed distances
    const int c0 = i1 + up1 - 1, r0 = S.row(i2 + up2 - 1), s0 = S.row(i2 - 1), w = S.stride();
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      ci[a] = c0 + a;
      ch[a] = i1 - 1 + a;
      ri[a] = r0 + a * w;
      rh[a] = s0 + a * w;
    }
  } else {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      ci[a] = S.col(i1 + up1 - 1 + a);
      ch[a] = S.col(i1 - 1 + a);
      ri[a] = S.row(i2 + up2 - 1 + a);
      rh[a] = S.row(i2 - 1 + a);
    }
  }
  R e1 = 0, e2 = 0, e3 = 0, b1 = 0, b2 = 0, b3 = 0;
#pragma unroll
  for (int b = 0; b < 3; ++b) {
    R s_e1 = 0, s_e2 = 0, s_e3 = 0, s_b1 = 0, s_b2 = 0, s_b3 = 0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const auto q0 = S.p0(ri[b], ch[a]);  // E1, B2 at (i1+1/2, i2)
      const auto q1 = S.p1(rh[b], ci[a]);  // E2, B1 at (i1, i2+1/2)
      s_e1 += wh1[a] * q0.x;
      s_b2 += wh1[a] * q0.y;
      s_e2 += wi1[a] * q1.x;
      s_b1 += wi1[a] * q1.y;
      s_e3 += wi1[a] * S.e3(ri[b], ci[a]);
      s_b3 += wh1[a] * S.b3(rh[b], ch[a]);
    }
    e1 += wi2[b] * s_e1;
    b2 += wi2[b] * s_b2;
    e2 += wh2[b] * s_e2;
    b1 += wh2[b] * s_b1;
    e3 += wi2[b] * s_e3;
    b3 += wh2[b] * s_b3;
  }
  Ef[0] = e1; Ef[1] = e2; Ef[2] = e3;
  Bf[0] = b1; Bf[1] = b2; Bf[2] = b3;
}

// Place the three stencil values s[] of nearest node m in a 4-node window
// starting at base (offset m - 1 - base in {0, 1}) without dynamic indexing.
template <class T>
__device__ __forceinline__ void place4(const T s[3], int off, T out[4]) {
  out[0] = off ? T(0) : s[0];
  out[1] = off ? s[0] : s[1];
  out[2] = off ? s[1] : s[2];
  out[3] = off ? s[2] : T(0);
}

// ---------------------------------------------------------------- current sinks
// A sink maps node indices (in the frame of the cell indices given to the
// deposit) to offsets with row(j) + col(i) and adds a value to component c at
// an offset.
struct GlobalFixed {
  gptr<unsigned long long> J;
  int n1, n2, cells;
  __device__ int row(int j) const { return wrap_small(j, n2) * n1; }
  __device__ int col(int i) const { return wrap_pow2(i, n1); }
  __device__ void add(int c, int off, long long v) const {
    if (v != 0)
      __scoped_atomic_fetch_add(J + c * cells + off, (unsigned long long)v, __ATOMIC_RELAXED,
                                __MEMORY_SCOPE_DEVICE);
  }
};
// Current box in LDS: rows of three component rows, [row][component][column],
// CS columns (a literal), or W where CS is 0.
template <int CS>
struct LdsFixed {
  lptr<unsigned long long> J;
  int W;
  __device__ int width() const { return CS > 0 ? CS : W; }
};
struct GlobalFp64 {
  double *J;
  int n1, n2, cells;
  __device__ int row(int j) const { return wrap_small(j, n2) * n1; }
  __device__ int col(int i) const { return wrap_pow2(i, n1); }
  __device__ void add(int c, int off, double v) const {
    if (v != 0.0) unsafeAtomicAdd(J + c * cells + off, v);
  }
};
template <int CS>
struct LdsFp64 {
  double *J;
  int W;
  __device__ int width() const { return CS > 0 ? CS : W; }
  __device__ int row(int j) const { return __mul24(j, 3 * width()); }
  __device__ int col(int i) const { return i; }
  __device__ void add(int c, int off, double v) const {
    if (v != 0.0) unsafeAtomicAdd(J + c * width() + off, v);
  }
};

// Fixed-point Esirkepov deposit of one particle (2D).  Integer shapes with
// exact sum 2^P make 2 (rho_new - rho_old) = div J hold exactly in the
// integers; j3 is FP32 rounded once per node.  The arithmetic is the one of the
// FP32-precision reference deposit, operation for operation.
//
// UNIT (|charge| 2^P < 2^23, so Q C1 and Q C2 fit 24 signed bits) selects the
// full-rate 24-bit integer products; it is a template parameter so that the
// general 64-bit products are not compiled into the common kernel.
template <bool UNIT, class Sink>
__device__ __forceinline__ void deposit2_fixed(const Sink &K, int P, float inv_wunit, float c3,
                                               int i1, int i2, float fa1, float fa2, int d1,
                                               int d2, float fb1, float fb2, float v3, float qw) {
#pragma clang fp contract(off)
  int sa1[3], sb1[3], sa2[3], sb2[3];
  const int na1 = fixed_shape<UNIT>(i1, fa1, P, sa1);
  const int nb1 = fixed_shape<UNIT>(i1 + d1, fb1, P, sb1);
  const int na2 = fixed_shape<UNIT>(i2, fa2, P, sa2);
  const int nb2 = fixed_shape<UNIT>(i2 + d2, fb2, P, sb2);
  const int base1 = min(na1, nb1) - 1, base2 = min(na2, nb2) - 1;
  int S0x[4], S1x[4], S0y[4], S1y[4];
  place4(sa1, na1 - 1 - base1, S0x);
  place4(sb1, nb1 - 1 - base1, S1x);
  place4(sa2, na2 - 1 - base2, S0y);
  place4(sb2, nb2 - 1 - base2, S1y);
  const float qs = qw * inv_wunit;
  const int Q = (int)rintf(qs);
  int C1[4], C2[4], A1[4], A2[4];
  int acc1 = 0, acc2 = 0;
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    acc1 += S1x[a] - S0x[a];
    acc2 += S1y[a] - S0y[a];
    C1[a] = acc1;
    C2[a] = acc2;
    A1[a] = S0x[a] + S1x[a];
    A2[a] = S0y[a] + S1y[a];
  }
  int ro[4], co[4];
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    ro[a] = K.row(base2 + a);
    co[a] = K.col(base1 + a);
  }
  // J1 = Q C1[a] A2[b], J2 = Q C2[b] A1[a]: exact integer products.  With
  // |Q C| <= 2^22 and A <= 1.5 2^P both factors fit 24 signed bits, so the
  // 48-bit product is one pair of full-rate 24-bit multiplies.
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const int qc = UNIT ? mul24_lo(Q, C1[a]) : 0;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      long long v;
      if (UNIT) v = mul24_wide(qc, A2[b]);
      else v = ((long long)Q * (long long)C1[a]) * (long long)A2[b];
      K.add(0, ro[b] + co[a], v);
    }
  }
#pragma unroll
  for (int b = 0; b < 3; ++b) {
    const int qc = UNIT ? mul24_lo(Q, C2[b]) : 0;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      long long v;
      if (UNIT) v = mul24_wide(qc, A1[a]);
      else v = ((long long)Q * (long long)C2[b]) * (long long)A1[a];
      K.add(1, ro[b] + co[a], v);
    }
  }
  // j3 = rint(x0[a] t0[b] + x1[a] t1[b]) with x = S h, t0 = 2 S0y + S1y,
  // t1 = S0y + 2 S1y: the product x1 t1 rounded, then one fused multiply-add.
  // |value| < 2^31 by the choice of c3, so it fits 32 bits.
  const float hv = qs * v3;
  const float h = hv * c3;
  float x0[4], x1[4];
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    x0[a] = (float)S0x[a] * h;
    x1[a] = (float)S1x[a] * h;
  }
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const float B0 = (float)S0y[b], B1 = (float)S1y[b];
    const float t0 = 2.0f * B0 + B1;
    const float t1 = B0 + 2.0f * B1;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const float p1 = x1[a] * t1;
      const float v = __builtin_fmaf(x0[a], t0, p1);
      K.add(2, ro[b] + co[a], (long long)(int)rintf(v));
    }
  }
}

// FP64 Esirkepov deposit of one particle (2D).
template <class Sink>
__device__ __forceinline__ void deposit2_fp64(const Sink &K, double jfx1, double jfx2, int i1,
                                              int i2, double fa1, double fa2, int d1, int d2,
                                              double fb1, double fb2, double v3, double qw) {
  double sa1[3], sb1[3], sa2[3], sb2[3];
  const int ua1 = fa1 >= 0.5, ub1 = fb1 >= 0.5, ua2 = fa2 >= 0.5, ub2 = fb2 >= 0.5;
  spline3<double>(fa1 - ua1, sa1);
  spline3<double>(fb1 - ub1, sb1);
  spline3<double>(fa2 - ua2, sa2);
  spline3<double>(fb2 - ub2, sb2);
  const int na1 = i1 + ua1, nb1 = i1 + d1 + ub1, na2 = i2 + ua2, nb2 = i2 + d2 + ub2;
  const int base1 = min(na1, nb1) - 1, base2 = min(na2, nb2) - 1;
  double S0x[4], S1x[4], S0y[4], S1y[4];
  place4(sa1, na1 - 1 - base1, S0x);
  place4(sb1, nb1 - 1 - base1, S1x);
  place4(sa2, na2 - 1 - base2, S0y);
  place4(sb2, nb2 - 1 - base2, S1y);
  int ro[4], co[4];
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    ro[a] = K.row(base2 + a);
    co[a] = K.col(base1 + a);
  }
  const double f1 = qw * jfx1, f2 = qw * jfx2;
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    double acc = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      acc += f1 * (S1x[a] - S0x[a]) * 0.5 * (S0y[b] + S1y[b]);
      K.add(0, ro[b] + co[a], acc);
    }
  }
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    double acc = 0.0;
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      acc += f2 * (S1y[b] - S0y[b]) * 0.5 * (S0x[a] + S1x[a]);
      K.add(1, ro[b] + co[a], acc);
    }
  }
  const double g3 = qw * v3;
#pragma unroll
  for (int b = 0; b < 4; ++b) {
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const double W3 = S0x[a] * S0y[b] * (1.0 / 3.0) + S1x[a] * S0y[b] * (1.0 / 6.0) +
                        S0x[a] * S1y[b] * (1.0 / 6.0) + S1x[a] * S1y[b] * (1.0 / 3.0);
      K.add(2, ro[b] + co[a], g3 * W3);
    }
  }
}

// What the fixed-point deposit needs of its run, read once per block.
struct Fix {
  int P;
  float inv_wunit, c3;
  float hz;  // |h| below which every j3 value rounds to zero
};
// every j3 value rounds to zero when |h| (S0x t0 + S1x t1) stays below 1/2: the
// bracket is at most 2 (3/4)(9/4) 2^(2P) = 3.375 2^(2P), and 0.45 leaves room
// for the FP32 rounding of the products
__device__ __forceinline__ Fix fix_of(const Run<float> &r) {
  return Fix{r.P, r.inv_wunit, r.c3, uniform((0.45f / 3.375f) / ((float)(1 << r.P) * (float)(1 << r.P)))};
}
struct NoFix {};
__device__ __forceinline__ NoFix fix_of(const Run<double> &) { return NoFix{}; }

// The same deposit into a workgroup's LDS box, giving the same integers bit for
// bit; only the addressing and which zero contributions are left out differ.
// In the window (first node min(nearest node before, after) - 1 per axis) both
// shapes cover nodes 0..2 unless the particle changes its nearest node along
// that axis, so apart from offsets exactly on a stencil edge the zero
// contributions are: along x1, column 3 of j2 and j3 and the running sum C1[2]
// of j1 (zero unless the lane switches nodes along x1); along x2, row 3 of j1
// and j3 and C2[2] of j2; all of j1 (j2) for a particle that does not move
// along x1 (x2) by a quantisation step; all of j3 when |h| is too small for
// any value to round away from zero.  The x1 column is left to the lanes that
// switch, in one block at the end; the x2 row is skipped for the whole wave
// when no lane switches along x2 (the common case for plasmas drifting along
// x1); a component for the lanes that do not move along its axis (a cold drift
// along x1 has no j2 and j3 outside the laser).  Every other node is added
// without a test (adding an exact zero changes nothing).  With a literal column
// stride every node of the three components is an immediate offset of one
// address.
template <bool UNIT, int CS>
__device__ __forceinline__ void deposit2_fixed_lds(const LdsFixed<CS> &K, const Fix &fx, int i1,
                                                   int i2, float fa1, float fa2, int d1, int d2,
                                                   float fb1, float fb2, float v3, float qw) {
#pragma clang fp contract(off)
  const int P = fx.P;
  int sa1[3], sb1[3], sa2[3], sb2[3];
  const int na1 = fixed_shape<UNIT>(i1, fa1, P, sa1);
  const int nb1 = fixed_shape<UNIT>(i1 + d1, fb1, P, sb1);
  const int na2 = fixed_shape<UNIT>(i2, fa2, P, sa2);
  const int nb2 = fixed_shape<UNIT>(i2 + d2, fb2, P, sb2);
  const int base1 = min(na1, nb1) - 1, base2 = min(na2, nb2) - 1;
  int S0x[4], S1x[4], S0y[4], S1y[4];
  place4(sa1, na1 - 1 - base1, S0x);
  place4(sb1, nb1 - 1 - base1, S1x);
  place4(sa2, na2 - 1 - base2, S0y);
  place4(sb2, nb2 - 1 - base2, S1y);
  const float qs = qw * fx.inv_wunit;
  const int Q = (int)rintf(qs);
  int C1[3], C2[3], A1[4], A2[4];
  int acc1 = 0, acc2 = 0;
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    acc1 += S1x[a] - S0x[a];
    acc2 += S1y[a] - S0y[a];
    if (a < 3) {
      C1[a] = acc1;
      C2[a] = acc2;
    }
    A1[a] = S0x[a] + S1x[a];
    A2[a] = S0y[a] + S1y[a];
  }
  const bool sw1 = na1 != nb1;                   // per lane
  const bool row3 = __ballot(na2 != nb2) != 0;  // wave-uniform
  // j1 (j2) vanishes when the quantised x1 (x2) shapes are the same before
  // and after the move (three integers summing to 2^P: two of them decide)
  const bool mv1 = (na1 != nb1) | (sa1[0] != sb1[0]) | (sa1[2] != sb1[2]);
  const bool mv2 = (na2 != nb2) | (sa2[0] != sb2[0]) | (sa2[2] != sb2[2]);
  const int W = K.width(), W3 = 3 * W;
  const lptr<unsigned long long> J1 = K.J + (__mul24(base2, W3) + base1);
  const lptr<unsigned long long> J2 = J1 + W, J3 = J2 + W;
  auto add = [](lptr<unsigned long long> q, long long v) {
    __hip_atomic_fetch_add(q, (unsigned long long)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  };
  auto prod = [&](int qc, int c, int f) -> long long {
    if (UNIT) return mul24_wide(qc, f);
    return ((long long)Q * (long long)c) * (long long)f;
  };
  int qc1[3], qc2[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    qc1[a] = UNIT ? mul24_lo(Q, C1[a]) : 0;
    qc2[a] = UNIT ? mul24_lo(Q, C2[a]) : 0;
  }
  // j1 = Q C1[a] A2[b], a = 0..2 (C1[3] = 0)
  if (mv1) {
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      if (b == 3 && !row3) break;
      const lptr<unsigned long long> row = J1 + b * W3;
      add(row, prod(qc1[0], C1[0], A2[b]));
      add(row + 1, prod(qc1[1], C1[1], A2[b]));
    }
  }
  // j2 = Q C2[b] A1[a], b = 0..2 (C2[3] = 0)
  if (mv2) {
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      if (b == 2 && !row3) break;
      const lptr<unsigned long long> row = J2 + b * W3;
      add(row, prod(qc2[b], C2[b], A1[0]));
      add(row + 1, prod(qc2[b], C2[b], A1[1]));
      add(row + 2, prod(qc2[b], C2[b], A1[2]));
    }
  }
  // j3 = rint(x0[a] t0[b] + x1[a] t1[b]) with the operation order of deposit2_fixed
  const float hv = qs * v3;
  const float h = hv * fx.c3;
  const bool on3 = !(fabsf(h) < fx.hz);
  auto j3 = [&](int a0, int a1) {
    float x0[4], x1[4];
#pragma unroll
    for (int a = a0; a < a1; ++a) {
      x0[a] = (float)S0x[a] * h;
      x1[a] = (float)S1x[a] * h;
    }
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      if (b == 3 && !row3) break;
      const float B0 = (float)S0y[b], B1 = (float)S1y[b];
      const float t0 = 2.0f * B0 + B1;
      const float t1 = B0 + 2.0f * B1;
      const lptr<unsigned long long> row = J3 + b * W3;
#pragma unroll
      for (int a = a0; a < a1; ++a) {
        const float p1 = x1[a] * t1;
        const float v = __builtin_fmaf(x0[a], t0, p1);
        add(row + a, (long long)(int)rintf(v));
      }
    }
  };
  if (on3) j3(0, 3);
  // the fourth column, of the lanes that switch nodes along x1 (they all move)
  if (sw1) {
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      if (b == 3 && !row3) break;
      add(J1 + b * W3 + 2, prod(qc1[2], C1[2], A2[b]));
    }
    if (mv2) {
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        if (b == 2 && !row3) break;
        add(J2 + b * W3 + 3, prod(qc2[b], C2[b], A1[3]));
      }
    }
    if (on3) j3(3, 4);
  }
}

template <bool UNIT, class Sink>
__device__ __forceinline__ void deposit_one(const Run<float> &r, const Fix &fx, const Sink &K,
                                            int i1, int i2, float fa1, float fa2, int d1, int d2,
                                            float fb1, float fb2, float v3, float qw) {
  deposit2_fixed<UNIT>(K, fx.P, fx.inv_wunit, fx.c3, i1, i2, fa1, fa2, d1, d2, fb1, fb2, v3, qw);
}
template <bool UNIT, int CS>
__device__ __forceinline__ void deposit_one(const Run<float> &r, const Fix &fx,
                                            const LdsFixed<CS> &K, int i1, int i2, float fa1,
                                            float fa2, int d1, int d2, float fb1, float fb2,
                                            float v3, float qw) {
  deposit2_fixed_lds<UNIT, CS>(K, fx, i1, i2, fa1, fa2, d1, d2, fb1, fb2, v3, qw);
}
template <bool UNIT, class Sink>
__device__ __forceinline__ void deposit_one(const Run<double> &r, const NoFix &, const Sink &K,
                                            int i1, int i2, double fa1, double fa2, int d1, int d2,
                                            double fb1, double fb2, double v3, double qw) {
  deposit2_fp64(K, r.jfx1, r.jfx2, i1, i2, fa1, fa2, d1, d2, fb1, fb2, v3, qw);
}

template <class R, int CS> struct Sinks;
template <int CS> struct Sinks<float, CS> { using G = GlobalFixed; using L = LdsFixed<CS>; using T = unsigned long long; };
template <int CS> struct Sinks<double, CS> { using G = GlobalFp64; using L = LdsFp64<CS>; using T = double; };

// A particle's deposit into an LDS box that does not hold every particle of the tile:
// at its cell (l1, l2) there, or at its cell (i1, i2) of the grid if it is outside.
template <class R>
struct SinkWide {
  typename Sinks<R, 0>::L lds;
  typename Sinks<R, 0>::T *J;
  bool in;
  int l1, l2;
};
// (The grid's half out of line, with plain arguments: it is rare, and takes no
// registers from the other so.)
template <bool UNIT>
__device__ __noinline__ void deposit_grid(const Run<float> *r, unsigned long long *J, int i1, int i2,
                                          float fa1, float fa2, int d1, int d2, float fb1, float fb2,
                                          float v3, float qw) {
  deposit2_fixed<UNIT>(GlobalFixed{G(J), r->n1, r->n2, r->cells}, r->P, r->inv_wunit, r->c3, i1, i2, fa1, fa2,
                       d1, d2, fb1, fb2, v3, qw);
}
template <bool UNIT>
__device__ __noinline__ void deposit_grid(const Run<double> *r, double *J, int i1, int i2, double fa1,
                                          double fa2, int d1, int d2, double fb1, double fb2, double v3,
                                          double qw) {
  deposit2_fp64(GlobalFp64{J, r->n1, r->n2, r->cells}, r->jfx1, r->jfx2, i1, i2, fa1, fa2, d1, d2, fb1, fb2, v3,
                qw);
}
template <bool UNIT>
__device__ __forceinline__ void deposit_one(const Run<float> &r, const Fix &fx, const SinkWide<float> &K,
                                            int i1, int i2, float fa1, float fa2, int d1, int d2,
                                            float fb1, float fb2, float v3, float qw) {
  if (K.in)
    deposit_one<UNIT>(r, fx, K.lds, K.l1, K.l2, fa1, fa2, d1, d2, fb1, fb2, v3, qw);
  else
    deposit_grid<UNIT>(&r, K.J, i1, i2, fa1, fa2, d1, d2, fb1, fb2, v3, qw);
}
template <bool UNIT>
__device__ __forceinline__ void deposit_one(const Run<double> &r, const NoFix &fx, const SinkWide<double> &K,
                                            int i1, int i2, double fa1, double fa2, int d1, int d2,
                                            double fb1, double fb2, double v3, double qw) {
  if (K.in)
    deposit_one<UNIT>(r, fx, K.lds, K.l1, K.l2, fa1, fa2, d1, d2, fb1, fb2, v3, qw);
  else
    deposit_grid<UNIT>(&r, K.J, i1, i2, fa1, fa2, d1, d2, fb1, fb2, v3, qw);
}

// Push one particle (state s): gather from S at the particle's cell (li1, li2)
// in S's frame, Boris, move, deposit into K in the same frame; s becomes the new
// state, (gi1, gi2) being the global cell.  Sets the cell moves (d1, d2), zero
// if the particle was rejected: a non-finite or a too-long move leaves it as it
// was, sets the error word and returns false.  One test of the velocities
// catches both: a non-finite momentum makes its velocity component NaN (inf *
// 0, or NaN throughout), and every comparison with NaN is false.
template <class R, bool UNIT, bool EC, class FX, class Src, class Sink>
__device__ __forceinline__ bool push_one(const Run<R> &r, const FX &fx, PState<R> &s, int gi1,
                                         int gi2, int li1, int li2, const Src &S, const Sink &K,
                                         unsigned *err, int &d1, int &d2) {
  R u[3] = {s.u1, s.u2, s.u3};
  R Ef[3], Bf[3];
  gather2<R, EC>(S, li1, li2, s.f1, s.f2, Ef, Bf);
  boris<R>(r.qmhdt * GATHER_SCALE<R, EC>, Ef, Bf, u);
  R v[3];
  velocity<R>(u, v);
  const R m1 = r.dtdx1 * v[0], m2 = r.dtdx2 * v[1];
  d1 = d2 = 0;
  if (!(fabs(m1) < R(1) && fabs(m2) < R(1) && fabs(v[2]) < R(2))) {
    const bool fin = isfinite(u[0]) && isfinite(u[1]) && isfinite(u[2]) && isfinite(m1) && isfinite(m2);
    atomicOr(err, fin ? ERR_RANGE : ERR_NUMERIC);
    return false;
  }
  R g1, g2;
  d1 = advance<R>(s.f1, m1, g1);
  d2 = advance<R>(s.f2, m2, g2);
  deposit_one<UNIT>(r, fx, K, li1, li2, s.f1, s.f2, d1, d2, g1, g2, v[2], s.qw);
  s.cell = (wrap_small(gi2 + d2, r.n2) << r.log2n1) | wrap_pow2(gi1 + d1, r.n1);
  s.f1 = g1;
  s.f2 = g2;
  s.u1 = u[0];
  s.u2 = u[1];
  s.u3 = u[2];
  return true;
}

__device__ __forceinline__ int wrap_delta_pow2(int d, int n) { return ((d + (n >> 1)) & (n - 1)) - (n >> 1); }
__device__ __forceinline__ int wrap_delta(int d, int n) {
  d += (d < -(n >> 1)) ? n : 0;
  d -= (d >= n - (n >> 1)) ? n : 0;
  return d;
}

// The workgroup's tile through LDS boxes with column strides CS (current) and
// CS - 2 (fields), or the box's own where CS is 0; the thread's first particle
// s0 (loaded before, so that its loads wait out the latency with the
// staging's).  box collects the particles' new cells in the frame.
template <class R, bool UNIT, bool EC, int CS>
__device__ __forceinline__ void push_tile(const Run<R> &r, const Parts<R> &P, int parity, int start,
                                          int end, PState<R> s0, int ref1, int ref2, int lo1,
                                          int lo2, int W, int H, unsigned char *smem,
                                          unsigned *err, int *nbox) {
  using SK = Sinks<R, CS>;
  using T = typename SK::T;
  constexpr int FS = CS > 0 ? CS - 2 : 0;
  const int n1 = r.n1, n2 = r.n2, cells = n1 * n2;
  const int FW = W - 2, FH = H - 2;
  const int cs = CS > 0 ? CS : W, fs = CS > 0 ? FS : FW;
  const int jrow = 3 * cs, fnodes = fs * FH;
  const int jbytes = (jrow * H * (int)sizeof(T) + 15) & ~15;
  // LDS layout: current accumulators first, then the fields (16-byte aligned)
  using LF = LdsFields<R, FS>;
  using T2 = typename LF::T2;
  const lptr<T> lj = (lptr<T>)smem;
  const lptr<T2> lp0 = (lptr<T2>)(smem + jbytes);
  const lptr<T2> lp1 = lp0 + fnodes;
  const lptr<R> le3 = (lptr<R>)(lp1 + fnodes);
  const lptr<R> lb3 = le3 + fnodes;
  const gptr<const R> F = G((const R *)r.F);
  const int o1 = ref1 + lo1 - 1, o2 = ref2 + lo2 - 1;  // global cell of the field-box origin
  for_box(FW, FH, [&](int b, int a) {
    const int g = wrap_any(o2 + b, n2) * n1 + wrap_pow2(o1 + a, n1), q = b * fs + a;
    const R e1 = F[g], e2 = F[cells + g], e3 = F[2 * cells + g];
    const R b1 = F[3 * cells + g], b2 = F[4 * cells + g], b3 = F[5 * cells + g];
    lp0[q] = T2{e1, b2};
    lp1[q] = T2{e2, b1};
    le3[q] = e3;
    lb3[q] = b3;
  });
  for (int q = threadIdx.x; q < jrow * H; q += PUSH_THREADS) lj[q] = 0;
  __syncthreads();
  // Particles use field-box coordinates (origin: cell lo-1).  The current box
  // starts one cell earlier, so its sink is shifted by one row and one column.
  const LF S{lp0, lp1, le3, lb3, fs};
  typename SK::L K;
  K.J = (decltype(K.J))(lj + jrow + 1);
  K.W = W;
  const int f1 = (n1 - r.T1) >> 1, f2 = (n2 - r.T2) >> 1;
  const auto fx = fix_of(r);
  CellBox box;
  PState<R> st = s0;
  for (int p = start + (int)threadIdx.x; p < end;) {
    // the next particle's loads are in flight while this one is pushed
    const int pn = p + PUSH_THREADS;
    PState<R> sn = st;
    if (pn < end) sn = load_state(P, pn);
    const int i1 = st.cell & (n1 - 1), i2 = st.cell >> r.log2n1;
    const int l1 = frame_pow2(i1 - ref1, f1, n1), l2 = frame_any(i2 - ref2, f2, n2);
    int d1, d2;
    const bool ok = push_one<R, UNIT, EC>(r, fx, st, i1, i2, l1 - lo1 + 1, l2 - lo2 + 1, S, K, err,
                                          d1, d2);
    box.add(l1 + d1, l2 + d2);
    arrived(sn);
    if (ok) store_state(P, p, st);
    st = sn;
    p = pn;
  }
  box.reduce(nbox);
  __syncthreads();
  // add the box to the global accumulators
  const auto J = G((T *)r.J[parity]);
  for_box(W, H, [&](int b, int a) {
    const int g = wrap_any(o2 - 1 + b, n2) * n1 + wrap_pow2(o1 - 1 + a, n1);
#pragma unroll
    for (int comp = 0; comp < 3; ++comp) {
      const T v = lj[b * jrow + comp * cs + a];
      if (v != 0)
        __scoped_atomic_fetch_add(J + comp * cells + g, v, __ATOMIC_RELAXED, __MEMORY_SCOPE_DEVICE);
    }
  });
}

// A tile whose particles have spread so far that the two boxes do not fit: fields
// through the cache, so that the LDS holds twice the current box, and only the particles
// outside that deposit into global memory.  (1024 x 512, eight particles a cell, sorted
// every 16 steps, push with a thermal spread of 0.3: 251 us, 1413 with such tiles in
// global memory; of 1: 338 and 2124; FP64 form of 0.3: 229 and 1831.)
template <class R, bool UNIT, bool EC>
__device__ __forceinline__ void push_wide(const Run<R> *run, int t, int parity, int pp, int lds_bytes,
                                       lptr<unsigned char> smem, lptr<int> nbox, unsigned *err) {
  using SK = Sinks<R, 0>;
  using T = typename SK::T;
  const Run<R> &r = *run;
  const Parts<R> P = r.pt[pp];
  const int n1 = r.n1, n2 = r.n2, cells = n1 * n2;
  const int f1 = (n1 - r.T1) >> 1, f2 = (n2 - r.T2) >> 1;
  const int start = G(r.tile_start)[t], end = G(r.tile_start)[t + 1];
  const int t2 = t / r.nt1, ref1 = (t - t2 * r.nt1) * r.T1, ref2 = t2 * r.T2;
  const auto tb = G(r.tile_box) + 6 * t;
  const WideBox w = wide_box(r, P, start, end, ref1, ref2, tb[0], tb[1], tb[2], tb[3], lds_bytes / 24,
                             (unsigned char *)smem);
  const lptr<T> lj = (lptr<T>)smem;
  const int jrow = 3 * w.W, o1 = ref1 + w.lo1 - 2, o2 = ref2 + w.lo2 - 2;
  for (int q = threadIdx.x; q < jrow * w.H; q += PUSH_THREADS) lj[q] = 0;
  __syncthreads();
  const GlobalFields<R> S{G((const R *)r.F), n1, n2, cells};
  const auto fx = fix_of(r);
  const gptr<T> J = G((T *)r.J[parity]);
  CellBox box;
  for (int p = start + (int)threadIdx.x; p < end; p += PUSH_THREADS) {
    PState<R> s = load_state(P, p);
    const int i1 = s.cell & (n1 - 1), i2 = s.cell >> r.log2n1;
    const int l1 = frame_pow2(i1 - ref1, f1, n1), l2 = frame_any(i2 - ref2, f2, n2);
    const SinkWide<R> K{{(decltype(SK::L::J))lj, w.W}, (T *)r.J[parity], w.holds(l1, l2), l1 - w.lo1 + 2, l2 - w.lo2 + 2};
    int d1, d2;
    if (push_one<R, UNIT, EC>(r, fx, s, i1, i2, i1, i2, S, K, err, d1, d2)) store_state(P, p, s);
    box.add(l1 + d1, l2 + d2);
  }
  box.reduce((int *)nbox);
  __syncthreads();
  for_box(w.W, w.H, [&](int b, int a) {
    const int g = wrap_any(o2 + b, n2) * n1 + wrap_pow2(o1 + a, n1);
#pragma unroll
    for (int comp = 0; comp < 3; ++comp) {
      const T v = lj[b * jrow + comp * w.W + a];
      if (v != 0)
        __scoped_atomic_fetch_add(J + comp * cells + g, v, __ATOMIC_RELAXED, __MEMORY_SCOPE_DEVICE);
    }
  });
}

// Out of line, where it would take registers from the paths of a tile that fits (8192 x
// 512, two particles a cell: push 222 us, 232 with it in line).
template <class R, bool UNIT>
__device__ __noinline__ void push_wide_call(const Run<R> *run, int t, int parity, int pp, int lds_bytes,
                                            lptr<unsigned char> smem, lptr<int> nbox, unsigned *err) {
  push_wide<R, UNIT, false>(run, t, parity, pp, lds_bytes, smem, nbox, err);
}

// One workgroup per (run, tile).  The tile's bounding box (from the previous
// push, or the tile itself right after a sort) sizes the LDS staging; the new
// box of the pushed particles is written back for the next step.  CS: the
// literal column stride of the boxes (the tile's width and its drift margin),
// used by every tile whose box is no wider; a wider one takes the box's own
// stride.
template <class R, bool UNIT, bool EC, int CS>
__global__ void __launch_bounds__(PUSH_THREADS, sizeof(R) == 4 ? 5 : 3)
k_push_deposit(const Run<R> *__restrict__ runs, const Item *__restrict__ items, int parity, int pp,
               int lds_bytes, unsigned *err, unsigned *stats) {
  __shared__ int nbox[4];
  const Item it = items[blockIdx.x];
  const Run<R> &r = runs[it.run];
  const Parts<R> P = r.pt[pp];
  const int t = it.a;
  const int start = r.tile_start[t], end = r.tile_start[t + 1];
  if (start >= end) return;
  PState<R> s0{};
  if (start + (int)threadIdx.x < end) s0 = load_state(P, start + (int)threadIdx.x);
  const int n1 = r.n1, n2 = r.n2;
  const int t2 = t / r.nt1, t1 = t - t2 * r.nt1;
  const int ref1 = t1 * r.T1, ref2 = t2 * r.T2;  // tile origin
  const int *box = r.tile_box + 6 * t;
  const int lo1 = box[0], hi1 = box[1], lo2 = box[2], hi2 = box[3];
  if (threadIdx.x == 0) {
    nbox[0] = 1 << 30; nbox[1] = -(1 << 30); nbox[2] = 1 << 30; nbox[3] = -(1 << 30);
  }
  // current box: lo-2 .. hi+3; field box: cells lo-1 .. hi+2
  const int W = hi1 - lo1 + 6, H = hi2 - lo2 + 6;
  auto need = [&](int w) { return push_box_bytes(w, H, sizeof(R)); };
  const int f1 = (n1 - r.T1) >> 1, f2 = (n2 - r.T2) >> 1;
  const bool local = need(W) <= lds_bytes;
  if (CS > 0 && W <= CS && need(CS) <= lds_bytes) {
    push_tile<R, UNIT, EC, CS>(r, P, parity, start, end, s0, ref1, ref2, lo1, lo2, W, H, smem_raw,
                               err, nbox);
  } else if (local) {
    push_tile<R, UNIT, EC, 0>(r, P, parity, start, end, s0, ref1, ref2, lo1, lo2, W, H, smem_raw,
                              err, nbox);
  } else {
    const lptr<unsigned char> smem = (lptr<unsigned char>)smem_raw;
    if constexpr (EC)
      push_wide<R, UNIT, true>(&r, t, parity, pp, lds_bytes, smem, (lptr<int>)nbox, err);
    else
      push_wide_call<R, UNIT>(&r, t, parity, pp, lds_bytes, smem, (lptr<int>)nbox, err);
  }
  // new bounding box of the tile's particles; one that reaches past the
  // frame's edge wraps, so it becomes the whole frame
  if (threadIdx.x < 2) {
    const int k = threadIdx.x, f = k ? f2 : f1, n = k ? n2 : n1;
    int lo = nbox[2 * k], hi = nbox[2 * k + 1];
    if (lo < -f || hi >= n - f) {
      lo = -f;
      hi = n - f - 1;
    }
    r.tile_box[6 * t + 2 * k] = lo;
    r.tile_box[6 * t + 2 * k + 1] = hi;
    // (counted last: nothing waits for these atomics)
    if (k == 0) {
      count_stat(stats, STAT_TILES);
      if (!local) count_stat(stats, STAT_FALLBACK);
    }
  }
}

// ---------------------------------------------------------------- tile sort
// Counting sort of the particles of every run by tile and cell of the tile: count,
// exclusive scan over the cells, scatter into the other particle buffer.  The
// order inside a cell is whatever the atomics give; the step's results do not
// depend on any of it.  Sorted by tile alone, particles kept their order of arrival,
// and the lanes of one LDS atomic met on the same nodes (24 runs, 34M particles
// loaded at random: push 667 us, 518 now) or came to (512 x 128 x 128 cells: 1380 us in
// the first 64 steps, 1540 after four sorts, with the push as it was).  What bounds
// it is the scatter's traffic, 80 bytes a particle in pieces of lines (the whole
// sort of the 24 runs 1110 us, 1600 when one workgroup a run scanned and cleared the
// counts and a wave's lanes went to the tiles one by one).

// a / b for 0 <= a < 2^30, 0 < b, and the remainder
__device__ __forceinline__ int div_small(int a, int b, int &rem) {
  return settle_quotient(a, b, (int)((float)a * __builtin_amdgcn_rcpf((float)b)), rem);
}
// Tile of a cell, and the cell's place in the tile.  (Even columns and rows first, so
// that lanes whose nearest node lies beside their cell still differ, moves more
// memory in the scatter and gains the push nothing: 2D 518 and 526 us.)
template <class R>
__device__ __forceinline__ int tile_of(const Run<R> &r, int cell, int &place) {
  int a1, a2, a3 = 0, t3 = 0, i2;
  if (r.dim == 3) {
    i2 = (cell >> r.log2n1) & ((1 << (r.sh3 - r.log2n1)) - 1);
    t3 = div_small(cell >> r.sh3, r.T3, a3);
  } else {
    i2 = cell >> r.log2n1;
  }
  const int t1 = div_small(cell & (r.n1 - 1), r.T1, a1), t2 = div_small(i2, r.T2, a2);
  place = r.area == 1 ? 0 : (a3 * r.T2 + a2) * r.T1 + a1;
  return (t3 * r.nt2 + t2) * r.nt1 + t1;
}

// Block b of n in an order that gives each of the eight dies, to which blocks go in
// turn, a contiguous run of them: the particles of a tile lie in a few blocks, so the
// pieces of a line that they write meet in one L2.  Whole sort, in turn and in runs:
// 2048 x 512 laser 440 and 367 us, its FP64 form at 1024 x 512 264 and 215, four 256 x
// 256 71 and 59, 1024 x 300 68 and 48, the 24 runs 1160 and 1110; 512 x 128 x 128 573
// and 574, as its blocks write few lines together.
__device__ __forceinline__ int die_run(int b, int n) {
  const int per = n >> 3;
  return b < 8 * per ? (b & 7) * per + (b >> 3) : b;
}

template <class R>
__global__ void __launch_bounds__(256) k_sort_clear(const Run<R> *runs, const Item *blocks) {
  const Item it = blocks[blockIdx.x];
  const Run<R> &r = runs[it.run];
  const gptr<int> c = G(r.cell_cnt) + (long long)it.a * SORT_BLOCK;
  const int n = min(SORT_BLOCK, r.ntiles * r.area - it.a * SORT_BLOCK);
  for (int i = threadIdx.x; i < n; i += 256) c[i] = 0;
}

template <class R>
__global__ void __launch_bounds__(256) k_sort_count(const Run<R> *runs, const Item *chunks, int pp) {
  const Item it = chunks[die_run(blockIdx.x, gridDim.x)];
  const Run<R> &r = runs[it.run];
  if (threadIdx.x >= (unsigned)it.b) return;
  int place;
  const int t = tile_of(r, *elem(r.pt[pp].cell, it.a + (int)threadIdx.x), place);
  (void)cell_inc(r.cell_cnt, t * r.area + place);
}

// Exclusive scan of the cell counts within blocks of SORT_BLOCK, and the blocks' sums.
template <class R>
__global__ void __launch_bounds__(256) k_sort_scan(const Run<R> *runs, const Item *blocks) {
  __shared__ int wsum[4];
  const Item it = blocks[blockIdx.x];
  const Run<R> &r = runs[it.run];
  const gptr<int> c = G(r.cell_cnt) + (long long)it.a * SORT_BLOCK;
  const int n = min(SORT_BLOCK, r.ntiles * r.area - it.a * SORT_BLOCK);
  constexpr int PER = SORT_BLOCK / 256;
  const int i0 = (int)threadIdx.x * PER, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int v[PER], s = 0;
#pragma unroll
  for (int k = 0; k < PER; ++k) v[k] = i0 + k < n ? c[i0 + k] : 0;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int x = v[k];
    v[k] = s;
    s += x;
  }
  int inc = s;
  for (int o = 1; o < 64; o <<= 1) {
    const int x = __shfl_up(inc, o);
    if (lane >= o) inc += x;
  }
  if (lane == 63) wsum[w] = inc;
  __syncthreads();
  int base = inc - s;
  for (int k = 0; k < w; ++k) base += wsum[k];
#pragma unroll
  for (int k = 0; k < PER; ++k)
    if (i0 + k < n) c[i0 + k] = base + v[k];
  if (threadIdx.x == 255) G(r.blk_sum)[it.a] = base + s;
}

// The blocks' first particles, and the tiles that start in them.
template <class R>
__global__ void __launch_bounds__(256) k_sort_tiles(const Run<R> *runs, const Item *blocks) {
  __shared__ int wsum[4];
  const Item it = blocks[blockIdx.x];
  const Run<R> &r = runs[it.run];
  int s = 0;
  for (int b = threadIdx.x; b < it.a; b += 256) s += G(r.blk_sum)[b];
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = s;
  __syncthreads();
  const int base = wsum[0] + wsum[1] + wsum[2] + wsum[3];
  if (threadIdx.x == 0) {
    G(r.blk_base)[it.a] = base;
    if (it.a == 0) G(r.tile_start)[r.ntiles] = r.np;
  }
  const int c0 = it.a * SORT_BLOCK, c1 = min(c0 + SORT_BLOCK, r.ntiles * r.area);
  const int first = (c0 + r.area - 1) / r.area;
  for (int t = first + (int)threadIdx.x; t < r.ntiles && t * r.area < c1; t += 256) {
    G(r.tile_start)[t] = base + G(r.cell_cnt)[t * r.area];
    // right after the sort every particle of tile t lies in the tile, which the
    // frame of the push (centred on the tile) always holds whole
    const int t3 = t / (r.nt1 * r.nt2), t12 = t - t3 * r.nt1 * r.nt2;
    const int t2 = t12 / r.nt1, t1 = t12 - t2 * r.nt1;
    const int w[3] = {min(r.T1, r.n1 - t1 * r.T1), min(r.T2, r.n2 - t2 * r.T2),
                      min(r.T3, r.n3 - t3 * r.T3)};
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      G(r.tile_box)[6 * t + 2 * d] = 0;
      G(r.tile_box)[6 * t + 2 * d + 1] = w[d] - 1;
    }
  }
}

template <class R>
__global__ void __launch_bounds__(256) k_sort_scatter(const Run<R> *runs, const Item *chunks, int pp) {
  const Item it = chunks[die_run(blockIdx.x, gridDim.x)];
  const Run<R> &r = runs[it.run];
  if (threadIdx.x >= (unsigned)it.b) return;
  const int p = it.a + (int)threadIdx.x;
  const Parts<R> &A = r.pt[pp];
  const Parts<R> &B = r.pt[pp ^ 1];
  const int c = *elem(A.cell, p);
  int place;
  const int t = tile_of(r, c, place), key = t * r.area + place;
  const int q = cell_inc(r.cell_cnt, key) + G(r.blk_base)[key / SORT_BLOCK];
  const int t0 = G(r.tile_start)[t], cnt = G(r.tile_start)[t + 1] - t0, rank = q - t0;
  // ragged transpose by the tile's particles per cell m: rank r = m j + k goes to
  // column k, row j, so that consecutive slots, the lanes of a wave, hold
  // particles of different cells
  int slot = q;
  if (cnt < 1 << 23) {
    int rem, rest, k;
    const int m = max(1, div_small(cnt + (r.area >> 1), r.area, rest));
    const int rows = div_small(cnt, m, rem), j = div_small(rank, m, k);
    slot = t0 + k * rows + min(k, rem) + j;
  }
  B.cell[slot] = c;
  B.id[slot] = A.id[p];
  B.f1[slot] = A.f1[p];
  B.f2[slot] = A.f2[p];
  if (r.dim == 3) B.f3[slot] = A.f3[p];
  B.u1[slot] = A.u1[p];
  B.u2[slot] = A.u2[p];
  B.u3[slot] = A.u3[p];
  B.qw[slot] = A.qw[p];
}

// ---------------------------------------------------------------- test hook
// Deposit alone on given moves (tests of the fixed-point deposit).
__global__ void k_debug_deposit(int n1, int n2, int P, float inv_wunit, float c3, int np,
                                const int *cell0, const float *off0, const int *cell1,
                                const float *off1, const float *v3, const float *qw,
                                long long *J, unsigned *err) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= np) return;
  const int a1 = cell0[p], a2 = cell0[np + p], b1 = cell1[p], b2 = cell1[np + p];
  const int d1 = wrap_delta_pow2(b1 - a1, n1);
  const int d2 = wrap_delta(b2 - a2, n2);
  if (d1 < -1 || d1 > 1 || d2 < -1 || d2 > 1 || a1 < 0 || a1 >= n1 || a2 < 0 || a2 >= n2) {
    atomicOr(err, ERR_RANGE);
    return;
  }
  const GlobalFixed K{G((unsigned long long *)J), n1, n2, n1 * n2};
  deposit2_fixed<false>(K, P, inv_wunit, c3, a1, a2, off0[p], off0[np + p], d1, d2, off1[p],
                 off1[np + p], v3[p], qw[p]);
}

// ---------------------------------------------------------------- charge density
__global__ void k_rho_fixed(const Run<float> *run, int pp, long long *rho) {
  const Run<float> &r = *run;
  const Parts<float> &P = r.pt[pp];
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= r.np) return;
  const int cell = P.cell[p];
  const int i1 = cell & (r.n1 - 1), i2 = cell >> r.log2n1;
  int s1[3], s2[3];
  const int m1 = fixed_shape<false>(i1, P.f1[p], r.P, s1);
  const int m2 = fixed_shape<false>(i2, P.f2[p], r.P, s2);
  const long long Q = (long long)rintf(P.qw[p] * r.inv_wunit);
#pragma unroll
  for (int b = 0; b < 3; ++b) {
    const int row = wrap_small(m2 - 1 + b, r.n2) * r.n1;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const long long v = Q * (long long)s1[a] * (long long)s2[b];
      if (v != 0)
        atomicAdd((unsigned long long *)(rho + row + wrap_pow2(m1 - 1 + a, r.n1)),
                  (unsigned long long)v);
    }
  }
}

__global__ void k_rho_fp64(const Run<double> *run, int pp, double *rho) {
  const Run<double> &r = *run;
  const Parts<double> &P = r.pt[pp];
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= r.np) return;
  const int cell = P.cell[p];
  const int i1 = cell & (r.n1 - 1), i2 = cell >> r.log2n1;
  const double f1 = P.f1[p], f2 = P.f2[p];
  const int u1 = f1 >= 0.5, u2 = f2 >= 0.5;
  double s1[3], s2[3];
  spline3<double>(f1 - u1, s1);
  spline3<double>(f2 - u2, s2);
#pragma unroll
  for (int b = 0; b < 3; ++b) {
    const int row = wrap_small(i2 + u2 - 1 + b, r.n2) * r.n1;
#pragma unroll
    for (int a = 0; a < 3; ++a)
      unsafeAtomicAdd(rho + row + wrap_pow2(i1 + u1 - 1 + a, r.n1), P.qw[p] * s1[a] * s2[b]);
  }
}

template <class R>
__global__ void k_kinetic(const Run<R> *run, int pp, double *partial) {
  const Run<R> &r = *run;
  const Parts<R> &P = r.pt[pp];
  __shared__ double red[256];
  double acc = 0;
  for (int p = blockIdx.x * blockDim.x + threadIdx.x; p < r.np; p += gridDim.x * blockDim.x) {
    const double u1 = P.u1[p], u2 = P.u2[p], u3 = P.u3[p];
    const double uu = u1 * u1 + u2 * u2 + u3 * u3;
    acc += (double)P.qw[p] * uu / (sqrt(1.0 + uu) + 1.0);  // qw (gamma - 1)
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int w = blockDim.x / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

// ---------------------------------------------------------------- launches
// Literal strides for the tile widths in use; other widths, and the
// energy-conserving gather, take the box's own stride (its kernel gains nothing by
// a literal one: 2048 x 512 laser 140 us without, 144 with; four 256 x 256 38.5 and
// 37.9).
template <class R>
void Launch<R>::push_deposit(const Run<R> *runs, const Item *items, int nitems, int parity, int pp,
                             int lds_bytes, int tile1, bool unit, bool ec, unsigned *err,
                             unsigned *stats, hipStream_t s) {
  if (nitems <= 0) return;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(nitems), dim3(PUSH_THREADS), lds_bytes, s, runs, items, parity,
                       pp, lds_bytes, err, stats);
  };
  constexpr bool F = std::is_same<R, float>::value;
  auto by_width = [&](auto u) {
    constexpr bool U = decltype(u)::value;
    if (ec) return go(k_push_deposit<R, U, true, 0>);
    switch (tile1) {
      case 8: return go(k_push_deposit<R, U, false, push_cols(8)>);
      case 16: return go(k_push_deposit<R, U, false, push_cols(16)>);
      case 32: return go(k_push_deposit<R, U, false, push_cols(32)>);
      case 64: return go(k_push_deposit<R, U, false, push_cols(64)>);
      default: return go(k_push_deposit<R, U, false, 0>);
    }
  };
  if (F && unit)
    by_width(std::integral_constant<bool, F>{});
  else
    by_width(std::false_type{});
}

template <class R>
void Launch<R>::sort(const Run<R> *runs, const Item *chunks, int nchunks, const Item *blocks,
                     int nblocks, int pp, hipStream_t s) {
  if (nchunks <= 0) return;
  hipLaunchKernelGGL(k_sort_clear<R>, dim3(nblocks), dim3(256), 0, s, runs, blocks);
  hipLaunchKernelGGL(k_sort_count<R>, dim3(nchunks), dim3(256), 0, s, runs, chunks, pp);
  hipLaunchKernelGGL(k_sort_scan<R>, dim3(nblocks), dim3(256), 0, s, runs, blocks);
  hipLaunchKernelGGL(k_sort_tiles<R>, dim3(nblocks), dim3(256), 0, s, runs, blocks);
  hipLaunchKernelGGL(k_sort_scatter<R>, dim3(nchunks), dim3(256), 0, s, runs, chunks, pp);
}

template struct Launch<float>;
template struct Launch<double>;

void launch_rho_fixed(const Run<float> *run_dev, int pp, int np, long long *rho, hipStream_t s) {
  if (np <= 0) return;
  hipLaunchKernelGGL(k_rho_fixed, dim3((np + 255) / 256), dim3(256), 0, s, run_dev, pp, rho);
}
void launch_rho_fp64(const Run<double> *run_dev, int pp, int np, double *rho, hipStream_t s) {
  if (np <= 0) return;
  hipLaunchKernelGGL(k_rho_fp64, dim3((np + 255) / 256), dim3(256), 0, s, run_dev, pp, rho);
}

template <class R>
void launch_kinetic(const Run<R> *run_dev, int pp, double *partial, int nblocks, hipStream_t s) {
  hipLaunchKernelGGL(k_kinetic<R>, dim3(nblocks), dim3(256), 0, s, run_dev, pp, partial);
}
template void launch_kinetic<float>(const Run<float> *, int, double *, int, hipStream_t);
template void launch_kinetic<double>(const Run<double> *, int, double *, int, hipStream_t);

void launch_debug_deposit(int n1, int n2, int P, float inv_wunit, float c3, int np,
                          const int *cell0, const float *off0, const int *cell1,
                          const float *off1, const float *v3, const float *qw, long long *J,
                          unsigned *err, hipStream_t s) {
  if (np <= 0) return;
  hipLaunchKernelGGL(k_debug_deposit, dim3((np + 255) / 256), dim3(256), 0, s, n1, n2, P,
                     inv_wunit, c3, np, cell0, off0, cell1, off1, v3, qw, J, err);
}

}  // namespace hp
