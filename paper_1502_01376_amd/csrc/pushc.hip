// pushc.hip -- 2D push with the cubic particle shape on gfx950: quadratic or
// cubic B-spline form factors of order l (Appendix A; Sec. 4 uses cubic
// shapes against the NCI modes the quadratic shape leaves), here l = 3:
// gather over 4 x 4 nodes (the energy-conserving variant drops to the
// quadratic shape along a component's staggered directions), relativistic
// Boris push, and the Esirkepov deposit over a 5 x 5 window.
//
// One workgroup per particle tile of the periodic tile sort, with the tile's
// fields and currents in LDS boxes that follow its particles, as in the
// quadratic push; where they do not fit, LDS holds the currents alone.  FP32
// form: integer cubic weights with exact sum 2^P and the integer Esirkepov
// products of the quadratic kernel, so 2 (rho_new - rho_old) = div J holds
// exactly in the integers and the sums do not depend on the order; FP64 form:
// physical current in FP64.
#include <type_traits>

#include "hpic_internal.h"

namespace hp {

namespace {

// Cubic B-spline weights of the nodes m-1, m, m+1, m+2 for a position m + d,
// d in [0, 1): S3 at the distances 1 + d, d, 1 - d, 2 - d.
template <class R>
__device__ __forceinline__ void cubic4(R d, R w[4]) {
  const R e = R(1) - d;
  w[0] = e * e * e * R(1.0 / 6.0);
  w[1] = (R(4) - R(6) * d * d + R(3) * d * d * d) * R(1.0 / 6.0);
  w[2] = (R(4) - R(6) * e * e + R(3) * e * e * e) * R(1.0 / 6.0);
  w[3] = d * d * d * R(1.0 / 6.0);
}
// Quadratic weights on the same four nodes (m-1 .. m+2) for m + d: the nearest
// node is m (d < 1/2) or m + 1.
template <class R>
__device__ __forceinline__ void quad4(R d, R w[4]) {
  const bool up = d >= R(0.5);
  const R q = up ? d - R(1) : d;
  const R a = R(0.5) - q, b = R(0.5) + q;
  const R s0 = R(0.5) * a * a, s1 = R(0.75) - q * q, s2 = R(0.5) * b * b;
  w[0] = up ? R(0) : s0;
  w[1] = up ? s0 : s1;
  w[2] = up ? s1 : s2;
  w[3] = up ? s2 : R(0);
}
// Stencil along one axis for a component with staggering h (0 or 1/2 cell) at
// cell i with offset f: first node and four weights.
template <class R>
__device__ __forceinline__ int stencil4(int i, R f, bool half, bool lower, R w[4]) {
  int m = i;
  R d = f;
  if (half) {
    if (f >= R(0.5)) {
      d = f - R(0.5);
    } else {
      d = f + R(0.5);
      m = i - 1;
    }
  }
  if (lower)
    quad4<R>(d, w);
  else
    cubic4<R>(d, w);
  return m - 1;
}

// Fields as seen by the gather: a node's pairs (E1, B2) on (i1+1/2, i2) and (E2, B1) on
// (i1, i2+1/2), E3 on (i1, i2), B3 on (i1+1/2, i2+1/2), from the grid or from the tile's
// field box in LDS (row stride FS, or W where FS is 0).
template <class R>
struct GlobalC {
  gptr<const R> F;
  int n1, n2, cells;
  __device__ int col(int i) const { return wrap_pow2(i, n1); }
  __device__ int row(int j) const { return wrap_small(j, n2) * n1; }
  __device__ R get(int c, int r, int a) const { return F[c * (long long)cells + r + col(a)]; }
  __device__ void p0(int r, int a, R &x, R &y) const { x = get(0, r, a); y = get(4, r, a); }
  __device__ void p1(int r, int a, R &x, R &y) const { x = get(1, r, a); y = get(3, r, a); }
  __device__ R e3(int r, int a) const { return get(2, r, a); }
  __device__ R b3(int r, int a) const { return get(5, r, a); }
};
template <class R, int FS>
struct LdsC {
  typedef R T2 __attribute__((ext_vector_type(2)));
  lptr<const T2> P0, P1;
  lptr<const R> E3, B3;
  int W;
  __device__ int row(int j) const { return __mul24(j, FS > 0 ? FS : W); }
  __device__ void p0(int r, int a, R &x, R &y) const { const T2 v = P0[r + a]; x = v.x; y = v.y; }
  __device__ void p1(int r, int a, R &x, R &y) const { const T2 v = P1[r + a]; x = v.x; y = v.y; }
  __device__ R e3(int r, int a) const { return E3[r + a]; }
  __device__ R b3(int r, int a) const { return B3[r + a]; }
};
template <class R> __device__ __forceinline__ R dot4c(const R w[4], const R v[4]) {
  return fmaq(w[3], v[3], fmaq(w[2], v[2], fmaq(w[1], v[1], w[0] * v[0])));
}
// Gather at cell (i1, i2) of the source's frame; EC lowers the order along the
// staggered directions.
template <class R, bool EC, class Src>
__device__ __forceinline__ void gather_c(const Src &S, int i1, int i2, R f1, R f2, R E[3], R B[3]) {
  R wi1[4], wh1[4], wi2[4], wh2[4];
  const int ci = stencil4<R>(i1, f1, false, false, wi1);
  const int ch = stencil4<R>(i1, f1, true, EC, wh1);
  const int ri = stencil4<R>(i2, f2, false, false, wi2);
  const int rh = stencil4<R>(i2, f2, true, EC, wh2);
#pragma unroll
  for (int c = 0; c < 3; ++c) E[c] = B[c] = R(0);
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const int rib = S.row(ri + b), rhb = S.row(rh + b);
    R e1[4], b2[4], e2[4], b1[4], e3[4], b3[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      S.p0(rib, ch + a, e1[a], b2[a]);
      S.p1(rhb, ci + a, e2[a], b1[a]);
      e3[a] = S.e3(rib, ci + a);
      b3[a] = S.b3(rhb, ch + a);
    }
    E[0] = fmaq(wi2[b], dot4c(wh1, e1), E[0]);
    E[1] = fmaq(wh2[b], dot4c(wi1, e2), E[1]);
    E[2] = fmaq(wi2[b], dot4c(wi1, e3), E[2]);
    B[0] = fmaq(wh2[b], dot4c(wi1, b1), B[0]);
    B[1] = fmaq(wi2[b], dot4c(wh1, b2), B[1]);
    B[2] = fmaq(wh2[b], dot4c(wh1, b3), B[2]);
  }
}

// Integer cubic weights of the nodes m-1 .. m+2 for a position m + d: the
// spline values in FP32 (no contraction, so every call site computes the same
// integers from the same offset) scaled by 2^P and rounded, the node m+1
// taking the remainder, so the four sum to 2^P exactly.  |error| of each is a
// few units of 2^-P.
__device__ __forceinline__ void cubic_fixed(float d, int P, int s[4]) {
#pragma clang fp contract(off)
  const float e = 1.0f - d;
  const float sc = (float)(1 << P) * (1.0f / 6.0f);
  s[0] = (int)rintf(e * e * e * sc);
  s[1] = (int)rintf((4.0f - 6.0f * d * d + 3.0f * d * d * d) * sc);
  s[3] = (int)rintf(d * d * d * sc);
  s[2] = (1 << P) - s[0] - s[1] - s[3];
}

// Deposit targets: window() gives row b of component c in the window from (i1, i2), add()
// adds to its column a; at() calls f with the window at the particle's cell plus
// (o1, o2).  LDS box: rows of three component rows, [row][component]
// [column], CS columns (a literal), or W where CS is 0; added to without a test (an
// exact zero changes nothing, and costs less than the test).
template <class A, int CS>
struct SinkLdsC {
  lptr<A> box;
  int W;
  struct Window {
    lptr<A> w;
    int W;
    __device__ __forceinline__ lptr<A> row(int c, int b) const { return w + (3 * b + c) * (CS > 0 ? CS : W); }
    __device__ __forceinline__ void add(lptr<A> r, int a, A v) const {
      __hip_atomic_fetch_add(r + a, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
  };
  __device__ __forceinline__ Window window(int i1, int i2) const {
    return Window{box + (__mul24(i2, 3 * (CS > 0 ? CS : W)) + i1), W};
  }
  template <class F> __device__ __forceinline__ void at(int i1, int i2, int o1, int o2, const F &f) const {
    f(window(i1 + o1, i2 + o2));
  }
};
template <class A>
struct SinkGlobC {
  A *J;
  long long cells;
  int n1, n2;
  struct Window {
    A *J;
    long long cells;
    int n1, n2, i1, i2;
    __device__ __forceinline__ gptr<A> row(int c, int b) const {
      return G(J) + (c * cells + (long long)wrap_small(i2 + b, n2) * n1);
    }
    __device__ __forceinline__ void add(gptr<A> r, int a, A v) const {
      if (v != A(0))
        __hip_atomic_fetch_add(r + wrap_pow2(i1 + a, n1), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  };
  __device__ __forceinline__ Window window(int i1, int i2) const { return Window{J, cells, n1, n2, i1, i2}; }
};
// A particle's deposit into an LDS box that does not hold every particle of the tile:
// at its cell (l1, l2) there, or at its cell of the grid if it is outside.
template <class A>
struct SinkWideC {
  SinkLdsC<A, 0> lds;
  SinkGlobC<A> grid;
  bool in;
  int l1, l2;
  template <class F> __device__ __forceinline__ void at(int i1, int i2, int o1, int o2, const F &f) const {
    if (in)
      f(lds.window(l1 + o1, l2 + o2));
    else
      f(grid.window(i1 + o1, i2 + o2));
  }
};

// Both deposits below leave out what is zero: a particle that keeps its cell along an
// axis has four-node stencils there, so that the window's fifth node and the
// fourth running sum along the axis are zero (the FP64 form's up to the rounding
// of 1 - 1).  The fifth column is left to the lanes that change their cell along
// x1, the fifth row to the waves with a lane that changes it along x2.

// FP64 Esirkepov deposit over the 5 x 5 window: J1 = C1 T2 g1, J2 = C2 T1 g2
// (C the running sums of S1 - S0, T = (S0 + S1)/2), J3 = W3 g3.
template <class Win>
__device__ __forceinline__ void deposit_c(const Win &K, const double S0x[5], const double S1x[5],
                                          const double S0y[5], const double S1y[5], bool sw1,
                                          bool row4, double g1, double g2, double g3) {
  double C1[4], C2[4], T1[5], T2[5];
  double a1 = 0, a2 = 0;
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    a1 = a1 + (S1x[k] - S0x[k]);
    a2 = a2 + (S1y[k] - S0y[k]);
    if (k < 4) {
      C1[k] = a1;
      C2[k] = a2;
    }
    T1[k] = 0.5 * (S0x[k] + S1x[k]);
    T2[k] = 0.5 * (S0y[k] + S1y[k]);
  }
  auto columns = [&](int c0, int c1) {  // of the window's nodes: J1 has one less
#pragma unroll
    for (int b = 0; b < 5; ++b) {
      if (b == 4 && !row4) break;
      const auto j1 = K.row(0, b), j2 = K.row(1, b), j3 = K.row(2, b);
#pragma unroll
      for (int a = c0; a < c1; ++a) {
        if (a > 0) K.add(j1, a - 1, C1[a - 1] * T2[b] * g1);
        if (b < (row4 ? 4 : 3)) K.add(j2, a, C2[b] * T1[a] * g2);
        const double W3 = S0x[a] * S0y[b] * (1.0 / 3.0) + S1x[a] * S0y[b] * (1.0 / 6.0) +
                          S0x[a] * S1y[b] * (1.0 / 6.0) + S1x[a] * S1y[b] * (1.0 / 3.0);
        K.add(j3, a, W3 * g3);
      }
    }
  };
  columns(0, 4);
  if (sw1) columns(4, 5);
}

// Fixed-point Esirkepov deposit over the 5 x 5 window from integer weights
// with exact sum 2^P: J1 = Q C1[a] A2[b], J2 = Q C2[b] A1[a] (C the running
// sums of S1 - S0, A = S0 + S1) as exact integer products, so the integer
// divergence equals twice the integer change of Q S_x S_y node by node; J3 as
// the quadratic kernel's: rint(x0 t0 + x1 t1), x = S h, t0 = 2 S0y + S1y,
// t1 = S0y + 2 S1y (|value| < 2^31 by the choice of c3), left out where |h| < hz
// rounds every value to zero.  UNIT: |Q C| and A fit 24 signed bits, so each
// product is one full-rate 24-bit pair.
template <bool UNIT, class Win>
__device__ __forceinline__ void deposit_cf(const Win &K, const int S0x[5], const int S1x[5],
                                           const int S0y[5], const int S1y[5], bool sw1, bool row4,
                                           int Q, float h, float hz) {
#pragma clang fp contract(off)
  int C1[4], C2[4], A1[5], A2[5];
  int a1 = 0, a2 = 0;
  bool mv2 = false;
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    a1 += S1x[k] - S0x[k];
    a2 += S1y[k] - S0y[k];
    if (k < 4) {
      C1[k] = a1;
      C2[k] = a2;
      mv2 |= a2 != 0;
    }
    A1[k] = S0x[k] + S1x[k];
    A2[k] = S0y[k] + S1y[k];
  }
  auto prod = [&](int c, int qc, int f) -> long long {
    if (UNIT) return mul24_wide(qc, f);
    return ((long long)Q * (long long)c) * (long long)f;
  };
  const bool on3 = !(fabsf(h) < hz);
  int q2[4];
#pragma unroll
  for (int b = 0; b < 4; ++b) q2[b] = UNIT ? mul24_lo(Q, C2[b]) : 0;
  auto columns = [&](int c0, int c1) {  // of the window's nodes: J1 has one less
#pragma unroll
    for (int a = c0 > 0 ? c0 - 1 : 0; a < c1 - 1; ++a) {
      const int qc = UNIT ? mul24_lo(Q, C1[a]) : 0;
#pragma unroll
      for (int b = 0; b < 5; ++b) {
        if (b == 4 && !row4) break;
        K.add(K.row(0, b), a, prod(C1[a], qc, A2[b]));
      }
    }
    if (mv2) {
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        if (b == 3 && !row4) break;
        const auto j2 = K.row(1, b);
#pragma unroll
        for (int a = c0; a < c1; ++a) K.add(j2, a, prod(C2[b], q2[b], A1[a]));
      }
    }
    if (on3) {
      float x0[5], x1[5];
#pragma unroll
      for (int a = c0; a < c1; ++a) {
        x0[a] = (float)S0x[a] * h;
        x1[a] = (float)S1x[a] * h;
      }
#pragma unroll
      for (int b = 0; b < 5; ++b) {
        if (b == 4 && !row4) break;
        const float B0 = (float)S0y[b], B1 = (float)S1y[b];
        const float t0 = 2.0f * B0 + B1;
        const float t1 = B0 + 2.0f * B1;
        const auto j3 = K.row(2, b);
#pragma unroll
        for (int a = c0; a < c1; ++a) {
          const float p1 = x1[a] * t1;
          const float v = __builtin_fmaf(x0[a], t0, p1);
          K.add(j3, a, (long long)(int)rintf(v));
        }
      }
    }
  };
  columns(0, 4);
  if (sw1) columns(4, 5);
}

template <class R>
__device__ __forceinline__ void place5(const R s[4], int off, R out[5]) {
  out[0] = off ? R(0) : s[0];
  out[1] = off ? s[0] : s[1];
  out[2] = off ? s[1] : s[2];
  out[3] = off ? s[2] : s[3];
  out[4] = off ? s[3] : R(0);
}

// Pushes one particle (state s) as the quadratic push does: gather from S and deposit into
// K at the cell (li1, li2) of their frame; false, with no move, if it was rejected.
template <class R, bool UNIT, bool EC, class Src, class Sink>
__device__ __forceinline__ bool push_one_c(const Run<R> &r, float hz, PState<R> &s, int gi1, int gi2,
                                           int li1, int li2, const Src &S, const Sink &K,
                                           unsigned *err, int &d1, int &d2) {
  R u[3] = {s.u1, s.u2, s.u3};
  R E[3], B[3];
  gather_c<R, EC>(S, li1, li2, s.f1, s.f2, E, B);
  boris<R>(r.qmhdt, E, B, u);
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
  // window: nodes from min(cell_old, cell_new) - 1, five per axis
  const int o1 = min(0, d1), o2 = min(0, d2);
  const bool row4 = __ballot(d2 != 0) != 0;
  if constexpr (sizeof(R) == 4) {
    int sa[4], sb[4], S0x[5], S1x[5], S0y[5], S1y[5];
    cubic_fixed(s.f1, r.P, sa);
    cubic_fixed(g1, r.P, sb);
    place5<int>(sa, 0 - o1, S0x);
    place5<int>(sb, d1 - o1, S1x);
    cubic_fixed(s.f2, r.P, sa);
    cubic_fixed(g2, r.P, sb);
    place5<int>(sa, 0 - o2, S0y);
    place5<int>(sb, d2 - o2, S1y);
    const float qs = s.qw * r.inv_wunit;
    const float hv = qs * v[2];
    K.at(li1, li2, o1 - 1, o2 - 1, [&](const auto &W) {
      deposit_cf<UNIT>(W, S0x, S1x, S0y, S1y, d1 != 0, row4, (int)rintf(qs), hv * r.c3, hz);
    });
  } else {
    R sa[4], sb[4], S0x[5], S1x[5], S0y[5], S1y[5];
    cubic4<R>(s.f1, sa);
    cubic4<R>(g1, sb);
    place5<R>(sa, 0 - o1, S0x);
    place5<R>(sb, d1 - o1, S1x);
    cubic4<R>(s.f2, sa);
    cubic4<R>(g2, sb);
    place5<R>(sa, 0 - o2, S0y);
    place5<R>(sb, d2 - o2, S1y);
    K.at(li1, li2, o1 - 1, o2 - 1, [&](const auto &W) {
      deposit_c(W, S0x, S1x, S0y, S1y, d1 != 0, row4, s.qw * r.jfx1, s.qw * r.jfx2, s.qw * v[2]);
    });
  }
  s.cell = (wrap_small(gi2 + d2, r.n2) << r.log2n1) | wrap_pow2(gi1 + d1, r.n1);
  s.f1 = g1;
  s.f2 = g2;
  s.u1 = u[0];
  s.u2 = u[1];
  s.u3 = u[2];
  return true;
}

// |h| below which every value of J3 rounds to zero: the bracket is at most 2 (2/3) (3 2/3)
// 2^(2P) = 2.667 2^(2P); 0.45 leaves room for the FP32 rounding of the products.
template <class R> __device__ __forceinline__ float j3_zero(const Run<R> &r) {
  return uniform((0.45f / 2.667f) / ((float)(1 << r.P) * (float)(1 << r.P)));
}

// The workgroup's tile through LDS boxes with column strides CS (current) and CS - 1
// (fields), or the boxes' own where CS is 0; s0 is the thread's first particle,
// loaded.  Both boxes start at cell lo - 2.
template <class R, bool UNIT, bool EC, int CS>
__device__ __forceinline__ void push_tile_c(const Run<R> &r, const Parts<R> &P, int parity, int start,
                                            int end, PState<R> s0, int ref1, int ref2, int lo1,
                                            int lo2, int W, int H, unsigned char *smem,
                                            unsigned *err, int *nbox) {
  using A = typename AccOf<R>::T;
  using LF = LdsC<R, (CS > 0 ? CS - 1 : 0)>;
  using T2 = typename LF::T2;
  const int n1 = r.n1, n2 = r.n2;
  const long long cells = r.cells;
  const int cs = CS > 0 ? CS : W, fs = cs - 1, jrow = 3 * cs, fnodes = fs * (H - 1);
  const lptr<A> lj = (lptr<A>)smem;
  const lptr<T2> lp0 = (lptr<T2>)(smem + ((jrow * H * (int)sizeof(A) + 15) & ~15));
  const lptr<T2> lp1 = lp0 + fnodes;
  const lptr<R> le3 = (lptr<R>)(lp1 + fnodes);
  const lptr<R> lb3 = le3 + fnodes;
  const gptr<const R> F = G((const R *)r.F);
  const int o1 = ref1 + lo1 - 2, o2 = ref2 + lo2 - 2;
  for_box(W - 1, H - 1, [&](int b, int a) {
    const long long g = (long long)wrap_any(o2 + b, n2) * n1 + wrap_pow2(o1 + a, n1);
    const int q = b * fs + a;
    const R e1 = F[g], e2 = F[cells + g], e3 = F[2 * cells + g];
    const R b1 = F[3 * cells + g], b2 = F[4 * cells + g], b3 = F[5 * cells + g];
    lp0[q] = T2{e1, b2};
    lp1[q] = T2{e2, b1};
    le3[q] = e3;
    lb3[q] = b3;
  });
  for (int q = threadIdx.x; q < jrow * H; q += PUSH_THREADS) lj[q] = 0;
  __syncthreads();
  const LF S{lp0, lp1, le3, lb3, fs};
  const SinkLdsC<A, CS> K{lj, cs};
  const int f1 = (n1 - r.T1) >> 1, f2 = (n2 - r.T2) >> 1;
  const float hz = j3_zero(r);
  CellBox box;
  PState<R> st = s0;
  for (int p = start + (int)threadIdx.x; p < end;) {
    // the next particle's loads are in flight while this one is pushed
    const int pn = p + PUSH_THREADS;
    PState<R> sn = st;
    if (pn < end) sn = load_state(P, pn);
    const int i1 = st.cell & (n1 - 1), i2 = st.cell >> r.log2n1;
    const int l1 = frame_pow2(i1 - ref1, f1, n1), l2 = frame_any(i2 - ref2, f2, n2);
    const int b1 = l1 - lo1 + 2, b2 = l2 - lo2 + 2;
    int d1, d2;
    const bool ok = push_one_c<R, UNIT, EC>(r, hz, st, i1, i2, b1, b2, S, K, err, d1, d2);
    box.add(l1 + d1, l2 + d2);
    arrived(sn);
    if (ok) store_state(P, p, st);
    st = sn;
    p = pn;
  }
  box.reduce(nbox);
  __syncthreads();
  const gptr<A> J = G((A *)r.J[parity]);
  for_box(W, H, [&](int b, int a) {
    const long long g = (long long)wrap_any(o2 + b, n2) * n1 + wrap_pow2(o1 + a, n1);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const A v = lj[b * jrow + c * cs + a];
      if (v != A(0))
        __hip_atomic_fetch_add(J + (c * cells + g), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  });
}

// A tile whose particles have spread so far that the two boxes do not fit: fields
// through the cache, so that the LDS holds twice the current box, and only the particles
// outside that deposit into global memory.  (1024 x 300, eight particles a cell, sorted
// every 16 steps, push with a thermal spread of 0.3: 189 us, 1563 with such tiles in
// global memory; of 1: 228 and 2304; FP64 form of 0.3: 182 and 1624.)
template <class R, bool UNIT, bool EC>
__device__ __forceinline__ void push_wide_c(const Run<R> &r, const Parts<R> &P, int parity, int start, int end,
                                         int ref1, int ref2, int lo1, int hi1, int lo2, int hi2,
                                         int lds_bytes, unsigned char *smem, unsigned *err, int *nbox) {
  using A = typename AccOf<R>::T;
  const int n1 = r.n1, n2 = r.n2;
  const long long cells = r.cells;
  const int f1 = (n1 - r.T1) >> 1, f2 = (n2 - r.T2) >> 1;
  const WideBox w = wide_box(r, P, start, end, ref1, ref2, lo1, hi1, lo2, hi2, lds_bytes / 24, smem);
  const lptr<A> lj = (lptr<A>)smem;
  const int jrow = 3 * w.W, o1 = ref1 + w.lo1 - 2, o2 = ref2 + w.lo2 - 2;
  for (int q = threadIdx.x; q < jrow * w.H; q += PUSH_THREADS) lj[q] = 0;
  __syncthreads();
  const GlobalC<R> S{G((const R *)r.F), n1, n2, r.cells};
  const float hz = j3_zero(r);
  CellBox box;
  for (int p = start + (int)threadIdx.x; p < end; p += PUSH_THREADS) {
    PState<R> s = load_state(P, p);
    const int i1 = s.cell & (n1 - 1), i2 = s.cell >> r.log2n1;
    const int l1 = frame_pow2(i1 - ref1, f1, n1), l2 = frame_any(i2 - ref2, f2, n2);
    const SinkWideC<A> K{{lj, w.W}, {r.J[parity], cells, n1, n2}, w.holds(l1, l2), l1 - w.lo1 + 2, l2 - w.lo2 + 2};
    int d1, d2;
    if (push_one_c<R, UNIT, EC>(r, hz, s, i1, i2, i1, i2, S, K, err, d1, d2)) store_state(P, p, s);
    box.add(l1 + d1, l2 + d2);
  }
  box.reduce(nbox);
  __syncthreads();
  const gptr<A> J = G((A *)r.J[parity]);
  for_box(w.W, w.H, [&](int b, int a) {
    const long long g = (long long)wrap_any(o2 + b, n2) * n1 + wrap_pow2(o1 + a, n1);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const A v = lj[b * jrow + c * w.W + a];
      if (v != A(0))
        __hip_atomic_fetch_add(J + (c * cells + g), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  });
}

}  // namespace

// One workgroup per particle tile (items: run, tile), as the quadratic push: the box of
// the tile's particles (from the previous push, or the tile itself after a sort)
// sizes the LDS boxes, with literal column strides CS for boxes that are no
// wider; where the two do not fit, the LDS holds the current box alone.
//
// What bounds it: the instructions, about 930 a particle (40 to 65 contributions and 96
// field values).  A pass of its own to bound the particles, divisions for every
// node staged and flushed, and a test for every contribution made them 1330: 1024
// x 300, four particles a cell, push 72 us, 49 now; 2048 x 512 189 and 127; FP64 form
// 340 and 232.
template <class R, bool UNIT, bool EC, int CS>
__global__ void __launch_bounds__(PUSH_THREADS, sizeof(R) == 4 ? 5 : 2)
k_push_deposit_cubic(const Run<R> *__restrict__ runs, const Item *__restrict__ items, int parity,
                     int pp, int lds_bytes, unsigned *err) {
  using A = typename AccOf<R>::T;
  __shared__ int nbox[4];
  const Item it = items[blockIdx.x];
  const Run<R> &r = runs[it.run];
  const int t = it.a;
  const int start = G(r.tile_start)[t], end = G(r.tile_start)[t + 1];
  if (start >= end) return;  // the whole workgroup
  const Parts<R> P = r.pt[pp];
  PState<R> s0{};
  if (start + (int)threadIdx.x < end) s0 = load_state(P, start + (int)threadIdx.x);
  const int n1 = r.n1, n2 = r.n2;
  const int t2 = t / r.nt1, t1 = t - t2 * r.nt1;
  const int ref1 = t1 * r.T1, ref2 = t2 * r.T2;
  const auto tbox = G(r.tile_box) + 6 * t;
  const int lo1 = tbox[0], hi1 = tbox[1], lo2 = tbox[2], hi2 = tbox[3];
  if (threadIdx.x == 0) {
    nbox[0] = nbox[2] = 1 << 30;
    nbox[1] = nbox[3] = -(1 << 30);
  }
  const int W = hi1 - lo1 + 6, H = hi2 - lo2 + 6;
  const int f1 = (n1 - r.T1) >> 1, f2 = (n2 - r.T2) >> 1;
  if (CS > 0 && W <= CS && push_box_bytes(CS, H, sizeof(R), 1) <= lds_bytes) {
    push_tile_c<R, UNIT, EC, CS>(r, P, parity, start, end, s0, ref1, ref2, lo1, lo2, W, H, smem_raw,
                                 err, nbox);
  } else if (push_box_bytes(W, H, sizeof(R), 1) <= lds_bytes) {
    push_tile_c<R, UNIT, EC, 0>(r, P, parity, start, end, s0, ref1, ref2, lo1, lo2, W, H, smem_raw, err,
                                nbox);
  } else {
    push_wide_c<R, UNIT, EC>(r, P, parity, start, end, ref1, ref2, lo1, hi1, lo2, hi2, lds_bytes, smem_raw,
                             err, nbox);
  }
  // new box of the tile's particles; one that reaches past the frame's edge wraps, so
  // it becomes the whole frame
  if (threadIdx.x < 2) {
    const int k = threadIdx.x, f = k ? f2 : f1, n = k ? n2 : n1;
    int lo = nbox[2 * k], hi = nbox[2 * k + 1];
    if (lo < -f || hi >= n - f) {
      lo = -f;
      hi = n - f - 1;
    }
    tbox[2 * k] = lo;
    tbox[2 * k + 1] = hi;
  }
}

// Charge density of a run's particles with the cubic shape in the deposit's
// units: FP32 form Q S_x S_y with the integer weights of the deposit (so the
// integer continuity check is exact), FP64 form q w S_x S_y.
template <class R>
__global__ void __launch_bounds__(256) k_rho_cubic(const Run<R> *__restrict__ run, int pp,
                                                   typename AccOf<R>::T *rho) {
  const Run<R> &r = *run;
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= r.np) return;
  const Parts<R> P = r.pt[pp];
  const int cell = P.cell[p];
  const int i1 = cell & (r.n1 - 1), i2 = cell >> r.log2n1;
  if constexpr (sizeof(R) == 4) {
    int w1[4], w2[4];
    cubic_fixed(P.f1[p], r.P, w1);
    cubic_fixed(P.f2[p], r.P, w2);
    const long long Q = (long long)rintf(P.qw[p] * r.inv_wunit);
    for (int b = 0; b < 4; ++b) {
      const long long row = (long long)wrap_small(i2 - 1 + b, r.n2) * r.n1;
      for (int a = 0; a < 4; ++a) {
        const long long v = Q * (long long)w1[a] * (long long)w2[b];
        if (v != 0)
          atomicAdd((unsigned long long *)(rho + row + wrap_pow2(i1 - 1 + a, r.n1)),
                    (unsigned long long)v);
      }
    }
  } else {
    double w1[4], w2[4];
    cubic4<double>(P.f1[p], w1);
    cubic4<double>(P.f2[p], w2);
    const double q = P.qw[p];
    for (int b = 0; b < 4; ++b) {
      const long long row = (long long)wrap_small(i2 - 1 + b, r.n2) * r.n1;
      for (int a = 0; a < 4; ++a)
        unsafeAtomicAdd(rho + row + wrap_pow2(i1 - 1 + a, r.n1), q * w1[a] * w2[b]);
    }
  }
}

template <class R>
void launch_push_cubic(const Run<R> *runs, const Item *items, int nitems, int parity, int pp,
                       int lds_bytes, int tile1, bool unit, bool ec, unsigned *err, hipStream_t s) {
  if (nitems <= 0) return;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(nitems), dim3(PUSH_THREADS), (size_t)lds_bytes, s, runs, items,
                       parity, pp, lds_bytes, err);
  };
  // UNIT selects the 24-bit integer products of the FP32 form; the FP64 form
  // has no integer products and is instantiated without it
  // (the energy-conserving gather gains nothing by a literal stride: 1024 x 300 54.4 us
  // without, 53.8 with)
  constexpr bool F = sizeof(R) == 4;
  auto by_width = [&](auto u) {
    constexpr bool U = decltype(u)::value;
    if (ec) return go(k_push_deposit_cubic<R, U, true, 0>);
    switch (tile1) {
      case 8: return go(k_push_deposit_cubic<R, U, false, push_cols(8)>);
      case 16: return go(k_push_deposit_cubic<R, U, false, push_cols(16)>);
      case 32: return go(k_push_deposit_cubic<R, U, false, push_cols(32)>);
      default: return go(k_push_deposit_cubic<R, U, false, 0>);
    }
  };
  if (F && unit)
    by_width(std::integral_constant<bool, F>{});
  else
    by_width(std::false_type{});
}
template <class R>
void launch_rho_cubic(const Run<R> *run_dev, int pp, int np, typename AccOf<R>::T *rho,
                      hipStream_t s) {
  if (np <= 0) return;
  hipLaunchKernelGGL(k_rho_cubic<R>, dim3((np + 255) / 256), dim3(256), 0, s, run_dev, pp, rho);
}
template void launch_push_cubic<float>(const Run<float> *, const Item *, int, int, int, int, int,
                                       bool, bool, unsigned *, hipStream_t);
template void launch_push_cubic<double>(const Run<double> *, const Item *, int, int, int, int, int,
                                        bool, bool, unsigned *, hipStream_t);
template void launch_rho_cubic<float>(const Run<float> *, int, int, long long *, hipStream_t);
template void launch_rho_cubic<double>(const Run<double> *, int, int, double *, hipStream_t);

}  // namespace hp
