// push3.hip -- particle side of the 3D hybrid Yee-FFT PIC step on gfx950:
// field gather + relativistic Boris push + Esirkepov current deposit in 3D,
// and the 3D charge density of the diagnostics.
//
// One workgroup per particle tile (T1 x T2 x T3 cells), in two passes that share
// one piece of LDS: the tile's particles gather the 27-node quadratic stencil of
// each field component from a copy of the tile's field box and get their new
// momenta; then they move and deposit into an LDS copy of the current box, which
// is added to the global accumulators with one atomic per touched node.  A tile
// whose boxes do not fit is pushed in slabs, or through global memory.
//
// FP32 form: the Esirkepov weights of the FP32 offsets are computed in FP64
// and each node's contribution is rounded once to an integer, accumulated in
// 64 bits: the result does not depend on the order of the atomics.  (An exact
// integer scheme as in 2D would need products of three shape factors plus the
// charge, more than 64 bits for general charges.)
#include "hpic_internal.h"

namespace hp {

// Cell minus tile origin in the tile's frame: the period [-o, n - o), o = (n -
// T) / 2, centred on the tile.
__device__ __forceinline__ int frame_pow2_3(int d, int o, int n) { return ((d + o) & (n - 1)) - o; }
__device__ __forceinline__ int frame_any_3(int d, int o, int n) {
  d += (d < -o) ? n : 0;
  d -= (d >= n - o) ? n : 0;
  return d;
}
// i mod n for any i (a loop of corrections: boxes that fit the LDS reach at
// most a few periods of a small grid)
__device__ __forceinline__ int wrap_any3(int i, int n) {
  while (i >= n) i -= n;
  while (i < 0) i += n;
  return i;
}

__device__ __forceinline__ int wave_min3(int v) {
  for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o));
  return v;
}
__device__ __forceinline__ int wave_max3(int v) {
  for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o));
  return v;
}

__device__ __forceinline__ float rsqrt3(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ double rsqrt3(double x) { return 1.0 / sqrt(x); }
__device__ __forceinline__ float rcp3(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double rcp3(double x) { return 1.0 / x; }

template <class R>
__device__ __forceinline__ void boris3(R qmhdt, const R E[3], const R B[3], R u[3]) {
  const R e0 = qmhdt * E[0], e1 = qmhdt * E[1], e2 = qmhdt * E[2];
  const R m0 = u[0] + e0, m1 = u[1] + e1, m2 = u[2] + e2;
  const R ig = rsqrt3(R(1) + m0 * m0 + m1 * m1 + m2 * m2);
  const R t0 = qmhdt * B[0] * ig, t1 = qmhdt * B[1] * ig, t2 = qmhdt * B[2] * ig;
  const R sf = R(2) * rcp3(R(1) + t0 * t0 + t1 * t1 + t2 * t2);
  const R s0 = t0 * sf, s1 = t1 * sf, s2 = t2 * sf;
  const R p0 = m0 + (m1 * t2 - m2 * t1);
  const R p1 = m1 + (m2 * t0 - m0 * t2);
  const R p2 = m2 + (m0 * t1 - m1 * t0);
  u[0] = m0 + (p1 * s2 - p2 * s1) + e0;
  u[1] = m1 + (p2 * s0 - p0 * s2) + e1;
  u[2] = m2 + (p0 * s1 - p1 * s0) + e2;
}

// FP64 shape factors of one coordinate at the nodes m-1, m, m+1 around the
// nearest node m = cell + (f >= 1/2); d = offset from m (exact).  No
// contraction: the FP32 form's integer deposit is defined operation by
// operation.
__device__ __forceinline__ int dshape3(int cell, double f, double s[3]) {
#pragma clang fp contract(off)
  const int up = (f >= 0.5) ? 1 : 0;
  const double d = up ? (f - 1.0) : f;
  const double a = 0.5 - d, b = 0.5 + d;
  s[0] = 0.5 * (a * a);
  s[1] = 0.75 - d * d;
  s[2] = 0.5 * (b * b);
  return cell + up;
}

template <class T>
__device__ __forceinline__ void place4_3(const T s[3], int off, T out[4]) {
  out[0] = off ? T(0) : s[0];
  out[1] = off ? s[0] : s[1];
  out[2] = off ? s[1] : s[2];
  out[3] = off ? s[2] : T(0);
}

// One node's contribution x y, and sums of two products, in the form's
// arithmetic.  FP32 form: every operation rounded once as written, the node's
// value rounded to an integer.
template <class A> struct Acc3;
template <> struct Acc3<unsigned long long> {
  static __device__ __forceinline__ double sum2(double a, double b, double c, double d) {
#pragma clang fp contract(off)
    const double x = a * b, y = c * d;
    return x + y;
  }
  static __device__ __forceinline__ unsigned long long node(double x, double y) {
#pragma clang fp contract(off)
    const double v = x * y;
    return (unsigned long long)rint_i64(v);
  }
};
template <> struct Acc3<double> {
  static __device__ __forceinline__ double sum2(double a, double b, double c, double d) {
    return __builtin_fma(a, b, c * d);
  }
  static __device__ __forceinline__ double node(double x, double y) { return x * y; }
};
template <class R> struct AccOf3;
template <> struct AccOf3<float> { using T = unsigned long long; };
template <> struct AccOf3<double> { using T = double; };

template <class T> using lptr3 = T __attribute__((address_space(3))) *;
typedef int int4v __attribute__((ext_vector_type(4)));

// Current sinks.  window(): the 4 x 4 x 4 nodes from (b1, b2, b3); put(): adds to
// component comp of the window's node (i, j, k).  The LDS box holds the three
// components of a row next to each other, [k][j][comp][i], so that a node's
// address is the window's plus a uniform offset and a literal one.  (Components
// next to each other at every node would save an addition per row, but put the
// nodes of a row on every third bank: 1866 against 1644 us, 512 x 128 x 128.)  Its atomic is
// issued for zero contributions too: adding an exact zero changes nothing, and
// costs less than the test.
template <class A>
struct Lds3 {
  lptr3<unsigned char> J;
  int CS, RS, PS;  // bytes from component to component, row to row, plane to plane
  struct Window {
    lptr3<unsigned char> w;
    int CS, RS, PS;
    __device__ __forceinline__ void put(int comp, int i, int j, int k, A v) const {
      __hip_atomic_fetch_add((lptr3<A>)(w + (comp * CS + j * RS + k * PS) + 8 * i), v,
                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
  };
  __device__ __forceinline__ Window window(int b1, int b2, int b3) const {
    return Window{J + b1 * 8 + __mul24(b2, RS) + __mul24(b3, PS), CS, RS, PS};
  }
};
template <class A>
struct Global3 {
  gptr<A> J;
  int n1, n2, n3;
  long long cells;
  struct Window {
    gptr<A> J;
    long long cells;
    int row[4][4], col[4];
    __device__ __forceinline__ void put(int comp, int i, int j, int k, A v) const {
      if (v != A(0))
        __hip_atomic_fetch_add(J + (comp * cells + row[k][j] + col[i]), v, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
    }
  };
  __device__ __forceinline__ Window window(int b1, int b2, int b3) const {
    Window w{J, cells};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      w.col[k] = wrap_pow2(b1 + k, n1);
#pragma unroll
      for (int j = 0; j < 4; ++j)
        w.row[k][j] = (wrap_small(b3 + k, n3) * n2 + wrap_small(b2 + j, n2)) * n1;
    }
    return w;
  }
};

// Esirkepov deposit of one particle in 3D.  l[] is the particle's cell in the
// sink's frame, fa[] the old offsets, dd[] the cell moves, fb[] the new
// offsets.  For component d, with (e, f) the other axes in cyclic order:
//   T[i][j] = S0e[i] (2 S0f[j] + S1f[j]) + S1e[i] (S0f[j] + 2 S1f[j])
//           (6 times the Esirkepov bracket), C[k] = running sum of S1d - S0d,
//   J_d[k][i][j] += C[k] g[d] T[i][j],  k = 0..2.
// FP32 form: the weights of the FP32 offsets in FP64, g = (qw inv_wunit) cj
// with cj = 2^40, every FP64 operation rounded once in the order written, the
// node value rounded to a 64-bit integer (j_d = -(dx_d/dt) J / (6 inv_wunit
// cj)): the sums are independent of the order of the atomics and continuity
// holds to about 2^-41 of a particle's charge per node and step (with FP32
// weights and a 2^28 scale, long drifting-beam runs grew a spurious k1 = 0
// mode).  FP64 form: g = qw (-dx_d/dt) / 6, physical current.
// Where no particle of the wave changes its nearest node along an axis, the
// stencil is three nodes wide there (the fourth row of S0 and S1 is zero, the
// last running sum C[2] along that axis only the rounding of 1 - 1) and both
// blocks of terms are skipped for the whole wave.  In the FP32 form the skip
// is exact: the skipped rows add exact zeros, and |C[2]| is a few units of
// 2^-53, so |C[2] g T| < 2^-53 x 8 x 2^40 x 3.4 stays far below the half
// unit that would round away from zero.  The nodes (i, j) of the two other
// axes are walked outside the three running sums, so only one bracket T is
// live at a time (the whole 4 x 4 block of brackets spilled registers).
template <class A, class Sink>
__device__ __forceinline__ void deposit3(const Sink &K, const double g[3], const int l[3],
                                         const double fa[3], const int dd[3], const double fb[3]) {
#pragma clang fp contract(off)
  using Op = Acc3<A>;
  double S0[3][4], S1[3][4], C[3][3];
  int base[3];
  bool w4[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    double sa[3], sb[3];
    const int na = dshape3(l[d], fa[d], sa);
    const int nb = dshape3(l[d] + dd[d], fb[d], sb);
    base[d] = min(na, nb) - 1;
    w4[d] = __ballot(na != nb) != 0;
    place4_3(sa, na - 1 - base[d], S0[d]);
    place4_3(sb, nb - 1 - base[d], S1[d]);
    double acc = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      acc = acc + (S1[d][k] - S0[d][k]);
      C[d][k] = acc;
    }
  }
  const auto W = K.window(base[0], base[1], base[2]);
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const int e = (d + 1) % 3, f = (d + 2) % 3;
    double u0[4], u1[4], cg[3];
#pragma unroll
    for (int j = 0; j < 4; ++j) {  // 2 S is exact
      u0[j] = __builtin_fma(2.0, S0[f][j], S1[f][j]);
      u1[j] = __builtin_fma(2.0, S1[f][j], S0[f][j]);
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) cg[k] = C[d][k] * g[d];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (i == 3 && !w4[e]) continue;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (j == 3 && !w4[f]) continue;
        const double T = Op::sum2(S0[e][i], u0[j], S1[e][i], u1[j]);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          if (k == 2 && !w4[d]) continue;
          const int x[3] = {d == 0 ? k : (e == 0 ? i : j), d == 1 ? k : (e == 1 ? i : j),
                            d == 2 ? k : (e == 2 ? i : j)};
          W.put(d, x[0], x[1], x[2], Op::node(cg[k], T));
        }
      }
    }
  }
}

__device__ __forceinline__ void unpack3(int cell, int log2n1, int sh3, int n1, int &i1, int &i2,
                                        int &i3) {
  i1 = cell & (n1 - 1);
  i2 = (cell >> log2n1) & ((1 << (sh3 - log2n1)) - 1);
  i3 = cell >> sh3;
}

// State of one particle as loaded: cell, offsets, momenta, charge.
template <class R> struct PState3 {
  int cell;
  R f[3], u[3], qw;
};
template <class R>
__device__ __forceinline__ PState3<R> load_state3(const Parts<R> &P, int p) {
  PState3<R> s;
  s.cell = *elem(P.cell, p);
  s.f[0] = *elem(P.f1, p);
  s.f[1] = *elem(P.f2, p);
  s.f[2] = *elem(P.f3, p);
  s.u[0] = *elem(P.u1, p);
  s.u[1] = *elem(P.u2, p);
  s.u[2] = *elem(P.u3, p);
  s.qw = *elem(P.qw, p);
  return s;
}
// Move of a particle of momentum u over a step, in cells.
template <class R>
__device__ __forceinline__ void move3(const Run<R> &r, const R u[3], R m[3]) {
#pragma clang fp contract(off)
  R s = R(1) + u[0] * u[0];
  s = s + u[1] * u[1];
  s = s + u[2] * u[2];
  const R ig = inv_gamma(s);
  m[0] = r.dtdx1 * (u[0] * ig);
  m[1] = r.dtdx2 * (u[1] * ig);
  m[2] = r.dtdx3 * (u[2] * ig);
}

// Sum of one staggered component over its 27 nodes: weights w along the axes,
// row(b, c) the first of three nodes along x1.
template <class R, class F>
__device__ __forceinline__ R gather3(const R w1[3], const R w2[3], const R w3[3], const F &row) {
  R acc = 0;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    R s2 = 0;
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      const auto r = row(b, c);
      s2 = fmaq(w2[b], dot3q(w1, R(r[0]), R(r[1]), R(r[2])), s2);
    }
    acc = fmaq(w3[c], s2, acc);
  }
  return acc;
}
// The same through wrapped node indices.
template <class R>
__device__ __forceinline__ R gather3_at(gptr<const R> F, const R w1[3], const int o1[3],
                                        const R w2[3], const int o2[3], const R w3[3],
                                        const int o3[3]) {
  R acc = 0;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    R s2 = 0;
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      const int r = o3[c] + o2[b];
      s2 = fmaq(w2[b], dot3q(w1, F[r + o1[0]], F[r + o1[1]], F[r + o1[2]]), s2);
    }
    acc = fmaq(w3[c], s2, acc);
  }
  return acc;
}

// a / b for 0 <= a < 1024, 0 < b: the quotient's distance from an integer is at least
// 1 / 2b before it is cut off, the product's error below 2^-12.
__device__ __forceinline__ int small_div(int a, int b) {
  return (int)(((float)a + 0.5f) * __builtin_amdgcn_rcpf((float)b));
}
// Walks the nodes of a box of w x h x d at the grid's (c1, c2, c3) with the workgroup's
// NT threads.  A thread keeps its column (i, j) and walks the planes, N at a time:
// get(u, node in the grid) for each of them, then put(u, i, j, k).
template <int N, int NT, class Get, class Put>
__device__ __forceinline__ void for_box3(int w, int h, int d, int c1, int c2, int c3, int n1, int n2,
                                         int n3, Get get, Put put) {
  const int wh = w * h, step = max(1, NT / wh);  // planes at once
  const int k0 = step > 1 ? small_div((int)threadIdx.x, wh) : 0;
  const int n12 = n1 * n2;
  c2 = wrap_any3(c2, n2);
  c3 = wrap_any3(c3, n3);
  for (int q = (int)threadIdx.x - k0 * wh; q < wh && k0 < step; q += NT) {
    const int j = wh <= 1024 ? small_div(q, w) : q / w, i = q - j * w;
    const int col = wrap_any3(c2 + j, n2) * n1 + wrap_pow2(c1 + i, n1);
    int g3 = wrap_any3(c3 + k0, n3);
    for (int k = k0; k < d; k += N * step) {
#pragma unroll
      for (int u = 0; u < N; ++u) {
        if (k + u * step < d) get(u, (long long)g3 * n12 + col);
        g3 += step;
        while (g3 >= n3) g3 -= n3;
      }
#pragma unroll
      for (int u = 0; u < N; ++u)
        if (k + u * step < d) put(u, i, j, k + u * step);
    }
  }
}

// A tile's place in its run.
struct Tile3 {
  int ref[3], fo[3];  // first cell; the frame along each axis is [-fo, n - fo), centred on the tile
  template <class R>
  __device__ __forceinline__ Tile3(const Run<R> &r, int t) {
    const int t3 = t / (r.nt1 * r.nt2), t12 = t - t3 * r.nt1 * r.nt2;
    const int t2 = t12 / r.nt1, t1 = t12 - t2 * r.nt1;
    ref[0] = t1 * r.T1;
    ref[1] = t2 * r.T2;
    ref[2] = t3 * r.T3;
    fo[0] = (r.n1 - r.T1) >> 1;
    fo[1] = (r.n2 - r.T2) >> 1;
    fo[2] = (r.n3 - r.T3) >> 1;
  }
  // cell of a particle in the grid and in the tile's frame
  template <class R>
  __device__ __forceinline__ void cell(const Run<R> &r, int cell, int gc[3], int l[3]) const {
    unpack3(cell, r.log2n1, r.sh3, r.n1, gc[0], gc[1], gc[2]);
    l[0] = frame_pow2_3(gc[0] - ref[0], fo[0], r.n1);
    l[1] = frame_any_3(gc[1] - ref[1], fo[1], r.n2);
    l[2] = frame_any_3(gc[2] - ref[2], fo[2], r.n3);
  }
};
// Stencil weights (doubled) of a particle, integer (i) and half (h) nodes per axis.
template <class R>
struct Weights3 {
  R wi[3][3], wh[3][3];
  int up[3];
  __device__ __forceinline__ Weights3(const R f[3], bool ec) {
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      up[d] = f[d] >= R(0.5);
      spline3x2<R>(f[d] - R(up[d]), wi[d]);
      half3x2<R>(f[d] - R(0.5), wh[d], ec);
    }
  }
};
// New momentum, and whether the particle moves: a non-finite or a too long move
// leaves it as it was.  (A non-finite momentum makes its move NaN, inf x 0, which
// fails every comparison.)
template <class R>
__device__ __forceinline__ bool kick3(const Run<R> &r, const R E[3], const R B[3], R u[3], unsigned *err) {
  boris3<R>(R(0.125) * r.qmhdt, E, B, u);
  R m[3];
  move3<R>(r, u, m);
  if (fabs(m[0]) < R(1) && fabs(m[1]) < R(1) && fabs(m[2]) < R(1)) return true;
  const bool fin = isfinite(u[0]) && isfinite(u[1]) && isfinite(u[2]) && isfinite(m[0]) &&
                   isfinite(m[1]) && isfinite(m[2]);
  atomicOr(err, fin ? ERR_RANGE : ERR_NUMERIC);
  return false;
}
// Scale of the deposit along each axis.
template <class R>
__device__ __forceinline__ void scale3(const Run<R> &r, R qw, double g[3]) {
  if constexpr (sizeof(R) == 4) {
#pragma clang fp contract(off)
    g[0] = g[1] = g[2] = ((double)qw * (double)r.inv_wunit) * (double)r.cj;
  } else {
    g[0] = qw * r.jfx1 * (1.0 / 6.0);
    g[1] = qw * r.jfx2 * (1.0 / 6.0);
    g[2] = qw * r.jfx3 * (1.0 / 6.0);
  }
}
template <class R>
__device__ __forceinline__ void store_place3(const Run<R> &r, const Parts<R> &P, int p, const int gc[3],
                                             const int dd[3], const R g[3]) {
  *elem(P.cell, p) = (wrap_small(gc[2] + dd[2], r.n3) << r.sh3) |
                     (wrap_small(gc[1] + dd[1], r.n2) << r.log2n1) | wrap_pow2(gc[0] + dd[0], r.n1);
  *elem(P.f1, p) = g[0];
  *elem(P.f2, p) = g[1];
  *elem(P.f3, p) = g[2];
}
// Bounding box of the cells a thread's particles move to, then of the
// workgroup's (nbox, initialised before a barrier).
struct CellBox3 {
  int lo[3] = {1 << 30, 1 << 30, 1 << 30}, hi[3] = {-(1 << 30), -(1 << 30), -(1 << 30)};
  __device__ __forceinline__ void add(const int l[3], const int dd[3]) {
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      lo[d] = min(lo[d], l[d] + dd[d]);
      hi[d] = max(hi[d], l[d] + dd[d]);
    }
  }
  __device__ __forceinline__ void reduce(lptr3<int> nbox) {
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      lo[d] = wave_min3(lo[d]);
      hi[d] = wave_max3(hi[d]);
      if ((threadIdx.x & 63) == 0) {
        __hip_atomic_fetch_min(nbox + 2 * d, lo[d], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __hip_atomic_fetch_max(nbox + 2 * d + 1, hi[d], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    }
  }
};

// A tile whose boxes do not fit the LDS: fields through the cache, current to global
// atomics.  Out of line, so that it takes no registers from the LDS path.
template <class R, int NT>
__device__ __noinline__ void push_tile3_global(const Run<R> *run, int t, int parity, int pp,
                                               lptr3<int> nbox, unsigned *err) {
  using A = typename AccOf3<R>::T;
  const Run<R> &r = *run;
  const Parts<R> P = r.pt[pp];
  const Tile3 T(r, t);
  const int n1 = r.n1, n2 = r.n2, n3 = r.n3, end = G(r.tile_start)[t + 1];
  const long long cells = r.cells;
  const gptr<const R> F = G((const R *)r.F);
  CellBox3 box;
  for (int p = G(r.tile_start)[t] + (int)threadIdx.x; p < end; p += NT) {
    PState3<R> st = load_state3(P, p);
    int gc[3], l[3], dd[3] = {0, 0, 0};
    T.cell(r, st.cell, gc, l);
    const Weights3<R> w(st.f, r.interp != 0);
    int oi[3][3], oh[3][3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      oi[0][a] = wrap_pow2(gc[0] + w.up[0] - 1 + a, n1);
      oh[0][a] = wrap_pow2(gc[0] - 1 + a, n1);
      oi[1][a] = wrap_small(gc[1] + w.up[1] - 1 + a, n2) * n1;
      oh[1][a] = wrap_small(gc[1] - 1 + a, n2) * n1;
      oi[2][a] = wrap_small(gc[2] + w.up[2] - 1 + a, n3) * (n1 * n2);
      oh[2][a] = wrap_small(gc[2] - 1 + a, n3) * (n1 * n2);
    }
    const R E[3] = {gather3_at<R>(F, w.wh[0], oh[0], w.wi[1], oi[1], w.wi[2], oi[2]),
                    gather3_at<R>(F + cells, w.wi[0], oi[0], w.wh[1], oh[1], w.wi[2], oi[2]),
                    gather3_at<R>(F + 2 * cells, w.wi[0], oi[0], w.wi[1], oi[1], w.wh[2], oh[2])};
    const R B[3] = {gather3_at<R>(F + 3 * cells, w.wi[0], oi[0], w.wh[1], oh[1], w.wh[2], oh[2]),
                    gather3_at<R>(F + 4 * cells, w.wh[0], oh[0], w.wi[1], oi[1], w.wh[2], oh[2]),
                    gather3_at<R>(F + 5 * cells, w.wh[0], oh[0], w.wh[1], oh[1], w.wi[2], oi[2])};
    if (kick3<R>(r, E, B, st.u, err)) {
      *elem(P.u1, p) = st.u[0];
      *elem(P.u2, p) = st.u[1];
      *elem(P.u3, p) = st.u[2];
      R m[3], g[3];
      move3<R>(r, st.u, m);
#pragma unroll
      for (int d = 0; d < 3; ++d) dd[d] = advance<R>(st.f[d], m[d], g[d]);
      store_place3<R>(r, P, p, gc, dd, g);
      double gq[3];
      scale3<R>(r, st.qw, gq);
      const double fa[3] = {(double)st.f[0], (double)st.f[1], (double)st.f[2]};
      const double fb[3] = {(double)g[0], (double)g[1], (double)g[2]};
      deposit3<A>(Global3<A>{G((A *)r.J[parity]), n1, n2, n3, cells}, gq, gc, fa, dd, fb);
    }
    box.add(l, dd);
  }
  box.reduce(nbox);
}

// The tile's particles from tile_first to tile_end through the LDS boxes; lo, hi the
// box of their cells, Z the planes of a slab (ONE: all of them, and at most 32
// particles a thread); st the thread's first particle, loaded.
//
// Two passes through one piece of LDS:
// first it holds the fields around the tile [6][k][j][i] (cells lo - 1 .. hi + 2 per
// axis, lo .. hi the tile's particles') and every particle gathers and gets its new
// momentum, then the current box [k][j][3][i] (cells lo - 2 .. hi + 3) and every
// particle moves and deposits.  Where the particles have spread so far that a box does
// not fit, the tile is pushed in slabs of planes that do, each particle in the slab of
// its old cell.
//
// What bounds it: the waits between a workgroup's phases, with the instructions
// (about 1100 a particle) and the LDS (240 accesses) each half busy.  Both boxes
// at once left the LDS to 12 waves of 168 registers on tiles of 8 x 4 x 4 cells;
// taking turns they leave it to 16 waves of 128 on tiles of 8 x 8 x 8, which also halves
// the halo nodes a particle stages and flushes.  512 x 128 x 128 cells, two particles
// a cell, mean over 128 steps: 1530 us before, 1160 now; 128 x 37 x 45, three
// a cell: 85 and 62, 220 and 155 once it is so hot that the boxes outgrow 53 KB; FP64
// form, 128 x 64 x 64: 234 us when it gathered through the cache, 147 now.  (The
// slabs' loops in the same body spilled 26 registers: 1460 us.)
template <class R, int NT, bool ONE>
__device__ __forceinline__ void push_tile3(const Run<R> &r, const Tile3 &T, int tile_first, int tile_end,
                                           int parity, int pp, const int lo[3], const int hi[3], int Z,
                                           PState3<R> st, lptr3<unsigned char> box, lptr3<int> nbox,
                                           unsigned *err) {
  using A = typename AccOf3<R>::T;
  const Parts<R> P = r.pt[pp];
  const int W = hi[0] - lo[0] + 6, H = hi[1] - lo[1] + 6, FW = W - 2, FH = H - 2;
  const int RS = 24 * W, PS = RS * H;
  const int FRS = (int)sizeof(R) * FW, FPS = FRS * FH, FCS = FPS * (Z + 3);
  CellBox3 cbox;
  // up to 32 particles a thread at a time, with a bit each
  for (int start = tile_first; start < tile_end; start += 32 * NT) {
    const int end = ONE ? tile_end : min(tile_end, start + 32 * NT);
    unsigned done = 0;  // pushed, in an earlier slab
    for (int z0 = lo[2]; z0 <= hi[2]; z0 += Z) {
      const int zn = ONE ? Z : min(Z, hi[2] + 1 - z0);
      if (!ONE && (start != tile_first || z0 != lo[2])) __syncthreads();
      {
        // four nodes' loads in flight before their LDS stores: most boxes of the
        // default tiles take one round of memory latency
        R v[4][6];
        const gptr<const R> F = G((const R *)r.F);
        const long long cells = r.cells;
        for_box3<4, NT>(
            FW, FH, zn + 3, T.ref[0] + lo[0] - 1, T.ref[1] + lo[1] - 1, T.ref[2] + z0 - 1, r.n1, r.n2,
            r.n3,
            [&](int u, long long g) {
#pragma unroll
              for (int c = 0; c < 6; ++c) v[u][c] = (F + c * cells)[g];
            },
            [&](int u, int i, int j, int k) {
              const lptr3<unsigned char> node = box + (i * (int)sizeof(R) + j * FRS + k * FPS);
#pragma unroll
              for (int c = 0; c < 6; ++c) *(lptr3<R>)(node + c * FCS) = v[u][c];
            });
      }
      __syncthreads();
      // ---- pass 1: new momenta
      unsigned here = 0, moves = 0;  // of this slab, and not rejected
      for (int p = start + (int)threadIdx.x, k = 0; p < end; p += NT, ++k) {
        if (p != tile_first + (int)threadIdx.x || (!ONE && z0 != lo[2])) st = load_state3(P, p);
        int gc[3], l[3];
        T.cell(r, st.cell, gc, l);
        if (!ONE) {
          if (done >> k & 1 || l[2] < z0 || l[2] >= z0 + Z) continue;
          here |= 1u << k;
        }
        const Weights3<R> w(st.f, r.interp != 0);
        const int u1 = w.up[0] ? (int)sizeof(R) : 0, u2 = w.up[1] ? FRS : 0, u3 = w.up[2] ? FPS : 0;
        const lptr3<unsigned char> hhh = box + (l[0] - lo[0]) * (int)sizeof(R) +
                                         __mul24(l[1] - lo[1], FRS) + __mul24(l[2] - z0, FPS);
        auto comp = [&](int c, int off, const R w1[3], const R w2[3], const R w3[3]) {
          const lptr3<unsigned char> f = hhh + off + c * FCS;
          return gather3(w1, w2, w3, [&](int b, int q) { return (lptr3<const R>)(f + (b * FRS + q * FPS)); });
        };
        R E[3], B[3];
        E[0] = comp(0, u2 + u3, w.wh[0], w.wi[1], w.wi[2]);
        E[1] = comp(1, u1 + u3, w.wi[0], w.wh[1], w.wi[2]);
        E[2] = comp(2, u1 + u2, w.wi[0], w.wi[1], w.wh[2]);
        B[0] = comp(3, u1, w.wi[0], w.wh[1], w.wh[2]);
        B[1] = comp(4, u2, w.wh[0], w.wi[1], w.wh[2]);
        B[2] = comp(5, u3, w.wh[0], w.wh[1], w.wi[2]);
        if (kick3<R>(r, E, B, st.u, err)) {
          *elem(P.u1, p) = st.u[0];
          *elem(P.u2, p) = st.u[1];
          *elem(P.u3, p) = st.u[2];
          moves |= 1u << k;
        }
      }
      __syncthreads();
      for (int q = 16 * (int)threadIdx.x; q < PS * (zn + 5); q += 16 * NT)
        *(lptr3<int4v>)(box + q) = int4v{0, 0, 0, 0};
      __syncthreads();
      // ---- pass 2: move and deposit, last particle first (the thread still holds it)
      const int last = end - 1 - start - (int)threadIdx.x;
      for (int k = last < 0 ? -1 : last / NT, held = 1; k >= 0; --k, held = 0) {
        const int p = start + (int)threadIdx.x + k * NT;
        if (!held) st = load_state3(P, p);
        if (!ONE && !(here >> k & 1)) continue;
        int gc[3], l[3], dd[3] = {0, 0, 0};
        T.cell(r, st.cell, gc, l);
        if (moves >> k & 1) {
          R m[3], g[3];
          move3<R>(r, st.u, m);
#pragma unroll
          for (int d = 0; d < 3; ++d) dd[d] = advance<R>(st.f[d], m[d], g[d]);
          store_place3<R>(r, P, p, gc, dd, g);
          double gq[3];
          scale3<R>(r, st.qw, gq);
          const int lb[3] = {l[0] - lo[0] + 2, l[1] - lo[1] + 2, l[2] - z0 + 2};
          const double fa[3] = {(double)st.f[0], (double)st.f[1], (double)st.f[2]};
          const double fb[3] = {(double)g[0], (double)g[1], (double)g[2]};
          deposit3<A>(Lds3<A>{box, 8 * W, RS, PS}, gq, lb, fa, dd, fb);
        }
        cbox.add(l, dd);
      }
      done |= here;
      __syncthreads();
      const gptr<A> J = G((A *)r.J[parity]);
      const long long cells = r.cells;
      long long g;
      for_box3<1, NT>(
          W, H, zn + 5, T.ref[0] + lo[0] - 2, T.ref[1] + lo[1] - 2, T.ref[2] + z0 - 2, r.n1, r.n2, r.n3,
          [&](int, long long node) { g = node; },
          [&](int, int i, int j, int k) {
            const lptr3<A> node = (lptr3<A>)(box + (i * 8 + j * RS + k * PS));
            const A v[3] = {node[0], node[W], node[2 * W]};
#pragma unroll
            for (int c = 0; c < 3; ++c)
              if (v[c] != A(0))
                __hip_atomic_fetch_add((J + c * cells) + g, v[c], __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
          });
      if (ONE) break;
    }
    if (ONE) break;
  }
  cbox.reduce(nbox);
}

// Slabs, or more particles, out of line as well.
template <class R, int NT>
__device__ __noinline__ void push_tile3_slabs(const Run<R> *run, int t, int parity, int pp, int Z,
                                              lptr3<unsigned char> box, lptr3<int> nbox,
                                              unsigned *err) {
  const Run<R> &r = *run;
  const int first = G(r.tile_start)[t], end = G(r.tile_start)[t + 1];
  const auto b = G(r.tile_box) + 6 * t;
  const int lo[3] = {b[0], b[2], b[4]}, hi[3] = {b[1], b[3], b[5]};
  PState3<R> st{};
  if (first + (int)threadIdx.x < end) st = load_state3(r.pt[pp], first + (int)threadIdx.x);
  push_tile3<R, NT, false>(r, Tile3(r, t), first, end, parity, pp, lo, hi, Z, st, box, nbox, err);
}

// One workgroup of NT threads per tile.
template <class R, int NT>
__global__ void __launch_bounds__(NT, Push3Occupancy<R>::WAVES_PER_SIMD)
k_push_deposit3(const Run<R> *__restrict__ runs, const Item *__restrict__ items, int parity, int pp,
                int lds_bytes, unsigned *err, unsigned *stats) {
  __shared__ int nbox[6];
  const Item it = items[blockIdx.x];
  const Run<R> &r = runs[it.run];
  const Parts<R> P = r.pt[pp];
  const int t = it.a;
  const int tile_first = G(r.tile_start)[t], tile_end = G(r.tile_start)[t + 1];
  if (tile_first >= tile_end) return;
  // the thread's first particle is loaded before the staging, so that its loads
  // wait out the memory latency together with the staging's
  PState3<R> st{};
  if (tile_first + (int)threadIdx.x < tile_end) st = load_state3(P, tile_first + (int)threadIdx.x);
  const Tile3 T(r, t);
  const auto tbox = G(r.tile_box) + 6 * t;
  int lo[3], hi[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    lo[d] = tbox[2 * d];
    hi[d] = tbox[2 * d + 1];
  }
  const int W = hi[0] - lo[0] + 6, H = hi[1] - lo[1] + 6, FW = W - 2, FH = H - 2;
  // Slabs of Z planes of cells whose two boxes both fit; none, or more of their nodes than
  // 64 a particle: through global memory (64 x 33 x 33, one particle a cell, thermal spread
  // 2: 160 us, 217 in slabs alone; from 32 a particle on: 166, 16: 181).
  const int all = hi[2] - lo[2] + 1;
  const int jplane = 24 * (int)min((long long)W * H, 1ll << 20);
  const int fplane = 6 * (int)sizeof(R) * (int)min((long long)FW * FH, 1ll << 20);
  int Z = min(all, min(lds_bytes / jplane - 5, lds_bytes / fplane - 3));
  if (Z > 0 && Z < all && (long long)((all + Z - 1) / Z) * (Z + 5) * W * H > 64ll * (tile_end - tile_first)) Z = 0;
  if (threadIdx.x == 0) {
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      nbox[2 * d] = 1 << 30;
      nbox[2 * d + 1] = -(1 << 30);
    }
    count_stat(stats, STAT_TILES);
    if (Z < 1) count_stat(stats, STAT_FALLBACK);
  }
  const lptr3<unsigned char> box = (lptr3<unsigned char>)smem_raw;
  if (Z == all && tile_end - tile_first <= 32 * NT) {
    push_tile3<R, NT, true>(r, T, tile_first, tile_end, parity, pp, lo, hi, Z, st, box, (lptr3<int>)nbox,
                            err);
  } else {
    __syncthreads();
    if (Z < 1)
      push_tile3_global<R, NT>(&r, t, parity, pp, (lptr3<int>)nbox, err);
    else
      push_tile3_slabs<R, NT>(&r, t, parity, pp, Z, box, (lptr3<int>)nbox, err);
  }
  __syncthreads();
  // the box of the pushed particles; one that reaches past the frame's edge
  // wraps, so it becomes the whole frame
  if (threadIdx.x < 3) {
    const int d = threadIdx.x, o = d == 0 ? T.fo[0] : d == 1 ? T.fo[1] : T.fo[2];
    const int n = d == 0 ? r.n1 : d == 1 ? r.n2 : r.n3;
    int a = nbox[2 * d], b = nbox[2 * d + 1];
    if (a < -o || b >= n - o) {
      a = -o;
      b = n - o - 1;
    }
    tbox[2 * d] = a;
    tbox[2 * d + 1] = b;
  }
}

template <class R>
void Launch<R>::push_deposit3(const Run<R> *runs, const Item *items, int nitems, int parity,
                              int pp, int lds_bytes, unsigned *err, unsigned *stats,
                              hipStream_t s) {
  if (nitems <= 0) return;
  const bool wide = lds_bytes > Push3Occupancy<R>::LDS_3;
  constexpr int NT = Push3Occupancy<R>::NT_MAX;
  hipLaunchKernelGGL((wide ? k_push_deposit3<R, NT> : k_push_deposit3<R, 256>), dim3(nitems),
                     dim3(wide ? NT : 256), lds_bytes, s, runs, items, parity, pp, lds_bytes, err,
                     stats);
}
template void Launch<float>::push_deposit3(const Run<float> *, const Item *, int, int, int, int,
                                           unsigned *, unsigned *, hipStream_t);
template void Launch<double>::push_deposit3(const Run<double> *, const Item *, int, int, int, int,
                                            unsigned *, unsigned *, hipStream_t);

// Charge density in FP64 (diagnostics): rho = qw S1 S2 S3 on the integer
// nodes, from the particles' cells and offsets (either form).
template <class R>
__global__ void k_rho3(const Run<R> *run, int pp, double *rho) {
  const Run<R> &r = *run;
  const Parts<R> &P = r.pt[pp];
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= r.np) return;
  int i1, i2, i3;
  unpack3(P.cell[p], r.log2n1, r.sh3, r.n1, i1, i2, i3);
  double s1[3], s2[3], s3[3];
  const int m1 = dshape3(i1, (double)P.f1[p], s1);
  const int m2 = dshape3(i2, (double)P.f2[p], s2);
  const int m3 = dshape3(i3, (double)P.f3[p], s3);
  const double q = (double)P.qw[p];
  for (int c = 0; c < 3; ++c) {
    const long long pl = (long long)wrap_small(m3 - 1 + c, r.n3) * r.n2;
    for (int b = 0; b < 3; ++b) {
      const long long row = (pl + wrap_small(m2 - 1 + b, r.n2)) * r.n1;
      for (int a = 0; a < 3; ++a)
        unsafeAtomicAdd(rho + row + wrap_pow2(m1 - 1 + a, r.n1), q * s1[a] * s2[b] * s3[c]);
    }
  }
}

template <class R>
void launch_rho3(const Run<R> *run_dev, int pp, int np, double *rho, hipStream_t s) {
  if (np <= 0) return;
  hipLaunchKernelGGL(k_rho3<R>, dim3((np + 255) / 256), dim3(256), 0, s, run_dev, pp, rho);
}
template void launch_rho3<float>(const Run<float> *, int, int, double *, hipStream_t);
template void launch_rho3<double>(const Run<double> *, int, int, double *, hipStream_t);

}  // namespace hp
