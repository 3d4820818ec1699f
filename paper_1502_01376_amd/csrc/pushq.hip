// pushq.hip -- particle side of the quasi-3D (r-z with azimuthal modes) step
// on gfx950: field gather from the modes, relativistic Boris push in Cartesian
// momenta, and the per-mode charge-conserving deposit (Sec. 5 runs the hybrid
// solver per mode; the particle scheme is that of the cited quasi-3D method).
//
// Mode convention F(z, r, th) = sum_m Re(F_m(z, r) e^{i m th}); the phase of a
// particle is P_m = e^{-i m th} = ((x - i y)/r)^m.  Node weights are quadratic
// B-spline products in (z, r) cell units.  The stencil row below the axis
// (row -1) is the mirror point of row 1 (integer-r nodes) or row 0 (half-r
// nodes): z components and scalars of mode m carry (-1)^m there, r and th
// components -(-1)^m.
//
// Deposit of one move (W^0, P^0) -> (W^1, P^1), per mode, with c_0 = 1 and
// c_m = 2: W^1 P^1 - W^0 P^0 = (W^1 - W^0)(P^0 + P^1)/2 + (W^0 + W^1)/2 (P^1 - P^0).
// The first part is split into z and r face fluxes by the Esirkepov
// decomposition in (z, r) index space with the mean phase (separable: the
// running sum of the shape change along one axis times the mean shape along
// the other), the second is an azimuthal flux i c_m q w Wbar (P^1 - P^0) / m.
// Where continuity sets no azimuthal current (m = 0, and m = 1 on the axis
// node) the azimuthal current is deposited directly from the azimuthal
// velocity with the time-averaged weight W3.  Ghost-row fold factors:
// (-1)^m for the z and azimuthal fluxes, -(-1)^m for the flux through the face
// at -dr/2 (it lands on the face at +dr/2) and for the direct azimuthal
// current.  The accumulators hold charge per step (flux times dt), scaled by
// wscale; the row-transform kernel converts them to current densities with
// the face areas and node volumes.
//
// One workgroup per particle tile (particles are counting-sorted by tiles of
// z columns x radial rows every few steps): the FP32 form stages the fields its
// particles gather in LDS, and both forms accumulate the current of the tile's
// box in LDS, which is then added to the global accumulators with one atomic per
// node (particles too far from the rest of their tile gather and deposit in global
// memory).  The deposit's arithmetic (shapes, phases and fluxes of the
// stored positions, their radius and direction in R) is FP64 in both forms;
// the FP32 form rounds each contribution once to a 64-bit integer on a fine
// scale (2^40 per unit charge), so the sums do not depend on the order and
// continuity holds to about 2^-41 of a particle's charge per node and step.
// (With FP32 weights and a 2^28 scale, long drifting-beam runs grew a spurious
// k1 = 0 mode.)
#include "hpic_q3d.h"

namespace hp {

namespace {

__device__ __forceinline__ float rsqrtq(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ double rsqrtq(double x) { return 1.0 / sqrt(x); }
__device__ __forceinline__ float rcpq(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double rcpq(double x) { return 1.0 / x; }

template <class R>
__device__ __forceinline__ void splineq(R d, R w[3]) {
  const R a = R(0.5) - d, b = R(0.5) + d;
  w[0] = R(0.5) * a * a;
  w[1] = fmaq(-d, d, R(0.75));
  w[2] = R(0.5) * b * b;
}

// Floor for the small non-negative arguments used here (r/dr + 1/2 >= 0).
template <class R> __device__ __forceinline__ int ifloorq(R x) { return (int)floor(x); }

// r / dr of a transverse position given as cells + offsets, as its nearest
// integer node m and the offset d = r/dr - m, and the direction (c, s).  The
// offset is formed from the exact integer part of (r/dr)^2 - m^2, so it keeps
// the resolution of the stored offsets anywhere in the column: with
// S = (ix + fx)^2 + (iy + fy)^2, d = (S - m^2) / (r/dr + m).
template <class R>
__device__ __forceinline__ void radial(int ix, R fx, int iy, R fy, int &m, R &d, R &c, R &s) {
#pragma clang fp contract(off)
  const int si = ix * ix + iy * iy;
  const R sf = fx * (R(2 * ix) + fx) + fy * (R(2 * iy) + fy);
  const R rho0 = sqrt(fmax(R(si) + sf, R(0)));
  m = (int)floor(rho0 + R(0.5));
  const R X = R(ix) + fx, Y = R(iy) + fy;
  // within half a cell of the axis ix, iy are 0 or -1 and X, Y are exact
  d = m == 0 ? sqrt(X * X + Y * Y) : (R(si - m * m) + sf) / (rho0 + R(m));
  const R rho = R(m) + d;
  c = rho > R(0) ? X / rho : R(1);
  s = rho > R(0) ? Y / rho : R(0);
}

// a b - c d, the second product rounded.
template <class R> __device__ __forceinline__ R crossq(R a, R b, R c, R d) { return fmaq(a, b, -(c * d)); }

template <class R>
__device__ __forceinline__ void borisq(R qmhdt, const R E[3], const R B[3], R u[3]) {
  const R m0 = fmaq(qmhdt, E[0], u[0]), m1 = fmaq(qmhdt, E[1], u[1]), m2 = fmaq(qmhdt, E[2], u[2]);
  const R ig = rsqrtq(fmaq(m2, m2, fmaq(m1, m1, fmaq(m0, m0, R(1)))));
  const R t0 = qmhdt * B[0] * ig, t1 = qmhdt * B[1] * ig, t2 = qmhdt * B[2] * ig;
  const R sf = R(2) * rcpq(fmaq(t2, t2, fmaq(t1, t1, fmaq(t0, t0, R(1)))));
  const R s0 = t0 * sf, s1 = t1 * sf, s2 = t2 * sf;
  const R p0 = m0 + crossq(m1, t2, m2, t1);
  const R p1 = m1 + crossq(m2, t0, m0, t2);
  const R p2 = m2 + crossq(m0, t1, m1, t0);
  u[0] = fmaq(qmhdt, E[0], m0 + crossq(p1, s2, p2, s1));
  u[1] = fmaq(qmhdt, E[1], m1 + crossq(p2, s0, p0, s2));
  u[2] = fmaq(qmhdt, E[2], m2 + crossq(p0, s1, p1, s0));
}

// Quadratic shape of a coordinate given as cell + offset f in [0,1) along z:
// nodes n-1, n, n+1 around the nearest node n = cell + (f >= 1/2).
template <class R>
__device__ __forceinline__ int zshape(int cell, R f, R s[3]) {
  const int up = f >= R(0.5);
  splineq<R>(f - R(up), s);
  return cell + up;
}
// The same along r for rho = r/dr >= 0 (integer-r nodes).
template <class R>
__device__ __forceinline__ int rshape(R rho, R s[3]) {
  const int n = ifloorq<R>(rho + R(0.5));
  splineq<R>(rho - R(n), s);
  return n;
}
template <class R>
__device__ __forceinline__ void place4(const R s[3], int off, R out[4]) {
  out[0] = off ? R(0) : s[0];
  out[1] = off ? s[0] : s[1];
  out[2] = off ? s[1] : s[2];
  out[3] = off ? s[2] : R(0);
}

// P_m to P_{m+1} = P_m (c - i s).
template <class R> __device__ __forceinline__ void next_phase(R c, R s, R &Pr, R &Pi) {
  const R t = fmaq(Pr, c, Pi * s);
  Pi = fmaq(Pi, c, -(Pr * s));
  Pr = t;
}

// One mode of one staggered component at the particle: the complex
// interpolated value (vx, vy) from weights wz/wr, node columns oz[3] and rows
// rr[3] (a ghost row already mirrored; ghost0: row 0 of the stencil is the
// ghost, whose sign depends on the mode parity and on whether the component is
// a z component or a transverse one).  F points at the mode's plane of the
// component, in global memory (row stride n1) or in a wave's LDS copy of the
// fields around its particles (row stride the box width, columns relative to
// the box).
template <class R, class PC, class I>
__device__ __forceinline__ void gather_q(PC F, const R wz[3], const int oz[3], const R wr[3],
                                         const int rr[3], bool ghost0, bool odd, bool vec,
                                         I rowstride, R &vx, R &vy) {
  vx = 0;
  vy = 0;
#pragma unroll
  for (int b = 0; b < 3; ++b) {
    const PC row = F + rr[b] * rowstride;
    const auto v0 = row[oz[0]], v1 = row[oz[1]], v2 = row[oz[2]];
    R w = wr[b];
    if (b == 0 && ghost0 && odd != vec) w = -w;  // (-1)^m for z components, -(-1)^m for r, th
    vx = fmaq(w, dot3q(wz, v0.x, v1.x, v2.x), vx);
    vy = fmaq(w, dot3q(wz, v0.y, v1.y, v2.y), vy);
  }
}

__device__ __forceinline__ int wmin(int v) {
  for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o));
  return v;
}
__device__ __forceinline__ int wmax(int v) {
  for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o));
  return v;
}
// A complex value as a clang vector (copyable to and from LDS).
template <class R> struct LdsC;
template <> struct LdsC<float> { typedef float T __attribute__((ext_vector_type(2))); };
template <> struct LdsC<double> { typedef double T __attribute__((ext_vector_type(2))); };

// One contribution x y in the accumulator's type: FP32 form the nearest 64-bit
// integer (|x y| < 2^44: charges are scaled to at most 2^40 and every weight
// factor is at most 4 in magnitude), rounded once by the fused multiply-add that
// brings it next to 1.5 2^52; FP64 form the product.
template <class A> __device__ __forceinline__ A acc_mul(double x, double y);
template <> __device__ __forceinline__ long long acc_mul<long long>(double x, double y) {
  return __double_as_longlong(__builtin_fma(x, y, 6755399441055744.0)) - 0x4338000000000000LL;
}
template <> __device__ __forceinline__ double acc_mul<double>(double x, double y) { return x * y; }

// Deposit targets: the tile's LDS box, or the global accumulators.  A node row is
// found once per move (row()) and serves every component, mode and part, whose
// slot() is a distance from it.
//
// LDS box: [row][slot][column], CW columns (a literal), slots in the order
// component, then m = 0, then the real and imaginary parts of m = 1, 2, ..
template <class A, int MC, int CW>
struct SinkLdsQ {
  lptr<A> box;  // the window's first column in row 0 (may lie below the LDS box)
  int M;
  using Row = lptr<A>;
  __device__ __forceinline__ int per() const { return MC > 0 ? 2 * MC - 1 : 2 * M - 1; }
  __device__ __forceinline__ Row row(int j) const { return box + __mul24(j, q_row(CW, MC > 0 ? MC : M)); }
  __device__ __forceinline__ int slot(int c, int m) const { return (c * per() + (m == 0 ? 0 : 2 * m - 1)) * CW; }
  __device__ __forceinline__ void put(Row r, int slot, int part, int a, double x, double y) const {
    __hip_atomic_fetch_add(r + slot + part * CW + a, acc_mul<A>(x, y), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_WORKGROUP);
  }
};
template <class A>
struct SinkGlobQ {
  A *J;
  long long plane;
  int n1, bz;
  using Row = long long;
  __device__ __forceinline__ Row row(int j) const { return (long long)j * n1; }
  __device__ __forceinline__ long long slot(int c, int m) const { return (m * 3 + c) * plane; }
  __device__ __forceinline__ void put(Row r, long long slot, int part, int a, double x, double y) const {
    const A q = acc_mul<A>(x, y);
    if (q != A(0))
      __hip_atomic_fetch_add(G(J) + 2 * (slot + r + wrap_pow2(bz + a, n1)) + part, q,
                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
};
__device__ __forceinline__ void glob_add(gptr<long long> p, long long v) {
  __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void glob_add(gptr<double> p, double v) {
  __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Per-mode deposit of one move (see the file header) through K, whose columns
// start at the window's: window shapes S0/S1 along z and r (first row br >= -1),
// the old and new directions (cta, sta), (ctb, stb) (phases P_m = (c - i s)^m by
// the same recurrence for both, so the new phase of one step is bit for bit the
// old phase of the next), scaled charge g and v_th dt.
//
// A particle that keeps its nearest node along an axis has three-node stencils
// there: the window's fourth node and the third running sum along the axis are
// zero (the sum up to the rounding of 1 - 1, which the FP32 form rounds away).
// The fourth column is left to the lanes that change their node along z (zswitch),
// the fourth row to the waves with a lane that changes it along r (rswitch, wave-
// uniform); everything else is added without a test.
template <int MC, class Sink>
__device__ __forceinline__ void deposit_q(const Sink &K, int M, double S0z[4],
                                          double S1z[4], double S0r[4],
                                          double S1r[4], int br, bool zswitch, bool rswitch,
                                          double cta, double sta, double ctb, double stb, double g,
                                          double vthdt) {
  using D = double;
  D Cz[3], Cr[3];
  {
    D az = 0, ar = 0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      az = az + (S1z[k] - S0z[k]);
      ar = ar + (S1r[k] - S0r[k]);
      Cz[k] = az;
      Cr[k] = ar;
    }
  }
  // rows: node rows |br + b|; the face below the axis lands on face 0
  const bool ghost = br < 0;
  typename Sink::Row row[4];
  row[0] = K.row(ghost ? 1 : br);
#pragma unroll
  for (int b = 1; b < 4; ++b) row[b] = K.row(br + b);
  const typename Sink::Row face0 = K.row(ghost ? 0 : br);
  const bool axis = __ballot(br <= 0) != 0;  // some lane's window holds the axis row
  D P0r = 1, P0i = 0;  // phase at the old position
  D P1r = 1, P1i = 0;  // phase at the new position
  if (MC > 0) M = MC;
  for (int m = 0; m < M; ++m) {
    if constexpr (MC == 0) {
#pragma unroll
      for (int a = 0; a < 4; ++a) asm volatile("" : "+v"(S0z[a]), "+v"(S1z[a]), "+v"(S0r[a]), "+v"(S1r[a]));
    }
    if (m > 0) {
      next_phase(cta, sta, P0r, P0i);
      next_phase(ctb, stb, P1r, P1i);
    }
    const D cm = m == 0 ? 1.0 : 2.0;
    const D even = (m & 1) ? -1.0 : 1.0;  // (-1)^m
    const D Pmr = 0.5 * (P0r + P1r), Pmi = 0.5 * (P0i + P1i);
    const D qr = -0.5 * cm * g * Pmr, qi = -0.5 * cm * g * Pmi;
    const D fold = ghost ? even : 1.0;    // of the first row's node fluxes
    // z faces: running sum along z times the mean radial shape
    {
      const auto s = K.slot(0, m);
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        if (b == 3 && !rswitch) break;
        const D T = (S0r[b] + S1r[b]) * (b == 0 ? fold : 1.0);
        const D xr = qr * T, xi = qi * T;
        K.put(row[b], s, 0, 0, xr, Cz[0]);
        K.put(row[b], s, 0, 1, xr, Cz[1]);
        if (m > 0) {
          K.put(row[b], s, 1, 0, xi, Cz[0]);
          K.put(row[b], s, 1, 1, xi, Cz[1]);
        }
        if (zswitch) {
          K.put(row[b], s, 0, 2, xr, Cz[2]);
          if (m > 0) K.put(row[b], s, 1, 2, xi, Cz[2]);
        }
      }
    }
    // r faces (face j at (j + 1/2) dr): running sum along r times the mean z shape
    {
      const auto s = K.slot(1, m);
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        if (b == 2 && !rswitch) break;
        const D T = b == 0 ? Cr[0] * (ghost ? -even : 1.0) : Cr[b];
        const D xr = qr * T, xi = qi * T;
        const auto f = b == 0 ? face0 : row[b];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          const D t = S0z[a] + S1z[a];
          K.put(f, s, 0, a, xr, t);
          if (m > 0) K.put(f, s, 1, a, xi, t);
        }
        if (zswitch) {
          const D t = S0z[3] + S1z[3];
          K.put(f, s, 0, 3, xr, t);
          if (m > 0) K.put(f, s, 1, 3, xi, t);
        }
      }
    }
    // azimuthal current: m = 0 from the azimuthal velocity with the weight W3,
    // m > 0 the flux i c_m q w Wbar (P1 - P0) / m (none on the axis row)
    {
      const auto s = K.slot(2, m);
      const D h = m == 0 ? g * vthdt * (1.0 / 6.0) : 0.5 * cm * g / (D)m;
      const D xr = m == 0 ? 1.0 : -(P1i - P0i), xi = P1r - P0r;
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        if (b == 3 && !rswitch) break;
        D k0, k1;
        if (m == 0) {
          const D hb = b == 0 && ghost ? -h : h;
          k0 = hb * (2.0 * S0r[b] + S1r[b]);
          k1 = hb * (S0r[b] + 2.0 * S1r[b]);
        } else {
          D hb = b == 0 ? h * fold : h;
          if (b < 2) hb = (b == 0 ? br == 0 : br == -1) ? 0.0 : hb;
          k0 = hb * S0r[b];
          k1 = hb * S1r[b];
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          const D w = fmaq(S0z[a], k0, S1z[a] * k1);
          K.put(row[b], s, 0, a, w, xr);
          if (m > 0) K.put(row[b], s, 1, a, w, xi);
        }
        if (zswitch) {
          const D w = fmaq(S0z[3], k0, S1z[3] * k1);
          K.put(row[b], s, 0, 3, w, xr);
          if (m > 0) K.put(row[b], s, 1, 3, w, xi);
        }
      }
      // m = 1 on the axis row: the direct current
      if (m == 1 && axis) {
        const D h1 = cm * g * vthdt * (1.0 / 6.0);
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          if (b == 0 ? br != 0 : br != -1) continue;
          const D k0 = h1 * (2.0 * S0r[b] + S1r[b]), k1 = h1 * (S0r[b] + 2.0 * S1r[b]);
#pragma unroll
          for (int a = 0; a < 4; ++a) {
            if (a == 3 && !zswitch) break;
            const D w = fmaq(S0z[a], k0, S1z[a] * k1);
            K.put(row[b], s, 0, a, w, Pmr);
            K.put(row[b], s, 1, a, w, Pmi);
          }
        }
      }
    }
  }
}

// One move of a particle: from cell cz with z offset fz, by dz cells to offset
// gz; radial nodes mri, mrb with offsets dri, drb; old and new directions; scaled
// charge g; v_th dt.
struct MoveQ {
  int cz, dz, mri, mrb;
  double fz, gz, dri, drb, ct, st, ctb, stb, g, vthdt;
};
// Builds the 4-node windows along z and r holding both stencils and deposits
// through the sink that sink(bz) gives for the window's first column bz.
template <int MC, class F>
__device__ __forceinline__ void deposit_move(const MoveQ &v, int M, const F &sink) {
  using D = double;
  D S0z[4], S1z[4], S0r[4], S1r[4];
  D sa[3], sb[3];
  const int na = zshape<D>(v.cz, v.fz, sa);
  const int nb = zshape<D>(v.cz + v.dz, v.gz, sb);
  const int bz = min(na, nb) - 1;
  place4<D>(sa, na - 1 - bz, S0z);
  place4<D>(sb, nb - 1 - bz, S1z);
  splineq<D>(v.dri, sa);
  splineq<D>(v.drb, sb);
  const int br = min(v.mri, v.mrb) - 1;
  place4<D>(sa, v.mri - 1 - br, S0r);
  place4<D>(sb, v.mrb - 1 - br, S1r);
  deposit_q<MC>(sink(bz), M, S0z, S1z, S0r, S1r, br, na != nb, __ballot(v.mri != v.mrb) != 0, v.ct,
                v.st, v.ctb, v.stb, v.g, v.vthdt);
}

// The rare global-atomic path out of line, with plain arguments (no array
// whose address is taken), so that it adds neither registers nor scratch
// memory to the LDS path.
template <class A>
__device__ __noinline__ void deposit_move_global(A *J, long long plane, int n1, int M, int cz,
                                                 double fz, int dz, double gz, int mri, double dri,
                                                 int mrb, double drb, double ct, double st,
                                                 double ctb, double stb, double g, double vthdt) {
  deposit_move<0>(MoveQ{cz, dz, mri, mrb, fz, gz, dri, drb, ct, st, ctb, stb, g, vthdt}, M,
                  [&](int bz) { return SinkGlobQ<A>{J, plane, n1, bz}; });
}

// State of one particle as loaded.
template <class R>
struct PStateQ {
  int cell, ix, iy;
  R fz, fx, fy, u[3], qw;
};
template <class R>
__device__ __forceinline__ PStateQ<R> load_q(const PartsQ<R> &P, int p) {
  PStateQ<R> s;
  s.cell = *elem(P.cell, p);
  s.ix = *elem(P.ix, p);
  s.iy = *elem(P.iy, p);
  s.fz = *elem(P.fz, p);
  s.fx = *elem(P.fx, p);
  s.fy = *elem(P.fy, p);
  s.u[0] = *elem(P.uz, p);
  s.u[1] = *elem(P.ux, p);
  s.u[2] = *elem(P.uy, p);
  s.qw = *elem(P.qw, p);
  return s;
}

// The columns (x .. y) and nearest nodes (z .. w) whose particles a push's LDS boxes
// hold where a segment's own box is too large for them: as many as fit, around the
// particles' mean.  Called by the whole workgroup.
template <class R>
__device__ __forceinline__ int4 q_window(const RunQ<R> &r, const QSeg *seg, int cols, int rows,
                                         lptr<unsigned char> smem) {
  const PartsQ<R> &P = r.pt;
  const auto s = G(seg);
  const int start = s->start, end = s->end, fo = (r.n1 - r.sbz) >> 1, z0 = s->tile / r.nbr * r.sbz;
  int4 w = make_int4(s->zlo, s->zhi, s->rlo, s->rhi);
  long long sz = 0, sr = 0;
  for (int p = start + (int)threadIdx.x; p < end; p += 256) {
    const float x = (float)*elem(P.ix, p) + (float)*elem(P.fx, p);
    const float y = (float)*elem(P.iy, p) + (float)*elem(P.fy, p);
    sz += frame_pow2(*elem(P.cell, p) - z0, fo, r.n1);
    sr += (int)(sqrtf(x * x + y * y) + 0.5f);
  }
  int mz, mr;
  group_mean(sz, sr, end - start, (unsigned char *)smem, mz, mr);
  auto clamp = [](int &lo, int &hi, int mean, int n) {
    if (hi - lo < n) return;
    lo = max(lo, min(mean - (n - 1) / 2, hi - (n - 1)));
    hi = lo + n - 1;
  };
  clamp(w.x, w.y, mz, cols);
  clamp(w.z, w.w, mr, rows);
  return w;
}

// A segment with boxes of CW columns for the particles in columns clo .. chi and at nodes
// mlo .. mhi: all of them (ALL), or the others gather and deposit in global memory.  st is
// the thread's first particle, loaded.
template <class R, int MC, int CW, bool ALL, bool STAGE>
__device__ __forceinline__ void q_push(const RunQ<R> &r, const QSeg *qseg, int parity, int clo, int chi,
                                       int mlo, int mhi, PStateQ<R> st, lptr<unsigned char> smem,
                                       lptr<int> nbox, unsigned *err) {
  constexpr int NT = 256;
  using A = typename AccQ<R>::T;
  using V2 = typename LdsC<R>::T;
  constexpr int FWD = CW - 2;
  const gptr<QSeg> seg = G((QSeg *)qseg);
  const int t = seg->tile, start = seg->start, end = seg->end;
  const PartsQ<R> P = r.pt;
  const int n1 = r.n1, M = MC > 0 ? MC : r.M;
  const long long plane = r.plane;
  const int z0 = (t / r.nbr) * r.sbz;   // first column of the tile
  const int fo = (n1 - r.sbz) >> 1;     // the tile's frame along z: [-fo, n1 - fo), centred on it
  const int per = 2 * M - 1, NS = 3 * per;
  const int RS = q_row(CW, M);                  // one row of the current box
  // one row of the field box: six components of mode 0 (the real part, all that
  // the gather takes of it), then of each further mode, complex; its used size
  const int FS = q_field_row(CW, M);
  const int zlo = clo - 2, W = chi - clo + 6, Wf = W - 2;
  const int rlo = max(0, mlo - 2), H = min(mhi + 2, r.n2) - rlo + 1, Hf = H - 1;
  const lptr<A> box = (lptr<A>)smem;
  const lptr<R> fbox = (lptr<R>)(smem + RS * H * (int)sizeof(A));
  const gptr<const V2> F = G((const V2 *)r.F);
  for (int q = threadIdx.x; q < RS * H; q += NT) box[q] = 0;
  if constexpr (STAGE) {
    // half a wave per (row, mode): its six components' loads all in flight
    // before their LDS stores
    const int cc = threadIdx.x & 31;
    if (cc < Wf)
      for (int e = (int)threadIdx.x >> 5; e < Hf * M; e += NT / 32) {
        const int j = e / M, m = e - j * M;
        const gptr<const V2> src = F + (long long)(6 * m) * plane + (long long)(rlo + j) * n1 +
                       wrap_pow2(z0 + zlo + 1 + cc, n1);
        V2 v[6];
#pragma unroll
        for (int c = 0; c < 6; ++c) v[c] = src[c * plane];
        const lptr<R> row = fbox + j * FS;
        if (m == 0) {
#pragma unroll
          for (int c = 0; c < 6; ++c) row[c * FWD + cc] = v[c].x;
        } else {
          const lptr<V2> crow = (lptr<V2>)(row + (12 * m - 6) * FWD);
#pragma unroll
          for (int c = 0; c < 6; ++c) crow[c * FWD + cc] = v[c];
        }
      }
  }
  __syncthreads();
  int blo = 1 << 30, bhi = -(1 << 30), rlo2 = 1 << 30, rhi2 = -(1 << 30);
  for (int p = start + (int)threadIdx.x; p < end; p += NT) {
    if (p != start + (int)threadIdx.x) st = load_q(P, p);
    const int cz = st.cell, ix = st.ix, iy = st.iy;
    const R fz = st.fz, fx = st.fx, fy = st.fy;
    R u[3] = {st.u[0], st.u[1], st.u[2]};
    const int relz = ((cz - z0 + fo) & (n1 - 1)) - fo;
    // nearest integer-r node mri with offset dri, nearest half-r node (j + 1/2)
    // mrh with offset drh, direction (ct, sn)
    int mri;
    R dri, ct, sn;
    radial<R>(ix, fx, iy, fy, mri, dri, ct, sn);
    const int mrh = dri >= R(0) ? mri : mri - 1;
    const R drh = dri >= R(0) ? dri - R(0.5) : dri + R(0.5);
    const bool in = ALL || (relz >= clo && relz <= chi && mri >= mlo && mri <= mhi);
    // ---- gather: integer (i) and half (h) stencils along z, weights halved, and r,
    // weights doubled
    R wzi[3], wzh[3], wri[3], wrh[3];
    const int upz = fz >= R(0.5);
    spline3h<R>(fz - R(upz), wzi);
    half3h<R>(fz - R(0.5), wzh, r.interp != 0);
    spline3x2<R>(dri, wri);
    half3x2<R>(drh, wrh, r.interp != 0);
    const bool gi = mri == 0, gh = mrh == 0;  // ghost row in the stencil
    // sum over the modes of Re(F_m e^{i m th}), with P_m = (ct - i sn)^m by
    // recurrence (m = 0: the real part alone)
    R Ec[3] = {0, 0, 0}, Bc[3] = {0, 0, 0};
    R Pr = 1, Pi = 0;
    // (four modes in line spill 17 registers of the FP32 form: push of 1024 x 160 198 us, 180 so)
    constexpr int MU = STAGE && MC > 3 ? 1 : MC > 0 ? MC : 1;
    int rri[3], rrh[3];
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      const int ji = mri - 1 + b, jh = mrh - 1 + b;
      rri[b] = ji < 0 ? -ji : ji;
      rrh[b] = jh < 0 ? -jh - 1 : jh;
    }
    if (STAGE && in) {
      // first node of each stencil row, integer (i) or half (h) along z and r
      int oi[3], oh[3];
      const int c0 = relz - zlo - 2;
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        oi[b] = __mul24(rri[b] - rlo, FS);
        oh[b] = __mul24(rrh[b] - rlo, FS);
      }
      {
        auto sum = [&](int z, const int o[3], int c, const R wz[3], const R wr[3], R sign) {
          R v = 0;
#pragma unroll
          for (int b = 0; b < 3; ++b) {
            const lptr<const R> row = fbox + (o[b] + z) + c * FWD;
            v = fmaq(b == 0 ? wr[0] * sign : wr[b], dot3q(wz, row[0], row[1], row[2]), v);
          }
          return v;
        };
        // ghost rows of mode 0: as they are for z components, negative for r, th
        const R si = gi ? R(-1) : R(1), sh = gh ? R(-1) : R(1);
        const int zi = c0 + upz, zh = c0;
        Ec[0] = sum(zh, oi, 0, wzh, wri, R(1));
        Ec[1] = sum(zi, oh, 1, wzi, wrh, sh);
        Ec[2] = sum(zi, oi, 2, wzi, wri, si);
        Bc[0] = sum(zi, oh, 3, wzi, wrh, R(1));
        Bc[1] = sum(zh, oi, 4, wzh, wri, si);
        Bc[2] = sum(zh, oh, 5, wzh, wrh, sh);
      }
#pragma unroll MU
      for (int m = 1; m < M; ++m) {
        next_phase(ct, sn, Pr, Pi);
        // ghost rows: (-1)^m for z components, -(-1)^m for r, th
        const R odd = (m & 1) ? R(-1) : R(1);
        const R szi = gi ? odd : R(1), svi = gi ? -odd : R(1);
        const R szh = gh ? odd : R(1), svh = gh ? -odd : R(1);
        const int zi = 2 * (c0 + upz), zh = 2 * c0;
        // Re(v e^{i m th}) with P = e^{-i m th}
        auto sum = [&](int z, const int o[3], int c, const R wz[3], const R wr[3], R sign) {
          R vx = 0, vy = 0;
#pragma unroll
          for (int b = 0; b < 3; ++b) {
            const lptr<const V2> row =
                (lptr<const V2>)(fbox + (o[b] + z)) + ((6 * m - 3) + c) * FWD;
            const V2 f0 = row[0], f1 = row[1], f2 = row[2];
            const R w = b == 0 ? wr[0] * sign : wr[b];
            vx = fmaq(w, dot3q<R>(wz, f0.x, f1.x, f2.x), vx);
            vy = fmaq(w, dot3q<R>(wz, f0.y, f1.y, f2.y), vy);
          }
          return fmaq(vx, Pr, vy * Pi);
        };
        Ec[0] += sum(zh, oi, 0, wzh, wri, szi);
        Ec[1] += sum(zi, oh, 1, wzi, wrh, svh);
        Ec[2] += sum(zi, oi, 2, wzi, wri, svi);
        Bc[0] += sum(zi, oh, 3, wzi, wrh, szh);
        Bc[1] += sum(zh, oi, 4, wzh, wri, svi);
        Bc[2] += sum(zh, oh, 5, wzh, wrh, svh);
      }
    } else {
      int ozi[3], ozh[3];
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        ozi[a] = wrap_pow2(cz + upz - 1 + a, n1);
        ozh[a] = wrap_pow2(cz - 1 + a, n1);
      }
#pragma unroll MU
      for (int m = 0; m < M; ++m) {
        // not all nodes' loads at once: they spilled with a general mode count, and cost FP64
        // pushes of one and two modes 2 to 4% (three and four gain 25% by them)
        constexpr bool FEW = MC == 0 || (sizeof(R) == 8 && MC < 3);
        if constexpr (MC == 0) {
          // keeps the nodes' addresses from being formed before the loop and spilled
#pragma unroll
          for (int a = 0; a < 3; ++a) asm volatile("" : "+v"(ozi[a]), "+v"(ozh[a]), "+v"(rri[a]), "+v"(rrh[a]));
        }
        if (m > 0) next_phase(ct, sn, Pr, Pi);
        const bool odd = m & 1;
        R vx[6], vy[6];
        const long long rs = n1;
        const gptr<const V2> Fm = F + 6 * m * plane;
        gather_q<R>(Fm, wzh, ozh, wri, rri, gi, odd, false, rs, vx[0], vy[0]);
        gather_q<R>(Fm + plane, wzi, ozi, wrh, rrh, gh, odd, true, rs, vx[1], vy[1]);
        if constexpr (FEW) asm volatile("" ::: "memory");
        gather_q<R>(Fm + 2 * plane, wzi, ozi, wri, rri, gi, odd, true, rs, vx[2], vy[2]);
        gather_q<R>(Fm + 3 * plane, wzi, ozi, wrh, rrh, gh, odd, false, rs, vx[3], vy[3]);
        if constexpr (FEW) asm volatile("" ::: "memory");
        gather_q<R>(Fm + 4 * plane, wzh, ozh, wri, rri, gi, odd, true, rs, vx[4], vy[4]);
        gather_q<R>(Fm + 5 * plane, wzh, ozh, wrh, rrh, gh, odd, true, rs, vx[5], vy[5]);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          Ec[c] += m > 0 ? fmaq(vx[c], Pr, vy[c] * Pi) : vx[c];
          Bc[c] += m > 0 ? fmaq(vx[c + 3], Pr, vy[c + 3] * Pi) : vx[c + 3];
        }
      }
    }
    const R E[3] = {Ec[0], crossq(Ec[1], ct, Ec[2], sn), fmaq(Ec[1], sn, Ec[2] * ct)};
    const R B[3] = {Bc[0], crossq(Bc[1], ct, Bc[2], sn), fmaq(Bc[1], sn, Bc[2] * ct)};
    borisq<R>(r.qmhdt, E, B, u);
    // moves in cells
    R mz, mx, my;
    {
#pragma clang fp contract(off)
      R s = R(1) + u[0] * u[0];
      s = s + u[1] * u[1];
      s = s + u[2] * u[2];
      const R ig = inv_gamma(s);
      mz = r.dtdz * (u[0] * ig);
      mx = r.dtdr * (u[1] * ig);
      my = r.dtdr * (u[2] * ig);
    }
    bool ok = true;
    if (!(isfinite(u[0]) && isfinite(u[1]) && isfinite(u[2]) && isfinite(mz) && isfinite(mx) &&
          isfinite(my))) {
      atomicOr(err, ERR_NUMERIC);
      ok = false;
    }
    R gz = fz, gx = fx, gy = fy;
    int dz = 0, dx = 0, dy = 0, mrb = mri;
    R drb = dri, ctb = ct, stb = sn;
    if (ok) {
      if (!(fabs(mz) < R(1)) || !(fabs(mx) < R(1)) || !(fabs(my) < R(1))) {
        atomicOr(err, ERR_RANGE);
        ok = false;
      } else {
        dz = advance<R>(fz, mz, gz);
        dx = advance<R>(fx, mx, gx);
        dy = advance<R>(fy, my, gy);
        radial<R>(ix + dx, gx, iy + dy, gy, mrb, drb, ctb, stb);
        // within the wall margin, and less than a cell in r (the deposit window
        // and the tile's box assume it)
        const R dmove = R(mrb - mri) + (drb - dri);
        if (!(R(mrb) + drb < r.rmax) || !(fabs(dmove) < R(1)) || abs(mrb - mri) > 1) {
          atomicOr(err, ERR_RANGE);
          ok = false;
        }
      }
    }
    const int nz = ok ? relz + dz : relz, nm = ok ? mrb : mri;
    blo = min(blo, nz);
    bhi = max(bhi, nz);
    rlo2 = min(rlo2, nm);
    rhi2 = max(rhi2, nm);
    if (ok) {
      // the new state first (fewer values live across the deposit)
      *elem(P.cell, p) = wrap_pow2(cz + dz, n1);
      *elem(P.fz, p) = gz;
      *elem(P.ix, p) = ix + dx;
      *elem(P.fx, p) = gx;
      *elem(P.iy, p) = iy + dy;
      *elem(P.fy, p) = gy;
      *elem(P.uz, p) = u[0];
      *elem(P.ux, p) = u[1];
      *elem(P.uy, p) = u[2];
    }
    // ---- deposit (FP64); a particle at rest adds nothing but exact zeros (512 x 128, three
    // modes, FP32, all at rest: 28 us, 40 with the zeros)
    if (ok && (mz != R(0) || mx != R(0) || my != R(0))) {
      using D = double;
      // azimuthal velocity at the mid point times dt: the move (mx, my) dr
      // projected on the azimuthal direction of the mid point
      const D xmid = D(ix) + (D)fx + 0.5 * (D)mx, ymid = D(iy) + (D)fy + 0.5 * (D)my;
      const D rmid = sqrt(fmaq(xmid, xmid, ymid * ymid));
      const D vthdt = rmid > 0.0 ? crossq(xmid, (D)my, ymid, (D)mx) / rmid * (D)r.dr : 0.0;
      const D g = (D)st.qw * (D)r.wscale;
      if (in) {
        deposit_move<MC>(MoveQ{cz, dz, mri, mrb, (D)fz, (D)gz, (D)dri, (D)drb, (D)ct, (D)sn, (D)ctb,
                               (D)stb, g, vthdt},
                         M, [&](int bz) {
                           return SinkLdsQ<A, MC, CW>{box + ((bz - cz + relz - zlo) - rlo * RS), M};
                         });
      } else {
        deposit_move_global<A>(r.J[parity], plane, n1, M, cz, (D)fz, dz, (D)gz, mri, (D)dri, mrb,
                               (D)drb, (D)ct, (D)sn, (D)ctb, (D)stb, g, vthdt);
      }
    }
  }
  blo = wmin(blo);
  bhi = wmax(bhi);
  rlo2 = wmin(rlo2);
  rhi2 = wmax(rhi2);
  if ((threadIdx.x & 63) == 0) {
    atomicMin((int *)nbox + 0, blo);
    atomicMax((int *)nbox + 1, bhi);
    atomicMin((int *)nbox + 2, rlo2);
    atomicMax((int *)nbox + 3, rhi2);
  }
  __syncthreads();
  // add the box to the global accumulators: half a wave per (row, slot)
  A *J = r.J[parity];
  const int cc = threadIdx.x & 31;
  if (cc < W) {
    const int col = wrap_pow2(z0 + zlo + cc, n1);
    for (int e = (int)threadIdx.x >> 5; e < H * NS; e += NT / 32) {
      const int j = e / NS, slot = e - j * NS;
      const A v = box[j * RS + slot * CW + cc];
      if (v == A(0)) continue;
      const int c = slot / per, s2 = slot - c * per;
      const int m = (s2 + 1) >> 1, part = s2 == 0 ? 0 : (s2 - 1) & 1;
      glob_add(G(J) + ((long long)(m * 3 + c) * plane + (long long)(rlo + j) * n1 + col) * 2 + part, v);
    }
  }
  // the box of the pushed particles; one that reaches past the frame's edge
  // wraps, so it becomes the whole frame
  if (threadIdx.x == 0) {
    int lo = nbox[0], hi = nbox[1];
    if (lo < -fo || hi >= n1 - fo) {
      lo = -fo;
      hi = n1 - fo - 1;
    }
    seg->zlo = lo;
    seg->zhi = hi;
    seg->rlo = nbox[2];
    seg->rhi = nbox[3];
  }
}
template <class R>
__device__ __noinline__ int4 q_window_call(const RunQ<R> *run, const QSeg *seg, int cols, int rows,
                                           lptr<unsigned char> smem) {
  return q_window<R>(*run, seg, cols, rows, smem);
}
// With the box laid around the particles' mean, as large as fits.  Out of line, so that it
// takes no registers from a segment that fits.  Up to three modes leave room for 32
// columns, up to two for the fields of the FP32 form; with more, the fields come through the
// cache.  (256 x 128, eight particles a cell, thermal spread 0.1, FP32, push: one mode 24 us,
// 37 with 24 columns; two 40 and 63; four 137, 213 with their fields in the LDS.)
template <class R, int MC, int CW>
__device__ __noinline__ void q_push_spread(const RunQ<R> *run, const QSeg *seg, int parity,
                                           lptr<unsigned char> smem, lptr<int> nbox, unsigned *err) {
  constexpr int CS = MC > 0 && MC < 4 && CW > 16 ? 32 : CW;
  constexpr bool STAGE = sizeof(R) == 4 && MC > 0 && MC < 3;
  const RunQ<R> &r = *run;
  const int first = G(seg)->start + (int)threadIdx.x;
  const int4 w = q_window<R>(r, seg, CS - 5, q_push_rows<R>(CS, MC > 0 ? MC : r.M, STAGE) - 4, smem);
  PStateQ<R> st{};
  if (first < G(seg)->end) st = load_q(r.pt, first);
  q_push<R, MC, CS, false, STAGE>(r, seg, parity, __builtin_amdgcn_readfirstlane(w.x),
                                  __builtin_amdgcn_readfirstlane(w.y), __builtin_amdgcn_readfirstlane(w.z),
                                  __builtin_amdgcn_readfirstlane(w.w), st, smem, nbox, err);
}

}  // namespace

// One workgroup per (run, segment of a tile).  A segment's box (from the previous push, or the
// whole tile right after a sort) bounds the cells of its particles: z columns
// relative to the tile and nearest integer-r nodes; a move is less than a cell,
// so the current box is columns lo - 2 .. hi + 3 and rows lo - 2 .. hi + 2 (ghost
// rows folded onto rows 0 and 1).  In the FP32 form the fields over columns
// lo - 1 .. hi + 2 and rows lo - 2 .. hi + 1 are staged next to it.  Every row of
// either box holds all components and modes, with CW columns each (CW - 2 of the
// fields), so that an address found for one row serves them all.  MC: the mode
// count when every run of the launch has it (the gather's mode loop is then
// unrolled and the deposit's has a constant trip count), or 0.
//
// What bounds it: the instructions and the LDS atomics of about 145 contributions
// a particle, with three modes.  On 2048 x 256 cells (8 particles each over 250
// rows, three modes, FP32) a push takes 385 us, 1098 with a box per wave of 64
// particles, which carried a halo of 8 x 8 nodes for 8 cells and tested every
// contribution; FP64 on 256 x 61 with two modes 36 us (28 in the 64 steps after a load,
// until the second sort), 56 before.  Of that:
// tiles in place of waves (a third of the nodes flushed and staged per particle)
// and contributions without tests, 744; particles in the order of their cells, so
// that the lanes of an atomic meet different nodes (LDS cycles 374 to 290 us) and
// 16 x 4 tiles, 672; workgroups of 256 threads, three per compute unit, 424; rows and
// order for the banks, 397; a path without global memory for the segments that fit,
// 385.  Warm columns, with a thermal spread of 0.1, sorted every 64 steps (512 x 160, eight a
// cell): 68 us with two modes, 588 with whole segments in global memory; with one mode 34
// and 212; FP64 form 110 and 681, 71 and 238.
template <class R, int MC, int CW, bool STAGE>
__global__ void __launch_bounds__(256, QPush<R>::WAVES_PER_SIMD)
    k_q_push_deposit(const RunQ<R> *__restrict__ runs, const Item *__restrict__ items, int parity,
                     unsigned *err) {
  __shared__ int nbox[4];
  const Item it = items[blockIdx.x];
  const RunQ<R> &r = runs[it.run];
  const gptr<const QSeg> seg = G((const QSeg *)r.seg) + it.a;
  const int start = seg->start, end = seg->end;
  if (start >= end) return;
  PStateQ<R> st{};
  if (start + (int)threadIdx.x < end) st = load_q(r.pt, start + (int)threadIdx.x);
  if (threadIdx.x == 0) {
    nbox[0] = nbox[2] = 1 << 30;
    nbox[1] = nbox[3] = -(1 << 30);
  }
  const int rows = q_push_rows<R>(CW, MC > 0 ? MC : r.M, STAGE);
  int clo = seg->zlo, chi = seg->zhi, mlo = seg->rlo, mhi = seg->rhi;
  const bool fits = chi - clo + 6 <= CW && min(mhi + 2, r.n2) - max(0, mlo - 2) < rows;
  const lptr<unsigned char> smem = (lptr<unsigned char>)smem_raw;
  // A path of its own for the segments that fit, with no global memory in it, is the faster
  // one in FP32 and with one or two modes (2048 x 256, three modes, FP32: 385 us, 411 in
  // one path; FP64 on 1024 x 160: 81 and 92 with one mode, 193 and 190 with three).
  if constexpr (sizeof(R) == 4 || MC == 1 || MC == 2) {
    if (fits)
      q_push<R, MC, CW, true, STAGE>(r, r.seg + it.a, parity, clo, chi, mlo, mhi, st, smem, (lptr<int>)nbox,
                                     err);
    else
      q_push_spread<R, MC, CW>(&r, r.seg + it.a, parity, smem, (lptr<int>)nbox, err);
  } else {
    if (!fits) {
      const int4 w = q_window_call<R>(&r, r.seg + it.a, CW - 5, rows - 4, smem);
      clo = __builtin_amdgcn_readfirstlane(w.x);
      chi = __builtin_amdgcn_readfirstlane(w.y);
      mlo = __builtin_amdgcn_readfirstlane(w.z);
      mhi = __builtin_amdgcn_readfirstlane(w.w);
    }
    q_push<R, MC, CW, false, false>(r, r.seg + it.a, parity, clo, chi, mlo, mhi, st, smem, (lptr<int>)nbox,
                                    err);
  }
}

// FP64 charge density of a run's particles (any form), added into rho.
template <class R>
__global__ void __launch_bounds__(256) k_q_rho(const RunQ<R> *__restrict__ run, int M,
                                               double2 *rho) {
  const RunQ<R> &r = *run;
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= r.np) return;
  const PartsQ<R> P = r.pt;
  const int n1 = r.n1;
  const double f = G(P.fz)[p], qw = G(P.qw)[p];
  const double x = (double)G(P.ix)[p] + (double)G(P.fx)[p];
  const double y = (double)G(P.iy)[p] + (double)G(P.fy)[p];
  const int cz = G(P.cell)[p];
  const double rr = sqrt(x * x + y * y);  // r / dr
  const double ct = rr > 0 ? x / rr : 1.0, st = rr > 0 ? y / rr : 0.0;
  double wz[3], wr[3];
  const int nz = zshape<double>(cz, f, wz);
  const int nr0 = rshape<double>(rr, wr);
  const double PI_ = 3.14159265358979323846;
  double Pr = 1, Pi = 0;
  for (int m = 0; m < M; ++m) {
    if (m > 0) {
      const double t = Pr * ct + Pi * st;
      Pi = Pi * ct - Pr * st;
      Pr = t;
    }
    const double cm = m == 0 ? 1.0 : 2.0;
    for (int b = 0; b < 3; ++b) {
      int row = nr0 - 1 + b;
      double s = cm * qw * wr[b];
      if (row < 0) {
        row = -row;
        if (m & 1) s = -s;
      }
      const double V = row == 0 ? 0.25 * PI_ * r.dr * r.dr * r.dz : 2.0 * PI_ * row * r.dr * r.dr * r.dz;
      for (int a = 0; a < 3; ++a) {
        double *o = (double *)(rho + (long long)m * r.plane + (long long)row * n1 +
                               wrap_pow2(nz - 1 + a, n1));
        const double w = s * wz[a] / V;
        atomicAdd(o, w * Pr);
        if (m > 0) atomicAdd(o + 1, w * Pi);
      }
    }
  }
}

// Co-drifting background current: jbg[j] -= q w v_z S_r / (n1 dz A_j).
template <class R>
__global__ void __launch_bounds__(256) k_q_jbg(const RunQ<R> *__restrict__ run, double *jbg) {
  const RunQ<R> &r = *run;
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= r.np) return;
  const PartsQ<R> P = r.pt;
  const double qw = G(P.qw)[p];
  const double x = (double)G(P.ix)[p] + (double)G(P.fx)[p];
  const double y = (double)G(P.iy)[p] + (double)G(P.fy)[p];
  const double uz = G(P.uz)[p], ux = G(P.ux)[p], uy = G(P.uy)[p];
  const double vz = uz / sqrt(1.0 + uz * uz + ux * ux + uy * uy);
  const double rr = sqrt(x * x + y * y);  // r / dr
  double wr[3];
  const int n0 = rshape<double>(rr, wr);
  const double PI_ = 3.14159265358979323846;
  for (int b = 0; b < 3; ++b) {
    int row = n0 - 1 + b;
    if (row < 0) row = -row;
    const double A = row == 0 ? 0.25 * PI_ * r.dr * r.dr : 2.0 * PI_ * row * r.dr * r.dr;
    atomicAdd(jbg + row, -qw * vz * wr[b] / ((double)r.n1 * r.dz * A));
  }
}

// ---------------------------------------------------------------- sort
// A periodic counting sort by the push's tiles, of sbz z columns x sbr radial
// rows, that also orders the particles within a tile: by their rank among the
// particles of their place, then by place, of which there is one per column and
// nearest row of nodes (the tile's last one together with its first).
// Consecutive particles, which the lanes of a wave take, then touch different
// accumulators: columns two apart, so that it does not matter where in its cell
// a particle is along z, and rows whose banks do not meet.  (By cell, with rows where
// the stride fell, half of the LDS cycles were conflicts: 2048 x 256, three modes,
// push 425 us, 397 now.)

// Even columns before odd, in each by row and column.
__device__ __forceinline__ int q_place_of(int z, int j, int tz, int tr) {
  const int even = (tz + 1) >> 1, odd = z & 1;
  return odd * even * tr + j * (odd ? tz - even : even) + (z >> 1);
}
// Tile and place of a particle.
template <class R>
__device__ __forceinline__ int q_sort_cell(const RunQ<R> &r, const PartsQ<R> &P, int p) {
  const float x = (float)*elem(P.ix, p) + (float)*elem(P.fx, p);
  const float y = (float)*elem(P.iy, p) + (float)*elem(P.fy, p);
  const float rr = sqrtf(x * x + y * y);
  const int j = min(max((int)rr, 0), r.n2 - 1), z = *elem(P.cell, p);
  const int tz = z / r.sbz, tr = j / r.sbr;
  const int near = min(max((int)(rr + 0.5f) - tr * r.sbr, 0), r.sbr);
  return (tz * r.nbr + tr) * (r.sbz * r.sbr) +
         q_place_of(z - tz * r.sbz, near == r.sbr ? 0 : near, r.sbz, r.sbr);
}

template <class R>
__global__ void k_q_sort_clear(const RunQ<R> *__restrict__ run) {
  const RunQ<R> &r = *run;
  const int n = r.nbins * r.sbz * r.sbr;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) r.ccnt[i] = 0;
}

template <class R>
__global__ void __launch_bounds__(256) k_q_sort_count(const RunQ<R> *__restrict__ run) {
  const RunQ<R> &r = *run;
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= r.np) return;
  const int c = q_sort_cell<R>(r, r.pt, p);
  r.skey[p] = c;
  // a wave within one cell (a dense beam) adds once
  const int c0 = __builtin_amdgcn_readfirstlane(c);
  const unsigned long long act = __ballot(1);
  int k;
  if (__ballot(c == c0) == act) {
    const int lane = threadIdx.x & 63, head = __builtin_ctzll(act);
    k = lane == head ? atomicAdd(r.ccnt + c, __popcll(act)) : 0;
    k = __builtin_amdgcn_readfirstlane(k) + __popcll(act & ((1ull << lane) - 1));
  } else {
    k = atomicAdd(r.ccnt + c, 1);
  }
  r.srank[p] = k;
}

// Particles per tile and the tile's levels, one wave a tile, a lane a cell.
template <class R>
__global__ void __launch_bounds__(256) k_q_sort_tiles(const RunQ<R> *__restrict__ run) {
  const RunQ<R> &r = *run;
  const int t = blockIdx.x * 4 + ((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (t >= r.nbins) return;
  const int area = r.sbz * r.sbr;
  const int cnt = lane < area ? G(r.ccnt)[t * area + lane] : 0;
  int base = 0;
  for (int k = 0; k < area; ++k) {
    const unsigned long long mask = __ballot(cnt > k);
    if (!mask) break;
    if (lane == 0) r.level[(long long)t * area + k] = QLevel{mask, base, 0};
    base += __popcll(mask);
  }
  int n = cnt;
  for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o);
  if (lane == 0) r.sbin[t] = n;
}

// Exclusive prefix sum of the bin counts in three launches: each block of
// 1024 threads scans its 1024 bins in LDS and records their sum; one block
// scans the block sums (a contiguous chunk per thread, then across threads);
// every block adds its offset.
__device__ __forceinline__ int block_scan_incl(int v, int *part) {
  const int t = threadIdx.x;
  part[t] = v;
  __syncthreads();
  for (int off = 1; off < 1024; off <<= 1) {
    const int w = t >= off ? part[t - off] : 0;
    __syncthreads();
    part[t] += w;
    __syncthreads();
  }
  return part[t];
}

template <class R>
__global__ void __launch_bounds__(1024) k_q_scan_local(const RunQ<R> *__restrict__ run) {
  __shared__ int part[1024];
  const RunQ<R> &r = *run;
  const int i = blockIdx.x * 1024 + threadIdx.x;
  const int v = i < r.nbins ? r.sbin[i] : 0;
  const int inc = block_scan_incl(v, part);
  if (i < r.nbins) r.sbin[i] = inc - v;
  if (threadIdx.x == 1023) r.ssum[blockIdx.x] = inc;
}

template <class R>
__global__ void __launch_bounds__(1024) k_q_scan_sums(const RunQ<R> *__restrict__ run) {
  __shared__ int part[1024];
  const RunQ<R> &r = *run;
  const int n = (r.nbins + 1023) / 1024, t = threadIdx.x;
  const int chunk = (n + 1023) / 1024, lo = min(n, t * chunk), hi = min(n, lo + chunk);
  int sum = 0;
  for (int i = lo; i < hi; ++i) sum += r.ssum[i];
  int run_sum = block_scan_incl(sum, part) - sum;  // exclusive prefix of this chunk
  for (int i = lo; i < hi; ++i) {
    const int c = r.ssum[i];
    r.ssum[i] = run_sum;
    run_sum += c;
  }
  if (t == 1023) r.sbin[r.nbins] = part[1023];
}

template <class R>
__global__ void __launch_bounds__(1024) k_q_scan_add(const RunQ<R> *__restrict__ run) {
  const RunQ<R> &r = *run;
  const int i = blockIdx.x * 1024 + threadIdx.x;
  if (i >= r.nbins) return;
  r.sbin[i] += r.ssum[blockIdx.x];
}

// The push's segments, one thread a tile; right after the sort a tile's particles
// lie in it.
template <class R>
__global__ void __launch_bounds__(256) k_q_sort_segments(const RunQ<R> *__restrict__ run) {
  const RunQ<R> &r = *run;
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t >= r.nbins) return;
  const int s0 = r.sbin[t], s1 = r.sbin[t + 1];
  const int tz = t / r.nbr, r0 = (t - tz * r.nbr) * r.sbr;
  QSeg g;
  g.tile = t;
  g.pad = 0;
  g.zlo = 0;
  g.zhi = min(r.sbz, r.n1 - tz * r.sbz) - 1;
  g.rlo = r0;
  g.rhi = max(r0, min(r0 + r.sbr, r.n2 - 3));  // no particle reaches r = n2 - 3
  const int parts = max(1, (s1 - s0 + Q_SEG - 1) / Q_SEG), len = (s1 - s0 + parts - 1) / parts;
  const int m0 = q_seg_more(s0), m1 = q_seg_more(s1);
  for (int k = 0; k <= m1 - m0; ++k) {
    g.start = min(s0 + k * len, s1);
    g.end = min(g.start + len, s1);
    r.seg[k == 0 ? t : r.nbins + m0 + k - 1] = g;
  }
}

// Scatter.  A particle of rank k in its cell comes after those of lower rank in
// any of the tile's cells and those of rank k in the cells before its own.
template <class R>
__global__ void __launch_bounds__(256) k_q_sort_scatter(const RunQ<R> *__restrict__ run) {
  const RunQ<R> &r = *run;
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= r.np) return;
  const int area = r.sbz * r.sbr, c = r.skey[p], t = c / area, place = c - t * area, k = r.srank[p];
  int d = r.sbin[t];
  if (k < area) {
    const QLevel l = r.level[(long long)t * area + k];
    d += l.base + __popcll(l.mask & ((1ull << place) - 1));
  } else {
    for (int i = 0; i < area; ++i) d += min(r.ccnt[t * area + i], i < place ? k + 1 : k);
  }
  const PartsQ<R> &A = r.pt, &B = r.pt2;
  G(B.cell)[d] = G(A.cell)[p];
  G(B.ix)[d] = G(A.ix)[p];
  G(B.iy)[d] = G(A.iy)[p];
  G(B.id)[d] = G(A.id)[p];
  G(B.fz)[d] = G(A.fz)[p];
  G(B.fx)[d] = G(A.fx)[p];
  G(B.fy)[d] = G(A.fy)[p];
  G(B.uz)[d] = G(A.uz)[p];
  G(B.ux)[d] = G(A.ux)[p];
  G(B.uy)[d] = G(A.uy)[p];
  G(B.qw)[d] = G(A.qw)[p];
}

template <class R>
__global__ void k_q_sort_swap(RunQ<R> *run) {
  const PartsQ<R> t = run->pt;
  run->pt = run->pt2;
  run->pt2 = t;
}

template <class R>
void LaunchQ<R>::sort(RunQ<R> *run_dev, int np, int nbins, hipStream_t s) {
  if (np <= 0 || nbins <= 0) return;
  const int pb = (np + 255) / 256;
  hipLaunchKernelGGL(k_q_sort_clear<R>, dim3(std::min(nbins, 1024)), dim3(256), 0, s, run_dev);
  hipLaunchKernelGGL(k_q_sort_count<R>, dim3(pb), dim3(256), 0, s, run_dev);
  hipLaunchKernelGGL(k_q_sort_tiles<R>, dim3((nbins + 3) / 4), dim3(256), 0, s, run_dev);
  const int sb = (nbins + 1023) / 1024;
  hipLaunchKernelGGL(k_q_scan_local<R>, dim3(sb), dim3(1024), 0, s, run_dev);
  hipLaunchKernelGGL(k_q_scan_sums<R>, dim3(1), dim3(1024), 0, s, run_dev);
  hipLaunchKernelGGL(k_q_scan_add<R>, dim3(sb), dim3(1024), 0, s, run_dev);
  hipLaunchKernelGGL(k_q_sort_segments<R>, dim3((nbins + 255) / 256), dim3(256), 0, s, run_dev);
  hipLaunchKernelGGL(k_q_sort_scatter<R>, dim3(pb), dim3(256), 0, s, run_dev);
  hipLaunchKernelGGL(k_q_sort_swap<R>, dim3(1), dim3(1), 0, s, run_dev);
}

template <class R>
void LaunchQ<R>::push_deposit(const RunQ<R> *runs, const Item *items, int nitems, int parity,
                              int modes, int tz, bool staged, unsigned *err, hipStream_t s) {
  if (nitems <= 0) return;
  // kernels with the mode loops unrolled for the common mode counts, and literal
  // column strides for the tile widths the runtime uses
  constexpr int C16 = q_push_cols(16), C8 = q_push_cols(8);
  constexpr bool S = sizeof(R) == 4;
  auto k = k_q_push_deposit<R, 0, C8, false>;
  if (S && !staged)
    ;  // (tiles of up to 8 columns)
  else if (tz > 8)
    k = modes == 1   ? k_q_push_deposit<R, 1, C16, S>
        : modes == 2 ? k_q_push_deposit<R, 2, C16, S>
        : modes == 3 ? k_q_push_deposit<R, 3, C16, S>
        : modes == 4 ? k_q_push_deposit<R, 4, C16, S>
                     : k_q_push_deposit<R, 0, C16, S>;
  else
    k = modes == 2   ? k_q_push_deposit<R, 2, C8, S>
        : modes == 3 ? k_q_push_deposit<R, 3, C8, S>
        : modes == 4 ? k_q_push_deposit<R, 4, C8, S>
                     : k_q_push_deposit<R, 0, C8, S>;
  hipLaunchKernelGGL(k, dim3(nitems), dim3(256), (size_t)QPush<R>::LDS, s, runs, items, parity, err);
}
template <class R>
void LaunchQ<R>::rho(const RunQ<R> *run_dev, int np, int M, double2 *rho, hipStream_t s) {
  if (np <= 0) return;
  hipLaunchKernelGGL(k_q_rho<R>, dim3((np + 255) / 256), dim3(256), 0, s, run_dev, M, rho);
}
template <class R>
void LaunchQ<R>::jbg(const RunQ<R> *run_dev, int np, double *jbg, hipStream_t s) {
  if (np <= 0) return;
  hipLaunchKernelGGL(k_q_jbg<R>, dim3((np + 255) / 256), dim3(256), 0, s, run_dev, jbg);
}

template void LaunchQ<float>::push_deposit(const RunQ<float> *, const Item *, int, int, int, int,
                                           bool, unsigned *, hipStream_t);
template void LaunchQ<double>::push_deposit(const RunQ<double> *, const Item *, int, int, int, int,
                                            bool, unsigned *, hipStream_t);
template void LaunchQ<float>::sort(RunQ<float> *, int, int, hipStream_t);
template void LaunchQ<double>::sort(RunQ<double> *, int, int, hipStream_t);
template void LaunchQ<float>::rho(const RunQ<float> *, int, int, double2 *, hipStream_t);
template void LaunchQ<double>::rho(const RunQ<double> *, int, int, double2 *, hipStream_t);
template void LaunchQ<float>::jbg(const RunQ<float> *, int, double *, hipStream_t);
template void LaunchQ<double>::jbg(const RunQ<double> *, int, double *, hipStream_t);

}  // namespace hp
