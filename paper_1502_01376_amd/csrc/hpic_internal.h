// hpic_internal.h -- device-side data layout and helpers of the MI355X hybrid
// Yee-FFT PIC library.  Shared by the kernels (kernels.hip) and the host
// runtime (runtime.cpp); not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hp {

// The dynamic LDS of every kernel.  It follows a kernel's static LDS, so without an
// alignment of its own it may start at any byte: behind the six ints of the 3D
// push's box the 16-byte stores that clear it lay 8 bytes off.
extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];

// ---------------------------------------------------------------- types
template <class R> struct Cplx;
template <> struct Cplx<float> { using T = float2; };
template <> struct Cplx<double> { using T = double2; };

// Deposit accumulator: 64-bit fixed point for the FP32 form, FP64 otherwise.
template <class R> struct AccOf;
template <> struct AccOf<float> { using T = long long; };
template <> struct AccOf<double> { using T = double; };

// One work item of a batched launch: run index and two item-specific ints.
struct Item {
  int run;
  int a;
  int b;
};

// Particle state (structure of arrays): cell[np] packed cell index
// i1 | i2 << log2n1 | i3 << sh3 (2D: i3 = 0, so the packed index is the
// linear one), f1/f2/f3[np] offsets in [0,1) (f3 only in 3D), u1..u3[np]
// momenta u = gamma v, qw[np] charge times weight, id[np] load index.
constexpr int SORT_BLOCK = 2048;

template <class R>
struct Parts {
  int *cell, *id;
  R *f1, *f2, *f3, *u1, *u2, *u3, *qw;
};

// Device-side description of one 2D run.  Arrays are owned by the host runtime.
//   pt:  particle buffers, ping-pong for the tile sort (index = particle parity)
//   tiles: T1 x T2 cells each, nt1 x nt2 of them; tile_start[ntiles + 1] is the
//        first particle of each tile after the last sort, cell_cnt[ntiles][area]
//        the histogram / scatter cursor of the sort (one key per cell of a tile,
//        or per tile), in blocks of SORT_BLOCK with their sums and first
//        particles blk_sum, blk_base; tile_box the bounding box of
//        the cells of each tile's particles (they drift out of the tile
//        between sorts)
//   F:   real-space fields [6][n2][n1] (E1 E2 E3 B1 B2 B3) for the gather
//   Fk:  k-space master copy [6][n2][nk] in FP64 for both forms (ping-pong,
//        index = step parity): the state that carries the field from step to
//        step, so its rounding does not accumulate into a phase drift
//        (FP32 storage of a mode rotated 1000 times drifts by ~1e-5)
//   J:   deposit accumulators [3][n2][n1] (ping-pong, index = step parity)
//   Jk:  corrected, filtered current [3][n2][nk]
template <class R>
struct Run {
  using C = typename Cplx<R>::T;
  using Acc = typename AccOf<R>::T;
  int dim;           // 2 or 3
  int interp;        // 0 momentum-conserving gather, 1 energy-conserving (3D
                     // kernel; the 2D kernel takes it as a template argument)
  int shape;         // particle shape order: 2 quadratic, 3 cubic (2D only)
  int n1, n2, n3, log2n1, nk;
  int sh3;           // 3D: shift of i3 in the packed cell index
  int rows;          // n2 * n3: rows of the x1 transforms
  int cells;         // n1 * rows
  int np;
  int P;             // fixed point: shape factors in units of 2^-P
  float inv_wunit;   // fixed point: integer charge = rint(qw * inv_wunit)
  float c3;          // fixed point: scale of the out-of-plane current
  int unit_charge;   // fixed point: |charge| * 2^P < 2^31, so Q*C products fit 32 bits
  R dt, hdt, idx2;   // dt, dt/2, 1/dx2
  R dtdx1, dtdx2;    // dt/dx1, dt/dx2 (position advance in cells per unit velocity)
  R qmhdt;           // (q/m) dt/2
  R jfx1, jfx2;      // FP64 form: -dx1/dt, -dx2/dt (current of a unit-charge move)
  R idx3, dtdx3, jfx3;  // 3D: 1/dx3, dt/dx3, -dx3/dt
  float cj;          // 3D FP32 form: integer scale of the per-node contributions
  R inv_m;           // 1/M, M = n1/2 (inverse real FFT normalisation)
  double jbgu[3];    // j_bg in accumulator units, added to every node before the
                     // row transform (so the transform sees the drift-free current)
  Parts<R> pt[2];
  int T1, T2, T3, nt1, nt2, nt3, ntiles;
  int area;          // sort keys per tile
  int *tile_start, *cell_cnt, *blk_sum, *blk_base;
  int *tile_box;     // [ntiles][6]: lo1, hi1, lo2, hi2, lo3, hi3 of the tile's particle cells
                     // relative to the tile origin (updated by every push)
  R *F;
  double2 *Fk[2];
  Acc *J[2];
  C *Jk;
  const C *tw;       // [n1]: exp(-2 pi i m / n1)
  const double *sym; // [nk][4]: i k1 xi+ (re, im), i k1 xi- (re, im)
  double mdt, mhdt, midx2, midx3;  // dt, dt/2, 1/dx2, 1/dx3 of the FP64 field update
  const R *jfac;     // [nk][3]: factor on the transformed accumulator per component
};

// Global-memory view of a pointer held in a descriptor: lets the compiler use
// global (not flat) loads, stores and atomics.
template <class T> using gptr = T __attribute__((address_space(1))) *;
template <class T> __device__ __forceinline__ gptr<T> G(T *p) { return (gptr<T>)p; }

// ---------------------------------------------------------------- complex
__device__ __forceinline__ float2 cmk(float x, float y) { return make_float2(x, y); }
__device__ __forceinline__ double2 cmk(double x, double y) { return make_double2(x, y); }
template <class C> __device__ __forceinline__ C cadd(C a, C b) { return cmk(a.x + b.x, a.y + b.y); }
template <class C> __device__ __forceinline__ C csub(C a, C b) { return cmk(a.x - b.x, a.y - b.y); }
template <class C> __device__ __forceinline__ C cmul(C a, C b) {
  return cmk(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
template <class C> __device__ __forceinline__ C cconj(C a) { return cmk(a.x, -a.y); }
template <class C, class R> __device__ __forceinline__ C cscale(C a, R s) { return cmk(a.x * s, a.y * s); }
__device__ __forceinline__ double2 to_d2(float2 a) { return make_double2(a.x, a.y); }
__device__ __forceinline__ double2 to_d2(double2 a) { return a; }
template <class C> __device__ __forceinline__ C from_d2(double2 a);
template <> __device__ __forceinline__ float2 from_d2<float2>(double2 a) {
  return make_float2((float)a.x, (float)a.y);
}
template <> __device__ __forceinline__ double2 from_d2<double2>(double2 a) { return a; }
// multiply by +i (inv = true) or -i
template <class C> __device__ __forceinline__ C cmuli(C a, bool plus) {
  return plus ? cmk(-a.y, a.x) : cmk(a.y, -a.x);
}

// Global loads and stores of pairs: element i of an array of complex values, and
// elements i, i + 1 (i even) of one of accumulators or reals.  (Through a generic
// pointer they would be flat accesses, which may alias the LDS and so cannot be
// moved across its stores: every load of a row transform waited alone.)
typedef float float2v __attribute__((ext_vector_type(2)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef double double2v __attribute__((ext_vector_type(2)));
typedef double double4v __attribute__((ext_vector_type(4)));
typedef long long long2v __attribute__((ext_vector_type(2)));
template <class T> struct Pair;
template <> struct Pair<float2> { using V = float2v; };
template <> struct Pair<double2> { using V = double2v; };
template <> struct Pair<double> { using V = double2v; };
template <> struct Pair<long long> { using V = long2v; };
template <class R> struct Quad;
template <> struct Quad<float> { using V = float4v; };
template <> struct Quad<double> { using V = double4v; };
template <class C> __device__ __forceinline__ C ldc(const C *p, long long i) {
  const auto v = ((gptr<const typename Pair<C>::V>)G(p))[i];
  return cmk(v.x, v.y);
}
template <class C> __device__ __forceinline__ void stc(C *p, long long i, C c) {
  typename Pair<C>::V v;
  v.x = c.x;
  v.y = c.y;
  ((gptr<typename Pair<C>::V>)G(p))[i] = v;
}
template <class A> __device__ __forceinline__ typename Pair<A>::V ldpair(const A *p, long long i) {
  return *(gptr<const typename Pair<A>::V>)(G(p) + i);
}
template <class A> __device__ __forceinline__ void zeropair(A *p, long long i) {
  *(gptr<typename Pair<A>::V>)(G(p) + i) = typename Pair<A>::V{0, 0};
}

// ---------------------------------------------------------------- LDS FFT
// NF independent complex transforms of length M = 2^log2M stored back to back
// in LDS (buf[f*M + j]), computed by the whole workgroup with Stockham
// auto-sort radix-4 passes and, for odd log2M, a final radix-2 pass.
// tw[m * tws] = exp(-2 pi i m / M); inverse = true uses the conjugate twiddles
// (no 1/M).  MAXB bounds the radix-4 butterflies per thread per pass.
template <class C, int MAXB>
__device__ __forceinline__ void lds_fft(C *buf, int M, int log2M, int NF, const C *__restrict__ tw, int tws,
                        bool inverse, int s0 = 0) {
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int Q = M >> 2;
  const int log2Q = log2M - 2;
  int s = s0;  // log2 of the span Ns already transformed
  for (; s + 2 <= log2M; s += 2) {
    const int Ns = 1 << s;
    C v[MAXB][4];
    int ob[MAXB];
    int cnt = 0;
    const int total = NF * Q;
#pragma unroll
    for (int it = 0; it < MAXB; ++it) {
      const int g = tid + it * nthr;
      if (g < total) {
        const int f = g >> log2Q;
        const int j = g & (Q - 1);
        C *x = buf + f * M;
        const int k = j & (Ns - 1);
        C a0 = x[j], a1 = x[j + Q], a2 = x[j + 2 * Q], a3 = x[j + 3 * Q];
        if (s > 0) {
          // twiddle w^(r k), w = exp(-+2 pi i / (4 Ns)) -> table index r k M / (4 Ns)
          const int e = k << (log2Q - s);
          C t1 = ldc(tw, e * tws), t2 = ldc(tw, 2 * e * tws), t3 = ldc(tw, 3 * e * tws);
          if (inverse) { t1 = cconj(t1); t2 = cconj(t2); t3 = cconj(t3); }
          a1 = cmul(a1, t1);
          a2 = cmul(a2, t2);
          a3 = cmul(a3, t3);
        }
        const C b0 = cadd(a0, a2), b1 = csub(a0, a2), b2 = cadd(a1, a3);
        const C b3 = cmuli(csub(a1, a3), inverse);
        v[it][0] = cadd(b0, b2);
        v[it][1] = cadd(b1, b3);
        v[it][2] = csub(b0, b2);
        v[it][3] = csub(b1, b3);
        ob[it] = f * M + ((j >> s) << (s + 2)) + k;
        cnt = it + 1;
      }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < MAXB; ++it) {
      if (it < cnt) {
#pragma unroll
        for (int q = 0; q < 4; ++q) buf[ob[it] + q * Ns] = v[it][q];
      }
    }
    __syncthreads();
  }
  if (s < log2M) {
    // final radix-2 pass: Ns = M/2, in place (each thread owns its pair)
    const int H = M >> 1;
    const int total = NF * H;
    for (int g = tid; g < total; g += nthr) {
      const int f = g >> (log2M - 1);
      const int j = g & (H - 1);
      C *x = buf + f * M;
      C t = ldc(tw, j * tws);
      if (inverse) t = cconj(t);
      const C a0 = x[j], a1 = cmul(x[j + H], t);
      x[j] = cadd(a0, a1);
      x[j + H] = csub(a0, a1);
    }
    __syncthreads();
  }
}

// 4-point DFT in place (forward: X_q = sum_r a_r exp(-2 pi i r q / 4)).
template <class C>
__device__ __forceinline__ void dft4(C &a0, C &a1, C &a2, C &a3, bool inverse) {
  const C b0 = cadd(a0, a2), b1 = csub(a0, a2), b2 = cadd(a1, a3);
  const C b3 = cmuli(csub(a1, a3), inverse);
  a0 = cadd(b0, b2);
  a1 = cadd(b1, b3);
  a2 = csub(b0, b2);
  a3 = csub(b1, b3);
}
// exp(-2 pi i m / 16) (conjugate for the inverse) of the 16-point DFT's
// inner twiddles, m = r2 q1 in {1, 2, 3, 4, 6, 9}
template <class C>
__device__ __forceinline__ C w16(int m, bool inverse) {
  using R = decltype(C().x);
  const R c1 = R(0.92387953251128675613), s1 = R(0.38268343236508977173);
  const R h = R(0.70710678118654752440);
  R x, y;
  switch (m) {
    case 1: x = c1; y = -s1; break;
    case 2: x = h; y = -h; break;
    case 3: x = s1; y = -c1; break;
    case 4: x = 0; y = -1; break;
    case 6: x = -h; y = -h; break;
    default: x = -c1; y = s1; break;  // 9
  }
  return cmk(x, inverse ? -y : y);
}
// 16-point DFT in registers as 4 x 4: a[r] -> y_q with q = q1 + 4 q2 stored
// at a[4 q1 + q2].
template <class C>
__device__ __forceinline__ void dft16(C a[16], bool inverse) {
#pragma unroll
  for (int r2 = 0; r2 < 4; ++r2) dft4(a[r2], a[4 + r2], a[8 + r2], a[12 + r2], inverse);
#pragma unroll
  for (int q1 = 1; q1 < 4; ++q1)
#pragma unroll
    for (int r2 = 1; r2 < 4; ++r2) a[4 * q1 + r2] = cmul(a[4 * q1 + r2], w16<C>(r2 * q1, inverse));
#pragma unroll
  for (int q1 = 0; q1 < 4; ++q1) dft4(a[4 * q1], a[4 * q1 + 1], a[4 * q1 + 2], a[4 * q1 + 3], inverse);
}
// NF transforms of length M in LDS, radix-16 Stockham passes (one 16-point
// butterfly per thread, all of them held in registers across the barrier)
// while they fit the block, then the radix-4/2 passes of lds_fft.  Same
// result as lds_fft.
template <class C, int MAXB>
__device__ __forceinline__ void lds_fft16(C *buf, int M, int log2M, int NF, const C *__restrict__ tw, int tws,
                          bool inverse) {
  int s = 0;
  if (NF * (M >> 4) <= (int)blockDim.x) {
    const int Q = M >> 4, log2Q = log2M - 4, g = threadIdx.x;
    for (; s + 4 <= log2M; s += 4) {
      const int Ns = 1 << s;
      C v[16];
      int ob = 0;
      const bool act = g < NF * Q;
      if (act) {
        const int f = g >> log2Q, j = g & (Q - 1), k = j & (Ns - 1);
        const C *x = buf + f * M;
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = x[j + r * Q];
        if (s > 0) {
          // twiddle w^(r k), w = exp(-+2 pi i / (16 Ns)): table index r k M / (16 Ns)
          const int e = k << (log2Q - s);
#pragma unroll
          for (int r = 1; r < 16; ++r) {
            C t = ldc(tw, r * e * tws);
            if (inverse) t = cconj(t);
            v[r] = cmul(v[r], t);
          }
        }
        dft16(v, inverse);
        ob = f * M + ((j >> s) << (s + 4)) + k;
      }
      __syncthreads();
      if (act) {
#pragma unroll
        for (int q1 = 0; q1 < 4; ++q1)
#pragma unroll
          for (int q2 = 0; q2 < 4; ++q2) buf[ob + (q1 + 4 * q2) * Ns] = v[4 * q1 + q2];
      }
      __syncthreads();
    }
  }
  lds_fft<C, MAXB>(buf, M, log2M, NF, tw, tws, inverse, s);
}

// NF transforms of length M in LDS (as lds_fft), one transform at a time when
// the radix-4 passes of all NF at once would need more than MAXB butterflies
// per thread (n1 = 8192 rows: three components of M = 4096).  The choice is
// uniform over the block, so the barriers inside stay uniform.
template <class C, int MAXB>
__device__ __forceinline__ void lds_fft_rows(C *buf, int M, int log2M, int NF, const C *__restrict__ tw, int tws,
                             bool inverse) {
  if (NF * (M >> 2) <= MAXB * (int)blockDim.x) {
    lds_fft16<C, MAXB>(buf, M, log2M, NF, tw, tws, inverse);
    return;
  }
  for (int f = 0; f < NF; ++f) lds_fft16<C, MAXB>(buf + f * M, M, log2M, 1, tw, tws, inverse);
}

// ---------------------------------------------------------------- shapes
// Quadratic B-spline weights of the nodes m-1, m, m+1 for a particle at signed
// distance d in [-1/2, 1/2) from its nearest node m.
template <class R> __device__ __forceinline__ void spline3(R d, R w[3]) {
  const R a = R(0.5) - d, b = R(0.5) + d;
  w[0] = R(0.5) * a * a;
  w[1] = R(0.75) - d * d;
  w[2] = R(0.5) * b * b;
}
// Linear B-spline on the same three nodes (energy-conserving gather along a
// staggered direction): for d in [-1/2, 1/2) the weights of m-1, m, m+1.
template <class R> __device__ __forceinline__ void line3(R d, R w[3]) {
  w[0] = d < R(0) ? -d : R(0);
  w[1] = R(1) - (d < R(0) ? -d : d);
  w[2] = d > R(0) ? d : R(0);
}
// Contractions spelled out: a tile whose box leaves the LDS takes another path through
// the code, and gives the same bits.
__device__ __forceinline__ float fmaq(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fmaq(double a, double b, double c) { return __builtin_fma(a, b, c); }
// Twice the quadratic weights (the gather scales its sums by 1/2 per
// axis), or twice the energy-conserving gather's along a staggered direction.
template <class R> __device__ __forceinline__ void spline3x2(R d, R w[3]) {
  const R a = R(0.5) - d, b = R(0.5) + d;
  w[0] = a * a;
  w[1] = fmaq(R(-2) * d, d, R(1.5));
  w[2] = b * b;
}
template <class R> __device__ __forceinline__ void half3x2(R d, R w[3], bool ec) {
  if (ec) {
    line3<R>(d, w);
#pragma unroll
    for (int k = 0; k < 3; ++k) w[k] = R(2) * w[k];
  } else {
    spline3x2<R>(d, w);
  }
}

// Half the quadratic weights, or the energy-conserving gather's: the other axis's doubled
// ones then need no factor, and no partial sum exceeds the largest field.
template <class R> __device__ __forceinline__ void spline3h(R d, R w[3]) {
  const R h = R(0.5) * d, a = R(0.25) - h, b = R(0.25) + h;
  w[0] = a * a;
  w[1] = fmaq(-h, d, R(0.375));
  w[2] = b * b;
}
template <class R> __device__ __forceinline__ void half3h(R d, R w[3], bool ec) {
  if (ec) {
    line3<R>(d, w);
#pragma unroll
    for (int k = 0; k < 3; ++k) w[k] = R(0.5) * w[k];
  } else {
    spline3h<R>(d, w);
  }
}

template <class R> __device__ __forceinline__ R dot3q(const R w[3], R a, R b, R c) {
  return fmaq(w[2], c, fmaq(w[1], b, w[0] * a));
}
// New offset in [0,1) and cell shift in {-1, 0, 1} after a move d (|d| < 1).
// The subtraction is exact above 1; below 0 it may round up to 1, and the
// position is then the next cell edge.
template <class R>
__device__ __forceinline__ int advance(R f, R d, R &g) {
  const R t = f + d, c = floor(t);
  g = t - c;
  const bool edge = g >= R(1);
  g = edge ? R(0) : g;
  return (int)c + (edge ? 1 : 0);
}

// Quantised quadratic shape of one coordinate (cell + FP32 offset): integers
// s[0..2] of the nodes m-1, m, m+1 with exact sum 2^P; returns m.  The same
// definition as the FP32-precision reference deposit:
//   s[0] = floor(((2^(P-1) - D)^2 + 2^P) / 2^(P+1)), s[2] likewise with +D,
// D = rint(d 2^P).  The squares differ by 4 2^(P-1) D = 2^(P+1) D, so
// s[2] = s[0] + D and s[1] = 2^P - 2 s[0] - D: one square per coordinate.
// SMALL (P <= 22): the square is a full-rate 24-bit multiply pair and
// floor((x^2 + 2^P) / 2^(P+1)) is evaluated as (floor(x^2 / 2^P) + 1) >> 1,
// which is the same integer.
template <bool SMALL>
__device__ __forceinline__ int fixed_shape(int cell, float f, int P, int s[3]) {
  const int up = (f >= 0.5f) ? 1 : 0;
  const float d = f - (float)up;                    // exact
  int D;                                            // |D| <= 2^(P-1)
  if (SMALL)  // |d 2^P| <= 2^21: 1.5 2^23 rounds it to an integer in the low bits
    D = __float_as_int(__builtin_fmaf(d, (float)(1 << P), 12582912.0f)) - 0x4b400000;
  else
    D = (int)rintf(d * (float)(1 << P));            // exact product
  const int lo = (1 << (P - 1)) - D;                // in [0, 2^P]
  if (SMALL) {
    const unsigned long long l2 = (unsigned long long)(unsigned)(lo & 0xffffff) * (unsigned)(lo & 0xffffff);
    const unsigned ql = __builtin_amdgcn_alignbit((unsigned)(l2 >> 32), (unsigned)l2, (unsigned)P);
    s[0] = (int)((ql + 1u) >> 1);
  } else {
    s[0] = (int)(((long long)lo * lo + (1ll << P)) >> (P + 1));
  }
  s[2] = s[0] + D;
  s[1] = (1 << P) - s[0] - s[2];
  return cell + up;
}

// Products of two integers in [-2^23, 2^23): the low half (the whole product
// where it fits 32 bits) and the 64-bit value.  The full-rate 24-bit multiplies
// are written out: from the C expression the compiler takes a quarter-rate
// 32-bit multiply, or adds sign extensions that these operands do not need.
__device__ __forceinline__ int mul24_lo(int a, int b) {
  int r;
  asm("v_mul_i32_i24 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ long long mul24_wide(int a, int b) {
  int lo, hi;
  asm("v_mul_i32_i24 %0, %1, %2" : "=v"(lo) : "v"(a), "v"(b));
  asm("v_mul_hi_i32_i24 %0, %1, %2" : "=v"(hi) : "v"(a), "v"(b));
  return ((long long)hi << 32) | (unsigned)lo;
}

// Nearest integer (ties to even) of |v| < 2^51 as a 64-bit integer: adding
// 1.5 2^52 rounds v to an integer held in the low mantissa bits (one FP64 add
// and one 64-bit subtract instead of the multi-instruction FP64 -> int64
// conversion).
__device__ __forceinline__ long long rint_i64(double v) {
#pragma clang fp contract(off)
  const double t = v + 6755399441055744.0;
  return __double_as_longlong(t) - 0x4338000000000000LL;
}

__device__ __forceinline__ double inv_gamma(double s) {
  const double g = sqrt(s);
  return 1.0 / g;
}
// 1/g with g = sqrt(s), both correctly rounded, for s >= 1: no scaling against
// underflow is needed there, which leaves half the instructions of the general
// square root and division.  The method is the usual one with a fused multiply-add
// (P. Markstein, Computation of elementary functions on the IBM RISC System/6000
// processor, IBM J. Res. Dev. 34, 1990): g, the hardware root is within one unit and
// the exact residuals of its neighbours decide; 1/g, two residual corrections of the
// hardware reciprocal.  (A test compares every significand with either parity of the
// exponent, beyond which both only scale; infinity gives 0.)
__device__ __forceinline__ float inv_gamma(float s) {
#pragma clang fp contract(off)
  float g = __builtin_amdgcn_sqrtf(s);
  const float gm = __int_as_float(__float_as_int(g) - 1), gp = __int_as_float(__float_as_int(g) + 1);
  const float rm = __builtin_fmaf(-gm, g, s), rp = __builtin_fmaf(-gp, g, s);
  g = rm <= 0.0f ? gm : g;
  g = rp > 0.0f ? gp : g;
  float q = __builtin_amdgcn_rcpf(g);
  q = __builtin_fmaf(__builtin_fmaf(-g, q, 1.0f), q, q);
  q = __builtin_fmaf(__builtin_fmaf(-g, q, 1.0f), q, q);
  return s <= 3.402823466e38f ? q : (s > 0.0f ? 0.0f : s);
}

// Element p of an array whose base is uniform: a 32-bit byte offset from a
// scalar base where every offset fits (at most 10^9 particles: 4-byte
// elements), which saves the 64-bit address of each access.
template <class T>
__device__ __forceinline__ gptr<T> elem(T *a, int p) {
  if constexpr (sizeof(T) == 4)
    return (gptr<T>)((gptr<char>)G((char *)a) + (unsigned)p * 4u);
  else
    return G(a) + p;
}

__device__ __forceinline__ int wrap_pow2(int i, int n) { return i & (n - 1); }
__device__ __forceinline__ int wrap_small(int i, int n) {
  i += (i < 0) ? n : 0;
  i -= (i >= n) ? n : 0;
  return i;
}

// Adds 1 per lane to cnt[key] and returns the lane's place in it; the active lanes
// are the wave's first ones.  Neighbouring lanes with equal keys (particles as loaded
// come cell by cell) share one atomic, which would serve them one after the other.
__device__ __forceinline__ int cell_inc(int *cnt, int key) {
  const int lane = threadIdx.x & 63, lanes = __popcll(__ballot(1));
  const int before = __shfl_up(key, 1);
  const unsigned long long heads = __ballot(lane == 0 || before != key);
  const int head = 63 - __clzll(heads & (~0ull >> (63 - lane)));
  const unsigned long long after = heads & (~1ull << lane);
  int base = 0;
  if (head == lane) base = atomicAdd(cnt + key, (after ? __ffsll((long long)after) - 1 : lanes) - lane);
  return __shfl(base, head) + lane - head;
}

// Error bits of the device error word.
enum : unsigned { ERR_RANGE = 1u, ERR_NUMERIC = 2u };

// Statistics of the push kernel: tiles that fell back to global memory
// (bounding box too large for LDS) and tiles processed, counted in STAT_SLOTS
// pairs of counters on cache lines of their own and added up by the host.
// (Device-scope atomics on one address are served every 12 ns: a single
// counter held a launch of 16384 tiles for 197 us, of 65536 for 790 us.)
enum { STAT_FALLBACK = 0, STAT_TILES = 1 };
constexpr int STAT_SLOTS = 256, STAT_STRIDE = 32, NSTAT = STAT_SLOTS * STAT_STRIDE;
__device__ __forceinline__ void count_stat(unsigned *stats, int which) {
  atomicAdd(stats + (blockIdx.x & (STAT_SLOTS - 1)) * STAT_STRIDE + which, 1u);
}

// LDS of one push+deposit workgroup: staged fields (24 B per node in FP32,
// 48 B in FP64) and current accumulators (3 x 8 B per node).  The budget is
// set per handle from the tile shape (push_lds_bytes), between the minimum
// and maximum here.
constexpr int PUSH_THREADS = 256;
template <class T> using lptr = T __attribute__((address_space(3))) *;

// 1/sqrt(x) and 1/x: hardware approximations (~1 ulp) in FP32, IEEE in FP64.
__device__ __forceinline__ float rsqrt_(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ double rsqrt_(double x) { return 1.0 / sqrt(x); }
__device__ __forceinline__ float rcp_(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double rcp_(double x) { return 1.0 / x; }

// Relativistic Boris rotation: u^{n-1/2} -> u^{n+1/2} with E^n, B^n.
template <class R>
__device__ __forceinline__ void boris(R qmhdt, const R E[3], const R B[3], R u[3]) {
  const R e0 = qmhdt * E[0], e1 = qmhdt * E[1], e2 = qmhdt * E[2];
  const R m0 = u[0] + e0, m1 = u[1] + e1, m2 = u[2] + e2;
  const R ig = rsqrt_(R(1) + m0 * m0 + m1 * m1 + m2 * m2);
  const R t0 = qmhdt * B[0] * ig, t1 = qmhdt * B[1] * ig, t2 = qmhdt * B[2] * ig;
  const R sf = R(2) * rcp_(R(1) + t0 * t0 + t1 * t1 + t2 * t2);
  const R s0 = t0 * sf, s1 = t1 * sf, s2 = t2 * sf;
  const R p0 = m0 + (m1 * t2 - m2 * t1);
  const R p1 = m1 + (m2 * t0 - m0 * t2);
  const R p2 = m2 + (m0 * t1 - m1 * t0);
  u[0] = m0 + (p1 * s2 - p2 * s1) + e0;
  u[1] = m1 + (p2 * s0 - p0 * s2) + e1;
  u[2] = m2 + (p0 * s1 - p1 * s0) + e2;
}

// Velocity from momentum, every operation rounded once in this order (the
// out-of-plane velocity enters the fixed-point deposit, which tests reproduce
// bit for bit on the host): g = sqrt(((1 + u1 u1) + u2 u2) + u3 u3) and
// v = u * (1/g), square root and reciprocal correctly rounded.
template <class R>
__device__ __forceinline__ void velocity(const R u[3], R v[3]) {
#pragma clang fp contract(off)
  R s = R(1) + u[0] * u[0];
  s = s + u[1] * u[1];
  s = s + u[2] * u[2];
  const R ig = inv_gamma(s);
  v[0] = u[0] * ig;
  v[1] = u[1] * ig;
  v[2] = u[2] * ig;
}

// State of one particle as loaded from the buffers.
template <class R>
struct PState {
  int cell;
  R f1, f2, u1, u2, u3, qw;
};

template <class R>
__device__ __forceinline__ PState<R> load_state(const Parts<R> &P, int p) {
  PState<R> s;
  s.cell = *elem(P.cell, p);
  s.f1 = *elem(P.f1, p);
  s.f2 = *elem(P.f2, p);
  s.u1 = *elem(P.u1, p);
  s.u2 = *elem(P.u2, p);
  s.u3 = *elem(P.u3, p);
  s.qw = *elem(P.qw, p);
  return s;
}

template <class R>
__device__ __forceinline__ void store_state(const Parts<R> &P, int p, const PState<R> &s) {
  *elem(P.cell, p) = s.cell;
  *elem(P.f1, p) = s.f1;
  *elem(P.f2, p) = s.f2;
  *elem(P.u1, p) = s.u1;
  *elem(P.u2, p) = s.u2;
  *elem(P.u3, p) = s.u3;
}
// Has the loads of s returned here.  Loads and stores are counted in one queue:
// a state still awaited when the next particle starts would wait out the stores
// issued after its loads as well (277 -> 265 us on 8192 x 512 cells, two
// particles a cell).
template <class R>
__device__ __forceinline__ void arrived(PState<R> &s) {
  asm volatile("" : "+v"(s.cell), "+v"(s.f1), "+v"(s.f2), "+v"(s.u1), "+v"(s.u2), "+v"(s.u3), "+v"(s.qw));
}

__device__ __forceinline__ int wave_min(int v) {
  for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o));
  return v;
}
__device__ __forceinline__ int wave_max(int v) {
  for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o));
  return v;
}

// Cell i (0 <= i < n) relative to a tile origin, in the tile's frame: the
// period [-o, n - o) with o = (n - T) / 2, i.e. centred on the tile, so that
// particles may drift half the rest of the box from their tile before the
// frame's edge splits them.
__device__ __forceinline__ int frame_pow2(int d, int o, int n) { return ((d + o) & (n - 1)) - o; }
__device__ __forceinline__ int frame_any(int d, int o, int n) {
  d += (d < -o) ? n : 0;
  d -= (d >= n - o) ? n : 0;
  return d;
}
// i mod n for any i within a few periods
__device__ __forceinline__ int wrap_any(int i, int n) {
  while (i >= n) i -= n;
  while (i < 0) i += n;
  return i;
}

// Walks the nodes of a W x H box with the workgroup's threads: f(row, column).
// Rows of up to 32 (64) nodes take half a wave (a wave) each, so that no
// thread divides; wider rows are walked in pieces of 64.
template <class F>
__device__ __forceinline__ void for_box(int W, int H, F f) {
  const int sh = W <= 32 ? 5 : 6, lanes = 1 << sh;
  for (int b = (int)threadIdx.x >> sh; b < H; b += PUSH_THREADS >> sh)
    for (int a = (int)threadIdx.x & (lanes - 1); a < W; a += lanes) f(b, a);
}

// Bounding box of the cells a thread's particles move to, then of the
// workgroup's (nbox, initialised before a barrier).
struct CellBox {
  int lo1 = 1 << 30, hi1 = -(1 << 30), lo2 = 1 << 30, hi2 = -(1 << 30);
  __device__ __forceinline__ void add(int d1, int d2) {
    lo1 = min(lo1, d1); hi1 = max(hi1, d1);
    lo2 = min(lo2, d2); hi2 = max(hi2, d2);
  }
  __device__ __forceinline__ void reduce(int *nbox) const {
    const int a = wave_min(lo1), b = wave_max(hi1), c = wave_min(lo2), d = wave_max(hi2);
    if ((threadIdx.x & 63) == 0) {
      atomicMin(&nbox[0], a); atomicMax(&nbox[1], b);
      atomicMin(&nbox[2], c); atomicMax(&nbox[3], d);
    }
  }
};

// Means of the n values whose parts of the sums the workgroup's threads hold.  smem: 16
// bytes of LDS, free again when this returns.
__device__ __forceinline__ void group_mean(long long s1, long long s2, int n, unsigned char *smem, int &m1,
                                           int &m2) {
  const lptr<unsigned long long> sum = (lptr<unsigned long long>)smem;
  if (threadIdx.x < 2) sum[threadIdx.x] = 0;
  __syncthreads();
  for (int o = 32; o > 0; o >>= 1) {
    s1 += __shfl_xor(s1, o);
    s2 += __shfl_xor(s2, o);
  }
  if ((threadIdx.x & 63) == 0) {
    __hip_atomic_fetch_add(sum, (unsigned long long)s1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __hip_atomic_fetch_add(sum + 1, (unsigned long long)s2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  __syncthreads();
  m1 = (int)((long long)sum[0] / n);
  m2 = (int)((long long)sum[1] / n);
  __syncthreads();
}

// The current box of a tile whose particles have spread too far for the boxes of
// fields and currents: all of its nodes where they number at most cap, or as many around
// the particles' mean cell, the margin about the tile the same on all sides.  Holds
// the deposits of the particles in cells lo .. hi; cells lo - 2 .. hi + 3.
struct WideBox {
  int lo1, hi1, lo2, hi2, W, H;
  __device__ __forceinline__ bool holds(int l1, int l2) const {
    return l1 >= lo1 && l1 <= hi1 && l2 >= lo2 && l2 <= hi2;
  }
};
// smem: 16 bytes of LDS.  Called by the whole workgroup.
template <class R>
__device__ __forceinline__ WideBox wide_box(const Run<R> &r, const Parts<R> &P, int start, int end,
                                            int ref1, int ref2, int lo1, int hi1, int lo2, int hi2,
                                            int cap, unsigned char *smem) {
  WideBox b{lo1, hi1, lo2, hi2, hi1 - lo1 + 6, hi2 - lo2 + 6};
  if ((long long)b.W * b.H > cap) {
    const int f1 = (r.n1 - r.T1) >> 1, f2 = (r.n2 - r.T2) >> 1;
    long long s1 = 0, s2 = 0;
    for (int p = start + (int)threadIdx.x; p < end; p += PUSH_THREADS) {
      const int cell = *elem(P.cell, p);
      s1 += frame_pow2((cell & (r.n1 - 1)) - ref1, f1, r.n1);
      s2 += frame_any((cell >> r.log2n1) - ref2, f2, r.n2);
    }
    int m1, m2;
    group_mean(s1, s2, end - start, smem, m1, m2);
    int W = min(b.W, r.T1 + 6), H = min(b.H, r.T2 + 6);
    if ((long long)W * H > cap) W = min(W, 64);  // a tile that is too large by itself
    for (;;) {
      const int w = min(b.W, W + 2), h = min(b.H, H + 2);
      if ((w == W && h == H) || (long long)w * h > cap) break;
      W = w;
      H = h;
    }
    H = min(b.H, cap / W);
    b.lo1 = max(lo1, min(m1 - (W - 6) / 2, hi1 - (W - 6)));
    b.lo2 = max(lo2, min(m2 - (H - 6) / 2, hi2 - (H - 6)));
    b.hi1 = b.lo1 + W - 6;
    b.hi2 = b.lo2 + H - 6;
    b.W = W;
    b.H = H;
  }
  return b;
}

__device__ __forceinline__ float uniform(float x) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x)));
}

// Columns of the 2D push's current box for tiles t wide: the tile, two cells of
// drift on each side, the stencil's six and one more, which makes the row
// stride odd for even widths (rows a multiple of 16 of the 8-byte bank slots
// apart put the rows a wave touches on the same banks: 191 instead of 153 us on
// 2048 x 512 cells).
__host__ __device__ constexpr int push_cols(int t) { return t + 11; }
// LDS bytes of its boxes for a current box of w columns and h rows: 64-bit
// accumulators of three components, then the six fields, two nodes less along
// each axis (one with the cubic shape).
__host__ __device__ constexpr long long push_box_bytes(int w, int h, size_t real, int less = 2) {
  return ((3ll * w * h * 8 + 15) & ~15ll) + (long long)(w - less) * (h - less) * 6 * (long long)real;
}
constexpr int PUSH_LDS_MIN = 16384;
constexpr int PUSH_LDS_MAX = 64512;  // with the static LDS, under 64 KiB
constexpr int LDS_PIECE = 1280, LDS_PIECES = 128;  // a compute unit's LDS is given out in pieces
// The 3D push.  FP32 form: 4 waves per SIMD (128 registers), four workgroups of 256
// threads per compute unit with LDS_256 bytes each (three with LDS_3), or two of NT_MAX =
// 512 with LDS_MAX for tiles that need more.  FP64 form: 2 waves per SIMD (256
// registers), two workgroups of 256.
template <class R> struct Push3Occupancy {
  static constexpr int WAVES_PER_SIMD = 2, NT_MAX = 256, LDS_256 = 80896, LDS_3 = 80896, LDS_MAX = 80896;
};
template <> struct Push3Occupancy<float> {
  static constexpr int WAVES_PER_SIMD = 4, NT_MAX = 512, LDS_256 = 40448, LDS_3 = 53248, LDS_MAX = 80896;
};

// ---------------------------------------------------------------- launches
// Host-side launch wrappers (kernels.hip), one instantiation per precision.
template <class R>
struct Launch {
  // unit: every run's charges satisfy the 24-bit product bound (FP32 form);
  // ec: energy-conserving gather (all runs of a handle share it)
  static void push_deposit(const Run<R> *runs, const Item *items, int nitems, int parity,
                           int pp, int lds_bytes, int tile1, bool unit, bool ec,
                           unsigned *err, unsigned *stats, hipStream_t s);
  // tile sort of the particles of all runs: items are (run, first particle,
  // count) chunks, and (run, b, 0) for every block b of SORT_BLOCK cell counts
  static void sort(const Run<R> *runs, const Item *chunks, int nchunks, const Item *blocks,
                   int nblocks, int pp, hipStream_t s);
  // row transforms: ncomp = 3 components per block (item = run, row[, group])
  // or 1 (item = run, row, component) for long rows
  static void fft_j(const Run<R> *runs, const Item *items, int nitems, int parity, int maxM,
                    int ncomp, hipStream_t s);
  static void kupdate(const Run<R> *runs, const Item *items, int nitems, int parity, int strip,
                      hipStream_t s);
  // 3D: the same update as two passes (E and the half-step B, then B)
  static void kupdate3(const Run<R> *runs, const Item *items, int nitems, int parity,
                       hipStream_t s);
  static void push_deposit3(const Run<R> *runs, const Item *items, int nitems, int parity,
                            int pp, int lds_bytes, unsigned *err, unsigned *stats,
                            hipStream_t s);
  static void ifft_eb(const Run<R> *runs, const Item *items, int nitems, int parity, int maxM,
                      int ncomp, hipStream_t s);
  static void fields_to_k(const Run<R> *runs, const Item *items, int nitems, int parity,
                          int maxM, int ncomp, hipStream_t s);
};


// Diagnostics and helpers (FP64 unless noted).
// 3D: charge density in FP64 from the particle state (any form).
template <class R>
void launch_rho3(const Run<R> *run_dev, int pp, int np, double *rho, hipStream_t s);
// 3D Gauss residual per row (i2, i3) of the k-space master copy; rows_out [rows][3].
template <class R>
void launch_gauss3(const Run<R> *run_dev, int rows, int n1, int parity, const double *rho,
                   const double2 *tw64, const double *sym64, const double *filt, double idx2,
                   double idx3, double *rows_out, hipStream_t s);
// 3D continuity residual max |(rho_n - rho_o)/dt + div j| with j = fac[d] * J.
template <class A>
void launch_cont3(const double *rn, const double *ro, const A *J, int n1, int n2, int n3,
                  double dt, double f1, double f2, double f3, double idx1, double idx2,
                  double idx3, double *partial, int nblocks, hipStream_t s);
void launch_rho_fixed(const Run<float> *run_dev, int pp, int np, long long *rho, hipStream_t s);
// 2D with the cubic shape: push + deposit (items: run, tile; unit: every
// run's |charge| 2^P fits the 24-bit products), and the charge density in the
// deposit's units (FP32 form: integers, FP64 form: physical)
template <class R>
void launch_push_cubic(const Run<R> *runs, const Item *items, int nitems, int parity, int pp,
                       int lds_bytes, int tile1, bool unit, bool ec, unsigned *err, hipStream_t s);
template <class R>
void launch_rho_cubic(const Run<R> *run_dev, int pp, int np, typename AccOf<R>::T *rho,
                      hipStream_t s);
void launch_rho_fp64(const Run<double> *run_dev, int pp, int np, double *rho, hipStream_t s);
// Moving antenna of a 2D run (see hp_set_antenna): device parameters.
struct AntennaDev {
  int run;             // run index in the handle
  int n1, n2;
  double dx1, dx2, dt;
  double x0, v, t0, T, K0, omega, phase, x2c, waist;
  double scale;        // physical j3 -> accumulator units
};
// Adds every antenna's current of the step (time (*step + 1/2) dt) to j3 of
// the run's accumulators of the given parity; then, in a separate launch,
// the step counter advances by one (both are captured in step graphs).
template <class R>
void launch_antenna(const Run<R> *runs, const AntennaDev *ants, int nant, int maxn2, int parity,
                    const long long *step, hipStream_t s);
void launch_step_tick(long long *step, hipStream_t s);
template <class R>
void launch_energy(const R *F, long long cells, double *partial, int nblocks, hipStream_t s);
template <class R>
void launch_kinetic(const Run<R> *run_dev, int pp, double *partial, int nblocks, hipStream_t s);
// Gauss residual per row: rho (physical, FP64, [n2][n1]) and the k-space E1,E2
// of a run; writes per-row [3]: sum |R|^2, max |R|, sum |f rho|^2.
template <class R>
void launch_gauss(const Run<R> *run_dev, int n2, int n1, int parity, const double *rho,
                  const double2 *tw64, const double *sym64, const double *filt, double idx2,
                  double *rows_out, hipStream_t s);
void launch_cont_fixed(const long long *rho_new, const long long *rho_old, const long long *J,
                       int n1, int n2, long long *partial_max, int nblocks, hipStream_t s);
void launch_cont_fp64(const double *rho_new, const double *rho_old, const double *J, int n1,
                      int n2, double dt, double idx1, double idx2, double *partial_max,
                      int nblocks, hipStream_t s);
void launch_debug_deposit(int n1, int n2, int P, float inv_wunit, float c3, int np,
                          const int *cell0, const float *off0, const int *cell1,
                          const float *off1, const float *v3, const float *qw, long long *J,
                          unsigned *err, hipStream_t s);
template <class R>
void launch_inverse_rows(const typename Cplx<R>::T *Xk, int nk, int n1, int nrows,
                         const typename Cplx<R>::T *tw, R scale, R *out, hipStream_t s);

// ---------------------------------------------------------------- device I/O
// (io.hip) Geometry of a Cartesian run for loading particles from FP64 device
// arrays: box lengths L = n dx, cell sizes, packing of the cell index.
struct LoadGeom {
  int dim, n1, n2, n3, log2n1, sh3;
  double L[3], dx[3];
};
// Validation pass over n particles (x[dim][n], u[3][n], w[n] in device memory):
// *bad |= 1 for a non-finite input, count[cells] += particles per cell,
// qbits[0] = max and qbits[1] = min of |(R)(q w)| as FP64 bit patterns.
template <class R>
void launch_scan_particles(const LoadGeom &g, long long n, const double *x, const double *u,
                           const double *w, double q, int *count, unsigned long long *qbits,
                           unsigned *bad, hipStream_t s);
void launch_max_int(const int *a, long long n, int *out, hipStream_t s);
template <class A>
void launch_current_out(const A *raw, long long n, double f, double bg, double *out, hipStream_t s);
template <class R>
void launch_real_to_double(const R *in, long long n, double *out, hipStream_t s);
void launch_zero_i64(long long *p, long long n, hipStream_t s);
// Conversion pass: the run's structure of arrays A in input order.
template <class R>
void launch_load_particles(const LoadGeom &g, long long n, const double *x, const double *u,
                           const double *w, double q, Parts<R> A, hipStream_t s);
// The run's particle state (buffer pp, current order) into device buffers.
template <class R>
void launch_unload_particles(const Run<R> *run_dev, int pp, int np, int *cell, R *off, R *u, R *qw,
                             int *id, hipStream_t s);

}  // namespace hp
