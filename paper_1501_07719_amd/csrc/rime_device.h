// Device-side numeric helpers shared by the kernels of librime.so: the
// precision traits of the two arithmetic paths (float64, and float32 with an
// accurate sine/cosine of turns and the gfx950 hardware exp2, reciprocal and
// reciprocal square root), the error-free phase argument, and float64
// compensated (two-sum) accumulation with wavefront and workgroup reductions.
#pragma once

#include "rime_internal.h"

namespace rime {

// ---------------------------------------------------------------------------
// Numeric helpers
// ---------------------------------------------------------------------------

constexpr double kLog2e = 1.44269504088896340735992468100189214;

// Pointers into the constant address space: loads through them at a
// wavefront-uniform address become scalar (SMEM) loads whose results are
// operands in SGPRs.  Only data written by an earlier kernel is read this way.
// (The host compilation pass parses the device code without address spaces.)
#if defined(__HIP_DEVICE_COMPILE__)
#define RIME_CONST __attribute__((address_space(4)))
#else
#define RIME_CONST
#endif

template <class T>
__device__ inline const RIME_CONST T *const_ptr(const void *p) {
  return (const RIME_CONST T *)(p);  // an address-space cast needs the C form
}

// Plain 4-vector for loads through constant-space pointers (the HIP vector
// types have no copy from that address space); copies merge into one wide
// scalar load.
template <class R>
struct alignas(4 * sizeof(R)) Quad {
  R x, y, z, w;
};

// Returns x unchanged in a VGPR the compiler cannot see through, so that a
// constant folded into x (an LDS region offset) stays in the per-lane base
// address instead of being re-added inside a loop.
__device__ inline uint32_t opaque_vgpr(uint32_t x) {
  asm volatile("" : "+v"(x));
  return x;
}

// A float64 constant in an SGPR pair: an operand of v_fma_f64, where hipcc
// otherwise copies the constant into the destination of a v_fmac_f64 each time.
__device__ inline double sgpr_const(double x) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm("" : "+s"(x));
#endif
  return x;
}

// The set descriptor of a work item, read through the constant space so that
// its fields are wavefront-uniform (scalar) values.
__device__ inline SetDesc load_set(const KParams &p, int set) {
  if (!p.sets) return p.one;
  const RIME_CONST SetDesc *q = const_ptr<SetDesc>(p.sets) + set;
  SetDesc d;
  d.lm = q->lm;
  d.stokes = q->stokes;
  d.alpha = q->alpha;
  d.gshape = q->gshape;
  d.xshape = q->xshape;
  d.npsrc = q->npsrc;
  d.ngsrc = q->ngsrc;
  d.nxsrc = q->nxsrc;
  d.src_off = q->src_off;
  return d;
}

template <class R> struct Num;

template <> struct Num<double> {
  using R2 = double2;
  using R4 = double4;
  // sin and cos of 2 pi r for r in [-1/2, 1/2] turns.  The quarter-turn
  // reduction r = q/4 + x is exact; with y = x^2 the polynomials interpolate
  // sin(2 pi x) / x and (cos(2 pi x) - 1) / y at the Chebyshev nodes of
  // y in [0, 1/64] (errors 4e-17 relative and 2e-17 with the coefficients
  // rounded to float64), so that each result carries the rounding of its last
  // two operations; the quadrant permutes and negates the pair.  About 30
  // instructions against 70 of sincospi() (8 antennas, 31 timesteps, 60
  // channels, 24 points, no beam, predict: 24.3 against 41.9 us with the beam's
  // own polynomials below; 64-antenna planes with k3 4.0 -> 3.4 ms).
  __device__ static inline void sincos_turns(double r, double *s, double *c) {
    const double q = rint(4.0 * r);
    const double x = fma(-0.25, q, r);
    const double y = x * x;
    double sp = 3.7808689593022957;
    sp = fma(sp, y, sgpr_const(-15.093804209987114));
    sp = fma(sp, y, sgpr_const(42.058685020160894));
    sp = fma(sp, y, sgpr_const(-76.70585970427454));
    sp = fma(sp, y, sgpr_const(81.60524927594804));
    sp = fma(sp, y, sgpr_const(-41.341702240399634));
    sp = fma(sp, y, sgpr_const(6.283185307179586));
    double cp = -1.6990343940660637;
    cp = fma(cp, y, sgpr_const(7.903206911569678));
    cp = fma(cp, y, sgpr_const(-26.426253275854723));
    cp = fma(cp, y, sgpr_const(60.24464135270201));
    cp = fma(cp, y, sgpr_const(-85.4568172066438));
    cp = fma(cp, y, sgpr_const(64.93939402266824));
    cp = fma(cp, y, sgpr_const(-19.739208802178716));
    const double sn = sp * x, cs = fma(cp, y, 1.0);
    // sin and cos of 2 pi x + iq pi/2
    const int iq = static_cast<int>(q);
    const double ss = (iq & 1) ? cs : sn, cc = (iq & 1) ? sn : cs;
    *s = (iq & 2) ? -ss : ss;
    *c = ((iq + 1) & 2) ? -cc : cc;
  }
  // expb(y) = exp(y / kExpScale) = 2^y for y <= 0.  2^y = 2^n 2^f with n the
  // nearest integer and f = y - n exact; 2^f on [-1/2, 1/2] is the polynomial
  // that interpolates it at the 12 Chebyshev nodes, 2.0e-17 relative with the
  // coefficients rounded to float64.  19 instructions against 24 of exp().
  // Below 2^-1100 the result is 0 (the cut keeps y = -infinity finite; a NaN
  // passes through).
  static constexpr double kExpScale = kLog2e;
  __device__ static inline double expb(double y) {
    y = y < -1100.0 ? -1100.0 : y;
    const double n = rint(y);
    const double f = y - n;
    double r = sgpr_const(4.4558179083360645e-10);
    r = fma(r, f, sgpr_const(7.074194297288521e-09));
    r = fma(r, f, sgpr_const(1.0178057087733941e-07));
    r = fma(r, f, sgpr_const(1.3215432535912375e-06));
    r = fma(r, f, sgpr_const(1.5252733841556773e-05));
    r = fma(r, f, sgpr_const(0.00015403530463724353));
    r = fma(r, f, sgpr_const(0.001333355814640647));
    r = fma(r, f, sgpr_const(0.009618129107587256));
    r = fma(r, f, sgpr_const(0.055504108664821625));
    r = fma(r, f, sgpr_const(0.24022650695910158));
    r = fma(r, f, sgpr_const(0.6931471805599453));
    r = fma(r, f, 1.0);
    return __builtin_amdgcn_ldexp(r, static_cast<int>(n));
  }
  // the 32 bits packed into the last word of a per-baseline record
  __device__ static inline uint32_t bits(double w) {
    return static_cast<uint32_t>(__double_as_longlong(w));
  }
  __device__ static inline double from_bits(uint32_t b) {
    return __longlong_as_double(static_cast<long long>(b));
  }
  // 1 / x for x well inside the exponent range: the hardware estimate and two
  // Newton steps
  __device__ static inline double rcp(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = fma(fma(-x, r, 1.0), r, r);
    return fma(fma(-x, r, 1.0), r, r);
  }
  __device__ static inline double rsqrt_(double x) { return rsqrt(x); }
};

template <> struct Num<float> {
  using R2 = float2;
  using R4 = float4;
  // sin and cos of 2 pi r for r in [-1/2, 1/2] turns, to about one float32
  // unit: the quarter-turn reduction r = q/4 + x is exact in float64, the
  // angle 2 pi x (|2 pi x| <= pi/4) is rounded once to float32, and the Taylor
  // series of sin to degree 9 and of cos to degree 10 leave truncation errors
  // below 2e-9 there; the quadrant then permutes and negates the pair.  (The
  // hardware v_sin_f32 / v_cos_f32 are several float32 units less accurate,
  // which shows in sums that cancel.)
  __device__ static inline void sincos_turns(double r, float *s, float *c) {
    const double q = rint(4.0 * r);
    const float th = static_cast<float>((r - 0.25 * q) * (2.0 * 3.14159265358979323846));
    const float t2 = th * th;
    const float sn =
        th * (1.0f + t2 * (-1.0f / 6.0f +
                           t2 * (1.0f / 120.0f + t2 * (-1.0f / 5040.0f + t2 * (1.0f / 362880.0f)))));
    const float cs =
        1.0f + t2 * (-0.5f + t2 * (1.0f / 24.0f +
                                   t2 * (-1.0f / 720.0f +
                                         t2 * (1.0f / 40320.0f + t2 * (-1.0f / 3628800.0f)))));
    // sin and cos of th + iq pi/2
    const int iq = static_cast<int>(q) & 3;
    const float ss = (iq & 1) ? cs : sn, cc = (iq & 1) ? sn : cs;
    *s = (iq & 2) ? -ss : ss;
    *c = ((iq + 1) & 2) ? -cc : cc;
  }
  static constexpr double kExpScale = kLog2e;
  __device__ static inline float expb(float y) { return __builtin_amdgcn_exp2f(y); }
  __device__ static inline uint32_t bits(float w) { return __float_as_uint(w); }
  __device__ static inline float from_bits(uint32_t b) { return __uint_as_float(b); }
  __device__ static inline float rcp(float x) { return __builtin_amdgcn_rcpf(x); }
  __device__ static inline float rsqrt_(float x) { return __builtin_amdgcn_rsqf(x); }
};

// Error-free transformations for the phase argument of eq. k_term.  The path
// length tau = u l + v m + w (n - 1) times nu / c spans hundreds to thousands of
// turns on the benchmark arrays; carried as an unevaluated float64 pair
// (hi + lo) through exact products and sums, its fraction of a turn is the
// exact fraction of the products of the float64 inputs to about 1e-16 turns,
// whatever the rounding order of a plain evaluation would have been.
// Every function here turns contraction off: fusing a product into a
// following sum (hipcc contracts by default) would round differently from
// the product that the error term is taken against, and break the identity.

// Error-free sum (Knuth): s + e == a + b exactly.
__device__ inline void two_sum(double a, double b, double &s, double &e) {
#pragma clang fp contract(off)
  s = a + b;
  const double bp = s - a;
  e = (a - (s - bp)) + (b - bp);
}

// Error-free product with one fused multiply-add: p + e == a b exactly.
__device__ inline void two_prod(double a, double b, double &p, double &e) {
#pragma clang fp contract(off)
  p = a * b;
  e = fma(a, b, -p);
}

struct Pair {
  double hi, lo;
};

// tau = u l + v m + w (n - 1) (metres) as hi + lo.
__device__ inline Pair path_length(double u, double v, double w, double l, double m,
                                   double nm1) {
#pragma clang fp contract(off)
  double p1, e1, p2, e2, p3, e3, s, es1, es2;
  two_prod(u, l, p1, e1);
  two_prod(v, m, p2, e2);
  two_prod(w, nm1, p3, e3);
  two_sum(p1, p2, s, es1);
  two_sum(s, p3, s, es2);
  Pair t;
  two_sum(s, (e1 + e2 + e3) + (es1 + es2), t.hi, t.lo);
  return t;
}

// tau nu / c in turns minus its nearest integer (ties to even), in
// [-1/2, 1/2] up to rounding: exp(-2 pi i x) has period 1 in x.
__device__ inline double phase_frac(Pair tau, double nuc) {
#pragma clang fp contract(off)
  double xh, xe;
  two_prod(tau.hi, nuc, xh, xe);
  const double xl = xe + tau.lo * nuc;
  return (xh - rint(xh)) + xl;
}

// The phase argument of one (antenna, source) pair, for its channels.
// EXACT (the float64 path): the error-free pair above.  Otherwise (the
// float32 path) one plain float64 evaluation: at a few thousand turns it is
// within about 1e-12 turns of the exact fraction, four orders of magnitude
// below what a float32 sine and cosine resolve, for a fifth of the work.
template <bool EXACT> struct PhaseArg;

template <> struct PhaseArg<true> {
  Pair tau;
  __device__ inline PhaseArg(double u, double v, double w, double l, double m, double nm1)
      : tau(path_length(u, v, w, l, m, nm1)) {}
  __device__ inline double turns(double nuc) const { return phase_frac(tau, nuc); }
};

template <> struct PhaseArg<false> {
  double tau;
  __device__ inline PhaseArg(double u, double v, double w, double l, double m, double nm1)
      : tau(fma(w, nm1, fma(v, m, u * l))) {}
  __device__ inline double turns(double nuc) const {
    const double x = tau * nuc;
    return x - rint(x);
  }
};

// Beam factors of the float32 path for a beam angle x in [0, beam_clip]
// (the plan accepts beam_clip <= 1.5 rad): e = cos^3(x) and, when wanted,
// tan(x)/x, the factor of d ln e / dl.  With z = x^2, cos x = C(z) and
// sin(x)/x = P(z) are their Taylor series to z^6, whose truncation errors
// stay below 5e-8 relative up to 1.5 rad (below 1e-10 up to 1.0881 rad);
// tan(x)/x = P(z) / C(z) needs no special case at x = 0.
__device__ inline void beam_f32(float x, bool want_tan, float *e, float *tx) {
  const float z = x * x;
  const float c =
      1.0f + z * (-1.0f / 2.0f +
                  z * (1.0f / 24.0f +
                       z * (-1.0f / 720.0f +
                            z * (1.0f / 40320.0f +
                                 z * (-1.0f / 3628800.0f + z * (1.0f / 479001600.0f))))));
  *e = c * c * c;
  if (want_tan) {
    const float sx =
        1.0f + z * (-1.0f / 6.0f +
                    z * (1.0f / 120.0f +
                         z * (-1.0f / 5040.0f +
                              z * (1.0f / 362880.0f +
                                   z * (-1.0f / 39916800.0f + z * (1.0f / 6227020800.0f))))));
    *tx = sx * __builtin_amdgcn_rcpf(c);
  }
}

// The same in float64: polynomials of z = x^2 in [0, 2.25] that interpolate
// (cos x - 1) / z and sin(x)/x at the Chebyshev nodes (errors 1.0e-17 in cos x
// and 3.2e-17 relative).  They take z, so that no square root of the radius is needed.
__device__ inline void beam_f64(double z, bool want_tan, double *e, double *tx) {
  double c = -1.5208314371212568e-16;
  c = fma(c, z, sgpr_const(4.7777511764295694e-14));
  c = fma(c, z, sgpr_const(-1.1470706408552252e-11));
  c = fma(c, z, sgpr_const(2.0876756468878697e-09));
  c = fma(c, z, sgpr_const(-2.755731921994676e-07));
  c = fma(c, z, sgpr_const(2.480158730156964e-05));
  c = fma(c, z, sgpr_const(-0.001388888888888885));
  c = fma(c, z, sgpr_const(0.041666666666666664));
  c = fma(c, z, -0.5);
  c = fma(c, z, 1.0);
  *e = c * c * c;
  if (want_tan) {
    double sx = -8.00323184555007e-18;
    sx = fma(sx, z, sgpr_const(2.810422181166706e-15));
    sx = fma(sx, z, sgpr_const(-7.647136389681425e-13));
    sx = fma(sx, z, sgpr_const(1.6059043399982724e-10));
    sx = fma(sx, z, sgpr_const(-2.5052108381120333e-08));
    sx = fma(sx, z, sgpr_const(2.755731922395986e-06));
    sx = fma(sx, z, sgpr_const(-0.00019841269841269752));
    sx = fma(sx, z, sgpr_const(0.008333333333333333));
    sx = fma(sx, z, sgpr_const(-0.16666666666666666));
    sx = fma(sx, z, 1.0);
    *tx = sx * Num<double>::rcp(c);
  }
}

// a^2 + b^2 with each product rounded on its own (l^2 + m^2 as written).
__device__ inline double sumsq_rn(double a, double b) {
#pragma clang fp contract(off)
  return a * a + b * b;
}

// Kernel modes.  MODE_RESID is the forward of the float64-residual mixed
// mode: float64 arithmetic over float32 data and weights, chi^2 partials and,
// when p.rho_b is set, the weighted residual in Stokes form (float32) per
// visibility and, with p.pme_adj, in the antenna-pair slots.  MODE_ADJ is its
// float32 adjoint: pass 2 alone, over the residual read from p.rho_b.
enum { MODE_PREDICT = 0, MODE_CHI2 = 1, MODE_GRAD = 2, MODE_RESID = 3, MODE_ADJ = 4 };

template <bool B, class X, class Y> struct Pick { using T = X; };
template <class X, class Y> struct Pick<false, X, Y> { using T = Y; };

// Source tiles of a set: points first, then Gaussians, then disks; tile k
// covers sources [s0, s0 + cnt) of one morphology.
struct SrcTile {
  int shape, s0, cnt;
};

__device__ inline SrcTile src_tile(const SetDesc &sd, int k, int ns, int npt, int ngt) {
  if (k < npt) return {SHAPE_POINT, k * ns, min(ns, sd.npsrc - k * ns)};
  if (k < npt + ngt) {
    const int s0 = sd.npsrc + (k - npt) * ns;
    return {SHAPE_GAUSS, s0, min(ns, sd.npsrc + sd.ngsrc - s0)};
  }
  const int s0 = sd.npsrc + sd.ngsrc + (k - npt - ngt) * ns;
  return {SHAPE_DISK, s0, min(ns, sd.npsrc + sd.ngsrc + sd.nxsrc - s0)};
}

// The per-antenna term of one (antenna, source) at channel c: a = e K and, for
// the adjoint, k3 with d ln e / d(l, m) = k3 (l - dl_p, m - dm_p).  The angles
// are formed in float64 and their sines and cosines to within about a unit of
// R (N::sincos_turns): each factor is reused by every baseline that holds the
// antenna.  r2b and rb: squared distance to the pointing centre and its root
// (float32 only).
template <class R, bool WITH_BETA>
__device__ inline void antenna_term(const KParams &p, const PhaseArg<sizeof(R) == 8> &tau,
                                    double r2b, double rb, int c, typename Num<R>::R2 &a, R &k3) {
  using N = Num<R>;
  const double r = tau.turns(p.nu_c[c]);
  R sn, cs;
  N::sincos_turns(r, &sn, &cs);
  R e = R(1);
  k3 = R(0);
  if (p.beam) {
    // x_b = bs r, bs = beam_k nu / beam_ref_freq, clipped at beam_clip
    // (eq. e_term); the clip is decided on r^2 against the per-channel
    // threshold (beam_clip / bs)^2.
    // d ln e / dl = -3 tan(x) dx/dl, dx/dl = bs (l - dl_p) / r
    //             = -3 bs^2 (l - dl_p) tan(x)/x ; zero past the clip.
    const double bs = p.bsc[c];
    const bool clipped = r2b >= p.clip_r2[c];
    R tx = R(0);
    if constexpr (sizeof(R) == 8) {
      double txd = 0.0;
      beam_f64(clipped ? p.beam_clip * p.beam_clip : bs * bs * r2b, WITH_BETA, &e, &txd);
      if (!clipped) tx = txd;
    } else {
      float txf = 0.0f;
      const double xr = clipped ? p.beam_clip : bs * rb;
      beam_f32(static_cast<float>(xr), WITH_BETA, &e, &txf);
      if (!clipped) tx = txf;
    }
    if (WITH_BETA) k3 = static_cast<R>(p.bk3[c]) * tx;
  }
  a.x = e * cs;
  a.y = -e * sn;
}

// Compensated float64 accumulator.
struct Comp {
  double s = 0.0, c = 0.0;
  __device__ inline void add(double x) {
    double e;
    two_sum(s, x, s, e);
    c += e;
  }
  __device__ inline void merge(double os, double oc) {
    double e;
    two_sum(s, os, s, e);
    c += oc + e;
  }
};

__device__ inline Comp wave_reduce(Comp v) {
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) {
    const double os = __shfl_xor(v.s, off, kWave);
    const double oc = __shfl_xor(v.c, off, kWave);
    v.merge(os, oc);
  }
  return v;
}

// Workgroup reduction of a compensated pair; the result is valid in thread 0.
template <int NT>
__device__ inline Comp block_reduce(Comp v, double2 *scratch) {
  constexpr int NW = NT / kWave;
  v = wave_reduce(v);
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  if (NW == 1) return v;
  __syncthreads();
  if (lane == 0) scratch[wave] = make_double2(v.s, v.c);
  __syncthreads();
  Comp r;
  if (wave == 0) {
    if (lane < NW) {
      r.s = scratch[lane].x;
      r.c = scratch[lane].y;
    }
    r = wave_reduce(r);
  }
  return r;
}

// 2x2 complex matrices in float64, entries (xx, xy, yx, yy) = ([0][0], [0][1],
// [1][0], [1][1]).
struct M22 {
  double re[4], im[4];
};

// a b
__device__ inline M22 m22_mul(const M22 &a, const M22 &b) {
  M22 r;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      double sr = 0.0, si = 0.0;
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int x = 2 * i + k, y = 2 * k + j;
        sr += a.re[x] * b.re[y] - a.im[x] * b.im[y];
        si += a.re[x] * b.im[y] + a.im[x] * b.re[y];
      }
      r.re[2 * i + j] = sr;
      r.im[2 * i + j] = si;
    }
  return r;
}

// a^H
__device__ inline M22 m22_herm(const M22 &a) {
  M22 r;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      r.re[2 * i + j] = a.re[2 * j + i];
      r.im[2 * i + j] = -a.im[2 * j + i];
    }
  return r;
}

__device__ inline M22 m22_load(const double2 *m) {
  M22 r;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const double2 v = m[k];
    r.re[k] = v.x;
    r.im[k] = v.y;
  }
  return r;
}

// V of one visibility from its Stokes sums S (re, im of I, Q, U, V), and, in
// the chi^2 modes, its weighted squared residual (added to `chi`) and, with
// RHO, the weighted residual in Stokes form `rho` that the adjoint takes.
//   PREDICT: V goes to p.vis.  DT: type of data and weights (and of vis).
//   gap, gaq: the baseline's antennas; gg: its diagonal gain products
//   g_pi conj(g_qj); c: channel (with !ok any valid one; nothing is then read
//   or written and rho = 0); vidx: index of the visibility's first correlation.
template <class R, class DT, class A, bool PREDICT, bool RHO, bool TERMS>
__device__ inline void visibility(const KParams &p, bool ok, int t, int gap, int gaq, int c,
                                  int64_t vidx, const double (&S)[8], const double2 (&gg)[4],
                                  Comp &chi, typename Num<A>::R2 (&rho)[4]) {
  using R2 = typename Num<R>::R2;
  using DT2 = typename Num<DT>::R2;
  // Stokes sums -> 2x2 coherency X (eq. brightness_term)
  const double SIr = S[0], SIi = S[1], SQr = S[2], SQi = S[3];
  const double SUr = S[4], SUi = S[5], SVr = S[6], SVi = S[7];
  M22 X;
  X.re[0] = SIr + SQr;  // xx
  X.im[0] = SIi + SQi;
  X.re[1] = SUr - SVi;  // xy = S_U + i S_V
  X.im[1] = SUi + SVr;
  X.re[2] = SUr + SVi;  // yx = S_U - i S_V
  X.im[2] = SUi - SVr;
  X.re[3] = SIr - SQr;  // yy
  X.im[3] = SIi - SQi;
  double Vr[4], Vi[4];
  // V = G_p X G_q^H (eq. 1's direction-independent term, outside the
  // source sum), or the plan's diagonal gains
  M22 Gp, Gq;
  if (TERMS && p.die) {
    const int64_t gi = (static_cast<int64_t>(t) * p.na) * p.nchan + c;
    Gp = m22_load(p.die + (gi + static_cast<int64_t>(gap) * p.nchan) * 4);
    Gq = m22_load(p.die + (gi + static_cast<int64_t>(gaq) * p.nchan) * 4);
    const M22 V = m22_mul(m22_mul(Gp, X), m22_herm(Gq));
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      Vr[k] = V.re[k];
      Vi[k] = V.im[k];
    }
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      Vr[k] = X.re[k] * gg[k].x - X.im[k] * gg[k].y;
      Vi[k] = X.re[k] * gg[k].y + X.im[k] * gg[k].x;
    }
  }
  if (PREDICT) {
    if (ok) {
      R2 *out = static_cast<R2 *>(p.vis) + vidx;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        R2 v;
        v.x = static_cast<R>(Vr[k]);
        v.y = static_cast<R>(Vi[k]);
        out[k] = v;
      }
    }
    return;
  }
  double Yr[4] = {0, 0, 0, 0}, Yi[4] = {0, 0, 0, 0};
  if (ok) {
    const DT2 *D = static_cast<const DT2 *>(p.data) + vidx;
    const DT *W = static_cast<const DT *>(p.weight) + vidx;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const DT2 d = D[k];
      const double w = static_cast<double>(W[k]);
      const double rr = Vr[k] - static_cast<double>(d.x);
      const double ri = Vi[k] - static_cast<double>(d.y);
      chi.add(w * (rr * rr + ri * ri));
      Yr[k] = w * rr;
      Yi[k] = w * ri;
    }
  }
  if (!RHO) return;
  // the residual carried to the coherency X: Z = G_p^H Y G_q (with
  // diagonal gains Z_ij = Y_ij conj(g_pi) g_qj = Y_ij conj(gg_ij)); then
  // rho_I = conj(Zxx) + conj(Zyy), rho_Q = conj(Zxx) - conj(Zyy),
  // rho_U = conj(Zxy) + conj(Zyx), rho_V = i (conj(Zxy) - conj(Zyx))
  double Zr[4], Zi[4];
  if (TERMS && p.die) {
    M22 Y;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      Y.re[k] = Yr[k];
      Y.im[k] = Yi[k];
    }
    const M22 Z = m22_mul(m22_mul(m22_herm(Gp), Y), Gq);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      Zr[k] = Z.re[k];
      Zi[k] = Z.im[k];
    }
    if (ok && p.die_part) {
      // d chi^2 / d conj(G) of this visibility: Y G_q X^H for antenna
      // p and Y^H G_p X for antenna q
      const M22 Ap = m22_mul(m22_mul(Y, Gq), m22_herm(X));
      const M22 Aq = m22_mul(m22_mul(m22_herm(Y), Gp), X);
      double2 *dp = p.die_part + vidx * 2;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        dp[k] = make_double2(Ap.re[k], Ap.im[k]);
        dp[4 + k] = make_double2(Aq.re[k], Aq.im[k]);
      }
    }
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      Zr[k] = Yr[k] * gg[k].x + Yi[k] * gg[k].y;
      Zi[k] = Yi[k] * gg[k].x - Yr[k] * gg[k].y;
    }
  }
  rho[0].x = static_cast<A>(Zr[0] + Zr[3]);
  rho[0].y = static_cast<A>(-(Zi[0] + Zi[3]));
  rho[1].x = static_cast<A>(Zr[0] - Zr[3]);
  rho[1].y = static_cast<A>(-(Zi[0] - Zi[3]));
  rho[2].x = static_cast<A>(Zr[1] + Zr[2]);
  rho[2].y = static_cast<A>(-(Zi[1] + Zi[2]));
  rho[3].x = static_cast<A>(Zi[1] - Zi[2]);
  rho[3].y = static_cast<A>(Zr[1] - Zr[2]);
}

// The plan's diagonal gain products of baseline (gap, gaq): g_pi conj(g_qj).
__device__ inline void gain_products(const KParams &p, int gap, int gaq, double2 (&gg)[4]) {
  const double2 gpi[2] = {make_double2(p.gains[4 * gap + 0], p.gains[4 * gap + 1]),
                          make_double2(p.gains[4 * gap + 2], p.gains[4 * gap + 3])};
  const double2 gqj[2] = {make_double2(p.gains[4 * gaq + 0], p.gains[4 * gaq + 1]),
                          make_double2(p.gains[4 * gaq + 2], p.gains[4 * gaq + 3])};
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const double2 a = gpi[i], b = gqj[j];
      gg[2 * i + j] = make_double2(a.x * b.x + a.y * b.y, a.y * b.x - a.x * b.y);
    }
}

// Workgroups are dealt round-robin to the 8 XCDs; renumbering them makes
// consecutive work items (which share operands through L2) land on one XCD.
__device__ inline int xcd_item(int nitems) {
  const int per_xcd = (nitems + 7) / 8;
  return static_cast<int>(blockIdx.x % 8) * per_xcd + static_cast<int>(blockIdx.x / 8);
}

// chi^2 of one set from its per-item (sum, compensation) partials, in a fixed
// order; all 256 threads of the workgroup take part.
__device__ inline void chi2_reduce(const KParams &p, int set, double2 *scr) {
  Comp acc;
  const double2 *part = p.chi2_part + static_cast<int64_t>(set) * p.chi2_items;
  // each thread merges items tid, tid + 256, ... in that order; four loads are
  // issued before they are merged
  int i = threadIdx.x;
  for (; i + 3 * 256 < p.chi2_items; i += 4 * 256) {
    double2 v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = part[i + k * 256];
#pragma unroll
    for (int k = 0; k < 4; ++k) acc.merge(v[k].x, v[k].y);
  }
  for (; i < p.chi2_items; i += 256) {
    const double2 v = part[i];
    acc.merge(v.x, v.y);
  }
  const Comp r = block_reduce<256>(acc, scr);
  if (threadIdx.x == 0) p.chi2_out[set] = r.s + r.c;
}

constexpr int nat_for(int nbt) { return nbt >= 1024 ? 64 : nbt >= 256 ? 32 : 16; }

}  // namespace rime
