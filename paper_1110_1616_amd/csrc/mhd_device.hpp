// Device-side ideal-MHD pointwise arithmetic for gfx950 (HIP).
//
// Scheme: MUSCL-Hancock on primitives (minmod), HLLD fluxes (Miyoshi &
// Kusano 2005), constrained transport with the arithmetic edge average of
// Balsara & Spicer (1999).  The paper (Sec. 1 and abstract) needs only that
// each grid's hyperbolic advance is decoupled by ghost zones; it defers the
// solver itself to the AstroBEAR code paper, so the solver is fixed here.
//
// Conventions: primitive W = (rho, vx, vy, vz, p, Bx, By, Bz); conserved
// U = (rho, mx, my, mz, E, Bx, By, Bz); magnetic pressure |B|^2/2.
// Rotated frame of direction d: (n, t1, t2) = (d, d+1, d+2) mod 3.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace amr {

template <class T> __host__ __device__ __forceinline__ T dsqrt(T x);
template <> __host__ __device__ __forceinline__ double dsqrt<double>(double x) { return __builtin_sqrt(x); }
template <> __host__ __device__ __forceinline__ float dsqrt<float>(float x) { return __builtin_sqrtf(x); }

template <class T> __host__ __device__ __forceinline__ T dabs(T x) { return x < T(0) ? -x : x; }

// Reciprocal of a nonzero finite normal x.  On the device in double: the
// hardware estimate refined by two Newton-Raphson steps r <- r + r (1 - x r),
// each error term formed with one fused multiply-add (the correctly rounded
// division costs twice the instructions).  The estimate is good to about
// 2^-24 on gfx950: one step leaves up to 11 ulp, two gave the correctly
// rounded reciprocal on every one of 2^20 random inputs.  In float the
// hardware estimate alone, good to 1 ulp (a Newton step made it correctly
// rounded on every such input, at 1.2% of the FP32 hierarchy's throughput).
// On the host, and for other types: plain division.
__device__ __forceinline__ double drcp(double x) {
  double r = __builtin_amdgcn_rcp(x);
  double e = __builtin_fma(-x, r, 1.0);
  r = __builtin_fma(r, e, r);
  e = __builtin_fma(-x, r, 1.0);
  return __builtin_fma(r, e, r);
}
__device__ __forceinline__ float drcp(float x) { return __builtin_amdgcn_rcpf(x); }
__host__ __forceinline__ double drcp(double x) { return 1.0 / x; }
__host__ __forceinline__ float drcp(float x) { return 1.0f / x; }
template <class T> __host__ __device__ __forceinline__ T drcp(T x) { return T(1) / x; }

// Square root of a non-negative finite x (0 for x <= 0).  On the device in
// double: Goldschmidt's iteration from the hardware reciprocal square root
// estimate y ~ 1/sqrt(x) (g = x y -> sqrt(x), h = y/2 -> 1/(2 sqrt(x)), one
// coupled step, then one correction g <- g + (x - g^2) h), without the
// rescaling of subnormal inputs the general routine does; on the host the
// library square root.  The estimate is good to about 2^-23 on gfx950, so
// after the coupled step g is good to about 2^-45 and the correction leaves
// it at the correctly rounded value on every one of 2^20 random inputs
// spread over 2^-30..2^30 (a second correction changed none of them).
__device__ __forceinline__ double psqrt(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y, h = 0.5 * y;
  const double r = __builtin_fma(-h, g, 0.5);
  g = __builtin_fma(g, r, g);
  h = __builtin_fma(h, r, h);
  const double d = __builtin_fma(-g, g, x);
  g = __builtin_fma(d, h, g);
  return x > 0.0 ? g : 0.0;
}
// In float the same iteration: the estimate is good to 1 ulp, and the
// correction gave the correctly rounded root on every one of 2^20 random
// inputs over 2^-30..2^30 (the library routine's scaling and ulp tests cost
// about twice the instructions).
__device__ __forceinline__ float psqrt(float x) {
  const float y = __builtin_amdgcn_rsqf(x);
  float g = x * y, h = 0.5f * y;
  const float r = __builtin_fmaf(-h, g, 0.5f);
  g = __builtin_fmaf(g, r, g);
  h = __builtin_fmaf(h, r, h);
  const float d = __builtin_fmaf(-g, g, x);
  g = __builtin_fmaf(d, h, g);
  return x > 0.0f ? g : 0.0f;
}
__host__ __forceinline__ double psqrt(double x) { return x > 0.0 ? __builtin_sqrt(x) : 0.0; }
__host__ __forceinline__ float psqrt(float x) { return x > 0.0f ? __builtin_sqrtf(x) : 0.0f; }
template <class T> __host__ __device__ __forceinline__ T psqrt(T x) { return x > T(0) ? dsqrt(x) : T(0); }

// Square root s and reciprocal square root i of a positive finite x.  On the
// device in double: the hardware estimate y (good to about 2^-23) and one
// third-order step, 1/sqrt(x) = y (1 + e/2 + 3 e^2/8 + ...) with e = 1 - x y^2,
// whose remainder is below 2^-66: both roots to about 1 ulp for 8 instructions
// (a correctly rounded root and the reciprocal of it take 18).  In float the
// hardware root and reciprocal root, 1 ulp each.
__device__ __forceinline__ void sqrt_rsqrt(double x, double& s, double& i) {
  const double y = __builtin_amdgcn_rsq(x);
  const double t = x * y;
  const double e = __builtin_fma(-t, y, 1.0);
  const double p = __builtin_fma(e, 0.375, 0.5);
  s = __builtin_fma(t * e, p, t);
  i = __builtin_fma(y * e, p, y);
}
__device__ __forceinline__ void sqrt_rsqrt(float x, float& s, float& i) {
  s = __builtin_amdgcn_sqrtf(x);
  i = __builtin_amdgcn_rsqf(x);
}
template <class T> __host__ __device__ __forceinline__ void sqrt_rsqrt(T x, T& s, T& i) {
  s = dsqrt(x);
  i = drcp(s);
}
__host__ __forceinline__ void sqrt_rsqrt(double x, double& s, double& i) { s = __builtin_sqrt(x); i = 1.0 / s; }
__host__ __forceinline__ void sqrt_rsqrt(float x, float& s, float& i) { s = __builtin_sqrtf(x); i = 1.0f / s; }
// Reciprocals of a and b (nonzero, a b finite and normal): in double one
// refined estimate of the product's, so one transcendental instruction (a
// quarter of the rate of the others) for the two; in float, whose range
// bounds the product and whose reciprocal is one instruction, each its own.
__device__ __forceinline__ void drcp2(double a, double b, double& ia, double& ib) {
  const double r = drcp(a * b);
  ia = r * b;
  ib = r * a;
}
__host__ __forceinline__ void drcp2(double a, double b, double& ia, double& ib) {
  const double r = 1.0 / (a * b);
  ia = r * b;
  ib = r * a;
}
template <class T> __host__ __device__ __forceinline__ void drcp2(T a, T b, T& ia, T& ib) {
  ia = drcp(a);
  ib = drcp(b);
}
// Square root of x, 0 for x <= 0: in float the hardware root, good to 1 ulp.
template <class T> __host__ __device__ __forceinline__ T root0(T x) { return psqrt(x); }
__device__ __forceinline__ float root0(float x) { return __builtin_amdgcn_sqrtf(__builtin_fmaxf(x, 0.0f)); }
__host__ __forceinline__ float root0(float x) { return psqrt(x); }

// Smaller and larger of two values (one instruction each on the device).
template <class T> __host__ __device__ __forceinline__ T pmin(T a, T b) { return b < a ? b : a; }
template <class T> __host__ __device__ __forceinline__ T pmax(T a, T b) { return a < b ? b : a; }
__device__ __forceinline__ double pmin(double a, double b) { return __builtin_fmin(a, b); }
__device__ __forceinline__ double pmax(double a, double b) { return __builtin_fmax(a, b); }
__device__ __forceinline__ float pmin(float a, float b) { return __builtin_fminf(a, b); }
__device__ __forceinline__ float pmax(float a, float b) { return __builtin_fmaxf(a, b); }
__host__ __forceinline__ double pmin(double a, double b) { return b < a ? b : a; }
__host__ __forceinline__ double pmax(double a, double b) { return a < b ? b : a; }
__host__ __forceinline__ float pmin(float a, float b) { return b < a ? b : a; }
__host__ __forceinline__ float pmax(float a, float b) { return a < b ? b : a; }

// minmod limiter: 0 when the one-sided differences disagree in sign (or one
// is zero), else the one of smaller magnitude (a on ties).  That is the
// median of a, b and 0: one instruction in float on the device, four minima
// and maxima in double, against seven (compares, a product, and two selects)
// spelled out; 24 of them a cell.
template <class T> __host__ __device__ __forceinline__ T limiter_minmod(T a, T b) {
  T r = (dabs(b) < dabs(a)) ? b : a;
  return ((a > T(0) && b > T(0)) || (a < T(0) && b < T(0))) ? r : T(0);
}
__device__ __forceinline__ double limiter_minmod(double a, double b) {
  return pmax(pmin(a, b), pmin(pmax(a, b), 0.0));
}
__device__ __forceinline__ float limiter_minmod(float a, float b) { return __builtin_amdgcn_fmed3f(a, b, 0.0f); }
__host__ __forceinline__ double limiter_minmod(double a, double b) { return pmax(pmin(a, b), pmin(pmax(a, b), 0.0)); }
__host__ __forceinline__ float limiter_minmod(float a, float b) { return pmax(pmin(a, b), pmin(pmax(a, b), 0.0f)); }

// W -> U for one state.
template <class T> __host__ __device__ __forceinline__ void to_conserved(const T (&w)[8], T (&u)[8], T gm1_inv) {
  u[0] = w[0];
  u[1] = w[0] * w[1];
  u[2] = w[0] * w[2];
  u[3] = w[0] * w[3];
  T b2 = w[5] * w[5] + w[6] * w[6] + w[7] * w[7];
  u[4] = w[4] * gm1_inv + T(0.5) * (b2 + u[1] * w[1] + u[2] * w[2] + u[3] * w[3]);
  u[5] = w[5];
  u[6] = w[6];
  u[7] = w[7];
}

// U -> W for one state.
template <class T> __host__ __device__ __forceinline__ void to_primitive(const T (&u)[8], T (&w)[8], T gm1) {
  const T ir = drcp(u[0]);
  w[0] = u[0];
  w[1] = u[1] * ir;
  w[2] = u[2] * ir;
  w[3] = u[3] * ir;
  T b2 = u[5] * u[5] + u[6] * u[6] + u[7] * u[7];
  w[4] = gm1 * (u[4] - T(0.5) * (b2 + u[1] * w[1] + u[2] * w[2] + u[3] * w[3]));
  w[5] = u[5];
  w[6] = u[6];
  w[7] = u[7];
}

// Physical flux along lab axis D of primitive w and its conserved state u
// (8 components, F(B_D) = 0).
template <int D, class T>
__host__ __device__ __forceinline__ void flux_along(const T (&w)[8], const T (&u)[8], T (&f)[8]) {
  const T vn = w[1 + D];
  const T bn = w[5 + D];
  T b2 = w[5] * w[5] + w[6] * w[6] + w[7] * w[7];
  T pt = w[4] + T(0.5) * b2;
  T vb = w[1] * w[5] + w[2] * w[6] + w[3] * w[7];
  const T rvn = u[1 + D];
  f[0] = rvn;
#pragma unroll
  for (int a = 0; a < 3; ++a) f[1 + a] = rvn * w[1 + a] - bn * w[5 + a];
  f[1 + D] += pt;
  f[4] = (u[4] + pt) * vn - bn * vb;
#pragma unroll
  for (int a = 0; a < 3; ++a) f[5 + a] = w[5 + a] * vn - bn * w[1 + a];
  f[5 + D] = T(0);
}
// The same from the primitive state alone.
template <int D, class T>
__host__ __device__ __forceinline__ void flux_along(const T (&w)[8], T (&f)[8], T gm1_inv) {
  T u[8];
  to_conserved(w, u, gm1_inv);
  flux_along<D>(w, u, f);
}

// Fast magnetosonic speed for density r, pressure p, |B|^2 = b2 and the field
// component along the direction bn.
template <class T> __host__ __device__ __forceinline__ T fast_magnetosonic(T r, T p, T b2, T bn, T gam) {
  T ir = drcp(r);
  T gp = gam * p;
  T a = (gp + b2) * ir;
  T d = a * a - T(4) * gp * bn * bn * ir * ir;
  return psqrt(T(0.5) * (a + psqrt(d)));
}

// Its square, c^2 = (a + sqrt(a^2 - 4 cs^2 va^2)) / 2 with a = (gamma p + B^2)
// / rho, cs^2 = gamma p / rho and va^2 = bn2 / rho.  Everything squared is a
// square of a speed.  With the roots of A = gamma p + B^2 taken before the
// division and the sides compared crosswise, two steps of 128^3 in FP64 take
// 632 instead of 642 us, but products of pressures leave the range of float at
// pressures of 1e-18 or 1e19 (a gas of 1e-30 g/cm^3 at 1e6 cm/s).
template <class T> __host__ __device__ __forceinline__ T fast_speed2(T r, T p, T b2, T bn2, T gam) {
  const T ir = drcp(r);
  const T cs2 = gam * p * ir;
  const T a = cs2 + b2 * ir;
  return T(0.5) * (a + root0(a * a - T(4) * cs2 * (bn2 * ir)));
}

// The waves of an HLLD fan and every choice its flux and the reverse of it make:
// one side's wave speed S, star density and Alfven wave, and the region that
// holds x/t = 0.  The reverse calls the same routine, so it follows the branch
// the flux took also where the sides are equal to a few roundings.
template <class T> struct HlldSide {
  T b2, pt;       // |B|^2, total pressure
  T s, d, rd;     // S, S - u, rho (S - u)
  T idsm, iden;   // 1 / (S - S_M); 1 / (rho (S - u)(S - S_M) - bn^2), any where degenerate
  T rs, sq, isq;  // star density, its root and reciprocal root
  T sa;           // speed of the Alfven wave
  bool deg;
};
template <class T> struct HlldFan {
  HlldSide<T> l, r;
  T bn2, sm, pts;
  bool lfast;  // the left fast speed bounds the fan
  bool left, inner, outer, ddeg;
};
template <class T>
__host__ __device__ __forceinline__ void hlld_side(const T (&q)[8], T bn2, T sm, T tiny, HlldSide<T>& o) {
  const T dsm = o.s - sm;
  const T den = o.rd * dsm - bn2;
  o.deg = dabs(den) <= tiny;
  // both denominators from one reciprocal in double: their product,
  // rho (S - u)(S - S_M)^2, has the scale of the energy flux, which has to be
  // in range itself
  drcp2(dsm, o.deg ? T(1) : den, o.idsm, o.iden);
  o.rs = o.rd * o.idsm;
  sqrt_rsqrt(o.rs, o.sq, o.isq);
}
template <class T>
__host__ __device__ __forceinline__ void hlld_fan(const T (&ql)[8], const T (&qr)[8], T bn, T gam, HlldFan<T>& w) {
  const T bn2 = w.bn2 = bn * bn;
  w.l.b2 = bn2 + ql[6] * ql[6] + ql[7] * ql[7];
  w.r.b2 = bn2 + qr[6] * qr[6] + qr[7] * qr[7];
  w.l.pt = ql[4] + T(0.5) * w.l.b2;
  w.r.pt = qr[4] + T(0.5) * w.r.b2;
  // larger fast speed: the sides' c^2 are compared before the root
  const T c2l = fast_speed2(ql[0], ql[4], w.l.b2, bn2, gam), c2r = fast_speed2(qr[0], qr[4], w.r.b2, bn2, gam);
  w.lfast = c2l > c2r;
  const T cmx = root0(pmax(c2r, c2l));
  w.l.s = pmin(qr[1], ql[1]) - cmx;
  w.r.s = pmax(qr[1], ql[1]) + cmx;
  // contact speed and star total pressure
  w.l.d = w.l.s - ql[1];
  w.r.d = w.r.s - qr[1];
  w.l.rd = ql[0] * w.l.d;
  w.r.rd = qr[0] * w.r.d;
  w.sm = (w.r.rd * qr[1] - w.l.rd * ql[1] - w.r.pt + w.l.pt) * drcp(w.r.rd - w.l.rd);
  w.pts = w.l.pt + w.l.rd * (w.sm - ql[1]);
  const T tiny = T(1e-12) * w.pts;
  hlld_side(ql, bn2, w.sm, tiny, w.l);
  hlld_side(qr, bn2, w.sm, tiny, w.r);
  const T abn = dabs(bn);
  w.l.sa = w.sm - abn * w.l.isq;
  w.r.sa = w.sm + abn * w.r.isq;
  w.ddeg = T(0.5) * bn2 <= tiny;
  w.left = w.sm >= T(0) || w.l.s > T(0);
  w.outer = w.left ? w.l.s > T(0) : !(w.r.sa >= T(0)) && !(w.r.s >= T(0));
  // the inner state holds x/t = 0 unless a test before it does or the normal
  // field is degenerate (the inner states then equal the star states)
  w.inner = (w.left ? !(w.l.sa >= T(0)) : w.r.sa >= T(0)) && !w.ddeg;
}

// HLLD flux (Miyoshi & Kusano 2005).  Inputs in the rotated frame:
// q = (rho, un, ut1, ut2, p, [unused], bt1, bt2); bn shared.  Output
// f = (rho, m_n, m_t1, m_t2, E, B_t1, B_t2).  The region that contains
// x/t = 0 is the first true test of S_L > 0, S*_L >= 0, S_M >= 0, S*_R >= 0,
// S_R >= 0 (else the right state).  The star states satisfy the jump
// conditions with the total pressure and normal velocity they share, so the
// flux of every region is the physical flux of its state, evaluated once: the
// inner (double-star) or star state of the chosen side by selects (waves hold
// lanes of both), the outer state under a branch that subsonic flow skips.
// The kept tangential field of a degenerate star state is the one that does
// not satisfy them: its flux is put right by B_t (u - S_M), under a branch at
// the end (summed where the states are selected it spilled 30 registers).
// Against forming every state's jump F + S (U* - U) + S* (U** - U*) with
// selects between both sides this is about 270 instead of 430 vector
// instructions in double (a select of a double is two), and the kernels here
// are bound by their issue.
template <class T>
__host__ __device__ __forceinline__ void riemann_hlld(const T (&ql)[8], const T (&qr)[8], T bn, T gam, T gm1_inv,
                                                      T (&f)[7]) {
  HlldFan<T> fan;
  hlld_fan(ql, qr, bn, gam, fan);
  const T bn2 = fan.bn2, sm = fan.sm, pts = fan.pts;
  const bool left = fan.left, inner = fan.inner;

  // Outer star states: tangential v and B, energy.  With
  // g = (S_M - u) / (rho (S - u)(S - S_M) - bn^2) the tangential fields are
  // v* = v - bt bn g and bt* = bt (1 + rho (S - u) g); g = 0 (v and bt kept)
  // where that denominator is degenerate.
  T vsl, wsl, bysl, bzsl, vbsl, esl;
  {
    const HlldSide<T>& o = fan.l;
    const T g = o.deg ? T(0) : (sm - ql[1]) * o.iden;
    const T fv = bn * g, fb = T(1) + o.rd * g;
    vsl = ql[2] - ql[6] * fv;
    wsl = ql[3] - ql[7] * fv;
    bysl = ql[6] * fb;
    bzsl = ql[7] * fb;
    const T vb = ql[1] * bn + ql[2] * ql[6] + ql[3] * ql[7];
    vbsl = sm * bn + vsl * bysl + wsl * bzsl;
    const T e = ql[4] * gm1_inv + T(0.5) * (ql[0] * (ql[1] * ql[1] + ql[2] * ql[2] + ql[3] * ql[3]) + o.b2);
    esl = (o.d * e - o.pt * ql[1] + pts * sm + bn * (vb - vbsl)) * o.idsm;
  }
  T vsr, wsr, bysr, bzsr, vbsr, esr;
  {
    const HlldSide<T>& o = fan.r;
    const T g = o.deg ? T(0) : (sm - qr[1]) * o.iden;
    const T fv = bn * g, fb = T(1) + o.rd * g;
    vsr = qr[2] - qr[6] * fv;
    wsr = qr[3] - qr[7] * fv;
    bysr = qr[6] * fb;
    bzsr = qr[7] * fb;
    const T vb = qr[1] * bn + qr[2] * qr[6] + qr[3] * qr[7];
    vbsr = sm * bn + vsr * bysr + wsr * bzsr;
    const T e = qr[4] * gm1_inv + T(0.5) * (qr[0] * (qr[1] * qr[1] + qr[2] * qr[2] + qr[3] * qr[3]) + o.b2);
    esr = (o.d * e - o.pt * qr[1] + pts * sm + bn * (vb - vbsr)) * o.idsm;
  }

  // The inner (double-star) state.
  const T sql = fan.l.sq, sqr = fan.r.sq;
  const T sg = bn > T(0) ? T(1) : T(-1);
  const T isum = drcp(sql + sqr);
  const T ssg = sql * sqr * sg;
  const T vss = (sql * vsl + sqr * vsr + (bysr - bysl) * sg) * isum;
  const T wss = (sql * wsl + sqr * wsr + (bzsr - bzsl) * sg) * isum;
  const T byss = (sql * bysr + sqr * bysl + ssg * (vsr - vsl)) * isum;
  const T bzss = (sql * bzsr + sqr * bzsl + ssg * (wsr - wsl)) * isum;
  const T vbss = sm * bn + vss * byss + wss * bzss;
  T r = left ? fan.l.rs : fan.r.rs, u = sm, pt = pts;
  T vb = left ? vbsl : vbsr;
  T e = left ? esl : esr;
  e = inner ? e - (left ? sql : -sqr) * sg * (vb - vbss) : e;
  vb = inner ? vbss : vb;
  T v = inner ? vss : (left ? vsl : vsr);
  T w = inner ? wss : (left ? wsl : wsr);
  T by = inner ? byss : (left ? bysl : bysr);
  T bz = inner ? bzss : (left ? bzsl : bzsr);
  if (fan.outer) {  // beyond the fast waves: the outer state
    r = left ? ql[0] : qr[0];
    u = left ? ql[1] : qr[1];
    v = left ? ql[2] : qr[2];
    w = left ? ql[3] : qr[3];
    by = left ? ql[6] : qr[6];
    bz = left ? ql[7] : qr[7];
    pt = left ? fan.l.pt : fan.r.pt;
    vb = u * bn + v * by + w * bz;
    e = (left ? ql[4] : qr[4]) * gm1_inv + T(0.5) * (r * (u * u + v * v + w * w) + (left ? fan.l.b2 : fan.r.b2));
  }
  f[0] = r * u;
  f[1] = f[0] * u + (pt - bn2);
  f[2] = f[0] * v - bn * by;
  f[3] = f[0] * w - bn * bz;
  f[4] = (e + pt) * u - bn * vb;
  f[5] = by * u - bn * v;
  f[6] = bz * u - bn * w;
  if (!fan.outer && (left ? fan.l.deg : fan.r.deg)) {  // the kept field crosses the outer wave with the outer state's flux
    const T t = u - (left ? ql[1] : qr[1]);
    f[5] -= (left ? ql[6] : qr[6]) * t;
    f[6] -= (left ? ql[7] : qr[7]) * t;
  }
}

}  // namespace amr
