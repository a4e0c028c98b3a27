// integrands.hpp -- per-event integrands f(x) on [0,1]^D for the gfx950 kernels.
//
// The paper evaluates a phase-space point and a matrix element times parton
// densities per event (Sec. 2.1); it prints neither.  The readings implemented
// here: Breit-Wigner mapping of resonant masses, the (tau, ln x1) mapping of the
// parton fractions, massless two-body decays with Lorentz boosts, chiral
// couplings, parametric PDFs A x^a (1-x)^b, and 3n-4 phase-space dimensions
// for n final-state particles (Sec. 3.2).  Every configuration-wide constant
// (couplings, mapping ranges) is computed once on the host into PhysConst and
// reaches the kernel as a by-value argument (constant/scalar memory).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "device_common.hpp"

namespace vg {

constexpr double kPi = 3.14159265358979323846;

struct PhysConst {
  int process, ndim, nbins, family;
  double conv;                // (hbar c)^2 in pb GeV^2
  // Breit-Wigner mapping of the first resonance: m^2 = M2 + MG tan(rho_lo + x rho_rng)
  double M2, MG, invMG, rho_lo, rho_rng, m2lo, tlo;
  // uniform products formed once on the host (the same roundings as in the kernels'
  // expressions), so that no per-thread copy of them takes vector registers: MG^2,
  // MG (1 + tlo^2), (MZ GZ)^2
  double MG2, MGt, mzgz2;
  // the constant factors of an event's weight, in one: conversion, flux, phase space,
  // couplings and the Breit-Wigner maps' ranges
  double wk = 1.0;
  double invS;                // 1 / S (hadronic)
  double pdfA, pdfa, pdfb;
  int pdf_pow;                // 1: a = a2/2 with integer a2 in [-8, 8] and integer b in [0, 16]
  int pdf_a2, pdf_b;
  // Drell-Yan
  double e4_12;               // e^4 / 12
  double dyA, dyB, dyC;       // sums over q, h, h' of (Q_q Q_l)^2, 2 Q_q Q_l g_q,h g_l,h', (g_q,h g_l,h')^2
  double mzgz, mz2;
  // W+
  double g4v2_24;             // g^4 |V|^2 / 24
  double ptmin2, th2;         // pT^2 cut, tanh(eta_max)^2
  // WW
  double rs, shat, gs;        // sqrt(shat), shat, g / sqrt(2)
  double i2rs = 1.0;          // 1 / (2 sqrt(shat))
  double cs_re[2][2], cs_im[2][2];  // s-channel photon+Z coefficient, [q][h]
  double ct;                  // exchange-diagram coefficient: -g^2 / 2
  double csR2;                // |Cs[u][R]|^2 + |Cs[d][R]|^2
  // hadronic WW: ln tau = Lhi + x8 * Lrng on [ln tau_lo, ln tau_hi] (Lrng = Llo - Lhi),
  // shat = tau S; per event the s-channel coefficients e^2 Q / shat + e^2 f (shat - MZ^2
  // - i MZ GZ) / |shat - MZ^2 + i MZ GZ|^2 from csq[q] = e^2 Q and csf[q][h] = e^2 f
  double S, Lhi, Lrng, Ldiff; // Ldiff = Lhi - Llo
  double csq[2], csf[2][2];
  // e+e- -> mu+mu-
  double s_ee, e4;
  // Gaussian test integrand
  double mu, inv2s2, gnorm;   // exp(-(x-mu)^2 inv2s2) * gnorm per dimension
  // Genz families
  double ga[16], gw[16];
};

// a polynomial coefficient materialised in a scalar register pair where it is used: an
// FMA then takes it as its SGPR operand, instead of a copy of a loop-invariant vector
// register into the accumulating FMA's destination before each step
__device__ __forceinline__ double poly_coef(double c) {
  VG_OPAQUE_SGPR(c);
  return c;
}

// ---------------------------------------------------------------------------
// atan(v) by the method of Moshier's Cephes library (atan.c): fold |v| to
// |x| <= 0.66 with atan(|v|) = pi/2 + atan(-1/|v|) above tan(3 pi/8) and
// pi/4 + atan((|v| - 1)/(|v| + 1)) above 0.66, then atan(x) = x + x z P(z)/Q(z),
// z = x^2, with its degree-4 / 5 rational fit; the low part of pi/2 (resp. half of
// it) is added last.  Branch-free here: the fold is one division (n / d with d = 1 on
// the low range), and P/Q the second; the coefficients are scalar-register operands.
// Relative error about 2 units in the last place (checked on the CPU against atanl).
// ---------------------------------------------------------------------------
__device__ __forceinline__ double atan_rr(double v) {
  VG_PRICED(atan, v);
  constexpr double kT3p8 = 2.41421356237309504880, kPio2 = 1.57079632679489661923,
                   kPio4 = 0.78539816339744830962, kMoreBits = 6.123233995736765886130e-17;
  const double a = fabs(v);
  const bool hi = a > kT3p8, mid = !hi && a > 0.66;
  const double x = div_nr(hi ? -1.0 : (mid ? a - 1.0 : a), hi ? a : (mid ? a + 1.0 : 1.0));
  const double z = x * x;
  double p = poly_coef(-8.750608600031904122785e-1);
  p = __fma_rn(p, z, poly_coef(-1.615753718733365076637e1));
  p = __fma_rn(p, z, poly_coef(-7.500855792314704667340e1));
  p = __fma_rn(p, z, poly_coef(-1.228866684490136173410e2));
  p = __fma_rn(p, z, poly_coef(-6.485021904942025371773e1));
  double q = z + poly_coef(2.485846490142306297962e1);
  q = __fma_rn(q, z, poly_coef(1.650270098316988542046e2));
  q = __fma_rn(q, z, poly_coef(4.328810604912902668951e2));
  q = __fma_rn(q, z, poly_coef(4.853903996359136964868e2));
  q = __fma_rn(q, z, poly_coef(1.945506571482613964425e2));
  const double r = __fma_rn(x, z * div_nr(p, q), x);
  const double y = hi ? kPio2 + (r + kMoreBits) : (mid ? kPio4 + (r + 0.5 * kMoreBits) : r);
  return copysign(y, v);
}

// ---------------------------------------------------------------------------
// tan(x) for |x| < pi/2 (the Breit-Wigner map's arguments): |x| > pi/4 is folded to
// y = pi/2 - |x| (pi/2 as the sum of two binary64 numbers; the first difference is
// exact, both being within a factor 2), and tan y = y + y z P(z)/Q(z), z = y^2, with the
// degree-2 / 4 rational fit of Moshier's Cephes library (tan.c) on |y| <= pi/4, taken
// here as N/Q with N = y (Q + z P): one division gives tan y = N/Q or cot y = Q/N.  A
// few units in the last place (checked on the CPU against tanl).
// ---------------------------------------------------------------------------
// sin y and cos y for |y| <= pi/4 by the minimax polynomials of the fdlibm / FreeBSD msun
// kernels (k_sin.c, k_cos.c; Sun Microsystems), by Horner's rule: sin y = y + y z S(z),
// z = y^2, and cos y = 1 + z (z C(z) - 1/2).  About one unit in the last place (checked on
// the CPU against sinl and cosl).
__device__ __forceinline__ void sincos_pio4(double y, double& sn, double& cs) {
  const double z = y * y;
  double s = __fma_rn(z, poly_coef(1.58969099521155010221e-10), poly_coef(-2.50507602534068634195e-08));
  s = __fma_rn(z, s, poly_coef(2.75573137070700676789e-06));
  s = __fma_rn(z, s, poly_coef(-1.98412698298579493134e-04));
  s = __fma_rn(z, s, poly_coef(8.33333333332248946124e-03));
  s = __fma_rn(z, s, poly_coef(-1.66666666666666324348e-01));
  sn = __fma_rn(z * y, s, y);
  double c = __fma_rn(z, poly_coef(-1.13596475577881948265e-11), poly_coef(2.08757232129817482790e-09));
  c = __fma_rn(z, c, poly_coef(-2.75573143513906633035e-07));
  c = __fma_rn(z, c, poly_coef(2.48015872894767294178e-05));
  c = __fma_rn(z, c, poly_coef(-1.38888888888741095749e-03));
  c = __fma_rn(z, c, poly_coef(4.16666666666666019037e-02));
  cs = __fma_rn(z, __fma_rn(z, c, -0.5), 1.0);
}

// tan y = nm / q on |y| <= pi/4 (the rational fit above)
__device__ __forceinline__ void tan_nq(double y, double& nm, double& q) {
  const double z = y * y;
  double p = poly_coef(-1.30936939181383777646e4);
  p = __fma_rn(p, z, poly_coef(1.15351664838587416140e6));
  p = __fma_rn(p, z, poly_coef(-1.79565251976484877988e7));
  q = z + poly_coef(1.36812963470692954678e4);
  q = __fma_rn(q, z, poly_coef(-1.32089234440210967447e6));
  q = __fma_rn(q, z, poly_coef(2.50083801823357915839e7));
  q = __fma_rn(q, z, poly_coef(-5.38695755929454629881e7));
  nm = y * __fma_rn(z, p, q);
}

// tan x = n / d for 0 <= x < pi/2, the division left to the caller
__device__ __forceinline__ void tan_halfpi_nd(double x, double& n, double& d) {
  constexpr double kPio4 = 0.78539816339744830962, kPio2Hi = 1.5707963267948966,
                   kPio2Lo = 6.123233995736766e-17;
  const bool big = x > kPio4;
  const double y = big ? (kPio2Hi - x) + kPio2Lo : x;
  double nm, q;
  tan_nq(y, nm, q);
  n = big ? q : nm;
  d = big ? nm : q;
}

__device__ __forceinline__ double tan_halfpi(double x) {
  VG_PRICED(tan, x);
  double n, d;
  tan_halfpi_nd(fabs(x), n, d);
  return copysign(div_nr(n, d), x);
}

// ---------------------------------------------------------------------------
// log, exp and expm1 for the parton fractions, without the libraries' extended precision
// and special cases: about one unit in the last place (checked on the CPU against logl and
// expm1l).  31, 16 and 20 vector instructions where the library's take 98, 42 and 53; the
// W+ and Drell-Yan integrands call log once and expm1 twice, the hadronic W+W- one exp once
// and expm1 twice.  Polynomials: interpolations at Chebyshev nodes, computed in 60 digits.
// ---------------------------------------------------------------------------
constexpr double kLn2 = 0.6931471805599453, kLn2Lo = 2.3190468138462996e-17;

// log x for normal x > 0: x = 2^k m with m in [sqrt(1/2), sqrt(2)), f = m - 1,
// s = f / (m + 1), z = s^2: log m = 2 atanh(s) = f - s (f - z G(z)) with
// G = 2 (1/3 + z/5 + ...) by a degree-6 polynomial (9.4e-18 of s)
__device__ __forceinline__ double log_pos(double x) {
  VG_PRICED(log, x);
  constexpr uint32_t kSqrtHalf = 0x3fe6a09e;  // high word of sqrt(1/2)
  uint64_t b;
  __builtin_memcpy(&b, &x, sizeof(b));
  const uint32_t h = static_cast<uint32_t>(b >> 32) + (0x3ff00000u - kSqrtHalf);
  const int k = static_cast<int>(h >> 20) - 1023;
  const double m = __hiloint2double(static_cast<int>((h & 0xfffffu) + kSqrtHalf), static_cast<int>(b));
  const double f = m - 1.0, s = f * rcp_nr(m + 1.0), z = s * s;
  double g = __fma_rn(z, poly_coef(0.146171283998073), poly_coef(0.15331666676597175));
  g = __fma_rn(z, g, poly_coef(0.1818289077802613));
  g = __fma_rn(z, g, poly_coef(0.22222211112104948));
  g = __fma_rn(z, g, poly_coef(0.2857142862611452));
  g = __fma_rn(z, g, poly_coef(0.399999999998992));
  g = __fma_rn(z, g, poly_coef(0.666666666666667));
  const double dk = static_cast<double>(k);
  const double u = __fma_rn(s, __fma_rn(-z, g, f), dk * -kLn2Lo);
  return __fma_rn(dk, kLn2, f - u);
}

// t = k ln 2 + r with |r| <= ln(2)/2; exp(r) - 1 = r + r^2 q(r), q of degree 9 (1.6e-17 of exp r)
constexpr double kExpQ[10] = {0.5000000000000001,     0.16666666666666669,    0.04166666666662413,    0.008333333333330062,
                              0.0013888888917213717,  0.00019841269863053618, 2.4801521295954376e-05, 2.7557268459997064e-06,
                              2.7620088445409746e-07, 2.510038549551032e-08};
__device__ __forceinline__ double exp_fold(double t, int& k, double& r) {
  constexpr double kRound = 0x1.8p52;  // a sum with it is rounded to an integer, its last bits
  const double kr = __fma_rn(t, 1.4426950408889634, kRound);
  uint64_t b;
  __builtin_memcpy(&b, &kr, sizeof(b));
  k = static_cast<int>(static_cast<uint32_t>(b));
  const double dk = kr - kRound;
  r = __fma_rn(-dk, kLn2Lo, __fma_rn(-dk, kLn2, t));
  double q = __fma_rn(r, poly_coef(kExpQ[9]), poly_coef(kExpQ[8]));
  q = __fma_rn(q, r, poly_coef(kExpQ[7]));
  q = __fma_rn(q, r, poly_coef(kExpQ[6]));
  q = __fma_rn(q, r, poly_coef(kExpQ[5]));
  q = __fma_rn(q, r, poly_coef(kExpQ[4]));
  q = __fma_rn(q, r, poly_coef(kExpQ[3]));
  q = __fma_rn(q, r, poly_coef(kExpQ[2]));
  q = __fma_rn(q, r, poly_coef(kExpQ[1]));
  return __fma_rn(q, r, poly_coef(kExpQ[0]));
}

// exp t and exp t - 1 for |t| < 1e9 (0 and inf, or -1 and inf, where they leave the range)
__device__ __forceinline__ double exp_fin(double t) {
  VG_PRICED(exp, t);
  int k;
  double r;
  const double q = exp_fold(t, k, r);
  return ldexp(__fma_rn(r * r, q, r) + 1.0, k);
}
__device__ __forceinline__ double expm1_fin(double t) {
  VG_PRICED(expm1, t);
  int k;
  double r;
  const double q = exp_fold(t, k, r), s = ldexp(double(1.0), k);
  return __fma_rn(s * r * r, q, __fma_rn(s, r, s - 1.0));  // 2^k - 1 + 2^k (r + r^2 q)
}

// ---------------------------------------------------------------------------
// mappings (rounding kept as in their plain definitions: no contraction)
// ---------------------------------------------------------------------------
// m^2 = M^2 + M G tan(rho_lo + r rrng) on the process's window (lower edge m2lo,
// rho_lo = atan(tlo)); its Jacobian is dm^2/dr = rrng ((m^2 - M^2)^2 + (M G)^2) / (M G), whose
// resonance factor the integrands cancel against the propagator's
template <bool TWO_DIV = false>
__device__ __forceinline__ double bw_mass(const PhysConst& c, double r, double rrng) {
#pragma clang fp contract(off)
  const double rho = c.rho_lo + r * rrng;
  // below the pole the mass is measured from the window's lower edge (tangent
  // addition theorem), free of the cancellation in M^2 + M G tan(rho) as m^2 -> m2lo;
  // one tangent per event either way (no divergent second call).  With the tangent as a
  // ratio t = n / d, t / (1 - tlo t) = n / (d - tlo n): one division for either form.
  // Both arguments lie in [0, pi/2).  TWO_DIV: the tangent rounded first (the binary32
  // amplitude's masses: an ulp here turns into another binary32 rounding there)
  const bool below = rho < 0.0;
  if constexpr (TWO_DIV) {
    const double t = tan_halfpi(below ? r * rrng : rho);
    return below ? c.m2lo + c.MGt * t * rcp_nr(1.0 - c.tlo * t) : c.M2 + c.MG * t;
  }
  double t;
  {
    VG_PRICED(tan, rho);
    double n, d;
    tan_halfpi_nd(below ? r * rrng : rho, n, d);
    t = div_nr(n, below ? __fma_rn(-c.tlo, n, d) : d);
  }
  return below ? __fma_rn(c.MGt, t, c.m2lo) : __fma_rn(c.MG, t, c.M2);
}

// ---------------------------------------------------------------------------
// product of the two parton densities, f(x1) f(x2) = A^2 tau^a ((1-x1)(1-x2))^b with
// tau = x1 x2, L = ln tau and P = (1-x1)(1-x2) (> 0).  For half-integer a and integer
// b (the usual parametrisations) the powers are products, square roots and one
// reciprocal; otherwise exp(a L + b ln P).
// ---------------------------------------------------------------------------
__device__ __forceinline__ double ipow_pos(double v, int k) {  // v^k, 0 <= k <= 16
  double r = 1.0;
  for (int i = 0; i < k; ++i) r *= v;
  return r;
}

__device__ __forceinline__ double pdf_pair(const PhysConst& c, double tau, double L, double P) {
  if (c.pdf_pow) {
    const int a2 = c.pdf_a2;
    const int ka = (a2 >= 0 ? a2 : -a2) >> 1;   // |a| rounded down
    double ta = ipow_pos(tau, ka);
    if (a2 < 0 && ka > 0) ta = rcp_nr(ta);
    if (a2 & 1) {
      double r, ir;
      sqrt_rsqrt_nr(tau, r, ir);
      ta *= a2 < 0 ? ir : r;
    }
    return c.pdfA * c.pdfA * ta * ipow_pos(P, c.pdf_b);
  }
  return c.pdfA * c.pdfA * exp(c.pdfa * L + c.pdfb * log(P));
}

// ---------------------------------------------------------------------------
// test integrands
// ---------------------------------------------------------------------------
template <int D>
__device__ __forceinline__ double f_gauss(const PhysConst& c, const double* x) {
  const int nd = D > 0 ? D : c.ndim;
  double s = 0.0, norm = 1.0;
#pragma unroll
  for (int d = 0; d < (D > 0 ? D : 16); ++d) {
    if (d >= nd) break;
    const double z = x[d] - c.mu;
    s += z * z;
    norm *= c.gnorm;
  }
  return norm * exp(-s * c.inv2s2);
}

template <int D>
__device__ __forceinline__ double f_genz(const PhysConst& c, const double* x) {
  const int nd = D > 0 ? D : c.ndim;
  double s = 0.0, f = 1.0;
  switch (c.family) {
    case 1:
      for (int d = 0; d < nd; ++d) s += c.ga[d] * x[d];
      return cos(2.0 * kPi * c.gw[0] + s);
    case 2:
      for (int d = 0; d < nd; ++d) {
        const double z = x[d] - c.gw[d];
        f *= 1.0 / (1.0 / (c.ga[d] * c.ga[d]) + z * z);
      }
      return f;
    case 3:
      for (int d = 0; d < nd; ++d) s += c.ga[d] * x[d];
      return pow(1.0 + s, -static_cast<double>(nd + 1));
    case 4:
      for (int d = 0; d < nd; ++d) {
        const double z = x[d] - c.gw[d];
        s += c.ga[d] * c.ga[d] * z * z;
      }
      return exp(-s);
    case 5:
      for (int d = 0; d < nd; ++d) s += c.ga[d] * fabs(x[d] - c.gw[d]);
      return exp(-s);
    case 6:
      if (x[0] > c.gw[0]) return 0.0;
      if (nd > 1 && x[1] > c.gw[1]) return 0.0;
      for (int d = 0; d < nd; ++d) s += c.ga[d] * x[d];
      return exp(s);
    default:
      return __builtin_nan("");
  }
}

// e+e- -> mu+mu-: <|M|^2> = e^4 (1 + c^2); flux 1/(2s), dPhi_2 = dOmega/(32 pi^2),
// solid-angle Jacobian 4 pi -> f = conv e^4 (1 + c^2) / (16 pi s)
__device__ __forceinline__ double f_eemumu(const PhysConst& c, const double* x) {
  const double cs = 2.0 * x[0] - 1.0;
  return c.conv * c.e4 * (1.0 + cs * cs) / (16.0 * kPi * c.s_ee);
}

// ---------------------------------------------------------------------------
// q qbar -> photon/Z -> l- l+ (both beam orderings).  With one PDF for all
// four flavours the two orderings sum to sum_{hh'} |A_hh'|^2 * 2 (1 + c^2).
// ---------------------------------------------------------------------------
// The map's Jacobian contains 1 / |shat - MZ^2 + i MZ GZ|^2's inverse, so with
// |Q Q'/shat + g g'/D|^2 summed over q, h, h' the weight needs no division by |D|^2:
// shat^2 |D|^2 sum = A |D|^2 + shat (B (shat - MZ^2) + C shat).
// obs_sq: the square of the observable, the lepton-pair mass m_ll^2
__device__ __forceinline__ double f_dy(const PhysConst& c, const double* x, double& obs_sq) {
  const double m2 = bw_mass(c, x[0], c.rho_rng);
  obs_sq = m2;
  const double tau = m2 * c.invS;
  double L, l1, l2;
  {
#pragma clang fp contract(off)
    L = log_pos(tau);
    l1 = x[1] * L;
    l2 = L - l1;
  }
  // f(x1) f(x2) with tau = x1 x2 = m2 / S and 1 - x = -expm1(ln x)
  const double ff = pdf_pair(c, tau, L, expm1_fin(l1) * expm1_fin(l2));
  const double cs = 2.0 * x[2] - 1.0;
  const double ds = m2 - c.mz2;
  const double me = __fma_rn(c.dyA, __fma_rn(ds, ds, c.mzgz2), m2 * __fma_rn(c.dyB, ds, c.dyC * m2));
  // conv * J_bw * J_tau * J_cos(2) * flux 1/(2 shat) * 2 pi / (32 pi^2)
  return (c.wk * me) * (-L * rcp_nr(m2)) * __fma_rn(cs, cs, 1.0) * ff;
}

// ---------------------------------------------------------------------------
// u dbar -> W+ -> e+ nu (both orderings) with e+ cuts pT > ptmin, |eta| < etamax.
// Orderings sum to g^4 |V|^2 shat^2 (1 + c^2) / (24 |D|^2); the cuts use the
// boost-invariant pT^2 = (shat/4)(1 - c^2) and the lab polar cosine
// (c + beta)/(1 + beta c), beta = (x1 - x2)/(x1 + x2).
// ---------------------------------------------------------------------------
// obs_sq: the square of the observable, the e+ transverse momentum (taken before the cuts)
__device__ __forceinline__ double f_w(const PhysConst& c, const double* x, double& obs_sq) {
  const double m2 = bw_mass(c, x[0], c.rho_rng);
  const double tau = m2 * c.invS;
  double L, l1, l2;
  {
#pragma clang fp contract(off)
    L = log_pos(tau);
    l1 = x[1] * L;
    l2 = L - l1;
  }
  const double cs = 2.0 * x[2] - 1.0;
  // x = 1 + expm1(ln x): beta = (x1 - x2)/(x1 + x2) and 1 - x from the same two values
  const double em1 = expm1_fin(l1), em2 = expm1_fin(l2);
  const double pt2 = 0.25 * m2 * (1.0 - cs) * (1.0 + cs);
  obs_sq = pt2;
  const double beta = div_nr(em1 - em2, 2.0 + em1 + em2);
  const double num = cs + beta, dnm = 1.0 + beta * cs;
  const bool pass = (pt2 > c.ptmin2) && (num * num < c.th2 * dnm * dnm);
  if (!pass) return 0.0;
  // |M|^2 / (2 shat) = g^4 |V|^2 / 24 * shat^2 (1 + cos^2) / |D|^2 / (2 shat), and the map's
  // Jacobian has the same |D|^2 = (shat - MW^2)^2 + (MW GW)^2 above the line
  const double ff = pdf_pair(c, tau, L, em1 * em2);
  // conv * J_bw * J_tau * |M|^2 / (2 shat) * (2 * 2 pi)/(32 pi^2)
  return (c.wk * tau) * -L * __fma_rn(cs, cs, 1.0) * ff;
}

// ---------------------------------------------------------------------------
// q qbar -> W+ W- -> e+ nu mu- nubar: helicity amplitudes in two-component
// (Weyl) form.  Quarks along +-z; lepton helicities fixed by V-A; the quark-pair
// currents are then j_L = rs (0, 1, -i, 0) and j_R = rs (0, 1, i, 0).  Two
// evaluations of the same amplitudes: in binary64 from products of the lepton spinors
// (ww_spinor_me2), in binary32 from the currents and the three-boson vertex
// (ww_me2; its roundings are what that option's results are made of, so it stays).
// ---------------------------------------------------------------------------
template <typename R>
struct cx {
  R re, im;
};
template <typename R>
__device__ __forceinline__ cx<R> cadd(cx<R> a, cx<R> b) { return {a.re + b.re, a.im + b.im}; }
template <typename R>
__device__ __forceinline__ cx<R> csub(cx<R> a, cx<R> b) { return {a.re - b.re, a.im - b.im}; }
template <typename R>
__device__ __forceinline__ cx<R> cmul(cx<R> a, cx<R> b) {
  return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
template <typename R>
__device__ __forceinline__ cx<R> cscale(cx<R> a, R s) { return {a.re * s, a.im * s}; }
template <typename R>
__device__ __forceinline__ cx<R> cconjmul(cx<R> a, cx<R> b) {  // conj(a) * b
  return {a.re * b.re + a.im * b.im, a.re * b.im - a.im * b.re};
}
template <typename R>
__device__ __forceinline__ R cabs2(cx<R> a) { return a.re * a.re + a.im * a.im; }

// helicity-minus massless 2-spinor (left-chiral), phase chosen per hemisphere: with
// r = sqrt(p0 + |p3|), (-(p1 - i p2) / r, r) for p3 >= 0 and (-r, (p1 + i p2) / r) below
// (the two differ by a phase, so |M|^2 does not depend on the choice; dividing by the
// larger of p0 +- p3 avoids the cancellation).  One square root and its reciprocal from
// the same estimate, and selects instead of branches (a wave holds both hemispheres).
template <typename R>
__device__ __forceinline__ void spinor_m(const R p[4], cx<R>& s0, cx<R>& s1) {
  const bool up = p[3] >= R(0);
  R r, ir;
  sqrt_rsqrt_nr(p[0] + fabs(p[3]), r, ir);
  const R a = p[1] * ir, b = p[2] * ir;
  s0 = {up ? -a : -r, up ? b : R(0)};
  s1 = {up ? r : a, up ? R(0) : b};
}

// J^mu = a^dagger sigma-bar^mu b (contravariant components)
template <typename R>
__device__ __forceinline__ void current(cx<R> a0, cx<R> a1, cx<R> b0, cx<R> b1, cx<R> J[4]) {
  const cx<R> t00 = cconjmul(a0, b0), t11 = cconjmul(a1, b1);
  const cx<R> t01 = cconjmul(a0, b1), t10 = cconjmul(a1, b0);
  J[0] = cadd(t00, t11);
  J[1] = {-(t01.re + t10.re), -(t01.im + t10.im)};
  const cx<R> d = csub(t01, t10);
  J[2] = {-d.im, d.re};  // i * d
  J[3] = csub(t11, t00);
}

template <typename R>
__device__ __forceinline__ cx<R> mdot(const cx<R> a[4], const cx<R> b[4]) {
  cx<R> s = cmul(a[0], b[0]);
  s = csub(s, cmul(a[1], b[1]));
  s = csub(s, cmul(a[2], b[2]));
  return csub(s, cmul(a[3], b[3]));
}

template <typename R>
__device__ __forceinline__ cx<R> mdot_r(const R a[4], const cx<R> b[4]) {
  return {a[0] * b[0].re - a[1] * b[1].re - a[2] * b[2].re - a[3] * b[3].re,
          a[0] * b[0].im - a[1] * b[1].im - a[2] * b[2].im - a[3] * b[3].im};
}

// [ (sigma-bar.e2)(sigma.k)(sigma-bar.e1) ]_{01}; sigma-bar.e = e^0 + sigma.e,
// sigma.k = k^0 - sigma.k (k real)
template <typename R>
__device__ __forceinline__ cx<R> chain01(const cx<R> e2[4], const R k[4], R B00, R B11, const cx<R> e1[4]) {
  const cx<R> A00 = cadd(e2[0], e2[3]);
  const cx<R> A01 = {e2[1].re + e2[2].im, e2[1].im - e2[2].re};  // e2^1 - i e2^2
  const cx<R> C01 = {e1[1].re + e1[2].im, e1[1].im - e1[2].re};  // e1^1 - i e1^2
  const cx<R> C11 = csub(e1[0], e1[3]);
  const cx<R> B01 = {-k[1], k[2]};   // -(k1 - i k2)
  const cx<R> B10 = {-k[1], -k[2]};  // -(k1 + i k2)
  const cx<R> y0 = cadd(cscale(C01, B00), cmul(B01, C11));
  const cx<R> y1 = cadd(cmul(B10, C01), cscale(C11, B11));
  return cadd(cmul(A00, y0), cmul(A01, y1));
}

// exchange-propagator invariants: t = k^2 and k^0 -+ k^3 for k = p1 - q(W+) (u quark)
// and k = p1 - q(W-) (d quark), formed in binary64 from the mapped masses
template <typename R>
struct ExchInv {
  R tu, td, b00u, b11u, b00d, b11d;
};

// the lepton current of one W decay, J = a^dagger sigma-bar b with a, b the
// helicity-minus spinors of pa, pb (formed as soon as the decay momenta are, so that
// only the current stays live)
template <typename R>
__device__ __forceinline__ void lepton_current(const double pa[4], const double pb[4], cx<R> J[4]) {
  R a[4], b[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    a[i] = static_cast<R>(pa[i]);
    b[i] = static_cast<R>(pb[i]);
  }
  cx<R> a0, a1, b0, b1;
  spinor_m(a, a0, a1);
  spinor_m(b, b0, b1);
  current(a0, a1, b0, b1, J);
}

// sum over q in {u, d} and quark helicity of |M|^2 (no averages) WITHOUT the two W
// propagators and couplings g/sqrt2 / (m^2 - MW^2 + i MW GW): every diagram is linear
// in each W's polarisation current, so they factor out of every amplitude as one complex
// number, and |.|^2 of it, g^4/4 / ((m+^2 - MW^2)^2 + (MW GW)^2) / ((m-^2 - MW^2)^2 +
// (MW GW)^2), cancels against the Breit-Wigner maps' Jacobians (the caller multiplies
// the remainder, (g^2/2)^2 / (MW GW)^2 times the maps' ranges, into the weight).  From the
// lepton currents Jp = ubar(nu) gamma P_L v(e+), Jm = ubar(mu-) gamma P_L v(nubar) (the
// polarisations ep, em up to those factors) and the W momenta qp, qm
template <typename R>
__device__ __forceinline__ R ww_me2(const PhysConst& c, const cx<R> ep[4], const cx<R> em[4], const R qp[4],
                                    const R qm[4], const ExchInv<R>& inv) {
  R Ppq[4], Pmq[4], dq[4];
#pragma unroll
  for (int mu = 0; mu < 4; ++mu) {
    const R PP = qp[mu] + qm[mu];
    Ppq[mu] = PP + qp[mu];
    Pmq[mu] = PP + qm[mu];
    dq[mu] = qm[mu] - qp[mu];
  }
  // triple-gauge vertex contracted with ep, em
  const cx<R> a1 = mdot_r(Ppq, em), a2 = mdot(ep, em), a3 = mdot_r(Pmq, ep);
  cx<R> V1, V2;
  V1 = csub(cadd(cmul(ep[1], a1), cscale(a2, dq[1])), cmul(em[1], a3));
  V2 = csub(cadd(cmul(ep[2], a1), cscale(a2, dq[2])), cmul(em[2], a3));
  const R rs = static_cast<R>(c.rs);
  // j_L.V = -rs (V1 - i V2), j_R.V = -rs (V1 + i V2)
  const cx<R> AL = {-rs * (V1.re + V2.im), -rs * (V1.im - V2.re)};
  const cx<R> AR = {-rs * (V1.re - V2.im), -rs * (V1.im + V2.re)};
  // exchange diagrams: u quark emits W+ first (k = p1 - qp), d quark emits W- first (k = p1 - qm);
  // p1 = (rs/2, 0, 0, rs/2); vbar(p2) ... u(p1) picks -rs * [..]_{01}
  const R half = rs * R(0.5);
  R ku[4] = {half - qp[0], -qp[1], -qp[2], half - qp[3]};
  R kd[4] = {half - qm[0], -qm[1], -qm[2], half - qm[3]};
  const R tu = inv.tu, td = inv.td, b00u = inv.b00u, b11u = inv.b11u, b00d = inv.b00d, b11d = inv.b11d;
  const cx<R> Tu = chain01(em, ku, b00u, b11u, ep);
  const cx<R> Td = chain01(ep, kd, b00d, b11d, em);
  const R ct = static_cast<R>(c.ct);
  const R rsct = -rs * ct;
  const R fu = rsct * rcp_nr(tu), fd = rsct * rcp_nr(td);
  // s-channel photon + Z, left-handed quark
  const cx<R> csuL = {static_cast<R>(c.cs_re[0][0]), static_cast<R>(c.cs_im[0][0])};
  const cx<R> csdL = {static_cast<R>(c.cs_re[1][0]), static_cast<R>(c.cs_im[1][0])};
  const cx<R> MuL = cadd(cmul(csuL, AL), cscale(Tu, fu));
  const cx<R> MdL = cadd(cmul(csdL, AL), cscale(Td, fd));
  return cabs2(MuL) + cabs2(MdL) + static_cast<R>(c.csR2) * cabs2(AR);
}

// ---------------------------------------------------------------------------
// the same sum over quark flavours and helicities in binary64, from the lepton spinors.
//
// A W decay's current J^mu = a^dagger sigma-bar^mu b contracts to a matrix of rank one,
// sigma-bar.J = 2 a~ b~^T with a~ = (a1*, -a0*), b~ = (b1, -b0), so an exchange diagram is
// a product of spinor components with the quarks' spinors along z: for the u quark
//   [sigma-bar.Jm sigma.k sigma-bar.Jp]_01 = -4 U,  U = l5_1* l3_0 K_u,
//   K_u = (l6_1, -l6_0) sigma.(p1 - qp) (l4_1*, -l4_0*)^T
// (3 e+, 4 nu, 5 mu-, 6 nubar), and D likewise for the d quark with the bosons exchanged.
// Contracted with the quark current, the three-boson vertex is the difference of the same
// two products, j_L.V = -4 rs (U - D), and for the right-handed quark j_R.V = -4 rs (U' - D')
// with the quark momenta exchanged: the gauge relation between the diagrams (the form in
// which Dixon, Kunszt and Signer, 1998, write these helicity amplitudes).
//
// Spinors: with the azimuths counted from the W+'s (a rotation of the whole event about
// the beam leaves |M|^2 as it is), the boost from a W's rest frame to (E, qx, 0, qz) takes a
// left-handed spinor by the real matrix (E + m - q.sigma) / sqrt(2 m (E + m)); a decay with
// cos(theta) = 2 x - 1 and azimuth phi has the rest spinors sqrt(m) (-s e^{-i phi}, x) / sqrt(x)
// and sqrt(m) (x, s e^{i phi}) / sqrt(x), s = sqrt(x (1 - x)).  Their scales leave every
// amplitude as the one factor 1 / (2 (E + m) x) per W, squared.
//
// Bound by the VALU's issue rate; against currents, boosted momenta, four spinor square
// roots and the vertex the event loop took about 870 instead of 1156 VALU instructions
// per 64 events and 137 instead of 157 registers: an iteration of 1e7 W+W- events 303 us
// instead of 378, of 3e6 hadronic ones 196 instead of 221.  (Since then the shorter
// divisions, roots and sines, and the weight's constant factors formed on the host, have
// taken it to 817 instructions, and with all other steps the W+W- iteration to 253 us.)
// ---------------------------------------------------------------------------
// light-cone components of the bosons (the W+ along qx, qz): W+ E -+ qz, W- E -+ qz (its
// momentum is -qx, -qz), each sum of positive terms or the quotient (m^2 + qx^2) over its
// partner, so forward bosons lose no digits; E+ + E- = rs turns every difference with rs
// that the diagrams contain into one of them
struct WWPoint {
  double qx, pm, pp, mm, mp;
};

// m0, m1 = mass + (E -+ qz), qx of the boson; x the decay's angular variable, z = s e^{i phi}:
// l = the spinor of the decay lepton along phi, n = the conjugate of its partner's
__device__ __forceinline__ void decay_spinors(double m0, double m1, double qx, double x, cx<double> z, cx<double> l[2],
                                              cx<double> n[2]) {
  const double ox = qx * x;
  const cx<double> a = {m0 * z.re, m0 * z.im}, b = {m1 * z.re, m1 * z.im};
  l[0] = {-a.re - ox, a.im};
  l[1] = {__fma_rn(qx, z.re, m1 * x), -qx * z.im};
  n[0] = {__fma_rn(-qx, z.re, m0 * x), qx * z.im};
  n[1] = {b.re - ox, -b.im};
}

__device__ __forceinline__ double ww_spinor_me2(const PhysConst& c, const WWPoint& w, const cx<double> l3[2],
                                                const cx<double> n4[2], const cx<double> n5[2], const cx<double> l6[2],
                                                const double cre[2], const double cim[2], double csR2, double ct_tu,
                                                double ct_td) {
  // pairwise products: the W+ neutrino with the antineutrino, the positron with the muon
  const cx<double> p11 = cmul(l6[1], n4[1]), p00 = cmul(l6[0], n4[0]);
  const cx<double> p10 = cmul(l6[1], n4[0]), p01 = cmul(l6[0], n4[1]);
  const cx<double> q11 = cmul(l3[1], n5[1]), q00 = cmul(l3[0], n5[0]);
  const cx<double> q10 = cmul(l3[1], n5[0]), q01 = cmul(l3[0], n5[1]);
  const cx<double> po = {w.qx * (p10.re + p01.re), w.qx * (p10.im + p01.im)};
  const cx<double> qo = {w.qx * (q10.re + q01.re), w.qx * (q10.im + q01.im)};
  const cx<double> ku = {w.mm * p00.re - w.pm * p11.re - po.re, w.mm * p00.im - w.pm * p11.im - po.im};
  const cx<double> kd = {w.pp * q00.re - w.mp * q11.re + qo.re, w.pp * q00.im - w.mp * q11.im + qo.im};
  const cx<double> kur = {w.mp * p11.re - w.pp * p00.re - po.re, w.mp * p11.im - w.pp * p00.im - po.im};
  const cx<double> kdr = {w.pm * q11.re - w.mm * q00.re + qo.re, w.pm * q11.im - w.mm * q00.im + qo.im};
  const cx<double> U = cmul(q01, ku), D = cmul(p01, kd);
  const cx<double> S = csub(U, D), SR = csub(cmul(q10, kur), cmul(p10, kdr));
  const cx<double> MuL = {cre[0] * S.re - cim[0] * S.im - ct_tu * U.re, cre[0] * S.im + cim[0] * S.re - ct_tu * U.im};
  const cx<double> MdL = {cre[1] * S.re - cim[1] * S.im - ct_td * D.re, cre[1] * S.im + cim[1] * S.re - ct_td * D.im};
  return cabs2(MuL) + cabs2(MdL) + csR2 * cabs2(SR);
}

// rest frame of Q (mass m, im = 1 / m) -> frame of Q, for k and its back-to-back partner
template <typename R>
__device__ __forceinline__ void boost_pair(const R Q[4], R m, R im, const R k[4], R a[4], R b[4]) {
  const R qk = Q[1] * k[1] + Q[2] * k[2] + Q[3] * k[3];
  const R iqm = rcp_nr(Q[0] + m);
  const R Ea = (Q[0] * k[0] + qk) * im;
  const R Eb = (Q[0] * k[0] - qk) * im;
  const R fa = (k[0] + Ea) * iqm, fb = (k[0] + Eb) * iqm;
  a[0] = Ea;
  b[0] = Eb;
#pragma unroll
  for (int i = 1; i < 4; ++i) {
    a[i] = k[i] + fa * Q[i];
    b[i] = -k[i] + fb * Q[i];
  }
}

// v with its sign changed where bit 31 of m is set
__device__ __forceinline__ double flip_sign(double v, uint32_t m) {
  uint64_t b;
  __builtin_memcpy(&b, &v, sizeof(b));
  b ^= static_cast<uint64_t>(m & 0x80000000u) << 32;
  __builtin_memcpy(&v, &b, sizeof(b));
  return v;
}

// sin and cos of 2 pi x for -1 <= x <= 1: x = q/4 + r with q = rint(4 x) and |r| <= 1/8
// (r exact: x and q/4 are within a factor 2 of each other when q is not 0), y = 2 pi r, then
// the rotation by q quarter turns.  q is rounded by adding 1.5 x 2^52, whose sum's last bits
// are q's: bit 0 exchanges sine and cosine, bit 1 of q and of q + 1 are their signs
__device__ __forceinline__ void sincos_2pi(double x, double& s, double& c) {
  VG_PRICED(sincos, x);
  constexpr double kRound = 0x1.8p52;
  const double t = __fma_rn(4.0, x, kRound);
  const double q = t - kRound;
  uint64_t bits;
  __builtin_memcpy(&bits, &t, sizeof(bits));
  const uint32_t qi = static_cast<uint32_t>(bits);
  const double y = __fma_rn(-0.25, q, x) * 6.283185307179586477;
  double sn, cs;
  sincos_pio4(y, sn, cs);
  const bool odd = qi & 1u;
  const double a = odd ? cs : sn, b = odd ? sn : cs;
  s = flip_sign(a, qi << 30);
  c = flip_sign(b, (qi + 1u) << 30);
}
__device__ __forceinline__ void sincos_2pi(float x, float& s, float& c) { sincospif(2.0f * x, &s, &c); }

// dPhi_2(P) (4 pi) = sl / (8 pi shat), dm+^2/(2 pi), dm-^2/(2 pi), [dPhi_2(W) (4 pi)]^2 =
// 1 / (64 pi^2), flux 1 / (2 shat), colour and spin average 1/12: one constant over shat^2;
// each Breit-Wigner Jacobian times its propagator's |g/sqrt2 / (m^2 - MW^2 + i MW GW)|^2
// is (g^2/2) / (MW GW) times the map's range
constexpr double kWWPS = 0.5 / (12.0 * 8.0 * kPi * 4.0 * kPi * kPi * 64.0 * kPi * kPi);

// WW_4L: x0 -> m+^2 (BW on [0, shat]), x1 -> m-^2 (BW on [0, (rs - m+)^2]),
// x2, x3 -> W+ direction, x4..x7 -> lepton directions in the W rest frames.
// obs_sq: the square of the observable, the e+ nu mass m_+^2 (0 where the map gives none)
// HAD: the hadronic integrand (10 dims): x8 -> ln tau, x9 -> ln x1, the partonic weight
// at shat = tau S times the luminosity 2 |dtau/dx8| (-ln tau) f(x1) f(x2) (the two beam
// orderings give the same integral)
template <bool HAD>
__device__ __forceinline__ double f_ww_double(const PhysConst& c, const double* x, double& obs_sq) {
  double rs = c.rs, sh = c.shat, rho_rng = c.rho_rng, lum = 1.0;
  if constexpr (HAD) {
    double L, l1, l2;
    {
#pragma clang fp contract(off)
      L = c.Lhi + x[8] * c.Lrng;
      l1 = x[9] * L;
      l2 = L - l1;
    }
    const double tau = exp_fin(L);
    sh = tau * c.S;
    rs = sqrt_nr(sh);
    rho_rng = atan_rr((sh - c.M2) * c.invMG) - c.rho_lo;
    lum = tau * -L * pdf_pair(c, tau, L, expm1_fin(l1) * expm1_fin(l2));
  }
  // the masses from the Breit-Wigner maps; their Jacobians' resonance factors cancel
  // the W propagators (see ww_me2): only the maps' ranges enter the weight
  const double mp2 = bw_mass(c, x[0], rho_rng);
  obs_sq = mp2 > 0.0 ? mp2 : 0.0;
  if (!(mp2 > 0.0)) return 0.0;
  const double mp = sqrt_nr(mp2);
  const double up = (rs - mp) * (rs - mp);
  const double rrng2 = atan_rr((up - c.M2) * c.invMG) - c.rho_lo;
  const double mm2 = bw_mass(c, x[1], rrng2);
  if (!(mm2 > 0.0)) return 0.0;
  const double mm = sqrt_nr(mm2);
  const double lam = (sh - mp2 - mm2) * (sh - mp2 - mm2) - 4.0 * mp2 * mm2;
  if (!(lam > 0.0)) return 0.0;
  const double sl = sqrt_nr(lam);
  const double ct = 2.0 * x[2] - 1.0, st = sqrt_nr((1.0 - ct) * (1.0 + ct));
  // s-channel photon + Z coefficients, left-handed quark [q], and the sum of the squares
  // of the right-handed ones; hadronic: e^2 Q / shat + e^2 f (shat - MZ^2 - i MZ GZ) /
  // |shat - MZ^2 + i MZ GZ|^2, the two reciprocals from one
  double cre[2] = {c.cs_re[0][0], c.cs_re[1][0]}, cim[2] = {c.cs_im[0][0], c.cs_im[1][0]}, csR2 = c.csR2;
  double wk = c.wk;
  if constexpr (HAD) {
    const double dr = sh - c.mz2, dd = dr * dr + c.mzgz2, r = rcp_nr(sh * dd);
    const double idd = r * sh, ish = r * dd;
    wk *= ish;
    csR2 = 0.0;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      cre[q] = c.csq[q] * ish + c.csf[q][0] * dr * idd;
      cim[q] = -c.csf[q][0] * c.mzgz * idd;
      const double rr = c.csq[q] * ish + c.csf[q][1] * dr * idd, ri = -c.csf[q][1] * c.mzgz * idd;
      csR2 += rr * rr + ri * ri;
    }
  }
  const double i2rs = HAD ? 0.5 * rcp_nr(rs) : c.i2rs;
  const double q = sl * i2rs;
  // E+ + E- = rs as rounded: the diagrams cancel by (shat / M_W^2)^2 at high energy, and
  // a mismatch of the energies would come through (measured on 1e5 hadronic events: the
  // 99th percentile of the error 4.2e-13 with it, 5.0e-13 without; the currents' form 4.0e-13)
  const double Ep = (sh + mp2 - mm2) * i2rs, Em = rs - Ep;
  const double qz = q * ct, qx = q * st, qx2 = qx * qx;
  WWPoint w;
  {
    const double Lp = Ep + fabs(qz), Lm = Em + fabs(qz), r = rcp_nr(Lp * Lm);
    const double Sp = (mp2 + qx2) * (r * Lm), Sm = (mm2 + qx2) * (r * Lp);
    const bool up = qz >= 0.0;
    w.qx = qx;
    w.pm = up ? Sp : Lp;
    w.pp = up ? Lp : Sp;
    w.mm = up ? Sm : Lm;
    w.mp = up ? Lm : Sm;
  }
  cx<double> l3[2], n4[2], n5[2], l6[2];
  // x bounded away from 0 (a grid edge; its bin has no width): the scale 1 / x stays finite
  const double xp = fmax(x[4], 0x1p-120), xm = fmax(x[6], 0x1p-120);
  const double mep = Ep + mp, mem = Em + mm;
  {
    double s, cc;
    sincos_2pi(x[5] - x[3], s, cc);
    const double r = sqrt_nr(xp * (1.0 - xp));
    decay_spinors(mp + w.pm, mp + w.pp, qx, xp, {r * cc, r * s}, l3, n4);
  }
  {
    double s, cc;
    sincos_2pi(x[7] - x[3], s, cc);
    const double r = sqrt_nr(xm * (1.0 - xm));
    // the muon's spinor is needed conjugated, the antineutrino's as it is: the roles of
    // l and n exchange under phi -> -phi
    cx<double> a[2], b[2];
    decay_spinors(mm + w.mp, mm + w.mm, -qx, xm, {r * cc, -r * s}, a, b);
    n5[0] = a[0];
    n5[1] = a[1];
    l6[0] = b[0];
    l6[1] = b[1];
  }
  // minus the exchange invariants, -t = sums of positive terms, and their reciprocals
  // with that of the spinors' scale from one
  const double tu = __fma_rn(w.pm, w.mm, qx2), td = __fma_rn(w.mp, w.pp, qx2);
  const double P = tu * td, N = (mep * xp) * (mem * xm);
  const double r = rcp_nr(P * N), iP = r * N, iN = r * P;
  const double me = ww_spinor_me2(c, w, l3, n4, n5, l6, cre, cim, csR2, -c.ct * (iP * td), -c.ct * (iP * tu));
  const double f = wk * (sl * me) * (iN * iN) * (rho_rng * rrng2);
  if constexpr (HAD) return f * lum;
  return f;
}

// the same point with the amplitude (spinors, currents, diagrams) in binary32; phase space
// (masses, momenta, lambda) is binary64
__device__ __forceinline__ double f_ww_single(const PhysConst& c, const double* x, double& obs_sq) {
  using R = float;
  const double rs = c.rs, sh = c.shat, rho_rng = c.rho_rng;
  const double mp2 = bw_mass<true>(c, x[0], rho_rng);
  obs_sq = mp2 > 0.0 ? mp2 : 0.0;
  if (!(mp2 > 0.0)) return 0.0;
  double mp, imp;
  sqrt_rsqrt_nr(mp2, mp, imp);
  const double up = (rs - mp) * (rs - mp);
  const double rrng2 = atan_rr((up - c.M2) * c.invMG) - c.rho_lo;
  const double mm2 = bw_mass<true>(c, x[1], rrng2);
  if (!(mm2 > 0.0)) return 0.0;
  double mm, imm;
  sqrt_rsqrt_nr(mm2, mm, imm);
  const double lam = (sh - mp2 - mm2) * (sh - mp2 - mm2) - 4.0 * mp2 * mm2;
  if (!(lam > 0.0)) return 0.0;
  const double sl = sqrt_nr(lam);
  const double i2rs = c.i2rs;
  const double q = sl * i2rs;
  const double Ep = (sh + mp2 - mm2) * i2rs, Em = (sh - mp2 + mm2) * i2rs;
  const double ct = 2.0 * x[2] - 1.0, st = sqrt_nr((1.0 - ct) * (1.0 + ct));
  double sf, cf;
  sincos_2pi(x[3], sf, cf);
  const double qp[4] = {Ep, q * st * cf, q * st * sf, q * ct};
  const double qm[4] = {Em, -qp[1], -qp[2], -qp[3]};
  // each W's decay leptons in the CM frame, turned into its lepton current at once
  cx<R> Jp[4], Jm[4];
  {
    const double c3 = 2.0 * x[4] - 1.0, s3 = sqrt_nr((1.0 - c3) * (1.0 + c3));
    double s, cc;
    sincos_2pi(x[5], s, cc);
    const double h = 0.5 * mp;
    const double k[4] = {h, h * s3 * cc, h * s3 * s, h * c3};
    double d3[4], d4[4];
    boost_pair<double>(qp, mp, imp, k, d3, d4);
    lepton_current<R>(d4, d3, Jp);
  }
  {
    const double c5 = 2.0 * x[6] - 1.0, s5 = sqrt_nr((1.0 - c5) * (1.0 + c5));
    double s, cc;
    sincos_2pi(x[7], s, cc);
    const double h = 0.5 * mm;
    const double k[4] = {h, h * s5 * cc, h * s5 * s, h * c5};
    double d5[4], d6[4];
    boost_pair<double>(qm, mm, imm, k, d5, d6);
    lepton_current<R>(d5, d6, Jm);
  }
  R qpr[4], qmr[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    qpr[i] = static_cast<R>(qp[i]);
    qmr[i] = static_cast<R>(qm[i]);
  }
  // the exchange invariants cancel for forward W bosons, so they are formed in binary64
  // without cancellation, E -+ q cos = m^2 / (E + q) + q (1 -+ cos) for the W+ (and with
  // cos -> -cos for the W-)
  const double epm = div_nr(mp2, Ep + q) + q * (1.0 - ct);  // Ep - q cos
  const double emm = div_nr(mm2, Em + q) + q * (1.0 + ct);  // Em + q cos
  ExchInv<R> iv;
  iv.tu = static_cast<R>(mp2 - rs * epm);
  iv.td = static_cast<R>(mm2 - rs * emm);
  iv.b00u = static_cast<R>(-epm);
  iv.b11u = static_cast<R>(rs - (Ep + q * ct));
  iv.b00d = static_cast<R>(-emm);
  iv.b11d = static_cast<R>(rs - (Em - q * ct));
  const double me = static_cast<double>(ww_me2(c, Jp, Jm, qpr, qmr, iv));
  const double gbw = (c.gs * c.gs) * c.invMG, ish = 1.0 / sh;
  return (c.conv * kWWPS) * (gbw * gbw) * (ish * ish) * (sl * me) * (rho_rng * rrng2);
}

template <typename R, bool HAD = false>
__device__ __forceinline__ double f_ww(const PhysConst& c, const double* x, double& obs_sq) {
  if constexpr (sizeof(R) < sizeof(double)) {
    static_assert(!HAD, "the hadronic amplitude is binary64 only");
    return f_ww_single(c, x, obs_sq);
  } else {
    return f_ww_double<HAD>(c, x, obs_sq);
  }
}

}  // namespace vg
