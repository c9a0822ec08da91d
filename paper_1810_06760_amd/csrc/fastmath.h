// Table-driven FP64 complex exponential exp(-g) (cos phi + i sin phi) for bounded
// arguments.
//
// exp: Tang's table-driven method.  x = -g = (256 m + j) ln2/256 + r with
//   |r| <= ln2/512, so exp(x) = 2^m 2^{j/256} (1 + r + r^2/2 + r^3/6 + r^4/24);
//   the omitted r^5/120 term is below 4e-17 relative.
// sin/cos: reduction by multiples of pi/128, |r| <= pi/256, Taylor polynomials of
//   r (through r^5 for sin, r^6 for cos, truncation below 1e-17 absolute), then the
//   angle-addition formulas with sin(j pi/128), cos(j pi/128) from a 256-entry table.
// The tables are filled per workgroup from the device library's exp2/sincos,
// so every entry is correctly rounded or within an ulp.
//
// cexp_neg_units takes the phase in units of pi/128 (v = phi 128/pi, so the
// reduction is v - rint(v) with no constant to split) and a mask; both
// roundings to an integer add 1.5 2^52, which leaves round-to-nearest(x) in
// the low mantissa bits for |x| < 2^51.
#pragma once

#include <hip/hip_runtime.h>

namespace fga {

constexpr int TRIG_N = 256;
struct TrigTables {
  double e2[TRIG_N];    // 2^(j/256)
  double2 sc[TRIG_N];   // (sin(j pi/128), cos(j pi/128)): one 16-byte read per lookup
};

// Fill the tables; call from every thread of the block, then __syncthreads().
__device__ __forceinline__ void fill_tables(TrigTables &t)
{
  for (int j = threadIdx.x; j < TRIG_N; j += blockDim.x) {
    t.e2[j] = exp2((double)j / 256.0);
    double s, c;
    sincospi((double)j / 128.0, &s, &c);
    t.sc[j] = make_double2(s, c);
  }
}

// 256/ln2, ln2/256 split so that k*LN2_256_HI is exact for |k| < 2^20
// (hi has 32 significant bits; hi + lo = ln2/256 to ~5e-30).
constexpr double INV_LN2_256 = 369.3299304675746;
constexpr double LN2_256_HI = 0.0027076061742263846;
constexpr double LN2_256_LO = -1.6409824502660487e-13;
constexpr double INV_PI_128 = 40.74366543152521;  // 128/pi

constexpr double RND_MAGIC = 6755399441055744.0;  // 1.5 * 2^52
constexpr double PI_128 = 0.02454369260617026;      // pi/128

// in ? exp(-g) (cos(v pi/128) + i sin(v pi/128)) : 0, for 0 <= g <~ 700 and
// |v| < 2^51 where in is true; where it is false g >= 0 and v may be any
// finite values (the magnitude is replaced by 0 before it meets the phase).
__device__ __forceinline__ void cexp_neg_units(const TrigTables &t, double g, double v, bool in, double &re,
                                               double &im)
{
  // exp(-g)
  const double tk = fma(g, -INV_LN2_256, RND_MAGIC);
  const double kd = tk - RND_MAGIC;
  const int k = __double2loint(tk);
  const int j = k & (TRIG_N - 1);
  const int m = k >> 8;  // floor(k / 256)
  double r = fma(-kd, LN2_256_HI, -g);
  r = fma(-kd, LN2_256_LO, r);
  double q = fma(r, 1.0 / 24.0, 1.0 / 6.0);
  q = fma(r, q, 0.5);
  q = fma(r, q, 1.0);
  q = q * r;  // p(r) - 1
  const double tj = t.e2[j];
  double ex = ldexp(fma(tj, q, tj), m);
  ex = in ? ex : 0.0;
  // sin / cos: v - rint(v) is exact, |u| <= pi/256
  const double tn = v + RND_MAGIC;
  const double nd = tn - RND_MAGIC;
  const int n = __double2loint(tn) & (TRIG_N - 1);
  const double u = (v - nd) * PI_128;
  const double u2 = u * u;
  const double sp = fma(u2, 1.0 / 120.0, -1.0 / 6.0);
  const double su = fma(u * u2, sp, u);
  double cp = fma(u2, -1.0 / 720.0, 1.0 / 24.0);
  cp = fma(u2, cp, -0.5);
  const double cu = fma(u2, cp, 1.0);
  const double2 scn = t.sc[n];
  const double sj = scn.x, cj = scn.y;
  const double sphi = fma(su, cj, cu * sj);
  const double cphi = fma(cu, cj, -(su * sj));
  re = ex * cphi;
  im = ex * sphi;
}

// Tables of cexp_scaled: as TrigTables, with the high word of 2^(j/256) less
// j 2^12, so that adding k 2^12 to it (k = 256 m + j) adds m to the exponent.
struct ScaledTables {
  uint2 e2[TRIG_N];     // (low, high - (j << 12)) words of 2^(j/256)
  double2 sc[TRIG_N];   // (sin(j pi/128), cos(j pi/128))
};

__device__ __forceinline__ void fill_tables(ScaledTables &t)
{
  for (int j = threadIdx.x; j < TRIG_N; j += blockDim.x) {
    const double e = exp2((double)j / 256.0);
    t.e2[j] = make_uint2((unsigned)__double2loint(e), (unsigned)__double2hiint(e) - ((unsigned)j << 12));
    double s, c;
    sincospi((double)j / 128.0, &s, &c);
    t.sc[j] = make_double2(s, c);
  }
}

// Coefficients of cexp_scaled's polynomials, held in registers over a loop:
// the compiler otherwise moves each into a fresh register pair at every use
// (7 moves in a term of 49 instructions).  An FMA takes one scalar operand, so
// the first step of each polynomial has its addend in a vector register.
struct ScaledCoeffs {
  double e4, e3, e2, e1;  // L^4/24, L^3/6, L^2/2, L with L = ln2/256
  double s5, s3, s1;      // P^5/120, -P^3/6, P with P = pi/128
  double c6, c4, c2;      // -P^6/720, P^4/24, -P^2/2
  __device__ __forceinline__ ScaledCoeffs()
  {
    constexpr double L = 0.0027076061740622863, P = PI_128;
    e4 = L * L * L * L / 24.0;
    e3 = L * L * L / 6.0;
    e2 = L * L / 2.0;
    e1 = L;
    s5 = P * P * P * P * P / 120.0;
    s3 = -P * P * P / 6.0;
    s1 = P;
    c6 = -P * P * P * P * P * P / 720.0;
    c4 = P * P * P * P / 24.0;
    c2 = -P * P / 2.0;
    asm volatile("" : "+v"(e3), "+v"(s3), "+v"(c4));
    asm volatile("" : "+s"(e4), "+s"(e2), "+s"(e1), "+s"(s5), "+s"(s1), "+s"(c6), "+s"(c2));
  }
};

// in ? exp(-C t ln2/256) (cos(v pi/128) + i sin(v pi/128)) : 0 for nc + ncl = -C,
// t >= 0 and C t < 1022 * 256 (the exponent must stay normal; WIDE: C t < 2^31),
// |v| < 2^51 where in is true; where it is false t >= 0 and v may be any finite
// values.  The same reductions and polynomials as cexp_neg_units with both
// arguments in table units: the remainders r = -C t - k and w = v - n are in units
// of ln2/256 and pi/128, which the coefficients carry, and k goes into the exponent
// by one shift-and-add on the table's high word.  C takes two numbers, since its
// rounding to one is an error of up to 2^-53 of the exponent, the same for all
// terms: with nc alone 4000 terms of exponents up to 25 were off by 1.32e-15 (root
// mean square, eps = 0.01) where they are now off by 7.2e-16.  WIDE
// scales by ldexp instead: below the normal range the values are subnormal, then 0.
template <bool WIDE>
__device__ __forceinline__ void cexp_scaled(const ScaledTables &tab, const ScaledCoeffs &K, double t, double nc,
                                            double ncl, double v, bool in, double &re, double &im)
{
  // both table reads first: the polynomials run while they are on their way
  const double tk = fma(t, nc, RND_MAGIC);
  const double tn = v + RND_MAGIC;
  const int k = __double2loint(tk);
  const uint2 e = tab.e2[k & (TRIG_N - 1)];
  const double2 scn = tab.sc[__double2loint(tn) & (TRIG_N - 1)];
  const double kd = tk - RND_MAGIC;
  const double nd = tn - RND_MAGIC;
  const double r = fma(t, ncl, fma(t, nc, -kd));
  const double w = v - nd;  // exact
  double q = fma(r, K.e4, K.e3);
  const double w2 = w * w;
  double sp = fma(w2, K.s5, K.s3);
  double cp = fma(w2, K.c6, K.c4);
  q = fma(r, q, K.e2);
  sp = fma(w2, sp, K.s1);
  cp = fma(w2, cp, K.c2);
  q = fma(r, q, K.e1);
  const double su = w * sp;
  const double cu = fma(w2, cp, 1.0);
  q = q * r;  // e^{rL} - 1
  const unsigned up = (unsigned)(WIDE ? k & (TRIG_N - 1) : k) << 12;
  const double tj = __hiloint2double((int)(up + e.y), (int)e.x);
  double ex = fma(tj, q, tj);
  if (WIDE) ex = ldexp(ex, k >> 8);
  ex = in ? ex : 0.0;
  const double sphi = fma(su, scn.y, cu * scn.x);
  const double cphi = fma(cu, scn.y, -(su * scn.x));
  re = ex * cphi;
  im = ex * sphi;
}

}  // namespace fga
