// The FP64 right-hand side of the FGA ODE system and the classic RK4 step,
// shared by the integrator and the interface step.  The right-hand side is,
// for sigma = +1 / -1 (Sec. 2.2):
//   dQ/dt = sigma c P/|P|,  dP/dt = -sigma |P| grad c         (eq:char_plus, eq:char_minus)
//   d(dzQ)/dt = sigma [dzQ (grad c (x) P)/|P| + c dzP (I - P (x) P/|P|^2)/|P|]
//   d(dzP)/dt = sigma [-|P| dzQ Hess c - dzP (P (x) grad c)/|P|]   (eq:DzDt)
//   da_P/dt = a_P (sigma grad c . P/|P| + tr(Z^{-1} dZ/dt)/2)       (eq:amp_P)
//   d(a_SV, a_SH)/dt = s (a_SV, a_SH) + omega (-a_SH, a_SV),
//     omega = dN_SH/dt . N_SV = sigma (P.e) e.(grad c x P)/|e x P|^2  (eq:amp_SV, eq:amp_SH)
//   dS/dt = P . dQ/dt - sigma c |P| = 0: H is homogeneous of degree one in P, so the
//     action keeps its value and no step touches it
// tr(Z^{-1} dZ/dt) is formed as (sum_ij cof(Z)_ij dZ_ij) / det Z, so no
// matrix inverse is built.  Frame-free S amplitudes (SV = 1): the physical
// polarisation A = a_SV N_SV + a_SH N_SH is advanced instead, by
//   dA/dt = s A - (A . dPhat/dt) Phat,  dPhat/dt = (dP/dt - Phat (Phat . dP/dt))/|P|,
// which is the framed system with the frame's rotation differentiated out.
#pragma once

#include "device_common.h"

namespace fga {
namespace rk {

constexpr int NS = 47;
enum { IQ = 0, IP = 3, IZQR = 6, IZQI = 15, IZPR = 24, IZPI = 33, IA = 42, IS = 46 };
// frame-free S state: A_x at IA, IA+1, A_y at IA+2, IA+3, A_z at IAZ, IAZ+1
constexpr int IAZ = 47;
template <int SV> constexpr int nstate() { return SV ? 49 : NS; }
constexpr double COS10 = 0.98480775301220805936;  // cos(10 degrees)

// One RK4 stage: k = f(stage input), acc += weight k, yt <- y + fraction dt k in
// place.  The derivative is folded in as soon as each group of components is
// complete, row by row for dzQ/dzP, so the live state stays at y, acc and yt.
//
// LAST: the fourth stage, which forms no further stage input and writes y itself;
// otherwise stage `st` of a loop.
// EXIT (layered media, LAST): true, and y as it was, where the step's end lies
// outside the beam's layer.
template <int MK, int SV = 0, bool LAST = false, bool EXIT = false>
__device__ __forceinline__ bool stage(const DevMedium &med, int sp, int layer, double sg, bool isS,
                                      const double e[3], double *__restrict__ y, double *__restrict__ yt,
                                      double *__restrict__ acc, int st, double dt,
                                      const MedBlock *blk = nullptr, CellCache *cells = nullptr,
                                      const Layer *lay = nullptr)
{
  const double h2 = 0.5 * dt, h6 = dt / 6.0;
  const double wacc = (st == 0 || st == 3) ? 1.0 : 2.0;
  const double cnext = st == 2 ? dt : (st == 3 ? 0.0 : h2);
  auto fold = [&](int f, double k) {
    if (LAST) {
      y[f] += h6 * (acc[f] + k);
    } else {
      acc[f] += wacc * k;
      yt[f] = y[f] + cnext * k;
    }
  };
  double c, g[3], H6[6];
  if (MK == MK_GRID && cells) {
    double v[10];
    cells->fields(v);
    const double scale = sp && !med.two_fields ? med.cs_ratio : 1.0;
    c = scale * v[0];
#pragma unroll
    for (int k = 0; k < 3; ++k) g[k] = scale * v[1 + k];
#pragma unroll
    for (int k = 0; k < 6; ++k) H6[k] = scale * v[4 + k];
  } else if (MK == MK_LAYERED && lay) {
    layer_eval(*lay, yt + IQ, c, g, H6);
  } else {
    medium_eval<MK>(med, sp, layer, yt + IQ, c, g, H6, blk);
  }
  const double H[3][3] = {{H6[0], H6[3], H6[4]}, {H6[3], H6[1], H6[5]}, {H6[4], H6[5], H6[2]}};
  const double P0 = yt[IP], P1 = yt[IP + 1], P2 = yt[IP + 2];
  const double np2 = P0 * P0 + P1 * P1 + P2 * P2;
  const double inp = fast_rsqrt(np2), np = np2 * inp;
  const double ph[3] = {P0 * inp, P1 * inp, P2 * inp};
  const double sc = sg * c;
  const double ci = sc * inp;
  // the ray first: the next stage's point (after the last stage the next step's)
  // is known before the Jacobians' work begins, and its cell is asked for (the
  // trilinear medium's steps are all peeled)
  if constexpr (EXIT) {
    double q[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) q[j] = y[IQ + j] + h6 * (acc[IQ + j] + sc * ph[j]);
    if (leaves_layer(*lay, q)) return true;
#pragma unroll
    for (int j = 0; j < 3; ++j) y[IQ + j] = q[j];
  } else {
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const double k = sc * ph[j];
      fold(IQ + j, k);
    }
  }
  if (MK == MK_GRID && cells) cells->request(med, sp, LAST ? y + IQ : yt + IQ);

  // cofactors of Z = dzQ + i dzP and det Z (cyclic index form carries the sign)
  double Cr[9], Ci[9];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const int i1 = (i + 1) % 3, i2 = (i + 2) % 3;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const int j1 = (j + 1) % 3, j2 = (j + 2) % 3;
      const int a = 3 * i1 + j1, b = 3 * i2 + j2, cc = 3 * i1 + j2, d = 3 * i2 + j1;
      const double ar = yt[IZQR + a] - yt[IZPI + a], ai = yt[IZQI + a] + yt[IZPR + a];
      const double br = yt[IZQR + b] - yt[IZPI + b], bi = yt[IZQI + b] + yt[IZPR + b];
      const double cr = yt[IZQR + cc] - yt[IZPI + cc], cim = yt[IZQI + cc] + yt[IZPR + cc];
      const double dr = yt[IZQR + d] - yt[IZPI + d], di = yt[IZQI + d] + yt[IZPR + d];
      Cr[3 * i + j] = (ar * br - ai * bi) - (cr * dr - cim * di);
      Ci[3 * i + j] = (ar * bi + ai * br) - (cr * di + cim * dr);
    }
  }
  double detr = 0.0, deti = 0.0;
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const double zr = yt[IZQR + j] - yt[IZPI + j], zi = yt[IZQI + j] + yt[IZPR + j];
    detr += zr * Cr[j] - zi * Ci[j];
    deti += zr * Ci[j] + zi * Cr[j];
  }

  // -sigma |P| Hess c and -sigma grad c
  double Hn[3][3], gn[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    gn[i] = -sg * g[i];
#pragma unroll
    for (int j = 0; j <= i; ++j) Hn[i][j] = Hn[j][i] = (-sg * np) * H[i][j];
  }
  double Tr = 0.0, Ti = 0.0;
#pragma unroll
  for (int m = 0; m < 3; ++m) {
    const double *qr = yt + IZQR + 3 * m, *qi = yt + IZQI + 3 * m, *pr = yt + IZPR + 3 * m, *pi = yt + IZPI + 3 * m;
    const double vr = pr[0] * ph[0] + pr[1] * ph[1] + pr[2] * ph[2];
    const double vi = pi[0] * ph[0] + pi[1] * ph[1] + pi[2] * ph[2];
    // sigma (row . grad c) - sigma c/|P| (row . Phat): what multiplies Phat in d(dzQ)/dt
    const double ur = -(qr[0] * gn[0] + qr[1] * gn[1] + qr[2] * gn[2]) - ci * vr;
    const double ui = -(qi[0] * gn[0] + qi[1] * gn[1] + qi[2] * gn[2]) - ci * vi;
    double kq_r[3], kq_i[3], kp_r[3], kp_i[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const int o = 3 * m + j;
      kq_r[j] = ur * ph[j] + ci * pr[j];
      kq_i[j] = ui * ph[j] + ci * pi[j];
      kp_r[j] = vr * gn[j] + qr[0] * Hn[0][j] + qr[1] * Hn[1][j] + qr[2] * Hn[2][j];
      kp_i[j] = vi * gn[j] + qi[0] * Hn[0][j] + qi[1] * Hn[1][j] + qi[2] * Hn[2][j];
      // dZ = d(dzQ) + i d(dzP); T += cof(Z) : dZ
      const double dr = kq_r[j] - kp_i[j], di = kq_i[j] + kp_r[j];
      Tr += Cr[o] * dr - Ci[o] * di;
      Ti += Cr[o] * di + Ci[o] * dr;
    }
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const int o = 3 * m + j;
      fold(IZQR + o, kq_r[j]);
      fold(IZQI + o, kq_i[j]);
      fold(IZPR + o, kp_r[j]);
      fold(IZPI + o, kp_i[j]);
    }
  }
  const double idd = fast_rcp(detr * detr + deti * deti);
  const double trr = (Tr * detr + Ti * deti) * idd;
  const double tri = (Ti * detr - Tr * deti) * idd;
  const double sr = sg * (g[0] * ph[0] + g[1] * ph[1] + g[2] * ph[2]) + 0.5 * trr;
  const double si = 0.5 * tri;
  double ka[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  if (SV && isS) {
    // parallel transport of A: dPhat/dt from dP/dt = -sigma |P| grad c
    const double dq0 = -sg * g[0], dq1 = -sg * g[1], dq2 = -sg * g[2];   // (dP/dt)/|P|
    const double pd = ph[0] * dq0 + ph[1] * dq1 + ph[2] * dq2;
    const double dph[3] = {dq0 - ph[0] * pd, dq1 - ph[1] * pd, dq2 - ph[2] * pd};
    const double Ar[3] = {yt[IA], yt[IA + 2], yt[IAZ]}, Ai[3] = {yt[IA + 1], yt[IA + 3], yt[IAZ + 1]};
    const double adr = Ar[0] * dph[0] + Ar[1] * dph[1] + Ar[2] * dph[2];
    const double adi = Ai[0] * dph[0] + Ai[1] * dph[1] + Ai[2] * dph[2];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      ka[2 * c] = sr * Ar[c] - si * Ai[c] - adr * ph[c];
      ka[2 * c + 1] = sr * Ai[c] + si * Ar[c] - adi * ph[c];
    }
  } else {
    const double a0r = yt[IA], a0i = yt[IA + 1], a1r = yt[IA + 2], a1i = yt[IA + 3];
    if (!isS) {
      ka[0] = sr * a0r - si * a0i;
      ka[1] = sr * a0i + si * a0r;
      ka[2] = 0.0;
      ka[3] = 0.0;
    } else {
      const double gx0 = g[1] * P2 - g[2] * P1, gx1 = g[2] * P0 - g[0] * P2, gx2 = g[0] * P1 - g[1] * P0;
      const double egp = e[0] * gx0 + e[1] * gx1 + e[2] * gx2;
      const double pe = P0 * e[0] + P1 * e[1] + P2 * e[2];
      const double x0 = e[1] * P2 - e[2] * P1, x1 = e[2] * P0 - e[0] * P2, x2 = e[0] * P1 - e[1] * P0;
      const double om = sg * pe * egp * fast_rcp(x0 * x0 + x1 * x1 + x2 * x2);
      ka[0] = sr * a0r - si * a0i - om * a1r;
      ka[1] = sr * a0i + si * a0r - om * a1i;
      ka[2] = sr * a1r - si * a1i + om * a0r;
      ka[3] = sr * a1i + si * a1r + om * a0i;
    }
  }
#pragma unroll
  for (int t = 0; t < (SV ? 6 : 4); ++t) fold(t < 4 ? IA + t : IAZ + t - 4, ka[t]);
#pragma unroll
  for (int j = 0; j < 3; ++j) fold(IP + j, np * gn[j]);
  return false;
}

// After a step: an S beam whose P has come within 10 degrees of its frame
// axis switches axis (e_z <-> e_x) and re-expresses (a_SV, a_SH) so that the
// physical polarisation a_SV N_SV + a_SH N_SH is unchanged.
__device__ __forceinline__ void reframe_s(const double P[3], double A[4], double e[3])
{
  const double inp = fast_rsqrt(P[0] * P[0] + P[1] * P[1] + P[2] * P[2]);
  const double pe = P[0] * e[0] + P[1] * e[1] + P[2] * e[2];
  if (fabs(pe) * inp > COS10) {
    double nsh[3], nsv[3];
    s_frame(P, e, nsh, nsv);
    double Ar[3], Ai[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      Ar[c] = A[0] * nsv[c] + A[2] * nsh[c];
      Ai[c] = A[1] * nsv[c] + A[3] * nsh[c];
    }
    const bool was_z = e[2] != 0.0 && e[0] == 0.0 && e[1] == 0.0;
    e[0] = was_z ? 1.0 : 0.0;
    e[1] = 0.0;
    e[2] = was_z ? 0.0 : 1.0;
    s_frame(P, e, nsh, nsv);
    A[0] = Ar[0] * nsv[0] + Ar[1] * nsv[1] + Ar[2] * nsv[2];
    A[1] = Ai[0] * nsv[0] + Ai[1] * nsv[1] + Ai[2] * nsv[2];
    A[2] = Ar[0] * nsh[0] + Ar[1] * nsh[1] + Ar[2] * nsh[2];
    A[3] = Ai[0] * nsh[0] + Ai[1] * nsh[1] + Ai[2] * nsh[2];
  }
}

__device__ __forceinline__ void reframe_s(double *y, double e[3]) { reframe_s(y + IP, y + IA, e); }

// One classic RK4 step of size dt in place, y' = y + dt/6 (k1 + 2 k2 + 2 k3 + k4).
// SV = 1: frame-free S amplitudes (y holds nstate<1>() values); after the
// step A is projected on the plane orthogonal to the new P, which the exact
// solution never leaves (the projection removes the step's truncation drift).
// PEEL: the fourth stage on its own after a loop of three.  The arithmetic
// reaches half of the register file, and y and acc live in the other half: the
// loop's fourth turn reads y for a stage input that nobody takes and the step's
// end reads y and acc once more (4.1 M beams x 16 steps in the trilinear medium:
// 12.0 ms as a loop of four, 11.5 peeled).  All four in a row are 65 KB of code,
// as much as the instruction cache holds for two compute units: 16.9 ms.  Callers
// with many steps in a row of code (the interface step) keep the loop.
// EXIT (layered media, with PEEL and the beam's layer): a step that would leave the beam's layer is
// not taken: y stays as it was and the result is true.
template <int MK, int SV = 0, bool PEEL = false, bool EXIT = false>
__device__ __forceinline__ bool rk4_step(const DevMedium &med, int sp, int layer, double sg, bool isS,
                                         const double e[3], double *y, double dt, const MedBlock *blk = nullptr,
                                         CellCache *cells = nullptr, const Layer *lay = nullptr)
{
  constexpr int N = nstate<SV>();
  double acc[N], yt[N];
#pragma unroll
  for (int f = 0; f < N; ++f) { yt[f] = y[f]; acc[f] = 0.0; }
#pragma nounroll
  for (int st = 0; st < (PEEL ? 3 : 4); ++st) {
    if (MK == MK_GRID && cells) cells->wait();
    stage<MK, SV>(med, sp, layer, sg, isS, e, y, yt, acc, st, dt, blk, cells, lay);
  }
  if constexpr (PEEL) {
    if (MK == MK_GRID && cells) cells->wait();
    if (stage<MK, SV, true, EXIT>(med, sp, layer, sg, isS, e, y, yt, acc, 3, dt, blk, cells, lay)) return true;
  } else {
    const double h6 = dt / 6.0;
#pragma unroll
    for (int f = 0; f < N; ++f)
      if (f != IS) y[f] += h6 * acc[f];
  }
  if (SV && isS) {
    const double inp = fast_rsqrt(y[IP] * y[IP] + y[IP + 1] * y[IP + 1] + y[IP + 2] * y[IP + 2]);
    const double ph[3] = {y[IP] * inp, y[IP + 1] * inp, y[IP + 2] * inp};
    const double apr = y[IA] * ph[0] + y[IA + 2] * ph[1] + y[IAZ] * ph[2];
    const double api = y[IA + 1] * ph[0] + y[IA + 3] * ph[1] + y[IAZ + 1] * ph[2];
    y[IA] -= apr * ph[0];
    y[IA + 2] -= apr * ph[1];
    y[IAZ] -= apr * ph[2];
    y[IA + 1] -= api * ph[0];
    y[IA + 3] -= api * ph[1];
    y[IAZ + 1] -= api * ph[2];
  }
  return false;
}

// The classic RK4 step where grad c = 0 (a homogeneous medium, or inside one layer
// of a layered medium).  There P and dzP have zero derivative and Q and dzQ
// constant ones, so Q and dzQ, and with it Z = dzQ + i dzP, move by h/6 X, X = 6
// times their rate, for as long as the beam stays in its layer.  The amplitudes' derivative is s a,
// s = tr(Z^{-1} dZ/dt)/2 at the stage's time: the two middle stages share one s and
// a step's last s is the next one's first, so a step needs two traces, and both
// amplitudes (complex a_P; a_SV and a_SH, omega = 0) grow by one complex factor.
// The formulas are those of rk4_step with the medium's gradient and Hessian at
// zero, so the two agree to rounding.  With four traces a step, K formed anew and
// one wavefront per SIMD 98 k beams x 50 steps in a homogeneous medium took 247 us
// and 898 k beams x 48 steps and records in a layered Earth 4.0 ms; so 132 us and
// 2.0 ms, the latter 3.5 TB/s of state and records.
// dzP is read through a functor (re(o), im(o) of entry o), from registers or LDS.
struct ConstRates {
  double xq[3];                          // 6 dQ/dt
  double qr[9], qi[9], xr[9], xi[9];     // dzQ and 6 d(dzQ)/dt, rows m (the derivative by one z_m)
  double sr, si;                         // s at dzQ

  // for speed c: dQ/dt = sigma c Phat (eq:char_plus, eq:char_minus), d(dzQ)/dt =
  // sigma c dzP (I - Phat (x) Phat)/|P| (eq:DzDt with grad c = 0)
  template <class ZP> __device__ __forceinline__ void init(double c, double sg, const double *y, const ZP &zp)
  {
    const double *P = y + IP, *pr = y + IZPR, *pi = y + IZPI;
    const double inp = fast_rsqrt(P[0] * P[0] + P[1] * P[1] + P[2] * P[2]);
    const double ph[3] = {P[0] * inp, P[1] * inp, P[2] * inp};
    const double sc = 6.0 * sg * c, ci = sc * inp;
#pragma unroll
    for (int j = 0; j < 3; ++j) xq[j] = sc * ph[j];
#pragma unroll
    for (int m = 0; m < 3; ++m) {
      const double vr = pr[3 * m] * ph[0] + pr[3 * m + 1] * ph[1] + pr[3 * m + 2] * ph[2];
      const double vi = pi[3 * m] * ph[0] + pi[3 * m + 1] * ph[1] + pi[3 * m + 2] * ph[2];
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        const int o = 3 * m + j;
        xr[o] = ci * (pr[o] - vr * ph[j]);
        xi[o] = ci * (pi[o] - vi * ph[j]);
        qr[o] = y[IZQR + o];
        qi[o] = y[IZQI + o];
      }
    }
    trace(zp, 0.0, sr, si);
  }

  // s at dzQ + h X
  template <class ZP> __device__ __forceinline__ void trace(const ZP &zp, double h, double &s_r, double &s_i) const
  {
    double ar[9], ai[9];
    zp.again();
#pragma unroll
    for (int o = 0; o < 9; ++o) {
      ar[o] = qr[o] - zp.im(o);
      ai[o] = qi[o] + zp.re(o);
      if (h != 0.0) {
        ar[o] += h * xr[o];
        ai[o] += h * xi[o];
      }
    }
    // cofactors (cyclic index form), det Z and T = cof(Z) : X
    double detr = 0.0, deti = 0.0, Tr = 0.0, Ti = 0.0;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const int i1 = (i + 1) % 3, i2 = (i + 2) % 3;
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        const int j1 = (j + 1) % 3, j2 = (j + 2) % 3;
        const int ia = 3 * i1 + j1, ib = 3 * i2 + j2, ic = 3 * i1 + j2, id = 3 * i2 + j1;
        const double Cr = (ar[ia] * ar[ib] - ai[ia] * ai[ib]) - (ar[ic] * ar[id] - ai[ic] * ai[id]);
        const double Ci = (ar[ia] * ai[ib] + ai[ia] * ar[ib]) - (ar[ic] * ai[id] + ai[ic] * ar[id]);
        if (i == 0) {
          detr += ar[j] * Cr - ai[j] * Ci;
          deti += ar[j] * Ci + ai[j] * Cr;
        }
        Tr += Cr * xr[3 * i + j] - Ci * xi[3 * i + j];
        Ti += Cr * xi[3 * i + j] + Ci * xr[3 * i + j];
      }
    }
    const double idd = (1.0 / 12.0) * fast_rcp(detr * detr + deti * deti);
    s_r = (Tr * detr + Ti * deti) * idd;
    s_i = (Ti * detr - Tr * deti) * idd;
  }

  // where a step of 6 h6 takes Q
  __device__ __forceinline__ void move(const double *Q, double h6, double q[3]) const
  {
#pragma unroll
    for (int j = 0; j < 3; ++j) q[j] = Q[j] + h6 * xq[j];
  }

  // dzQ and the amplitudes a[4] = (re, im) of a_P or of (a_SV, a_SH) over a step dt
  template <class ZP> __device__ __forceinline__ void step(double a[4], bool isS, double dt, const ZP &zp)
  {
    const double h2 = 0.5 * dt, h6 = dt / 6.0;
    double mr, mi;
    trace(zp, 0.5 * h6, mr, mi);
    double kr = sr, ki = si;  // the stages' derivatives for a = 1
    double gr = kr, gi = ki;
#pragma unroll
    for (int st = 1; st < 3; ++st) {
      const double ur = 1.0 + h2 * kr, ui = h2 * ki;
      kr = mr * ur - mi * ui;
      ki = mr * ui + mi * ur;
      gr += 2.0 * kr;
      gi += 2.0 * ki;
    }
#pragma unroll
    for (int o = 0; o < 9; ++o) {
      qr[o] += h6 * xr[o];
      qi[o] += h6 * xi[o];
    }
    trace(zp, 0.0, sr, si);
    const double ur = 1.0 + dt * kr, ui = dt * ki;
    gr = h6 * (gr + (sr * ur - si * ui));
    gi = h6 * (gi + (sr * ui + si * ur));
    const double a0 = a[0], a1 = a[1];
    a[0] += gr * a0 - gi * a1;
    a[1] += gr * a1 + gi * a0;
    if (isS) {
      const double a2 = a[2], a3 = a[3];
      a[2] += gr * a2 - gi * a3;
      a[3] += gr * a3 + gi * a2;
    }
  }

  __device__ __forceinline__ void store(double *y) const
  {
#pragma unroll
    for (int o = 0; o < 9; ++o) {
      y[IZQR + o] = qr[o];
      y[IZQI + o] = qi[o];
    }
  }
};

// dzP in the state y
struct ZpOf {
  const double *y;
  __device__ __forceinline__ double re(int o) const { return y[IZPR + o]; }
  __device__ __forceinline__ double im(int o) const { return y[IZPI + o]; }
  __device__ __forceinline__ void again() const {}
};

// dzP of the wavefront's beams in LDS, [9][64] of (re, im): the registers it would
// take through the steps are what keeps a second wavefront off the SIMD
struct ZpLds {
  double2 *lds;
  // returns whether all are finite
  __device__ __forceinline__ bool put(const double *y) const
  {
    bool finite = true;
#pragma unroll
    for (int o = 0; o < 9; ++o) {
      lds[o * 64 + threadIdx.x] = double2{y[IZPR + o], y[IZPI + o]};
      finite = finite && isfinite(y[IZPR + o]) && isfinite(y[IZPI + o]);
    }
    return finite;
  }
  __device__ __forceinline__ double re(int o) const { return lds[o * 64 + threadIdx.x].x; }
  __device__ __forceinline__ double im(int o) const { return lds[o * 64 + threadIdx.x].y; }
  // what follows reads LDS (and does not keep what was read or written before)
  __device__ __forceinline__ void again() const { asm volatile("" ::: "memory"); }
};

// One classic RK4 step of the whole state y where grad c = 0, in place.
template <int MK>
__device__ __forceinline__ void rk4_step_pc(const DevMedium &med, int sp, int layer, double sg, bool isS, double *y,
                                            double dt)
{
  double c, g[3], H6[6];
  medium_eval<MK>(med, sp, layer, y + IQ, c, g, H6);
  ConstRates r;
  const ZpOf zp{y};
  r.init(c, sg, y, zp);
  double q[3];
  r.move(y + IQ, dt / 6.0, q);
  r.step(y + IA, isS, dt, zp);
#pragma unroll
  for (int j = 0; j < 3; ++j) y[IQ + j] = q[j];
  r.store(y);
}

}  // namespace rk
}  // namespace fga
