// What a receiver sum needs of a beam.
#pragma once

#include "fastmath.h"
#include "rk4.h"

namespace fga {

// Record of the state y: Q (3), P 128/(pi eps) (3), B = W A (3 complex),
// W = w e^{iS/eps} (S does not change, so W is formed once per launch).
// SV = 1: an S beam's state holds A itself (frame-free form).
// Returns whether all of it is finite: a beam with a non-finite record never
// enters a window, so no sum takes a NaN from it.
template <int SV = 0>
__device__ __forceinline__ bool beam_record(const double *y, const double e[3], double Wr, double Wi, bool isS,
                                            double ieps, double r[12])
{
  using namespace rk;
  double A[6];
  if (SV && isS) {
    A[0] = y[IA];
    A[1] = y[IA + 1];
    A[2] = y[IA + 2];
    A[3] = y[IA + 3];
    A[4] = y[IAZ];
    A[5] = y[IAZ + 1];
  } else if (!isS) {
    const double inp = fast_rsqrt(y[IP] * y[IP] + y[IP + 1] * y[IP + 1] + y[IP + 2] * y[IP + 2]);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const double nh = y[IP + c] * inp;
      A[2 * c] = y[IA] * nh;
      A[2 * c + 1] = y[IA + 1] * nh;
    }
  } else {
    double nsh[3], nsv[3];
    s_frame(y + IP, e, nsh, nsv);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      A[2 * c] = y[IA] * nsv[c] + y[IA + 2] * nsh[c];
      A[2 * c + 1] = y[IA + 1] * nsv[c] + y[IA + 3] * nsh[c];
    }
  }
  const double pscale = ieps * INV_PI_128;
#pragma unroll
  for (int f = 0; f < 3; ++f) {
    r[f] = y[IQ + f];
    r[3 + f] = y[IP + f] * pscale;  // the phase (P/eps).(x - Q) in units of pi/128
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    r[6 + 2 * c] = Wr * A[2 * c] - Wi * A[2 * c + 1];
    r[7 + 2 * c] = Wr * A[2 * c + 1] + Wi * A[2 * c];
  }
  bool finite = true;
#pragma unroll
  for (int f = 0; f < 12; ++f) finite = finite && isfinite(r[f]);
  return finite;
}

// W = w e^{iS/eps}
__device__ __forceinline__ void emit_weight(double wr, double wi, double S, double ieps, double &Wr, double &Wi)
{
  double sn, cs;
  sincos(S * ieps, &sn, &cs);
  Wr = wr * cs - wi * sn;
  Wi = wr * sn + wi * cs;
}

}  // namespace fga
