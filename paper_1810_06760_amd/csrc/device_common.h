// Device-side helpers shared by the gfx950 kernels: medium evaluation and
// polarisation frames.
#pragma once

#include "fga_internal.h"

namespace fga {

// 1/x and 1/sqrt(x) of a normal positive x: the hardware's estimate (about 24
// bits) and one third-order step, e the residual: r + r (e + e^2), and
// y + y e (1/2 + 3/8 e).  Within two units in the last place in 4 and 6
// instructions; the library's division and square root take about 10 and 16 for
// the last half unit and for subnormals.  Against 80 bits nothing is further off
// for it: an S beam's record 1.2e-16 (1.3e-16 with the library's), a state after 28
// to 142 steps the same to 0.1 %.
__device__ __forceinline__ double fast_rcp(double x)
{
  const double r = __builtin_amdgcn_rcp(x);
  const double e = fma(-x, r, 1.0);
  return fma(r, fma(e, e, e), r);
}
__device__ __forceinline__ double fast_rsqrt(double x)
{
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * y, y, 1.0);
  return fma(y * e, fma(e, 0.375, 0.5), y);
}

// Medium kinds a kernel is specialised for.
// MK_GRID: trilinear node records; MK_GRID3: cubic B-spline of the node values.
enum { MK_HOMOG = 0, MK_GRID = 1, MK_LAYERED = 2, MK_GRID3 = 3 };

// Layered media: if Q lies outside layer L, the interface crossed and the
// layer beyond it (points on an interface count as inside).  Flat: interface
// i is z = bound[i] between layer i (below) and i+1; spherical: |x| = bound[i]
// between layer i (outside) and i+1 (inside).  The free surface, if any, is
// interface IFACE_SURFACE with the beam's own layer beyond it.
constexpr int IFACE_SURFACE = -1;
__device__ __forceinline__ bool layer_exit(const DevMedium &m, int L, const double Q[3], int &iface, int &newL)
{
  const int nl = m.nlayer;
  if (m.geometry == 1) {
    const double r = sqrt(Q[0] * Q[0] + Q[1] * Q[1] + Q[2] * Q[2]);
    if (L < nl - 1 && r < m.bound[L]) { iface = L; newL = L + 1; return true; }
    if (L > 0 && r > m.bound[L - 1]) { iface = L - 1; newL = L - 1; return true; }
    if (L == 0 && m.surface > 0.0 && r > m.surface) { iface = IFACE_SURFACE; newL = 0; return true; }
  } else {
    if (L < nl - 1 && Q[2] > m.bound[L]) { iface = L; newL = L + 1; return true; }
    if (L > 0 && Q[2] < m.bound[L - 1]) { iface = L - 1; newL = L - 1; return true; }
    if (L == nl - 1 && m.surface > 0.0 && Q[2] > m.surface) { iface = IFACE_SURFACE; newL = L; return true; }
  }
  return false;
}

// Larger of a and b over two halves (pairs of 16-lane rows): of two values each
// reduced half way, the lower halves (the even rows) hold a's and the upper b's.
__device__ __forceinline__ double swap_max32(double a, double b)
{
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false,
                                                   false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false,
                                                   false);
  return fmax(__hiloint2double((int)hi[0], (int)lo[0]), __hiloint2double((int)hi[1], (int)lo[1]));
}
__device__ __forceinline__ double swap_max16(double a, double b)
{
  const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false,
                                                   false);
  const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false,
                                                   false);
  return fmax(__hiloint2double((int)hi[0], (int)lo[0]), __hiloint2double((int)hi[1], (int)lo[1]));
}
template <int ROR> __device__ __forceinline__ double row_max(double a)
{
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(a), 0x120 + ROR, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(a), 0x120 + ROR, 0xf, 0xf, true);
  return fmax(a, __hiloint2double(hi, lo));
}

// The bounding box lo[3], hi[3] of the q of the wavefront's lanes with `in`, into
// box[6] (+inf / -inf without any).  All 64 lanes take part.
__device__ __forceinline__ void store_tile_box(const double q[3], bool in, double *__restrict__ box)
{
  double v[6];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    v[d] = in ? -q[d] : -INFINITY;
    v[3 + d] = in ? q[d] : -INFINITY;
  }
  const double w0 = swap_max32(v[0], v[1]), w1 = swap_max32(v[2], v[3]), w2 = swap_max32(v[4], v[5]);
  // rows of 16 lanes: v0 v2 v1 v3, and v4 v4 v5 v5
  double x0 = swap_max16(w0, w1), x1 = swap_max16(w2, w2);
  x0 = row_max<1>(row_max<2>(row_max<4>(row_max<8>(x0))));
  x1 = row_max<1>(row_max<2>(row_max<4>(row_max<8>(x1))));
  const int lane = threadIdx.x & 63, row = lane >> 4;
  const int k = (lane & 1) ? 4 + (row >> 1) : (row == 0 ? 0 : (row == 1 ? 2 : (row == 2 ? 1 : 3)));
  if ((lane & 15) < ((row & 1) ? 1 : 2)) box[k] = (lane & 1) ? x1 : (k < 3 ? -x0 : x0);
}

// Level (z or radius) of interface iface, or of the free surface.
__device__ __forceinline__ double iface_level(const DevMedium &m, int iface)
{
  return iface == IFACE_SURFACE ? m.surface : m.bound[iface];
}

// Speed of wave type sp (0 = P, 1 = S) at x: c, gradient g and Hessian H
// (xx, yy, zz, xy, xz, yz).  Grid media interpolate the ten precomputed node
// fields trilinearly (periodic); each node is one 128-byte record.
// Cubic media: a block of MEDBLK3^3 spline coefficients per node field held in LDS
// by a workgroup, the c_S field (two_fields) after the c_P field; rows and planes at
// odd strides, so that neighbouring cells' reads meet on few banks.
constexpr int MEDBLK3 = 16, MEDROW = 17, MEDPLANE = 277;
struct MedBlock {
  const double *lds;  // NULL: no block
  int o[3];
};

// Cell (node i0, periodic) and offsets t in it of a point of a grid medium.
__device__ __forceinline__ void grid_cell(const DevMedium &m, const double *x, int i0[3], double t[3])
{
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const double u = (x[d] - m.lo[d]) * m.ih[d];
    const double fl = floor(u);
    t[d] = u - fl;
    int ii = (int)fl;
    if (ii < 0 || ii >= m.n[d]) ii = ((ii % m.n[d]) + m.n[d]) % m.n[d];  // periodic (rare)
    i0[d] = ii;
  }
}

// The eight node records of the cell each lane's beam is in, held in LDS over a
// launch.  A beam stays in a cell for several steps (c dt is a fraction of h),
// so a stage's trilinear sum reads its forty 16-byte pieces from the lane's own
// column of rec (consecutive lanes, no bank conflicts, one address for all) and
// memory is touched only where a beam has moved on: then its forty pieces go from
// the table straight to LDS (no registers), requested as soon as the stage before
// knows where the ray goes, a whole stage's arithmetic ahead.
constexpr int CELL_PIECES = 40;  // 8 corners x 5 pairs of fields
static_assert(FGA_GRID_NODE_DOUBLES * sizeof(double) == 128, "node records are addressed by shifts");
typedef double v2d __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) v2d lds_v2d;
struct CellCache {
  // the wavefront's pieces, [CELL_PIECES][64] (the workgroup is one wavefront); a
  // constant address, so the LDS side of a request costs no vector instruction
  static __device__ __forceinline__ lds_v2d *rec()
  {
    __shared__ v2d pieces[CELL_PIECES * 64];
    return (lds_v2d *)pieces;
  }
  int cell[3];   // the cell the lane's column holds (-1: none)
  double t[3];   // offsets in it of the point asked for last
  template <int K> static __device__ __forceinline__ void piece(const char *p, lds_v2d *col)
  {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)p,
                                     (__attribute__((address_space(3))) void *)(col + 63 * K), 16, 16 * K, 0);
  }
  __device__ __forceinline__ void request(const DevMedium &m, int sp, const double *x)
  {
    int i0[3];
    grid_cell(m, x, i0, t);
    if (i0[0] == cell[0] && i0[1] == cell[1] && i0[2] == cell[2]) return;
    // pieces arrive in LDS on their own time, not in the order of the wavefront's LDS
    // instructions: what is still to be read of the column is waited for first
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    const char *tab = reinterpret_cast<const char *>(m.table + (sp && m.two_fields ? m.field_stride : 0));
    int i1[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      cell[d] = i0[d];
      i1[d] = i0[d] + 1 == m.n[d] ? 0 : i0[d] + 1;
    }
#pragma unroll
    for (int row = 0; row < 4; ++row) {
      const uint64_t r = ((uint64_t)(unsigned)((row & 2) ? i1[2] : i0[2]) * (unsigned)m.n[1] +
                          (unsigned)((row & 1) ? i1[1] : i0[1])) * (unsigned)m.n[0];
#pragma unroll
      for (int cx = 0; cx < 2; ++cx) {
        const int corner = 2 * row + cx;
        const char *p = tab + ((r + (unsigned)(cx ? i1[0] : i0[0])) << 7);  // 128-byte records
        // one address a corner: the pieces' offsets are the instruction's, which
        // also moves the LDS address by as much
        lds_v2d *col = rec() + 64 * 5 * corner;
        piece<0>(p, col);
        piece<1>(p, col);
        piece<2>(p, col);
        piece<3>(p, col);
        piece<4>(p, col);
      }
    }
  }
  // every request has arrived (vmcnt 0)
  __device__ __forceinline__ void wait() const
  {
    __builtin_amdgcn_s_waitcnt(0x0f70);
    asm volatile("" ::: "memory");
  }
  // the ten fields at the point asked for last
  __device__ __forceinline__ void fields(double v[10]) const
  {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int f = 0; f < 10; ++f) v[f] = 0.0;
#pragma unroll
    for (int corner = 0; corner < 8; ++corner) {
      const double w = ((corner & 1) ? t[0] : 1.0 - t[0]) * ((corner & 2) ? t[1] : 1.0 - t[1]) *
                       ((corner & 4) ? t[2] : 1.0 - t[2]);
#pragma unroll
      for (int k = 0; k < 5; ++k) {
        const v2d a = rec()[64 * (5 * corner + k) + lane];
        v[2 * k] += w * a.x;
        v[2 * k + 1] += w * a.y;
      }
    }
  }
};

// Cubic B-spline weights of the nodes i-1 .. i+2 at the fraction t of cell i,
// and their first and second derivatives in x (ih = 1/h).
__device__ __forceinline__ void bspline_weights(double t, double ih, double w[4], double d1[4], double d2[4])
{
  const double s = 1.0 - t, t2 = t * t, t3 = t2 * t, i6 = 1.0 / 6.0, ih2 = ih * ih;
  w[0] = s * s * s * i6;
  w[1] = (3.0 * t3 - 6.0 * t2 + 4.0) * i6;
  w[2] = (-3.0 * t3 + 3.0 * t2 + 3.0 * t + 1.0) * i6;
  w[3] = t3 * i6;
  d1[0] = -0.5 * s * s * ih;
  d1[1] = (1.5 * t2 - 2.0 * t) * ih;
  d1[2] = (-1.5 * t2 + t + 0.5) * ih;
  d1[3] = 0.5 * t2 * ih;
  d2[0] = s * ih2;
  d2[1] = (3.0 * t - 2.0) * ih2;
  d2[2] = (1.0 - 3.0 * t) * ih2;
  d2[3] = t * ih2;
}

// Tensor-product sum of the 4x4x4 coefficients ld(a, b, c) (x, y, z offsets)
// giving c, grad c and the Hessian (xx, yy, zz, xy, xz, yz) in v[10]: the x
// sums first (value, first, second derivative per row), then y, then z.  Two
// rows are read while the two before are summed (and kept there by the
// scheduling barriers): left alone the compiler reads each pair of
// coefficients where it is used, and one wavefront per SIMD waits for it
// (532 k beams x 16 steps of a point source 2.60 ms, so 2.13).
template <class Load>
__device__ __forceinline__ void bspline_sum(const double w[3][4], const double d1[3][4], const double d2[3][4],
                                            Load ld, double v[10])
{
#pragma unroll
  for (int k = 0; k < 10; ++k) v[k] = 0.0;
  double q[2][2][4];
  auto rows = [&](int g, double (&to)[2][4]) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int a = 0; a < 4; ++a) to[h][a] = ld(a, 2 * (g & 1) + h, g >> 1);
  };
  rows(0, q[0]);
  double y00 = 0.0, y10 = 0.0, y01 = 0.0, y20 = 0.0, y11 = 0.0, y02 = 0.0;
#pragma unroll
  for (int g = 0; g < 8; ++g) {
    if (g < 7) rows(g + 1, q[(g + 1) & 1]);
    __builtin_amdgcn_sched_barrier(0);
    if ((g & 1) == 0) y00 = y10 = y01 = y20 = y11 = y02 = 0.0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int b = 2 * (g & 1) + h;
      double x0 = 0.0, x1 = 0.0, x2 = 0.0;
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        x0 += w[0][a] * q[g & 1][h][a];
        x1 += d1[0][a] * q[g & 1][h][a];
        x2 += d2[0][a] * q[g & 1][h][a];
      }
      y00 += w[1][b] * x0;
      y10 += w[1][b] * x1;
      y20 += w[1][b] * x2;
      y01 += d1[1][b] * x0;
      y11 += d1[1][b] * x1;
      y02 += d2[1][b] * x0;
    }
    if (g & 1) {
      const int c = g >> 1;
      v[0] += w[2][c] * y00;
      v[1] += w[2][c] * y10;
      v[2] += w[2][c] * y01;
      v[3] += d1[2][c] * y00;
      v[4] += w[2][c] * y20;
      v[5] += w[2][c] * y02;
      v[6] += d2[2][c] * y00;
      v[7] += w[2][c] * y11;
      v[8] += d1[2][c] * y10;
      v[9] += d1[2][c] * y01;
    }
  }
}

// What the speed of one wave type in one layer is made of, and the levels the
// layer lies between (the tests of layer_exit).  The integrator reads them once a
// launch: from the medium's tables at every stage they cost the one or two
// wavefronts of a SIMD their latency (40 steps of 553 k beams in the crosswell
// model 2.85 ms against 2.74, 48 of 898 k in the layered Earth 1.98 against 1.83).
struct Layer {
  double c0, gm, al, be, x0[3], w[3];
  double lo, hi;
  bool sphere;
};
__device__ __forceinline__ Layer layer_of(const DevMedium &m, int sp, int L)
{
  Layer l;
  l.c0 = sp == 0 ? m.cpl[L] : m.csl[L];
  l.gm = m.gradl[L];
  l.al = m.anom_amp[L];
  l.be = m.anom_beta[L];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    l.x0[d] = m.anom_x[L][d];
    l.w[d] = m.anom_w[L][d];
  }
  l.sphere = m.geometry == 1;
  const int nl = m.nlayer;
  const double in = L < nl - 1 ? m.bound[L] : (l.sphere ? -INFINITY : (m.surface > 0.0 ? m.surface : INFINITY));
  const double out = L > 0 ? m.bound[L - 1] : (l.sphere ? (m.surface > 0.0 ? m.surface : INFINITY) : -INFINITY);
  l.lo = l.sphere ? in : out;
  l.hi = l.sphere ? out : in;
  return l;
}
__device__ __forceinline__ bool leaves_layer(const Layer &l, const double Q[3])
{
  const double v = l.sphere ? sqrt(Q[0] * Q[0] + Q[1] * Q[1] + Q[2] * Q[2]) : Q[2];
  return v < l.lo || v > l.hi;
}

__device__ __forceinline__ void layer_eval(const Layer &l, const double *x, double &c, double g[3], double H[6])
{
  g[0] = g[1] = g[2] = 0.0;
#pragma unroll
  for (int i = 0; i < 6; ++i) H[i] = 0.0;
  c = l.c0;
  if (l.gm != 0.0) {
    if (l.sphere) {
      // c = l.c0 (1 + l.gm r): grad c = l.c0 l.gm x/r, Hess c = l.c0 l.gm (I - x x^T/r^2)/r
      const double r = sqrt(x[0] * x[0] + x[1] * x[1] + x[2] * x[2]);
      const double k = l.c0 * l.gm / r;
      c = l.c0 * (1.0 + l.gm * r);
#pragma unroll
      for (int d = 0; d < 3; ++d) g[d] = k * x[d];
      const double ir2 = 1.0 / (r * r);
      H[0] = k * (1.0 - x[0] * x[0] * ir2);
      H[1] = k * (1.0 - x[1] * x[1] * ir2);
      H[2] = k * (1.0 - x[2] * x[2] * ir2);
      H[3] = -k * x[0] * x[1] * ir2;
      H[4] = -k * x[0] * x[2] * ir2;
      H[5] = -k * x[1] * x[2] * ir2;
    } else {
      c = l.c0 * (1.0 + l.gm * x[2]);
      g[2] = l.c0 * l.gm;
    }
  }
  const double al = l.al;
  if (al != 0.0) {
    // times f = 1 - al E, E = exp(-beta q), q = sum_d w_d d_d^2: grad f = 2 al beta E w d,
    // Hess f = al E (2 beta diag(w) - 4 beta^2 (w d)(w d)^T); the product rule for c f
    const double be = l.be;
    double wd[3], q = 0.0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const double dd = x[d] - l.x0[d];
      wd[d] = l.w[d] * dd;
      q += wd[d] * dd;
    }
    const double E = exp(-be * q);
    const double f = 1.0 - al * E;
    const double k1 = 2.0 * al * be * E, k2 = 4.0 * al * be * be * E;
    const double gf[3] = {k1 * wd[0], k1 * wd[1], k1 * wd[2]};
    const int ii[6] = {0, 1, 2, 0, 0, 1}, jj[6] = {0, 1, 2, 1, 2, 2};
#pragma unroll
    for (int t = 0; t < 6; ++t) {
      const int i = ii[t], j = jj[t];
      const double hf = (i == j ? al * E * 2.0 * be * l.w[i] : 0.0) - k2 * wd[i] * wd[j];
      H[t] = f * H[t] + g[i] * gf[j] + gf[i] * g[j] + c * hf;
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) g[d] = f * g[d] + c * gf[d];
    c *= f;
  }
}

template <int MK>
__device__ __forceinline__ void medium_eval(const DevMedium &m, int sp, int layer, const double *x,
                                            double &c, double g[3], double H[6], const MedBlock *blk = nullptr)
{
  if constexpr (MK == MK_HOMOG) {
    c = sp == 0 ? m.cp : m.cs;
    g[0] = g[1] = g[2] = 0.0;
#pragma unroll
    for (int i = 0; i < 6; ++i) H[i] = 0.0;
  } else if constexpr (MK == MK_LAYERED) {
    layer_eval(layer_of(m, sp, layer), x, c, g, H);
  } else if constexpr (MK == MK_GRID3) {
    const double *cf = m.coef;
    double scale = 1.0;
    if (sp) {
      if (m.two_fields) cf += m.coef_stride;
      else scale = m.cs_ratio;
    }
    int i0[3];
    double t[3], w[3][4], d1[3][4], d2[3][4];
    grid_cell(m, x, i0, t);
#pragma unroll
    for (int d = 0; d < 3; ++d) bspline_weights(t[d], m.ih[d], w[d], d1[d], d2[d]);
    // the 4x4x4 stencil from the LDS block when it lies in it for every lane
    bool inblk = blk != nullptr && blk->lds != nullptr;
    int l[3] = {0, 0, 0};
    if (inblk) {
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        int li = i0[d] - 1 - blk->o[d];
        if (li < 0) li += m.n[d];
        l[d] = li;
        inblk = inblk && li <= MEDBLK3 - 4;
      }
    }
    double v[10];
    if (__all(inblk)) {
      const double *b0 = blk->lds + ((sp && m.two_fields) ? MEDBLK3 * MEDPLANE : 0) + l[2] * MEDPLANE + l[1] * MEDROW + l[0];
      bspline_sum(w, d1, d2, [&](int ia, int ib, int ic) { return b0[ic * MEDPLANE + ib * MEDROW + ia]; }, v);
    } else {
      int ix[4], iy[4], iz[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        ix[k] = i0[0] - 1 + k;
        iy[k] = i0[1] - 1 + k;
        iz[k] = i0[2] - 1 + k;
        ix[k] += ix[k] < 0 ? m.n[0] : (ix[k] >= m.n[0] ? -m.n[0] : 0);
        iy[k] += iy[k] < 0 ? m.n[1] : (iy[k] >= m.n[1] ? -m.n[1] : 0);
        iz[k] += iz[k] < 0 ? m.n[2] : (iz[k] >= m.n[2] ? -m.n[2] : 0);
      }
      bspline_sum(w, d1, d2,
                  [&](int ia, int ib, int ic) { return cf[((size_t)iz[ic] * m.n[1] + iy[ib]) * m.n[0] + ix[ia]]; }, v);
    }
    c = scale * v[0];
#pragma unroll
    for (int k = 0; k < 3; ++k) g[k] = scale * v[1 + k];
#pragma unroll
    for (int k = 0; k < 6; ++k) H[k] = scale * v[4 + k];
  } else {
    const double *tab = m.table;
    double scale = 1.0;
    if (sp) {
      if (m.two_fields) tab += m.field_stride;
      else scale = m.cs_ratio;
    }
    int i0[3], i1[3];
    double t[3];
    grid_cell(m, x, i0, t);
#pragma unroll
    for (int d = 0; d < 3; ++d) i1[d] = i0[d] + 1 == m.n[d] ? 0 : i0[d] + 1;
    double v[10];
#pragma unroll
    for (int f = 0; f < 10; ++f) v[f] = 0.0;
#pragma unroll 2
    for (int corner = 0; corner < 8; ++corner) {
      const int ix = (corner & 1) ? i1[0] : i0[0];
      const int iy = (corner & 2) ? i1[1] : i0[1];
      const int iz = (corner & 4) ? i1[2] : i0[2];
      const double w = ((corner & 1) ? t[0] : 1.0 - t[0]) * ((corner & 2) ? t[1] : 1.0 - t[1]) *
                       ((corner & 4) ? t[2] : 1.0 - t[2]);
      const double2 *p = reinterpret_cast<const double2 *>(
          tab + (size_t)FGA_GRID_NODE_DOUBLES * (((size_t)iz * m.n[1] + iy) * m.n[0] + ix));
#pragma unroll
      for (int k = 0; k < 5; ++k) {
        const double2 a = p[k];
        v[2 * k] += w * a.x;
        v[2 * k + 1] += w * a.y;
      }
    }
    c = scale * v[0];
#pragma unroll
    for (int k = 0; k < 3; ++k) g[k] = scale * v[1 + k];
#pragma unroll
    for (int k = 0; k < 6; ++k) H[k] = scale * v[4 + k];
  }
}

// SH/SV frame: N_SH = (e x P)/|e x P|, N_SV = (P/|P|) x N_SH.
__device__ __forceinline__ void s_frame(const double P[3], const double e[3], double nsh[3], double nsv[3])
{
  double x0 = e[1] * P[2] - e[2] * P[1];
  double x1 = e[2] * P[0] - e[0] * P[2];
  double x2 = e[0] * P[1] - e[1] * P[0];
  double in = fast_rsqrt(x0 * x0 + x1 * x1 + x2 * x2);
  nsh[0] = x0 * in; nsh[1] = x1 * in; nsh[2] = x2 * in;
  double ip = fast_rsqrt(P[0] * P[0] + P[1] * P[1] + P[2] * P[2]);
  double p0 = P[0] * ip, p1 = P[1] * ip, p2 = P[2] * ip;
  nsv[0] = p1 * nsh[2] - p2 * nsh[1];
  nsv[1] = p2 * nsh[0] - p0 * nsh[2];
  nsv[2] = p0 * nsh[1] - p1 * nsh[0];
}

// Rank of this lane among the lanes of its 256-thread block with keep = true,
// and the block total.  Uses wavefront ballots; must be called by all threads.
__device__ __forceinline__ int block_rank(bool keep, int *total)
{
  __shared__ int wsum[4];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const unsigned long long m = __ballot(keep);
  const unsigned long long lt = lane ? (~0ull >> (64 - lane)) : 0ull;
  const int r = __popcll(m & lt);
  if (lane == 0) wsum[w] = __popcll(m);
  __syncthreads();
  int off = 0;
  for (int k = 0; k < w; ++k) off += wsum[k];
  *total = wsum[0] + wsum[1] + wsum[2] + wsum[3];
  __syncthreads();
  return off + r;
}

}  // namespace fga
