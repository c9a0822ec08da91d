// Step 3 at scattered points (eq:FGA): receivers and seismograms.
//
// Beam-major layout.  A wavefront owns RW points (four, or eight with 32-bit
// sums) and walks a range of beams 64 at a time, one beam per lane, each lane
// holding its beam's emission record (Q, P 128/(pi eps), B = w e^{iS/eps} A) in
// registers and RW complex 3-vector sums.  The beam set is kept in Morton order
// of Q, so the 64 beams of a tile are close together: the tile's bounding box
// decides, per point, whether the tile is skipped, summed whole, or summed with
// a window test per beam.  A workgroup covers one sample, the points of two
// wavefronts and one beam range; workgroups sharing a beam range are dealt to
// one XCD so its records are read from HBM once.  After the beam range the sums
// are reduced over the lanes in a fixed order and written once per wavefront;
// per-workgroup partials are then reduced in a fixed order, so the sums are
// bitwise reproducible and need no atomics.
#include <algorithm>
#include <type_traits>

#include "device_common.h"
#include "fastmath.h"
#include "record.h"

namespace fga {
namespace {

// Two wavefronts per workgroup: a new workgroup needs a free wavefront slot
// on as many SIMDs as it has wavefronts, and the wavefronts of one finish at
// different times (their points skip different tiles), so smaller workgroups
// keep more of the four slots per SIMD busy (6 % faster than four, as fast
// as one; the sums are identical).
constexpr int WPW = 2;  // wavefronts per workgroup

// Workgroup -> (point group, beam range, sample).  Workgroups are dealt to
// the 8 XCDs round-robin by id; the point groups of one (beam range, sample)
// unit get consecutive ids on the same XCD, so that unit's records come from
// HBM once and are then served by that XCD's L2.
struct PointsWork {
  int pg;
  int64_t blk;
  int s;
  bool valid;
};
__device__ __forceinline__ PointsWork points_work(int64_t id, int groups, int64_t nblk, int m)
{
  PointsWork w;
  const int64_t xcd = id & 7, j = id >> 3;
  w.pg = (int)(j % groups);
  const int64_t unit = (j / groups) * 8 + xcd;
  w.blk = unit % nblk;
  w.s = (int)(unit / nblk);
  w.valid = w.s < m;
  return w;
}

// Summation modes: FP64 throughout; MIXED (FP32 exp / sin / cos, FP64
// products and sums); MIXED32 (FP32 exp / sin / cos, products and per-lane
// sums, the lane and block reductions in FP64).  FP64_WIDE: FP64 for windows
// so wide that exp(-3 tau) leaves the normal range; its magnitudes go on through
// the subnormal numbers to 0.
enum { SUM_FP64 = 0, SUM_MIXED = 1, SUM_MIXED32 = 2, SUM_FP64_WIDE = 3 };
constexpr double MAX_EXPONENT = 700.0;   // the magnitude stays normal up to here
constexpr double ZERO_EXPONENT = 800.0;  // and is 0 from here on (the smallest subnormal is e^-744.4)

// Points per wavefront.  FP64 sums take 12 registers a point: four points fit
// four wavefronts per SIMD (122 registers); eight fit three and lose what the
// halved record reads give (33 M beams, 256 points: 25.3 against 27.8 ms per
// launch).  With 32-bit sums eight points fit as well as four, and each tile's
// records are read half as often: a launch over 524 k beams, 8 samples and 385
// points takes 1.83 ms with eight and 2.35 ms with four.
constexpr int points_per_wave(int mode) { return mode == SUM_MIXED32 ? 8 : 4; }

// One term's complex factor exp(-|d|^2/(2 eps) + i P.d/eps), zero outside the
// window (in false); v: the phase in units of pi/128 (FP64 sums) or of 2 pi.  Mixed
// modes: the exponent and the phase (reduced to [-1/2, 1/2] revolutions) are
// formed in FP64, then exp2 / sin / cos run on the FP32 transcendental unit.
// FP64: the table-driven exponential.  nc + ncl: minus the exponent's scale for
// |d|^2 in the units that the exponential takes (ln2/256, or ln2 for the mixed
// modes, to which ncl is nothing).
// T is the accumulation type (float only for MIXED32).
template <int MODE, typename T>
__device__ __forceinline__ void point_term(const ScaledTables &tab, const ScaledCoeffs &K, const double (&dd)[3],
                                           const double (&pe)[3], double nc, double ncl, double tmax, bool in, T &er,
                                           T &ei)
{
  double t = dd[0] * dd[0] + dd[1] * dd[1] + dd[2] * dd[2];
  const double v = pe[0] * dd[0] + pe[1] * dd[1] + pe[2] * dd[2];
  if constexpr (MODE == SUM_MIXED || MODE == SUM_MIXED32) {
    const float r = (float)(v - rint(v));
    const float amp = in ? __builtin_amdgcn_exp2f((float)(t * nc)) : 0.0f;
    er = (T)(amp * __builtin_amdgcn_cosf(r));
    ei = (T)(amp * __builtin_amdgcn_sinf(r));
  } else {
    if constexpr (MODE == SUM_FP64_WIDE) t = fmin(t, tmax);
    cexp_scaled<MODE == SUM_FP64_WIDE>(tab, K, t, nc, ncl, v, in, er, ei);
  }
}

// u_c += (er + i ei) B_c, c = 0..2 (complex)
template <typename T>
__device__ __forceinline__ void accumulate_term(T (&u)[6], const T (&B)[6], T er, T ei)
{
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    u[2 * c] = fma(er, B[2 * c], fma(-ei, B[2 * c + 1], u[2 * c]));
    u[2 * c + 1] = fma(er, B[2 * c + 1], fma(ei, B[2 * c], u[2 * c + 1]));
  }
}

// Sums 24 values over the 64 lanes, halving the values held with the lanes
// summed: a swap of half-waves (then of 16-lane rows) leaves each half with one
// of two values' sums, so the first two levels take 18 additions and 36 swaps in
// place of 48 and 96, and the last four run within the rows by DPP.  Row g of
// the wavefront (lanes 16 g ..) ends with the totals of six values in all of its
// lanes: value 12 (g / 2) + 6 (g % 2) + i in out[i].
__device__ __forceinline__ double swap_add32(double a, double b)
{
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false,
                                                   false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false,
                                                   false);
  return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
__device__ __forceinline__ double swap_add16(double a, double b)
{
  const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false,
                                                   false);
  const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false,
                                                   false);
  return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
template <int ROR> __device__ __forceinline__ double row_add(double a)
{
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(a), 0x120 + ROR, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(a), 0x120 + ROR, 0xf, 0xf, true);
  return a + __hiloint2double(hi, lo);
}
__device__ __forceinline__ void reduce24(const double (&v)[24], double (&out)[6])
{
  double h[12];
#pragma unroll
  for (int i = 0; i < 12; ++i) h[i] = swap_add32(v[i], v[12 + i]);
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    double t = swap_add16(h[i], h[6 + i]);
    t = row_add<8>(t);
    t = row_add<4>(t);
    t = row_add<2>(t);
    out[i] = row_add<1>(t);
  }
}

// MODE: one of the SUM_ modes (the term and its sum as stated at point_term;
// MIXED32 holds the tile's records B and the sums in FP32).
//
// Bound by vector issue where tiles lie wholly in windows (busy in 82 % of the
// cycles on 66 k beams x 16 samples x 512 points): a term inside the window costs 49
// instructions, 12 of them the accumulation, and reads 24 bytes of tables.  What a
// term does not need is decided per tile by one lane each, 64 tiles at a time: a
// point whose window the tile's box misses is not visited, and one whose window holds
// the whole box is summed without the window test and mask.  With 63 instructions a
// term and the test on every beam the same launch took 1.36 ms; it takes 1.17 ms, and
// one over 4.1 M beams x 16 samples x 256 points 25.8 ms in place of 29.9.  There the
// vector unit is busy in 77 % of the cycles, 3.3 of four wavefronts are resident and
// wait 37 % of their time, on a tile's twelve record loads among others.
template <int MODE>
__global__ __launch_bounds__(64 * WPW) __attribute__((amdgpu_waves_per_eu(4))) void k_sum_points(PointsArgs a, int groups, int64_t nblk)
{
  using Acc = typename std::conditional<MODE == SUM_MIXED32, float, double>::type;
  constexpr int RW = points_per_wave(MODE), PG = RW * WPW;
  constexpr bool MIXED = MODE == SUM_MIXED || MODE == SUM_MIXED32;
  __shared__ ScaledTables tab;
  if constexpr (!MIXED) {
    fill_tables(tab);
    __syncthreads();
  }

  const PointsWork wk = points_work(blockIdx.x, groups, nblk, a.m);
  if (!wk.valid) return;  // whole workgroup: padding of the last XCD round
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform: points live in SGPRs
  const int64_t r0 = (int64_t)wk.pg * PG + w * RW;
  if (r0 >= a.n) return;  // no point of this wavefront exists (no barrier follows)
  double xr[RW][3];
#pragma unroll
  for (int k = 0; k < RW; ++k)
#pragma unroll
    for (int d = 0; d < 3; ++d) xr[k][d] = r0 + k < a.n ? a.xyz[3 * (r0 + k) + d] : 1.0e30;
  const double R = sqrt(2.0 * a.tau * a.eps);
  const double nc = a.nc, ncl = a.ncl;
  const double tmax = 2.0 * ZERO_EXPONENT * a.eps;
  const int64_t b0 = wk.blk * a.beams_per_block;
  const int64_t b1 = b0 + a.beams_per_block < a.nb ? b0 + a.beams_per_block : a.nb;
  const int s = wk.s;
  const double *E = a.emit + (int64_t)s * 12 * a.ld;
  const double *TB = a.tile_box + (int64_t)s * a.ntiles * 6;
  const ScaledCoeffs K;
  uint64_t cnt = 0;          // wave-uniform in-window count
  Acc u[RW][6];
#pragma unroll
  for (int k = 0; k < RW; ++k)
#pragma unroll
    for (int c = 0; c < 6; ++c) u[k][c] = (Acc)0;

  const int64_t tb0 = b0 >> 6, tb1 = (b1 + 63) >> 6;  // b0 is a multiple of 64
  for (int64_t base = tb0; base < tb1; base += 64) {
    // Lane = tile.  A tile whose box lies more than R away from the point along
    // some axis holds no term of it; one whose corners are all within R of it
    // holds only terms in its window (the rounded differences are monotone, so
    // both agree with the per-beam test).  A tile without live beams has an
    // empty box (+inf / -inf): neither.
    uint64_t reach[RW], whole[RW], any = 0;
    {
      const int64_t tt = base + lane;
      const bool ok = tt < tb1;
      double lo[3], hi[3];
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        lo[d] = ok ? TB[tt * 6 + d] : INFINITY;
        hi[d] = ok ? TB[tt * 6 + 3 + d] : -INFINITY;
      }
#pragma unroll
      for (int k = 0; k < RW; ++k) {
        bool rch = true, whl = true;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          const double dl = xr[k][d] - lo[d], dh = xr[k][d] - hi[d];
          rch = rch && !(-dl > R) && !(dh > R);
          whl = whl && fabs(dl) <= R && fabs(dh) <= R;
        }
        reach[k] = __ballot(rch);
        whole[k] = __ballot(whl);
        any |= reach[k];
      }
    }
    for (; any; any &= any - 1) {
      const int bit = __ffsll((long long)any) - 1;
      // records of the lane's beam: 12 loads off wave-uniform addresses, all in
      // flight together (the last lanes of a ragged tile read its last beam's)
      const int64_t t0 = (base + bit) << 6;
      const int left = (int)(b1 - t0 < 64 ? b1 - t0 : 64);
      const unsigned jl = lane < left ? lane : left - 1;
      const double *Et = E + t0;
      double q[3], pe[3], Bd[6];
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        q[d] = (Et + d * a.ld)[jl];
        pe[d] = (Et + (3 + d) * a.ld)[jl];
      }
#pragma unroll
      for (int c = 0; c < 6; ++c) Bd[c] = (Et + (6 + c) * a.ld)[jl];
      // dead beams and the ragged tail take a corner of the box as their place,
      // without phase or weight
      const bool mine = q[0] > -1.0e299 && lane < left;
      const uint64_t live = __ballot(mine);
      if (live != ~0ull) {
        const double *tb = TB + (base + bit) * 6;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          const double corner = tb[d];
          q[d] = mine ? q[d] : corner;
          pe[d] = mine ? pe[d] : 0.0;
        }
#pragma unroll
        for (int c = 0; c < 6; ++c) Bd[c] = mine ? Bd[c] : 0.0;
      }
      Acc B[6];
#pragma unroll
      for (int c = 0; c < 6; ++c) B[c] = (Acc)Bd[c];
      if constexpr (MIXED) {
#pragma unroll
        for (int d = 0; d < 3; ++d) pe[d] *= 1.0 / 256.0;  // exact: from units of pi/128 to revolutions
      }
#pragma unroll
      for (int k = 0; k < RW; ++k) {
        if (!((reach[k] >> bit) & 1)) continue;
        double dd[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) dd[d] = xr[k][d] - q[d];
        Acc er, ei;
        if ((whole[k] >> bit) & 1) {
          point_term<MODE>(tab, K, dd, pe, nc, ncl, tmax, true, er, ei);
          cnt += __popcll(live);
        } else {
          const bool in = (fabs(dd[0]) <= R) & (fabs(dd[1]) <= R) & (fabs(dd[2]) <= R);
          const uint64_t bal = __ballot(in) & live;
          if (!bal) continue;
          cnt += __popcll(bal);
          point_term<MODE>(tab, K, dd, pe, nc, ncl, tmax, in, er, ei);
        }
        accumulate_term(u[k], B, er, ei);
      }
    }
  }
  // lane reduction in FP64 in a fixed order, four points at a time
  const int g = lane >> 4, c = lane & 15;
#pragma unroll
  for (int h = 0; h < RW; h += 4) {
    double all[24], tot[6];
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int cc = 0; cc < 6; ++cc) all[k * 6 + cc] = (double)u[h + k][cc];
    reduce24(all, tot);
    // row g holds the six sums of point h + g; lane c of the row writes component c
    double v = tot[0];
#pragma unroll
    for (int i = 1; i < 6; ++i) v = c == i ? tot[i] : v;
    if (c < 6 && r0 + h + g < a.n) a.partial[((wk.blk * a.m + s) * a.n + r0 + h + g) * 6 + c] = v;
  }
  if (a.evals && lane == 0 && cnt) atomicAdd(a.evals + blockIdx.x % EVAL_SLOTS * EVAL_STRIDE, (unsigned long long)cnt);
}

// Per sample and 64-beam tile: bounding box of the live beams' centres Q
// (lo[3], hi[3]; an all-dead tile gets an empty box +inf / -inf).  Bound by the
// read of the centres: 4.1 M beams x 16 samples 322 us (4.9 TB/s; 691 with each of
// the six values reduced by itself through LDS shuffles).
__global__ __launch_bounds__(256) void k_tile_box(const double *__restrict__ emit, int64_t nb, int64_t ld, int64_t ntiles,
                                                  double *__restrict__ box)
{
  const int lane = threadIdx.x & 63;
  const int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int s = blockIdx.y;
  if (t >= ntiles) return;
  const double *E = emit + (int64_t)s * 12 * ld;
  const int64_t j = t * 64 + lane;
  double q[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) q[d] = E[d * ld + (j < nb ? j : 0)];
  // a dead record's q are all -1e300
  store_tile_box(q, j < nb && q[0] > -1.0e299, box + ((int64_t)s * ntiles + t) * 6);
}

// out[perm[r]][s0 + s][c] (+)= sum over blocks of partial[blk][s][r][c].
// A workgroup takes 64 consecutive outputs (one per lane, so every block row
// is read coalesced); its RG wavefronts sum the blocks b = w, w + RG, ... in
// order, and lane l of wavefront 0 adds the RG partial sums in order: a
// fixed summation order, bitwise reproducible, with RG times the parallelism
// of one thread per output.
constexpr int RG = 16;
__global__ __launch_bounds__(64 * RG) void k_reduce_points(const double *__restrict__ partial, int nblk, int m,
                                                           int64_t n, const int32_t *__restrict__ perm,
                                                           double *__restrict__ out, int64_t out_samples, int s0,
                                                           int accumulate)
{
  __shared__ double part[RG][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t id = (int64_t)blockIdx.x * 64 + lane;  // (s, r, c6)
  const int64_t total = (int64_t)m * n * 6;
  const int64_t row = (int64_t)m * n * 6;  // doubles per block
  double v = 0.0;
  if (id < total)
#pragma unroll 8  // loads of eight rows in flight, added in order (1498 rows of 78 outputs: 15 us one by one)
    for (int b = w; b < nblk; b += RG) v += partial[(int64_t)b * row + id];
  part[w][lane] = v;
  __syncthreads();
  if (w == 0 && id < total) {
    double t = 0.0;
#pragma unroll
    for (int k = 0; k < RG; ++k) t += part[k][lane];
    const int c6 = (int)(id % 6);
    const int64_t r = (id / 6) % n;
    const int s = (int)(id / (6 * n));
    const int64_t ro = perm ? perm[r] : r;
    double *o = out + (ro * out_samples + s0 + s) * 6 + c6;
    *o = accumulate ? *o + t : t;
  }
}

// A small sum in one launch, out[r][c] over all beams.  Each wavefront forms the
// records of one 64-beam tile and sums them at four points; the wavefronts of a
// workgroup take neighbouring tiles, whose sums are added in LDS; the last
// workgroup of a point group to finish adds the groups' sums in order, so the
// result does not depend on who is last.  arrived counts them modulo their number:
// a launch leaves a counter as it found it, and so do launches that overlap,
// since all that use one have the same number (small_counters).
// The sums pass the L2s of the eight XCDs by device-scope stores and loads: a
// device-scope fence in each workgroup writes a whole L2 back (204 workgroups:
// 21 us).
// Such a sum is bound by launches and latencies: 3000 beams at 65 points take
// 8.2 us a call, 13.8 as records, sums and their reduction in three launches.
constexpr int SMALL_TILES = 4, SMALL_POINTS = 4;
template <int MODE>
__global__ __launch_bounds__(64 * SMALL_TILES) void k_points_small(const double *__restrict__ F,
                                                                   const int32_t *__restrict__ I, int64_t cap,
                                                                   int64_t nb, double ieps, PointsArgs a, int groups,
                                                                   int nblk, double *__restrict__ out,
                                                                   unsigned *__restrict__ arrived)
{
  using Acc = typename std::conditional<MODE == SUM_MIXED32, float, double>::type;
  constexpr bool MIXED = MODE == SUM_MIXED || MODE == SUM_MIXED32;
  constexpr int OUT = 6 * SMALL_POINTS, SEG = 64 * SMALL_TILES / OUT;
  __shared__ ScaledTables tab;
  __shared__ double part[SEG > SMALL_TILES ? SEG : SMALL_TILES][OUT];
  __shared__ bool last;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int pg = blockIdx.x % groups, blk = blockIdx.x / groups;
  const int64_t i = ((int64_t)blk * SMALL_TILES + w) * 64 + lane;
  const int64_t ii = i < nb ? i : nb - 1;
  const bool alive = i < nb && (I[FGA_FLAGS * cap + ii] & FGA_FLAG_ALIVE);
  const bool isS = I[FGA_BRANCH * cap + ii] != 0;
  double y[rk::NS];
#pragma unroll
  for (int f = 0; f < rk::NS; ++f)
    if (f < rk::IZQR || f >= rk::IA) y[f] = F[f * cap + ii];
  const double e[3] = {F[(FGA_E + 0) * cap + ii], F[(FGA_E + 1) * cap + ii], F[(FGA_E + 2) * cap + ii]};
  const double wr = F[FGA_W_RE * cap + ii], wi = F[FGA_W_IM * cap + ii];
  const int64_t r0 = (int64_t)pg * SMALL_POINTS;
  double xr[SMALL_POINTS][3];
#pragma unroll
  for (int k = 0; k < SMALL_POINTS; ++k)
#pragma unroll
    for (int d = 0; d < 3; ++d) xr[k][d] = r0 + k < a.n ? a.xyz[3 * (r0 + k) + d] : 1.0e30;
  if constexpr (!MIXED) fill_tables(tab);
  double Wr, Wi, r[12];
  emit_weight(wr, wi, y[rk::IS], ieps, Wr, Wi);
  const bool mine = beam_record(y, e, Wr, Wi, isS, ieps, r) && alive;
  double q[3], pe[3];
  Acc B[6];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    q[d] = mine ? r[d] : 0.0;
    pe[d] = mine ? r[3 + d] : 0.0;
    if (MIXED) pe[d] *= 1.0 / 256.0;  // exact: from units of pi/128 to revolutions
  }
#pragma unroll
  for (int c = 0; c < 6; ++c) B[c] = (Acc)(mine ? r[6 + c] : 0.0);
  if constexpr (!MIXED) __syncthreads();
  const double R = sqrt(2.0 * a.tau * a.eps);
  const double nc = a.nc, ncl = a.ncl;
  const double tmax = 2.0 * ZERO_EXPONENT * a.eps;
  const ScaledCoeffs K;
  unsigned long long cnt = 0;
  double all[OUT], tot[6];
#pragma unroll
  for (int k = 0; k < SMALL_POINTS; ++k) {
    Acc u[6];
#pragma unroll
    for (int c = 0; c < 6; ++c) u[c] = (Acc)0;
    double dd[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) dd[d] = xr[k][d] - q[d];
    const bool in = mine & (fabs(dd[0]) <= R) & (fabs(dd[1]) <= R) & (fabs(dd[2]) <= R);
    const uint64_t bal = __ballot(in);
    if (bal) {
      cnt += __popcll(bal);
      Acc er, ei;
      point_term<MODE>(tab, K, dd, pe, nc, ncl, tmax, in, er, ei);
      accumulate_term(u, B, er, ei);
    }
#pragma unroll
    for (int c = 0; c < 6; ++c) all[k * 6 + c] = (double)u[c];
  }
  reduce24(all, tot);
  const int g = lane >> 4, c = lane & 15;
  double v = tot[0];
#pragma unroll
  for (int k = 1; k < 6; ++k) v = c == k ? tot[k] : v;
  if (c < 6) part[w][g * 6 + c] = v;
  if (a.evals && lane == 0 && cnt) atomicAdd(a.evals + blockIdx.x % EVAL_SLOTS * EVAL_STRIDE, cnt);
  __syncthreads();
  const int t = threadIdx.x;
  const bool valid = t < OUT && r0 + t / 6 < a.n;
  double *P = a.partial + r0 * 6 + t;
  if (valid) {
    double s = part[0][t];
#pragma unroll
    for (int k = 1; k < SMALL_TILES; ++k) s += part[k][t];
    if (nblk > 1) __hip_atomic_store(P + (int64_t)blk * a.n * 6, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else out[r0 * 6 + t] = s;
  }
  if (nblk == 1) return;
  // wavefront 0 wrote the row, past the L2s: it waits for those stores and counts
  if (w == 0) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0);
    if (t == 0)
      last = atomicInc(arrived + pg, (unsigned)nblk - 1) == (unsigned)nblk - 1;
  }
  __syncthreads();
  if (!last) return;
  const int seg = t / OUT, o = t % OUT;
  if (seg < SEG) {
    double s = 0.0;
    if (r0 + o / 6 < a.n) {
      double *Q = a.partial + r0 * 6 + o;
#pragma unroll 8
      for (int b = seg; b < nblk; b += SEG)
        s += __hip_atomic_load(Q + (int64_t)b * a.n * 6, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    part[seg][o] = s;
  }
  __syncthreads();
  if (valid) {
    double s = part[0][t];
#pragma unroll
    for (int k = 1; k < SEG; ++k) s += part[k][t];
    out[r0 * 6 + t] = s;
  }
}

}  // namespace

// The exponent -|d|^2/(2 eps) in units of ln2/256 (mixed modes: of ln2) is (nc + ncl) |d|^2.
static void exponent_scale(PointsArgs &a)
{
  const bool mixed = a.precision == FGA_FP32 || a.precision == FGA_FP32_ACC32;
  const long double c = -(mixed ? 1.0L : 256.0L) * 0.72134752044448170367996234050094L / (long double)a.eps;  // 1/(2 ln2)
  a.nc = (double)c;
  a.ncl = (double)(c - (long double)a.nc);
}

int points_small_blocks(int64_t nb, int64_t n)
{
  const int64_t blocks = (nb + 64 * SMALL_TILES - 1) / (64 * SMALL_TILES);
  const int64_t groups = (n + SMALL_POINTS - 1) / SMALL_POINTS;
  return nb > 0 && n > 0 && groups <= MAX_SMALL && blocks <= MAX_SMALL && blocks * groups <= MAX_SMALL ? (int)blocks : 0;
}

// The first of the counters of a sum of nblk rows.  Counters are by (nblk, point
// group): 1024 groups for each nblk below 32, and 32 above, as nblk times the
// groups is at most MAX_SMALL.
static int small_counters(int nblk) { return nblk < 32 ? nblk * MAX_SMALL : 32 * MAX_SMALL + nblk * 32; }
static_assert(MAX_SMALL == 1024 && SMALL_COUNTERS == 32 * MAX_SMALL + (MAX_SMALL + 1) * 32, "counters cover every sum");

hipError_t launch_points_small(const fga_beams *b, PointsArgs a, double *out, unsigned *counters, hipStream_t st)
{
  const int nblk = points_small_blocks(b->count, a.n);
  if (nblk == 0) return hipErrorInvalidValue;
  unsigned *arrived = counters + small_counters(nblk);
  exponent_scale(a);
  const int groups = (int)((a.n + SMALL_POINTS - 1) / SMALL_POINTS);
  ProfScope prof(FGA_K_SUM_POINTS, st);
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, (unsigned)(nblk * groups), 64 * SMALL_TILES, 0, st, b->f64, b->i32, b->capacity, b->count,
                       1.0 / a.eps, a, groups, nblk, out, arrived);
  };
  if (a.precision == FGA_FP32) go(k_points_small<SUM_MIXED>);
  else if (a.precision == FGA_FP32_ACC32) go(k_points_small<SUM_MIXED32>);
  else if (3.0 * a.tau > MAX_EXPONENT - 1.0) go(k_points_small<SUM_FP64_WIDE>);
  else go(k_points_small<SUM_FP64>);
  return hipGetLastError();
}

namespace {
constexpr int RANGE_GROUP = 4 * WPW;  // the FP64 sums' points per workgroup, for every mode
constexpr int64_t MANY_RANGES = 8192, FILL_RANGES = 2048;
constexpr int LONG_RANGE = 1024, MAX_RANGE = 8192;
}  // namespace

int points_beams_per_block(int64_t nb, int64_t n, int m, int least)
{
  // enough workgroups (about 8192) that the last partial round of resident
  // workgroups is a small fraction of the launch; ranges are whole 64-beam tiles.
  // Sums too small for 8192 ranges of 1024 beams take shorter ranges, down to
  // `least`, until the chip holds one workgroup per slot (about 2048): beyond
  // that a workgroup's tables and final reduction (about 500 instructions, against
  // 200 for a tile) outweigh what the extra workgroups give.
  const int64_t groups = (n + RANGE_GROUP - 1) / RANGE_GROUP;
  const int64_t pairs = nb * groups * (m > 0 ? m : 1);
  int64_t bpb = (pairs + MANY_RANGES - 1) / MANY_RANGES;
  if (bpb < LONG_RANGE) {
    const int64_t fill = (pairs + FILL_RANGES - 1) / FILL_RANGES;
    bpb = std::max(bpb, std::min<int64_t>(fill, LONG_RANGE));
  }
  bpb = (bpb + 63) / 64 * 64;
  if (bpb < least) bpb = least;
  if (bpb > MAX_RANGE) bpb = MAX_RANGE;
  return (int)bpb;
}

size_t points_partial_most(int64_t nb, int64_t n)
{
  // A sum takes at most F / groups + 1 rows of n points, so fewer than F groups' points
  // and a row, for F = FILL_RANGES (ranges of 64 beams or more) or F = MANY_RANGES
  // (LONG_RANGE or more), or ranges of MAX_RANGE.  The rows themselves go down where
  // the range grows by a tile (14,561 beams at 65 points: 228, 14,568: 114).
  auto rows = [nb](int64_t range) { return (nb + range - 1) / range; };
  const int64_t fill = std::min(rows(64) * n, FILL_RANGES * RANGE_GROUP + n);
  const int64_t many = std::min(rows(LONG_RANGE) * n, MANY_RANGES * RANGE_GROUP + n);
  return (size_t)6 * std::max(std::max(fill, many), rows(MAX_RANGE) * n);
}

hipError_t launch_sum_points(PointsArgs a, int *nblk_out, hipStream_t st)
{
  exponent_scale(a);
  const int64_t nblk = (a.nb + a.beams_per_block - 1) / a.beams_per_block;
  *nblk_out = (int)nblk;
  if (a.nb == 0 || a.n == 0 || a.m == 0) return hipSuccess;
  if (a.m > 65535) return hipErrorInvalidConfiguration;
  const int64_t ntiles = (a.nb + 63) / 64;
  if (ntiles != a.ntiles || a.ld < a.nb) return hipErrorInvalidValue;
  if (!a.boxes_ready) {
    hipLaunchKernelGGL(k_tile_box, dim3((unsigned)((ntiles + 3) / 4), (unsigned)a.m), 256, 0, st, a.emit, a.nb,
                       a.ld, ntiles, a.tile_box);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  const int mode = a.precision == FGA_FP32 ? SUM_MIXED : (a.precision == FGA_FP32_ACC32 ? SUM_MIXED32 : SUM_FP64);
  const int PG = points_per_wave(mode) * WPW;
  const int groups = (int)((a.n + PG - 1) / PG);
  const int64_t units = (nblk * a.m + 7) / 8 * 8;
  const int64_t nwg = units * groups;
  if (nwg > 0x7fffffff) return hipErrorInvalidConfiguration;
  ProfScope prof(FGA_K_SUM_POINTS, st);
  const bool wide = 3.0 * a.tau > MAX_EXPONENT - 1.0;  // an offset in the window has |d|^2 <= 3 R^2
  if (a.precision == FGA_FP32)
    hipLaunchKernelGGL(k_sum_points<SUM_MIXED>, dim3((unsigned)nwg), 64 * WPW, 0, st, a, groups, nblk);
  else if (a.precision == FGA_FP32_ACC32)
    hipLaunchKernelGGL(k_sum_points<SUM_MIXED32>, dim3((unsigned)nwg), 64 * WPW, 0, st, a, groups, nblk);
  else if (wide)
    hipLaunchKernelGGL(k_sum_points<SUM_FP64_WIDE>, dim3((unsigned)nwg), 64 * WPW, 0, st, a, groups, nblk);
  else
    hipLaunchKernelGGL(k_sum_points<SUM_FP64>, dim3((unsigned)nwg), 64 * WPW, 0, st, a, groups, nblk);
  return hipGetLastError();
}

hipError_t launch_reduce_points(const double *partial, int nblk, int m, int64_t n, const int32_t *perm, double *out,
                                int64_t out_samples, int s0, int accumulate, hipStream_t st)
{
  const int64_t total = (int64_t)m * n * 6;
  if (total == 0) return hipSuccess;
  hipLaunchKernelGGL(k_reduce_points, (unsigned)((total + 63) / 64), 64 * RG, 0, st, partial, nblk, m, n, perm, out,
                     out_samples, s0, accumulate);
  return hipGetLastError();
}

}  // namespace fga
