// One-thread-per-beam FP64 integrator of the FGA ODE system on gfx950.
//
// Each thread loads one beam's 47-double state from the structure-of-arrays
// planes (coalesced), advances it by `nsteps` classic RK4 steps held entirely
// in registers, optionally writes an emission record (Q, P, w e^{iS/eps} A)
// after every sample step for the receiver summation, and stores the state
// back (the right-hand side and the RK4 step are in rk4.h).  In layered media
// a beam stops at the step that would take its centre out of its layer, for the
// interface step (layered_body).
//
// The general step is bound by instruction issue at the one wavefront per SIMD
// its registers allow, so what it waits for is paid in full.  In the trilinear
// medium it waited for its gathers: with a block of nodes staged per workgroup
// and global memory for the rest, 4.1 M beams x 16 steps took 13.6 ms (9.7 with
// the gathers left out) and 66 k beams of a point source, which share no block,
// 517 us (182 without gathers).  With each lane's cell kept in LDS and the next
// one fetched a stage ahead (CellCache) they take 11.5 ms and 235 us.
#include "fastmath.h"
#include "record.h"

namespace fga {
namespace {

using namespace rk;

// Writes the record of the current state (beam_record) as beam j's; one with a
// non-finite entry is written as a dead one.  Returns whether it is a live one.
template <int SV = 0>
__device__ __forceinline__ bool emit_record(double *__restrict__ out, int64_t nb, int64_t j,
                                            const double *y, const double e[3], double Wr, double Wi,
                                            bool isS, double ieps)
{
  double r[12];
  const bool finite = beam_record<SV>(y, e, Wr, Wi, isS, ieps, r);
#pragma unroll
  for (int f = 0; f < 12; ++f) out[f * nb + j] = finite ? r[f] : (f < 3 ? -1.0e300 : 0.0);
  return finite;
}

__device__ __forceinline__ void emit_dead(double *__restrict__ out, int64_t nb, int64_t j)
{
  // dead beams sit at -1e300 (idle point lanes use +1e300), never in any window
#pragma unroll
  for (int f = 0; f < 3; ++f) out[f * nb + j] = -1.0e300;
#pragma unroll
  for (int f = 3; f < 12; ++f) out[f * nb + j] = 0.0;
}

// Whether the quantities a step's sample is formed from (Q, P and the
// amplitudes) are finite: 0 x is zero for a finite x and NaN otherwise.
template <int SV = 0>
__device__ __forceinline__ bool emitted_finite(const double *y)
{
  double z = 0.0;
#pragma unroll
  for (int d = 0; d < 3; ++d) z = fma(y[IQ + d], 0.0, fma(y[IP + d], 0.0, z));
#pragma unroll
  for (int t = 0; t < 4; ++t) z = fma(y[IA + t], 0.0, z);
  if (SV) z = fma(y[IAZ], 0.0, fma(y[IAZ + 1], 0.0, z));
  return z == 0.0;
}

// Frame-free S amplitudes: (a_SV, a_SH) in the beam's frame -> A in y, and back.
__device__ __forceinline__ void frame_to_vector(double *y, const double e[3])
{
  double nsh[3], nsv[3];
  s_frame(y + IP, e, nsh, nsv);
  const double a0r = y[IA], a0i = y[IA + 1], a1r = y[IA + 2], a1i = y[IA + 3];
  y[IA] = a0r * nsv[0] + a1r * nsh[0];
  y[IA + 1] = a0i * nsv[0] + a1i * nsh[0];
  y[IA + 2] = a0r * nsv[1] + a1r * nsh[1];
  y[IA + 3] = a0i * nsv[1] + a1i * nsh[1];
  y[IAZ] = a0r * nsv[2] + a1r * nsh[2];
  y[IAZ + 1] = a0i * nsv[2] + a1i * nsh[2];
}

// Back to the frame: the axis switched first if P has come within 10 degrees
// of it (the rule of reframe_s), then (a_SV, a_SH) = (A . N_SV, A . N_SH).
__device__ __forceinline__ void vector_to_frame(double *y, double e[3])
{
  const double np = sqrt(y[IP] * y[IP] + y[IP + 1] * y[IP + 1] + y[IP + 2] * y[IP + 2]);
  const double pe = y[IP] * e[0] + y[IP + 1] * e[1] + y[IP + 2] * e[2];
  if (fabs(pe) / np > COS10) {
    const bool was_z = e[2] != 0.0 && e[0] == 0.0 && e[1] == 0.0;
    e[0] = was_z ? 1.0 : 0.0;
    e[1] = 0.0;
    e[2] = was_z ? 0.0 : 1.0;
  }
  double nsh[3], nsv[3];
  s_frame(y + IP, e, nsh, nsv);
  const double Ar[3] = {y[IA], y[IA + 2], y[IAZ]}, Ai[3] = {y[IA + 1], y[IA + 3], y[IAZ + 1]};
  y[IA] = Ar[0] * nsv[0] + Ar[1] * nsv[1] + Ar[2] * nsv[2];
  y[IA + 1] = Ai[0] * nsv[0] + Ai[1] * nsv[1] + Ai[2] * nsv[2];
  y[IA + 2] = Ar[0] * nsh[0] + Ar[1] * nsh[1] + Ar[2] * nsh[2];
  y[IA + 3] = Ai[0] * nsh[0] + Ai[1] * nsh[1] + Ai[2] * nsh[2];
}

// Threads per workgroup: one wavefront, except in cubic media, where four share the
// block of coefficients.  (In the trilinear medium a wavefront's cells take 40 KB
// of LDS, so four fill a compute unit.)
template <int MK> constexpr int block_of() { return MK == MK_GRID3 ? 256 : 64; }

template <int MK, int SV = 0>
__device__ __forceinline__ void integrate_body(const DevMedium &med, const IntegrateArgs &a)
{
  const int64_t i = a.beg + (int64_t)blockIdx.x * block_of<MK>() + threadIdx.x;
  const bool active = i < a.end;
  unsigned long long steps_done = 0, culled = 0, quar = 0;
  MedBlock blk{nullptr, {0, 0, 0}};
  if constexpr (MK == MK_GRID3) {
    // The workgroup's beams are neighbours in Morton order, so the nodes they
    // interpolate from for the whole launch mostly lie in one small block around
    // them; that MEDBLK3^3 block of spline coefficients (of both node fields when
    // there are two) is staged in LDS once and the 4x4x4 stencils read it (stencils
    // outside it fall back to global memory).
    constexpr int B3 = MEDBLK3 * MEDBLK3 * MEDBLK3;
    __shared__ double lds_cf[2 * MEDBLK3 * MEDPLANE];
    __shared__ int bb[6];
    if (threadIdx.x < 3) {
      bb[threadIdx.x] = 0x7fffffff;
      bb[3 + threadIdx.x] = -0x7fffffff;
    }
    __syncthreads();
    if (active && (a.i32[FGA_FLAGS * a.cap + i] & FGA_FLAG_ALIVE)) {
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const double u = (a.f64[(FGA_Q + d) * a.cap + i] - med.lo[d]) * med.ih[d];
        const int cell = (int)fmax(fmin(floor(u), 1.0e9), -1.0e9);
        atomicMin(&bb[d], cell);
        atomicMax(&bb[3 + d], cell);
      }
    }
    __syncthreads();
    if (bb[0] <= bb[3]) {
      int o[3];
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const int c0 = bb[d] / 2 + bb[3 + d] / 2 - MEDBLK3 / 2 + 1;
        o[d] = ((c0 % med.n[d]) + med.n[d]) % med.n[d];
      }
      const int nf = med.two_fields ? 2 : 1;
      for (int idx = threadIdx.x; idx < nf * B3; idx += 256) {
        const int f = idx / B3, r = idx - f * B3;
        const int lx = r % MEDBLK3, ly = (r / MEDBLK3) % MEDBLK3, lz = r / (MEDBLK3 * MEDBLK3);
        const int nx = (o[0] + lx) % med.n[0], ny = (o[1] + ly) % med.n[1], nz = (o[2] + lz) % med.n[2];
        lds_cf[f * MEDBLK3 * MEDPLANE + lz * MEDPLANE + ly * MEDROW + lx] = med.coef[f * med.coef_stride + ((int64_t)nz * med.n[1] + ny) * med.n[0] + nx];
      }
      __syncthreads();
      blk.lds = lds_cf;
      blk.o[0] = o[0];
      blk.o[1] = o[1];
      blk.o[2] = o[2];
    }
  }
  if (active) {
    const int64_t cap = a.cap;
    const int64_t nb = a.end - a.beg;
    const int64_t j = i - a.beg;
    double *__restrict__ F = a.f64;
    int32_t flags = a.i32[FGA_FLAGS * cap + i];
    const int first_emit = a.stride ? a.step0 / a.stride : 0;
    if (!(flags & FGA_FLAG_ALIVE)) {
      if (a.stride)
        for (int s = 0; s < a.nsteps; ++s)
          if ((a.step0 + s + 1) % a.stride == 0)
            emit_dead(a.emit + (int64_t)((a.step0 + s + 1) / a.stride - 1 - first_emit) * 12 * nb, nb, j);
    } else {
      const int br = a.i32[FGA_BRANCH * cap + i];
      const double sg = (double)a.i32[FGA_SIGMA * cap + i];
      const int layer = a.i32[FGA_LAYER * cap + i];
      const int sp = br == 0 ? 0 : 1;
      const bool isS = br != 0;
      double y[nstate<SV>()];
#pragma unroll
      for (int f = 0; f < NS; ++f) y[f] = F[f * cap + i];
      double e[3] = {F[(FGA_E + 0) * cap + i], F[(FGA_E + 1) * cap + i], F[(FGA_E + 2) * cap + i]};
      if (SV) {
        y[nstate<SV>() - 2] = 0.0;
        y[nstate<SV>() - 1] = 0.0;
        if (isS) frame_to_vector(y, e);
      }
      const double wr = F[FGA_W_RE * cap + i], wi = F[FGA_W_IM * cap + i];
      const double dt = a.dt;
      const double ieps = 1.0 / a.eps_emit;
      const double wabs = sqrt(wr * wr + wi * wi);
      // After every step: a beam whose sampled quantities are no longer finite
      // is quarantined, and one with |w| max|a| below the cutoff is dropped;
      // either stops stepping and emits dead records from that step's sample on.
      CellCache cells{{-1, -1, -1}, {0.0, 0.0, 0.0}};
      bool live = isfinite(wabs) && isfinite(e[0]) && isfinite(e[1]) && isfinite(e[2]);
      if (!live) {
        flags = FGA_FLAG_QUARANTINED;
        quar = 1;
      }
      const double S = y[IS];
      const bool s_finite = isfinite(S);
      double Wr = 0.0, Wi = 0.0;
      if (a.stride) emit_weight(wr, wi, S, ieps, Wr, Wi);
      if constexpr (MK == MK_GRID) {
        if (live) cells.request(med, sp, y + IQ);
      }
      for (int s = 0; s < a.nsteps; ++s) {
        if (live) {
          if constexpr (MK == MK_GRID) rk4_step<MK, SV, true>(med, sp, layer, sg, isS, e, y, dt, nullptr, &cells);
          else rk4_step<MK, SV, true>(med, sp, layer, sg, isS, e, y, dt, &blk);
          if (isS && !SV) reframe_s(y, e);
          ++steps_done;
          if (!(emitted_finite<SV>(y) && s_finite)) {
            live = false;
            flags = FGA_FLAG_QUARANTINED;
            quar = 1;
          } else if (a.cutoff_abs > 0.0) {
            const double m0 = y[IA] * y[IA] + y[IA + 1] * y[IA + 1];
            double m1 = y[IA + 2] * y[IA + 2] + y[IA + 3] * y[IA + 3];
            // frame-free S: the magnitude of the polarisation vector
            const double mm = (SV && isS) ? m0 + m1 + y[nstate<SV>() - 2] * y[nstate<SV>() - 2] +
                                                y[nstate<SV>() - 1] * y[nstate<SV>() - 1]
                                          : (m0 > m1 ? m0 : m1);
            if (wabs * sqrt(mm) < a.cutoff_abs) {
              live = false;
              flags = 0;
              culled = 1;
            }
          }
        }
        if (a.stride && (a.step0 + s + 1) % a.stride == 0) {
          double *rec = a.emit + (int64_t)((a.step0 + s + 1) / a.stride - 1 - first_emit) * 12 * nb;
          if (live) emit_record<SV>(rec, nb, j, y, e, Wr, Wi, isS, ieps);
          else emit_dead(rec, nb, j);
        }
      }
      if (SV && isS) vector_to_frame(y, e);
      // the steps leave S as it was: not stored (the addresses are formed anew: kept from the loads they would take a
      // hundred registers through the steps)
      int64_t io = i;
      asm volatile("" : "+v"(io));
      if (live) {
        bool finite = true;
#pragma unroll
        for (int f = 0; f < NS; ++f) finite = finite && isfinite(y[f]);
        if (!finite) {
          flags = FGA_FLAG_QUARANTINED;
          quar = 1;
        }
      }
#pragma unroll
      for (int f = 0; f < NS; ++f)
        if (f != IS) F[f * cap + io] = y[f];
#pragma unroll
      for (int d = 0; d < 3; ++d) F[(FGA_E + d) * cap + io] = e[d];
      a.i32[FGA_FLAGS * cap + i] = flags;
    }
  }
  // wavefront-level reduction of the counters, one atomic per wavefront
  for (int off = 32; off > 0; off >>= 1) {
    steps_done += __shfl_down(steps_done, off);
    culled += __shfl_down(culled, off);
    quar += __shfl_down(quar, off);
  }
  if ((threadIdx.x & 63) == 0 && a.counters) {
    if (steps_done) atomicAdd(a.counters + 0, steps_done);
    if (culled) atomicAdd(a.counters + 1, culled);
    if (quar) atomicAdd(a.counters + 2, quar);
  }
}

template <int MK, int SV = 0>
__global__ __launch_bounds__(block_of<MK>()) void k_integrate(DevMedium med, IntegrateArgs a)
{
  integrate_body<MK, SV>(med, a);
}

// The steps of a chunk in a layered medium.  As in the other media the state stays
// in registers from step to step and each sample's record is written as it comes;
// a beam whose next step would end outside its layer stops there: its state at
// that step's start is stored, the flags get FGA_FLAG_CROSS and the step's number,
// and its slot joins the list of the interface kernels.  Their children come back
// in a launch over that list and the slots appended, and go on with the step after
// (their flags name it); a slot's samples before that are its parent's, or, where
// it was appended (FLAG_BORN), dead records.
//
// GRAD: some layer has a speed gradient (rays bend): the general RK4 step.  Else
// ConstRates, with two wavefronts per SIMD; a homogeneous medium is that without
// layers (LAYERS false).  One step per launch, with the state's 0.6 to
// 0.9 KB a beam to and from memory, a scan of all beams for those that stopped and
// the interface kernels each time, was bound by memory and launches: 898 k beams of
// a point source in a layered Earth took 410 us a step and sample beside the sums,
// chunks of 16 steps 66; 553 k beams in the crosswell model (GRAD) 190 and 77.
template <bool LAYERS, bool GRAD, int SV>
__device__ __forceinline__ void layered_body(const DevMedium &med, const IntegrateArgs &a)
{
  const int64_t idx = (int64_t)blockIdx.x * 64 + threadIdx.x;
  const int64_t cap = a.cap;
  double *__restrict__ F = a.f64;
  const bool active = idx < a.nlist + (a.end - a.beg);
  const int64_t i = !active ? 0 : (LAYERS && idx < a.nlist ? (int64_t)a.list[idx] : a.beg + (idx - a.nlist));
  unsigned long long steps_done = 0, culled = 0, quar = 0;
  int32_t flags = active ? a.i32[FGA_FLAGS * cap + i] : 0;
  const bool fresh = !LAYERS || (idx >= a.nlist && i < a.fresh_end);
  const int resume = fresh ? 0 : flags >> RESUME_SHIFT;
  // the first step whose sample this launch writes, and the step whose end the
  // state is at (if of this chunk)
  const int first = (fresh || (flags & FLAG_BORN)) ? 0 : (resume > 0 ? resume - 1 : 0);
  const int born = fresh ? 0 : resume - 1;
  flags &= FGA_FLAG_ALIVE | FGA_FLAG_QUARANTINED;
  const bool alive = active && (flags & FGA_FLAG_ALIVE);
  const int first_emit = a.stride ? a.step0 / a.stride : 0;
  const double dt = a.dt;
  const double ieps = 1.0 / a.eps_emit;
  __shared__ double2 zp_lds[GRAD ? 1 : 9 * 64];
  const ZpLds zp{zp_lds};
  ConstRates rates;
  Layer lay;
  int layer = 0, sp = 0;
  bool isS = false, live = alive, cross = false, s_finite = false, zp_finite = true;
  double sg = 0.0, wabs = 0.0, Wr = 0.0, Wi = 0.0;
  double y[nstate<SV>()], e[3];
  if (alive) {
    const int br = a.i32[FGA_BRANCH * cap + i];
    sg = (double)a.i32[FGA_SIGMA * cap + i];
    layer = a.i32[FGA_LAYER * cap + i];
    sp = br == 0 ? 0 : 1;
    isS = br != 0;
#pragma unroll
    for (int f = 0; f < NS; ++f) y[f] = F[f * cap + i];
#pragma unroll
    for (int d = 0; d < 3; ++d) e[d] = F[(FGA_E + d) * cap + i];
    if (SV) {
      y[nstate<SV>() - 2] = 0.0;
      y[nstate<SV>() - 1] = 0.0;
    }
    const double wr = F[FGA_W_RE * cap + i], wi = F[FGA_W_IM * cap + i];
    wabs = sqrt(wr * wr + wi * wi);
    const double S = y[IS];
    s_finite = isfinite(S);
    if (a.stride) emit_weight(wr, wi, S, ieps, Wr, Wi);
    if (!LAYERS && !(isfinite(wabs) && isfinite(e[0]) && isfinite(e[1]) && isfinite(e[2]))) {
      live = false;
      flags = FGA_FLAG_QUARANTINED;
      quar = 1;
    }
    if (LAYERS) lay = layer_of(med, sp, layer);
    if constexpr (!GRAD) {
      zp_finite = zp.put(y);
      rates.init(LAYERS ? lay.c0 : (isS ? med.cs : med.cp), sg, y, zp);
    }
  }
  for (int s = 0; s < a.nsteps; ++s) {
    if (s >= resume && live && !cross) {
      if constexpr (GRAD) {
        double A0[4];
        if (SV) {
#pragma unroll
          for (int t = 0; t < 4; ++t) A0[t] = y[IA + t];
          if (isS) frame_to_vector(y, e);
        }
        cross = rk4_step<MK_LAYERED, SV, true, true>(med, sp, layer, sg, isS, e, y, dt, nullptr, nullptr, &lay);
        if (SV && cross) {
#pragma unroll
          for (int t = 0; t < 4; ++t) y[IA + t] = A0[t];
        } else if (isS && SV) {
          vector_to_frame(y, e);
        } else if (isS && !cross) {
          reframe_s(y, e);
        }
      } else {
        double q[3];
        rates.move(y + IQ, dt / 6.0, q);
        if (LAYERS) cross = leaves_layer(lay, q);
        if (!cross) {
#pragma unroll
          for (int d = 0; d < 3; ++d) y[IQ + d] = q[d];
          rates.step(y + IA, isS, dt, zp);
          if (isS) reframe_s(y, e);
        }
      }
      ++steps_done;
      if (cross) {
        flags = FGA_FLAG_ALIVE | FGA_FLAG_CROSS | (s << RESUME_SHIFT);
      } else if (!(emitted_finite(y) && s_finite)) {
        live = false;
        flags = FGA_FLAG_QUARANTINED;
        quar = 1;
      } else if (a.cutoff_abs > 0.0) {
        const double m0 = y[IA] * y[IA] + y[IA + 1] * y[IA + 1];
        const double m1 = y[IA + 2] * y[IA + 2] + y[IA + 3] * y[IA + 3];
        if (wabs * sqrt(m0 > m1 ? m0 : m1) < a.cutoff_abs) {
          live = false;
          flags = 0;
          culled = 1;
        }
      }
    }
    if (a.stride && active && s >= first && !cross && (a.step0 + s + 1) % a.stride == 0) {
      double *rec = a.emit + (int64_t)((a.step0 + s + 1) / a.stride - 1 - first_emit) * 12 * a.ld;
      if (live && s >= born) emit_record(rec, a.ld, i - a.rec0, y, e, Wr, Wi, isS, ieps);
      else emit_dead(rec, a.ld, i - a.rec0);
    }
  }
  if (alive) {
    if constexpr (!GRAD) rates.store(y);
    if (live && !cross) {
      bool finite = zp_finite && s_finite;
#pragma unroll
      for (int f = 0; f < NS; ++f)
        if (f != IS && (GRAD || f < IZPR || f >= IZPR + 18)) finite = finite && isfinite(y[f]);
      if (!finite) {
        flags = FGA_FLAG_QUARANTINED;
        quar = 1;
      }
    }
    // the addresses are formed anew: kept from the loads they would take a
    // hundred registers through the steps
    int64_t io = i;
    asm volatile("" : "+v"(io));
#pragma unroll
    for (int f = 0; f < NS; ++f)
      if (f != IS && (GRAD || !((f >= IP && f < IP + 3) || (f >= IZPR && f < IZPR + 18)))) F[f * cap + io] = y[f];
#pragma unroll
    for (int d = 0; d < 3; ++d) F[(FGA_E + d) * cap + io] = e[d];
  }
  if (active) a.i32[FGA_FLAGS * cap + i] = flags;
  const int lane = threadIdx.x & 63;
  const unsigned long long stopped = __ballot(cross);
  if (stopped) {
    unsigned long long base = 0;
    if (lane == 0) base = atomicAdd(a.ncross, (unsigned long long)__popcll(stopped));
    base = __shfl(base, 0);
    if (cross) a.cross[base + __popcll(stopped & ((1ull << lane) - 1))] = (int32_t)i;
  }
  for (int off = 32; off > 0; off >>= 1) {
    steps_done += __shfl_down(steps_done, off);
    culled += __shfl_down(culled, off);
    quar += __shfl_down(quar, off);
  }
  if (lane == 0 && a.counters) {
    if (steps_done) atomicAdd(a.counters + 0, steps_done);
    if (culled) atomicAdd(a.counters + 1, culled);
    if (quar) atomicAdd(a.counters + 2, quar);
  }
}

__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_layered(DevMedium med,
                                                                                           IntegrateArgs a)
{
  layered_body<true, false, 0>(med, a);
}

template <int SV>
__global__ __launch_bounds__(64) void k_layered_grad(DevMedium med, IntegrateArgs a)
{
  layered_body<true, true, SV>(med, a);
}

// A homogeneous medium: the same body without layers to leave.
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_homog(DevMedium med, IntegrateArgs a)
{
  layered_body<false, false, 0>(med, a);
}

// Emission records of the current state (no stepping), e.g. for t = 0
// samples.  With box: each wavefront is one 64-beam tile of the records and
// also writes that tile's bounding box of the live centres Q (lo[3], hi[3];
// +inf / -inf when no beam of the tile is live), as k_tile_box would from
// the records.
__global__ __launch_bounds__(256) void k_emit(const double *__restrict__ F, const int32_t *__restrict__ I,
                                              int64_t cap, int64_t beg, int64_t end, double ieps,
                                              double *__restrict__ out, double *__restrict__ box)
{
  const int64_t i = beg + (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t nb = end - beg, j = i - beg;
  double q[3] = {0.0, 0.0, 0.0};
  bool in = false;
  if (i < end) {
    if (!(I[FGA_FLAGS * cap + i] & FGA_FLAG_ALIVE)) {
      emit_dead(out, nb, j);
    } else {
      double y[NS];
#pragma unroll
      for (int f = 0; f < NS; ++f) y[f] = F[f * cap + i];
      const double e[3] = {F[(FGA_E + 0) * cap + i], F[(FGA_E + 1) * cap + i], F[(FGA_E + 2) * cap + i]};
      double Wr, Wi;
      emit_weight(F[FGA_W_RE * cap + i], F[FGA_W_IM * cap + i], y[IS], ieps, Wr, Wi);
      in = emit_record(out, nb, j, y, e, Wr, Wi, I[FGA_BRANCH * cap + i] != 0, ieps);
#pragma unroll
      for (int d = 0; d < 3; ++d) q[d] = y[IQ + d];
    }
  }
  const int64_t t0 = j - (threadIdx.x & 63);  // this wavefront's tile
  if (box && t0 < nb) store_tile_box(q, in, box + (t0 >> 6) * 6);
}

}  // namespace

hipError_t launch_integrate(const DevMedium &m, const IntegrateArgs &a, hipStream_t st)
{
  const int64_t n = a.end - a.beg;
  if (n + a.nlist <= 0) return hipSuccess;
  const unsigned blocks = (unsigned)((n + 255) / 256);
  const unsigned waves = (unsigned)((n + a.nlist + 63) / 64);
  ProfScope prof(FGA_K_INTEGRATE, st);
  switch (m.kind) {
  case FGA_MEDIUM_HOMOGENEOUS: hipLaunchKernelGGL(k_homog, waves, 64, 0, st, m, a); break;
  case FGA_MEDIUM_GRID:
    // frame-free S amplitudes: a variant of the grid-medium kernels (in a
    // homogeneous medium P is constant and the two forms are one)
    if (m.smooth && a.s_vector) hipLaunchKernelGGL((k_integrate<MK_GRID3, 1>), blocks, 256, 0, st, m, a);
    else if (m.smooth) hipLaunchKernelGGL(k_integrate<MK_GRID3>, blocks, 256, 0, st, m, a);
    else if (a.s_vector) hipLaunchKernelGGL((k_integrate<MK_GRID, 1>), waves, 64, 0, st, m, a);
    else hipLaunchKernelGGL(k_integrate<MK_GRID>, waves, 64, 0, st, m, a);
    break;
  default:
    if (a.nsteps > MAX_LAYERED_CHUNK) return hipErrorInvalidValue;
    if (m.any_grad && a.s_vector) hipLaunchKernelGGL(k_layered_grad<1>, waves, 64, 0, st, m, a);
    else if (m.any_grad) hipLaunchKernelGGL(k_layered_grad<0>, waves, 64, 0, st, m, a);
    else hipLaunchKernelGGL(k_layered, waves, 64, 0, st, m, a);
    break;
  }
  return hipGetLastError();
}

hipError_t launch_emit(const double *f64, const int32_t *i32, int64_t cap, int64_t beg, int64_t end,
                       double eps, double *emit, double *box, hipStream_t st)
{
  const int64_t n = end - beg;
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_emit, (unsigned)((n + 255) / 256), 256, 0, st, f64, i32, cap, beg, end, 1.0 / eps, emit,
                     box);
  return hipGetLastError();
}

}  // namespace fga
