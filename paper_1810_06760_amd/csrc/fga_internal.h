// Internal declarations of the gfx950 FGA library (host launchers, device
// helpers, error reporting).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <string>

#include "fga.h"

namespace fga {

// ---------------------------------------------------------------- errors --
void set_error(const char *fmt, ...);
fga_status fail(fga_status st, const char *fmt, ...);

#define FGA_HIP(call)                                                                  \
  do {                                                                                 \
    hipError_t e_ = (call);                                                            \
    if (e_ != hipSuccess)                                                              \
      return ::fga::fail(FGA_EDEVICE, "%s failed: %s (%s:%d)", #call,                  \
                         hipGetErrorString(e_), __FILE__, __LINE__);                   \
  } while (0)

#define FGA_LAUNCH_CHECK()                                                             \
  do {                                                                                 \
    hipError_t e_ = hipGetLastError();                                                 \
    if (e_ != hipSuccess)                                                              \
      return ::fga::fail(FGA_EDEVICE, "kernel launch failed: %s (%s:%d)",              \
                         hipGetErrorString(e_), __FILE__, __LINE__);                   \
  } while (0)

// --------------------------------------------------------------- timing --
// Records a start event on construction and a stop event on destruction
// (around one kernel launch) when profiling is enabled.
struct ProfScope {
  int k;
  hipStream_t st;
  hipEvent_t a = nullptr;
  ProfScope(int kernel, hipStream_t s);
  ~ProfScope();
};

// ------------------------------------------------------------- workspace --
// Bump allocator over a caller workspace; every sub-buffer is 256-byte aligned.
struct Arena {
  char *base = nullptr;
  size_t size = 0, used = 0;
  Arena(void *b, size_t s) : base(static_cast<char *>(b)), size(s) {}
  template <class T> T *take(size_t n) {
    size_t off = (used + 255) & ~size_t(255);
    used = off + n * sizeof(T);
    if (base == nullptr || used > size) return nullptr;
    return reinterpret_cast<T *>(base + off);
  }
  static size_t need(size_t bytes) { return (bytes + 255) & ~size_t(255); }
};

// ----------------------------------------------------------- media (GPU) --
// Device view of a medium; passed by value to kernels.
struct DevMedium {
  int kind;
  double cp, cs;
  // grid
  const double *table;
  int n[3];
  double lo[3], ih[3];
  int64_t field_stride;   // doubles between the c_P and c_S tables
  int two_fields;
  double cs_ratio;
  int smooth;             // 1: cubic B-spline of the node values (coef), 0: trilinear records
  const double *coef;     // spline coefficients, c_P then c_S (coef_stride apart)
  int64_t coef_stride;
  // layered
  int geometry, nlayer;
  double bound[FGA_MAX_LAYERS];
  double cpl[FGA_MAX_LAYERS], csl[FGA_MAX_LAYERS], rhol[FGA_MAX_LAYERS];
  double gradl[FGA_MAX_LAYERS];  // relative speed gradient per layer (0: constant)
  double anom_amp[FGA_MAX_LAYERS], anom_beta[FGA_MAX_LAYERS];  // Gaussian anomaly per layer (0: none)
  double anom_x[FGA_MAX_LAYERS][3], anom_w[FGA_MAX_LAYERS][3];
  int any_grad;                  // some layer has a gradient: the general RK4 step
  double surface;                // > 0: traction-free surface closing the outermost region
};

fga_status make_dev_medium(const fga_medium *m, DevMedium *out);

// -------------------------------------------------------------- launchers --
hipError_t launch_grid_build(const int n[3], const double h[3], const double *c, double *table,
                             hipStream_t st);
hipError_t launch_spline_coefficients(const int n[3], const double *c, double *coef, hipStream_t st);

struct IntegrateArgs {
  double *f64;
  int32_t *i32;
  int64_t cap;
  int64_t beg, end;          // beams [beg, end)
  double dt;
  int nsteps;
  int step0;                 // global index of the first step of this launch
  int stride;                // emit after steps with (step+1) % stride == 0 (0: never)
  double *emit;              // [n_emit][12][end-beg]
  double eps_emit;
  double cutoff_abs;
  unsigned long long *counters;  // [0] beam-steps, [1] culled, [2] quarantined
  int s_vector;              // 1: frame-free S amplitudes (grid media)
  int64_t rec0, ld;          // slot of the first record, and the records' plane stride (emit is [n_emit][12][ld])
  // layered media: the beams are list[0, nlist), then the slots [beg, end)
  const int32_t *list;
  int64_t nlist;
  int64_t fresh_end;         // slots below it start the chunk anew: their flags hold no resume step
  int32_t *cross;            // slots that stopped at an interface, in no order
  unsigned long long *ncross;
};
// Layered media, within a chunk: the flags of a beam that stopped at an
// interface hold the step (of the chunk) that would leave the layer, those of a
// beam that comes from an interface the step it goes on with, from bit
// RESUME_SHIFT on; FLAG_BORN: the slot held no beam before that step.
enum { FLAG_BORN = 0x80, RESUME_SHIFT = 8, FLAG_MASK = 0x7f };
constexpr int MAX_LAYERED_CHUNK = 65535;  // samples that one launch of the sums takes
hipError_t launch_integrate(const DevMedium &m, const IntegrateArgs &a, hipStream_t st);

// A sum's term counter: workgroups add to one of EVAL_SLOTS words, a cache line
// apart, and the host adds them up.  One word takes an addition every 10 ns or so,
// which a small sum with many workgroups waited for (2190 beams at 349 points,
// FP32: 42 us with one word, 9.3 so).
constexpr int EVAL_SLOTS = 64, EVAL_STRIDE = 8, EVAL_WORDS = EVAL_SLOTS * EVAL_STRIDE;
struct PointsArgs {
  const double *emit;        // [m][12][ld] records
  int64_t nb;                // beams in the batch
  int64_t ld;                // plane stride of the records (>= nb)
  int m;                     // samples in the batch
  const double *xyz;         // [n][3]
  int64_t n;
  double eps, tau;
  double nc, ncl;            // set by the launch: minus the exponent's scale for |x - Q|^2, and what its rounding left
  double *partial;           // [nblk][m][n][6]
  int beams_per_block;
  unsigned long long *evals; // NULL, or EVAL_WORDS counters whose sum takes the in-window terms
  double *tile_box;          // scratch [m][ntiles][6], ntiles = ceil(nb / 64)
  int64_t ntiles;
  int boxes_ready;           // tile_box already holds the boxes (written with the records)
  int precision;             // FGA_FP64, or FGA_FP32: FP32 exp/sin/cos of FP64-reduced arguments
};
hipError_t launch_sum_points(PointsArgs a, int *nblk_out, hipStream_t st);
// beams walked by one point-sum workgroup for nb beams, n points and m samples
// per launch (a multiple of 64 in [least, 8192], least itself a multiple of 64
// up to 1024); partial holds ceil(nb / that) * m * n * 6 doubles
int points_beams_per_block(int64_t nb, int64_t n, int m, int least);
// The doubles of partial that sums of at most nb beams at at most n points take (m 1, least 64).
size_t points_partial_most(int64_t nb, int64_t n);
// A sum small enough for one launch: the rows of partial it takes, else 0.
// partial: [that][n][6]; counters: SMALL_COUNTERS words at 0, which are 0 again
// when no launch that uses them is on its way.
// Up to MAX_SMALL workgroups (256 beams by 4 points), about what the chip holds at
// once: 1016 (65,000 beams, 16 points) take 19.7 us against 35.3 in three launches,
// 1000 (10,000 by 100) 14.1 against 20.2.  Each four points form the records anew,
// so at 1975 (20,000 by 100) the two are even (22.8, 23.6), at 5925 it is 45 against 34.
constexpr int MAX_SMALL = 1024, SMALL_COUNTERS = 32 * MAX_SMALL + (MAX_SMALL + 1) * 32;
int points_small_blocks(int64_t nb, int64_t n);
hipError_t launch_points_small(const fga_beams *b, PointsArgs a, double *out, unsigned *counters, hipStream_t st);
// seis[perm[r]][s0 + s][c] (+)= sum_blk partial[blk][s][r][c]   (perm NULL: identity)
hipError_t launch_reduce_points(const double *partial, int nblk, int m, int64_t n, const int32_t *perm,
                                double *out, int64_t out_samples, int s0, int accumulate, hipStream_t st);
// Copies n points (device [n][3]) into xyz_sorted in Morton order of their
// positions and sets perm[k] = original index of sorted point k.  Synchronises st.
// xyz_sorted holds 3 n + 1 doubles (the last for the check of the points).
fga_status sort_points(const double *xyz, int64_t n, double *xyz_sorted, int32_t *perm, hipStream_t st);
constexpr int MAX_RANKED = 1024;
hipError_t launch_rank_points(const double *xyz, int n, double *sorted, int32_t *perm, int64_t *bad, hipStream_t st);
// rtp (device [n][3]: radius, longitude, latitude) -> xyz (device [n][3])
hipError_t launch_spherical_to_cartesian(const double *rtp, int64_t n, double *xyz, hipStream_t st);

// beams -> emission records (current state, one sample)
// box (may be NULL): also the tile boxes of the records, [ceil((end - beg) / 64)][6]
hipError_t launch_emit(const double *f64, const int32_t *i32, int64_t cap, int64_t beg, int64_t end,
                       double eps, double *emit, double *box, hipStream_t st);

// decomposition
struct DecompArgs {
  const fga_mesh *mesh;
  const double *Ft;          // complex [3][nz*npz][ny*npy][nx*npx] (see k_decompose)
  const double *Gt;          // NULL or complex [2][3][...] (FBI[g/c_P], FBI[g/c_S])
  double *f64;
  int32_t *i32;
  int64_t *lineage;
  int64_t cap;
};
fga_status decompose_impl(const DevMedium &dm, const fga_mesh *mesh, const double *f, const double *g,
                          fga_beams *beams, Arena &ar, hipStream_t st, bool size_only, size_t *need);

// Interface step of a layered medium: beams that would leave their layer in the
// step their flags name (flag FGA_FLAG_CROSS, state at the start of the step) are
// split into children (Snell, elastic boundary
// problem, Jacobian map) which finish the step in their own layers.
struct InterfaceArgs {
  double *f64;
  int32_t *i32;
  int64_t *lineage;
  int64_t cap;
  int64_t n;                 // beams in the set before the step
  const int32_t *list;       // [nlist] the crossing beams' slots, increasing
  int64_t nlist;
  double dt;
  int gen_max;
  double child_cut;
  int64_t *blk_extra;        // [ceil(nlist / 256)] extra slots per workgroup (pass 1 output)
  int64_t *blk_off;          // [ceil(nlist / 256)] exclusive scan of blk_extra (pass 2 input)
  unsigned long long *counters;  // [0] crossings, [1] children, [2] retired at the generation cap
  unsigned long long *ncross;    // pass 1 sets it to 0
};
// pass 1 (write = 0): per-workgroup counts of extra slots; pass 2 (write = 1):
// children written (first child in the parent's slot, the others appended at
// n + blk_off + rank)
hipError_t launch_interface(const DevMedium &m, const InterfaceArgs &a, int write, hipStream_t st);
// The *count slots in list in increasing order into sorted (tmp:
// cross_sort_bytes(cap) bytes); *ncross is their number.  Synchronises st.
size_t cross_sort_bytes(int64_t cap);
hipError_t sort_crossers(const int32_t *list, int32_t *sorted, const unsigned long long *count, void *tmp,
                         size_t tmp_bytes, hipStream_t st, int64_t *ncross);
// The resume steps out of the flags of [0, n) (after a failure within a chunk).
hipError_t launch_clear_resume(int32_t *flags, int64_t n, hipStream_t st);

// exclusive scan of n int64 values (one workgroup); total = sum
hipError_t launch_scan(const int64_t *in, int64_t *out, int64_t n, int64_t *total, hipStream_t st);

// Morton-order the beam set by Q (dead beams dropped; count updated; synchronises st).
// scratch (256-byte aligned, may be NULL): memory free during the call beside the
// arena's; the more planes it holds the fewer launches the re-ordering takes
// (least: the size is what the call takes at least)
fga_status sort_beams_spatial(fga_beams *b, Arena &ar, void *scratch, size_t scratch_bytes, hipStream_t st,
                              bool size_only, size_t *need, bool least = false);
// The least workspace fga_evolve takes; its query gives more for small sets.
size_t evolve_least_bytes(const fga_beams *beams, int nsteps, const fga_evolve_opts *opts, const fga_receivers *rec);

// stable compaction of the beam set by FLAGS & ALIVE
fga_status compact_beams(fga_beams *b, Arena &ar, hipStream_t st, bool size_only, size_t *need);
// counts for fga_beams_info into ctr[6] (device)
hipError_t launch_beams_info(const fga_beams *b, unsigned long long *ctr, hipStream_t st);

// grid summation
fga_status grid_sum_impl(const fga_beams *b, double eps, double tau, const int n[3], const double lo[3],
                         const double h[3], int precision, double *out, Arena &ar, hipStream_t st,
                         bool size_only, size_t *need, int64_t *evals, bool add = false);

}  // namespace fga
