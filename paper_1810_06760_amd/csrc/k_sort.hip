// Spatial ordering of the beam set.
//
// Beams are independent, so their order in memory is free.  Sorting them
// along a Morton curve of their centres Q puts beams that share medium cells
// into the same wavefronts and workgroups: the trilinear gathers of the
// integrator then hit the same cache lines, and the receiver sums see
// compact beam tiles.  Dead beams sort last and are dropped, which is also
// the compaction step.  The radix sort is stable, so the order (and every
// result) is reproducible run to run.
#include <hipcub/hipcub.hpp>

#include "device_common.h"

namespace fga {
namespace {

__global__ __launch_bounds__(256) void k_bbox_partial(const double *__restrict__ F, const int32_t *__restrict__ I,
                                                      int64_t cap, int64_t n, double *__restrict__ part)
{
  __shared__ double red[6][4];
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  double b[6] = {HUGE_VAL, HUGE_VAL, HUGE_VAL, -HUGE_VAL, -HUGE_VAL, -HUGE_VAL};
  if (i < n && (I[FGA_FLAGS * cap + i] & FGA_FLAG_ALIVE)) {
    for (int d = 0; d < 3; ++d) {
      const double q = F[(FGA_Q + d) * cap + i];
      b[d] = q;
      b[3 + d] = q;
    }
  }
  for (int off = 32; off > 0; off >>= 1)
    for (int d = 0; d < 3; ++d) {
      b[d] = fmin(b[d], __shfl_xor(b[d], off));
      b[3 + d] = fmax(b[3 + d], __shfl_xor(b[3 + d], off));
    }
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0)
    for (int k = 0; k < 6; ++k) red[k][w] = b[k];
  __syncthreads();
  if (threadIdx.x < 6) {
    const int k = threadIdx.x;
    double v = red[k][0];
    for (int ww = 1; ww < 4; ++ww) v = k < 3 ? fmin(v, red[k][ww]) : fmax(v, red[k][ww]);
    part[(int64_t)blockIdx.x * 6 + k] = v;
  }
}

__global__ __launch_bounds__(256) void k_bbox_final(const double *__restrict__ part, int64_t nblk,
                                                    double *__restrict__ box)
{
  __shared__ double red[6][256];
  double b[6] = {HUGE_VAL, HUGE_VAL, HUGE_VAL, -HUGE_VAL, -HUGE_VAL, -HUGE_VAL};
  for (int64_t k = threadIdx.x; k < nblk; k += 256)
    for (int d = 0; d < 6; ++d) b[d] = d < 3 ? fmin(b[d], part[k * 6 + d]) : fmax(b[d], part[k * 6 + d]);
  for (int d = 0; d < 6; ++d) red[d][threadIdx.x] = b[d];
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s)
      for (int d = 0; d < 6; ++d)
        red[d][threadIdx.x] = d < 3 ? fmin(red[d][threadIdx.x], red[d][threadIdx.x + s])
                                    : fmax(red[d][threadIdx.x], red[d][threadIdx.x + s]);
    __syncthreads();
  }
  if (threadIdx.x < 6) box[threadIdx.x] = red[threadIdx.x][0];
}

__device__ __forceinline__ uint32_t spread3(uint32_t v)
{
  v &= 0x3ff;
  v = (v | (v << 16)) & 0x030000ff;
  v = (v | (v << 8)) & 0x0300f00f;
  v = (v | (v << 4)) & 0x030c30c3;
  v = (v | (v << 2)) & 0x09249249;
  return v;
}

__global__ __launch_bounds__(256) void k_morton(const double *__restrict__ F, const int32_t *__restrict__ I,
                                                int64_t cap, int64_t n, const double *__restrict__ box,
                                                uint32_t *__restrict__ keys, int32_t *__restrict__ vals)
{
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  uint32_t key = 0xffffffffu;
  if (I[FGA_FLAGS * cap + i] & FGA_FLAG_ALIVE) {
    uint32_t c[3];
    for (int d = 0; d < 3; ++d) {
      const double span = box[3 + d] - box[d];
      double u = span > 0 ? (F[(FGA_Q + d) * cap + i] - box[d]) / span * 1023.0 : 0.0;
      u = u < 0.0 ? 0.0 : (u > 1023.0 ? 1023.0 : u);
      c[d] = (uint32_t)u;
    }
    key = spread3(c[0]) | (spread3(c[1]) << 1) | (spread3(c[2]) << 2);
  }
  keys[i] = key;
  vals[i] = (int32_t)i;
}

__global__ __launch_bounds__(256) void k_count_alive(const uint32_t *__restrict__ keys, int64_t n,
                                                     int64_t *__restrict__ out)
{
  // keys are sorted: the first dead key marks the end of the live beams
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const bool live = keys[i] != 0xffffffffu;
  const bool next_dead = i + 1 == n || keys[i + 1] == 0xffffffffu;
  if (i == 0 && !live) *out = 0;
  if (live && next_dead) *out = i + 1;
}

// All planes of a beam set by one number: the FGA_NF64 double planes, the
// lineage, then the FGA_NI32 int32 planes.
constexpr int NPLANE = FGA_NF64 + 1 + FGA_NI32;
constexpr int NWIDE = FGA_NF64 + 1;  // planes of 8-byte entries

struct PlaneSet {
  double *f64;
  int32_t *i32;
  int64_t *lineage;
  int64_t cap;
};

// Scratch slots of one plane each (8-byte stride), in two separate regions.
struct Slots {
  uint64_t *a, *b;
  int na, nb;
  int64_t stride;  // entries
  __host__ __device__ uint64_t *at(int s) const { return s < na ? a + s * stride : b + (s - na) * stride; }
};

__device__ __forceinline__ void *plane_ptr(const PlaneSet &p, int id)
{
  if (id < FGA_NF64) return p.f64 + (int64_t)id * p.cap;
  if (id == FGA_NF64) return p.lineage;
  return p.i32 + (int64_t)(id - NWIDE) * p.cap;
}

// Re-orders planes through scratch: planes [g0, g1) are gathered,
// slot[gs + p - g0][i] = plane p[perm[i]], and the slots of the planes
// [c0, c1), gathered by the launch before, are copied back to their planes.
// blockIdx.y takes G planes.  The planes of a large set stream through the
// 256 MB last-level cache one or two at a time, which serves the scattered reads
// of the first ordering (33 M beams: 22.8 ms for one and two planes per block,
// 29.9 ms for eight; one plane per launch and a copy kernel, 23.6 ms; 66 k
// beams: 28 us against 116 launches of 3 us each).
constexpr int G = 2;
__global__ __launch_bounds__(256) void k_permute(PlaneSet ps, const int32_t *__restrict__ perm, int64_t n,
                                                 Slots sl, int g0, int g1, int gs, int c0, int c1, int cs)
{
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const int ng = (g1 - g0 + G - 1) / G;
  const bool gather = (int)blockIdx.y < ng;
  const int y = gather ? blockIdx.y : blockIdx.y - ng;
  const int b = gather ? g0 : c0, e = gather ? g1 : c1, s0 = gather ? gs : cs;
  const int64_t src = gather ? perm[i] : i;
  uint64_t v[G];
#pragma unroll
  for (int k = 0; k < G; ++k) {
    const int p = b + y * G + k;
    v[k] = 0;
    if (p < e) {
      const void *from = gather ? plane_ptr(ps, p) : sl.at(s0 + p - b);
      v[k] = p < NWIDE ? static_cast<const uint64_t *>(from)[src] : static_cast<const uint32_t *>(from)[src];
    }
  }
#pragma unroll
  for (int k = 0; k < G; ++k) {
    const int p = b + y * G + k;
    if (p < e) {
      void *to = gather ? sl.at(s0 + p - b) : plane_ptr(ps, p);
      if (p < NWIDE) static_cast<uint64_t *>(to)[i] = v[k];
      else static_cast<uint32_t *>(to)[i] = (uint32_t)v[k];
    }
  }
}

// The permutation of all planes in as few launches as the scratch allows: with
// NPLANE slots one gather and one copy; with fewer, groups of half the slots, each
// launch gathering one group while it copies the group before back.  The sort's own
// buffers always give two slots.
hipError_t permute_planes(const PlaneSet &ps, const int32_t *perm, int64_t n, const Slots &sl, hipStream_t st)
{
  const int slots = sl.na + sl.nb;
  if (slots < 2) return hipErrorInvalidValue;
  const int per = slots >= NPLANE ? NPLANE : slots / 2;
  const unsigned nblk = (unsigned)((n + 255) / 256);
  auto launch = [&](int g0, int g1, int gs, int c0, int c1, int cs) {
    const int y = (g1 - g0 + G - 1) / G + (c1 - c0 + G - 1) / G;
    hipLaunchKernelGGL(k_permute, dim3(nblk, (unsigned)y), 256, 0, st, ps, perm, n, sl, g0, g1, gs, c0, c1, cs);
    return hipGetLastError();
  };
  int prev0 = 0, prev1 = 0, prevs = 0;
  for (int g0 = 0, k = 0; g0 < NPLANE; g0 += per, ++k) {
    const int g1 = g0 + per < NPLANE ? g0 + per : NPLANE, gs = (k & 1) * per;
    hipError_t e = launch(g0, g1, gs, prev0, prev1, prevs);
    if (e != hipSuccess) return e;
    prev0 = g0;
    prev1 = g1;
    prevs = gs;
  }
  return launch(0, 0, 0, prev0, prev1, prevs);
}

// Points in Morton order of their positions, up to MAX_RANKED of them, in one launch
// without a step between workgroups: each forms the bounding box and all keys for
// itself, and a thread's point goes to the number of points before it (n^2
// comparisons; 16 bytes of LDS, the same for all lanes, give four).  That is in place
// of a copy to the host, the sort there and two copies back: a sum of 20 k beams takes
// 83 us in place of 97 at 40 points, 107 for 121 at 349, 157 for 159 at 1024, where
// the line lies.  bad: the first point that is not finite, else n.
__global__ __launch_bounds__(256) void k_rank_points(const double *__restrict__ xyz, int n, double *__restrict__ sorted,
                                                     int32_t *__restrict__ perm, int64_t *__restrict__ bad)
{
  __shared__ alignas(16) uint32_t key[MAX_RANKED];  // read four at a time
  __shared__ double red[4][6];
  __shared__ int first_bad;
  const int t = threadIdx.x;
  if (t == 0) first_bad = n;
  __syncthreads();
  double b[6] = {HUGE_VAL, HUGE_VAL, HUGE_VAL, -HUGE_VAL, -HUGE_VAL, -HUGE_VAL};
  for (int i = t; i < n; i += 256) {
    bool finite = true;
    for (int d = 0; d < 3; ++d) {
      const double v = xyz[3 * i + d];
      finite = finite && isfinite(v);
      b[d] = fmin(b[d], v);
      b[3 + d] = fmax(b[3 + d], v);
    }
    if (!finite) atomicMin(&first_bad, i);
  }
  for (int off = 32; off > 0; off >>= 1)
    for (int d = 0; d < 3; ++d) {
      b[d] = fmin(b[d], __shfl_xor(b[d], off));
      b[3 + d] = fmax(b[3 + d], __shfl_xor(b[3 + d], off));
    }
  if ((t & 63) == 0)
    for (int k = 0; k < 6; ++k) red[t >> 6][k] = b[k];
  __syncthreads();
  double lo[3], span[3];
  for (int d = 0; d < 3; ++d) {
    lo[d] = fmin(fmin(red[0][d], red[1][d]), fmin(red[2][d], red[3][d]));
    const double hi = fmax(fmax(red[0][3 + d], red[1][3 + d]), fmax(red[2][3 + d], red[3][3 + d]));
    span[d] = hi > lo[d] ? hi - lo[d] : 1.0;
  }
  const int padded = (n + 3) & ~3;
  for (int i = t; i < padded; i += 256) {
    uint32_t k = 0xffffffffu;  // the padding goes last
    if (i < n) {
      uint32_t c[3];
      for (int d = 0; d < 3; ++d) {
        double u = (xyz[3 * i + d] - lo[d]) / span[d] * 1023.0;
        u = u < 0.0 ? 0.0 : (u > 1023.0 ? 1023.0 : u);
        c[d] = (uint32_t)u;
      }
      k = spread3(c[0]) | (spread3(c[1]) << 1) | (spread3(c[2]) << 2);
    }
    key[i] = k;
  }
  __syncthreads();
  const int i = blockIdx.x * 256 + t;
  if (i < n) {
    const uint32_t mine = key[i];
    int rank = 0;
    const uint4 *k4 = reinterpret_cast<const uint4 *>(key);
    for (int j = 0; j < padded; j += 4) {
      const uint4 k = k4[j >> 2];
      rank += (k.x < mine || (k.x == mine && j < i)) + (k.y < mine || (k.y == mine && j + 1 < i)) +
              (k.z < mine || (k.z == mine && j + 2 < i)) + (k.w < mine || (k.w == mine && j + 3 < i));
    }
    for (int d = 0; d < 3; ++d) sorted[3 * rank + d] = xyz[3 * i + d];
    perm[rank] = i;
  }
  if (i == 0) *bad = first_bad;
}

struct SortBufs {
  uint32_t *k1, *k2;
  int32_t *v1, *v2;
  double *part, *box;
  double *room;  // nothing of its own: with it the free bytes hold two planes
  int64_t *alive;
  void *sort_tmp;
  size_t sort_bytes;
  size_t free_bytes;  // from k1 to the workspace's end: free once the keys are sorted and the live beams counted
};

// Beams of a set for whose sort a workspace query counts a slot for every plane
// (at most 122 MB) unless the caller has memory to lend, as its launches cost more
// than its bytes: 98 k beams without receivers' buffers to borrow took 30 launches
// of 5 us for the planes, now two.  The call takes less, down to a query without them.
constexpr int64_t SMALL_SET = 1 << 18;

SortBufs sort_layout(int64_t n, Arena &ar)
{
  SortBufs b{};
  const int64_t nblk = (n + 255) / 256;
  b.v2 = ar.take<int32_t>(n + 1);
  b.part = ar.take<double>(6 * nblk + 6);
  b.box = ar.take<double>(6);
  b.alive = ar.take<int64_t>(1);
  const size_t keep = Arena::need(ar.used);
  b.k1 = ar.take<uint32_t>(n + 1);
  b.k2 = ar.take<uint32_t>(n + 1);
  b.v1 = ar.take<int32_t>(n + 1);
  b.room = ar.take<double>(n + 1);
  b.sort_bytes = 0;
  // size query only (no device work): the bytes come back in sort_bytes
  (void)hipcub::DeviceRadixSort::SortPairs(nullptr, b.sort_bytes, b.k1, b.k2, b.v1, b.v2, (int)(n > 0 ? n : 1), 0,
                                           32);
  b.sort_tmp = ar.take<char>(b.sort_bytes + 1);
  b.free_bytes = ar.size > keep ? ar.size - keep : 0;  // and the rest of the workspace
  return b;
}

}  // namespace

hipError_t launch_rank_points(const double *xyz, int n, double *sorted, int32_t *perm, int64_t *bad, hipStream_t st)
{
  if (n < 1 || n > MAX_RANKED) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_rank_points, (unsigned)((n + 255) / 256), 256, 0, st, xyz, n, sorted, perm, bad);
  return hipGetLastError();
}

fga_status sort_beams_spatial(fga_beams *b, Arena &ar, void *scratch, size_t scratch_bytes, hipStream_t st,
                              bool size_only, size_t *need, bool least)
{
  const int64_t n = b->count;
  SortBufs s = sort_layout(n, ar);
  if (size_only) {
    if (!least && scratch_bytes < (size_t)NPLANE * 8 * n && n <= SMALL_SET)
      ar.take<double>((size_t)NPLANE * ((n + 31) & ~(int64_t)31));
    *need = ar.used;
    return FGA_OK;
  }
  if (!s.k1 || !s.k2 || !s.v1 || !s.v2 || !s.part || !s.box || !s.room || !s.alive || !s.sort_tmp)
    return fail(FGA_ENOMEM, "beam sort workspace too small (%zu bytes given)", ar.size);
  if (n == 0) return FGA_OK;
  if (n > 0x7fffffff) return fail(FGA_EUNSUPPORTED, "more than 2^31 beams in one sort");
  const int64_t nblk = (n + 255) / 256;
  const int64_t cap = b->capacity;
  hipLaunchKernelGGL(k_bbox_partial, (unsigned)nblk, 256, 0, st, b->f64, b->i32, cap, n, s.part);
  FGA_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_bbox_final, 1, 256, 0, st, s.part, nblk, s.box);
  FGA_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_morton, (unsigned)nblk, 256, 0, st, b->f64, b->i32, cap, n, s.box, s.k1, s.v1);
  FGA_LAUNCH_CHECK();
  // dead beams carry key 0xffffffff: sort all 32 bits so they land last
  size_t bytes = s.sort_bytes;
  FGA_HIP(hipcub::DeviceRadixSort::SortPairs(s.sort_tmp, bytes, s.k1, s.k2, s.v1, s.v2, (int)n, 0, 32, st));
  FGA_HIP(hipMemsetAsync(s.alive, 0, sizeof(int64_t), st));
  hipLaunchKernelGGL(k_count_alive, (unsigned)nblk, 256, 0, st, s.k2, n, s.alive);
  FGA_LAUNCH_CHECK();
  Slots sl{};
  sl.stride = (n + 31) & ~(int64_t)31;
  const size_t slot_bytes = (size_t)sl.stride * 8;
  auto slots_in = [&](size_t bytes) { return (int)(bytes / slot_bytes < NPLANE ? bytes / slot_bytes : NPLANE); };
  sl.a = static_cast<uint64_t *>(scratch);
  sl.na = scratch ? slots_in(scratch_bytes) : 0;
  sl.b = reinterpret_cast<uint64_t *>(s.k1);
  sl.nb = slots_in(s.free_bytes);
  FGA_HIP(permute_planes(PlaneSet{b->f64, b->i32, b->lineage, cap}, s.v2, n, sl, st));
  int64_t alive = 0;
  FGA_HIP(hipMemcpyAsync(&alive, s.alive, sizeof alive, hipMemcpyDeviceToHost, st));
  FGA_HIP(hipStreamSynchronize(st));
  b->count = alive;
  return FGA_OK;
}

}  // namespace fga
