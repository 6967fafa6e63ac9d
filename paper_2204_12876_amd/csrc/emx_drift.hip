// Height drift compensation (Sec. II-D).
//
// The map's heights are shifted by the mean error between a frame's points and
// the map on flat ground, measured before the frame is fused.  Two launches:
//   1. per 1024-point chunk, the float64 sum of the errors and their count,
//      each thread summing its four points (256 apart) in index order and the
//      workgroup combining them by a fixed butterfly;
//   2. every valid cell adds the mean, rounded once to float32.  Each workgroup
//      combines the chunk partials itself, in the same fixed way: 12 bytes a
//      chunk from the L2 cost less than a launch between the two (300k points on
//      400 x 400 cells: 5.8 -> 4.2 us).  (A last workgroup of launch 1 that
//      combined them would need an agent-scope release from every other one, and
//      on this chip each writes back the L2.)
// The order of every sum depends only on the number of points, so the result
// is the same on every call.  The point decisions (transform, validity,
// binning) are the fusion's own, from the shared device helpers.
#include "emx_kernels.h"

namespace emx {

namespace {

constexpr int kNTd = 256;                 // threads per chunk workgroup
constexpr int kPerD = kChunk / kNTd;      // points per thread
// Shift workgroups at most: each reads all chunk partials, so half as many for large
// frames (12M points on 2000 x 2000 cells: 55 against 62 us a call; 60k there: 19.6
// against 18.0, 1.5M 23.4 against 21.4).
constexpr unsigned kShiftGroups = 2048;
constexpr int64_t kManyChunks = 2048;
// Chunk partials requested together: one after the other, 4M points on 2000 x 2000
// cells took 37.1 instead of 34.7 us a call, 12M on 100 x 100 49.6 instead of 41.1.
constexpr int kAheadD = 8;

struct DriftArgs {
  Item it;
  float trav_min;
  double* part_sum;     // [B]
  uint32_t* part_cnt;   // [B]
  double* out_mean;     // optional
  int64_t* out_count;   // optional
};

// Fixed-shape sum over the workgroup: a butterfly within each wave, then the
// wave totals in wave order.  Thread 0 ends with the total; the order of the
// additions never changes.
__device__ __forceinline__ void block_sum(double& sum, int64_t& cnt, double* s_sum,
                                          int64_t* s_cnt) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    sum = sum + __shfl_xor(sum, o, 64);
    cnt = cnt + __shfl_xor(cnt, o, 64);
  }
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    s_sum[wave] = sum;
    s_cnt[wave] = cnt;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    sum = s_sum[0];
    cnt = s_cnt[0];
    for (int w = 1; w < kNTd / 64; ++w) {
      sum = sum + s_sum[w];
      cnt = cnt + s_cnt[w];
    }
  }
}

__global__ __launch_bounds__(kNTd) void k_drift_partial(DriftArgs a) {
  __shared__ double s_sum[kNTd / 64];
  __shared__ int64_t s_cnt[kNTd / 64];
  const Item& it = a.it;
  const int tid = threadIdx.x;
  const int64_t base = (int64_t)blockIdx.x * kChunk;
  double sum = 0.0;
  int64_t cnt = 0;
  // the four points' cells first, then their layers, so that the gathers of
  // all four are in flight together
  float zm[kPerD];
  int64_t cell[kPerD];
  bool use[kPerD];
#pragma unroll
  for (int j = 0; j < kPerD; ++j) {
    const int64_t i = base + (int64_t)j * kNTd + tid;  // a thread's points in index order
    use[j] = false;
    cell[j] = 0;
    zm[j] = 0.0f;
    if (i < it.n) {
      const PointEval e = eval_point(it.P, it.c, it.x[i], it.y[i], it.z[i]);
      int ix, iy;
      use[j] = e.valid && bin_xy(e.xm, e.ym, it.c, ix, iy);
      if (use[j]) cell[j] = pcell(it.c, ix, iy);  // physical: the layers
      zm[j] = e.zm;
    }
  }
#pragma unroll
  for (int j = 0; j < kPerD; ++j) {
    const uint8_t vc = it.L.valid[cell[j]];
    const float tr = it.L.trav[cell[j]];
    const float hc = it.L.h[cell[j]];
    // NaN traversability never passes
    if (use[j] && vc && tr > a.trav_min) {
      sum = sum + ((double)zm[j] - (double)hc);
      ++cnt;
    }
  }
  block_sum(sum, cnt, s_sum, s_cnt);
  if (tid == 0) {
    a.part_sum[blockIdx.x] = sum;
    a.part_cnt[blockIdx.x] = (uint32_t)cnt;
  }
}

__global__ __launch_bounds__(kNTd) void k_drift_shift(DriftArgs a, int64_t cells) {
  __shared__ double s_sum[kNTd / 64];
  __shared__ int64_t s_cnt[kNTd / 64];
  __shared__ double s_mean;
  __shared__ int64_t s_n;
  // the chunk partials: strided sums in chunk order, then a fixed tree
  const int tid = threadIdx.x;
  double sum = 0.0;
  int64_t cnt = 0;
  for (int64_t b = tid; b < a.it.B; b += kAheadD * kNTd) {
    double p[kAheadD];
    uint32_t c[kAheadD];
#pragma unroll
    for (int j = 0; j < kAheadD; ++j) {
      const bool in = b + j * kNTd < a.it.B;  // past the end: nothing (a sum is never -0.0)
      p[j] = in ? a.part_sum[b + j * kNTd] : 0.0;
      c[j] = in ? a.part_cnt[b + j * kNTd] : 0u;
    }
#pragma unroll
    for (int j = 0; j < kAheadD; ++j) {
      sum = sum + p[j];
      cnt += c[j];
    }
  }
  block_sum(sum, cnt, s_sum, s_cnt);
  if (tid == 0) {
    s_n = cnt;
    s_mean = cnt > 0 ? sum / (double)cnt : 0.0;
    if (blockIdx.x == 0) {
      if (a.out_mean) *a.out_mean = s_mean;
      if (a.out_count) *a.out_count = cnt;
    }
  }
  __syncthreads();
  if (s_n <= 0) return;
  const float mean = (float)s_mean;
  const Layers& L = a.it.L;
  for (int64_t i = (int64_t)blockIdx.x * kNTd + tid; i < cells; i += (int64_t)gridDim.x * kNTd)
    if (L.valid[i]) L.h[i] = L.h[i] + mean;
}

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

}  // namespace

size_t drift_scratch_layout(int64_t max_points, char* base, DriftScratch* out) {
  const int64_t B = (max_points + kChunk - 1) / kChunk;
  size_t off = 256;  // kept free: the size contract of emx_drift_scratch_bytes
  const size_t o_sum = off;
  off = align256(off + (size_t)B * sizeof(double));
  const size_t o_cnt = off;
  off = align256(off + (size_t)B * sizeof(uint32_t));
  if (out && base) {
    out->part_sum = (double*)(base + o_sum);
    out->part_cnt = (uint32_t*)(base + o_cnt);
  }
  return off;
}

hipError_t launch_drift(const Item& it, float trav_min, const DriftScratch& ds,
                        double* out_mean, int64_t* out_count, hipStream_t stream) {
  DriftArgs a;
  a.it = it;
  a.trav_min = trav_min;
  a.part_sum = ds.part_sum;
  a.part_cnt = ds.part_cnt;
  a.out_mean = out_mean;
  a.out_count = out_count;
  hipError_t err;
  if (it.B > 0) {
    TimedLaunch tl("k_drift_partial", stream);
    hipLaunchKernelGGL(k_drift_partial, dim3(it.B), dim3(kNTd), 0, stream, a);
  }
  if ((err = hipGetLastError()) != hipSuccess) return err;
  const int64_t cells = (int64_t)it.c.nx * it.c.ny;
  const int64_t groups = (cells + kNTd - 1) / kNTd;
  const unsigned most = it.B > kManyChunks ? kShiftGroups / 2 : kShiftGroups;
  {
    TimedLaunch tl("k_drift_shift", stream);
    hipLaunchKernelGGL(k_drift_shift,
                       dim3(groups < most ? (unsigned)groups : most), dim3(kNTd), 0, stream, a,
                       cells);
  }
  return hipGetLastError();
}

}  // namespace emx
