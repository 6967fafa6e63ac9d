// Post-processing filters for legged locomotion (Sec. II-I).
//
// Minimum-filter inpainting: the invalid cells form regions connected through
// their edge neighbours; each region takes the smallest height on its border.
// A union-find over the grid labels the regions.  Links only ever point from
// a larger cell index to a smaller one (an integer atomic minimum), so there
// are no cycles and each region ends with its smallest cell as the root,
// whatever the order of the unions.  Four launches, all but the first on the
// scratch arrays alone, in logical cell order:
//   1. local: per 32 x 32 tile, in LDS, the union of the tile's invalid cells
//      and, per tile-local region, the minimum border height offered from
//      inside the tile.  Writes each invalid cell's parent (its local root; -1
//      marks a valid cell), the local minimum at each local root, and the valid
//      cells' output;
//   2. seams, one thread per pair of cells across a tile edge: invalid pairs
//      unite in the global parent array, a valid cell offers its height to the
//      local region across the edge (any cell on its chain of parents is a
//      local root, which the next launch collects);
//   3. collect: local roots pass their minimum to their final root;
//   4. fill: invalid cells read their final root's minimum (NaN if none).
// Minima are integer atomics over an order-preserving key of the float, so
// the output is deterministic.
// What bounds it: the four launches' chains of dependent loads.  Measured on a
// 400 x 400 map, before and after: local 21.3 -> 9.9 us (a wave's offers were
// reduced region by region), seams 10.1 -> 10.4 us with the offers across the
// edges in them, collect 12.1 -> 4.7 us (it made those offers, and followed every
// chain through the atomics path), fill 3.9 us.
//
// Smoothing.  Box and Gaussian work on 16 x 16 output tiles: a workgroup stages
// the tile and its mirrored halo in LDS and runs a pass along x into LDS and a
// pass along y to the output.  The median works in registers, a column per lane.
#include "emx_kernels.h"

namespace emx {

namespace {

constexpr int kNTi = 256;

// Order-preserving key of a float: larger float, larger key.  The all-ones
// key is "none" and decodes to NaN.
__device__ __forceinline__ uint32_t f32_key(float f) {
  const uint32_t b = __float_as_uint(f);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float key_f32(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}
constexpr uint32_t kNoKey = 0xffffffffu;

struct InpaintArgs {
  Consts c;
  Layers L;
  int32_t* parent;  // [cells] parent chain of invalid cells (global indices); -1: valid
  uint32_t* best;   // [cells] at local roots: key of the smallest border height
  float* out;       // [cells]
  int tiles_x;
};

constexpr int kIT = 32;                // inpainting tile side
constexpr int kNTl = kIT * kIT;        // one thread per tile cell

// Root of cell x once no union runs any more.
__device__ __forceinline__ int32_t find_root(const int32_t* parent, int32_t x) {
  int32_t p = parent[x];
  while (p != x) {
    x = p;
    p = parent[x];
  }
  return x;
}

// A parent while unions run: past the L2, which is not shared by all the chip.
__device__ __forceinline__ int32_t load_parent(const int32_t* parent, int32_t x) {
  return __hip_atomic_load(parent + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Unites the regions of cells a and b.  Both chains of parents are followed at
// the same time, one step of each to a round trip, and halved on the way: each
// visited cell is pointed at its grandparent.  The write is an atomic minimum,
// so it can never undo a link made meanwhile (parents only decrease, and stay
// ancestors).
__device__ __forceinline__ void unite(int32_t* parent, int32_t a, int32_t b) {
  int32_t pa = load_parent(parent, a), pb = load_parent(parent, b);
  while (a != b) {
    const bool ra = pa == a, rb = pb == b;
    if (ra && rb) {
      if (a < b) {
        const int32_t t = a;
        a = b;
        b = t;
      }
      // link root a below b; if a is no longer a root, follow its new parent
      const int32_t old = atomicMin(parent + a, b);
      if (old == a) return;
      a = old;
      pa = load_parent(parent, a);
      pb = load_parent(parent, b);
      continue;
    }
    const int32_t ga = load_parent(parent, pa), gb = load_parent(parent, pb);
    if (!ra) {
      if (ga != pa) atomicMin(parent + a, ga);
      a = pa;
    }
    if (!rb) {
      if (gb != pb) atomicMin(parent + b, gb);
      b = pb;
    }
    pa = ga;
    pb = gb;
  }
}

// The same union-find on a tile's LDS array of local indices.
__device__ __forceinline__ int lds_find(volatile int* par, int x) {
  int p = par[x];
  while (p != x) {
    x = p;
    p = par[x];
  }
  return x;
}

__device__ __forceinline__ void lds_unite(int* par, int a, int b) {
  volatile int* vp = par;
  while (true) {
    a = lds_find(vp, a);
    b = lds_find(vp, b);
    if (a == b) return;
    if (a < b) {
      const int t = a;
      a = b;
      b = t;
    }
    const int old = atomicMin(par + a, b);
    if (old == a) return;
    a = old;
  }
}

__global__ __launch_bounds__(kNTl) void k_inp_local(InpaintArgs a) {
  __shared__ int s_par[kNTl];
  __shared__ uint32_t s_best[kNTl];
  const int nx = a.c.nx;
  const int ny = a.c.ny;
  const int tid = threadIdx.x;
  const int lx = tid % kIT;
  const int ly = tid / kIT;
  const int x0 = (int)(blockIdx.x % a.tiles_x) * kIT;
  const int y0 = (int)(blockIdx.x / a.tiles_x) * kIT;
  const int gx = x0 + lx;
  const int gy = y0 + ly;
  const bool in = gx < nx && gy < ny;
  const int64_t pc = in ? pcell(a.c, gx, gy) : 0;
  const bool ok = in && a.L.valid[pc];
  const float height = in ? a.L.h[pc] : 0.0f;
  const bool hole = in && !ok;
  // Rows first, without atomics: a hole's parent is the first cell of its
  // run of holes along the row (a tile row is half a wave: one ballot).
  const uint64_t bal = __ballot(hole);
  const uint32_t row = (uint32_t)(bal >> (tid & 32));
  const uint32_t gaps = ~row & ((1u << lx) - 1u);   // non-holes left of lx
  const int start = gaps ? 32 - __builtin_clz(gaps) : 0;
  s_par[tid] = hole ? ly * kIT + start : -1;
  s_best[tid] = kNoKey;
  __syncthreads();
  // Then columns: join a run to the run above where they first overlap.
  if (hole && ly > 0 && s_par[tid - kIT] >= 0 && (lx == start || s_par[tid - kIT - 1] < 0))
    lds_unite(s_par, ly * kIT + start, tid - kIT);
  __syncthreads();
  // the roots, then each hole's own root in place of its parent
  const int root = hole ? lds_find(s_par, tid) : -1;
  __syncthreads();
  s_par[tid] = root;
  __syncthreads();
  // valid cells offer their height to the holes beside them, each by an LDS
  // atomic of its own (reducing a wave's offers region by region first cost
  // seven cross-lane steps for every region that the wave met)
  if (ok) {
    const uint32_t k = f32_key(height);
    const int nb[4] = {lx > 0 ? s_par[tid - 1] : -1, lx + 1 < kIT ? s_par[tid + 1] : -1,
                       ly > 0 ? s_par[tid - kIT] : -1, ly + 1 < kIT ? s_par[tid + kIT] : -1};
#pragma unroll
    for (int d = 0; d < 4; ++d)
      if (nb[d] >= 0) atomicMin(s_best + nb[d], k);
  }
  __syncthreads();
  if (!in) return;
  const int64_t i = (int64_t)gy * nx + gx;
  a.parent[i] = hole ? (int32_t)((int64_t)(y0 + root / kIT) * nx + x0 + root % kIT) : -1;
  a.best[i] = root == tid ? s_best[tid] : kNoKey;
  if (ok) a.out[i] = height;
}

// Seam pairs: ny to each vertical seam, then nx to each horizontal one.
__host__ __device__ inline int64_t seam_pairs(int nx, int ny) {
  return (int64_t)((nx - 1) / kIT) * ny + (int64_t)((ny - 1) / kIT) * nx;
}

__global__ __launch_bounds__(kNTi) void k_inp_seams(InpaintArgs a) {
  const int nx = a.c.nx;
  const int ny = a.c.ny;
  const int64_t q = (int64_t)blockIdx.x * kNTi + threadIdx.x;
  if (q >= seam_pairs(nx, ny)) return;
  const int nv = ((nx - 1) / kIT) * ny;  // at most 511 * 16384
  const bool vertical = q < nv;
  const int u = (int)(vertical ? q : q - nv);
  const int len = vertical ? ny : nx;
  const int seam = u / len;
  const int along = u - seam * len;
  const int across = (seam + 1) * kIT - 1;
  const int32_t i = vertical ? along * nx + across : across * nx + along;
  const int32_t j = i + (vertical ? 1 : nx);
  const int32_t back = vertical ? nx : 1;  // the pair before this one along the seam
  // (whatever unions these loads see, they give an ancestor of a hole, -1 of a
  // valid cell)
  const bool first = along % kIT == 0;
  const int32_t pi = a.parent[i], pj = a.parent[j];
  const int32_t bi = first ? -1 : a.parent[i - back], bj = first ? -1 : a.parent[j - back];
  if (pi >= 0 && pj >= 0) {
    // pairs next to each other along a tile edge are already joined on both
    // sides: only the first pair of each run of pairs unites
    if (bi < 0 || bj < 0) unite(a.parent, pi, pj);
  } else if (pi >= 0) {
    atomicMin(a.best + pi, f32_key(a.out[j]));
  } else if (pj >= 0) {
    atomicMin(a.best + pj, f32_key(a.out[i]));
  }
}

__global__ __launch_bounds__(kNTi) void k_inp_collect(InpaintArgs a) {
  const int64_t i = (int64_t)blockIdx.x * kNTi + threadIdx.x;
  if (i >= (int64_t)a.c.nx * a.c.ny) return;
  const uint32_t k = a.best[i];
  if (k == kNoKey) return;
  const int32_t r = find_root(a.parent, (int32_t)i);
  if (r != (int32_t)i) atomicMin(a.best + r, k);
}

__global__ __launch_bounds__(kNTi) void k_inp_fill(InpaintArgs a) {
  const int64_t i = (int64_t)blockIdx.x * kNTi + threadIdx.x;
  if (i >= (int64_t)a.c.nx * a.c.ny) return;
  const int32_t p = a.parent[i];
  if (p >= 0) a.out[i] = key_f32(a.best[find_root(a.parent, p)]);
}

// -------------------------------------------------------------- smoothing
constexpr int kFT = 16;                      // output tile side
constexpr int kMaxR = 15;                    // largest radius (ksize 31)
constexpr int kFH = kFT + 2 * kMaxR;         // largest staged side

struct SmoothArgs {
  const float* in;
  float* out;
  int nx, ny;
  int r;                 // ksize / 2
  float w[2 * kMaxR + 1];  // per-axis weights (box: all 1)
  float scale;           // applied after both passes (box: 1/ksize^2)
};

// Index i mirrored into [0, n) about the edge cells.  Positions a partial
// tile stages beyond what its outputs read are clamped, to stay in bounds.
__device__ __forceinline__ int mirror(int i, int n) {
  i = i < 0 ? -i : i;
  i = i > n - 1 ? 2 * (n - 1) - i : i;
  return min(max(i, 0), n - 1);
}

// Stage the tile at (x0, y0) with a halo of r, mirrored at the grid's edges.
__device__ __forceinline__ void stage(float (*s)[kFH], const SmoothArgs& a, int x0, int y0) {
  const int side = kFT + 2 * a.r;
  for (int idx = threadIdx.x; idx < side * side; idx += kNTi) {
    const int ly = idx / side;
    const int lx = idx - ly * side;
    const int gx = mirror(x0 - a.r + lx, a.nx);
    const int gy = mirror(y0 - a.r + ly, a.ny);
    s[ly][lx] = a.in[(int64_t)gy * a.nx + gx];
  }
}

// Box and Gaussian: weighted sum along x (into LDS), then along y.
__global__ __launch_bounds__(kNTi) void k_smooth_sep(SmoothArgs a) {
  __shared__ float s[kFH][kFH];
  __shared__ float t[kFH][kFT + 1];
  __shared__ float w[2 * kMaxR + 1];  // the weights, indexed at run time
  const int x0 = blockIdx.x * kFT;
  const int y0 = blockIdx.y * kFT;
  if (threadIdx.x < 2 * kMaxR + 1) w[threadIdx.x] = a.w[threadIdx.x];
  stage(s, a, x0, y0);
  __syncthreads();
  const int k = 2 * a.r + 1;
  const int rows = kFT + 2 * a.r;
  for (int idx = threadIdx.x; idx < rows * kFT; idx += kNTi) {
    const int ly = idx / kFT;
    const int lx = idx - ly * kFT;
    float acc = 0.0f;
    for (int j = 0; j < k; ++j) acc = acc + w[j] * s[ly][lx + j];
    t[ly][lx] = acc;
  }
  __syncthreads();
  const int lx = threadIdx.x % kFT;
  const int ly = threadIdx.x / kFT;
  const int gx = x0 + lx;
  const int gy = y0 + ly;
  if (gx >= a.nx || gy >= a.ny) return;
  float acc = 0.0f;
  for (int j = 0; j < k; ++j) acc = acc + w[j] * t[ly + j][lx];
  a.out[(int64_t)gy * a.nx + gx] = acc * a.scale;
}

// ------------------------------------------------------------------ median
// A wave takes one row of 64 - (K - 1) outputs, a column per lane.  A lane sorts
// its column of K values; the sorted columns of the K - 1 lanes beside it come by
// DPP moves.  Selecting from sorted columns takes about a fifth of the
// comparisons of ranking every value against every other: 15.7 -> 4.1 us for
// ksize 5 on 400 x 400 cells.
__device__ __forceinline__ void order(float& a, float& b) {
  const float lo = fminf(a, b);
  b = fmaxf(a, b);
  a = lo;
}

__device__ __forceinline__ void sort3(float& a, float& b, float& c) {
  order(a, b);
  order(b, c);
  order(a, b);
}

// Nine exchanges.
__device__ __forceinline__ void sort5(float (&v)[5]) {
  order(v[0], v[1]);
  order(v[3], v[4]);
  order(v[2], v[4]);
  order(v[2], v[3]);
  order(v[1], v[4]);
  order(v[0], v[3]);
  order(v[0], v[2]);
  order(v[1], v[3]);
  order(v[1], v[2]);
}

// The middle of n (odd) values, of which the first n / 2 + 2 are held: their
// smallest and largest cannot be the middle and go, and the next value comes in.
template <int n>
__device__ __forceinline__ float middle(float* v) {
  constexpr int held = n / 2 + 2;
  if constexpr (n == 3) {
    return __builtin_amdgcn_fmed3f(v[0], v[1], v[2]);
  } else {
#pragma unroll
    for (int i = 1; i < held; ++i) order(v[0], v[i]);       // smallest to v[0]
#pragma unroll
    for (int i = 1; i + 1 < held; ++i) order(v[i], v[held - 1]);  // largest to the end
    // what is left: v[1 .. held - 2], then the values not seen yet
#pragma unroll
    for (int i = 0; i < held - 2; ++i) v[i] = v[i + 1];
#pragma unroll
    for (int i = held - 2; i < n - 2; ++i) v[i] = v[i + 2];
    return middle<n - 2>(v);
  }
}

// The lane's value of the column `step` to the right (below: to the left); lanes
// at the wave's ends get a value they do not use.
template <int step>
__device__ __forceinline__ float column(float v) {
  int x = __float_as_int(v);
#pragma unroll
  for (int i = 0; i < (step < 0 ? -step : step); ++i)
    x = step < 0 ? __builtin_amdgcn_update_dpp(0, x, 0x138 /* wave_shr:1 */, 0xf, 0xf, false)
                 : __builtin_amdgcn_update_dpp(0, x, 0x130 /* wave_shl:1 */, 0xf, 0xf, false);
  return __int_as_float(x);
}

// Median of a K x K window: the middle value; NaN if the window holds a NaN.
constexpr int kNTm = 64 * kFT;  // a wave to a row, kFT rows to a workgroup

template <int K>
__global__ __launch_bounds__(kNTm) void k_smooth_median(SmoothArgs a) {
  constexpr int R = K / 2;
  const int lane = threadIdx.x & 63;
  const int gx = (int)blockIdx.x * (64 - 2 * R) - R + lane;
  const int gy = (int)blockIdx.y * kFT + (int)(threadIdx.x >> 6);
  if (gy >= a.ny) return;  // whole waves
  const int cx = mirror(gx, a.nx);
  float v[K];
  bool nan = false;
#pragma unroll
  for (int j = 0; j < K; ++j) {
    v[j] = a.in[(int64_t)mirror(gy + j - R, a.ny) * a.nx + cx];
    nan = nan || isnan(v[j]);
  }
  uint64_t bad = __ballot(nan);
  float med;
  if constexpr (K == 3) {
    bad |= (bad << 1) | (bad >> 1);
    sort3(v[0], v[1], v[2]);
    const float lo = fmaxf(fmaxf(column<-1>(v[0]), v[0]), column<1>(v[0]));
    const float mi = __builtin_amdgcn_fmed3f(column<-1>(v[1]), v[1], column<1>(v[1]));
    const float hi = fminf(fminf(column<-1>(v[2]), v[2]), column<1>(v[2]));
    med = __builtin_amdgcn_fmed3f(lo, mi, hi);
  } else {
    bad |= (bad << 1) | (bad >> 1) | (bad << 2) | (bad >> 2);
    sort5(v);
    float r[5][5];  // by rank in the column, then sorted across the columns
#pragma unroll
    for (int i = 0; i < 5; ++i) {
      r[i][0] = column<-2>(v[i]);
      r[i][1] = column<-1>(v[i]);
      r[i][2] = v[i];
      r[i][3] = column<1>(v[i]);
      r[i][4] = column<2>(v[i]);
      sort5(r[i]);
    }
    // Sorted both ways, r[i][j] has (i + 1)(j + 1) - 1 values not above and
    // (5 - i)(5 - j) - 1 not below it.  Where one of them is over 12 it is not the
    // middle of 25: six values below and six above it go, 13 are left.
    float c[13] = {r[0][3], r[0][4], r[1][2], r[1][3], r[1][4], r[2][1], r[2][2],
                   r[2][3], r[3][0], r[3][1], r[3][2], r[4][0], r[4][1]};
    med = middle<13>(c);
  }
  if (lane >= R && lane < 64 - R && gx < a.nx)
    a.out[(int64_t)gy * a.nx + gx] = ((bad >> lane) & 1u) ? __builtin_nanf("") : med;
}

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

}  // namespace

size_t inpaint_scratch_bytes(int nx, int ny) {
  const size_t C = (size_t)nx * (size_t)ny;
  return align256(C * 4) + align256(C * 4);
}

hipError_t launch_inpaint(const Consts& c, const Layers& L, float* out, char* scratch,
                          hipStream_t stream) {
  const int64_t C = (int64_t)c.nx * c.ny;
  InpaintArgs a;
  a.c = c;
  a.L = L;
  a.parent = (int32_t*)scratch;
  a.best = (uint32_t*)(scratch + align256((size_t)C * 4));
  a.out = out;
  a.tiles_x = (c.nx + kIT - 1) / kIT;
  const unsigned tiles = (unsigned)(a.tiles_x * ((c.ny + kIT - 1) / kIT));
  const dim3 grid((unsigned)((C + kNTi - 1) / kNTi));
  hipError_t e;
  {
    TimedLaunch tl("k_inp_local", stream);
    hipLaunchKernelGGL(k_inp_local, dim3(tiles), dim3(kNTl), 0, stream, a);
  }
  if ((e = hipGetLastError()) != hipSuccess) return e;
  // a map of one tile has no seams: its local minima are final
  if (const int64_t pairs = seam_pairs(c.nx, c.ny)) {
    {
      TimedLaunch tl("k_inp_seams", stream);
      hipLaunchKernelGGL(k_inp_seams, dim3((unsigned)((pairs + kNTi - 1) / kNTi)), dim3(kNTi), 0,
                         stream, a);
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
    {
      TimedLaunch tl("k_inp_collect", stream);
      hipLaunchKernelGGL(k_inp_collect, grid, dim3(kNTi), 0, stream, a);
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  {
    TimedLaunch tl("k_inp_fill", stream);
    hipLaunchKernelGGL(k_inp_fill, grid, dim3(kNTi), 0, stream, a);
  }
  return hipGetLastError();
}

// kind: 0 box, 1 Gaussian, 2 median (validated by the caller).
hipError_t launch_smooth(const float* in, float* out, int nx, int ny, int kind, int ksize,
                         float sigma, hipStream_t stream) {
  SmoothArgs a;
  a.in = in;
  a.out = out;
  a.nx = nx;
  a.ny = ny;
  a.r = ksize / 2;
  a.scale = 1.0f;
  for (int j = 0; j < 2 * kMaxR + 1; ++j) a.w[j] = 0.0f;
  if (kind == 0) {
    for (int j = 0; j < ksize; ++j) a.w[j] = 1.0f;
    a.scale = (float)(1.0 / ((double)ksize * (double)ksize));
  } else if (kind == 1) {
    double w[2 * kMaxR + 1], sum = 0.0;
    const double s = (double)sigma;
    for (int j = 0; j < ksize; ++j) {
      const double i = (double)(j - a.r);
      w[j] = exp(-(i * i) / (2.0 * s * s));
      sum += w[j];
    }
    for (int j = 0; j < ksize; ++j) a.w[j] = (float)(w[j] / sum);
  }
  const dim3 grid((unsigned)((nx + kFT - 1) / kFT), (unsigned)((ny + kFT - 1) / kFT));
  if (kind == 2) {
    TimedLaunch tl("k_smooth_median", stream);
    const int wide = 64 - 2 * a.r;
    const dim3 rows((unsigned)((nx + wide - 1) / wide), grid.y);
    if (ksize == 3) hipLaunchKernelGGL(k_smooth_median<3>, rows, dim3(kNTm), 0, stream, a);
    else hipLaunchKernelGGL(k_smooth_median<5>, rows, dim3(kNTm), 0, stream, a);
  } else {
    TimedLaunch tl("k_smooth_sep", stream);
    hipLaunchKernelGGL(k_smooth_sep, grid, dim3(kNTi), 0, stream, a);
  }
  return hipGetLastError();
}

}  // namespace emx
