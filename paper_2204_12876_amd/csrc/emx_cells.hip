// Per-cell passes: prior fill, robot-centric move (alone; before a fusion it
// runs in that launch), 3x3 normals, conv traversability.
//
// The stencils (normals, traversability) work in registers: a wave holds a strip
// of rows, one column per lane (see "stencil tile").  The batched launch computes
// both from one set of loads.
#include "emx_kernels.h"

namespace emx {

namespace {

// ------------------------------------------------------- XCD-aware unit order
// Workgroups are dispatched to the chip's 8 XCDs (each with its own L2) in
// turn: workgroup b goes to XCD b % 8.  Stencil tiles share their halos with
// their neighbours, so each XCD is given a contiguous range of the n units
// (unit order is row-major over tiles), and neighbouring tiles meet in one L2.
constexpr int kXcds = 8;

// The unit of workgroup b in a launch of exactly n workgroups, a bijection of
// [0, n).
__device__ __forceinline__ int64_t xcd_unit(int64_t b, int64_t n) {
  const int64_t q = n / kXcds, r = n % kXcds;
  const int64_t x = b % kXcds;
  return x * q + (x < r ? x : r) + b / kXcds;
}

// The k-th unit of workgroup b in a launch of g workgroups over n
// units, or -1 past its share.  With g a multiple of 8, the g/8 workgroups of
// XCD x walk that XCD's contiguous range in turn; otherwise units go round
// robin (b, b + g, ...).
__device__ __forceinline__ int64_t xcd_unit_k(int64_t b, int64_t g, int64_t n, int64_t k) {
  if (g % kXcds != 0) {
    const int64_t u = b + k * g;
    return u < n ? u : -1;
  }
  const int64_t q = n / kXcds, r = n % kXcds;
  const int64_t x = b % kXcds;
  const int64_t cnt = q + (x < r ? 1 : 0);
  const int64_t j = b / kXcds + k * (g / kXcds);
  return j < cnt ? x * q + (x < r ? x : r) + j : -1;
}

constexpr int kNTf = 256;

// ------------------------------------------------------------------ prior fill
struct FillArgs {
  Consts c;
  Layers L;
  int64_t cells;
  uint32_t* ctl;
  int nctl;
};

__global__ __launch_bounds__(kNTf) void k_fill_prior(FillArgs a) {
  const int64_t i = (int64_t)blockIdx.x * kNTf + threadIdx.x;
  if (i < a.nctl) a.ctl[i] = 0u;
  if (i >= a.cells) return;
  const float qnan = __builtin_nanf("");
  a.L.h[i] = a.c.h_init;
  a.L.v[i] = a.c.v_init;
  a.L.t[i] = 0;
  a.L.nx[i] = qnan;
  a.L.ny[i] = qnan;
  a.L.nz[i] = qnan;
  a.L.trav[i] = qnan;
  a.L.valid[i] = 0;
  a.L.mark[i] = 0;
  if (a.L.ub) a.L.ub[i] = INFINITY;
  ulonglong2* f = reinterpret_cast<ulonglong2*>(a.L.fx + kFxWords * i);
  f[0] = f[1] = make_ulonglong2(0u, 0u);
}

// ------------------------------------------------------------ overlap clearance
// Valid cells within a horizontal radius of the robot whose height differs
// from the robot's by more than the threshold return to the prior.
__global__ __launch_bounds__(kNTf) void k_overlap(OverlapArgs a) {
  const int64_t i = (int64_t)blockIdx.x * kNTf + threadIdx.x;  // logical cell
  const int64_t C = (int64_t)a.c.nx * a.c.ny;
  if (i >= C) return;
  const int iy = (int)(i / a.c.nx);
  const int ix = (int)(i - (int64_t)iy * a.c.nx);
  const int64_t p = pcell(a.c, ix, iy);
  const float dx = ((float)ix + 0.5f) * a.r32 - a.rx;
  const float dy = ((float)iy + 0.5f) * a.r32 - a.ry;
  const bool hit = a.L.valid[p] && ((dx * dx + dy * dy) <= a.rad2) &&
                   (fabsf(a.L.h[p] - a.rz) > a.thr);
  if (hit) {
    a.L.h[p] = a.c.h_init;
    a.L.v[p] = a.c.v_init;
    a.L.valid[p] = 0;
  }
  if (a.out) a.out[i] = hit ? 1 : 0;
}

// ---------------------------------------------------------------- stencil tile
// A wave takes kRows rows of 62 cells: its lanes are the columns x0 - 1 .. x0 +
// 62, so the neighbours of lanes 1..62 lie in the lanes beside them (one DPP
// move each) and nothing is staged in LDS.  Every load of the kRows + 2 rows of
// heights and validity is issued at once, a cell's window is valid where three
// rows' validity masks and their shifts by a lane agree (a few scalar
// instructions a row), and the filter's weights are scalar operands.  The four
// waves of a workgroup lie below each other, so a halo row is in the first-level
// cache of its other user.
// What bounds it: the bytes on large maps (1533 x 1277 cells: 13.7 -> 9.9 us, 4.2
// TB/s of its 21 bytes a cell), the one round trip on small ones (400 x 400: 8.6 ->
// 4.4 us), in a batch both (16 maps, 6.2M cells: 55 -> 38 us).  Before, a 66 x 18
// tile in LDS took five dependent rounds of loads per wave and 89 LDS reads of
// weights per cell.
constexpr int kSW = 62;            // columns of a tile
// Rows of a wave.  A map alone: two, for more waves in flight (128 x 128: 4.2
// against 5.1 us with four; 1533 x 1277: 9.9 against 10.6; 2000 x 2000: 14.8
// against 15.3).  A batch: four, which halve the fixed part of a unit (16 maps:
// 38 against 48 us).
constexpr int kRowsPlain = 2;
constexpr int kRowsBatch = 4;

constexpr int tile_rows(int rows) { return rows * (kNTf / 64); }  // of a workgroup

// The value of the lane below (left column) or above (right column).
__device__ __forceinline__ float from_left(float v) {
  return __int_as_float(
      __builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138 /* wave_shr:1 */, 0xf, 0xf, false));
}
__device__ __forceinline__ float from_right(float v) {
  return __int_as_float(
      __builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130 /* wave_shl:1 */, 0xf, 0xf, false));
}

// A row of heights: the lane's column and its neighbours.
struct Row {
  float l, m, r;
};

__device__ __forceinline__ void normal_at(const Row& a, const Row& b, const Row& c, float inv6r,
                                          float& nx, float& ny, float& nz) {
  const float dxm = a.r - a.l;
  const float dx0 = b.r - b.l;
  const float dxp = c.r - c.l;
  const float dym = c.l - a.l;
  const float dy0 = c.m - a.m;
  const float dyp = c.r - a.r;
  const float gxv = ((dxm + dx0) + dxp) * inv6r;
  const float gyv = ((dym + dy0) + dyp) * inv6r;
  const float q = (gxv * gxv + gyv * gyv) + 1.0f;
  const float inv = 1.0f / sqrtf(q);
  nx = -gxv * inv;
  ny = -gyv * inv;
  nz = inv;
}

// The weights through the scalar cache: uniform, and written by no kernel of
// this launch.
typedef const __attribute__((address_space(4))) float* Weights;

// Normals and/or traversability of one output tile.
template <int kRows>
__device__ __forceinline__ void cells_body(const Item& it, int64_t unit, bool do_n, bool do_t) {
  const Consts& c = it.c;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int ux = (c.nx + kSW - 1) / kSW;
  const int uy = (int)(unit / ux);
  const int gx = (int)(unit - (int64_t)uy * ux) * kSW - 1 + lane;
  const int y0 = uy * tile_rows(kRows) + wave * kRows;
  if (y0 >= c.ny) return;
  const bool col = gx >= 0 && gx < c.nx;
  int px = gx + c.ox;
  px = col ? px - (px >= c.nx ? c.nx : 0) : 0;
  // physical cells of rows y0 - 1 .. y0 + kRows; a row outside the map reads row 0
  uint32_t o[kRows + 2];
  float h[kRows + 2];
  uint8_t ok[kRows + 2];
#pragma unroll
  for (int r = 0; r < kRows + 2; ++r) {
    const int gy = y0 - 1 + r;
    int py = gy + c.oy;
    py = gy >= 0 && gy < c.ny ? py - (py >= c.ny ? c.ny : 0) : 0;
    o[r] = (uint32_t)py * (uint32_t)c.nx + (uint32_t)px;
    h[r] = it.L.h[o[r]];
    ok[r] = it.L.valid[o[r]];
  }
  uint64_t m[kRows + 2];  // the row's valid cells whose neighbours in the row are valid
#pragma unroll
  for (int r = 0; r < kRows + 2; ++r) {
    const int gy = y0 - 1 + r;
    const uint64_t v = gy >= 0 && gy < c.ny ? __ballot(col && ok[r] != 0) : 0ull;
    m[r] = v & (v << 1) & (v >> 1);
  }
  Row row[kRows + 2];
#pragma unroll
  for (int r = 0; r < kRows + 2; ++r) row[r] = Row{from_left(h[r]), h[r], from_right(h[r])};
  const bool out = col && lane >= 1 && lane <= kSW;
  const float qnan = __builtin_nanf("");
  bool win[kRows];
  uint64_t any = 0;
#pragma unroll
  for (int j = 0; j < kRows; ++j) {
    const uint64_t w = m[j] & m[j + 1] & m[j + 2];
    any |= w;
    win[j] = (w >> lane) & 1u;
  }
  if (do_n) {
#pragma unroll
    for (int j = 0; j < kRows; ++j) {
      float nx = qnan, ny = qnan, nz = qnan;
      if (win[j]) normal_at(row[j], row[j + 1], row[j + 2], c.inv6r, nx, ny, nz);
      if (out && y0 + j < c.ny) {
        it.L.nx[o[j + 1]] = nx;
        it.L.ny[o[j + 1]] = ny;
        it.L.nz[o[j + 1]] = nz;
      }
    }
  }
  if (do_t) {
    const Weights w = (Weights)(uintptr_t)it.w;
    float T[kRows];
    if (any) {  // some window of the wave is valid
#pragma unroll
      for (int j = 0; j < kRows; ++j) T[j] = w[88];
#pragma unroll
      for (int ch = 0; ch < 8; ++ch) {
#pragma unroll
        for (int j = 0; j < kRows; ++j) {
          float acc = w[72 + ch];
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            acc = fmaf(w[ch * 9 + 3 * k], row[j + k].l, acc);
            acc = fmaf(w[ch * 9 + 3 * k + 1], row[j + k].m, acc);
            acc = fmaf(w[ch * 9 + 3 * k + 2], row[j + k].r, acc);
          }
          T[j] = fmaf(w[80 + ch], fmaxf(acc, 0.0f), T[j]);
        }
      }
    }
#pragma unroll
    for (int j = 0; j < kRows; ++j)
      if (out && y0 + j < c.ny) it.L.trav[o[j + 1]] = win[j] ? T[j] : qnan;
  }
}

// ---------------------------------------------------------------- launches
__global__ __launch_bounds__(kNTf) void k_move(Item it) {
  move_body<kNTf>(it, blockIdx.x);
}
// One workgroup per output tile, each XCD taking a contiguous range of tiles.
__global__ __launch_bounds__(kNTf) void k_cells(Item it, bool do_n, bool do_t) {
  cells_body<kRowsPlain>(it, xcd_unit(blockIdx.x, gridDim.x), do_n, do_t);
}

// Each XCD takes a contiguous range of the batch's tiles (xcd_unit_k).
__global__ __launch_bounds__(kNTf) void k_cells_b(const Batch* bt) {
  const UnitFinder units(bt, kBCells);
  for (int64_t k = 0;; ++k) {
    const int64_t w = xcd_unit_k(blockIdx.x, gridDim.x, units.total(), k);
    if (w < 0) break;
    int64_t unit;
    const int i = units.find(w, unit);
    const Item& it = bt->items[i];
    cells_body<kRowsBatch>(it, unit, (it.stages & kStageNormals) != 0,
                          (it.stages & kStageTrav) != 0);
  }
}

}  // namespace

static int64_t cells_tiles(int nx, int ny, int rows) {
  return (int64_t)((nx + kSW - 1) / kSW) * ((ny + tile_rows(rows) - 1) / tile_rows(rows));
}
int64_t cells_units(int nx, int ny) { return cells_tiles(nx, ny, kRowsBatch); }

hipError_t launch_fill_prior(const Consts& c, const Layers& L, uint32_t* ctl, int nctl,
                             hipStream_t stream) {
  FillArgs a;
  a.c = c;
  a.L = L;
  a.cells = (int64_t)c.nx * c.ny;
  a.ctl = ctl;
  a.nctl = ctl ? nctl : 0;
  const int64_t n = a.cells > a.nctl ? a.cells : a.nctl;
  TimedLaunch tl("k_fill_prior", stream);
  hipLaunchKernelGGL(k_fill_prior, dim3((unsigned)((n + kNTf - 1) / kNTf)), dim3(kNTf), 0, stream,
                     a);
  return hipGetLastError();
}

hipError_t launch_overlap(const OverlapArgs& a, hipStream_t stream) {
  const int64_t C = (int64_t)a.c.nx * a.c.ny;
  TimedLaunch tl("k_overlap", stream);
  hipLaunchKernelGGL(k_overlap, dim3((unsigned)((C + kNTf - 1) / kNTf)), dim3(kNTf), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_move(const Item& it, hipStream_t stream) {
  const int64_t units = (strips_of(it).cells + kNTf - 1) / kNTf;
  if (units == 0) return hipSuccess;
  TimedLaunch tl("k_move", stream);
  hipLaunchKernelGGL(k_move, dim3((unsigned)units), dim3(kNTf), 0, stream, it);
  return hipGetLastError();
}

static hipError_t launch_cells(const Item& it, const char* name, bool do_n, bool do_t,
                               hipStream_t stream) {
  TimedLaunch tl(name, stream);
  const int nx = it.c.nx, ny = it.c.ny;
  hipLaunchKernelGGL(k_cells, dim3((unsigned)cells_tiles(nx, ny, kRowsPlain)), dim3(kNTf), 0,
                     stream, it, do_n, do_t);
  return hipGetLastError();
}

hipError_t launch_normals(const Item& it, hipStream_t stream) {
  return launch_cells(it, "k_normals", true, false, stream);
}

hipError_t launch_trav(const Item& it, hipStream_t stream) {
  return launch_cells(it, "k_trav", false, true, stream);
}

hipError_t launch_normals_trav(const Item& it, hipStream_t stream) {
  return launch_cells(it, "k_normals_trav", true, true, stream);
}

hipError_t launch_cells_batch(const Batch* d_batch, int grid, hipStream_t stream) {
  {
    TimedLaunch tl("k_cells_b", stream);
    hipLaunchKernelGGL(k_cells_b, dim3(grid), dim3(kNTf), 0, stream, d_batch);
  }
  return hipGetLastError();
}

}  // namespace emx
