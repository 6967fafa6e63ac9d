// Device-side definitions shared by the emx kernels (gfx950, wave64).
//
// Every file of this library is compiled with -ffp-contract=off and correctly
// rounded float32 division/sqrt.  Kernels that take decisions (binning, gate,
// ray samples, clearing predicate) rely on that to reproduce the operation
// order the ABI documents exactly.
//
// Every kernel body works on one `Item`: one map with one frame.  It is called
// either from a plain launch (the Item passed by value, one workgroup per unit
// of work) or from a batched launch that looks its units up in a
// device-resident `Batch` table.  The arithmetic is the same code either way,
// so a map's results are identical alone and in a batch.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace emx {

// Points per fusion work unit (one workgroup of pass 1, the wall counts and
// the drift partials).
constexpr int kChunk = 1024;
// Map tiles of 32 x 8 cells: pass 2 of the fusion visits only the tiles the
// frame touched (a 400 x 400 map has 13 x 50 = 650 tiles).
constexpr int kTileLogX = 5;
constexpr int kTileLogY = 3;
constexpr int kTileW = 1 << kTileLogX;
constexpr int kTileH = 1 << kTileLogY;
constexpr int kTileCells = kTileW * kTileH;

// One buffer set of map layers, row-major [ny][nx].
// The map's layers, [ny][nx] each in the ring layout (pcell).
struct Layers {
  float* h;
  float* v;
  int32_t* t;
  float* nx;
  float* ny;
  float* nz;
  float* trav;
  uint8_t* valid;
  uint8_t* mark;  // the fusion's per-cell flags (kMark*); all zero between calls
  float* cmax;    // per logical block: max height over cells a ray may clear (transient)
  float* smax;    // the same per logical superblock (transient)
  float* ub;      // upper bound of the ground height (+inf: none), or null
  float* clr;     // per logical cell: h, or -inf if a ray may not clear it; or pairs of that
                  // and v (with the bound layer {NaN, bound} without an estimate) (transient)
  uint64_t* fx;   // the fusion's fixed-point sums: kFxWords words per physical cell; all
                  // zero between calls
};

// Fixed-point sums of a cell, its words side by side.  A value x enters as the
// integer X = round(x * 2^S) (S: the item's shift for that sum), split as
// X = hi * 2^32 + lo with 0 <= lo < 2^32; the hi and lo parts are summed in
// separate words (hi as two's complement).  Integer addition is associative,
// so the sums do not depend on the order of the atomics that form them: the
// fused result is the same in every run, alone or batched.
enum FxWord { kFxWhi = 0, kFxWlo, kFxZhi, kFxZlo, kFxWords };  // sum 1/sp2; sum rz/sp2

// Clearing prunes samples by square blocks of 8 x 8 cells and superblocks of
// 32 x 32 cells (one workgroup of the setup each).
constexpr int kBlockLog = 3;
constexpr int kSuperLog = 5;
__host__ __device__ inline int blocks_of(int n, int b) { return (n + (1 << b) - 1) >> b; }

// Float32 constants derived once on the host from emx_params.
struct Consts {
  float inv_r;     // float32(1/r)
  float rmin2;     // float32(min_range^2)
  float k2;        // float32(gate_k^2)
  float alpha;     // noise_alpha
  float an2;       // float32(clear_normal_alpha^2)
  float inv_step;  // float32(1/ray_step)
  float inv6r;     // float32(1/(6 r))
  float h_init;
  float v_init;
  float nxf, nyf;  // nx, ny as float (exact)
  int nx, ny;
  int32_t tau;     // clear_min_age_ms
  float var_t;     // time variance per fusion, 0 = off
  int32_t wall;    // wall/edge rule threshold, 0 = off
  int32_t excl_on;     // exclusion area on
  float excl_slope;    // float32(tan(theta_a))
  float excl_b, excl_c, excl_d;
  float var_o;     // outlier variance per fusion, 0 = off
  int ox, oy;      // ring origin: physical column and row of logical cell (0, 0)
};

// Sensor -> map-local transform, float32.
struct Pose32 {
  float R[9];
  float t[3];
};

struct FuseScratch {
  uint32_t* tcnt;       // [T] nonzero if pass 1 added to a cell of the tile; part of the
                        // map state, zero between calls (pass 2 resets it)
  uint32_t* count;      // [nx * ny] the frame's valid points per cell (wall rule), or null
};

// Stages of one frame, in pipeline order.
constexpr uint32_t kStageMove = 1u;
constexpr uint32_t kStageFuse = 2u;
constexpr uint32_t kStageClear = 4u;
constexpr uint32_t kStageNormals = 8u;
constexpr uint32_t kStageTrav = 16u;

// One map with one frame: everything a kernel body reads.
struct Item {
  Consts c;
  Pose32 P;
  Layers L;     // the map's layers (ring layout; c holds the origin after any move)
  const float* x;
  const float* y;
  const float* z;
  int64_t n;
  int32_t t_now;
  int sx, sy;   // move shift in cells (the cells entering the map)
  uint32_t stages;
  const float* w;  // traversability weights (89)
  int32_t* out_cell;
  uint8_t* out_accept;
  uint8_t* out_cleared;
  FuseScratch fs;
  int fxw, fxz;      // fixed-point shifts S of the sums of 1/sp2 and rz/sp2 (FxWord)
  int tiles_x, T, B;
  int bx, by;        // clearing blocks
  int sbx, sby;      // clearing superblocks
  int grp;           // clearing samples to a group: at most 7 cells of travel; 0 if these
                     // would be fewer than 3 (each sample by itself)
  int32_t index;     // position in its batch
};

// Batched launches: a device-resident table of items and, per stage, the
// prefix of work units over the items.
constexpr int kMaxItems = 64;
// kBZero, kBCount: the wall/edge rule's per-cell counts (zeroed, then
// counted); kBVar: the per-cell time and outlier variance after the fusion.
enum BatchStage {
  kBMove = 0, kBZero, kBCount, kBChunk, kBTile, kBVar, kBSetup, kBRays, kBSparse, kBCells,
  kBNum
};

// Only the header and the first n items are uploaded for a batch of n.  Units fit 32
// bits: the smallest hold 128 points or 256 cells, of 64 items of less than 2^31
// points and at most 2^28 cells each.
struct Batch {
  int n;
  int32_t off[kBNum][kMaxItems + 1];
  Item items[kMaxItems];
};

struct PointEval {
  float xm, ym, zm, d2, sp2;
  float rz;  // the rotated point's height (zm before the translation is added)
  bool valid;
};

// Transform, range and noise of one sensor-frame point, in the ABI's order.
__device__ __forceinline__ PointEval eval_point(const Pose32& P, const Consts& c, float xs,
                                                float ys, float zs) {
  PointEval e;
  e.xm = ((P.R[0] * xs + P.R[1] * ys) + P.R[2] * zs) + P.t[0];
  e.ym = ((P.R[3] * xs + P.R[4] * ys) + P.R[5] * zs) + P.t[1];
  e.rz = (P.R[6] * xs + P.R[7] * ys) + P.R[8] * zs;
  e.zm = e.rz + P.t[2];
  e.d2 = (xs * xs + ys * ys) + zs * zs;
  e.sp2 = c.alpha * e.d2;
  e.valid = isfinite(xs) && isfinite(ys) && isfinite(zs) && isfinite(e.d2) &&
            (e.d2 >= c.rmin2) && isfinite(e.sp2);
  return e;
}

// Exclusion area: the point lies above the line around the sensor origin
// (Pose32::t), in the ABI's float32 order.
__device__ __forceinline__ bool excluded_point(const Pose32& P, const Consts& c,
                                               const PointEval& e) {
  const float dxr = e.xm - P.t[0];
  const float dyr = e.ym - P.t[1];
  const float rho = sqrtf(dxr * dxr + dyr * dyr);
  const float eup = e.zm - P.t[2];
  const float line = fminf(c.excl_b + c.excl_slope * fmaxf(rho - c.excl_c, 0.0f), c.excl_d);
  return eup > line;
}

// Mark layer bits between the fusion's passes and its per-cell pass.
constexpr uint8_t kMarkUpdated = 1;   // pass 2 updated the cell
constexpr uint8_t kMarkOutlier = 2;   // a gate-rejected point fell in the (valid) cell

// Half-open binning of map-local float32 coordinates; false outside.
__device__ __forceinline__ bool bin_xy(float xm, float ym, const Consts& c, int& ix, int& iy) {
  const float fx = xm * c.inv_r;
  const float fy = ym * c.inv_r;
  if (!(fx >= 0.0f && fx < c.nxf && fy >= 0.0f && fy < c.nyf)) return false;
  ix = (int)floorf(fx);
  iy = (int)floorf(fy);
  return true;
}

// ---------------------------------------------------------------- ring layout
// The map is stored as a ring (a circular buffer in both axes): logical cell
// (ix, iy) lives at physical cell pcell(c, ix, iy), with the origin (ox, oy)
// the physical column and row of logical (0, 0).  A move turns the ring
// instead of copying the layers; only the cells that enter the map are reset.
__host__ __device__ __forceinline__ int64_t pcell(const Consts& c, int ix, int iy) {
  int px = ix + c.ox;
  px -= (px >= c.nx) ? c.nx : 0;
  int py = iy + c.oy;
  py -= (py >= c.ny) ? c.ny : 0;
  return (int64_t)py * c.nx + px;
}

// Physical cell o back to the prior: no estimate, no normal or
// traversability, no bound; the mark is cleared.
__device__ __forceinline__ void prior_cell(const Consts& c, const Layers& L, int64_t o) {
  const float qnan = __builtin_nanf("");
  L.h[o] = c.h_init;
  L.v[o] = c.v_init;
  L.t[o] = 0;
  L.nx[o] = qnan;
  L.ny[o] = qnan;
  L.nz[o] = qnan;
  L.trav[o] = qnan;
  L.valid[o] = 0;
  L.mark[o] = 0;
  if (L.ub) L.ub[o] = INFINITY;
}

// ------------------------------------------------------------------------ move
// The ring has already turned (it.c holds the new origin); the cells that
// enter the map go back to the prior.  With a shift (sx, sy) they are the
// logical columns [nx - sx, nx) (sx > 0) or [0, -sx) (sx < 0) in every row,
// and the logical rows [ny - sy, ny) or [0, -sy) in every column; a shift of a
// whole side resets every cell.  One thread per cell: the column strip, then
// the row strip (their corner twice, with the same values).  Where the move is
// followed by a fusion, its pass 1 resets the cells in the same launch and
// takes the prior for entering cells itself (entering).
struct Strips {
  int ncol, nrow;   // entering columns and rows
  bool all;         // every cell enters
  int64_t cells;    // threads needed
};

__host__ __device__ __forceinline__ Strips strips_of(const Item& it) {
  Strips s;
  const int ax = it.sx < 0 ? -it.sx : it.sx;
  const int ay = it.sy < 0 ? -it.sy : it.sy;
  s.ncol = ax < it.c.nx ? ax : it.c.nx;
  s.nrow = ay < it.c.ny ? ay : it.c.ny;
  s.all = s.ncol == it.c.nx || s.nrow == it.c.ny;
  s.cells = s.all ? (int64_t)it.c.nx * it.c.ny
                  : (int64_t)s.ncol * it.c.ny + (int64_t)s.nrow * it.c.nx;
  return s;
}

// Whether logical cell (ix, iy) has entered the map with the item's move.
__device__ __forceinline__ bool entering(const Item& it, int ix, int iy) {
  return (it.sx > 0 && ix >= it.c.nx - it.sx) || (it.sx < 0 && ix < -it.sx) ||
         (it.sy > 0 && iy >= it.c.ny - it.sy) || (it.sy < 0 && iy < -it.sy);
}

// Unit `unit` of kT of the entering cells, one per thread.
template <int kT>
__device__ __forceinline__ void move_body(const Item& it, int64_t unit) {
  const Strips st = strips_of(it);
  const int64_t q = unit * kT + threadIdx.x;
  if (q >= st.cells) return;
  int ix, iy;
  if (st.all) {
    iy = (int)(q / it.c.nx);
    ix = (int)(q - (int64_t)iy * it.c.nx);
  } else if (q < (int64_t)st.ncol * it.c.ny) {
    iy = (int)(q / st.ncol);
    const int k = (int)(q - (int64_t)iy * st.ncol);
    ix = it.sx > 0 ? it.c.nx - st.ncol + k : k;
  } else {
    const int64_t q2 = q - (int64_t)st.ncol * it.c.ny;
    const int k = (int)(q2 / it.c.nx);
    ix = (int)(q2 - (int64_t)k * it.c.nx);
    iy = it.sy > 0 ? it.c.ny - st.nrow + k : k;
  }
  prior_cell(it.c, it.L, pcell(it.c, ix, iy));
}

// ------------------------------------------------------------- batched units
// The item that holds a global work unit of a stage.  Each lane of a wave keeps
// the end of one item's units (kMaxItems lanes), so that finding an item is one
// comparison and a ballot; a search in memory would put six dependent loads,
// each a trip to the L2, before every unit's work.  Every lane of the wave
// calls both members, with the same w.
class UnitFinder {
 public:
  __device__ __forceinline__ UnitFinder(const Batch* bt, int stage) {
    static_assert(kMaxItems == 64, "one lane per item");
    const int lane = threadIdx.x & 63;
    n_ = bt->n;
    total_ = bt->off[stage][n_];
    end_ = lane < n_ ? bt->off[stage][lane + 1] : total_;
  }
  __device__ __forceinline__ int64_t total() const { return total_; }
  // The item of unit w < total(), and the unit's number within it.
  __device__ __forceinline__ int find(int64_t w, int64_t& unit) const {
    const int i = __builtin_amdgcn_readfirstlane(__popcll(__ballot(end_ <= (int)w)));
    const int before = __builtin_amdgcn_readlane(end_, i > 0 ? i - 1 : 0);
    unit = (int)w - (i > 0 ? before : 0);
    return i;
  }

 private:
  int n_;
  int total_, end_;
};

}  // namespace emx
