// Height fusion (Sec. II-C, Eq. 1 and Eq. 2) with exact integer sums and no
// float atomics.
//
// Eq. 2 fuses a cell's accepted points through two sums, of 1/sp2 and of
// zm/sp2.  Both are formed in fixed point: a term x enters as the integer
// round(x * 2^S), held as hi * 2^32 + lo (FxWord), with one shift S per sum and
// frame chosen on the host so that no sum can overflow (fuse_fixed_shifts).
// Integer addition is associative, so the sums come out the same whatever the
// order the additions land in: results are bitwise identical from run to run,
// alone or batched, whatever the grid shape.
//
// Pass 1, chunk body: one workgroup per chunk of consecutive points, consecutive
// points in consecutive lanes.
//   - Takes the per-point decisions: transform, range, bin, exclusion area,
//     wall/edge rule, and the Mahalanobis gate against the frame-start prior.
//   - Converts an accepted point's 1/sp2 and rz/sp2 to fixed point (rz: the
//     rotated point's height, zm = rz + tz; tz * sum 1/sp2 is added back in
//     pass 2, which keeps the terms independent of the sensor's height).
//   - Sums the chunk's points per cell in an LDS table: the first lane of each
//     run of one cell finds the run's slot (sensors emit points in scan order,
//     so most runs span several points), then every lane adds its own words
//     with LDS integer atomics.  Words that are zero, as the low words of most
//     terms are at these scales, are not added.  A segmented scan of the four
//     words over the wave in front of the table cost 54 cross-lane moves per
//     wave and four such scans in a row per thread: 15 against 9 us for a 300k
//     frame, 144 against 80 us for a batch of 16 maps, each at the time.
//   - Adds the chunk's sums to the cells' words (FxWord) with integer atomics,
//     from a list of the slots taken, four neighbouring lanes to a cell: its
//     words lie side by side, so a cell's atomics are one request, and the pass
//     has no idle lanes.  With a plane for each word and a scan of all slots the
//     atomics were a fourth to a third of the pass (300k points: 9.6 -> 6.9 us,
//     4M: 42 -> 41, 16 maps: 80 -> 75; pass 2, which takes a cell's words in two
//     loads, 21 -> 18 us for 16 maps).  The cells' tiles are flagged.
//   - Where the call moves the map first, further workgroups of the same launch
//     reset the entering cells, and points in them take the prior (a launch of
//     its own took 3 us of every frame).
// Pass 2, tile body: per 32 x 8-cell tile of the physical layout, a workgroup
// with one thread per cell (plain calls) or one wave with four cells per lane
// (batches).  An unflagged tile returns after one load;
// otherwise the flag is reset, and each cell with a nonzero sum converts its
// sums back to floating point, applies the information-form update once and
// resets its words to zero for the next call.
#include <math.h>

#include "emx_kernels.h"

namespace emx {

namespace {

constexpr uint32_t kNoCell = 0xFFFFFFFFu;   // lanes without an accepted point

// The integer X = round(x * 2^S) (ties to even) of an x with 24 significant bits,
// as X = hi * 2^32 + lo with 0 <= lo < 2^32.  Every step is exact in float64: the
// choice of S keeps |X| < 2^94.
__device__ __forceinline__ void fx_split(double x, int S, int64_t& hi, uint64_t& lo) {
  const double d = rint(ldexp(x, S));
  const double h = floor(d * 0x1p-32);
  hi = (int64_t)h;
  lo = (uint64_t)(uint32_t)fma(h, -0x1p32, d);
}

// (hi * 2^32 + lo) * 2^-S in float64.
__device__ __forceinline__ double fx_value(int64_t hi, uint64_t lo, int S) {
  return ldexp((double)hi * 4294967296.0 + (double)lo, -S);
}

// ------------------------------------------------------------------ pass 1
// A chunk's sums are gathered per cell in an LDS table before they go to the
// map: kAggSlots slots of (cell + 1, four words), open addressing with at most
// kAggProbes probes.  A run that finds no slot adds to the map directly.
constexpr int kAggLog = 9;
constexpr int kAggSlots = 1 << kAggLog;
constexpr int kAggProbes = 8;
constexpr uint32_t kNoSlot = 0xFFFFFFFFu;

// Chunks.  A frame alone takes one point per thread: its few workgroups wait for
// each step of their chain, and four points per thread put four of each step in
// a row.  Up to one 256-point chunk for each compute unit (20k points on 128 x
// 128 cells: 4.6 against 5.9 us with 1024; 43k on 250 x 250: 4.9 against 6.7);
// above, 1024-point chunks, whose table joins more of a cell's runs before the
// map's atomics (300k on 400 x 400: 9.1 against 13.2 us with 256).  A batch has
// workgroups to spare, and 256 threads with four points each leave more of them
// in flight (16 maps, 4.6M points: 80 against 91 us; 512 threads with four points
// 72 against 75, but 38 against 36 for a server's batch of 8 maps).  They take 128
// registers, four waves to a SIMD; a bound of five spills (75 -> 108 us).
constexpr int64_t kSmallFrame = 65536;
constexpr int kThreadsLarge = 1024;
constexpr int kThreadsBatch = 256;
constexpr int kPointsBatch = 4;

struct AggTable {
  uint32_t key[kAggSlots];                   // physical cell + 1; 0 = free
  // the words, a plane each; the stride keeps eight slots' words in distinct banks
  unsigned long long v[kFxWords][kAggSlots + 8];
  uint32_t used[kAggSlots];                   // the slots taken
  int n;                                      // how many, over all chunks of the workgroup
};

__device__ __forceinline__ void add_to_map(const Item& it, uint32_t cell, const uint64_t (&v)[4]) {
#pragma unroll
  for (int k = 0; k < kFxWords; ++k)
    if (v[k]) atomicAdd((unsigned long long*)(it.L.fx + kFxWords * (int64_t)cell + k), v[k]);
}

__device__ __forceinline__ uint32_t tile_of_cell(const Item& it, uint32_t cell) {
  const uint32_t py = cell / (uint32_t)it.c.nx;
  const uint32_t px = cell - py * (uint32_t)it.c.nx;
  return (py >> kTileLogY) * (uint32_t)it.tiles_x + (px >> kTileLogX);
}

// Zeroes the table (every thread of the block; the caller synchronises).
template <int kT>
__device__ __forceinline__ void agg_clear(AggTable& t) {
  if (threadIdx.x == 0) t.n = 0;
  for (int s = threadIdx.x; s < kAggSlots; s += kT) {
    t.key[s] = 0u;
#pragma unroll
    for (int k = 0; k < kFxWords; ++k) t.v[k][s] = 0ull;
  }
}

// One chunk of kT * kP points; a thread takes kP of them, kT apart, so that
// consecutive points lie in consecutive lanes.  On entry the table is zero but
// for n, which is n0; so it is again on return, with the next n0 (a count that
// goes on needs no reset, and so no barrier between the flush and the next chunk's
// first slot).
template <int kT, int kP>
__device__ __forceinline__ void chunk_body(const Item& it, int64_t chunk, AggTable& tab, int& n0) {
  const int lane = threadIdx.x & 63;
  float x[kP], y[kP], z[kP];
#pragma unroll
  for (int j = 0; j < kP; ++j) {
    const int64_t i = (chunk * kP + j) * kT + threadIdx.x;
    const bool in = i < it.n;  // past the end: a point at the sensor, never valid
    x[j] = in ? it.x[i] : 0.0f;
    y[j] = in ? it.y[i] : 0.0f;
    z[j] = in ? it.z[i] : 0.0f;
  }
  // the priors of the thread's points, every load issued before any is used
  PointEval e[kP];
  uint32_t pc[kP], cnt[kP];
  int cell[kP];
  float h0[kP], v0[kP];
  uint8_t vd[kP];
  bool gated[kP];
#pragma unroll
  for (int j = 0; j < kP; ++j) {
    e[j] = eval_point(it.P, it.c, x[j], y[j], z[j]);
    int ix = 0, iy = 0;
    const bool inmap = e[j].valid && bin_xy(e[j].xm, e[j].ym, it.c, ix, iy);
    cell[j] = inmap ? iy * it.c.nx + ix : -1;
    // points of the exclusion area are ignored
    gated[j] = inmap && (!it.c.excl_on || !excluded_point(it.P, it.c, e[j]));
    pc[j] = 0;
    h0[j] = it.c.h_init;
    v0[j] = it.c.v_init;
    cnt[j] = 0u;
    vd[j] = 0;
    if (gated[j]) {
      pc[j] = (uint32_t)pcell(it.c, ix, iy);
      if (!entering(it, ix, iy)) {  // else the prior, which this launch is storing
        h0[j] = it.L.h[pc[j]];
        v0[j] = it.L.v[pc[j]];
        if (it.fs.count) cnt[j] = it.fs.count[pc[j]];
        if (it.fs.count || it.c.var_o != 0.0f) vd[j] = it.L.valid[pc[j]];
      }
    }
  }
#pragma unroll
  for (int j = 0; j < kP; ++j) {
    const int64_t i = (chunk * kP + j) * kT + threadIdx.x;
    uint32_t key = kNoCell;  // the accepted point's physical cell
    uint64_t v[kFxWords] = {0, 0, 0, 0};
    bool acc = false;
    if (gated[j]) {
      const float d = e[j].zm - h0[j];
      const bool inside = (d * d) <= (it.c.k2 * (v0[j] + e[j].sp2));
      // wall/edge rule: in a crowded cell that holds an estimate, points
      // below the estimate are ignored (before the gate)
      const bool walled =
          it.fs.count && e[j].zm < h0[j] && cnt[j] > (uint32_t)it.c.wall && vd[j];
      acc = inside && !walled;
      // a gate-rejected point in a cell with an estimate flags the cell for
      // the outlier variance (a plain store: every writer stores 2)
      if (it.c.var_o != 0.0f && !inside && !walled && vd[j]) it.L.mark[pc[j]] = kMarkOutlier;
      if (acc) {
        key = pc[j];
        const float w = 1.0f / e[j].sp2;
        int64_t hi;
        fx_split(w, it.fxw, hi, v[kFxWlo]);
        v[kFxWhi] = (uint64_t)hi;
        if (hi == 0 && v[kFxWlo] == 0) v[kFxWlo] = 1;  // an accepted point adds at least one unit
        // a term past float32's range counts as 2^128, the power above it (w itself
        // is bounded by 1/sp2 of the nearest point, which is in range)
        const float u = w * e[j].rz;
        fx_split(isinf(u) ? copysign(0x1p128, (double)u) : (double)u, it.fxz, hi, v[kFxZlo]);
        v[kFxZhi] = (uint64_t)hi;
      }
    }
    if (i < it.n) {
      if (it.out_cell) it.out_cell[i] = cell[j];
      if (it.out_accept) it.out_accept[i] = acc ? 1 : 0;
    }
    // the first lane of each run of one cell finds the run's slot ...
    const uint32_t prev = (uint32_t)__shfl_up((int)key, 1, 64);
    const bool head = key != kNoCell && (lane == 0 || prev != key);
    const uint64_t heads = __ballot(head);
    if (heads == 0) continue;
    uint32_t slot = kNoSlot;
    bool fresh = false;
    if (head) {
      uint32_t h = (key * 2654435761u) >> (32 - kAggLog);
      for (int p = 0; p < kAggProbes; ++p) {
        const uint32_t was = atomicCAS(&tab.key[h], 0u, key + 1u);
        if (was == 0u || was == key + 1u) {
          slot = h;
          fresh = was == 0u;
          break;
        }
        h = (h + 1u) & (kAggSlots - 1);
      }
    }
    const uint64_t fr = __ballot(fresh);
    if (fr != 0) {  // slots taken: one atomic per wave
      int at = 0;
      if (lane == 0) at = atomicAdd(&tab.n, __popcll(fr));
      at = __builtin_amdgcn_readfirstlane(at) - n0;
      if (fresh)
        tab.used[at + __builtin_amdgcn_mbcnt_hi((uint32_t)(fr >> 32),
                                                __builtin_amdgcn_mbcnt_lo((uint32_t)fr, 0u))] =
            slot;
    }
    // ... and its lanes add to it, or straight to the map
    const uint64_t upto = heads & (~0ull >> (63 - lane));
    slot = (uint32_t)__shfl((int)slot, upto ? 63 - __builtin_clzll(upto) : 0, 64);
    if (key != kNoCell) {
      if (slot != kNoSlot) {
#pragma unroll
        for (int k = 0; k < kFxWords; ++k)
          if (v[k]) atomicAdd(&tab.v[k][slot], (unsigned long long)v[k]);
      } else {
        add_to_map(it, key, v);
        it.fs.tcnt[tile_of_cell(it, key)] = 1u;
      }
    }
  }
  __syncthreads();
  // the table's cells to the map, the table back to zero
  const int n1 = tab.n;
  const int items = (n1 - n0) * kFxWords;
  n0 = n1;
  for (int f = threadIdx.x; f < items; f += kT) {
    const uint32_t s = tab.used[f / kFxWords];
    const int k = f % kFxWords;
    const uint32_t c = tab.key[s] - 1u;
    const unsigned long long t = tab.v[k][s];
    if (t) {
      atomicAdd((unsigned long long*)(it.L.fx + kFxWords * (int64_t)c + k), t);
      tab.v[k][s] = 0ull;
    }
    // a slot's four lanes lie in one wave: all have read its key before the first of
    // them resets it (order for the compiler; no instructions)
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (k == 0) {
      it.fs.tcnt[tile_of_cell(it, c)] = 1u;
      tab.key[s] = 0u;
    }
  }
  __syncthreads();
}

// ------------------------------------------------------------------ pass 2
constexpr int kNT2 = kTileCells;               // plain pass 2: one thread per cell of the tile
constexpr int kNT2b = 256;                     // batched pass 2: one wave per tile
constexpr int kTilesPerGroup = kNT2b / 64;
constexpr int kCellsPerLane = kTileCells / 64;  // 4: lane l owns cells l, l + 64, ...

// Information-form update of physical cell `cell` from its sums (Σw's words
// whi, wlo given, not both zero); the sums are reset to zero.
__device__ __forceinline__ void update_cell(const Item& it, int64_t cell, int64_t whi,
                                            uint64_t wlo, int64_t zhi, uint64_t zlo, float h0,
                                            float v0) {
  ulonglong2* f = reinterpret_cast<ulonglong2*>(it.L.fx + kFxWords * cell);
  f[0] = f[1] = make_ulonglong2(0u, 0u);
  const double sw = fx_value(whi, wlo, it.fxw);
  const double srz = fx_value(zhi, zlo, it.fxz);
  const float acc_w = (float)sw;
  const float acc_wz = (float)(srz + (double)it.P.t[2] * sw);
  const float W = (1.0f / v0) + acc_w;
  const float v1 = 1.0f / W;
  const float h1 = ((h0 / v0) + acc_wz) * v1;
  it.L.h[cell] = h1;
  it.L.v[cell] = v1;
  it.L.t[cell] = it.t_now;
  it.L.valid[cell] = 1;
  // updated: no time variance (the owning thread keeps pass 1's outlier flag)
  if (it.c.var_t != 0.0f) it.L.mark[cell] = it.L.mark[cell] | kMarkUpdated;
}

// Tile t, by a workgroup of kNT2 threads, one cell each: the plain call's
// form, where a single frame's tiles are few and each cell's loads should be
// in flight at once.
__device__ __forceinline__ void tile_body_group(const Item& it, int64_t t) {
  if (it.fs.tcnt[t] == 0u) return;  // uniform: the frame added to no cell of the tile
  __syncthreads();                  // every thread has read the flag
  if (threadIdx.x == 0) it.fs.tcnt[t] = 0u;  // zero again for the next call
  const int l = threadIdx.x;
  const int tx = (int)(t % it.tiles_x);
  const int ty = (int)(t / it.tiles_x);
  // the owned cell, physical (tiles cover the ring layout as stored)
  const int px = (tx << kTileLogX) + (l & (kTileW - 1));
  const int py = (ty << kTileLogY) + (l >> kTileLogX);
  if (px >= it.c.nx || py >= it.c.ny) return;
  const int64_t cell = (int64_t)py * it.c.nx + px;
  const ulonglong2* f = reinterpret_cast<const ulonglong2*>(it.L.fx + kFxWords * cell);
  const ulonglong2 w = f[0], z = f[1];
  if (w.x == 0 && w.y == 0) return;  // no accepted point: every term is positive
  update_cell(it, cell, (int64_t)w.x, w.y, (int64_t)z.x, z.y, it.L.h[cell], it.L.v[cell]);
}

// Tile t, by one wave: lane l takes cells l + 64 i of the tile (two rows of 32
// per step), their loads issued together.  The batched form: a batch holds tens
// of thousands of tiles, many untouched, so a workgroup's waves take one tile
// each and an untouched tile costs one wave one load.  The same update_cell as
// the plain form: the same bits.  (Tiles of 32 x 16 cells took a wave two rounds
// of loads: 17.7 against 13.9 us for a server's batch of 8 maps, 24.1 against 21.8 us
// for 16 maps.)
__device__ __forceinline__ void tile_body_wave(const Item& it, int64_t t) {
  const int lane = threadIdx.x & 63;
  if (it.fs.tcnt[t] == 0u) return;  // wave-uniform: the frame added to no cell of the tile
  // the flag's load has completed for the whole wave (the branch used it)
  if (lane == 0) it.fs.tcnt[t] = 0u;  // zero again for the next call
  const int tx = (int)(t % it.tiles_x);
  const int ty = (int)(t / it.tiles_x);
  int64_t cell[kCellsPerLane];
  ulonglong2 w[kCellsPerLane];
#pragma unroll
  for (int i = 0; i < kCellsPerLane; ++i) {
    const int c = lane + 64 * i;
    // the cell, physical (tiles cover the ring layout as stored)
    const int px = (tx << kTileLogX) + (c & (kTileW - 1));
    const int py = (ty << kTileLogY) + (c >> kTileLogX);
    cell[i] = (int64_t)py * it.c.nx + px;
    w[i] = make_ulonglong2(0u, 0u);
    if (px < it.c.nx && py < it.c.ny)
      w[i] = reinterpret_cast<const ulonglong2*>(it.L.fx + kFxWords * cell[i])[0];
  }
  // cells with an accepted point (every term is positive): the rest of
  // their sums and their prior, all loads issued before any is used
  bool hit[kCellsPerLane];
  ulonglong2 z[kCellsPerLane];
  float h0[kCellsPerLane], v0[kCellsPerLane];
#pragma unroll
  for (int i = 0; i < kCellsPerLane; ++i) {
    hit[i] = w[i].x != 0 || w[i].y != 0;
    z[i] = make_ulonglong2(0u, 0u);
    h0[i] = 0.0f;
    v0[i] = 1.0f;
    if (hit[i]) {
      z[i] = reinterpret_cast<const ulonglong2*>(it.L.fx + kFxWords * cell[i])[1];
      h0[i] = it.L.h[cell[i]];
      v0[i] = it.L.v[cell[i]];
    }
  }
#pragma unroll
  for (int i = 0; i < kCellsPerLane; ++i)
    if (hit[i])
      update_cell(it, cell[i], (int64_t)w[i].x, w[i].y, (int64_t)z[i].x, z[i].y, h0[i], v0[i]);
}

// ------------------------------------------------------- wall rule: counts
// The frame's valid in-map points per cell.  Near the sensor thousands of
// points share a cell, and global atomics on one address serialise, so each
// workgroup first counts its chunk in an LDS hash table (open addressing,
// twice as many slots as points: a free slot always exists) and then adds one
// count per distinct cell.  Integer sums do not depend on their order.  The
// counts are zeroed by the launch before.
// As in pass 1, a frame alone takes one point per thread, a batch four (300k
// points on 400 x 400 cells: 7.4 -> 5.7 us).
constexpr int kCountSlotsLog = 11;
constexpr int kCountSlots = 1 << kCountSlotsLog;
static_assert(kCountSlots >= 2 * kChunk, "the table must keep a free slot");

template <int kT>
__device__ __forceinline__ void count_body(const Item& it, int64_t chunk) {
  __shared__ uint32_t s_key[kCountSlots];  // cell + 1, 0 = empty
  __shared__ uint32_t s_cnt[kCountSlots];
  for (int j = threadIdx.x; j < kCountSlots; j += kT) {
    s_key[j] = 0u;
    s_cnt[j] = 0u;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kChunk / kT; ++j) {
    const int64_t i = chunk * kChunk + j * kT + threadIdx.x;
    if (i >= it.n) continue;
    const PointEval e = eval_point(it.P, it.c, it.x[i], it.y[i], it.z[i]);
    int ix, iy;
    if (!e.valid || !bin_xy(e.xm, e.ym, it.c, ix, iy)) continue;
    if (it.c.excl_on && excluded_point(it.P, it.c, e)) continue;
    const uint32_t key = (uint32_t)pcell(it.c, ix, iy) + 1u;
    uint32_t h = (key * 2654435761u) >> (32 - kCountSlotsLog);
    while (true) {
      const uint32_t prev = atomicCAS(s_key + h, 0u, key);
      if (prev == 0u || prev == key) {
        atomicAdd(s_cnt + h, 1u);
        break;
      }
      h = (h + 1u) & (kCountSlots - 1);
    }
  }
  __syncthreads();
  for (int j = threadIdx.x; j < kCountSlots; j += kT) {
    const uint32_t key = s_key[j];
    if (key) atomicAdd(it.fs.count + (key - 1u), s_cnt[j]);
  }
}

// ------------------------------------- per-cell variances after a fusion
// Time variance: valid cells that the fusion did not update (no kMarkUpdated)
// gain sigma_t^2.  Outlier variance: cells flagged kMarkOutlier by pass 1
// then gain sigma_o^2.  The flags are cleared: marks are zero between calls.
constexpr int kNTv = 256;

__device__ __forceinline__ void timevar_body(const Item& it, int64_t unit) {
  const int64_t i = unit * kNTv + threadIdx.x;
  if (i >= (int64_t)it.c.nx * it.c.ny) return;
  const uint8_t m = it.L.mark[i];
  if (m) it.L.mark[i] = 0;
  const bool grow = it.c.var_t != 0.0f && !(m & kMarkUpdated) && it.L.valid[i];
  const bool outl = (m & kMarkOutlier) != 0;
  if (!grow && !outl) return;
  float v = it.L.v[i];
  if (grow) v = v + it.c.var_t;
  if (outl) v = v + it.c.var_o;
  it.L.v[i] = v;
}

__global__ __launch_bounds__(kChunk) void k_fuse_count(Item it) {
  count_body<kChunk>(it, blockIdx.x);
}

__global__ __launch_bounds__(kNTv) void k_time_variance(Item it) { timevar_body(it, blockIdx.x); }

__global__ __launch_bounds__(256) void k_zero_u32(uint32_t* p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = 0u;
}

// ---------------------------------------------------------------- launches
// The first `chunks` workgroups take points, the others the cells of the move.
template <int kT>
__global__ __launch_bounds__(kT) void k_fuse_chunk(Item it, uint32_t chunks) {
  __shared__ AggTable tab;
  if (blockIdx.x >= chunks) {
    move_body<kT>(it, blockIdx.x - chunks);
    return;
  }
  agg_clear<kT>(tab);
  __syncthreads();
  int n0 = 0;
  chunk_body<kT, 1>(it, blockIdx.x, tab, n0);
}

__global__ __launch_bounds__(kNT2) void k_fuse_tile(Item it) { tile_body_group(it, blockIdx.x); }

__global__ __launch_bounds__(kThreadsBatch, 4) void k_fuse_chunk_b(const Batch* bt) {
  __shared__ AggTable tab;
  agg_clear<kThreadsBatch>(tab);
  __syncthreads();
  const UnitFinder units(bt, kBChunk), moves(bt, kBMove);
  int n0 = 0;
  for (int64_t w = blockIdx.x; w < moves.total() + units.total(); w += gridDim.x) {
    int64_t unit;
    if (w < moves.total()) {
      const int i = moves.find(w, unit);
      move_body<kThreadsBatch>(bt->items[i], unit);
    } else {
      const int i = units.find(w - moves.total(), unit);
      chunk_body<kThreadsBatch, kPointsBatch>(bt->items[i], unit, tab, n0);
    }
  }
}

__global__ __launch_bounds__(256) void k_zero_b(const Batch* bt) {
  const UnitFinder units(bt, kBZero);
  for (int64_t w = blockIdx.x; w < units.total(); w += gridDim.x) {
    int64_t unit;
    const int i = units.find(w, unit);
    const Item& it = bt->items[i];
    const int64_t c = unit * 256 + threadIdx.x;
    if (c < (int64_t)it.c.nx * it.c.ny) it.fs.count[c] = 0u;
  }
}

__global__ __launch_bounds__(kThreadsBatch) void k_fuse_count_b(const Batch* bt) {
  const UnitFinder units(bt, kBCount);
  for (int64_t w = blockIdx.x; w < units.total(); w += gridDim.x) {
    int64_t unit;
    const int i = units.find(w, unit);
    count_body<kThreadsBatch>(bt->items[i], unit);
    __syncthreads();
  }
}

__global__ __launch_bounds__(kNTv) void k_time_variance_b(const Batch* bt) {
  const UnitFinder units(bt, kBVar);
  for (int64_t w = blockIdx.x; w < units.total(); w += gridDim.x) {
    int64_t unit;
    const int i = units.find(w, unit);
    timevar_body(bt->items[i], unit);
  }
}

// Each wave takes its own tiles: units w = (workgroup * kTilesPerGroup +
// wave) + k * (grid * kTilesPerGroup).
__global__ __launch_bounds__(kNT2b) void k_fuse_tile_b(const Batch* bt) {
  const UnitFinder units(bt, kBTile);
  const int64_t step = (int64_t)gridDim.x * kTilesPerGroup;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  for (int64_t w = (int64_t)blockIdx.x * kTilesPerGroup + wave; w < units.total(); w += step) {
    int64_t unit;
    const int i = units.find(w, unit);
    tile_body_wave(bt->items[i], unit);
  }
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Smallest E with x < 2^E, for finite x > 0.
int exp_above(double x) {
  int e = 0;
  const double f = frexp(x, &e);  // x = f * 2^e, 0.5 <= f < 1
  (void)f;
  return e;
}

// Largest shift S with n * bound * 2^S <= 2^93: then every term is below
// 2^94 / n (fx_split's range), and n such terms, plus the unit an accepted
// point may add, stay below 2^94 in total, so the hi words stay below 2^62
// and the lo words, each below 2^32, sum below 2^63 for n < 2^31.
int fixed_shift(double bound, int64_t n) {
  int ln = 0;
  while (((int64_t)1 << ln) < n) ++ln;
  return 93 - ln - exp_above(bound);
}

}  // namespace

int tiles_x_of(int nx) { return (nx + kTileW - 1) >> kTileLogX; }
int tiles_y_of(int ny) { return (ny + kTileH - 1) >> kTileLogY; }

void fuse_fixed_shifts(const Consts& c, const Pose32& P, int64_t n, int* fxw, int* fxz) {
  // Every accepted point has d2 >= rmin2 (float32 comparison), so its float32
  // 1/sp2 is at most 1/fl(alpha * rmin2): rounding is monotone.
  const float sp2min = c.alpha * c.rmin2;
  const double wmax = (double)(1.0f / sp2min);
  // |rz| <= |R20 xs| + |R21 ys| + |R22 zs| <= L1 * sqrt(d2) with the rounding of
  // the three products, two sums, d2 and sp2 bounded by a factor 1 + 2^-20,
  // so |fl(w * rz)| <= L1 / (alpha * sqrt(d2)) * (1 + 2^-20), largest at
  // d2 = rmin2.  The bound below adds a further margin.
  // A row with a non-finite entry makes every rz NaN or infinite: the gate
  // rejects every point, and any shift serves.
  const double l1 = fabs((double)P.R[6]) + fabs((double)P.R[7]) + fabs((double)P.R[8]);
  const double l1b = (l1 > 0.0 && isfinite(l1)) ? l1 : 1.0;
  const double zmax = l1b / ((double)c.alpha * sqrt((double)c.rmin2)) * (1.0 + 1.0 / 1024.0);
  const int64_t nn = n > 1 ? n : 1;
  *fxw = fixed_shift(wmax * (1.0 + 1.0 / 1024.0), nn);
  *fxz = fixed_shift(zmax, nn);
}

size_t fuse_scratch_layout(int64_t count_cells, char* base, FuseScratch* out) {
  if (out && base) out->count = count_cells > 0 ? (uint32_t*)base : nullptr;
  return align256((size_t)count_cells * sizeof(uint32_t));
}

hipError_t launch_fuse(const Item& it, hipStream_t stream) {
  hipError_t err = hipSuccess;
  const int64_t cells = (int64_t)it.c.nx * it.c.ny;
  if (it.n > 0) {
    if (it.fs.count) {  // wall/edge rule: the frame's points per cell first
      {
        TimedLaunch tl("k_zero_u32", stream);
        hipLaunchKernelGGL(k_zero_u32, dim3((unsigned)((cells + 255) / 256)), dim3(256), 0,
                           stream, it.fs.count, cells);
      }
      if ((err = hipGetLastError()) != hipSuccess) return err;
      {
        TimedLaunch tl("k_fuse_count", stream);
        hipLaunchKernelGGL(k_fuse_count, dim3(it.B), dim3(kChunk), 0, stream, it);
      }
      if ((err = hipGetLastError()) != hipSuccess) return err;
    }
    {
      TimedLaunch tl("k_fuse_chunk", stream);
      const int64_t entering = strips_of(it).cells;
      const auto go = [&](auto kernel, int threads) {
        const int64_t chunks = (it.n + threads - 1) / threads;
        const int64_t moves = (entering + threads - 1) / threads;
        hipLaunchKernelGGL(kernel, dim3((unsigned)(chunks + moves)), dim3((unsigned)threads), 0,
                           stream, it, (uint32_t)chunks);
      };
      if (it.n <= kSmallFrame) go(k_fuse_chunk<256>, 256);
      else go(k_fuse_chunk<kThreadsLarge>, kThreadsLarge);
    }
    if ((err = hipGetLastError()) != hipSuccess) return err;
    {
      TimedLaunch tl("k_fuse_tile", stream);
      hipLaunchKernelGGL(k_fuse_tile, dim3(it.T), dim3(kNT2), 0, stream, it);
    }
    if ((err = hipGetLastError()) != hipSuccess) return err;
  }
  if (it.c.var_t != 0.0f || (it.c.var_o != 0.0f && it.n > 0)) {
    // time variance (also after an empty frame) and outlier variance
    TimedLaunch tl("k_time_variance", stream);
    hipLaunchKernelGGL(k_time_variance, dim3((unsigned)((cells + kNTv - 1) / kNTv)), dim3(kNTv),
                       0, stream, it);
    err = hipGetLastError();
  }
  return err;
}

int64_t move_units(const Item& it) {
  return (strips_of(it).cells + kThreadsBatch - 1) / kThreadsBatch;
}
int64_t chunk_units(int64_t n) {
  return (n + kThreadsBatch * kPointsBatch - 1) / (kThreadsBatch * kPointsBatch);
}
int64_t zero_units(int64_t cells) { return (cells + 255) / 256; }
int64_t var_units(int64_t cells) { return (cells + kNTv - 1) / kNTv; }

hipError_t launch_fuse_batch(const Batch* d_batch, const int grid[5], hipStream_t stream) {
  // grid: zero, count, chunk, tile, var; the first two and the last may be 0
  // (no item needs the stage: no launch)
  const int grid_chunk = grid[2], grid_tile = grid[3];
  if (grid[0] > 0) {
    TimedLaunch tl("k_zero_b", stream);
    hipLaunchKernelGGL(k_zero_b, dim3(grid[0]), dim3(256), 0, stream, d_batch);
  }
  if (grid[1] > 0) {
    TimedLaunch tl("k_fuse_count_b", stream);
    hipLaunchKernelGGL(k_fuse_count_b, dim3(grid[1]), dim3(kThreadsBatch), 0, stream, d_batch);
  }
  {
    TimedLaunch tl("k_fuse_chunk_b", stream);
    hipLaunchKernelGGL(k_fuse_chunk_b, dim3(grid_chunk), dim3(kThreadsBatch), 0, stream, d_batch);
  }
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  {
    TimedLaunch tl("k_fuse_tile_b", stream);
    // grid_tile counts tiles in flight; a workgroup holds kTilesPerGroup
    hipLaunchKernelGGL(k_fuse_tile_b, dim3((unsigned)((grid_tile + kTilesPerGroup - 1) / kTilesPerGroup)),
                       dim3(kNT2b), 0, stream, d_batch);
  }
  if (grid[4] > 0) {
    TimedLaunch tl("k_time_variance_b", stream);
    hipLaunchKernelGGL(k_time_variance_b, dim3(grid[4]), dim3(kNTv), 0, stream, d_batch);
  }
  return hipGetLastError();
}

}  // namespace emx
