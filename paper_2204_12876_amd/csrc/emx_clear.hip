// Visibility clean-up by ray casting (Sec. II-E, Eq. 3 and Eq. 4).
//
// The samples of a ray are q_k = o + (k/K) d for k = 1..K-1, in float32.  Most
// of them pass above every cell that a ray could still remove: on 400 x 400
// maps in use a ray has 22 samples in the map, of which 0.1 to 2 lie below the
// largest removable height of their 8 x 8 block.  The work is therefore to find
// those samples without evaluating the others.
//
// setup: one workgroup per 32 x 32 cells, one wave per row of four 8 x 8
// blocks, a lane's four cells two rows apart in one column (128-byte rows of
// loads, and the block maxima in four shuffles for four blocks).
//   - Per 8 x 8 block (cmax) and per 32 x 32 superblock (smax): the largest
//     height of a cell that a ray could still remove: valid, older than the
//     minimum age, with a normal.  It is -inf if there is none.
//   - Each cell's clearing record: h, or -inf if no ray may remove it, so that
//     the march's height test takes one load.  A map alone keeps {that, v}, which
//     stops most of what passes the test of the height alone (4M rays: the march
//     271 against 285 us); a batch keeps 4 bytes, which is what bounds its setup
//     (16 maps: 39 -> 28 us, the march the same).
//   - Loads come in two rounds: validity, then the update time, normal z, height
//     and variance of valid cells (or the upper bound of invalid ones); on maps of up
//     to kAllCells all in one.
//   - The caller's removed-cell mask is zeroed here.
// march: one workgroup per 32, 64, 128 or (in a batch) 256 rays, consecutive ones or,
// where rays can be long, from several parts of the frame (kLongRay).
//   - The ray is cut into groups of Item::grp consecutive samples, at most 7
//     cells of travel, and spans of four groups.  Lower bounds of a group's
//     cells and height come from the ray's line, widened by more than the
//     samples' float32 evaluation can differ from it.  If the height is not
//     below the maxima of the 2 x 2 blocks from the lowest cell on, no sample of
//     the group can act: the group is skipped.  Long rays' spans are tested
//     first, the same way, against the superblocks.  This is exact pruning: it
//     never skips a sample that could act, and costs no sample evaluation.
//   - Three phases hand lists in LDS to each other, so that every phase has an
//     equal share for each thread whatever the rays' lengths: spans (one ray, or a
//     part of one, per thread), groups (one surviving span per thread; rays of one
//     span take theirs in the first phase), samples (one surviving group per thread).  One
//     thread per ray through all phases was 1.5 times slower on 400 x 400 maps:
//     the longest ray's chain of lookups, a microsecond each, set the time.
//   - Every sample of a surviving group is evaluated exactly and compared
//     with its cell's record, eight samples' records requested together (4M
//     rays: 260 against 273 us for half groups of four; four, where longer steps
//     leave a group no more: 600k rays on 2000 x 2000 with steps of two cells 63
//     against 67); the few below it read the cell's variance and normal.
//   - Steps so long that a group would hold fewer than three samples take a march
//     without groups (sparse march, below).
//   - A sample that removes its cell resets the cell to the prior on the spot
//     (and flags it in the caller's mask).  Of what it resets the march reads
//     only the variance, of a cell that it may be about to remove: a ray that
//     sees it reset finds a cell that is removed already.  All else are the
//     setup's records and the normals, so every ray tests the state as it was
//     when the call started, and resets are idempotent stores of the same
//     values: their order never shows in the result.
// Measured on MI355X, setup + march, against a queue of 16-sample segments whose
// every sample was evaluated: 4M LiDAR rays on 2000 x 2000 cells 1197 -> 276 us,
// 300k rays on 400 x 400 cells 25.4 -> 22.9 us, 16 maps with 4.6M rays in a batch
// 302 -> 148 us.  The march is bound by VALU issue on the large frames (0.83 of
// the SIMDs' issue slots) and by its chain of lookups on the small ones.
// There is no separate pass to apply the removals.
//
// Upper bound layer (Sec. II-H), on maps that keep one: a sample in a cell
// without an estimate lowers the cell's bound to the sample height, by an
// integer atomic minimum (order-free, so deterministic).  Such cells count in
// the maxima with their current bound, so pruning stays exact: a sample at or
// above it can neither remove a cell nor lower a bound.
#include "emx_kernels.h"

namespace emx {

namespace {

constexpr int kNTc = 256;
// Rays of a march workgroup.  A single frame's workgroups are balanced better by
// 128 than by 256 (400 x 400: 17.0 against 19.4 us); a batch has enough of them,
// and 256 halve the work's fixed part (16 maps: 137 against 167 us).  4M rays
// alone: the same.  64 keep the longest rays' workgroups short, which pays while
// 128 would leave fewer than 4 workgroups to a CU (a whole call, 60k rays on
// 200 x 200: 12.0 against 14.6 us; 100k on 2000 x 2000: 34.6 against 38.9; 200k:
// the same; 300k on 400 x 400: 18.5 against 17) and with an upper bound layer,
// where most samples over unseen ground act (400 x 400: 22 against 27 us).  32 for
// the fewest, where 64 leave compute units idle: 32 against 64, 13k rays on 1770 x
// 1979 21.9 against 23.7 us, 40k on 847 x 1070 15.3 against 16.2, but 60k on 200 x 200
// 12.6 against 11.4.  (With consecutive rays; the other form below gains the most at
// the same widths.)
constexpr int kRaysPlain = 128;
constexpr int kRaysShort = 64;
constexpr int kRaysFew = 32;
constexpr int kRaysBatch = 256;
constexpr int64_t kShortRays = 1 << 17;  // 4 x 256 workgroups of 128
constexpr int64_t kFewRays = 3 << 14;    // 6 x 256 workgroups of 32
// Where rays can be long (samples to a map side) and the workgroups are few, the
// march takes another form: a workgroup's rays come from several parts of the frame,
// since a LiDAR's beam is a run of rays of one length and a workgroup that holds only
// long ones sets the march's time; and all of its threads share its rays' spans, where
// a thread to each ray left the others waiting for rounds of eight spans.  A whole
// call, consecutive against shared: 13k LiDAR rays on 1770 x 1979 cells 27.6 -> 23.3
// us, 60k on 2000 x 2000 35.7 -> 29.5, 178k on 827 x 749 30.4 -> 22.5, 300k on 1500 x
// 1500 46.3 -> 35.0, 600k on 2000 x 2000 68 -> 61.  With more workgroups than the chip
// holds they balance each other, and consecutive rays share more of their lookups (4M
// on 2000 x 2000 229 against 237; 800k camera and LiDAR rays on 1200 x 1000 32 against
// 34; 500k on 520 x 520 25 against 28), and where a ray has few spans to share the one
// barrier more shows (with the bound, 300k on 400 x 400: 23.1 against 25.5; 43k on 250 x
// 250: 15.9 against 16.2).  Between the two, two runs of 64 rays and a thread to each
// ray: 600k LiDAR rays on 900 x 900 41.4 -> 32.2 us, 400k on 700 x 700 32.9 -> 27.5, but
// 800k camera and LiDAR rays on 1200 x 1000 34.2 against 33.9 and 4M LiDAR rays 231
// against 226.  On shorter maps only while the chip holds all workgroups at once: 200k
// LiDAR rays on 400 x 400 23.0 -> 20.0, on 330 x 330 22.0 -> 18.8, but 300k camera and
// LiDAR rays on 400 x 400 the same to 1% slower.
constexpr double kLongRay = 320.0;     // samples to the longer side
constexpr double kLongMap = 448.0;     // the same, with more rays than ...
constexpr int64_t kHeldRays = 1 << 18; // ... 7 workgroups of 128 for each of 256 CUs (2^17.8)
constexpr double kSharedRays = 384.0;  // rays to one of those samples: all threads share spans
constexpr double kSpreadRays = 896.0;  // runs of 64
constexpr int kRunShared = 32;         // runs; 16 share fewer lookups (100k rays 5% slower)
constexpr int kRunSpread = 64;
// Maps up to this size load a cell's fields without waiting for its validity: the
// 16 bytes that most cells then load for nothing cost less than the round trip
// (128 x 128: 6.1 -> 5.1 us, 400 x 400 with the bound: 6.6 -> 5.5 us).
constexpr int64_t kAllCells = 1 << 18;
constexpr int kSpanGroups = 4;  // groups in a span
constexpr int kSpans = 8;       // spans of a ray that a thread looks up together

// A ray: direction from the sensor origin (Pose32::t), 1/K correctly rounded
// in double, the last sample that can lie in the map, and the end point's cell.
struct Ray {
  float dx, dy, dz;
  int end_cell;  // or -1
  double rK;
  int k1;
};

// t = float32(k / K), correctly rounded, without a float32 division.
// For integers 1 <= k < K < 2^24, k/K lies more than 2^-49 (relative) from
// every float32 rounding boundary: a boundary is an odd multiple of half an
// ulp, and k/K equal to one would need K > k >= 2^24.  The double product
// k * RN(1/K) carries at most 2^-52 relative error, so it rounds to the same
// float32 as k/K.
__device__ __forceinline__ float t_of(double rK, int k) { return (float)((double)k * rK); }

// Lowers *a to v if v is smaller (v not NaN), as an integer atomic on the
// float's bits: non-negative floats order like their bits as signed
// integers, negative ones inversely to their bits as unsigned integers, and
// every negative float's bits exceed every non-negative one's.
__device__ __forceinline__ void atomic_min_f32(float* a, float v) {
  if (!signbit(v)) atomicMin(reinterpret_cast<int*>(a), __float_as_int(v));
  else atomicMax(reinterpret_cast<unsigned int*>(a), __float_as_uint(v));
}

// Whether q lowers the bound b, in the order of atomic_min_f32: of the two zeros the
// negative one is the lower.
__device__ __forceinline__ bool lowers(float q, float b) {
  return q < b || (__float_as_uint(q) == 0x80000000u && __float_as_uint(b) == 0u);
}

// A cell can be removed only if it is valid, older than the minimum age and
// has a normal (its validity, update time and normal z given).
__device__ __forceinline__ bool clearable(const Item& it, uint8_t valid, int32_t t_upd, float nz) {
  return valid && (((int64_t)it.t_now - (int64_t)t_upd) > (int64_t)it.c.tau) && !isnan(nz);
}

// Removal of a cell: back to the prior, invalid (physical index pc); flagged
// in the caller's mask (logical index lc).
__device__ __forceinline__ void clear_cell(const Item& it, int64_t pc, int lc) {
  it.L.h[pc] = it.c.h_init;
  it.L.v[pc] = it.c.v_init;
  it.L.valid[pc] = 0;
  if (it.out_cleared) it.out_cleared[lc] = 1;
}

// Narrows [lo, hi], in samples, to where o + (k/K) d lies in [0, W], widened
// by more than the float32 evaluation of a sample and of this line can be off:
// the samples outside are certainly outside the map, those inside are tested
// one by one.  A coordinate that does not change (d = 0) keeps or empties the
// whole range.
__device__ __forceinline__ void clip(float o, float d, float W, float K, float& lo, float& hi) {
  const float eps = (fabsf(o) + fabsf(d) + W) * 0x1p-18f;
  const float s = K * __builtin_amdgcn_rcpf(d);
  const float a = (-eps - o) * s;
  const float b = ((W + eps) - o) * s;
  lo = fmaxf(lo, fminf(a, b));
  hi = fminf(hi, fmaxf(a, b));
}

// The ray of point i of the item and its first sample k0.  False if the point
// casts no ray (not valid, too long a ray, or K < 2: no samples) or no sample
// can lie in the map.
__device__ __forceinline__ bool ray_of(const Item& it, int64_t i, Ray& r, int& k0) {
  const PointEval e = eval_point(it.P, it.c, it.x[i], it.y[i], it.z[i]);
  r.dx = e.xm - it.P.t[0];
  r.dy = e.ym - it.P.t[1];
  r.dz = e.zm - it.P.t[2];
  const float m = fmaxf(fabsf(r.dx), fabsf(r.dy));
  const float ks = m * it.c.inv_step;
  if (!e.valid || !(ks < 16777216.0f)) return false;
  const float Kf = ceilf(ks);
  if (!(Kf >= 2.0f)) return false;
  float lo = 1.0f, hi = Kf - 1.0f;
  const float r32 = __builtin_amdgcn_rcpf(it.c.inv_r);
  clip(it.P.t[0], r.dx, it.c.nxf * r32, Kf, lo, hi);
  clip(it.P.t[1], r.dy, it.c.nyf * r32, Kf, lo, hi);
  lo = fmaxf(lo - (fabsf(lo) * 0x1p-18f + 2.0f), 1.0f);
  hi = fminf(hi + (fabsf(hi) * 0x1p-18f + 2.0f), Kf - 1.0f);
  if (!(lo <= hi)) return false;
  k0 = (int)lo;
  r.k1 = (int)hi;
  r.rK = 1.0 / (double)Kf;
  int ex, ey;
  r.end_cell = bin_xy(e.xm, e.ym, it.c, ex, ey) ? ey * it.c.nx + ex : -1;
  return true;
}

// Lower bounds of the samples of a step: x and y, in blocks of 2^kLog cells, and
// the height z of the exact samples k .. k + step of the ray are at least
// line(k).  The samples' float32 evaluation and this one differ by less than
// 2^-21 of the magnitudes entering them; the margins are 2^-19.
struct Line {
  float x, dx, y, dy, z, dz;
  float zmin;  // no sample of the ray is lower; NaN if a step spans more than
               // one block along an axis (it is not looked up: it may act)
};

template <int kLog>
__device__ __forceinline__ Line line_of(const Item& it, const Ray& r, int step) {
  const float scale = it.c.inv_r * (1.0f / (float)(1 << kLog));
  const float rk = (float)r.rK;
  const float s = (float)step;
  const float ox = it.P.t[0] * scale, oy = it.P.t[1] * scale, oz = it.P.t[2];
  const float tx = r.dx * scale, ty = r.dy * scale;
  const float ex = (fabsf(ox) + fabsf(tx)) * 0x1p-19f;
  const float ey = (fabsf(oy) + fabsf(ty)) * 0x1p-19f;
  // (the least denormal: a bound of -0.0 must not look equal to a maximum of 0.0)
  const float ez = fmaf(fabsf(oz) + fabsf(r.dz), 0x1p-19f, 0x1p-149f);
  Line l;
  l.dx = tx * rk;
  l.dy = ty * rk;
  l.dz = r.dz * rk;
  l.x = (ox - ex) + fminf(l.dx * s, 0.0f);
  l.y = (oy - ey) + fminf(l.dy * s, 0.0f);
  l.z = (oz - ez) + fminf(l.dz * s, 0.0f);
  const bool fits = fabsf(l.dx) * s + 2.0f * ex < 0.999f && fabsf(l.dy) * s + 2.0f * ey < 0.999f;
  l.zmin = fits ? fminf(oz, fmaf(l.dz, (float)r.k1, oz)) - ez : __builtin_nanf("");
  return l;
}

// Which of kN consecutive steps of `step` samples from sample k on (bit j: the
// j-th) may hold a sample below the maximum of its block (`mx`, w x h blocks).  A
// step's samples lie in the 2 x 2 blocks from its line's on, two 8-byte lookups;
// clamping keeps every in-map cell among them.  Every lookup is requested before
// any is used.  Where there is one column the pair's second value is the next row's
// (past the last row, set_layout's spare one), and where there is one row the second
// pair is the first: a value too many only keeps a step.
struct __attribute__((packed, aligned(4))) Pair {
  float a, b;
};

template <int kN>
__device__ __forceinline__ uint32_t may_act(const Line& l, int k, int k1, int step,
                                            const float* mx, int w, int h) {
  uint32_t live = 0;
#pragma unroll
  for (int j = 0; j < kN; ++j) live |= (k + j * step <= k1) ? 1u << j : 0u;
  const float xm = (float)max(w - 2, 0), ym = (float)max(h - 2, 0);
  const float* up = mx + (h > 1 ? w : 0);
  Pair lo[kN], hi[kN];
  float z[kN];
#pragma unroll
  for (int j = 0; j < kN; ++j) {
    const float kf = (float)(k + j * step);
    const int x = (int)__builtin_amdgcn_fmed3f(fmaf(kf, l.dx, l.x), 0.0f, xm);
    const int y = (int)__builtin_amdgcn_fmed3f(fmaf(kf, l.dy, l.y), 0.0f, ym);
    z[j] = fmaf(kf, l.dz, l.z);
    const uint32_t o = (__umul24(y, w) + (uint32_t)x) * 4u;
    lo[j] = *(const Pair*)((const char*)mx + o);
    hi[j] = *(const Pair*)((const char*)up + o);
  }
  uint32_t bits = 0;
#pragma unroll
  for (int j = 0; j < kN; ++j) {
    const float m = fmaxf(fmaxf(lo[j].a, lo[j].b), fmaxf(hi[j].a, hi[j].b));
    // a NaN height may act (fmaxf would drop zmin's)
    bits |= !(z[j] >= m || l.zmin >= m) ? 1u << j : 0u;
  }
  if (isnan(l.zmin)) bits = ~0u;
  return bits & live;
}

// A sample of ray r, as the ABI evaluates it; in the map truncation is floor
// (`lim`: the largest float32 below nx and ny, so that clamping to it changes
// exactly the coordinates outside the map).
struct Sample {
  int ix, iy;
  float qz;
  bool in;
};

__device__ __forceinline__ Sample sample_of(const Item& it, const Ray& r, int k, float2 lim) {
  const float t = t_of(r.rK, k);
  const float fx = (it.P.t[0] + t * r.dx) * it.c.inv_r;
  const float fy = (it.P.t[1] + t * r.dy) * it.c.inv_r;
  const float cx = __builtin_amdgcn_fmed3f(fx, 0.0f, lim.x);
  const float cy = __builtin_amdgcn_fmed3f(fy, 0.0f, lim.y);
  Sample q;
  q.qz = it.P.t[2] + t * r.dz;
  q.in = (cx == fx) & (cy == fy);
  q.ix = (int)cx;
  q.iy = (int)cy;
  return q;
}

constexpr int kUnroll = 8;  // samples evaluated together
constexpr int kHalf = 4;    // in groups of up to four

// Samples [ka, kb] of ray r against the map, kU at a time.  Their cells are
// found without branches, then their clearing records are all requested
// together: the height, or -inf for a cell no ray may clear, which fails hd > 0
// for every finite sample height.  With kPair the record also holds the
// variance; on maps with an upper bound layer (kBound, always pairs) a cell
// without an estimate holds {NaN, its bound at the call's start} (no other
// record holds NaN).  The few samples that pass go through one loop, a lane's
// next one each time, so that a wave waits for its fullest lane and not for
// every position.  Without pairs that loop reads the variance from the layer:
// another ray may have removed the cell meanwhile, but then it is removed
// whatever this ray finds.
template <int kU, bool kBound, bool kPair>
__device__ __forceinline__ void test_samples(const Item& it, const Ray& r, int ka, int kb) {
  const float2 lim = make_float2(__uint_as_float(__float_as_uint(it.c.nxf) - 1u),
                                 __uint_as_float(__float_as_uint(it.c.nyf) - 1u));
  for (int k = ka; k <= kb; k += kU) {
    float qz[kU];
    bool cand[kU];
    float rec[kU], v[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const Sample q = sample_of(it, r, k + u, lim);
      const uint32_t cell = __umul24(q.iy, it.c.nx) + (uint32_t)q.ix;
      qz[u] = q.qz;
      cand[u] = (k + u <= kb) & q.in & ((int)cell != r.end_cell);
      v[u] = -INFINITY;
      if (kPair) {
        const float2 p = *(const float2*)((const char*)it.L.clr + cell * 8u);
        rec[u] = p.x;
        v[u] = p.y;
      } else {
        rec[u] = *(const float*)((const char*)it.L.clr + cell * 4u);
      }
    }
    uint32_t remove = 0, bound = 0;
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const float hd = rec[u] - qz[u];
      if (cand[u] & (hd > 0.0f) & (!kPair || (hd * hd) > v[u])) remove |= 1u << u;
      // lowers(), but for a pair of zeros in the other order, which the loop below
      // sorts out (in full here it takes 110 registers instead of 66)
      const bool low = (qz[u] <= v[u]) & (__float_as_int(qz[u]) != __float_as_int(v[u]));
      if (kBound && (cand[u] & isnan(rec[u]) & low)) bound |= 1u << u;
    }
    while (remove | bound) {
      const int u = __builtin_ctz(remove | bound);
      const Sample q = sample_of(it, r, k + u, lim);
      const int64_t pc = pcell(it.c, q.ix, q.iy);
      if ((remove >> u) & 1u) {
        bool below = true;
        if (!kPair) {
          const float hd = it.L.clr[__umul24(q.iy, it.c.nx) + (uint32_t)q.ix] - q.qz;
          below = (hd * hd) > it.L.v[pc];
        }
        const float an2dd = it.c.an2 * ((r.dx * r.dx + r.dy * r.dy) + r.dz * r.dz);
        const float dot = (r.dx * it.L.nx[pc] + r.dy * it.L.ny[pc]) + r.dz * it.L.nz[pc];
        if (below && (dot * dot) > an2dd) clear_cell(it, pc, q.iy * it.c.nx + q.ix);
      } else if (lowers(q.qz, it.L.ub[pc])) {  // another ray may have lowered it further
        atomic_min_f32(it.L.ub + pc, q.qz);
      }
      remove &= ~(1u << u);
      bound &= ~(1u << u);
    }
  }
}

// ------------------------------------------------------------------- setup
// Superblock `unit` of item `it`: its block maxima, its own, and the records.
// kAll: every cell's fields are loaded along with its validity.
// kPair: the records are pairs.
template <bool kAll, bool kBound, bool kPair>
__device__ __forceinline__ void setup_body(const Item& it, int unit, float* s_max) {
  constexpr int kRows = 4;  // rows of a lane's column, two apart
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int sy = unit / it.sbx;
  const int sx = unit - sy * it.sbx;
  const int ix = (sx << kSuperLog) + (lane & 31);
  const int iy0 = (sy << kSuperLog) + (wave << kBlockLog) + (lane >> 5);
  int c[kRows];       // logical cell: the mask, the records
  int64_t p[kRows];   // physical cell: the layers
  bool in[kRows];
  uint8_t vd[kRows];
#pragma unroll
  for (int j = 0; j < kRows; ++j) {
    const int iy = iy0 + 2 * j;
    in[j] = ix < it.c.nx && iy < it.c.ny;
    c[j] = in[j] ? iy * it.c.nx + ix : 0;
    p[j] = in[j] ? pcell(it.c, ix, iy) : 0;
    vd[j] = in[j] ? it.L.valid[p[j]] : 0;
  }
  // then what a valid cell's tests and record need, or a cell without an
  // estimate's bound; cells that cannot matter load nothing more
  int32_t tu[kRows];
  float nz[kRows], h[kRows], v[kRows], ub[kRows];
#pragma unroll
  for (int j = 0; j < kRows; ++j) {
    tu[j] = 0;
    nz[j] = h[j] = v[j] = 0.0f;
    ub[j] = INFINITY;
    if (kAll || vd[j]) {
      tu[j] = it.L.t[p[j]];
      nz[j] = it.L.nz[p[j]];
      h[j] = it.L.h[p[j]];
      if (kPair) v[j] = it.L.v[p[j]];
    }
    if (kBound && in[j] && (kAll || !vd[j])) ub[j] = it.L.ub[p[j]];
  }
  float rec[kRows];
  float m = -INFINITY;
#pragma unroll
  for (int j = 0; j < kRows; ++j) {
    if (in[j] && it.out_cleared) it.out_cleared[c[j]] = 0;  // the march sets removals
    const bool ok = in[j] && clearable(it, vd[j], tu[j], nz[j]);
    // a NaN height can never be cleared (hd > 0 fails), so -inf serves
    rec[j] = ok && !isnan(h[j]) ? h[j] : -INFINITY;
    m = fmaxf(m, rec[j]);
    if (kBound && in[j] && !vd[j]) {
      // a sample below the bound of a cell without an estimate lowers it:
      // such cells take part in the maximum too
      rec[j] = __builtin_nanf("");
      v[j] = ub[j];
      m = fmaxf(m, ub[j]);
    }
  }
  m = fmaxf(m, __shfl_xor(m, 1, 64));
  m = fmaxf(m, __shfl_xor(m, 2, 64));
  m = fmaxf(m, __shfl_xor(m, 4, 64));
  m = fmaxf(m, __shfl_xor(m, 32, 64));
#pragma unroll
  for (int j = 0; j < kRows; ++j)
    if (in[j]) {
      if (kPair) ((float2*)it.L.clr)[c[j]] = make_float2(rec[j], v[j]);
      else it.L.clr[c[j]] = rec[j];
    }
  const int b = (sx << (kSuperLog - kBlockLog)) + (lane >> kBlockLog);
  const int by = (sy << (kSuperLog - kBlockLog)) + wave;
  if (lane < 32 && (lane & 7) == 0 && b < it.bx && by < it.by) it.L.cmax[by * it.bx + b] = m;
  m = fmaxf(m, __shfl_xor(m, 8, 64));
  m = fmaxf(m, __shfl_xor(m, 16, 64));
  if (lane == 0) s_max[wave] = m;
  __syncthreads();
  if (threadIdx.x == 0)
    it.L.smax[unit] = fmaxf(fmaxf(s_max[0], s_max[1]), fmaxf(s_max[2], s_max[3]));
}

// ------------------------------------------------------------------- march
// Arrays by field: lanes that read different rays then meet different banks.
template <int kRays, int kParts>
struct MarchShared {
  float dx[kRays], dy[kRays], dz[kRays];
  double rK[kRays];
  int k1[kRays], end_cell[kRays];
  float line[7][kRays];  // of the groups, for rays of more than one span
  // the samples of such rays, none for others (where several threads share a ray)
  int from[kParts > 1 ? kRays : 1], to[kParts > 1 ? kRays : 1];
  // entries: ray << 24 | first sample
  uint32_t spans[kSpans * kRays * kParts];
  uint32_t groups[kSpanGroups * (kRays + kNTc)];
  int nspans, ngroups;
};

// Appends the steps of each lane's `bits` (kN of them) to a list with room for
// them, by one LDS atomic per wave (an atomic per lane with its own count would
// be expanded into a loop over the lanes).  The j-th steps of all lanes come
// together: neighbouring rays, whose lookups share cache lines.  The lanes of a
// wave that call it are those from lane 0 up to some lane: all, or in workgroups of
// 32 rays the first half in the march's first phase.
template <int kN>
__device__ __forceinline__ void append(uint32_t* list, int* n, uint32_t bits, uint32_t ray, int k,
                                       int step) {
  if (__ballot(bits != 0) == 0) return;
  uint64_t b[kN];
  int total = 0;
#pragma unroll
  for (int j = 0; j < kN; ++j) {
    b[j] = __ballot((bits >> j) & 1u);
    total += __popcll(b[j]);
  }
  int at = 0;
  if ((threadIdx.x & 63) == 0) at = atomicAdd(n, total);
  at = __builtin_amdgcn_readfirstlane(at);
  const uint32_t e = (ray << 24) | (uint32_t)k;
#pragma unroll
  for (int j = 0; j < kN; ++j) {
    if (b[j] == 0) continue;
    const int below = (int)__builtin_amdgcn_mbcnt_hi(
        (uint32_t)(b[j] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b[j], 0u));
    if ((bits >> j) & 1u) list[at + below] = e + (uint32_t)(j * step);
    at += __popcll(b[j]);
  }
}

// The ray in slot `slot` of workgroup `unit` of `units`, which takes runs of kRun
// consecutive rays from kRays / kRun parts of the frame.
template <int kRun>
__device__ __forceinline__ int64_t spread_ray(int64_t unit, int64_t units, int slot) {
  return ((int64_t)(slot / kRun) * units + unit) * kRun + slot % kRun;
}

// The rays of workgroup `unit` of the item: consecutive ones (kRun 0), or runs of
// kRun from all over the frame (spread_ray, `units` workgroups), with kParts threads
// to the spans of each.  The counts in s are zero on entry and on return (every
// thread passes a barrier after they were reset).
template <int kRays, int kRun, int kParts, bool kPair>
__device__ __forceinline__ void march_body(const Item& it, int64_t unit, int64_t units,
                                           MarchShared<kRays, kParts>& s) {
  const int tid = threadIdx.x;
  const int grp = it.grp, span = kSpanGroups * it.grp;
  Ray r;
  int k = 1, k1 = 0;  // the ray's first sample that no span covers yet, its last
  if (tid < kRays) {
    const int64_t i =
        kRun > 0 ? spread_ray<(kRun > 0 ? kRun : 1)>(unit, units, tid) : unit * kRays + tid;
    uint32_t gb = 0;
    int first = 1;
    if (i < it.n && ray_of(it, i, r, first)) {
      s.dx[tid] = r.dx;
      s.dy[tid] = r.dy;
      s.dz[tid] = r.dz;
      s.rK[tid] = r.rK;
      s.k1[tid] = r.k1;
      s.end_cell[tid] = r.end_cell;
      const Line l = line_of<kBlockLog>(it, r, grp);
      if (r.k1 - first < span) {
        // one span, as most rays: its groups at once
        gb = may_act<kSpanGroups>(l, first, r.k1, grp, it.L.cmax, it.bx, it.by);
      } else {
        s.line[0][tid] = l.x;
        s.line[1][tid] = l.dx;
        s.line[2][tid] = l.y;
        s.line[3][tid] = l.dy;
        s.line[4][tid] = l.z;
        s.line[5][tid] = l.dz;
        s.line[6][tid] = l.zmin;
        k = first;
        k1 = r.k1;
      }
    }
    append<kSpanGroups>(s.groups, &s.ngroups, gb, (uint32_t)tid, first, grp);
    if (kParts > 1) {
      s.from[tid] = k;
      s.to[tid] = k1;
    }
  }
  int slot = tid;
  if (kParts > 1) {
    __syncthreads();
    slot = tid % kRays;
    k = s.from[slot] + tid / kRays * (kSpans * span);
    k1 = s.to[slot];
    if (k <= k1) r = Ray{s.dx[slot], s.dy[slot], s.dz[slot], 0, s.rK[slot], k1};
  }
  bool more = true;
  while (more) {
    // spans: at most kSpans of each long ray's share
    uint32_t bits = 0;
    if (k <= k1)
      bits = k1 - k < 2 * span ? (k1 - k < span ? 1u : 3u)  // straight to the groups
                               : may_act<kSpans>(line_of<kSuperLog>(it, r, span), k, k1, span,
                                                 it.L.smax, it.sbx, it.sby);
    append<kSpans>(s.spans, &s.nspans, bits, (uint32_t)slot, k, span);
    k += kParts * kSpans * span;
    more = __syncthreads_or(k <= k1);
    const int ns = s.nspans;
    int b = 0;
    do {
      if (b < ns) {
        // groups: of at most one span per thread
        uint32_t gb = 0, w = 0;
        int ks = 0;
        if (b + tid < ns) {
          const uint32_t e = s.spans[b + tid];
          w = e >> 24;
          ks = (int)(e & 0xFFFFFFu);
          const Line l = {s.line[0][w], s.line[1][w], s.line[2][w], s.line[3][w],
                          s.line[4][w], s.line[5][w], s.line[6][w]};
          gb = may_act<kSpanGroups>(l, ks, s.k1[w], grp, it.L.cmax, it.bx, it.by);
        }
        append<kSpanGroups>(s.groups, &s.ngroups, gb, w, ks, grp);
        __syncthreads();
      }
      const int ng = s.ngroups;
      for (int g = tid; g < ng; g += kNTc) {
        const uint32_t e = s.groups[g];
        const uint32_t w = e >> 24;
        const Ray q = {s.dx[w], s.dy[w], s.dz[w], s.end_cell[w], s.rK[w], s.k1[w]};
        const int ka = (int)(e & 0xFFFFFFu);
        const int kb = min(ka + grp - 1, q.k1);
        if (it.L.ub) test_samples<kUnroll, true, true>(it, q, ka, kb);
        else if (grp > kHalf) test_samples<kUnroll, false, kPair>(it, q, ka, kb);
        else test_samples<kHalf, false, kPair>(it, q, ka, kb);
      }
      __syncthreads();  // the groups have been read
      if (tid == 0) s.ngroups = 0;
      __syncthreads();
      b += kNTc;
    } while (b < ns);
    if (tid == 0) s.nspans = 0;
    __syncthreads();
  }
}

// ------------------------------------------------------------- sparse march
// For steps so long that fewer than three samples lie within 7 cells (Item::grp is
// 0): a group would hold one or two, and its lookups cost more than they spare.  A
// workgroup's rays are cut into runs of eight samples, one per thread at a time,
// found by a search in the prefix of the rays' runs.  Each sample is compared with
// the maximum of its own block, and the few below it with their cells.
// What bounds it: on small frames the chain of round trips, on large ones VALU issue
// (50 registers, 8 waves to a SIMD; eight records requested together like the dense
// march took 104 and 10 to 30% longer).  A whole call against the dense march with
// groups of one sample: 300k rays on 400 x 400 cells, steps of 4 cells 23.4 -> 17.1 us
// (a queue of segments took 17.1), of 12 cells 20.6 -> 14.6 (14.6); 600k on 2000 x
// 2000, 4 cells 80 -> 53 (56), 20 cells 80 -> 33 (36).  At steps of 2 cells the dense
// march is the better one (600k on 2000 x 2000: 65 against 113), and so the line is
// drawn at three samples.
template <int kRays>
struct SparseShared {
  float dx[kRays], dy[kRays], dz[kRays];
  double rK[kRays];
  int k0[kRays], k1[kRays], end_cell[kRays];
  int first[kRays];  // runs of the rays before
  int sum[kNTc / 64];
};

// Rays come from all over the frame (spread_ray), in workgroups of 128 and, up to
// kShortRays and kFewRays, of 64 and 32: a beam's rays are of one length here too.
// Runs of 16 against 32 rays: 600k on 2000 x 2000, steps of 4 cells 53 against 57 us;
// consecutive rays 69.
constexpr int kRunSparse = 16;

// Samples [ka, kb] (at most kUnroll) of ray r.
template <bool kBound, bool kPair>
__device__ __forceinline__ void sparse_samples(const Item& it, const Ray& r, int ka, int kb) {
  const float2 lim = make_float2(__uint_as_float(__float_as_uint(it.c.nxf) - 1u),
                                 __uint_as_float(__float_as_uint(it.c.nyf) - 1u));
  uint32_t act = 0;
  float qz[kUnroll], m[kUnroll];
#pragma unroll
  for (int u = 0; u < kUnroll; ++u) {
    const Sample q = sample_of(it, r, ka + u, lim);
    const uint32_t cell = __umul24(q.iy, it.c.nx) + (uint32_t)q.ix;
    m[u] = it.L.cmax[__umul24(q.iy >> kBlockLog, it.bx) + (uint32_t)(q.ix >> kBlockLog)];
    qz[u] = q.qz;
    act |= ((ka + u <= kb) & q.in & ((int)cell != r.end_cell)) ? 1u << u : 0u;
  }
#pragma unroll
  for (int u = 0; u < kUnroll; ++u)  // (equal: zeros of either sign, see lowers)
    if (!(qz[u] <= m[u])) act &= ~(1u << u);
  while (act) {
    const Sample q = sample_of(it, r, ka + __builtin_ctz(act), lim);
    act &= act - 1u;
    const uint32_t lc = __umul24(q.iy, it.c.nx) + (uint32_t)q.ix;
    const int64_t pc = pcell(it.c, q.ix, q.iy);
    float h, v = 0.0f;
    if (kPair) {
      const float2 p = *(const float2*)((const char*)it.L.clr + lc * 8u);
      h = p.x;
      v = p.y;
    } else {
      h = *(const float*)((const char*)it.L.clr + lc * 4u);
    }
    const float hd = h - q.qz;
    if (kBound && isnan(h)) {
      if (lowers(q.qz, v) && lowers(q.qz, it.L.ub[pc])) atomic_min_f32(it.L.ub + pc, q.qz);
    } else if (hd > 0.0f) {
      if (!kPair) v = it.L.v[pc];  // (see test_samples)
      const float an2dd = it.c.an2 * ((r.dx * r.dx + r.dy * r.dy) + r.dz * r.dz);
      if ((hd * hd) > v) {
        const float dot = (r.dx * it.L.nx[pc] + r.dy * it.L.ny[pc]) + r.dz * it.L.nz[pc];
        if ((dot * dot) > an2dd) clear_cell(it, pc, (int)lc);
      }
    }
  }
}

// The rays of workgroup `unit` of `units` of the item.  Ends with a barrier.
template <int kRays, bool kBound, bool kPair>
__device__ __forceinline__ void sparse_body(const Item& it, int64_t unit, int64_t units,
                                            SparseShared<kRays>& s) {
  const int tid = threadIdx.x;
  int n = 0;  // the ray's runs
  if (tid < kRays) {
    const int64_t i = spread_ray<kRunSparse>(unit, units, tid);
    Ray r;
    int k0 = 1;
    if (i < it.n && ray_of(it, i, r, k0)) {
      s.dx[tid] = r.dx;
      s.dy[tid] = r.dy;
      s.dz[tid] = r.dz;
      s.rK[tid] = r.rK;
      s.k0[tid] = k0;
      s.k1[tid] = r.k1;
      s.end_cell[tid] = r.end_cell;
      n = (r.k1 - k0) / kUnroll + 1;
    }
  }
  const int lane = tid & 63, wave = tid >> 6;
  int x = n;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) s.sum[wave] = x;
  __syncthreads();
  int before = 0, total = 0;
#pragma unroll
  for (int w = 0; w < kNTc / 64; ++w) {
    before += w < wave ? s.sum[w] : 0;
    total += s.sum[w];
  }
  if (tid < kRays) s.first[tid] = before + x - n;
  __syncthreads();
  for (int g = tid; g < total; g += kNTc) {
    int w = 0;  // the last ray with first <= g: the one that has run g
#pragma unroll
    for (int h = kRays / 2; h > 0; h >>= 1)
      if (s.first[w + h] <= g) w += h;
    const Ray q = {s.dx[w], s.dy[w], s.dz[w], s.end_cell[w], s.rK[w], s.k1[w]};
    const int ka = s.k0[w] + (g - s.first[w]) * kUnroll;
    sparse_samples<kBound, kPair>(it, q, ka, min(ka + kUnroll - 1, q.k1));
  }
  __syncthreads();
}

// ---------------------------------------------------------------- launches
template <bool kAll>
__global__ __launch_bounds__(kNTc) void k_clear_setup(Item it) {
  __shared__ float s_max[kNTc / 64];
  if (it.L.ub) setup_body<kAll, true, true>(it, blockIdx.x, s_max);
  else setup_body<kAll, false, true>(it, blockIdx.x, s_max);
}

// The maxima are read through the caches: they are small and shared by every
// workgroup, and staging them in LDS per workgroup costs more than it saves.
template <int kRays, int kRun, int kParts>
__global__ __launch_bounds__(kNTc) void k_clear_march(Item it) {
  __shared__ MarchShared<kRays, kParts> s;
  if (threadIdx.x == 0) s.nspans = s.ngroups = 0;
  __syncthreads();
  march_body<kRays, kRun, kParts, true>(it, blockIdx.x, gridDim.x, s);
}

template <int kRays>
__global__ __launch_bounds__(kNTc, 8) void k_clear_sparse(Item it) {
  __shared__ SparseShared<kRays> s;
  if (it.L.ub) sparse_body<kRays, true, true>(it, blockIdx.x, gridDim.x, s);
  else sparse_body<kRays, false, true>(it, blockIdx.x, gridDim.x, s);
}

__global__ __launch_bounds__(kNTc) void k_clear_setup_b(const Batch* bt) {
  __shared__ float s_max[kNTc / 64];
  const UnitFinder units(bt, kBSetup);
  for (int64_t w = blockIdx.x; w < units.total(); w += gridDim.x) {
    int64_t unit;
    const int i = units.find(w, unit);
    const Item& it = bt->items[i];
    if (it.L.ub) setup_body<false, true, true>(it, (int)unit, s_max);
    else setup_body<false, false, false>(it, (int)unit, s_max);
    __syncthreads();
  }
}

__global__ __launch_bounds__(kNTc) void k_clear_march_b(const Batch* bt) {
  __shared__ MarchShared<kRaysBatch, 1> s;
  if (threadIdx.x == 0) s.nspans = s.ngroups = 0;
  __syncthreads();
  const UnitFinder units(bt, kBRays);
  for (int64_t w = blockIdx.x; w < units.total(); w += gridDim.x) {
    int64_t unit;
    const int i = units.find(w, unit);
    march_body<kRaysBatch, 0, 1, false>(bt->items[i], unit, 0, s);
  }
}

__global__ __launch_bounds__(kNTc, 8) void k_clear_sparse_b(const Batch* bt) {
  __shared__ SparseShared<kRaysPlain> s;
  const UnitFinder units(bt, kBSparse);
  for (int64_t w = blockIdx.x; w < units.total(); w += gridDim.x) {
    int64_t unit;
    const int i = units.find(w, unit);
    const Item& it = bt->items[i];
    const int64_t of = (it.n + kRaysPlain - 1) / kRaysPlain;
    if (it.L.ub) sparse_body<kRaysPlain, true, true>(it, unit, of, s);
    else sparse_body<kRaysPlain, false, false>(it, unit, of, s);
  }
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

}  // namespace

// What a caller's scratch must hold for a clearing call: the size contract of
// emx_scratch_bytes and emx_batch_scratch_bytes.  The kernels keep their work
// lists in LDS and use none of it.
size_t clear_scratch_bytes(int64_t max_points, int seg) {
  const int64_t segs = (max_points * 128 + seg - 1) / seg + 2 * max_points;
  const int64_t cap = (segs + segs / 8 + 63) / 64;
  return align256((size_t)cap * 64 * 8) + align256((size_t)max_points * 16);
}

int64_t sparse_units(const Item& it) {
  return it.grp > 0 ? 0 : (it.n + kRaysPlain - 1) / kRaysPlain;
}
int64_t setup_units(const Item& it) { return (int64_t)it.sbx * it.sby; }
int64_t ray_units(const Item& it) {
  return it.grp > 0 ? (it.n + kRaysBatch - 1) / kRaysBatch : 0;
}

hipError_t launch_clear(const Item& it, hipStream_t stream) {
  // with no rays the setup still zeroes the caller's mask
  if (it.n <= 0 && !it.out_cleared) return hipSuccess;
  {
    TimedLaunch tl("k_clear_setup", stream);
    hipLaunchKernelGGL((int64_t)it.c.nx * it.c.ny <= kAllCells ? k_clear_setup<true>
                                                               : k_clear_setup<false>,
                       dim3((unsigned)setup_units(it)), dim3(kNTc), 0, stream, it);
  }
  hipError_t err = hipGetLastError();
  if (err != hipSuccess || it.n <= 0) return err;
  TimedLaunch tl("k_clear_march", stream);
  const int side = it.c.nx > it.c.ny ? it.c.nx : it.c.ny;
  const double samples = (double)side / (double)it.c.inv_r * (double)it.c.inv_step;
  const double rays = (double)it.n / samples;
  const bool far = samples >= kLongRay && rays <= kSharedRays;
  const bool near = !(samples >= (it.n > kHeldRays ? kLongMap : kLongRay) && rays <= kSpreadRays);
  const auto go = [&](auto kernel, int width) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)((it.n + width - 1) / width)), dim3(kNTc), 0, stream,
                       it);
  };
  if (it.grp == 0) {
    if (it.n <= kFewRays) go(k_clear_sparse<kRaysFew>, kRaysFew);
    else if (it.n <= kShortRays) go(k_clear_sparse<kRaysShort>, kRaysShort);
    else go(k_clear_sparse<kRaysPlain>, kRaysPlain);
    return hipGetLastError();
  }
  const auto form = [&](auto consecutive, auto shared, int rays) {
    if (far) go(shared, rays);
    else go(consecutive, rays);
  };
  if (it.L.ub || (it.n > kFewRays && it.n <= kShortRays))
    form(k_clear_march<kRaysShort, 0, 1>,
         k_clear_march<kRaysShort, kRunShared, kNTc / kRaysShort>, kRaysShort);
  else if (it.n <= kFewRays)
    form(k_clear_march<kRaysFew, 0, 1>, k_clear_march<kRaysFew, kRunShared, kNTc / kRaysFew>,
         kRaysFew);
  else if (far || near)
    form(k_clear_march<kRaysPlain, 0, 1>,
         k_clear_march<kRaysPlain, kRunShared, kNTc / kRaysPlain>, kRaysPlain);
  else
    go(k_clear_march<kRaysPlain, kRunSpread, 1>, kRaysPlain);
  return hipGetLastError();
}

hipError_t launch_clear_batch(const Batch* d_batch, int grid_setup, int grid_march,
                              int grid_sparse, hipStream_t stream) {
  {
    TimedLaunch tl("k_clear_setup_b", stream);
    hipLaunchKernelGGL(k_clear_setup_b, dim3(grid_setup), dim3(kNTc), 0, stream, d_batch);
  }
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  {
    TimedLaunch tl("k_clear_march_b", stream);
    hipLaunchKernelGGL(k_clear_march_b, dim3(grid_march), dim3(kNTc), 0, stream, d_batch);
  }
  if (grid_sparse > 0) {  // no item needs it: no launch
    TimedLaunch tl("k_clear_sparse_b", stream);
    hipLaunchKernelGGL(k_clear_sparse_b, dim3(grid_sparse), dim3(kNTc), 0, stream, d_batch);
  }
  return hipGetLastError();
}

}  // namespace emx
