// Internal declarations shared by the kernels and the host library.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "vlbm.h"

namespace vlbm {

// Scheme parameters shared by every instance of a context.
struct Scheme {
  double gamma, alpha, beta, a_fixed, eps, rlmp_lo, rlmp_hi;
  int a_mode, order, limiters, bc_x, bc_y, sponge;
};

// One problem instance inside the state buffers.
struct Inst {
  long long off;   // element offset of cell (0, 0) inside every plane
  long long item0; // first work item (strip) of this instance
  double dx;
  int nx, ny;
  int xs, ys;      // strips along x and y
  int strip_h;     // rows per strip of this instance
  int pad_;
};

// Boundary description of one instance: per-cell kinds and Dirichlet moments
// of the four sides (west, east, south, north; null: zero-gradient), see
// lbm_set_boundary.
struct BndDesc {
  const uint8_t* kind[4];
  const double* state[4];
};

// Per-instance device scalars.  lam and t rotate over three slots: step n
// reads slot n % 3, writes slot (n + 1) % 3 and clears slot (n + 2) % 3.
struct alignas(128) Slots {
  unsigned long long lam[3]; // bit patterns of non-negative doubles
  double t[3];
  // guard, limited, bad, bouchut, lmp, non-finite, rho <= 0 (cumulative); of
  // the bad cells, those neither non-finite nor with rho <= 0 have p <= 0
  unsigned long long cnt[7];
};
enum {
  CNT_GUARD = 0,
  CNT_LIMITED = 1,
  CNT_BAD = 2,
  CNT_BOUCHUT = 3,
  CNT_LMP = 4,
  CNT_NONFINITE = 5,
  CNT_RHO = 6,
  CNT_N = 7
};
static_assert(sizeof(Slots) == 128, "one 128-byte record per instance");

// Shards: the step kernels raise lambda and the counters of an instance in
// kShards further records of the same form (t unused).  Atomics of many waves
// on one cache line queue at 40-100 ns each (the L2s of the XCDs are not
// shared, so they meet at the memory side): with one record the last waves of a
// short launch waited for the others' counts, 53 us a step on a 400^2 grid
// under LMP, where most waves hold a limited face, against 38 us with the
// records spread; 293 against 276 us at 2048^2.  8 records: 40 us, 16: 38.4,
// 32 and 64: 38.0.  The next step takes the largest of the shards' lambdas;
// launch_fold folds the shards into the instance's own record before the host
// reads that.
constexpr int kShards = 32;  // at most the wave's 64 lanes, a power of two
// Shards in use for an instance of `strips` strips of four rows (fixed for a
// context): one for every 16 strips; a single one is the slot record itself.  On the smallest grids, whose few waves
// do not queue, reading 32 lines instead of one at the start of every step
// costs more than it saves (64^2: 0.8 us of 17).
inline int shards_for(long long strips) {
  int n = 1;
  while (n < kShards && n * 16 < strips) n *= 2;
  return n;
}

struct StepArgs {
  const void* src;
  void* dst;
  long long plane;        // elements per plane (sum of all instances' cells)
  Slots* slots;           // [n_inst]
  const Inst* insts;      // [n_inst], device memory
  const int* item_inst;   // [n_items] instance of every item (batches), or null
  Inst inst0;             // the instance when n_inst == 1
  long long n_items;
  int n_inst;
  int slot;               // step index mod 3
  int waves_per_group;
  int xcd_remap;          // map consecutive groups onto one XCD
  int groups;             // launched workgroups
  double* theta_x;        // optional face output (single instance)
  double* theta_y;
  // boundary descriptions: a single instance's in bnd1, an ensemble's in the
  // device table bnd_table (one entry per instance)
  union {
    BndDesc bnd1;
    const BndDesc* bnd_table;
  };
  int bnd;                // 1 if any instance has a boundary description
  int blocked;            // src and dst hold the blocked layout (a context's own
                          // buffers; every width a multiple of 64, no boundary
                          // descriptions), else planar
  Scheme sc;
  // (What follows stands at the end because the place of the descriptions above
  // decides how the compiler groups the loads of a ghost's state: with these
  // fields ahead of them the described marches loaded one of a halo cell's
  // twelve values behind the others, 2000^2 float32 PP in strips of 64 rows 378
  // us a step, so 325.)
  int past;               // 1: the new state is stored past the caches (store_past)
  int rows;               // 1: the row kernel (one row of a strip per wave; the
                          // strips are kRowsPerGroup rows high and groups counts
                          // them), 0: the marches
  Slots* shards;          // [n_inst][shard_mask + 1]; the slots themselves (mask 0) where
                          // the launch's records are parked or there are no others
  int shard_mask;
};

// Whether a step stores the new state past the caches (non-temporal) rather than
// through L2.  cells: of all instances; even: see even_rows; rows: the row
// kernel.  us a step, past / through:
// - A small state (17 MB, half of what the XCDs' L2s hold) is better not left
//   dirty in an L2 whose lines the launch's end writes back: float32 384^2 PP
//   8.8 / 9.7, 448^2 10.1 / 11.4, 401^2 LMP 11.8 / 12.6; float64 256^2 PP 7.65 /
//   8.2, 320^2 10.2 / 11.2, but 352^2 14.8 / 13.6.
// - Beyond that, while the old and the new state fit the last-level cache, the
//   next step finds there what went through: float32 640^2 PP 20.4 / 18.7,
//   896^2 33.6 / 29.0, 1280^2 67.4 / 59.2, LMP 79.9 / 75; float64 512^2 PP 25.3 /
//   19.4, LMP 31 / 23.8.
// - Larger float32 states are read from memory anyway: 4096^2 PP 509 / 525,
//   8192^2 2% in favour of past.  Float64 there is within 1.5% either way with even
//   rows (8192^2 PP 3936 / 3925, LMP 3979 / 4036, 2048^2 277 / 275) and loses with
//   others (2001^2 353 / 299), so it goes through.
// - A row that starts off 64 bytes leaves a partial line at both ends of each
//   strip, which past the caches costs a read-modify-write and through L2 is
//   completed by the neighbouring strip: float32 2001 x 2047 PP 208 / 172, LMP
//   247 / 191; 4001^2 801 / 618, 933 / 730; 801 x 799 35 / 27; float64 257^2
//   10.9 / 10.1 (small float32 states are better past all the same).
inline bool store_past(int precision, long long cells, bool even, bool rows) {
  const bool small = cells * (precision == 0 ? 160 : 80) <= 17000000;
  if (precision == 0) return rows && small && even;
  return small || (even && cells * 160 > (256ll << 20));
}

// Whether an instance's rows in the planar layout start on multiples of 16
// elements only (64 bytes with the float32 state).
inline bool even_rows(const Inst& in, long long plane) { return ((in.nx | in.off | plane) & 15) == 0; }

// Rows of a strip that one workgroup of the row kernel takes, one per wave.
constexpr int kRowsPerGroup = 4;

// Workgroups of 256 threads that one launch can have: its threads must count
// fewer than 2^32, and the groups are rounded up to the 8 XCDs.
constexpr long long kMaxGroups = (1ll << 24) - 8;

// What the rules of the launch look at in a context's instances.
struct Extent {
  int n_inst = 0;
  long long strip_rows = 0;  // 64-column strip rows
  long long edge_rows = 0;   // those that read ghosts (two layers, as under density bounds)
  long long row_groups = 0;  // workgroups of the row kernel
  long long cells = 0;
  int max_ny = 0;
  void add(int nx, int ny) {
    const long long xs = (nx + 63ll) / 64;
    n_inst += 1;
    cells += (long long)nx * ny;
    max_ny = ny > max_ny ? ny : max_ny;
    strip_rows += xs * ny;
    const long long inner = nx >= 130 ? (nx - 66) / 64 : 0;
    edge_rows += xs * ny - inner * (ny > 4 ? ny - 4 : 0);
    row_groups += xs * ((ny + kRowsPerGroup - 1) / kRowsPerGroup);
  }
};

// Whether a launch whose shape nobody set takes the row kernel.  A march needs some
// 1024 strips of several rows to fill the chip and spends two (four under
// density bounds) further rows on each; the row kernel has a wave for every
// row, evaluates the faces between rows twice and reads its neighbours' rows
// through the caches, which it needs to hold both states.  us a step, row kernel /
// best march (strips of 4 to 16 rows), near-vacuum rarefaction: float64 PP 64^2
// 7.3 / 19.7, 512^2 19.8 / 23.5, 901^2 47.7 / 51.7 (13515 strip rows), 960^2 69.6 /
// 65.7; LMP 512^2 24.6 / 31.9, 901^2 68.4 / 71.1, 960^2 91 / 78; float32 PP 832^2
// 25.8 / 32.0, 1024^2 34.1 / 36.0; LMP 896^2 43.8 / 47.6, 960^2 49.2 / 48.3, 1024^2
// 58 / 49.  Ensembles, whose march strips end ragged at every instance: float64
// PP 24 of 128..512 (33920 strip rows) 161 / 173, 20 of 200..600 (56415) 260 / 283;
// LMP 64 of 40..200 (19502) 113 / 138, 24 of 128..512 187 / 183; float32 PP 88 /
// 89.4 with 33920 and 112 / 106 with 44544, LMP 105 / 107 and 137 / 126.
// With boundary descriptions every row of a march looks for ghosts, here only the
// rows and strips at the edges, but those read them in up to nine chains of loads
// one after the other, so the share of such rows decides under density bounds
// (row kernel / best march).  Described on four sides (walls and zero gradient):
// - PP: 400^2 float64 18 / 58, float32 13 / 57; 64 x 200000 1179 / 1228, 707 / 655; 256
//   of 64^2 111 / 118; 8192^2 float64 5381 / 5660.  Large float32 grids are the march's:
//   3500^2 650 / 647, 4096^2 747 / 743, 5000^2 1301 / 1227, 6000^2 1930 / 1705.
// - LMP float64: squares 400^2 24 / 82, 2000^2 415 / 478, 8192^2 6584 / 6873; 300 of
//   64..512 (41% of the rows) 3219 / 3358.  Three strips wide (67%): 130 x 8333 228 /
//   237, x 33333 897 / 850, x 66666 1809 / 1515.  One or two strips: 64 x 4000 44 / 61,
//   x 8000 88 / 82, x 100000 1003 / 844; 128 of 64^2 81 / 83, of 128^2 321 / 246.
// - LMP float32: squares 400^2 19 / 72, 2000^2 267 / 284, 3500^2 814 / 775, 4096^2 1004 /
//   858, 8192^2 3825 / 3434; 500 x 25000 (25%) 1005 / 994; 130 x 66666 1044 / 914; one or
//   two strips 100 x 6000 78 / 97, 64 x 12000 74 / 83, x 25000 148 / 126, x 200000 1177 /
//   793; 300 of 64..512 1953 / 1765.
// Grids of a few columns and more than 2^26 rows have more groups of four rows
// than a launch can hold (a march's strips of 64 rows stay below).
inline bool use_rows(const Extent& x, bool bnd, int precision, const Scheme& sc) {
  if (x.row_groups > kMaxGroups) return false;
  const bool lmp = (sc.limiters & 6) != 0 && sc.order == 2;
  if (bnd) {
    const double rows = (double)x.strip_rows, edge = (double)x.edge_rows / rows;
    if (!lmp) return precision == 0 || rows <= 300e3;
    if (precision == 0) return edge <= 0.45 || rows <= 9e3 + 300e3 * (1.0 - edge);
    return rows <= __builtin_fmin(200e3, 13e3 + 400e3 * (1.0 / edge - 1.0));
  }
  if (x.n_inst > 1) return x.strip_rows <= (precision != 0 ? 36000 : lmp ? 24000 : 57000);
  return x.strip_rows <= (precision == 0 ? 13600 : lmp ? 12600 : 16400);
}

// Rows per strip of a march whose launch shape nobody set: the height with the
// least estimated time.  `strips(h)` gives the number of strips of height h.
// One round of 1024 waves (float64; 2048 with the float32 state: one or two a
// SIMD) takes a time proportional to the strip's rows and e rows of halo, with
// the float32 state and PP a little more per row on tall strips (1 + g h); a
// round that fills only a part phi of the chip runs faster per row, but not
// below a fraction c of a full one, since a lone wave's chain of rows takes
// that long.  c, e and g are fitted to 240 timings (15 grids of 960^2 to
// 8192^2 and 4 : 1, strips of 4 to 64 rows, the four classes): the height
// chosen is within 0.7% of the best on average, 13% at worst.  The tallest
// strips that fill one round, the rule before, left a nearly empty second
// round where a little more than one was needed: 1536^2 float64 PP 215 us a
// step with strips of 32 rows (1.13 rounds), 161 with 12 (3 rounds); 3072^2
// float32 PP 399 with 64 and 309 with 24; 3072^2 float64 LMP 720 / 604.  Heights
// whose groups of four waves a launch cannot hold are left out, but for the
// tallest.
// The fits hold for full strips.  Where a tenth or more of their lanes is idle
// (narrow instances) memory sets the pace less and less: a row of halo then
// costs as much as any other (two a strip, three under density bounds) and tall
// strips lose nothing, so e and g move there as the lanes in use (n) become
// few.  And a strip has no more rows than its instance.  us a step with the
// fits as they stand / so / the best of the heights: 10^6 rows of one column,
// float32 PP 1719 / 1528 / 1519; 4 x 100000 257 / 219 / 203; 20 x 200000 413 /
// 375 / 372; 3000 instances of 32^2 217 / 194 / 194; 60 of 2000 x 20, float32 LMP 152 /
// 105 / 105; 100000 x 20, float64 PP 194 / 163 / 163.  Over such grids and ensembles and those
// above, 168 in all, the choice is within 1.5% of the best on average; the
// choices for the grids above are the same.
// Nor does memory set the pace with boundary descriptions: n = 1 there, and c is
// fitted to timings of 130 such grids and ensembles (1% from the best on average:
// float32 PP 6000^2 1705 us with 48 rows, 1852 with the 12 of the other fit).
template <class Strips>
int march_rows(const Extent& x, bool bnd, int precision, bool lmp, const Strips& strips) {
  const double slots = precision == 0 ? 1024.0 : 2048.0;
  const double c = bnd ? 0.6 : lmp ? 0.44 : (precision == 0 ? 0.54 : 0.48);
  const double n = bnd ? 1.0 : __builtin_fmax(0.0, 1.0 - (double)x.cells / (64.0 * x.strip_rows) / 0.9);
  const double full = precision == 0 ? (lmp ? 1.5 : 0.75) : (lmp ? 0.75 : 0.4);
  const double e = full + ((lmp ? 3.0 : 2.0) - full) * n;
  const double g = (precision != 0 && !lmp ? 0.004 : 0.0) * (1.0 - n);
  int best = 64;
  double least = HUGE_VAL;
  for (int h : {4, 8, 12, 16, 24, 32, 48, 64}) {
    if (strips(h) > 4 * kMaxGroups) continue;
    const double rounds = (double)strips(h) / slots;
    const double whole = __builtin_floor(rounds), phi = rounds - whole;
    const double part = phi > 0.0 ? __builtin_cbrt(phi * phi * phi + c * c * c) : 0.0;
    const int tall = h < x.max_ny ? h : x.max_ny;
    const double t = (whole + part) * (tall + e) * (1.0 + g * tall);
    if (t <= least) {
      least = t;
      best = h;
    }
  }
  return best;
}

enum { BND_ZERO_GRADIENT = 0, BND_WALL = 1, BND_DIRICHLET = 2 };

// Launchers (step.hip).
hipError_t launch_step(const StepArgs& a, int precision, hipStream_t s);
// `blocked`: the state S is in the blocked layout (see step.hip), else
// planar.
hipError_t launch_init(const Scheme& sc, const Inst* insts_host, int n_inst,
                       const Inst* insts_dev, long long plane, const double* u0,
                       void* S, Slots* slots, int precision, int blocked, hipStream_t s);
// (insts_dev: the same table in device memory, used for n_inst > 1)
hipError_t launch_lambda_state(const Scheme& sc, const Inst* insts_host, const Inst* insts_dev, int n_inst,
                               long long plane, const void* S, Slots* slots, int slot, int precision,
                               int blocked, int count, hipStream_t s);
hipError_t launch_moments(const Inst& in, long long plane, const void* S,
                          double* out, int precision, int blocked, hipStream_t s);
// Every instance's state (widths multiples of 64) from src to dst, planar ->
// blocked (to_blocked = 1) or blocked -> planar (0).
hipError_t launch_relayout(const Inst* insts_host, const Inst* insts_dev, int n_inst, long long plane, const void* src, void* dst,
                           int precision, int to_blocked, hipStream_t s);
// Per-cell blending step (an ablation): state A.src -> A.dst with the face
// factors A.theta_x / A.theta_y of the same state, single instance; also
// the step's slot bookkeeping.
hipError_t launch_percell(const StepArgs& a, int precision, hipStream_t s);
// Block minima of rho and of rho e = E - |m|^2 / (2 rho) over the finite
// cells of the moment slot, part[blocks][2].
hipError_t launch_minima(const Inst& in, long long plane, const void* S, double* part,
                         int blocks, int precision, int blocked, hipStream_t s);
// Double-double partial totals of the moment slot, part[blocks][4][2]; the
// grid is `blocks` workgroups of 256 threads.
hipError_t launch_totals(const Inst& in, long long plane, const void* S, double* part,
                         int blocks, int precision, int blocked, hipStream_t s);
hipError_t launch_clear_counts(Slots* slots, long long n, hipStream_t s);
hipError_t launch_fold(Slots* slots, Slots* shards, int n_shards, int n_inst, int clear, hipStream_t s);
hipError_t launch_fill_u32(unsigned int* p, unsigned int v, long long n, hipStream_t s);
// Raises each instance's lam[slot] to the largest wavespeed of its Dirichlet
// boundary states.
hipError_t launch_bnd_lambda(const StepArgs& a, int slot, hipStream_t s);
hipError_t launch_fill_f64(double* p, double v, long long n, hipStream_t s);
// Adjoint (adjoint.hip).  Boundary kinds per side (west, east, south,
// north), uint8 device arrays as in StepArgs; NULL: zero-gradient.
struct BndKinds {
  const uint8_t* k[4];
};
hipError_t launch_adjoint_step(const Scheme& sc, const Inst& in, long long plane,
                               const double* U, const double* Ubar1, double* Ubar0,
                               const double* theta_x, const double* theta_y,
                               const Slots* slot_src, int slot, const BndKinds& kinds,
                               hipStream_t s);
hipError_t launch_adjoint_init(const Scheme& sc, const Inst& in, const double* u0,
                               const double* Ubar0, double* u0bar,
                               const Slots* slots, int slot, hipStream_t s);

// Host helpers of the C ABI (api.hip): parameter checks (NULL when valid),
// the kernels' scheme record, and the message lbm_last_error(NULL) returns.
const char* host_check_params(const lbm_params* p);
Scheme host_make_scheme(const lbm_params* p);
void host_set_error(const char* m);

}  // namespace vlbm
