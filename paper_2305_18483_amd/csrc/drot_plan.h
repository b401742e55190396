// Launch planning for the Douglas-Rachford OT solver: which kernel runs which sweep.
//
// Pure host logic, no HIP in here: drot.hip includes this header and enqueues what it decides, and
// the same header compiles with a plain C++ compiler so that every path and every switch between
// paths can be exercised without a GPU (drot_plan_host.cpp wraps it for that).
//
// One iteration of the method is a sweep over the plan (eq. (8)) followed by the vector update of
// eq. (6).  The arithmetic of an iteration is fixed; what varies is the kernel that performs it:
//
//   Resident    tiny problems: one workgroup, X and C in registers, a whole stretch per launch
//   Pro32       small problems: 32-row tiles, the vector update of the previous iteration fused
//               into the head of the sweep (one launch per iteration)
//   Plain32     32-row tiles, every byte moved; also the first sweep of every cold start and the
//               two sweeps of an even/odd pair (mode 1 stores X - rho*C, mode 2 reads it, no C)
//   Tall64      64-row tiles; all-zero row segments of X neither read nor written back
//   Screened8   the same tiles; row segments certified to stay zero also skip their reads of C;
//               with `refresh` it reads all of C and records the bounds the certificates use
//   Lean        one wave per 64 x 256 tile, reads and writes 128-byte lines, for plans that are thinning out or sparse;
//               renews its bounds itself
//   Points      cost recomputed from point clouds on the matrix cores (32-row tiles); with `refresh` it
//               also records the screening bounds
//   PointsLean  the same cost for the rows a certificate does not cover only (256-row strips)
//   (Active     entries that hold something or may come to, listed and kept on the chip: many iterations in one launch)
//   Slab        group lasso, a whole class x 32 columns resident in one workgroup
//   TwoPass     group lasso, any labels: norms first, then the scaled update
//
// Where X and C fit the registers of the whole chip, a stretch of Pro32 or Tall64 sweeps and their vector updates run in
// one cooperative launch (make_static's grid_tiles, grid_head); the sweeps planned are the same.
//
// The choice depends on the problem (sizes, regularizer, alignment), on the options, on what the
// previous sweeps left in memory (row-segment sums, line flags, bounds) and, where the host reads
// the status block during the solve, on the density of the plan it reports.
#ifndef DROT_PLAN_H_
#define DROT_PLAN_H_

#include <cmath>
#include <cstddef>
#include <vector>

namespace drot_plan {

// Geometry the kernels are written for (drot.hip checks these against the kernels' own constants).
constexpr int kSegCols = 256;         // columns of a row segment / of a tile
constexpr int kTileRows = 32;         // rows of the small tile
constexpr int kTallTileRows = 64;     // rows of the tile of Tall64, Screened8 and Lean
constexpr int kAlignElems = 32;       // rows must start on 128-byte lines
constexpr int kSlabCols = 32;         // columns of a group-lasso slab
constexpr int kSlabLanes = 8;         // lanes along them
constexpr int kSlabRowLanes = 128;    // row lanes of the slab kernel (K = 1, 2, 4, 8 rows per lane)
constexpr int kSlabMaxRows = 1024;    // longest class the slab kernel holds
// The fused update has every slab's workgroup add up all the partial sums of its rows and columns again: cheap as long as
// the workgroups run side by side, one per compute unit; in a second round all of it comes on top.  Per iteration, fused
// and with the merged update: 2000 x 1500, 5 classes (235 slabs) 10.7 and 11.3 us, 10 classes (470) 15.2 and 10.6,
// 40 classes 44.8 and 16.6; 2000 x 2000, 4 classes (252) 12.7 and 12.6, 8 classes 17.7 and 11.3.
constexpr int kFusedSlabs = 256;
// Classes that are not runs of rows go through the slab kernel where their rows fill at least this part of its row lanes
// (128 K per class, whatever the class's size).  Per iteration, slabs and two passes: 2000 x 1500 with 40 classes of 50
// rows (0.39) 17 and 36 us; 5000 x 5000, 100 classes of 50 (0.39) 85 and 91, 156 of 32 (0.25) 120 and 93;
// 10000 x 8000, 100 of 100 (0.78) 204 and 337, 300 of 33 (0.26) 405 and 345.
constexpr double kMappedFill = 0.375;
constexpr int kResidentMaxRows = 128, kResidentCols = 256;
constexpr int kColGroup = 4;          // the lean sweep adds the column sums of four tiles before it stores
constexpr int kStripRows = 256;       // rows of a strip of the point-cloud variant's screened sweep
constexpr int kPointsColGroup = 8;    // ... which adds the column sums of its eight 32-row tiles before it stores
constexpr size_t kScreenFrom = (size_t)11 << 20;  // screening on automatic: from this many entries up
constexpr int kFirstRefreshPeriod = 8, kMaxRefreshPeriod = 1024;
constexpr int kFirstPeriodLines = 6;  // ... where the sweep by lines takes over after the second epoch's first sweep
// Grid-resident stretches (drot_grid.h): tiles a workgroup holds in registers and LDS, one workgroup per compute unit.
// (At the largest size that fits an iteration takes 9.8 us against 30 in single launches on 32-row tiles, 7.9 against
// 18.6 on 64-row tiles, and at the smallest 2.6 against 6.5: no size below the limit is better off without.)
constexpr int kGridTiles32 = 5;       // 32-row tiles (two rows per wave, 16 waves of 128 registers)
constexpr int kGridTiles64 = 3;       // 64-row tiles (eight rows per wave, 8 waves of 256 registers)
constexpr int kGridWaves32 = 16, kGridWaves64 = 8;
constexpr int kGridMostUnits = 256;   // workgroups at most
constexpr int kGridBlock = 8;         // rows or columns whose part of eq. (6) a wave forms
// Slabs (drot_grid_slab.h): rows per thread at least (idle ones cost little), and at most, over a workgroup's slabs (registers
// hold X, the LDS C).  Half slabs to a workgroup where all of them are on the chip at once, else whole ones, else two.
constexpr int kGridSlabLeastK = 4, kGridSlabRows = 8;
// Shorter stretches are not worth fetching the plan and the cost for.  Per iteration, in single launches and in one launch,
// stretches of 4, 6, 8 and 10 sweeps: 200 x 300 10.4 and 13.6 us, 8.9 and 10.1, 8.3 and 8.5, 7.9 and 7.4; 1000 x 1000 11.3
// and 13.7, 9.9 and 10.2, 9.9 and 8.5, 9.4 and 7.5 (one tile a workgroup); 2048 x 3072 24.0 and 18.5 at 4, 64-row tiles of
// 2300 x 2500 17.8 and 17.8, 2999 x 3307 21.3 and 21.3.  Slabs, and point clouds of one tile a workgroup, have the line of the one
// tile; whole calls of 4, 6 and 8 sweeps, single launches and one: point clouds 400 x 400 115 and 103 us, 145 and 115, 166 and 120;
// slabs 1500 x 1000 193 and 178, 212 and 184, 234 and 190; 2000 x 1500, five classes in no order 268 and 250, 297 and 257, 332
// and 262.  So their line could lie at 4, too.
constexpr int kGridMinSweeps = 4, kGridMinSweepsOneTile = 8;
// (a full sweep takes 230 to 260 us at 12000 x 12000, d = 32, the screened one 7 for every percent of the row segments left)
constexpr double kPointsSparse = 0.33;
// Active entries (drot_active.h): 16 x 16 workgroups of at most kActiveLocal groups of 256 rows and segments of 256 columns
constexpr int kActiveSide = 16, kActiveLocal = 5;
constexpr int kActiveEntries = 4096;   // ... and so many entries each
constexpr double kActiveFill = 0.6;    // point clouds: of them, on average, from the row segments that hold something
// Stored costs: of them, expected in the busiest workgroup where the entries of a list have been counted in advance, those within the slack among
// them, and else by what the plan holds.  Of 240 calls of 3000 x 5595 to 20000 x 20000, each listed at the first count below a higher line: at
// iteration 16, whose fast rise does not last, the lists held up to 1.18 (of 73 calls, 10 in vain, in few dimensions) and of 25 above once (1.27);
// later, where the plan alone held no more than 0.56, up to 1.12 (all of 33), and where it held more up to 0.85, in vain from 0.95 on (8).
constexpr double kActiveForecastEarly = 1.2, kActiveForecastThin = 1.12, kActiveForecast = 0.94, kActiveThin = 0.58, kActiveExpected = 0.75;
constexpr int kActiveEarly = 32;
// ... of point clouds below this many nonzero row segments: 12000 x 12000, d = 32, 276 us a full sweep: listed at 0.31, iteration 32, 15.1 ms for
// 500 iterations; at 0.53, iteration 24, 13.5; tried in vain at 0.88 and listed at 0.53 15.4.
constexpr double kActivePoints = 0.6;
constexpr int kActiveLeast = 16;       // shorter calls are not worth a list
// Iterations a list is meant to last: longer lists are made less often, and hold more.  At 48, 28 and 20: 10000 x 10000 (1000
// iterations) 14.6, 13.6, 13.7 ms; 20000 x 20000 (500) 18.45, 18.6, 18.8; point clouds 4001 x 3999 (400) 7.7, 6.1, 5.0; 12000 x 12100, quadratic
// (400) 16.25, 15.9, 15.5 (does not fit at 48).
constexpr int kActiveTarget = 20;
// ... and has to last to be worth making.  A list takes 25 to 80 us in a workgroup, the slowest one's counts; of point clouds of few dimensions 150 to 300.  A sweep over everything takes
// 12 to 20 us longer than an iteration on the active entries over a stored cost (7000 x 7100 with lists of 8 iterations and up 11.9 ms, with
// sweeps alone 10.2, with lists of 16 and up 10.3); over point clouds, d = 2 or 3, a third of a nanosecond per row segment.  Point clouds with lists
// of 3, of 6 and of 10 iterations and up, ms (and with sweeps alone): 75000 row segments (7552 x 2460, 211 iterations) 14.6, 12.2, 9.0 (12.1);
// 80000 (5000 x 4000, 400) 16.9, 16.9, 15.8 (16.6); 128000 (3875 x 8384, 200) 17.6, 11.3, 11.1 (13.4); 200000 (7480 x 6816, 200) 10.7, 10.7, 13.9
// (18.7); 324000 (9000 x 9000, 400) 51.8, 47.8, 47.6 (44.8); 564000 (12000 x 12000, 200) 13.5, 13.6, 17.1 (30.3), with d = 2 39.5, 35.8, 35.5 (40.3).
constexpr int kActiveShortest = 16, kActiveShortestPoints = 10, kActiveShortestPointsLarge = 6, kActivePointsLarge = 150000;
// Point clouds whose entries did not fit are tried again early where this share, or less, of the row segments is left that held something then.
constexpr double kActiveFallen = 0.8;
constexpr int kPromptLooksUntil = 128; // ... of which the host waits for those of a point-cloud solve until the plan is sparse
constexpr int kEarlyLooksUntil = 512;  // cold starts: extra density readings over this many iterations

inline int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Rows of column sums that the slabs leave: one per run, two per class whose rows are fetched through a table (its sums in
// two parts).  There are at most m / (kMappedFill 128) such classes.
inline int slab_col_rows(int nruns, bool mapped) { return mapped ? 2 * nruns : nruns; }
inline int most_col_rows(int m) {
  const int tiles = ceil_div(m, kTileRows), parts = slab_col_rows((int)(m / (kMappedFill * kSlabRowLanes)), true);
  return tiles > parts ? tiles : parts;
}

enum Regularizer { kNone = 0, kQuadratic = 1, kGroupLasso = 2 };

struct Options {
  int check_every = 100;
  int resident = -1;        // -1 automatic, 0 never
  int fused_update = -1;    // -1 automatic, 0 never
  int skip_cost = -1;       // even/odd pairs: -1 by density, 0 never, 1 wherever they apply
  int skip_unchanged = -1;  // zero-segment skipping: -1/1 on, 0 off
  int screening = -1;       // -1 from kScreenFrom entries up, 0 never, 1 always, k >= 2 always, renewed at least every k
  int nontemporal = -1;     // -1 by size, 0 never, 1 always
  int force_two_pass = 0;   // group lasso: never the slab kernel
  int gap_every = 0;        // objective / gap / dual residual at every gap_every-th residual check (0: only at the end)
};

struct Problem {
  int m = 0, n = 0;
  int reg_kind = kNone;
  bool from_points = false;   // cost recomputed from point clouds
  bool warm = false;          // caller-supplied starting point
  bool resume = false;        // continues the previous solve on the handle
  bool has_weights = false;   // weighted l1 term: the solve runs on a working copy C + W
  bool c_on_lines = true;     // base address of C is a multiple of 128
  bool x_on_lines = true;     // base address of X_out is a multiple of 128
  int slab_k = 0;             // group lasso: rows per lane of the slab kernel, 0 = two-pass path
  int nruns = 0;              // group lasso: runs of equal labels
  bool mapped_rows = false;   // group lasso: the slab kernel fetches the rows of a class through a table
  size_t tilesum_half = 0;    // capacity of one half of the tile-total buffer
  float rho = 0.f;            // stepsize
  bool feedback = true;       // the host reads the status block during the solve
  bool checking = false;      // a tolerance was given
  int max_iters = 0;
  int compute_units = 0;      // workgroups of a cooperative launch that are on the chip together (0: no such launches)
  bool line_bounds = false;      // the workspace holds the bounds by line, without which there is no lean sweep
  bool single_launches = false;  // every sweep in a launch of its own all the same (profile mode, callers that may capture)
};

// What a solve hands to the next one on the same handle (continued solves).
struct Carry {
  bool dense_plan = false;
  double plan_density = -1.0;
  long long epoch_gen = -1;      // sweep that last recorded the screening bounds
  int refresh_period = kFirstRefreshPeriod;
  bool bounds_from_points = false;  // ... from a cost formed from point clouds (no bounds by line then), or a stored one
  float bounds_rho = 0.f;           // ... with this stepsize
  bool sums_valid = false;       // the row-segment sums of the last sweep describe the X in memory
  int sums_strip = 0;            // ... in pieces of this many columns
  bool lines_valid = false;      // the same for the lean sweep's line flags
  bool by_lines = false;         // the plan has thinned out enough for the lean sweep
  bool drift_valid = false;      // the last vector update left the drift of varphi for it
  double lines = -1.0;           // fraction of nonzero lines last reported
  long long bound_gen = -1;      // iteration whose varphi the bounds by line that a launch of active entries left are against
  long long recorded_gen = -1;   // sweep over point clouds that last recorded bounds by line
  long long iters_done = 0;
};

// Decisions that hold for the whole call.
struct Static {
  int nseg = 0, ntr = 0, ntiles = 0, ntr_tall = 0;
  int nbm = 0, nbn = 0;          // workgroups of the reduction: 64 rows resp. 64 columns each
  int ld_pad = 0;                // pitch of the padded working copies
  bool nt = false;               // non-temporal accesses
  bool resident = false;
  bool pad_c = false, pad_x = false;
  int nstrips = 0;
  bool small_slab = false, small = false, fused = false;
  bool can_pair = false, adaptive_pairs = false, may_screen = false, adaptive = false;
  bool points_screen = false;    // point-cloud variant: screened sweeps once the plan is known to be sparse
  bool active = false;           // active entries once the plan is known to be sparse
  int refresh_max = kMaxRefreshPeriod;
  bool lean_fits = false;        // the rows of a tile of the lean sweep are within 32 bits of bytes from its first one
  bool early_lines = false;      // the lean sweep does not wait for a sparse plan
  double pairs_until = 0.5;      // the pairs end below this fraction of nonzero row segments, where they would not start
  int sums_strip = kSegCols;
  int grid_tiles = 0;            // grid-resident stretches: tiles per workgroup, 0: none
  int grid_wgs = 0;              // ... and workgroups
  bool grid_tall = false;        // ... of 64 rows each (else 32)
  int grid_points = 0;           // the same with the cost formed from point clouds: 32-row tiles per workgroup
  int grid_slab_lanes = 0;       // slabs in place of tiles: lanes along the columns of a workgroup (8, or 4: half a slab), else 0
  int grid_slab_k = 0;           // ... and rows per thread
  bool status_at_checks = false; // the stretches end with a status kernel (stopping test and / or density)
};

// Non-temporal accesses pay off once X and C together no longer fit the 256 MB memory-side cache.
// Measured crossover on MI355X: cacheable wins at 8mn = 290 MB (7.2 vs 6.1 TB/s), non-temporal at
// 393 MB (6.1 vs 5.7 TB/s).
inline bool use_nontemporal(int m, int n) { return 8.0 * (double)m * (double)n > 320.0 * 1024 * 1024; }

inline Static make_static(const Problem& P, const Options& O) {
  Static S;
  const int m = P.m, n = P.n;
  S.nseg = ceil_div(n, kSegCols);
  S.ntr = ceil_div(m, kTileRows);
  S.ntiles = S.nseg * S.ntr;
  S.ntr_tall = ceil_div(m, kTallTileRows);
  S.nbm = ceil_div(m, 64);
  S.nbn = ceil_div(n, 64);
  S.ld_pad = ceil_div(n, kAlignElems) * kAlignElems;
  S.nt = O.nontemporal < 0 ? use_nontemporal(m, n) : O.nontemporal != 0;
  S.resident = O.resident != 0 && P.reg_kind != kGroupLasso && !P.from_points && m <= kResidentMaxRows &&
               n <= kResidentCols;
  const bool rows_off_lines = n % kAlignElems != 0;
  S.pad_c = P.has_weights || (!S.resident && !P.from_points && (rows_off_lines || !P.c_on_lines));
  S.pad_x = !S.resident && (rows_off_lines || !P.x_on_lines);
  S.nstrips = ceil_div(n, kSlabCols);
  S.small_slab = P.slab_k && S.nstrips <= 64 && P.nruns <= 64 && S.nstrips * P.nruns <= kFusedSlabs;
  S.small = S.small_slab || (P.reg_kind != kGroupLasso && !P.from_points && S.ntr <= 64 && S.ntiles <= 4096);
  S.fused = S.small && O.fused_update != 0;
  S.can_pair = P.reg_kind != kGroupLasso && !S.fused && !P.from_points;
  S.may_screen = S.can_pair && !S.small && O.skip_cost != 1 && O.skip_unchanged != 0 &&
                 (O.screening > 0 || (O.screening == -1 && (size_t)m * (size_t)n >= kScreenFrom));
  // X and C stay in the registers of the whole chip from one check to the next where they fit: the sweeps of the fused
  // small-problem path on 32-row tiles, those that only skip zero segments on 64-row tiles (the same bits either way).
  // Above their size a problem is screened or streamed.
  const bool sweeps64 = S.can_pair && !S.small && O.skip_cost != 1 && O.skip_unchanged != 0 && !S.may_screen;
  S.points_screen = P.from_points && O.skip_unchanged != 0 &&
                    (O.screening > 0 || (O.screening == -1 && (size_t)m * (size_t)n >= kScreenFrom));
  // (a launch has room for the squared residuals of the blocks that so many workgroups own)
  const int units = P.compute_units < kGridMostUnits ? P.compute_units : kGridMostUnits;
  if (units > 0 && !S.resident && ((S.fused && !P.slab_k) || sweeps64)) {
    const int tiles = sweeps64 ? S.nseg * S.ntr_tall : S.ntiles;
    const int per_wg = ceil_div(tiles, units);
    // (the first workgroup keeps theta, the waves of the others own the blocks of eq. (6): workgroups without a tile where
    // an oblong problem has more blocks than its tiles' workgroups have waves)
    const int owners = ceil_div(ceil_div(m, kGridBlock) + ceil_div(n, kGridBlock), sweeps64 ? kGridWaves64 : kGridWaves32);
    const int wgs = ceil_div(tiles, per_wg) > 1 + owners ? ceil_div(tiles, per_wg) : 1 + owners;
    if (per_wg <= (sweeps64 ? kGridTiles64 : kGridTiles32) && wgs <= units) {
      S.grid_tiles = per_wg;
      S.grid_wgs = wgs;
      S.grid_tall = sweeps64;
    }
  }
  if (units > 0 && P.from_points && O.fused_update != 0 && O.skip_unchanged != 0 && !S.points_screen) {
    const int per_wg = ceil_div(S.ntiles, units);
    const int owners = ceil_div(ceil_div(m, kGridBlock) + ceil_div(n, kGridBlock), kGridWaves32);
    const int wgs = ceil_div(S.ntiles, per_wg) > 1 + owners ? ceil_div(S.ntiles, per_wg) : 1 + owners;
    if (per_wg <= kGridTiles32 && wgs <= units) {
      S.grid_points = per_wg;
      S.grid_wgs = wgs;
    }
  }
  // (group lasso: every workgroup holds slabs, none owns blocks only.  Here and above the option that asks for the vector
  // update in a launch of its own is the one that keeps a call off launches that hold every compute unit)
  if (units > 0 && P.slab_k && O.fused_update != 0 && (S.small || (size_t)S.nstrips * (size_t)P.nruns <= P.tilesum_half)) {
    const int k = P.slab_k < kGridSlabLeastK ? kGridSlabLeastK : P.slab_k;
    const int slabs = S.nstrips * P.nruns, blocks = ceil_div(m, kGridBlock) + ceil_div(n, kGridBlock);
    auto take = [&](int lanes, int per_wg) {
      const int wgs = ceil_div(slabs * (kSlabLanes / lanes), per_wg), owners = ceil_div(blocks, kSlabRowLanes * lanes / 64);
      if (S.grid_tiles || wgs > units || 1 + owners > wgs) return;
      S.grid_tiles = per_wg;
      S.grid_wgs = wgs;
      S.grid_slab_lanes = lanes;
      S.grid_slab_k = k;
    };
    take(4, 1);
    take(8, 1);
    if (k * 2 <= kGridSlabRows) take(8, 2);
  }
  S.adaptive_pairs = P.feedback && S.can_pair && !S.small && O.skip_cost == -1 && O.skip_unchanged != 0 && !S.grid_tiles;
  S.adaptive = P.feedback && (S.adaptive_pairs || S.may_screen || S.points_screen);
  // (smaller problems, screened when asked to, lie in the caches: lines gain nothing over row segments there)
  // (offsets of 32 bits within a tile: rows of up to 16.7 million columns; wider ones stay with the 8-wave tiles)
  S.lean_fits = (size_t)kTallTileRows * 4 * (size_t)S.ld_pad <= 0xffffffffu;
  S.early_lines = S.lean_fits && P.line_bounds && S.may_screen && (size_t)m * (size_t)n >= kScreenFrom;
  // (one workgroup per compute unit; the option that asks for the vector update in a launch of its own keeps a call off
  // launches that hold every compute unit, here as elsewhere)
  S.active = units >= kActiveSide * kActiveSide && O.fused_update != 0 && O.screening == -1 && P.feedback && O.gap_every < 1 &&
             (S.early_lines || S.points_screen) && S.nseg <= kActiveSide * kActiveLocal &&
             ceil_div(m, 256) <= kActiveSide * kActiveLocal;
  if (S.early_lines) S.pairs_until = 0.995;  // (the sweep by lines waits: whatever does not start the pairs ends them)
  S.refresh_max = O.screening >= 2 ? O.screening : kMaxRefreshPeriod;
  S.sums_strip = P.slab_k ? kSlabCols : kSegCols;
  S.status_at_checks = P.checking || S.adaptive || O.gap_every > 0;
  return S;
}

// What changes from sweep to sweep.
struct State {
  long long k_base = 0;          // iterations the state on the handle had seen before this call
  int k = 0;                     // iterations enqueued by this call
  long long sums_gen = -1;       // sweep whose row-segment sums describe the plain X in memory, or -1
  long long lines_gen = -1;      // the same for the lean sweep's line flags
  long long epoch_gen = -1;      // sweep that last recorded the screening bounds (host's record)
  int refresh_period = kFirstRefreshPeriod;
  bool dense_plan = false;       // the last status reported a dense plan: even/odd pairs
  double plan_density = -1.0;    // fraction of nonzero row segments, once a status has come back
  bool by_lines = false;         // the lean sweep may run (with line bounds): two epochs of bounds, or a sparse plan reported
  long long drift_gen = -1;      // sweep whose vector update left the drift of varphi since the epoch of the bounds
  bool dense_lines = false;      // ... but the last status found most lines nonzero
  double lines = -1.0;           // fraction of nonzero lines the last status that counted them reported
  long long bound_gen = -1;      // iteration whose varphi the bounds by line that a launch of active entries left are against
  long long recorded_gen = -1;   // sweep over point clouds that last recorded bounds by line: not every epoch of theirs has some
  int active_from = 0;           // no such launch before this iteration of the call
  int active_again = 0;          // ... or, once the plan has thinned out since, before this one
  double active_density = -1.0;  // plan_density when the last one that ended early started
  int forecast_k = -1;           // iteration of the call at which the entries of a list were last counted in advance ...
  int forecast_age = 0;          // ... how old the bounds are, which the sweep by lines renews by itself ...
  double forecast = 0.0;         // ... and how many the busiest workgroup would have, of kActiveEntries
  int active_left = 0;           // launches of them that ended early
  bool active_ran = false;
  bool last_lean = false;        // the sweep before the next status is a lean one
  bool materialized = true;      // phi, varphi, a, b, theta in memory are complete for the sweeps done
  bool norms_pending = false;    // the last vector update left the residual norms as per-workgroup sums
};

// The bounds by line a launch of active entries would start from, the newer ones of two: what the last such launch left (against the
// varphi it left, which stays with them), or what the last sweep to record any did, against the varphi of the last epoch.  Over a
// stored cost every epoch has bounds by line; over point clouds those of calls that could take such a launch.
enum ActiveBounds { kNoBounds = 0, kLeftBounds, kRecordedBounds };
inline ActiveBounds active_bounds(const Problem& P, const State& T) {
  const long long recorded = P.from_points ? T.recorded_gen : T.epoch_gen;
  if (T.bound_gen >= 0 && T.bound_gen >= recorded) return kLeftBounds;
  return recorded >= 0 && recorded == T.epoch_gen ? kRecordedBounds : kNoBounds;
}

inline State start_state(const Static& S, const Problem& P, const Carry& carry) {
  State T;
  T.k_base = P.resume ? carry.iters_done : 0;
  T.dense_plan = P.resume && carry.dense_plan;
  T.plan_density = P.resume ? carry.plan_density : -1.0;
  T.by_lines = P.resume && carry.by_lines;
  // (the bounds are of varphi_j - rho C_ij as the sweep that recorded them formed it, and the sweeps over point clouds
  // record none by line: where the cost comes from elsewhere now, or the stepsize is another, new ones come first)
  const bool bounds_hold = P.resume && carry.bounds_from_points == P.from_points && carry.bounds_rho == P.rho;
  T.drift_gen = bounds_hold && carry.drift_valid ? T.k_base : -1;
  // (a continued solve starts from the X the last one returned, so its row-segment sums still hold;
  // the warm start's sums are those of 256-column segments)
  T.sums_gen = P.warm ? (P.slab_k ? -1 : 0)
                      : (P.resume && carry.sums_valid && carry.sums_strip == S.sums_strip) ? T.k_base : -1;
  T.lines = P.resume ? carry.lines : -1.0;
  T.bound_gen = bounds_hold ? carry.bound_gen : -1;
  T.recorded_gen = bounds_hold ? carry.recorded_gen : -1;
  T.lines_gen = (P.resume && carry.lines_valid && T.sums_gen >= 0) ? T.k_base : -1;
  T.epoch_gen = bounds_hold ? carry.epoch_gen : -1;
  // (an epoch without bounds by line is none where active entries may come: the next full sweep records both)
  if (S.active && P.from_points && active_bounds(P, T) == kNoBounds) T.epoch_gen = -1;
  T.refresh_period = bounds_hold ? carry.refresh_period : S.early_lines ? kFirstPeriodLines : kFirstRefreshPeriod;
  if (T.refresh_period > S.refresh_max) T.refresh_period = S.refresh_max;
  return T;
}

// A stretch: the sweeps up to the next status (stopping test at the multiples of check_every; over
// the first iterations of a cold start also looks at the density only, after 16 and then every 32
// iterations: a plan goes through phases -- empty, dense, then as sparse as it will be -- and a wrong
// choice of sweep should not last a whole check interval).
//
// A launch that runs on through the checks, and one of point clouds or slabs whatever the call, has at most kRunSweeps sweeps
// (or reaches one check): the largest tiles take 10 us, the largest slabs 14, so that other work on the GPU waits no longer
// than 60 ms.
constexpr int kRunSweeps = 4096, kRunChecks = 256;
// (... on active entries: an iteration of 11 to 15 us and its share of the lists, 300 us at most for 16 iterations, over point clouds for 6)
constexpr int kRunActive = 2048, kRunActivePoints = 1024;
struct Stretch {
  int chunk = 0;
  bool prompt = false;     // the host waits for the status at its end before it plans on
  bool probe = false;      // ends with a status for the host's choice of sweep only (no stopping test)
  bool skip_cost = false;  // even/odd pairs in this stretch
  bool tall = false;       // 64-row tiles in this stretch
  bool gap = false;        // the status at its end carries objective, gap and dual residual
};

inline Stretch next_stretch(const Static& S, const Problem& P, const Options& O, const State& T) {
  Stretch R;
  const int k = T.k;
  R.chunk = P.max_iters - k;
  if (S.status_at_checks) {
    const int to_check = O.check_every - k % O.check_every;  // the tests stay at multiples of check_every
    if (to_check < R.chunk) R.chunk = to_check;
    if (S.adaptive && !P.resume && k < kEarlyLooksUntil) {
      // (point clouds: every 8 iterations at first, read at once.  Not to know for 32 to 64 sweeps that the plan has
      // become sparse costs 10 ms of 44 at 12000 x 12000, waiting 10 us a look)
      const bool often = P.from_points && k < kPromptLooksUntil && !(T.plan_density >= 0.0 && T.plan_density < kPointsSparse);
      const int next = k < 16 ? 16 : often ? (k / 8 + 1) * 8 : (k / 32 + 1) * 32;
      // (and where the active entries could be listed: a sweep by lines takes three times an iteration of theirs; over point clouds, where
      // they did not fit: the plan soon fills up then, 13.7 ms in place of 17.0 for 400 iterations of 3585 x 3329 in two dimensions)
      R.prompt = often || (S.active && !P.single_launches && next <= kPromptLooksUntil && (P.from_points ? T.active_left > 0 : !T.active_ran));
      if (next - k < R.chunk) {
        R.chunk = next - k;
        R.probe = true;
      }
    }
  }
  // (a call without checks, in launches of a bounded length where its sweeps were launches of their own)
  if (!S.status_at_checks && (S.grid_points || S.grid_slab_lanes) && R.chunk > kRunSweeps) R.chunk = kRunSweeps;
  R.skip_cost = S.can_pair && (O.skip_cost == 1 || (S.adaptive_pairs && T.dense_plan));
  R.tall = !S.small && !R.skip_cost && !P.from_points && P.reg_kind != kGroupLasso && O.skip_unchanged != 0;
  const int end = k + R.chunk;
  R.gap = !R.probe && O.gap_every > 0 && end % O.check_every == 0 && (end / O.check_every) % O.gap_every == 0;
  return R;
}

enum Sweep { kResident = 0, kPro32, kPlain32, kTall64, kScreened8, kLean, kPoints, kSlab, kTwoPass, kPointsLean };
enum Update { kNoUpdate = 0, kSeparate, kMergedSlab, kMergedTiles };

struct Step {
  Sweep sweep = kPlain32;
  long long sw = 0;        // this sweep produces X_sw; its sums live in the buffers of parity sw & 1
  bool first = false;      // X_0 = 0: nothing to read
  int mode = 0;            // even/odd scheme: 0 plain, 1 stores X - rho*C, 2 reads it without C
  bool prev_sums = false;  // the row-segment sums of sweep sw - 1 tell which pieces of X are zero
  bool lines_in = false;   // lean: the line flags of sweep sw - 1 are valid
  bool refresh = false;    // Screened8: reads all of C and records the bounds
  bool pro = false;        // the vector update of sweep sw - 1 rides along at the head of this sweep
  bool tilesum = false;    // the sweep stores the totals of its tiles
  Update update = kNoUpdate;
  int ra_ntr = 0;          // rows of column partials the sweep leaves, and how the reduction groups them
  int ra_cgroup = 1;
  int tt_rows = 0, tt_group = 1;  // merged update: rows of tile totals and their grouping
  int ctl_mode = 0;        // merged update: 0 nothing, 1 after a host-ordered refresh, 2 after a lean sweep
  bool drift = false;      // merged update: leave the drift of varphi per line of columns for the lean sweep
  int profile_kind = 0;    // what drot_get_profile reports for this sweep
  int iters = 1;           // iterations the launch covers (a resident stretch: all of it)
};

// The c-th sweep of stretch R (c = 0 .. chunk-1).  Advances T.
inline Step next_sweep(const Static& S, const Problem& P, const Options& O, State& T, const Stretch& R, int c) {
  Step Q;
  const long long sw = T.k_base + T.k + 1;
  Q.sw = sw;
  Q.first = sw == 1 && !P.warm;
  Q.tilesum = S.small;
  Q.ra_ntr = P.slab_k ? slab_col_rows(P.nruns, P.mapped_rows) : S.ntr;
  Q.ra_cgroup = 1;
  const bool skipping = O.skip_unchanged != 0;
  bool tiles64 = false, lean = false, slab_totals = false;
  if (S.resident) {
    Q.sweep = kResident;
    Q.iters = R.chunk;
    Q.first = sw == 1 && !P.warm;
    Q.profile_kind = 3;
    T.k += R.chunk;
    return Q;  // (the resident kernel does its own vector updates)
  }
  if (P.from_points) {
    Q.sweep = kPoints;
    Q.prev_sums = T.sums_gen == sw - 1 && skipping;
    T.sums_gen = sw;
    // (the reduction adds the eight 32-row tiles of a 256-row strip first, as the screened sweep stores them: the
    // same bits with and without the screening)
    Q.ra_cgroup = kPointsColGroup;
    if (S.points_screen) {
      // full sweeps record the bounds; the screened sweep runs on them while the plan is
      // known to be sparse, until they are due for renewal (after 8, 16, 32, ... sweeps: varphi moves fast at first).
      // Only the last full sweep before a look at the density need record them, every other one is a tenth faster without
      // (12000 x 12000: 285 instead of 320 us)
      const bool due = T.epoch_gen < 0 || sw - T.epoch_gen >= T.refresh_period;
      const bool sparse = T.plan_density >= 0.0 && T.plan_density < kPointsSparse;
      const bool lean_points = !Q.first && !due && Q.prev_sums && sparse;
      if (lean_points) {
        Q.sweep = kPointsLean;
        Q.profile_kind = 8;
        Q.ra_ntr = ceil_div(P.m, kStripRows);
        Q.ra_cgroup = 1;
      } else if (!Q.first && (sparse || c == R.chunk - 1)) {
        Q.refresh = true;
        Q.profile_kind = 9;
        if (T.epoch_gen >= 0 && due && sparse)
          T.refresh_period = T.refresh_period * 2 < S.refresh_max ? T.refresh_period * 2 : S.refresh_max;
        T.epoch_gen = sw;
        if (S.active) T.recorded_gen = sw;
      }
    }
  } else if (P.slab_k) {
    Q.sweep = kSlab;
    // (large problems: the slab totals give eta, one launch then does the whole vector update)
    slab_totals = !S.small && (size_t)S.nstrips * (size_t)P.nruns <= P.tilesum_half;
    if (slab_totals) Q.tilesum = true;
    Q.prev_sums = T.sums_gen == sw - 1 && skipping;
    Q.pro = !T.materialized;
    T.sums_gen = sw;
  } else if (P.reg_kind == kGroupLasso) {
    Q.sweep = kTwoPass;
  } else if (!T.materialized) {
    Q.sweep = kPro32;
    Q.pro = true;
    T.sums_gen = sw;
  } else {
    // even/odd scheme: inside a stretch the sweeps pair up as (store X - rho*C, then read it without
    // C); an odd stretch starts with one plain sweep, so X is plain at every stretch end
    int mode = 0;
    if (R.skip_cost) {
      const int paired_from = R.chunk & 1;
      if (c >= paired_from) mode = ((c - paired_from) & 1) ? 2 : 1;
    }
    Q.mode = mode;
    const bool screened = mode == 0 && R.tall && !Q.first && S.may_screen;
    Q.prev_sums = mode == 0 && T.sums_gen == sw - 1 && skipping;
    T.sums_gen = mode == 1 ? -1 : sw;
    // once the plan is known to be sparse (and bounds exist): one wave per tile
    // (by lines: from the second epoch of bounds on -- sweep 9 of a cold start, with 70 to 80 % of the lines and all of the
    // row segments still nonzero.  At 20000 x 20000 sweeps 9 to 96 took 24 ms in row segments and take 9 by lines)
    const bool sparse = T.plan_density >= 0.0 && T.plan_density < 0.25;
    lean = screened && S.lean_fits && T.epoch_gen >= 0 && Q.prev_sums && T.drift_gen == sw - 1 && (sparse || (S.early_lines && T.by_lines && !T.dense_lines));
    Q.refresh = screened && !lean && (T.epoch_gen < 0 || sw - T.epoch_gen >= T.refresh_period);
    tiles64 = R.tall && !Q.first && mode == 0;
    if (tiles64) Q.tilesum = true;
    Q.profile_kind = screened ? (Q.refresh ? 6 : 5) : tiles64 ? 4 : mode;
    if (screened) {
      if (Q.refresh) {
        // (varphi moves fast at first: the bounds are renewed after 8 sweeps, then 16, 32, ...)
        if (T.epoch_gen >= 0) {
          T.refresh_period = T.refresh_period * 2 < S.refresh_max ? T.refresh_period * 2 : S.refresh_max;
          T.by_lines = true;
        }
        T.epoch_gen = sw;
        if (P.line_bounds) T.lines_gen = sw;  // (it leaves the line flags, too)
      }
      if (lean) {
        Q.sweep = kLean;
        Q.lines_in = T.lines_gen == sw - 1;
        T.lines_gen = sw;
        Q.profile_kind = 7;
      } else {
        Q.sweep = kScreened8;
      }
    } else if (tiles64) {
      Q.sweep = kTall64;
    } else {
      Q.sweep = kPlain32;
    }
    // (the 64-row tiles leave fewer rows of column partials, which the reduction adds up in groups
    // of four; the lean sweep stores one row per group)
    Q.ra_ntr = lean ? ceil_div(S.ntr_tall, kColGroup) : tiles64 ? S.ntr_tall : S.ntr;
    Q.ra_cgroup = (tiles64 && !lean) ? kColGroup : 1;
  }
  T.last_lean = lean;
  // the vector update: separate kernels, one merged launch, or left to the head of the next sweep
  if (!S.fused || c == R.chunk - 1) {
    if (slab_totals) {
      Q.update = kMergedSlab;
      Q.tt_rows = P.nruns;
      Q.tt_group = 1;
    } else if (tiles64) {
      Q.update = kMergedTiles;
      Q.tt_rows = lean ? ceil_div(S.ntr_tall, kColGroup) : S.ntr_tall;
      Q.tt_group = lean ? 1 : kColGroup;
      Q.ctl_mode = lean ? 2 : Q.refresh ? 1 : 0;
      if (P.line_bounds && S.may_screen && T.epoch_gen >= 0) {
        Q.drift = true;
        T.drift_gen = sw;
      }
    } else if (P.from_points) {
      // (the point-cloud sweeps store the totals of their 32-row tiles, the screened one of its strips of eight)
      Q.update = kMergedTiles;
      Q.tilesum = true;
      Q.tt_rows = Q.sweep == kPointsLean ? ceil_div(P.m, kStripRows) : S.ntr;
      Q.tt_group = Q.sweep == kPointsLean ? 1 : kPointsColGroup;
    } else {
      Q.update = kSeparate;
    }
    T.norms_pending = true;
    T.materialized = true;
  } else {
    T.materialized = false;
  }
  T.k += 1;
  return Q;
}

// Checks inside the launch: where the sweeps between two checks are one launch anyway and nothing but the residual test hangs
// on a check, the launch runs on through the checks and tests by itself.  Per check that saves the launch, the last vector
// update, the norms, the status and its copy, and the fetching of X and C: 40 us in grid-resident stretches, 17 in the
// resident kernel, of stretches of 100 sweeps that take 300 and 95.  The host looks at the checks after kRunSweeps sweeps or
// kRunChecks checks.
inline bool runs_through_checks(const Static& S, const Problem& P, const Options& O) {
  return (S.resident || S.grid_tiles > 0 || S.grid_points > 0) && P.feedback && P.checking && !P.single_launches && !S.adaptive && O.gap_every < 1;
}

// Stretch R, which ends at a check or with the call, drawn out over the checks that follow.
inline Stretch draw_out(const Problem& P, const Options& O, const State& T, Stretch R, int sweeps = kRunSweeps) {
  for (int checks = 1; checks < kRunChecks && T.k + R.chunk < P.max_iters; ++checks) {
    const int left = P.max_iters - (T.k + R.chunk), more = O.check_every < left ? O.check_every : left;
    if (R.chunk > sweeps - more) break;
    R.chunk += more;
  }
  return R;
}

// How many sweeps of stretch R are launched one by one before a single grid-resident launch takes the rest, or -1 if
// there is no such launch in it.  (The first sweep of a cold start has its own tiles and vector update where the others
// run on 64-row tiles.)
inline int grid_head(const Static& S, const Problem& P, const State& T, const Stretch& R) {
  if ((!S.grid_tiles && !S.grid_points) || P.single_launches) return -1;
  const bool cold = T.k_base + T.k == 0 && !P.warm;
  const int head = S.grid_tall && cold ? 1 : 0;
  const int least = S.grid_slab_lanes || (!S.grid_tall && S.grid_tiles + S.grid_points == 1) ? kGridMinSweepsOneTile : kGridMinSweeps;
  return R.chunk - head >= least ? head : -1;
}

// Rows (or columns) of the workgroup that has the most: every kActiveSide-th group of 256, the last one of all may be shorter.
inline int active_side_most(int m) {
  const int groups = ceil_div(m, 256), most = ceil_div(groups, kActiveSide), others = (groups - 1) % kActiveSide;
  return others != 0 || most == 1 ? (256 * most < m ? 256 * most : m) : 256 * (most - 1) + m - 256 * (groups - 1);
}

// Entries that the busiest workgroup is expected to hold where so many lines of 32 hold something, each entry by its own chance.
inline double active_expected(const Problem& P, double lines) {
  const double one = lines < 1.0 ? -std::expm1(std::log1p(-lines) / 32.0) : 1.0;
  return one * active_side_most(P.m) * active_side_most(P.n);
}

// Whether a look counts in advance what a list over a stored cost would hold: where such a launch may come next.
inline bool active_forecast(const Static& S, const Problem& P, const State& T) {
  return S.active && !P.single_launches && !P.from_points && P.max_iters - T.k >= kActiveLeast && T.k >= T.active_from && T.materialized &&
         T.by_lines && T.epoch_gen >= 0 && T.sums_gen == T.k_base + T.k && active_bounds(P, T) == kRecordedBounds;
}

inline double active_forecast_limit(int k, double held) {
  return k < kActiveEarly ? kActiveForecastEarly : held <= kActiveThin ? kActiveForecastThin : kActiveForecast;
}

// Whether the next iterations run on the active entries: the plan is known to be thin enough, X in memory is plain, its
// flags and the screening bounds describe it, and the call is not about to end.
inline bool active_next(const Static& S, const Problem& P, const State& T) {
  if (!S.active || P.single_launches || P.max_iters - T.k < kActiveLeast) return false;
  if (T.k < T.active_from && (T.k < T.active_again || T.plan_density > kActiveFallen * T.active_density)) return false;
  const long long now = T.k_base + T.k;
  if (!T.materialized || T.dense_plan || T.sums_gen != now || T.epoch_gen < 0 || T.epoch_gen > now) return false;
  if (active_bounds(P, T) == kNoBounds) return false;
  const double room = kActiveFill * (double)kActiveEntries * (kActiveSide * kActiveSide);
  if (P.from_points) return T.plan_density >= 0.0 && T.plan_density < kActivePoints && T.plan_density * P.m * S.nseg <= room;
  if (!T.by_lines || T.dense_lines || T.lines < 0.0) return false;
  const double held = active_expected(P, T.lines) / kActiveEntries;
  return T.forecast_k == T.k ? held <= 1.0 && T.forecast <= active_forecast_limit(T.k, held) : held <= kActiveExpected;
}

// ... iterations a list of its entries has to last.
inline int active_shortest(const Problem& P, const Static& S) {
  if (!P.from_points) return kActiveShortest;
  return (long long)P.m * S.nseg >= kActivePointsLarge ? kActiveShortestPointsLarge : kActiveShortestPoints;
}

// ... the age of the bounds it starts from, at most.
inline int active_age(const Problem& P, const State& T) {
  const bool left = active_bounds(P, T) == kLeftBounds;
  const long long age = T.k_base + T.k - (left ? T.bound_gen : T.epoch_gen);
  const long long most = !left && T.forecast_k == T.k && T.forecast_age < age ? T.forecast_age : age;
  return most > 0 ? (int)most : 1;
}

// ... the iterations it may take: up to a check or the end of the call, drawn out over the checks that follow.
inline Stretch active_stretch(const Problem& P, const Options& O, const State& T) {
  Stretch R;
  R.chunk = P.max_iters - T.k;
  const int to_check = O.check_every - T.k % O.check_every;
  if (to_check < R.chunk) R.chunk = to_check;
  return draw_out(P, O, T, R, P.from_points ? kRunActivePoints : kRunActive);
}

// ... and it has come back, `iters` iterations later.  left: the entries no longer fit (or never did): the sweeps take over for
// a while, longer every time.
inline void active_done(State& T, const Problem& P, int iters, bool left) {
  T.k += iters;
  T.active_ran = true;
  const long long now = T.k_base + T.k;
  T.sums_gen = now;
  if (!P.from_points && iters > 0) T.lines_gen = now;
  T.bound_gen = now;
  if (iters > 0) {
    T.drift_gen = -1;
    T.norms_pending = false;
    T.last_lean = false;
  }
  if (left) {
    // (early in a point-cloud solve a look may find a thinner plan, and a sweep over everything costs half as much as an attempt;
    // tried again whatever the look has found, 9000 x 9000 in two dimensions spent 2 ms of 48 on three more attempts in vain)
    const int times = T.active_left < 6 ? T.active_left : 6;
    T.active_from = T.k + (512 << times);
    T.active_again = P.from_points && T.k < kPromptLooksUntil ? T.k + (8 << times) : T.active_from;
    T.active_density = T.plan_density;
    // (what the last look found is as old as the launch was long, and the plan has filled up where the entries no longer fit: over point clouds
    // the sweeps that go by certificates, 120 us at 5000 x 4000 where the others take 27, wait for the next look)
    if (P.from_points && iters > 0) T.plan_density = -1.0;
    ++T.active_left;
  }
}

// ... or it has been counted in advance.  Where the entries that hold something would fit by half and those within the slack do not let them, a
// list waits as long as behind a launch that ended early: they lie that close for hundreds of iterations.
inline void on_forecast(State& T, const Problem& P, int k, double entries, int age) {
  T.forecast_k = k;
  T.forecast_age = age;
  T.forecast = entries / kActiveEntries;
  const double held = T.lines >= 0.0 ? active_expected(P, T.lines) / kActiveEntries : 1.0;
  if (k == T.k && !T.dense_lines && T.forecast > active_forecast_limit(k, held) && held <= 0.5 * kActiveForecast) {
    T.active_ran = true;
    T.active_again = T.active_from = T.k + (512 << (T.active_left < 6 ? T.active_left : 6));
    ++T.active_left;
  }
}

// A status has come back: the density of the plan it reports steers the next stretches
// (hysteresis; the early looks never start the pairs: every plan is dense in its first iterations; where the sweep by lines
// waits they end them below 99.5 %, the checks, which see the same number, where they would not start them).  Above 90 % of the row
// segments nonzero: the sweeps that skip what is zero leave out a few percent of the bytes there, the pairs a sixth.
// lines: fraction of the lines of X that hold a nonzero, where the last sweep counted them (else negative).  It is the
// better measure (at 8191 x 8191 with a strong quadratic term 95 % of the row segments but 34 % of the lines are nonzero
// after 100 sweeps: 54 us a sweep by lines, 104 in pairs, 123 in row segments); above 92 % the streaming sweeps are faster (131 us
// against 158 with all lines nonzero).
inline void on_status(const Static& S, State& T, double density, double lines, bool was_probe) {
  if (!S.adaptive) return;
  T.plan_density = density;
  if (lines >= 0.0) T.lines = lines;
  if (lines >= 0.0) T.dense_lines = lines > 0.92 && (T.dense_lines || !was_probe);
  else if (density < 0.995) T.dense_lines = false;  // (independent lines: 0.995 of the row segments are half of the lines)
  const bool dense = lines >= 0.0 ? lines > 0.85 : density > 0.9;
  if (dense && !was_probe) T.dense_plan = S.adaptive_pairs;
  else if (lines >= 0.0 ? lines < 0.5 : density < S.pairs_until) T.dense_plan = false;
}

// What the handle keeps for a continued solve.  iters: what the final status reports (an early stop
// leaves the sweeps queued behind it undone: be conservative about everything they would have left).
inline Carry finish(const Static& S, const Problem& P, const State& T, bool converged, int iters) {
  Carry C;
  const bool epoch_ran = T.epoch_gen <= T.k_base + (long long)iters;
  const bool epoch_kept = !converged && epoch_ran;
  C.dense_plan = T.dense_plan;
  C.plan_density = T.plan_density;
  C.by_lines = T.by_lines;
  C.lines = T.lines;
  C.bound_gen = (converged || T.bound_gen > T.k_base + (long long)iters) ? -1 : T.bound_gen;
  C.recorded_gen = (converged || T.recorded_gen > T.k_base + (long long)iters) ? -1 : T.recorded_gen;
  C.drift_valid = !converged && epoch_kept && P.max_iters > 0 && T.drift_gen == T.k_base + T.k;
  C.epoch_gen = (converged || !epoch_ran) ? -1 : T.epoch_gen;
  C.refresh_period = (converged || !epoch_ran) ? kFirstRefreshPeriod : T.refresh_period;
  C.bounds_from_points = P.from_points;
  C.bounds_rho = P.rho;
  C.sums_valid = !converged && P.max_iters > 0 && T.sums_gen == T.k_base + T.k;
  C.lines_valid = C.sums_valid && T.lines_gen == T.k_base + T.k;
  C.sums_strip = S.sums_strip;
  C.iters_done = T.k_base + (P.max_iters == 0 ? 0 : iters);
  return C;
}

// Which pass evaluates the terms of the duality gap for the state after the sweeps enqueued so far.  The
// lean pass visits only the row segments a screening bound does not certify to contribute nothing; it
// needs the bounds of an epoch and flags that describe the X in memory: the line flags of a lean sweep,
// or the row-segment sums of any sweep that leaves them per 256 columns.  (After a stop raised on the
// device the sweeps enqueued behind it did not run and the host's record of the flags is ahead of the
// memory: the caller falls back to the dense pass then.)
enum GapPass { kGapDense = 0, kGapLeanLines, kGapLeanSums };

inline GapPass gap_pass(const Static& S, const Problem& P, const State& T) {
  const long long cur = T.k_base + T.k;
  if (!S.may_screen || P.from_points || P.reg_kind == kGroupLasso || P.slab_k) return kGapDense;
  if (T.epoch_gen < 0 || T.epoch_gen > cur || cur < 1) return kGapDense;
  if (T.lines_gen == cur) return kGapLeanLines;
  if (T.sums_gen == cur) return kGapLeanSums;
  return kGapDense;
}

// Group lasso: the labels of the m rows as runs of equal labels.  The slab kernel applies when every
// class is one run of at most kSlabMaxRows rows (and the runs fit the workspace); where a class lies in
// several runs, on the classes themselves, their rows fetched through a table.
struct LabelRuns {
  bool valid = true;              // every label in [0, num_classes)
  std::vector<int> start, len;    // the runs; with a table the non-empty classes: len their rows, start not used
  int slab_k = 0;                 // rows per lane of the slab kernel, 0: two-pass path
  std::vector<int> rows;          // empty, or [classes][kSlabRowLanes * slab_k] the rows of every class, ascending, then -1
};

// Two-pass path (any labels): the rows of every class, in ascending order, cut into chunks of at most
// kNormChunkRows rows.  The first pass adds up the squared entries of one chunk per wave, the second
// adds the chunks of a class in order: the group norms come out the same in every run (no atomics).
constexpr int kNormChunkRows = 16;
struct ClassChunks {
  std::vector<int> perm;          // [m] the rows sorted by (class, row)
  std::vector<int> chunk_start;   // [nchunks + 1] offsets into perm
  std::vector<int> class_first;   // [num_classes + 1] the chunks of class c are class_first[c] .. class_first[c+1] - 1
  int nchunks() const { return (int)chunk_start.size() - 1; }
};

inline ClassChunks chunk_classes(const int* labels, int m, int num_classes) {
  ClassChunks K;
  std::vector<int> count((size_t)num_classes + 1, 0);
  for (int i = 0; i < m; ++i) ++count[(size_t)labels[i] + 1];
  for (int c = 0; c < num_classes; ++c) count[(size_t)c + 1] += count[(size_t)c];  // first position of every class
  K.perm.resize((size_t)m);
  std::vector<int> next(count.begin(), count.end() - 1);
  for (int i = 0; i < m; ++i) K.perm[(size_t)next[(size_t)labels[i]]++] = i;       // stable: rows stay in order
  K.class_first.push_back(0);
  K.chunk_start.push_back(0);
  for (int c = 0; c < num_classes; ++c) {
    for (int b = count[(size_t)c]; b < count[(size_t)c + 1]; b += kNormChunkRows) {
      const int e = b + kNormChunkRows < count[(size_t)c + 1] ? b + kNormChunkRows : count[(size_t)c + 1];
      K.chunk_start.push_back(e);
    }
    K.class_first.push_back(K.nchunks());
  }
  return K;
}

inline LabelRuns analyze_labels(const int* labels, int m, int num_classes, int max_runs, bool force_two_pass) {
  LabelRuns L;
  std::vector<char> seen((size_t)num_classes, 0);
  bool one_run_per_class = true;
  int maxlen = 0;
  for (int i = 0; i < m;) {
    const int c = labels[i];
    if (c < 0 || c >= num_classes) {
      L.valid = false;
      return L;
    }
    int e = i + 1;
    while (e < m && labels[e] == c) ++e;
    if (seen[(size_t)c]) one_run_per_class = false;
    seen[(size_t)c] = 1;
    L.start.push_back(i);
    L.len.push_back(e - i);
    if (e - i > maxlen) maxlen = e - i;
    i = e;
  }
  if (!force_two_pass && one_run_per_class && maxlen <= kSlabMaxRows && (int)L.start.size() <= max_runs) {
    L.slab_k = 1;
    while (kSlabRowLanes * L.slab_k < maxlen) L.slab_k *= 2;
  } else if (!force_two_pass && !one_run_per_class) {
    std::vector<int> count((size_t)num_classes, 0);
    for (int i = 0; i < m; ++i) ++count[(size_t)labels[i]];
    int classes = 0, most = 0;
    for (const int c : count) {
      classes += c > 0;
      if (c > most) most = c;
    }
    int k = 1;
    while (kSlabRowLanes * k < most) k *= 2;
    if (most <= kSlabMaxRows && classes <= max_runs && (double)m >= kMappedFill * kSlabRowLanes * k * (double)classes) {
      L.slab_k = k;
      L.start.assign((size_t)classes, 0);
      L.len.clear();
      L.rows.assign((size_t)classes * (size_t)(kSlabRowLanes * k), -1);
      std::vector<size_t> next((size_t)num_classes, 0);
      for (size_t c = 0; c < count.size(); ++c) {
        if (count[c] == 0) continue;
        next[c] = L.len.size() * (size_t)(kSlabRowLanes * k);
        L.len.push_back(count[c]);
      }
      for (int i = 0; i < m; ++i) L.rows[next[(size_t)labels[i]]++] = i;
    }
  }
  return L;
}

}  // namespace drot_plan
#endif  // DROT_PLAN_H_
