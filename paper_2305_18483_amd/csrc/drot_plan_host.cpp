// Host-only wrapper of the launch planner (drot_plan.h) and of the screening certificates (drot_bounds.h) for tests that
// run without a GPU.
//
// drot_plan_trace() replays the host loop of a solve -- stretches, sweeps, statuses read one stretch
// late -- with the densities and the stop a test scripts in place of what a GPU would report, and
// writes down what the planner decided for every sweep.  Built with a plain C++ compiler into
// libdrot_plan.so; the product library includes the same header and does not use this file.
#include <cmath>
#include <cstring>

#include "drot_plan.h"

#define DROT_FN inline
#include "drot_bounds.h"

using namespace drot_plan;

extern "C" {

// problem[16]: m, n, reg_kind, from_points, warm, resume, has_weights, c_on_lines, x_on_lines, slab_k,
//              nruns, feedback, checking, max_iters, line_bounds, rho * 1e9
// options[9]:  check_every, resident, fused_update, skip_cost, skip_unchanged, screening, nontemporal,
//              force_two_pass, gap_every
// carry[12] (in and out): dense_plan, plan_density * 1e6, epoch_gen, refresh_period, sums_valid, sums_strip,
//              lines_valid, iters_done, by_lines, drift_valid, bounds_from_points, bounds_rho * 1e9
// densities[nstatus]: what the k-th status of the call reports (fraction of nonzero row segments), lines[nstatus] (or null)
//              the fraction of nonzero lines, reported where the last sweep was a lean one; statuses past the end repeat the
//              last one.  stop_at_status >= 0: that status reports convergence.
// rows [capacity][12]: sweep, mode, first, prev_sums, lines_in, refresh, pro, tilesum, update, ra_ntr * 16 + ra_cgroup,
//              profile_kind, flags (1: last sweep of a stretch, 2: that stretch is a probe, 4: its status carries the gap,
//              8: a gap evaluated there may take the lean pass, 16: with the lean sweep's line flags)
// statics[10]: nseg, ntr, resident, pad_c, pad_x, small, fused, may_screen, adaptive, nt
// Returns the number of sweeps (launches) planned, or -1 if capacity was too small.
int drot_plan_trace(const int* problem, const int* options, long long* carry, const double* densities,
                    const double* lines, int nstatus, int stop_at_status, int* rows, int capacity, int* statics, int* iters_done) {
  Problem P;
  P.m = problem[0];
  P.n = problem[1];
  P.reg_kind = problem[2];
  P.from_points = problem[3] != 0;
  P.warm = problem[4] != 0;
  P.resume = problem[5] != 0;
  P.has_weights = problem[6] != 0;
  P.c_on_lines = problem[7] != 0;
  P.x_on_lines = problem[8] != 0;
  P.slab_k = problem[9];
  P.nruns = problem[10];
  P.feedback = problem[11] != 0;
  P.checking = problem[12] != 0;
  P.max_iters = problem[13];
  P.line_bounds = problem[14] != 0;
  P.rho = (float)problem[15] * 1e-9f;
  P.tilesum_half = (size_t)ceil_div(P.n, kSegCols) * (size_t)ceil_div(P.m, kTileRows);
  if (P.tilesum_half < 4096) P.tilesum_half = 4096;
  Options O;
  O.check_every = options[0];
  O.resident = options[1];
  O.fused_update = options[2];
  O.skip_cost = options[3];
  O.skip_unchanged = options[4];
  O.screening = options[5];
  O.nontemporal = options[6];
  O.force_two_pass = options[7];
  O.gap_every = options[8];
  Carry C;
  C.dense_plan = carry[0] != 0;
  C.plan_density = (double)carry[1] * 1e-6;
  C.epoch_gen = carry[2];
  C.refresh_period = (int)carry[3];
  C.sums_valid = carry[4] != 0;
  C.sums_strip = (int)carry[5];
  C.lines_valid = carry[6] != 0;
  C.iters_done = carry[7];
  C.by_lines = carry[8] != 0;
  C.drift_valid = carry[9] != 0;
  C.bounds_from_points = carry[10] != 0;
  C.bounds_rho = (float)carry[11] * 1e-9f;


  const Static S = make_static(P, O);
  statics[0] = S.nseg;
  statics[1] = S.ntr;
  statics[2] = S.resident;
  statics[3] = S.pad_c;
  statics[4] = S.pad_x;
  statics[5] = S.small;
  statics[6] = S.fused;
  statics[7] = S.may_screen;
  statics[8] = S.adaptive;
  statics[9] = S.nt;
  State T = start_state(S, P, C);
  int nrows = 0, checks = 0;
  bool converged = false;
  bool was_probe[2] = {false, false}, was_lean[2] = {false, false};
  int slot = 0, stop_iters = -1;
  while (T.k < P.max_iters && !converged) {
    const Stretch R = next_stretch(S, P, O, T);
    const int k_end = T.k + R.chunk;
    for (int c = 0; T.k < k_end; ++c) {
      const Step Q = next_sweep(S, P, O, T, R, c);
      if (nrows >= capacity) return -1;
      int* r = rows + (size_t)nrows * 12;
      r[0] = Q.sweep;
      r[1] = Q.mode;
      r[2] = Q.first;
      r[3] = Q.prev_sums;
      r[4] = Q.lines_in;
      r[5] = Q.refresh;
      r[6] = Q.pro;
      r[7] = Q.tilesum;
      r[8] = Q.update;
      r[9] = Q.ra_ntr * 16 + Q.ra_cgroup;
      r[10] = Q.profile_kind;
      const GapPass G = T.k == k_end ? gap_pass(S, P, T) : kGapDense;
      r[11] = (T.k == k_end ? 1 : 0) | (T.k == k_end && R.probe ? 2 : 0) | (T.k == k_end && R.gap ? 4 : 0) |
              (G != kGapDense ? 8 : 0) | (G == kGapLeanLines ? 16 : 0);
      ++nrows;
    }
    if (S.status_at_checks) {
      was_probe[slot] = R.probe;
      was_lean[slot] = T.last_lean;
      if (checks == stop_at_status && stop_iters < 0) stop_iters = T.k;  // (the device raises its stop flag here)
      auto read_status = [&](int which, int slot_of) {
        if (stop_at_status >= 0 && which >= stop_at_status) converged = true;
        const int e = which < nstatus ? which : nstatus - 1;
        on_status(S, T, nstatus > 0 ? densities[e] : 0.0, nstatus > 0 && lines && was_lean[slot_of] ? lines[e] : -1.0,
                  was_probe[slot_of]);
      };
      // the host reads the previous stretch's status while this one is queued, and where it waits for it this one's too
      if (checks > 0 && P.feedback) read_status(checks - 1, slot ^ 1);
      if (P.feedback && R.prompt) read_status(checks, slot);
      slot ^= 1;
      ++checks;
    }
  }
  const bool stopped = stop_iters >= 0;
  const int reported = stopped ? stop_iters : T.k;
  const Carry F = finish(S, P, T, stopped, reported);
  carry[0] = F.dense_plan;
  carry[1] = (long long)(F.plan_density * 1e6);
  carry[2] = F.epoch_gen;
  carry[3] = F.refresh_period;
  carry[4] = F.sums_valid;
  carry[5] = F.sums_strip;
  carry[6] = F.lines_valid;
  carry[7] = F.iters_done;
  carry[8] = F.by_lines;
  carry[9] = F.drift_valid;
  carry[10] = F.bounds_from_points;
  carry[11] = (long long)(F.bounds_rho * 1e9 + 0.5);
  *iters_done = reported;
  return nrows;
}

// The lean sweep's certificates for `count` row segments resp. lines.  lines: below is encoded and decoded with rho first.
void drot_certify_segments(int count, const float* m1, const float* m2, const float* drift1, const float* drift, const float* mag,
                           const float* phi, unsigned char* out) {
  for (int k = 0; k < count; ++k) out[k] = certified_segment(m1[k], m2[k], drift1[k], drift[k], mag[k], phi[k]);
}
void drot_certify_lines(int count, float rho, const float* m1, const float* below, const float* drift, const float* mag,
                        const float* phi, unsigned char* out) {
  const int base = line_code_base(rho);
  for (int k = 0; k < count; ++k)
    out[k] = certified_line(m1[k], line_decode(line_code(below[k], base), base), drift[k], mag[k], phi[k]);
}

// Which of `count` zero entries, and lines of entries, a list of active entries would hold; the rises it is checked with.
void drot_active_entries(int count, const float* t, const float* varphi, const float* phi, const float* tau, unsigned char* out) {
  for (int k = 0; k < count; ++k) out[k] = active_entry(t[k], varphi[k], phi[k], tau[k]);
}
void drot_active_lines(int count, const float* bound, const float* rise, const float* mag, const float* phi, const float* tau, unsigned char* out) {
  for (int k = 0; k < count; ++k) out[k] = active_line(bound[k], rise[k], mag[k], phi[k], tau[k]);
}
void drot_active_rises(int count, const float* now, const float* from, const float* other, float* rise, float* both) {
  for (int k = 0; k < count; ++k) both[k] = active_rises(rise[k] = active_rise(now[k], from[k]), other[k]);
}

// The renewals of `count` lean sweeps, waste[k] the lines the k-th reads in vain unless it renews the bounds: renewed[k].
void drot_renewals(int count, const int* waste, int price, int max_since, unsigned char* renewed) {
  Renewal R{0, 0, 0};
  for (int k = 0; k < count; ++k) {
    renewed[k] = R.renew != 0;
    R = after_lean_sweep(R, waste[k], price, max_since);
  }
}

// Active entries: problem, options as in drot_plan_trace.  state[9]: iterations of the call so far, density and lines reported
// * 1e6 (negative: none), by_lines, generation of the bounds (negative: none), launches that ended early, iterations since the
// last of them, the density it started from * 1e6, entries counted in advance at this look * 1e6 (of kActiveEntries; negative: not
// counted).  out[8]: iterations of a launch now (0: none), and if it ends early after 10: before which
// iteration of the call no other starts, launches that ended early, the density that is known then * 1e6 (negative: none), whether the host
// waits for the next look; iterations that a list has to last; whether a look here counts in advance, and what the plan alone has * 1e6.  Returns whether the call could ever take one.
int drot_plan_active(const int* problem, const int* options, int compute_units, int single_launches, const int* state, int* out) {
  Problem P;
  P.m = problem[0];
  P.n = problem[1];
  P.reg_kind = problem[2];
  P.from_points = problem[3] != 0;
  P.feedback = problem[11] != 0;
  P.checking = problem[12] != 0;
  P.max_iters = problem[13];
  P.line_bounds = true;
  P.compute_units = compute_units;
  P.single_launches = single_launches != 0;
  Options O;
  O.check_every = options[0];
  O.fused_update = options[2];
  O.skip_cost = options[3];
  O.skip_unchanged = options[4];
  O.screening = options[5];
  O.gap_every = options[8];
  const Static S = make_static(P, O);
  State T = start_state(S, P, Carry{});
  T.k = state[0];
  T.sums_gen = state[0];
  T.plan_density = state[1] * 1e-6;
  T.lines = state[2] * 1e-6;
  T.by_lines = state[3] != 0;
  T.epoch_gen = T.recorded_gen = state[4];
  T.active_left = state[5];
  T.active_density = state[7] * 1e-6;
  if (state[5]) {
    T.active_from = state[0] - state[6] + (512 << (state[5] - 1));
    T.active_again = P.from_points && state[0] - state[6] < kPromptLooksUntil ? state[0] - state[6] + (8 << (state[5] - 1)) : T.active_from;
  }
  out[6] = active_forecast(S, P, T);
  out[7] = (int)(active_expected(P, T.lines) / kActiveEntries * 1e6 + 0.5);
  if (state[8] >= 0) on_forecast(T, P, T.k, state[8] * 1e-6 * kActiveEntries, state[0] - state[4]);
  out[0] = active_next(S, P, T) ? active_stretch(P, O, T).chunk : 0;
  if (T.active_left == state[5]) active_done(T, P, 10, true);  // (else it waits as if it had ended)
  out[1] = T.active_again;
  out[2] = T.active_left;
  out[3] = T.plan_density < 0.0 ? -1 : (int)(T.plan_density * 1e6 + 0.5);
  out[4] = next_stretch(S, P, O, T).prompt;
  out[5] = active_shortest(P, S);
  return S.active;
}

// Continued calls of one handle (problem as in drot_plan_trace; options[ncalls][9], iters[ncalls]), every status of which reports
// density and lines (* 1e6), every launch of active entries lasting to its end.  events[capacity][4]: 0, sweep, whether bounds by line
// were recorded, 0: a sweep that started an epoch; 1, iterations before it, iterations after it, where its bounds come from
// (ActiveBounds): a launch of active entries.  Returns the number of events, or -1 if capacity was too small.
int drot_plan_active_calls(const int* problem, int ncalls, const int* options, const int* iters, int compute_units, int density, int lines,
                           long long* events, int capacity) {
  Carry C;
  int count = 0;
  auto event = [&](long long a, long long b, long long c, long long d) {
    if (count < capacity) {
      events[4 * count] = a;
      events[4 * count + 1] = b;
      events[4 * count + 2] = c;
      events[4 * count + 3] = d;
    }
    ++count;
  };
  for (int call = 0; call < ncalls; ++call) {
    Problem P;
    P.m = problem[0];
    P.n = problem[1];
    P.reg_kind = problem[2];
    P.from_points = problem[3] != 0;
    P.resume = call > 0;
    P.feedback = true;
    P.checking = problem[12] != 0;
    P.line_bounds = true;
    P.compute_units = compute_units;
    P.max_iters = iters[call];
    P.rho = 1e-3f;
    P.tilesum_half = (size_t)ceil_div(P.n, kSegCols) * (size_t)ceil_div(P.m, kTileRows);
    const int* o = options + 9 * call;
    Options O;
    O.check_every = o[0];
    O.fused_update = o[2];
    O.skip_cost = o[3];
    O.skip_unchanged = o[4];
    O.screening = o[5];
    O.gap_every = o[8];
    const Static S = make_static(P, O);
    State T = start_state(S, P, C);
    while (T.k < P.max_iters) {
      if (active_next(S, P, T)) {
        const long long before = T.k_base + T.k;
        const ActiveBounds from = active_bounds(P, T);
        active_done(T, P, active_stretch(P, O, T).chunk, false);
        event(1, before, T.k_base + T.k, from);
        continue;
      }
      const Stretch R = next_stretch(S, P, O, T);
      for (int c = 0, end = T.k + R.chunk; T.k < end; ++c) {
        const Step Q = next_sweep(S, P, O, T, R, c);
        if (Q.refresh) event(0, Q.sw, P.from_points ? (S.active ? 1 : 0) : 1, 0);
      }
      if (S.status_at_checks) on_status(S, T, density * 1e-6, T.last_lean ? lines * 1e-6 : -1.0, R.probe);
    }
    C = finish(S, P, T, false, P.max_iters);
  }
  return count <= capacity ? count : -1;
}

// Grid-resident stretches: problem, options as in drot_plan_trace.  out[4]: tiles per workgroup (0: none), rows per tile,
// sweeps launched one by one at the head of the first stretch (-1: all of them), automatic even/odd pairs.
void drot_plan_grid(const int* problem, const int* options, int compute_units, int single_launches, int* out) {
  Problem P;
  P.m = problem[0];
  P.n = problem[1];
  P.reg_kind = problem[2];
  P.from_points = problem[3] != 0;
  P.warm = problem[4] != 0;
  P.slab_k = problem[9];
  P.nruns = problem[10];
  P.tilesum_half = (size_t)ceil_div(P.n, kSegCols) * (size_t)ceil_div(P.m, kTileRows);
  P.feedback = problem[11] != 0;
  P.checking = problem[12] != 0;
  P.max_iters = problem[13];
  P.compute_units = compute_units;
  P.single_launches = single_launches != 0;
  Options O;
  O.check_every = options[0];
  O.resident = options[1];
  O.fused_update = options[2];
  O.skip_cost = options[3];
  O.skip_unchanged = options[4];
  O.screening = options[5];
  const Static S = make_static(P, O);
  const State T = start_state(S, P, Carry{});
  out[0] = S.grid_tiles;
  out[1] = S.grid_tall ? kTallTileRows : kTileRows;
  out[2] = grid_head(S, P, T, next_stretch(S, P, O, T));
  out[3] = S.adaptive_pairs;
}

// Grid-resident slabs of a group-lasso problem.  out[4]: slabs per workgroup (0: none), lanes along the columns, rows per
// thread, workgroups.
void drot_plan_slabs(int m, int n, int slab_k, int nruns, int mapped, int fused_update, int compute_units, int* out) {
  Problem P;
  P.m = m;
  P.n = n;
  P.reg_kind = kGroupLasso;
  P.slab_k = slab_k;
  P.nruns = nruns;
  P.mapped_rows = mapped != 0;
  P.tilesum_half = 4096;
  P.compute_units = compute_units;
  Options O;
  O.fused_update = fused_update;
  const Static S = make_static(P, O);
  out[0] = S.grid_tiles;
  out[1] = S.grid_slab_lanes;
  out[2] = S.grid_slab_k;
  out[3] = S.grid_wgs;
}

// Launches that make the residual checks themselves: the sweeps of the first one of a call that has done k iterations (0: it
// makes none), problem and options as in drot_plan_trace.
int drot_plan_run(const int* problem, const int* options, int compute_units, int single_launches, int k) {
  Problem P;
  P.m = problem[0];
  P.n = problem[1];
  P.reg_kind = problem[2];
  P.from_points = problem[3] != 0;
  P.feedback = problem[11] != 0;
  P.checking = problem[12] != 0;
  P.max_iters = problem[13];
  P.compute_units = compute_units;
  P.single_launches = single_launches != 0;
  Options O;
  O.check_every = options[0];
  O.resident = options[1];
  O.fused_update = options[2];
  O.skip_unchanged = options[4];
  O.screening = options[5];
  O.gap_every = options[8];
  const Static S = make_static(P, O);
  if (!runs_through_checks(S, P, O)) return 0;
  State T = start_state(S, P, Carry{});
  T.k = k;
  return draw_out(P, O, T, next_stretch(S, P, O, T)).chunk;
}

// Sweeps of the next stretch of a call that has done k iterations: problem and options as in drot_plan_trace.
int drot_plan_stretch(const int* problem, const int* options, int compute_units, int k) {
  Problem P;
  P.m = problem[0];
  P.n = problem[1];
  P.reg_kind = problem[2];
  P.from_points = problem[3] != 0;
  P.slab_k = problem[9];
  P.nruns = problem[10];
  P.tilesum_half = 4096;
  P.checking = problem[12] != 0;
  P.max_iters = problem[13];
  P.compute_units = compute_units;
  Options O;
  O.check_every = options[0];
  O.fused_update = options[2];
  const Static S = make_static(P, O);
  State T = start_state(S, P, Carry{});
  T.k = k;
  return next_stretch(S, P, O, T).chunk;
}

// Label analysis of the group-lasso path: returns slab_k (0: two-pass), -1 for a label out of range;
// *nruns receives the number of runs.
int drot_plan_labels(const int* labels, int m, int num_classes, int max_runs, int force_two_pass, int* nruns) {
  const LabelRuns L = analyze_labels(labels, m, num_classes, max_runs, force_two_pass != 0);
  if (!L.valid) return -1;
  *nruns = (int)L.start.size();
  return L.slab_k;
}

// The same for classes that are not runs: the table of their rows, [classes][128 slab_k] (capacity cap).  Returns its
// length, 0 where there is none.
int drot_plan_label_rows(const int* labels, int m, int num_classes, int max_runs, int* rows, int cap) {
  const LabelRuns L = analyze_labels(labels, m, num_classes, max_runs, false);
  if ((int)L.rows.size() > cap) return -1;
  if (!L.rows.empty()) std::memcpy(rows, L.rows.data(), sizeof(int) * L.rows.size());
  return (int)L.rows.size();
}

// The chunk tables of the two-pass group-lasso path: perm[m], chunk_start[nchunks + 1] (capacity
// cap_chunks + 1), class_first[num_classes + 1].  Returns the number of chunks, or -1 if they do not fit.
int drot_plan_chunks(const int* labels, int m, int num_classes, int* perm, int* chunk_start, int cap_chunks,
                     int* class_first) {
  const ClassChunks K = chunk_classes(labels, m, num_classes);
  if (K.nchunks() > cap_chunks) return -1;
  std::memcpy(perm, K.perm.data(), sizeof(int) * (size_t)m);
  std::memcpy(chunk_start, K.chunk_start.data(), sizeof(int) * K.chunk_start.size());
  std::memcpy(class_first, K.class_first.data(), sizeof(int) * K.class_first.size());
  return K.nchunks();
}

}  // extern "C"
