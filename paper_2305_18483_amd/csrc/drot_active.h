// Active entries on the chip: many iterations of a large sparse problem in one cooperative launch.
// Part of drot.hip (included there, inside its anonymous namespace, in this order); not a stand-alone header.

// ------------------------------------------------------------------------------------------
// Once the plan of a large problem has thinned out, nearly all of its entries stay zero for dozens of iterations: of
// 20000 x 20000 some 30000 hold something, and few others come to.  The screened sweeps read little more than those, but
// pay two launches, the bounds and the sums of every row segment in every iteration (18 to 45 us).  Here the entries that
// hold something or may come to, the active ones, are listed, and X and C of those alone stay on the chip (the LDS and the
// registers of 256 workgroups, one per compute unit, 4096 entries each); an iteration is their arithmetic (2 to 4 us) and the
// two hops of the exchange (drot_grid.h), and moves no matrix.
//
// Which entries.  With t_ij = varphi_j - rho C_ij at the time of listing, an entry that is zero and has t_ij + phi_i + tau
// < 0 stays zero as long as phi_i and varphi_j together have risen by less than the slack tau.  A workgroup checks that
// for all of its rows and columns whenever it has new phi and varphi, before it sweeps with them, and lists anew where it
// does not hold: so no entry is ever missed, and the iterates are those of the sweeps over everything, bit for bit.
// Listing anew is cheapest for everybody at once (everybody waits for whoever does): a workgroup that will need it soon
// says so with its sums, and one workgroup, the keeper, has all of them do it behind that iteration.
//
// How they are found.  Per 128-byte line of C (32 columns of a row) a bound is kept in memory, no smaller than the largest t_ij of
// the line: exact when the line was last looked at, and then raised by how far varphi has moved since, which is kept per
// line of columns (the largest rise of its 32, added up from listing to listing).  Listing reads the bounds (32 bytes for
// a row segment), fetches the lines whose bound says so, lists their entries one by one and makes their bounds exact again:
// a line is looked at again only when the drift has used up its distance.  No pass over all of C renews them.
//
// Who holds what.  Workgroup (a, b) of 16 x 16 holds the groups of 256 rows a, a + 16, ... and the segments of 256 columns
// b, b + 16, ...  The reductions add up a row's partial sums in 16 interleaved shares, share c the segments c, c + 16, ...,
// and a column's the same way over groups of 256 rows: so what a workgroup has of a row or column is one whole share, added up in
// its order in fp64, and what is exchanged is 16 shares per row and column, whatever the size.
//
// Orders of addition, those of the sweeps: a row segment's entries in the binary tree of wave_sum over the column number; a
// column's entries within 256 rows by groups of 8 rows, tiles of 64 and their four tiles (point clouds: pairs, tiles of 32, eight
// tiles), each in order.  Zeros drop out of all of these, and where two entries at most are not zero any order is the same.
//
// What bounds it, per iteration of 10000 x 10000, by the clock of one workgroup (profiles): the sweep and its sums 1.9 to 2.7 us (chains of lane
// exchanges; 6 where 3000 entries are held), hop 1 2.4 to 2.8 (of the keeper, with its sum of the totals, 5.1), hop 2 1.3 to 3.0, the rest
// 1.3, and the lists, 25 to 38 us each in one workgroup, one in 22 iterations: 10.8 us in all (20000 x 20000 13, point clouds of 12000 12).
// In place of sweeps launched one by one: 10000 x 10000 (1000 iterations) 20.1 -> 13.6 ms; 20000 x 20000 (500) 24.4 -> 18.7; point clouds of 12000
// (500, d = 32) 30.3 -> 12.9, of 4001 x 3999 (400, d = 8) 28.2 -> 4.6.
// Waiting: a workgroup that polls without a rest can keep another's write from being seen for as long as it polls, so polls that
// have failed 32 times rest in between (kGridRest).
// ------------------------------------------------------------------------------------------
constexpr int kActSide = 16;                   // workgroups along the rows, and along the columns
constexpr int kActWgs = kActSide * kActSide;
constexpr int kActWaves = 16, kActThreads = 64 * kActWaves;
constexpr int kActLocal = 5;                   // groups of 256 rows, segments of 256 columns of a workgroup at most
constexpr int kActRows = 256 * kActLocal;
constexpr int kActSlots = 4, kActEntries = kActSlots * kActThreads;
constexpr int kActTasks = 3;                   // a wave's shares of 64 rows or 64 columns: 2 * 4 * kActLocal over 16 waves
constexpr int kActOwned = 2;                   // blocks of eight rows or columns per owner wave
constexpr int kActLines = 8192;                // lines of C a workgroup looks at while listing
constexpr int kActPause = 2;
constexpr int kActShortest = 16;               // iterations a list over a stored cost has to last (point clouds: ActiveArgs)
static_assert(kActEntries == 64 * 64 && kActLocal <= 5, "packed places; the units of a row");
constexpr int kActTotals = 32;                 // words of a workgroup for its totals
constexpr int kActSquares = 16;                // ... of an owned block for its squared residuals
static_assert(kActLocal * kActLocal < kActTotals, "the last word is the workgroup's request");
static_assert(2 * 4 * kActLocal <= kActTasks * kActWaves, "tasks");

enum { kActDone = 0, kActLeave = 1, kActAbort = 2 };
struct ActiveRecord {
  int iters;    // iterations done
  int why;      // kActDone: all, or a check passed; kActLeave: a list would not have lasted; kActAbort: the entries do not fit
  int lists;    // times listed
};

struct ActiveArgs {
  SweepArgs S;            // X, C, phi, varphi, rowpart: read at the start, left up to date at the end
  PointArgs points;       // where the cost is formed from point clouds
  const float* p;
  const float* q;
  double* a_in;           // eq. (6) state before the first update, and the other halves (as in GridArgs)
  double* b_in;
  double* a_alt;
  double* b_alt;
  double* theta_in;
  double* theta_alt;
  const double* sum_p;
  DeviceStatus* status;
  int* done;
  ActiveRecord* record;
  // the exchange buffer, two halves of half_words words: [row blocks, then column blocks][16 shares][8] shares, then from
  // these words on [row blocks, then column blocks][8] a - 2r and b - 2s, [workgroups][32] totals of its 256 x 256
  // pieces and, last, what it asks for, squared residuals [blocks][16], two words each, [kGridCopies][32]: 2 eta - theta, what to do
  // next, whether a check passes.  All zero at the start.
  u64* xchg;
  unsigned half_words, ent_word, tot_word, sq_word, cst_word;
  int nseg, ngroups;      // segments of 256 columns, groups of 256 rows
  int nblk_m, nblk_n;     // blocks of eight rows, of eight columns
  int iters;              // iterations to run at most (>= 1)
  unsigned tag0;
  int polls;
  CheckArgs check;
  float* phi_out;
  float* varphi_out;
  double* r;
  double* s;
  float* bound;           // [nseg][mp][8] bounds by line, against the varphi of `since`; left against bound_varphi, varphi at the end
  const float* since;
  float* bound_varphi;
  const float* m1;        // non-null: the bounds are those a sweep recorded (ScreenArgs), and `since` is its varphi
  const uint2* codes;
  unsigned char* lines;   // line flags of X, or null: none are kept
  int lines_known;        // they hold; else the row-segment sums do
  int age;                // iterations since `since`, at most
  float tau0;             // slack where nothing is known about how fast phi and varphi rise
  int target;             // iterations a list is meant to last
  float shortest;         // ... and has to, to be worth making (point clouds; over a stored cost the same everywhere)
};

// How the 64 entries of a wave's lanes, sorted, are added up.  Made when the entries are listed, good for as long as the list.
// Rows: in rounds, a lane adding the value `off` lanes up in each (0: it does not); what is added in round r, at least one
// entry and at most 2^r, lies no further up than that.  Columns: chains, over the lanes marked as the first of a group, of a tile, of a unit.
struct ActiveTree {
  unsigned offs;       // rows: the offsets, kActOffset bits
  unsigned units;      // six bits a round: of the units of a row or column (fp64), in order; bit 27: no entry here, 28: first of a
                       // group of rows, 29: of a tile, 30: of a unit, 31: of a row or column
  int rounds;          // the wave's most: rows: rounds; columns: of the groups' chains | tiles' << 4 | units' << 9; of `units` << 16
  bool fits;
};
__device__ __forceinline__ int active_offset_at(int r) { return r < 6 ? (r * (r + 1)) >> 1 : 6 * r - 15; }
__device__ __forceinline__ unsigned active_offset_mask(int r) { return r < 5 ? (2u << r) - 1u : r == 7 ? 31u : 63u; }
// One pass over the sums that are left (live, one lane each): a sum and the next one join where `same` says they belong together.
// CHAIN: only the first of those that belong together takes in its next one.  False: there was none.
template <bool CHAIN, typename Same, typename Join>
__device__ __forceinline__ bool active_pass(unsigned id, int lane, unsigned long long& live, Same same, Join join) {
  const unsigned long long below = (1ull << lane) - 1ull, at = 1ull << lane;
  const bool alive = (live & at) != 0;
  const unsigned long long after = live & ~(below | at), before = live & below;
  const int nx = after ? (int)__builtin_ctzll(after) : lane, pv = before ? 63 - (int)__builtin_clzll(before) : lane;
  const unsigned idn = (unsigned)__shfl((int)id, nx, 64), idp = (unsigned)__shfl((int)id, pv, 64);
  const bool can = alive && nx != lane && same(idn) && !(CHAIN && pv != lane && same(idp));
  const unsigned long long joins = __builtin_amdgcn_ballot_w64(can);
  join(can, nx);
  live &= ~__builtin_amdgcn_ballot_w64(alive && pv != lane && ((joins >> pv) & 1ull) != 0);
  return joins != 0;
}
// The most over the wave's lanes.
__device__ __forceinline__ int active_most(int v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = max(v, __shfl_xor(v, off, 64));
  return __builtin_amdgcn_readfirstlane(v);
}
// The lanes behind this one (32 at most), up to the next of `upper`, that are in `members`; none for a lane that is not in `upper`.
__device__ __forceinline__ unsigned active_chain(unsigned long long members, unsigned long long upper, int lane) {
  const unsigned next = (unsigned)(upper >> lane >> 1), in = (unsigned)(members >> lane >> 1) & ((next & (0u - next)) - 1u);
  return ((upper >> lane) & 1ull) ? in : 0u;
}
// ROWS: the binary tree over the eight bits of the column number.  Columns: groups of 2^G rows, tiles of 2^T, units of 256, each
// in order.  id: row | column << 16 of the lane's entry, or all bits.
template <bool ROWS, int G, int T>
__device__ __forceinline__ ActiveTree active_tree(unsigned id, int lane) {
  ActiveTree A{0, 0, 0, true};
  unsigned long long live = __builtin_amdgcn_ballot_w64(id != ~0u);
  if constexpr (ROWS) {
    int depth = 0;
#pragma unroll 1
    for (int d = 1; d <= 8; ++d)
      active_pass<false>(id, lane, live, [&](unsigned o) { return ((o ^ id) & 0xffffu) == 0 && ((o ^ id) >> (16 + d)) == 0; }, [&](bool can, int nx) {
        const int round = max(depth, __shfl(depth, nx, 64));
        if (can) {
          const unsigned off = (unsigned)(nx - lane);
          A.offs |= off << active_offset_at(round);
          A.fits = A.fits && off <= active_offset_mask(round);
          depth = round + 1;
        }
      });
    A.rounds = active_most(depth);
    A.fits = __builtin_amdgcn_ballot_w64(!A.fits) == 0;
  } else {
    const unsigned long long none = ~live;
    const unsigned before = (unsigned)__shfl_up((int)id, 1, 64);
    auto first = [&](int shift) { return (id != ~0u) & ((lane == 0) | (((before ^ id) >> 16) != 0) | ((((before ^ id) & 0xffffu) >> shift) != 0)); };
    const bool g = first(G), t = first(T), u = first(8);
    A.units = (id == ~0u ? 1u << 27 : 0u) | (g ? 1u << 28 : 0u) | (t ? 1u << 29 : 0u);
    const unsigned long long mg = __builtin_amdgcn_ballot_w64(g) | none, mt = __builtin_amdgcn_ballot_w64(t) | none,
                             mu = __builtin_amdgcn_ballot_w64(u) | none;
    A.rounds = active_most(__builtin_popcount(active_chain(~0ull, mg, lane))) | active_most(__builtin_popcount(active_chain(mg, mt, lane))) << 4 |
               active_most(__builtin_popcount(active_chain(mt, mu, lane))) << 9;
    // (no chain past 32 lanes: less than 33 entries in a unit)
    const unsigned after = (unsigned)(mu >> lane >> 1);
    A.fits = __builtin_amdgcn_ballot_w64(u && lane < 32 && after == 0) == 0;
    live = mu & ~none;
  }
  if ((live >> lane) & 1ull) A.units |= 1u << 30;
  int n = 0;
  auto line = [&](unsigned o) { return ROWS ? ((o ^ id) & 0xffffu) == 0 : ((o ^ id) >> 16) == 0; };
  while (active_pass<true>(id, lane, live, line, [&](bool can, int nx) {
           if (can) A.units |= (unsigned)(nx - lane) << (6 * n);  // (kActLocal units at most: four rounds)
           ++n;
         })) {}
  if ((live >> lane) & 1ull) A.units |= 1u << 31;
  A.rounds |= (n > 0 ? n - 1 : 0) << 16;
  return A;
}
// ... and they are added up, two waves' worth side by side.  v: the lane's entries, in the end the sums of their units (first of a
// unit); share: of their rows or columns.
struct ActiveSums {
  float v[2];
  double share[2];
};
template <bool ROWS>
__device__ __forceinline__ ActiveSums active_sums(float v0, float v1, unsigned offs0, unsigned offs1, unsigned units0, unsigned units1, int rounds0,
                                                  int rounds1, int lane) {
  auto up = [&](float x, unsigned off) { return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute((int)(4u * ((unsigned)lane + off)), fbits(x))); };
  const int units = max(rounds0 >> 16, rounds1 >> 16);
  if constexpr (ROWS) {
    const int rounds = max(rounds0 & 0xffff, rounds1 & 0xffff);
#pragma unroll 1
    for (int r = 0; r < rounds; ++r) {
      const int at = active_offset_at(r);
      const unsigned mask = active_offset_mask(r), off0 = (offs0 >> at) & mask, off1 = (offs1 >> at) & mask;
      const float w0 = up(v0, off0), w1 = up(v1, off1);
      v0 = off0 != 0 ? v0 + w0 : v0;
      v1 = off1 != 0 ? v1 + w1 : v1;
    }
  } else {
    unsigned long long members0 = ~0ull, members1 = ~0ull;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const unsigned bits = 1u << 27 | 1u << (28 + c);
      const unsigned long long upper0 = __builtin_amdgcn_ballot_w64((units0 & bits) != 0), upper1 = __builtin_amdgcn_ballot_w64((units1 & bits) != 0);
      unsigned m0 = active_chain(members0, upper0, lane), m1 = active_chain(members1, upper1, lane);
      members0 = upper0;
      members1 = upper1;
      const int from = c == 0 ? 0 : c == 1 ? 4 : 9, most = c == 1 ? 31 : 15;
      const int rounds = max((rounds0 >> from) & most, (rounds1 >> from) & most);
#pragma unroll 1
      for (int r = 0; r < rounds; ++r) {
        const float w0 = up(v0, m0 != 0 ? (unsigned)__builtin_ctz(m0) + 1u : 0u), w1 = up(v1, m1 != 0 ? (unsigned)__builtin_ctz(m1) + 1u : 0u);
        v0 = m0 != 0 ? v0 + w0 : v0;
        v1 = m1 != 0 ? v1 + w1 : v1;
        m0 &= m0 - 1u;
        m1 &= m1 - 1u;
      }
    }
  }
  ActiveSums A{{v0, v1}, {(double)v0, (double)v1}};
#pragma unroll 1
  for (int u = 0; u < units; ++u) {
    const unsigned off0 = (units0 >> (6 * u)) & 63u, off1 = (units1 >> (6 * u)) & 63u;
    const float w0 = up(v0, off0), w1 = up(v1, off1);
    A.share[0] += off0 != 0 ? (double)w0 : 0.0;
    A.share[1] += off1 != 0 ? (double)w1 : 0.0;
  }
  return A;
}

// Four costs of a lane, columns j .. j + 3 (j a multiple of four) of row i: the inner products as chains of fused
// multiply-adds over the coordinates in order, which is what v_mfma_f32_16x16x4_f32 makes of them (the sweeps' bits).
__device__ __forceinline__ f4v active_points_cost(const PointArgs& Pt, int i, int j, int n) {
  const int ng = Pt.dq >> 2;
  const int cb = min(j >> 4, Pt.ncb - 1);
  const float* __restrict__ ap = Pt.xs_pack + (size_t)i * 4 * Pt.dq;
  const float* __restrict__ bp = Pt.xt_pack + ((size_t)cb * ng * 64 + (j & 15)) * 4;
  f4v dot = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
  for (int g = 0; g < ng; ++g) {
    f4v av[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) av[k] = *reinterpret_cast<const f4v*>(ap + g * 16 + k * 4);
#pragma unroll
    for (int col = 0; col < 4; ++col) {
      f4v bv[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) bv[k] = *reinterpret_cast<const f4v*>(bp + g * 256 + k * 64 + col * 4);
      if (col > 0) __builtin_amdgcn_sched_barrier(0);  // (one column's operands at a time: registers)
      float d = dot[col];
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int k = 0; k < 4; ++k) d = fmaf(av[k][s], bv[k][s], d);
      dot[col] = d;
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  const float* __restrict__ ysq = Pt.xt_sq;  // (columns past n: another's, masked out like their cost)
  return points_cost(Pt, dot, Pt.xs_sq[i], f4v{ysq[min(j, n - 1)], ysq[min(j + 1, n - 1)], ysq[min(j + 2, n - 1)], ysq[min(j + 3, n - 1)]});
}

// f(0), f(STEP), ..., below N, the numbers known to the compiler: what is kept per task or piece stays in registers of its own.
template <int N, int STEP = 1, int K = 0, typename F>
__device__ __forceinline__ void active_each(F f) {
  if constexpr (K < N) {
    f(std::integral_constant<int, K>{});
    active_each<N, STEP, K + STEP>(f);
  }
}
// A number that all lanes hold alike, in a scalar register.
__device__ __forceinline__ float active_uniform(float v) { return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(fbits(v))); }
// The arguments once more, fetched where they are used (late_args).
__device__ __forceinline__ const ActiveArgs& late_active_args() {
  auto p = __builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const ActiveArgs*)p;
}

// The words of the shares and of a - 2r, b - 2s are the numbers themselves, with one bit to tell an iteration's from the one before
// in the same place (two iterations earlier): half the words, and the words are what the hops cost (20000 x 20000, an iteration:
// numbers and their halves' tags in two words 17 us, so 12, with what else has changed since).  The launch starts from zeroed words.
__device__ __forceinline__ unsigned active_phase(int it) { return 1u ^ ((unsigned)it >> 1 & 1u); }
__device__ __forceinline__ void active_store(u64* half, unsigned word, u64 v) {
  __hip_atomic_store(reinterpret_cast<u64*>(reinterpret_cast<char*>(half) + word * 8u), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// A share, a sum of numbers that are not negative, needs no sign.
__device__ __forceinline__ u64 active_word(double share, unsigned phase) {
  return (__builtin_bit_cast(u64, share) & ~(1ull << 63)) | (u64)phase << 63;
}
__device__ __forceinline__ double active_share(u64 w) { return __builtin_bit_cast(double, w & ~(1ull << 63)); }
// a - 2r is of the size of sums of fp32 numbers (or zero, or not finite): ten bits of exponent do, and what is below 2^-511 becomes zero.
// [phase][sign][exponent][fraction]
__device__ __forceinline__ u64 active_signed_word(double v, unsigned phase) {
  const u64 b = __builtin_bit_cast(u64, v);
  const int e = (int)(b >> 52 & 0x7ffu);
  const int e10 = e == 0x7ff ? 0x3ff : min(max(e - 511, 0), 0x3fe);
  const u64 fraction = e10 == 0 ? 0ull : b & ((1ull << 52) - 1ull);
  return (u64)phase << 63 | (b >> 63) << 62 | (u64)e10 << 52 | fraction;
}
__device__ __forceinline__ double active_signed(u64 w) {
  const int e10 = (int)(w >> 52 & 0x3ffu);
  const int e = e10 == 0 ? 0 : e10 == 0x3ff ? 0x7ff : e10 + 511;
  return __builtin_bit_cast(double, (w >> 62 & 1ull) << 63 | (u64)e << 52 | (w & ((1ull << 52) - 1ull)));
}
// grid_gather for such words.
template <int N, int PAUSE>
__device__ __forceinline__ void active_gather(const u64* half, u64 (&v)[N], const unsigned (&at)[N], unsigned phase, int limit, bool& lost) {
  for (int polls = 1;; ++polls) {
    bool there = true;
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] = grid_load(half, at[k]);
#pragma unroll
    for (int k = 0; k < N; ++k) there = there && (unsigned)(v[k] >> 63) == phase;
    if (__builtin_amdgcn_ballot_w64(!there) == 0) return;
    if (polls >= limit) {
      lost = true;
      return;
    }
    if (polls >= kGridPatience) {
      __builtin_amdgcn_s_sleep(kGridRest);
      polls += kGridRestPolls - 1;
    } else if (PAUSE > 0) {
      __builtin_amdgcn_s_sleep(PAUSE);
    }
  }
}

template <bool POINTS>
__global__ __launch_bounds__(kActThreads) void grid_active_kernel(ActiveArgs args) {
  constexpr int kLines = 8 * kActLocal;          // lines of a row of the workgroup
  constexpr int kGroupBits = POINTS ? 1 : 3, kTileBits = POINTS ? 5 : 6;
  __shared__ float dual[2 * kActRows];           // phi of the workgroup's rows, varphi of its columns
  __shared__ float val[kActEntries];             // X of the entries, rows in order and columns within a row
  __shared__ unsigned idx[kActEntries];          // row of the workgroup | column of the workgroup << 16; all bits: no entry
  __shared__ unsigned flags[kActLocal * kActRows / 4];  // [segment][row], a byte each: lines of X that hold something
  __shared__ __align__(16) float rise[kLines];   // how far varphi has risen since `since`, the largest of a line added up
  __shared__ __align__(16) float mags[kLines];   // ... and the magnitude of that with the largest of varphi, at the last list
  union Shared {
    struct {
      float rowseg[kActLocal][kActRows];         // sums of the row segments
      double share[2 * kActRows];                // ... of the rows, then of the columns
      float totals[kActSide * kActLocal * kActSide * kActLocal];  // the keeper: of all pieces of 256 x 256
      float old[kActEntries];                    // X before the sweep
    } f;
    struct {                                     // while listing
      union {
        unsigned lines[kActLines];               // lines to fetch (row | line << 16); then
        struct {
          float cost[kActEntries];               // C of the entries
          unsigned short loose[kActEntries];     // the entries by row, then by column, in no order there
          unsigned short colpos[kActEntries];    // the entries by column, rows in order
        };
      };
      float x[kActEntries], c[kActEntries];      // the entries as they are found
      unsigned id[kActEntries];
    } l;
  };
  __shared__ Shared U;
  __shared__ unsigned counts[2 * kActRows];  // while listing: entries of the rows, then of the columns (and places taken << 16)
  __shared__ __align__(8) unsigned short starts[2 * kActRows];  // ... and the place of their first one
  __shared__ int pieces[kActTasks * kActWaves];  // ... and how many times 64 places the rows or columns of a task take
  __shared__ int rounds[2][kActSlots][kActWaves];  // of the sums along the rows, along the columns
  __shared__ int nlines, nfound, nofit, left;
  __shared__ float risen[2][kActWaves];          // largest rise of phi, of varphi since the list
  __shared__ double red[kActWaves];
  __shared__ int asked;                          // the keeper: what the others ask for
  __shared__ int failed[2];                      // a word that never came: of the keeper's; of the others
  __shared__ double state[2][kActWaves][kActOwned][kGridBlock];  // eq. (6) state of the owned blocks, and before the last update
  __shared__ float target[kActWaves][kActOwned][kGridBlock];  // ... and their entries of p, q
  __shared__ double thetas[3];                   // the keeper: theta, and before the last update; 1^T p
  __shared__ double constant;                    // 2 eta - theta, as it has come
  __shared__ unsigned to_do;                     // ... and what to do next
  // (otherwise: phi and varphi of the list's time; the keeper, at a check: squared residuals of 64 rows or columns)
  float* const ref = reinterpret_cast<float*>(counts);
  double* const sq64 = reinterpret_cast<double*>(starts);
  static_assert(sizeof(counts) == 4 * 2 * kActRows && sizeof(starts) >= sizeof(double) * 2 * kActSide * kActRows / 64, "one each");

  const ActiveArgs& A = late_active_args();
  const SweepArgs& S = A.S;
  if (*A.done) return;
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wa = blockIdx.x / kActSide, wb = blockIdx.x % kActSide;
  const bool some = wa < A.ngroups && wb < A.nseg;  // (it holds part of the plan)
  const int nla = some ? (A.ngroups - wa + kActSide - 1) / kActSide : 0;
  const int nlb = some ? (A.nseg - wb + kActSide - 1) / kActSide : 0;
  const int nrc = 4 * nla, ntask = nrc + 4 * nlb;
  const bool keeper = blockIdx.x == kActWgs - 1;  // (the one with the fewest groups and segments)

  // a wave's tasks: 64 rows or 64 columns each (wave-uniform but for the lane)
  struct Task {
    bool live, rows;
    int first, count, local;  // first of the 64 in the matrix; how many exist; first in `dual`
  };
  auto task = [&](int k) __attribute__((always_inline)) {
    Task T;
    const int q = wave + kActWaves * k, c = q < nrc ? q : q - nrc;
    T.live = q < ntask;
    T.rows = q < nrc;
    T.first = ((T.rows ? wa : wb) + kActSide * (c >> 2)) * 256 + (c & 3) * 64;
    T.count = T.live ? min(max((T.rows ? S.m : S.n) - T.first, 0), 64) : 0;
    T.local = (T.rows ? 0 : kActRows) + c * 64;
    return T;
  };
  auto row_of = [&](unsigned id) { return (wa + kActSide * (int)((id & 0xffffu) >> 8)) * 256 + (int)(id & 255u); };
  auto col_of = [&](unsigned id) { return (wb + kActSide * (int)(id >> 24)) * 256 + (int)((id >> 16) & 255u); };

  // ---- state ----
  // the entries: a wave holds the places 64 (wave + 16 k) .. + 63, rows in order; the same places once more, columns in order
  float c[kActSlots];         // C (X is in `val`)
  unsigned row_offs[kActSlots], row_units[kActSlots], col_units[kActSlots];  // ActiveTree
  unsigned col_at[kActSlots]; // place of the entry that is here in the columns' order | its column << 16
  active_each<kActSlots>([&](auto k) __attribute__((always_inline)) {
    c[k] = 0.f;
    row_offs[k] = row_units[k] = col_units[k] = 0;
    col_at[k] = 0;
  });
  active_each<kActTasks>([&](auto k) __attribute__((always_inline)) {
    const Task T = task(k);
    if (T.live) {
      const int i = T.first + lane;
      const float v = lane < T.count ? (T.rows ? S.phi[i] : S.varphi[i]) : kMaskedOut;
      dual[T.local + lane] = v;
      ref[T.local + lane] = T.rows ? v : lane < T.count ? A.since[i] : kMaskedOut;
    }
  });
  for (int e = t; e < kLines; e += kActThreads) rise[e] = 0.f;
  if (t < 2) failed[t] = 0;
  if (t == 2) asked = 0;
  if (keeper && t == 0) {
    thetas[0] = thetas[1] = *A.theta_in;
    thetas[2] = *A.sum_p;
  }
  const int nblk = A.nblk_m + A.nblk_n;
  auto block = [&](int o) { return wave * (kActWgs - 1) + (int)blockIdx.x + o * (kActWgs - 1) * kActWaves; };
#pragma unroll
  for (int o = 0; o < kActOwned; ++o) {
    const int blk = block(o);
    if (!keeper && blk < nblk && lane < kGridBlock) {
      const bool own_rows = blk < A.nblk_m;
      const int entry = min((own_rows ? blk : blk - A.nblk_m) * kGridBlock + lane, (own_rows ? S.m : S.n) - 1);
      state[0][wave][o][lane] = own_rows ? A.a_in[entry] : A.b_in[entry];
      target[wave][o][lane] = own_rows ? A.p[entry] : A.q[entry];
    }
  }

  int row_pieces = 0, col_pieces = 0;  // 64 places each
  int cnt = 0;               // entries listed
  float tau = A.tau0;
  float rate = -1.f;         // rise per iteration (not known: negative)
  float risen_last = 0.f;    // ... of phi and varphi together since the list, at the last look
  int since_list = 0, lists = 0;
  int ask = 0;               // 1: a new list soon; 2: leave behind the next iteration; 4: this workgroup has no list
  bool relist = true, have_list = false;
  __syncthreads();

  // The list's entries into X, the sums of the row segments and the line flags into memory (and into `flags`).
  auto put_back = [&]() __attribute__((always_inline)) {
    const ActiveArgs& A = late_active_args();
    const SweepArgs& S = A.S;
    const int lane = lane_again(), t = wave * 64 + lane;
    for (int e = t; e < kActLocal * kActRows / 4; e += kActThreads) flags[e] = 0;
    __syncthreads();
    active_each<kActSlots>([&](auto k) __attribute__((always_inline)) {
      if (wave + kActWaves * k >= row_pieces) return;
      const unsigned id = idx[t + kActThreads * k];
      if (id != ~0u) {
        const unsigned lr = id & 0xffffu, lc = id >> 16;
        const float x = val[t + kActThreads * k];
        S.X[(size_t)row_of(id) * S.ldx + col_of(id)] = x;
        if (fbits(x) != 0) atomicOr(&flags[(lc >> 8) * (kActRows / 4) + (lr >> 2)], 1u << (8 * (lr & 3) + ((lc >> 5) & 7)));
      }
    });
    __syncthreads();
#pragma unroll 1
    for (int q = wave; q < nrc * nlb; q += kActWaves) {
      const int ls = q / nrc, lr = (q - ls * nrc) * 64 + lane, row = (wa + kActSide * (lr >> 8)) * 256 + (lr & 255);
      if (row < S.m) {
        const size_t at = (size_t)(wb + kActSide * ls) * S.mp + row;
        S.rowpart[at] = U.f.rowseg[ls][lr];
        if (A.lines) A.lines[at] = (unsigned char)(flags[ls * (kActRows / 4) + (lr >> 2)] >> (8 * (lr & 3)));
      }
    }
  };
  // How far varphi has risen since the list, line by line of columns (the largest of 32), is added to what is known.
  auto add_rise = [&]() __attribute__((always_inline)) {
    const int lane = lane_again();
    active_each<kActTasks>([&](auto k) __attribute__((always_inline)) {
      const Task T = task(k);
      if (!T.live || T.rows) return;
      const float v = dual[T.local + lane];
      const float from = ref[T.local + lane];
      float d = lane < T.count ? active_rise(v, from) : -INFINITY, mag = lane < T.count ? fabsf(v) : 0.f;
#pragma unroll
      for (int off = 16; off > 0; off >>= 1) {
        d = fmaxf(d, __shfl_xor(d, off, 64));
        mag = fmaxf(mag, __shfl_xor(mag, off, 64));
      }
      if ((lane & 31) == 0) {
        const int line = (T.local - kActRows + lane) >> 5;
        const float risen = d == -INFINITY ? 0.f : active_rises(rise[line], d);
        rise[line] = risen;
        mags[line] = fabsf(risen) + mag;
      }
      ref[T.local + lane] = v;
    });
  };

  // ---- a new list ----
  auto make_list = [&]() __attribute__((always_inline)) {
    if (have_list) put_back();
    const ActiveArgs& A = late_active_args();
    auto shortest = [&]() __attribute__((always_inline)) { return POINTS ? A.shortest : (float)kActShortest; };
    const SweepArgs& S = A.S;
    const int lane = lane_again(), t = wave * 64 + lane;
    const bool fresh = lists == 0;
    if (fresh) {  // which lines hold something: from memory
      for (int e = t; e < kActLocal * kActRows / 4; e += kActThreads) {
        unsigned w = 0;
        const int ls = e / (kActRows / 4), lr = 4 * (e % (kActRows / 4));
        const int row = (wa + kActSide * (lr >> 8)) * 256 + (lr & 255), seg = wb + kActSide * ls;
        if (some && ls < nlb && lr < 256 * nla) {
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (row + u < S.m) {
              const size_t at = (size_t)seg * S.mp + row + u;
              const unsigned f = (A.lines && A.lines_known) ? A.lines[at] : fbits(S.rowpart[at]) != 0 ? 0xffu : 0u;
              w |= f << (8 * u);
            }
        }
        flags[e] = w;
      }
      if (!(A.lines && A.lines_known)) {  // (a line of X costs less to read than one of the cost, from points above all)
        __syncthreads();
#pragma unroll 1
        for (int q = wave; q < nrc * nlb; q += kActWaves) {
          const int ls = q / nrc, lr0 = (q - ls * nrc) * 64, j = (wb + kActSide * ls) * kSegCols + 4 * lane;
          unsigned char* const f = reinterpret_cast<unsigned char*>(flags) + ls * kActRows + lr0;
          unsigned long long held = __builtin_amdgcn_ballot_w64(f[lane] != 0);
          while (held != 0) {
            int at[4];
            f4v x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              at[u] = held != 0 ? (int)__builtin_ctzll(held) : u > 0 ? at[u - 1] : 0;
              held &= held - 1ull;
              const int lr = lr0 + at[u], row = (wa + kActSide * (lr >> 8)) * 256 + (lr & 255);
              x[u] = f4v{0.f, 0.f, 0.f, 0.f};
              if (j < S.n) x[u] = *reinterpret_cast<const f4v*>(S.X + (size_t)row * S.ldx + j);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              unsigned long long b = __builtin_amdgcn_ballot_w64((fbits(x[u].x) | fbits(x[u].y) | fbits(x[u].z) | fbits(x[u].w)) != 0);
              unsigned lines = 0;
#pragma unroll
              for (int l = 0; l < 8; ++l) lines |= (b >> (8 * l) & 0xffull) != 0 ? 1u << l : 0u;
              if (lane == 0) f[at[u]] = (unsigned char)lines;
            }
          }
        }
      }
    }
    add_rise();
    have_list = false;
    __syncthreads();
    if (fresh) {  // (nothing better is known yet: phi is taken to rise as varphi has)
      float most_risen = 0.f;
      for (int e = 0; e < 8 * nlb; ++e) most_risen = fmaxf(most_risen, rise[e]);
      if (most_risen > 0.f) rate = active_uniform(2.f * most_risen / (float)A.age);
    }
    if (since_list > 0) rate = active_uniform(fmaxf(risen_last, 0.f) / (float)since_list);
    if (rate >= 0.f) tau = active_uniform(fmaxf(1.25f * rate * (float)A.target, 0.0625f * A.tau0));
    bool fits = false;
    // The entries found into their places, and how they are added up.
    auto order = [&]() __attribute__((always_inline)) {
      bool simple = true;
#pragma unroll 1
      for (int k = 0; k < kActTasks; ++k) {
        const Task T = task(k);
        if (!T.live) break;
        int base = 0;
        for (int q = T.rows ? 0 : nrc; q < wave + kActWaves * k; ++q) base += pieces[q];
        starts[T.local + lane] = (unsigned short)(starts[T.local + lane] + 64 * base);
      }
      for (int e = t; e < kActEntries; e += kActThreads) idx[e] = ~0u;
      __syncthreads();
      // rows in order, columns within a row: an entry's place is its row's plus how many of the row's lie before it
      unsigned place[kActSlots];
      active_each<kActSlots>([&](auto k) __attribute__((always_inline)) {
        const int e = t + kActThreads * k;
        if (e < cnt) {
          const unsigned lr = U.l.id[e] & 0xffffu;
          U.l.loose[starts[lr] + (atomicAdd(&counts[lr], 1u << 16) >> 16)] = (unsigned short)e;
        }
      });
      __syncthreads();
      active_each<kActSlots>([&](auto k) __attribute__((always_inline)) {
        const int e = t + kActThreads * k;
        place[k] = 0;
        if (e < cnt) {
          const unsigned id = U.l.id[e], first = starts[id & 0xffffu], count = counts[id & 0xffffu] & 0xffffu;
          unsigned before = 0;
          for (unsigned o = 0; o < count; ++o) before += U.l.id[U.l.loose[first + o]] < id ? 1u : 0u;  // (the same row: by column)
          place[k] = first + before;
          val[place[k]] = U.l.x[e];
          idx[place[k]] = id;
          U.l.cost[place[k]] = U.l.c[e];
        }
      });
      __syncthreads();
      active_each<kActSlots>([&](auto k) __attribute__((always_inline)) {
        const int e = t + kActThreads * k;
        if (e < cnt) {
          const unsigned lc = U.l.id[e] >> 16;
          U.l.loose[starts[kActRows + lc] + (atomicAdd(&counts[kActRows + lc], 1u << 16) >> 16)] = (unsigned short)e;
        }
      });
      for (int e = t; e < kActEntries; e += kActThreads) U.l.colpos[e] = 0xffff;
      __syncthreads();
      active_each<kActSlots>([&](auto k) __attribute__((always_inline)) {
        const int e = t + kActThreads * k;
        if (e < cnt) {
          const unsigned id = U.l.id[e], lc = id >> 16, first = starts[kActRows + lc], count = counts[kActRows + lc] & 0xffffu;
          unsigned before = 0;
          for (unsigned o = 0; o < count; ++o) before += U.l.id[U.l.loose[first + o]] < id ? 1u : 0u;  // (the same column: by row)
          U.l.colpos[first + before] = (unsigned short)place[k];
        }
      });
      __syncthreads();
      active_each<kActSlots>([&](auto k) __attribute__((always_inline)) {
        const int e = t + kActThreads * k;
        if (wave + kActWaves * k < row_pieces) {
          const unsigned id = idx[e];
          c[k] = id != ~0u ? U.l.cost[e] : 0.f;
          const ActiveTree R = active_tree<true, kGroupBits, kTileBits>(id, lane);
          row_offs[k] = R.offs;
          row_units[k] = R.units;
          simple = simple && R.fits;
          if (lane == 0) rounds[0][k][wave] = R.rounds;
        }
        if (wave + kActWaves * k < col_pieces) {
          const unsigned at = U.l.colpos[e], id = at != 0xffffu ? idx[at] : ~0u;
          const ActiveTree R = active_tree<false, kGroupBits, kTileBits>(id, lane);
          col_units[k] = R.units;
          simple = simple && R.fits;
          if (lane == 0) rounds[1][k][wave] = R.rounds;
          col_at[k] = id != ~0u ? at | (id >> 16) << 16 : 0xffffu;
        }
      });
      if (!simple) nofit = 1;
      __syncthreads();
      fits = nofit == 0;  // (else more than 32 entries of a column within 256 rows, or two halves of a row's sum of as many)
    };
#pragma unroll 1
    for (int attempt = 0; attempt < 5; ++attempt) {
      active_each<kActSlots>([&](auto k) __attribute__((always_inline)) {  // (no registers for these while listing)
        c[k] = 0.f;
        row_offs[k] = row_units[k] = col_units[k] = 0;
        col_at[k] = 0;
      });
      for (int e = t; e < 2 * kActRows; e += kActThreads) counts[e] = 0;
      if (t < 4) (t == 0 ? nlines : t == 1 ? nfound : t == 2 ? nofit : left) = 0;
      __syncthreads();
      // the lines that may hold an active entry: 64 rows x a segment to a wave at a time, until there is no room for more
      if (lane == 0) rounds[0][0][wave] = wave;  // (where a wave goes on: its own word, not in use yet)
      for (bool more = true; more;) {
        int q = __builtin_amdgcn_readfirstlane(rounds[0][0][wave]);
#pragma unroll 1
        for (; q < nrc * nlb; q += kActWaves) {
          const int ls = q / nrc, lr = (q - ls * nrc) * 64 + lane, row = (wa + kActSide * (lr >> 8)) * 256 + (lr & 255);
          const int seg = wb + kActSide * ls;
          unsigned held = 0;
          if (row < S.m) {
            const size_t at = (size_t)seg * S.mp + row;
            float* __restrict__ bp = A.bound + 8 * at;
            f4v lo, hi;
            if (fresh && A.codes && attempt == 0) {
              const float m1 = A.m1[at];
              const uint2 cd = A.codes[at];
              const int base = line_code_base(S.rho);
#pragma unroll
              for (int l = 0; l < 4; ++l) {
                lo[l] = m1 - line_decode((cd.x >> (8 * l)) & 0xffu, base);
                hi[l] = m1 - line_decode((cd.y >> (8 * l)) & 0xffu, base);
              }
              *reinterpret_cast<f4v*>(bp) = lo;
              *reinterpret_cast<f4v*>(bp + 4) = hi;
            } else {
              lo = *reinterpret_cast<const f4v*>(bp);
              hi = *reinterpret_cast<const f4v*>(bp + 4);
            }
            const float ph = dual[lr];
            held = flags[ls * (kActRows / 4) + (lr >> 2)] >> (8 * (lr & 3)) & 0xffu;
#pragma unroll
            for (int l = 0; l < 8; ++l) {
              const float b = l < 4 ? lo[l & 3] : hi[l & 3], s = rise[8 * ls + l];
              if (active_line(b, s, mags[8 * ls + l], ph, tau)) held |= 1u << l;
            }
            // (columns past n: no line, whatever the flags made of row-segment sums say)
            held &= (1u << min((S.n - seg * kSegCols + 31) / 32, 8)) - 1u;
          }
          if (__builtin_amdgcn_ballot_w64(held != 0) == 0) continue;
          int all = 0;
#pragma unroll
          for (int l = 0; l < 8; ++l) all += __builtin_popcountll(__builtin_amdgcn_ballot_w64((held >> l) & 1u));
          int at = 0;
          if (lane == 0) {
            at = nlines;
            for (int seen = -1; at != seen && at + all <= kActLines;) {
              seen = at;
              at = (int)atomicCAS((unsigned*)&nlines, (unsigned)seen, (unsigned)(seen + all));
            }
          }
          at = __builtin_amdgcn_readfirstlane(at);
          if (at + all > kActLines) {  // (these are found once more)
            if (lane == 0) left = 1;
            break;
          }
#pragma unroll
          for (int l = 0; l < 8; ++l) {
            const unsigned long long b = __builtin_amdgcn_ballot_w64((held >> l) & 1u);
            const int mine = at + __builtin_popcountll(b & ((1ull << lane) - 1ull));
            if ((held >> l) & 1u) U.l.lines[mine] = (unsigned)lr | (unsigned)(8 * ls + l) << 16;
            at += __builtin_popcountll(b);
          }
        }
        if (lane == 0) rounds[0][0][wave] = q;
        __syncthreads();
        // ... are fetched, eight lanes a line: their entries, and exact bounds
        const int nl = nfound <= kActEntries ? nlines : 0;  // (too many: the bounds of the rest only)
        constexpr int kAtOnce = POINTS ? 1 : 4;
        const int l4 = 4 * (lane & 7);
#pragma unroll 1
        for (int k0 = 8 * wave; k0 < nl; k0 += 8 * kActWaves * kAtOnce) {
          unsigned code[kAtOnce];
          f4v cc[kAtOnce], xx[kAtOnce];
#pragma unroll
          for (int s = 0; s < kAtOnce; ++s) {
            code[s] = U.l.lines[min(k0 + 8 * kActWaves * s + (lane >> 3), nl - 1)];
            const unsigned lr = code[s] & 0xffffu, line = code[s] >> 16;
            const int row = (wa + kActSide * (int)(lr >> 8)) * 256 + (int)(lr & 255u);
            const int j = (wb + kActSide * (int)(line >> 3)) * kSegCols + (int)(line & 7u) * 32 + l4;
            if constexpr (POINTS) cc[s] = active_points_cost(A.points, row, j, S.n);
            else cc[s] = *reinterpret_cast<const f4v*>(S.C + (size_t)row * S.ldc + j);
            xx[s] = f4v{0.f, 0.f, 0.f, 0.f};
            if (flags[(line >> 3) * (kActRows / 4) + (lr >> 2)] >> (8 * (lr & 3) + (line & 7u)) & 1u)
              xx[s] = *reinterpret_cast<const f4v*>(S.X + (size_t)row * S.ldx + j);
          }
#pragma unroll
          for (int s = 0; s < kAtOnce; ++s) {
            const int k = k0 + 8 * kActWaves * s + (lane >> 3);
            const unsigned lr = code[s] & 0xffffu, line = code[s] >> 16;
            const f4v vp = *reinterpret_cast<const f4v*>(&dual[kActRows + line * 32 + l4]);
            const float ph = dual[lr], rho = S.rho;
            const f4v tv = {fmaf(-rho, cc[s].x, vp.x), fmaf(-rho, cc[s].y, vp.y), fmaf(-rho, cc[s].z, vp.z), fmaf(-rho, cc[s].w, vp.w)};
            unsigned act = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const bool in = fbits(xx[s][e]) != 0 || active_entry(tv[e], vp[e], ph, tau);
              act |= in && k < nl ? 1u << e : 0u;
            }
            const float top = line_max(tv);
            if (k < nl && (lane & 7) == 0) {
              const int row = (wa + kActSide * (int)(lr >> 8)) * 256 + (int)(lr & 255u);
              A.bound[8 * ((size_t)(wb + kActSide * (int)(line >> 3)) * S.mp + row) + (line & 7u)] = top - rise[line];
            }
            if (__builtin_amdgcn_ballot_w64(act != 0) == 0) continue;
            int all = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) all += __builtin_popcountll(__builtin_amdgcn_ballot_w64((act >> e) & 1u));
            int at = 0;
            if (lane == 0) at = atomicAdd(&nfound, all);
            at = __builtin_amdgcn_readfirstlane(at);
            if (act != 0) atomicAdd(&counts[lr], (unsigned)__builtin_popcount(act));
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const unsigned long long b = __builtin_amdgcn_ballot_w64((act >> e) & 1u);
              const int mine = at + __builtin_popcountll(b & ((1ull << lane) - 1ull));
              if ((act >> e) & 1u) {
                const unsigned lc = line * 32 + (unsigned)(l4 + e);
                if (mine < kActEntries) {
                  U.l.x[mine] = xx[s][e];
                  U.l.c[mine] = cc[s][e];
                  U.l.id[mine] = lr | lc << 16;
                }
                atomicAdd(&counts[kActRows + lc], 1u);
              }
              at += __builtin_popcountll(b);
            }
          }
        }
        __syncthreads();
        more = left != 0;
        __syncthreads();
        if (t < 2) (t == 0 ? nlines : left) = 0;
        __syncthreads();
      }
      // places: a row's entries lie within 64 of them, a column's too; the pieces a task takes
#pragma unroll 1
      for (int k = 0; k < kActTasks; ++k) {
        const Task T = task(k);
        if (!T.live) break;
        const int mine = (int)counts[T.local + lane];
        int upto = mine;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
          const int other = __shfl_up(upto, off, 64);
          upto += lane >= off ? other : 0;
        }
        if (__builtin_amdgcn_ballot_w64(mine > 64) != 0) nofit = 1;
        int piece = 0, taken = 0, place = 0;
        unsigned long long left = __builtin_amdgcn_ballot_w64(mine > 0);
        while (left != 0 && piece < 64) {
          const unsigned long long now = left & __builtin_amdgcn_ballot_w64(upto - taken <= 64);
          if (now == 0) break;  // (a row of more than 64)
          if ((now >> lane) & 1ull) place = 64 * piece + upto - mine - taken;
          left &= ~now;
          taken = __builtin_amdgcn_readlane(upto, 63 - (int)__builtin_clzll(now));
          ++piece;
        }
        starts[T.local + lane] = (unsigned short)place;
        if (lane == 0) pieces[wave + kActWaves * k] = piece;
      }
      __syncthreads();
      row_pieces = col_pieces = 0;
      for (int q = 0; q < ntask; ++q) (q < nrc ? row_pieces : col_pieces) += pieces[q];
      cnt = nfound;
      fits = nfound <= kActEntries && row_pieces <= 64 && col_pieces <= 64 && nofit == 0;
      if (fits) order();
      if (fits) break;
      row_pieces = col_pieces = 0;
      if (tau == 0.f || (rate >= 0.f && ((fresh && !POINTS) || 0.5f * tau < shortest() * rate))) break;
      tau = active_uniform(rate >= 0.f ? fmaxf(0.3f * tau, shortest() * rate) : attempt == 3 ? 0.f : 0.25f * tau);
      __syncthreads();
    }
    active_each<kActTasks>([&](auto k) __attribute__((always_inline)) {
      const Task T = task(k);
      if (T.live) ref[T.local + lane] = dual[T.local + lane];
    });
    ask = 0;
    if (!fits) {  // (what the old list held is in memory)
      ask = 4;
      return;
    }
    if (rate >= 0.f ? tau < shortest() * rate : tau == 0.f) ask = 2;  // (a list that does not last)
    for (int e = t; e < kActLocal * kActRows; e += kActThreads) (&U.f.rowseg[0][0])[e] = 0.f;
    for (int e = t; e < 4 * kActRows; e += kActThreads) reinterpret_cast<float*>(U.f.share)[e] = 0.f;
    have_list = true;
    ++lists;
    since_list = 0;
    risen_last = 0.f;
    __syncthreads();
  };

  // ---- the sums of the rows' segments and of the rows ----
  auto row_sums = [&](int k, float x0, float x1, unsigned id0, unsigned id1, int lane) __attribute__((always_inline)) {  // of pieces k and k + 1
    const int r0 = __builtin_amdgcn_readfirstlane(rounds[0][k][wave]);
    const int r1 = wave + kActWaves * (k + 1) < row_pieces ? __builtin_amdgcn_readfirstlane(rounds[0][k + 1][wave]) : 0;
    const ActiveSums A = active_sums<true>(x0, x1, row_offs[k], row_offs[k + 1], row_units[k], row_units[k + 1], r0, r1, lane);
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const unsigned id = p ? id1 : id0, u = row_units[k + p];
      if ((u >> 30) & 1u) U.f.rowseg[id >> 24][id & 0xffffu] = A.v[p];
      if (u >> 31) U.f.share[id & 0xffffu] = A.share[p];
    }
  };

  int it = 0, why = kActDone;
  int upto = A.check.first;  // (the next iteration with a check behind it)
  int nchecks = 0;
  bool aborted = false, broken = false;
  for (;; ++it) {
    if (relist) make_list();
    relist = false;
    const ActiveArgs& A = late_active_args();
    const int lane = lane_again(), t = wave * 64 + lane;
    const int nblk = A.nblk_m + A.nblk_n;
    const float rho = A.S.rho, scale = A.S.scale;
    const bool check = it == upto;
    const unsigned tag = A.tag0 + (unsigned)it, phase = active_phase(it);
    u64* __restrict__ half = A.xchg + (size_t)(tag & 1u) * A.half_words;
    if (t == 0) grid_store(half, A.tot_word + kActTotals * blockIdx.x + kActTotals - 1, (unsigned)ask, tag);

    // ---- sweep, and the sums along the rows (without a list, sums of nothing go out: nobody uses them) ----
    active_each<kActSlots, 2>([&](auto k) __attribute__((always_inline)) {
      if (wave + kActWaves * k >= row_pieces) return;
      unsigned id[2];
      float x[2];
#pragma unroll
      for (int p = 0; p < 2; ++p) id[p] = wave + kActWaves * (k + p) < row_pieces ? idx[t + kActThreads * (k + p)] : ~0u;
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        const bool there = id[p] != ~0u;
        const float ph = dual[there ? id[p] & 0xffffu : 0u], vp = dual[kActRows + (there ? id[p] >> 16 : 0u)];
        const int e = t + kActThreads * (k + p);
        const float was = val[e];
        x[p] = there ? fmaxf(was + fmaf(-rho, c[k + p], vp + ph), 0.f) * scale : 0.f;
        if (there) {
          U.f.old[e] = was;
          val[e] = x[p];
        }
      }
      row_sums(k, x[0], x[1], id[0], id[1], lane);
    });
    __syncthreads();
    // ---- the totals of 256 rows x 256 columns: half a wave each, lane h its rows 8 h .. 8 h + 7 ----
    for (int e0 = 2 * wave; e0 < nla * nlb; e0 += 2 * kActWaves) {
      const int e = min(e0 + (lane >> 5), nla * nlb - 1), la = e / nlb, ls = e - la * nlb, h = lane & 31;
      const f4v r0 = *reinterpret_cast<const f4v*>(&U.f.rowseg[ls][256 * la + 8 * h]);
      const f4v r1 = *reinterpret_cast<const f4v*>(&U.f.rowseg[ls][256 * la + 8 * h + 4]);
      float sum = 0.f;
      if constexpr (POINTS) {
        // pairs of rows, tiles of 32 rows (four lanes), their eight
        const float p0 = r0.x + r0.y, p1 = r0.z + r0.w, p2 = r1.x + r1.y, p3 = r1.z + r1.w;
        float tile = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const int from = (lane & 60) | w;
          tile += __shfl(p0, from, 64);
          tile += __shfl(p1, from, 64);
          tile += __shfl(p2, from, 64);
          tile += __shfl(p3, from, 64);
        }
#pragma unroll
        for (int w = 0; w < 8; ++w) sum += __shfl(tile, (lane & 32) | 4 * w, 64);
      } else {
        // groups of 8 rows, tiles of 64 (eight lanes), their four
        const float g8 = ((((((r0.x + r0.y) + r0.z) + r0.w) + r1.x) + r1.y) + r1.z) + r1.w;
        float tile = 0.f;
#pragma unroll
        for (int w = 0; w < 8; ++w) tile += __shfl(g8, (lane & 56) | w, 64);
#pragma unroll
        for (int w = 0; w < 4; ++w) sum += __shfl(tile, (lane & 32) | 8 * w, 64);
      }
      if (h == 0 && e0 + (lane >> 5) < nla * nlb)
        grid_store(half, A.tot_word + kActTotals * blockIdx.x + (unsigned)(la * kActLocal + ls), (unsigned)fbits(sum), tag);
    }

    // ---- the sums along the columns ----
    active_each<kActSlots, 2>([&](auto k) __attribute__((always_inline)) {
      if (wave + kActWaves * k >= col_pieces) return;
      float v[2];
#pragma unroll
      for (int p = 0; p < 2; ++p) {  // (no entry here: kActEntries or more, and nothing is added to anything)
        const unsigned at = col_at[k + p] & 0xffffu;
        v[p] = val[at & (kActEntries - 1)];
      }
      const int r0 = __builtin_amdgcn_readfirstlane(rounds[1][k][wave]);
      const int r1 = wave + kActWaves * (k + 1) < col_pieces ? __builtin_amdgcn_readfirstlane(rounds[1][k + 1][wave]) : 0;
      const ActiveSums A = active_sums<false>(v[0], v[1], 0, 0, col_units[k], col_units[k + 1], r0, r1, lane);
#pragma unroll
      for (int p = 0; p < 2; ++p)
        if (col_units[k + p] >> 31) U.f.share[kActRows + (col_at[k + p] >> 16)] = A.share[p];
    });
    __syncthreads();
    // ---- publish the shares of the rows and columns ----
#pragma unroll 1
    for (int k = 0; k < kActTasks; ++k) {
      const Task T = task(k);
      if (!T.live) break;
      const double share = U.f.share[T.local + lane];
      const unsigned blk = (unsigned)((T.rows ? 0 : A.nblk_m) + T.first / kGridBlock + (lane >> 3));
      const unsigned word = (blk * kActSide + (unsigned)(T.rows ? wb : wa)) * kGridBlock + (unsigned)(lane & 7);
      if (lane < T.count) active_store(half, word, active_word(share, phase));
    }
    // ---- hop 1: the shares of the owned entries; the totals and what everybody asks for ----
    bool lost = false;
    if (!keeper && block(0) < nblk) {
      const ActiveArgs& A = late_active_args();
      const SweepArgs& S = A.S;
      u64 v[2 * kActOwned];
      unsigned at[2 * kActOwned];
#pragma unroll
      for (int o = 0; o < kActOwned; ++o) {
        const int blk = block(o) < nblk ? block(o) : block(0);
        const bool own_rows = blk < A.nblk_m;
        const int e = min(lane & 7, (own_rows ? S.m : S.n) - 1 - (own_rows ? blk : blk - A.nblk_m) * kGridBlock);
        const int shares = min(own_rows ? A.nseg : A.ngroups, kActSide);
#pragma unroll
        for (int w = 0; w < 2; ++w) at[2 * o + w] = (unsigned)((blk * kActSide + min((lane >> 3) + 8 * w, shares - 1)) * kGridBlock + e);
      }
      active_gather<2 * kActOwned, kActPause>(half, v, at, phase, A.polls, lost);
#pragma unroll
      for (int o = 0; o < kActOwned; ++o) {
        const int blk = block(o);
        if (blk >= nblk) continue;
        const bool own_rows = blk < A.nblk_m;
        const int shares = min(own_rows ? A.nseg : A.ngroups, kActSide);
        const int entry = (own_rows ? blk : blk - A.nblk_m) * kGridBlock + (lane & 7);
        const bool exists = entry < (own_rows ? S.m : S.n);
        const double s0 = (lane >> 3) < shares ? active_share(v[2 * o]) : 0.0;
        const double s1 = (lane >> 3) + 8 < shares ? active_share(v[2 * o + 1]) : 0.0;
        // (the tree of sum_partials_16)
        const double total = add_lane_bit3(add_lane_bit4(add_lane_bit5(s0 + s1)));
        const double res = total - (double)target[wave][o][lane & 7];
        const double was = state[0][wave][o][lane & 7];
        if (lane < kGridBlock) {
          state[1][wave][o][lane] = was;
          state[0][wave][o][lane] = was - res;
        }
        if (exists && lane < kGridBlock)
          active_store(half, A.ent_word + (unsigned)(blk * kGridBlock + lane), active_signed_word(was - 2.0 * res, phase));
        if (check) {
          double sq = exists ? res * res : 0.0;
          sq += dpp_mov_f64<0xB1, 0xF>(sq);
          sq += dpp_mov_f64<0x4E, 0xF>(sq);
          sq += dpp_mov_f64<0x141, 0xF>(sq);
          const u64 w = __builtin_bit_cast(u64, sq);
          if (lane < 2) grid_store(half, A.sq_word + (unsigned)(blk * kActSquares + lane), lane == 0 ? (unsigned)(w >> 32) : (unsigned)w, tag);
          if (exists && lane < kGridBlock) (own_rows ? A.r : A.s)[entry] = res;
        }
      }
    }
    if (keeper) {
      const ActiveArgs& A = late_active_args();
      const SweepArgs& S = A.S;
      // a workgroup's words are two lines: a wave takes two of them at a time
      {
        u64 v[8];
        unsigned at[8];
        // the b-th of the wave's words: which workgroup's, and which piece of its (or none: what the workgroup asks for)
        const int ngroups = A.ngroups, nseg = A.nseg;
        auto word = [&](int ln, int b, int& e) __attribute__((always_inline)) {
          const int slot = ln & (kActTotals - 1), la = slot / kActLocal, ls = slot - la * kActLocal;
          const int grp = wave + kActSide * la, seg = 2 * b + (ln >> 5) + kActSide * ls;
          e = grp * nseg + seg;
          return ((slot < kActLocal * kActLocal) & (grp < ngroups) & (seg < nseg)) != 0;
        };
        static_assert(kActWaves == kActSide, "a wave takes the words of a row of workgroups");
#pragma unroll
        for (int b = 0; b < 8; ++b) {
          int e;
          const int off = word(lane, b, e) ? lane : lane | (kActTotals - 1);
          at[b] = A.tot_word + (unsigned)((kActSide * wave + 2 * b) * kActTotals + off);
        }
        grid_gather<8, kActPause, true>(half, v, at, tag, A.polls, lost);
        const int ln = lane_again();
        unsigned wants = 0;
#pragma unroll
        for (int b = 0; b < 8; ++b) {
          int e;
          const bool there = word(ln, b, e);
          if (there) U.f.totals[e] = grid_value(v[b]);
          wants |= there ? 0u : (unsigned)v[b];
        }
        const int all = (__builtin_amdgcn_ballot_w64(wants & 1u) != 0 ? 1 : 0) | (__builtin_amdgcn_ballot_w64(wants & 2u) != 0 ? 2 : 0) |
                        (__builtin_amdgcn_ballot_w64(wants & 4u) != 0 ? 4 : 0);
        if (ln == 0 && all != 0 && !lost) atomicOr(&asked, all);
      }
      if (check) {
        for (int side_n = 0; side_n < 2; ++side_n) {
          const int blocks = side_n ? A.nblk_n : A.nblk_m;
          const unsigned word = A.sq_word + (side_n ? kActSquares * (unsigned)A.nblk_m : 0u);
          for (int b0 = 64 * wave; b0 < blocks && !lost; b0 += kActThreads) {
            const unsigned w0 = word + kActSquares * (unsigned)min(b0 + lane, blocks - 1);
            u64 v[2];
            const unsigned at[2] = {w0, w0 + 1};
            grid_gather<2, kActPause, true>(half, v, at, tag, A.polls, lost);
            double sq = b0 + lane < blocks ? grid_value(v[0], v[1]) : 0.0;
            sq += dpp_mov_f64<0xB1, 0xF>(sq);
            sq += dpp_mov_f64<0x4E, 0xF>(sq);
            sq += dpp_mov_f64<0x141, 0xF>(sq);
            if ((lane & 7) == 0 && b0 + lane < blocks) sq64[(side_n ? (A.nblk_m + 7) / 8 : 0) + (b0 + lane) / 8] = sq;
          }
        }
      }
      if (lost) failed[0] = 1;
      __syncthreads();
      if (failed[0]) {
        broken = true;
        break;
      }
      const double recip = reciprocal_of((double)S.m + (double)S.n);
      {  // 1024 shares of the totals: share 64 wave + lane takes the totals that many and every 1024 further
        const int ntot = A.ngroups * A.nseg;
        constexpr int kMost = (kActSide * kActLocal * kActSide * kActLocal + kActThreads - 1) / kActThreads;
        float v[kMost];
        active_each<kMost>([&](auto k) __attribute__((always_inline)) { v[k] = U.f.totals[min(t + kActThreads * k, ntot - 1)]; });
        double acc = 0.0;
        active_each<kMost>([&](auto k) __attribute__((always_inline)) { acc = t + kActThreads * k < ntot ? acc + (double)v[k] : acc; });
        acc = wave_sum_f64(acc);
        if (lane == 0) red[wave] = acc;
      }
      __syncthreads();
      if (wave == 0) {
        double sum_x = 0.0;
#pragma unroll
        for (int k = 0; k < kActWaves; ++k) sum_x += red[k];
        const double theta = thetas[0];
        const double eta = divide_by(sum_x - thetas[2], (double)S.m + (double)S.n, recip);
        const u64 cst = __builtin_bit_cast(u64, 2.0 * eta - theta);
        if (lane == 0) {
          thetas[1] = theta;
          thetas[0] = theta - eta;
        }
        const int wants = asked;
        const unsigned next = (wants & 4) ? 4u : (unsigned)(wants & 3);
        const unsigned at = A.cst_word + 32u * (unsigned)(lane >> 1) + (unsigned)(lane & 1);
        grid_store(half, at, (lane & 1) ? (unsigned)cst : (unsigned)(cst >> 32), tag);
        if (lane < kGridCopies) grid_store(half, A.cst_word + 32u * (unsigned)lane + 2u, next, tag);
        if (check) {
          double norm2[2];
          for (int side_n = 0; side_n < 2; ++side_n) {
            const int rows64 = (A.nblk_m + 7) / 8, from = side_n ? rows64 : 0, count = side_n ? (A.nblk_n + 7) / 8 : rows64;
            double sum = 0.0;
            for (int k = 0; k < count; k += 64) sum += butterfly_f64(k + lane < count ? sq64[from + k + lane] : 0.0);
            norm2[side_n] = sum;
          }
          bool pass = false;
          if (lane == 0 && next != 4u) pass = make_check<true>(A.check, nchecks, it, norm2[0], norm2[1]);
          const unsigned word = __builtin_amdgcn_ballot_w64(pass) != 0 ? 1u : 0u;
          if (lane < kGridCopies) grid_store(half, A.cst_word + 32u * (unsigned)lane + 3u, word, tag);
        }
      }
    }

    // ---- hop 2: phi and varphi, and what to do next ----
    unsigned next;
    {
      const ActiveArgs& A = late_active_args();
      const SweepArgs& S = A.S;
      // (the words that are the same for everybody: one wave asks for them, the last, which has the least to do.  A wave that has lost a
      // word asks once for the others: what the waits of a launch add up to is one in hop 1 and one in hop 2, of another wave)
      u64 v[kActTasks];
      unsigned at[kActTasks];
#pragma unroll
      for (int k = 0; k < kActTasks; ++k) {  // (a task of nothing asks for the wave's first word, or for the first of all)
        const Task T = task(k);
        const unsigned ent = A.ent_word + (unsigned)((T.rows ? 0 : A.nblk_m * kGridBlock) + T.first + min(lane, T.count - 1));
        at[k] = T.count > 0 ? ent : k > 0 ? at[0] : A.ent_word;
      }
      const int polls = lost ? 1 : A.polls;
      active_gather<kActTasks, kActPause>(half, v, at, phase, polls, lost);
      if (wave == kActWaves - 1) {
        u64 w[3];
        const unsigned cst_at = A.cst_word + 32u * (blockIdx.x % kGridCopies);
        const unsigned at_w[3] = {cst_at, cst_at + 1u, cst_at + 2u};
        grid_gather<3, 1, true>(half, w, at_w, tag, lost ? 1 : polls, lost);
        if (lane == 0) {
          constant = grid_value(w[0], w[1]);
          to_do = (unsigned)w[2];
        }
      }
      const double recip_n = reciprocal_of((double)S.n), recip_m = reciprocal_of((double)S.m);
      __syncthreads();
      const double cst = constant;
      next = (unsigned)__builtin_amdgcn_readfirstlane((int)to_do);
      float up_rows = -INFINITY, up_cols = -INFINITY;
      active_each<kActTasks>([&](auto k) __attribute__((always_inline)) {
        const Task T = task(k);
        if (T.count <= 0 || next == 4u) return;
        const float d = (float)divide_by(active_signed(v[k]) + cst, T.rows ? (double)S.n : (double)S.m, T.rows ? recip_n : recip_m);
        const float from = ref[T.local + lane];
        const float r = active_rise(d, from);
        if (lane < T.count) {
          dual[T.local + lane] = d;
          if (T.rows) up_rows = fmaxf(up_rows, r);
          else up_cols = fmaxf(up_cols, r);
        }
      });
      up_rows = wave_max(up_rows);
      up_cols = wave_max(up_cols);
      if (lane == 0) {
        risen[0][wave] = up_rows;
        risen[1][wave] = up_cols;
      }
    }
    bool passes = false;
    if (check && next != 4u && !lost) {
      u64 v[1];
      const unsigned at[1] = {A.cst_word + 32u * (blockIdx.x % kGridCopies) + 3u};
      grid_gather<1, kActPause, true>(half, v, at, tag, A.polls, lost);
      passes = !lost && (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)v[0]) != 0;
    }
    if (lost) failed[1] = 1;
    if (keeper && t == 0) asked = 0;  // (read before the hop by this wave alone)
    __syncthreads();
    if (failed[1]) {
      broken = true;
      break;
    }
    if (next == 4u) {  // (somebody's entries did not fit: this iteration has not been)
      aborted = true;
      why = kActAbort;
      break;
    }
    if (check) {
      ++nchecks;
      upto = min(it + A.check.every, A.iters - 1);
    }
    if (passes || it == A.iters - 1) {
      ++it;
      break;
    }
    if (next & 2u) {
      why = kActLeave;
      ++it;
      break;
    }
    // (columns and rows that do not exist have not risen; a wave without any neither)
    float rr = lane < kActWaves ? risen[0][lane] : -INFINITY, rc = lane < kActWaves ? risen[1][lane] : -INFINITY;
    rr = wave_max(rr);
    rc = wave_max(rc);
    ++since_list;
    if (some) {
      const float now = active_rises(rr, rc);
      const float step = fmaxf(now - risen_last, 0.f);
      risen_last = active_uniform(now);
      relist = !(now < tau);
      ask = now + 2.5f * step < tau ? 0 : 1;
    }
    if (next & 1u) relist = true;
  }
  if (broken || failed[0] || failed[1]) {
    if (wave == 0 && lane_again() == 0) {
      A.status->broken = 1;
      __threadfence();
      *A.done = 1;
    }
    return;
  }

  // ---- leave the plan, its sums and flags, the bounds and the state behind the last update in memory ----
  const int lane_end = lane_again();
  if (aborted && have_list) {
    // X as it was before the sweep that nobody counts, and the sums of its rows (a workgroup whose entries did not fit has
    // made none, and has left its plan in memory)
    const int t_end = wave * 64 + lane_end;
    active_each<kActSlots, 2>([&](auto k) __attribute__((always_inline)) {
      if (wave + kActWaves * k >= row_pieces) return;
      unsigned id[2];
      float x[2];
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        const int e = t_end + kActThreads * (k + p);
        id[p] = wave + kActWaves * (k + p) < row_pieces ? idx[e] : ~0u;
        x[p] = id[p] != ~0u ? U.f.old[e] : 0.f;
        if (id[p] != ~0u) val[e] = x[p];
      }
      row_sums(k, x[0], x[1], id[0], id[1], lane_end);
    });
    __syncthreads();
  }
  if (have_list) put_back();
  add_rise();
#pragma unroll
  for (int k = 0; k < kActTasks; ++k) {
    const Task T = task(k);
    if (lane_end >= T.count) continue;
    const float v = dual[T.local + lane_end];
    if (T.rows && wb == 0) A.phi_out[T.first + lane_end] = v;
    if (!T.rows && wa == 0) A.varphi_out[T.first + lane_end] = A.bound_varphi[T.first + lane_end] = v;
  }
  __syncthreads();
  // (the bounds: against varphi as it is now)
#pragma unroll 1
  for (int q = wave; q < nrc * nlb; q += kActWaves) {
    const int ls = q / nrc, lr = (q - ls * nrc) * 64 + lane_end, row = (wa + kActSide * (lr >> 8)) * 256 + (lr & 255);
    if (row >= S.m) continue;
    f4v* const bp = reinterpret_cast<f4v*>(A.bound + 8 * ((size_t)(wb + kActSide * ls) * S.mp + row));
    f4v b[2] = {bp[0], bp[1]};
#pragma unroll
    for (int l = 0; l < 8; ++l) {
      const float s = rise[8 * ls + l], w = b[l >> 2][l & 3];
      b[l >> 2][l & 3] = w == -INFINITY ? w : active_rises(w, s);
    }
    bp[0] = b[0];
    bp[1] = b[1];
  }
  const bool alt = (it & 1) != 0;  // (behind an odd number of updates)
#pragma unroll
  for (int o = 0; o < kActOwned; ++o) {
    const int blk = block(o);
    if (keeper || blk >= nblk || lane_end >= kGridBlock) continue;
    const bool own_rows = blk < A.nblk_m;
    const int entry = (own_rows ? blk : blk - A.nblk_m) * kGridBlock + lane_end;
    if (entry < (own_rows ? S.m : S.n)) (own_rows ? (alt ? A.a_alt : A.a_in) : (alt ? A.b_alt : A.b_in))[entry] = state[aborted ? 1 : 0][wave][o][lane_end];
  }
  if (keeper && wave == 0 && lane_end == 0) {
    *(alt ? A.theta_alt : A.theta_in) = aborted ? thetas[1] : thetas[0];
    A.record->iters = it;
    A.record->why = why;
    A.record->lists = lists;
  }
}

// Whether a first list over a stored cost would fit, before a launch is made for it: the lines that it would look at, counted as make_list does,
// and from their share the entries of the busiest workgroup (each entry by its own chance; one a line at least).  A launch whose
// entries do not fit costs 0.13 to 0.3 ms, 1 to 4 % of a call, this 5 us.
constexpr int kForecastBits = 11;
static_assert(kActRows * kActRows < 1 << (32 - kForecastBits), "entries and an age in a word");
struct ForecastArgs {
  const float* phi;
  const float* varphi;
  const float* since;          // varphi the bounds are against
  const float* m1;             // bounds (ScreenArgs)
  const uint2* codes;
  const unsigned char* lines;  // line flags of X, or null
  DeviceStatus* status;
  const int* done;
  int m, n, mp, nseg, ngroups;
  float rho, tau0;
  int age;                     // iterations since `since`, at most
  int target;
  const int* ctl;              // control words of the sweep by lines, which renews the bounds by itself
  int k;                       // iteration of the call
};
__global__ __launch_bounds__(kActThreads) void active_forecast_kernel(ForecastArgs A) {
  constexpr int kLines = 8 * kActLocal;
  __shared__ float rise[kLines], mags[kLines];
  __shared__ int lines_found;
  if (*A.done) return;
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wa = blockIdx.x / kActSide, wb = blockIdx.x % kActSide;
  if (wa >= A.ngroups || wb >= A.nseg) return;
  const int nla = (A.ngroups - wa + kActSide - 1) / kActSide, nlb = (A.nseg - wb + kActSide - 1) / kActSide;
  if (t == 0) lines_found = 0;
  for (int e = 2 * wave + (lane >> 5); e < 8 * nlb; e += 2 * kActWaves) {
    const int j = (wb + kActSide * (e >> 3)) * kSegCols + (e & 7) * 32 + (lane & 31);
    const float v = j < A.n ? A.varphi[j] : 0.f;
    float d = j < A.n ? active_rise(v, A.since[j]) : -INFINITY, mag = fabsf(v);
#pragma unroll
    for (int off = 16; off > 0; off >>= 1) {
      d = fmaxf(d, __shfl_xor(d, off, 64));
      mag = fmaxf(mag, __shfl_xor(mag, off, 64));
    }
    if ((lane & 31) == 0) {
      rise[e] = d == -INFINITY ? 0.f : d;
      mags[e] = fabsf(rise[e]) + mag;
    }
  }
  __syncthreads();
  float most_risen = 0.f;
  for (int e = 0; e < 8 * nlb; ++e) most_risen = fmaxf(most_risen, rise[e]);
  const int age = min(A.age, A.ctl[kCtlSince] + 1);
  const float tau = most_risen > 0.f ? fmaxf(2.5f * most_risen / (float)age * (float)A.target, 0.0625f * A.tau0) : A.tau0;
  const int nrc = 4 * nla, base = line_code_base(A.rho);
  int found = 0;
  for (int q = wave; q < nrc * nlb; q += kActWaves) {
    const int ls = q / nrc, lr = (q - ls * nrc) * 64 + lane, row = (wa + kActSide * (lr >> 8)) * 256 + (lr & 255), seg = wb + kActSide * ls;
    if (row >= A.m) continue;
    const size_t at = (size_t)seg * A.mp + row;
    const float m1 = A.m1[at], ph = A.phi[row];
    const uint2 cd = A.codes[at];
    unsigned held = A.lines ? A.lines[at] : 0u;
#pragma unroll
    for (int l = 0; l < 8; ++l) {
      const float b = m1 - line_decode(((l < 4 ? cd.x : cd.y) >> (8 * (l & 3))) & 0xffu, base);
      if (active_line(b, rise[8 * ls + l], mags[8 * ls + l], ph, tau)) held |= 1u << l;
    }
    found += __builtin_popcount(held & ((1u << min((A.n - seg * kSegCols + 31) / 32, 8)) - 1u));
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) found += __shfl_xor(found, off, 64);
  if (lane == 0) atomicAdd(&lines_found, found);
  __syncthreads();
  if (t == 0) {
    int rows = 0, cols = 0, lines = 0;
    for (int g = wa; g < A.ngroups; g += kActSide) rows += min(A.m - 256 * g, 256);
    for (int g = wb; g < A.nseg; g += kActSide) {
      cols += min(A.n - kSegCols * g, kSegCols);
      lines += min((A.n - kSegCols * g + 31) / 32, 8);
    }
    const float share = (float)lines_found / ((float)rows * (float)lines);
    const float one = share < 1.f ? 1.f - exp2f(log2f(1.f - share) / 32.f) : 1.f;
    const unsigned entries = (unsigned)fmaxf(one * (float)rows * (float)cols, (float)lines_found);
    atomicMax(&A.status->forecast, (u64)(unsigned)A.k << 32 | entries << kForecastBits | (unsigned)min(age, (1 << kForecastBits) - 1));
  }
}
