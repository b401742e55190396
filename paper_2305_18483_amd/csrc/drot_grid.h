// Grid-resident solver: a whole stretch of iterations in one cooperative launch, X and C in registers.
// Part of drot.hip (included there, inside its anonymous namespace, in this order); not a stand-alone header.

// ------------------------------------------------------------------------------------------
// Problems too large for one workgroup but whose X and C fit the register files of the whole chip (8 bytes per
// entry; 256 compute units hold 10 to 12 million entries).  One workgroup per compute unit keeps TW tiles of X and C in
// registers for all the iterations of a call, so an iteration moves no matrix at all; what is left of it is the
// arithmetic (a microsecond) and the trip of the partial sums to whoever forms eq. (6), and of phi and varphi back.
//
// That trip is what bounds the kernel.  The eight L2s are not coherent with one another, so the exchanged words go
// through the memory-side cache (relaxed agent-scope accesses), and no flag or barrier stands beside them: every word
// is 64 bits, half of them payload and half the number of the iteration they belong to, and a reader asks for the word
// until the number is the one it waits for.  Two hops per iteration: (1) every workgroup publishes the row sums, column
// sums and totals of its tiles; the owner of a block of eight rows or columns (a wave) gathers the partial sums of its
// entries, the first workgroup the tile totals, which give eta; (2) the owners publish a - 2r and b - 2s, the first
// workgroup 2 eta - theta (in several copies: every workgroup asks for it), and everybody fetches the ones of their
// tiles and forms phi and varphi.  Measured with an empty sweep: 2.5 us per iteration for 32 workgroups, 2.9 for 128,
// 4.3 for 256; one hop (everybody gathers all the partial sums they need) costs 4.3 to 8.8 us because of its traffic,
// and a counter-based barrier across the grid 8 to 14 us.  (With the tile totals fetched by every workgroup instead of
// one, hop 1 alone took 2.9 to 3.6 us instead of 1.7 to 2.0 at 2000 x 2000: hundreds of readers of the same lines queue up.)
//
// Measured on MI355X, per iteration, before (single launches) and now: 500 x 500 6.7 -> 3.1 us (0.55 sweep, 0.2 fold
// and publish, 1.0 hop 1, 1.2 hop 2), 1000 x 1000 6.7 -> 3.0, 2048 x 3072 22.6 -> 6.4, 2999 x 3307 18.6 -> 7.8 (2.4 of
// it the sweep: 8 operations for each of the 49000 entries of a compute unit).
//
// The launch runs on through the residual checks (GridArgs::check).  At a check the owners publish the squared residuals of
// their entries, too, the first workgroup adds them up, tests, and sends the answer behind 2 eta - theta: one hop more,
// 2 us.  Ending the launch at every check instead (the launch, fetching X and C, the last vector update, norms, status and
// its copy to the host) cost 40 us: 1000 x 1000, 1000 sweeps checked every 100 3.48 -> 3.11 ms, every 10 7.18 -> 3.39.
// The sweeps without a check are a loop of their own, without its branches; its registers are the kernel's, though (kFull).
//
// Two halves of the exchange buffers, used in turn, are enough: a word of iteration k is overwritten in iteration
// k + 2, whose sweep needs the 2 eta - theta of k + 1, which needs the total of every tile of k + 1, which every
// workgroup publishes after it has read all it needs of k.  (A workgroup without tiles, which only owns blocks, forms
// nothing of k + 2 before that either, and nobody gets past k + 1 without what it publishes there; the answer of a check that
// it still has to read is overwritten at a later check only, for which the first workgroup needs its squared residuals.)  The words of eight entries and one partial sum lie together
// (64 bytes), the partial sums of a block of eight one after the other: a wave reads 512 contiguous bytes per load.
//
// The arithmetic and its order are those of the launches this kernel stands for, so that the results are the same
// bits: 32-row tiles of 16 waves x 2 rows (small problems, update fused into the sweep) or 64-row tiles of 8 waves x 8
// rows (the sweeps that skip zero row segments).  The last sweep leaves X, its partial sums and the state after its vector
// update in memory as those launches do.
//
// The workgroups wait for one another, so they must all be on the chip: a cooperative launch, at most one workgroup per
// compute unit.  Every wait is bounded: a word that has not come after GridArgs::polls attempts (2^25 as a rule, about half a
// minute) ends the kernel with the `broken` mark in the status block and the stop flag up.  The host goes back to single
// launches then, as it does where the launch is refused.
// This kernel has not been seen to give up of itself.  The same exchange, in a first form for the slabs of the group lasso
// (three slabs, five workgroups that only owned blocks, a kernel with spilled registers), has, and neither reading it nor
// running it on a CPU showed why (drot_grid_slab.h has the present form): a wait that runs out is taken for possible here.
// No kernel with such waits uses scratch memory any more (a test of the built library holds them to it); workgroups that only
// own blocks are left, in this kernel, for oblong problems.
// ------------------------------------------------------------------------------------------
typedef unsigned long long u64;
constexpr int kGridPolls = 1 << 25;
constexpr int kGridPollsMax = 1 << 30;
// Attempts without a rest.  A word on its way can be held up for as long as every wave on the GPU asks without one: with 4000 waves
// waiting for the answer of a check, the words of one owner out of 2500 did not reach the memory-side cache in 300000
// attempts (a third of a second), one check in ten, and in none of hundreds once the waves rest between attempts.
// So the waits for a check's answer, in which everybody waits for one workgroup, rest in every kernel (quad 1000 x 1000, ten checks, 3.06 ms
// either way).  With the others resting as well, which are over in 1 to 2 us, this kernel and the slabs' took 1 to 2.5 % longer (one
// more way out of the loops that poll), and a form of the slabs' spilled.
constexpr int kGridPatience = 32, kGridRest = 64;  // (rest: 4096 cycles, 1.7 us)
constexpr int kGridRestPolls = 3;  // ... and an attempt behind one, 2.6 us where others take 0.9, counts for three of them:
static_assert((long long)kGridPolls / kGridRestPolls * 2600 < 30000000000ll, "half a minute");
constexpr int kGridBlock = 8;    // rows or columns per owner wave
constexpr int kGridCopies = 32;  // of 2 eta - theta: workgroup b reads copy b % kGridCopies

struct GridArgs {
  SweepArgs S;            // rowpart, colpart, tilesum: where the last sweep leaves its sums
  const float* p;
  const float* q;
  double* a_in;           // eq. (6) state before the first sweep's update
  double* b_in;
  double* a_alt;          // ... and the other halves: the state after 1, 3, 5, ... updates goes there, after 2, 4, 6, ... back
  double* b_alt;          // to where it came from
  double* theta_in;
  double* theta_alt;
  const double* sum_p;
  DeviceStatus* status;
  int* done;
  // the exchange buffer, two halves of half_words words: [row blocks][nseg][8] row sums, [column blocks][ntr][8] column
  // sums, [groups of tiles][G] totals, [row blocks][8][2] a - 2r, [column blocks][8][2] b - 2s, [kGridCopies][16][2]
  // 2 eta - theta (each copy on a 256-byte stretch of its own; the answer of a check behind it), starting at these words of a half
  u64* xchg;
  unsigned half_words, col_word, tot_word, ent_word, cst_word;
  int nseg, ntr;          // ntr: rows of tiles (32 or 64 rows each)
  int nblk_m, nblk_n;     // blocks of eight rows, of eight columns
  int iters;              // sweeps to run (>= 2)
  int first;              // X_0 = 0: nothing to read
  unsigned tag0;          // the exchange of sweep k (counted from 0) carries the number tag0 + k; never 0
  int polls;              // attempts before a wait is given up (>= 1)
  // checks inside the launch: the last sweep's vector update is made here, too, and the state left is that of the iterate
  // of the check the launch ends at
  CheckArgs check;
  unsigned sq_word;       // [row blocks][2], [column blocks][2]: squared residuals of eight entries
  float* phi_out;
  float* varphi_out;
  double* r;
  double* s;
  PointArgs points;       // where the cost is formed from point clouds (G = kPointsColGroup), once per launch
};

// The arguments once more, fetched where they are used: what only a check or the end of the launch needs would sit in
// registers all the while otherwise, or in spilled ones.
__device__ __forceinline__ const GridArgs& late_args() {
  auto p = __builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const GridArgs*)p;
}
// Blocks of 64 rows or columns that the owner waves of 256 workgroups (the planner takes no more) stand for.
template <int NW>
constexpr int kGridSquares = 32 * NW + 2;

// a / b by the steps of the division (reciprocal refined twice, quotient, one correction), the reciprocal formed once: b is the
// same in every iteration.  The same bits for the magnitudes here (b a number of rows or columns, a and a / b far from the
// ends of the range, where the division would scale its operands; against it over 2e8 quotients, with the reciprocal off by a
// unit either way: no difference).  Per iteration 2048 x 3072 6.50 -> 6.30 us, 2999 x 3307 8.45 -> 8.34, 1000 x 1000 3.10 -> 3.05.
__device__ __forceinline__ double reciprocal_of(double b) {
  double r = __builtin_amdgcn_rcp(b);
  r = fma(fma(-b, r, 1.0), r, r);
  return fma(fma(-b, r, 1.0), r, r);
}
__device__ __forceinline__ double divide_by(double a, double b, double r) {
  const double q = a * r;
  return fma(fma(-b, q, a), r, q);
}

// (a word is addressed by its number in the buffer's half: a scalar base and 32 bits of offset)
__device__ __forceinline__ u64 grid_load(const u64* half, unsigned word) {
  return __hip_atomic_load(reinterpret_cast<const u64*>(reinterpret_cast<const char*>(half) + word * 8u), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void grid_store(u64* half, unsigned word, unsigned v, unsigned tag) {
  __hip_atomic_store(reinterpret_cast<u64*>(reinterpret_cast<char*>(half) + word * 8u), ((u64)tag << 32) | v, __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float grid_value(u64 w) { return __builtin_bit_cast(float, (int)(unsigned)w); }
__device__ __forceinline__ double grid_value(u64 hi, u64 lo) { return __builtin_bit_cast(double, (hi << 32) | (unsigned)lo); }

// The number of the lane in a form that the compiler can't lift out of a loop, nor what is made of it.
__device__ __forceinline__ int lane_again() {
  int zero = 0;
  asm volatile("" : "+v"(zero));
  return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, (unsigned)zero));
}

// Fetches the words at[0 .. N-1] until every lane has all of its own with the number `tag`.  All of them are asked for
// again together: a word waited for by itself would cost a trip to the memory-side cache each.  PAUSE: between two
// attempts, in units of 64 cycles.  REST: and a long one once kGridPatience attempts have been in vain.
template <int N, int PAUSE = 0, bool REST = false>
__device__ __forceinline__ void grid_gather(const u64* half, u64 (&v)[N], const unsigned (&at)[N], unsigned tag, int limit, bool& lost) {
  for (int polls = 1;; ++polls) {
    bool there = true;
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] = grid_load(half, at[k]);
#pragma unroll
    for (int k = 0; k < N; ++k) there = there && (unsigned)(v[k] >> 32) == tag;
    if (__builtin_amdgcn_ballot_w64(!there) == 0) return;
    if (polls >= limit) {
      lost = true;
      return;
    }
    if (REST && polls >= kGridPatience) {
      __builtin_amdgcn_s_sleep(kGridRest);
      polls += kGridRestPolls - 1;
    } else if (PAUSE > 0) {
      __builtin_amdgcn_s_sleep(PAUSE);
    }
  }
}

// The sums over the 64 lanes of U values (U = 2 or 8) at once; lane l ends up with that of value l % U.  Each value's
// lanes are added up as wave_sum adds them, by the bits of the lane number from the lowest up (the same bits), but the
// lanes share the work: after the first step half of them carry one value and half the other.
template <int U>
__device__ __forceinline__ float wave_sums(const float (&s)[U], int lane) {
  static_assert(U == 2 || U == 8, "rows per wave");
  float a[U / 2];
  const bool b0 = lane & 1;
#pragma unroll
  for (int k = 0; k < U / 2; ++k) {
    const float keep = b0 ? s[2 * k + 1] : s[2 * k], send = b0 ? s[2 * k] : s[2 * k + 1];
    a[k] = keep + dpp_mov<0xB1, 0xF>(send);  // quad_perm [1,0,3,2]
  }
  float v;
  if constexpr (U == 8) {
    const bool b1 = lane & 2, b2 = lane & 4;
    float c[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const float keep = b1 ? a[2 * k + 1] : a[2 * k], send = b1 ? a[2 * k] : a[2 * k + 1];
      c[k] = keep + dpp_mov<0x4E, 0xF>(send);  // quad_perm [2,3,0,1]
    }
    const float keep = b2 ? c[1] : c[0], send = b2 ? c[0] : c[1];
    // the lane four up for the lower four of eight, four down for the upper four
    const int up = __builtin_amdgcn_update_dpp(0, fbits(send), 0x104, 0xF, 0x5, false);  // row_shl:4, banks 0 and 2
    const int other = __builtin_amdgcn_update_dpp(up, fbits(send), 0x114, 0xF, 0xA, false);  // row_shr:4, banks 1 and 3
    v = keep + __builtin_bit_cast(float, other);
  } else {
    v = a[0] + dpp_mov<0x4E, 0xF>(a[0]);
    const int up = __builtin_amdgcn_update_dpp(0, fbits(v), 0x104, 0xF, 0x5, false);
    const int other = __builtin_amdgcn_update_dpp(up, fbits(v), 0x114, 0xF, 0xA, false);
    v += __builtin_bit_cast(float, other);
  }
  v += dpp_mov<0x128, 0xF>(v);  // row_ror:8
  const auto h4 = __builtin_amdgcn_permlane16_swap((unsigned)fbits(v), (unsigned)fbits(v), false, false);
  v = __builtin_bit_cast(float, (int)h4[0]) + __builtin_bit_cast(float, (int)h4[1]);
  const auto h5 = __builtin_amdgcn_permlane32_swap((unsigned)fbits(v), (unsigned)fbits(v), false, false);
  return __builtin_bit_cast(float, (int)h5[0]) + __builtin_bit_cast(float, (int)h5[1]);
}

// Sum of a double over lanes that differ in one bit of their number, from the top bit down (the order of a butterfly);
// the steps below bit 4 rotate within a row of 16 lanes, which is the same once the higher lanes agree.
__device__ __forceinline__ double add_lane_bit5(double v) {
  const u64 b = __builtin_bit_cast(u64, v);
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)b, (unsigned)b, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
  return __builtin_bit_cast(double, ((u64)hi[0] << 32) | lo[0]) + __builtin_bit_cast(double, ((u64)hi[1] << 32) | lo[1]);
}
__device__ __forceinline__ double add_lane_bit4(double v) {
  const u64 b = __builtin_bit_cast(u64, v);
  const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)b, (unsigned)b, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
  return __builtin_bit_cast(double, ((u64)hi[0] << 32) | lo[0]) + __builtin_bit_cast(double, ((u64)hi[1] << 32) | lo[1]);
}
__device__ __forceinline__ double add_lane_bit3(double v) { return v + dpp_mov_f64<0x128, 0xF>(v); }  // row_ror:8
__device__ __forceinline__ double butterfly_f64(double v) {  // the bits of the wave part of block_sum_f64
  v = add_lane_bit3(add_lane_bit4(add_lane_bit5(v)));
  v += dpp_mov_f64<0x124, 0xF>(v);  // row_ror:4
  v += dpp_mov_f64<0x122, 0xF>(v);  // row_ror:2
  v += dpp_mov_f64<0x121, 0xF>(v);  // row_ror:1
  return v;
}

// G = kPointsColGroup: the cost comes from point clouds, formed tile by tile at the start of the launch as
// sweep_points_kernel forms it in every sweep (the same instructions per element, the same bits), and the sums are grouped as
// that kernel's are.  Calls of 300 sweeps, single launches and so: 400 x 400, d = 8 3.18 and 1.36 ms; 1000 x 1000, d = 32 3.50 and
// 1.37; 2000 x 2000 3.84 and 2.00; 2500 x 2500 4.94 and 3.31.
// NW waves; a tile is NT stacks of U rows, one stack per wave, so the workgroup works on NW / NT tiles at a time and on
// TW such sets; C of the first CL of them sits in LDS (registers are what limits the size).  G consecutive tile rows are added up in fp32 before anything else (1, or kColGroup for 64-row tiles).
template <int NW, int NT, int U, int TW, int CL, int G>
__global__ __launch_bounds__(64 * NW) void grid_resident_kernel(GridArgs A) {
  constexpr int kRows = NT * U;          // rows of a tile
  constexpr int kSide = NW / NT;         // tiles side by side in the workgroup's waves
  constexpr int kTiles = kSide * TW;     // tiles of the workgroup
  constexpr int kShareBlocks = 1024 / 64, kSB = kShareBlocks / NW;  // the tile totals are dealt out to 1024 shares
  // Pauses between the attempts of a wait leave the memory-side cache to the words on their way.  Where the workgroups differ
  // in the tiles they hold, or a tile takes long, the waits are long: per iteration without a pause, with 64, 128, 256 and 512
  // cycles 2048 x 2048 (two tiles) 4.96, 4.89, 4.88, 4.85, 4.92 us, 2048 x 3072 (three) 6.55, 6.48, 6.43, 6.37, 6.35,
  // 2999 x 3307 (64 rows) 8.50, 8.33, 8.33, 8.34, 8.38, 2100 x 1800 6.10, 5.94, 5.96, 5.94, 6.01.  With one tile of 32 rows
  // each attempt is of use (1000 x 1000 3.11, 3.13, 3.17, 3.24, 3.41), and with four or five it makes no difference.
  constexpr int kPause = U == 8 ? 2 : TW == 2 || TW == 3 ? 4 : 0;
  static_assert(kRows <= 64 && NW % NT == 0 && kShareBlocks % NW == 0, "layout");
  __shared__ f4v c_lds[CL > 0 ? CL : 1][NW * U][64];
  __shared__ float cs[kTiles][NT][kSegCols];  // column sums of a wave's rows
  __shared__ float lds_varphi[kTiles][kSegCols];
  __shared__ float lds_phi[kTiles][kRows];
  __shared__ float lds_row[kTiles][kRows];
  __shared__ float wt[kTiles][NT];            // totals of a wave's rows
  // (inner products of a tile: in the column sums' place where that is large enough)
  constexpr bool kPoints = G == kPointsColGroup;
  static_assert(!kPoints || (NW == kSweepWaves && NT == kSweepWaves && U == kSweepRows), "tiles of sweep_points_kernel");
  constexpr bool kDotsApart = kPoints && kTiles * NT * kSegCols < kTileRows * kDotPitch;
  __shared__ float dots_apart[kDotsApart ? kTileRows * kDotPitch : 1];
  __shared__ double red[kShareBlocks];
  // kFull: X and C fill the registers.  What a check, the end of the launch and the keeper alone need (constants, addresses) is
  // formed there then; the compiler keeps it in registers, or in scratch memory, through all the sweeps otherwise.  kTight: the
  // lane numbers of the exchange, too, and theta lies in LDS.  Registers without the checks, with them, and so (in brackets
  // the bytes of scratch memory): one tile 85, 116, 116; two 104, 128 (24), 120; three 124, 128 (24), 111; four 128 (28),
  // 128 (88), 108; five 128 (96), 128 (140), 121; three of 64 rows 249, 256 (56), 246; point clouds of two to five tiles
  // 128 (76 to 172) with the checks, 127, 114, 114, 128 so.  Times per iteration, with the scratch memory and without: 2048 x 3072
  // 6.20 and 6.21 us, 2999 x 3307 7.97 and 7.95, 2047 x 5101 9.25 and 9.36; point clouds 1400 x 1400 5.18 and 5.08, 3000 x 3300
  // 12.55 and 12.45.
  constexpr bool kFull = U == 8 ? TW == 3 : TW > 1, kTight = U == 2 && (TW >= 4 || (kPoints && TW >= 3));
  __shared__ double theta_sum[2];  // (kTight, the first workgroup: theta, 1^T p)
  __shared__ double sq64[kGridSquares<NW>];  // checks: squared residuals of 64 entries each
  __shared__ int failed[2];  // a word that never came: among the tile totals; among the others
  const SweepArgs& S = A.S;
  if (*A.done) return;
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int side = wave / NT, stack = wave % NT;
  const int ntiles = A.nseg * A.ntr;
  const int tile0 = blockIdx.x * kTiles;  // tiles are numbered down the columns of tiles
  const float rho = S.rho, scale = S.scale;

  // ---- fetch X, C, phi, varphi of the tiles, the eq. (6) state of the owned entries ----
  f4v x[TW][U], c[TW - CL][U];
#pragma unroll
  for (int q = 0; q < TW; ++q) {
    const int tl = tile0 + q * kSide + side;
    const int seg = tl / A.ntr, tr = tl - seg * A.ntr;
    const int j0 = seg * kSegCols + lane * 4;
    const int r0 = tr * kRows + stack * U;
    float (*dots)[kDotPitch] = nullptr;
    f4v ysq = {0.f, 0.f, 0.f, 0.f};
    if constexpr (kPoints) {
      dots = reinterpret_cast<float (*)[kDotPitch]>(kDotsApart ? dots_apart : &cs[0][0][0]);
      if (q > 0) __syncthreads();  // (the last tile's have been read)
      if (tl < ntiles) {           // (the same for the whole workgroup)
        points_tile(A.points, dots, lane, wave, seg, tr, S.m);
        ysq = load4(A.points.xt_sq + j0, min(max(S.n - j0, 0), 4));
      }
      __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      x[q][u] = f4v{0.f, 0.f, 0.f, 0.f};
      f4v cc = {0.f, 0.f, 0.f, 0.f};
      if (tl < ntiles && r0 + u < S.m && j0 < S.n_mem) {
        if constexpr (!kPoints) cc = *reinterpret_cast<const f4v*>(S.C + (size_t)(r0 + u) * S.ldc + j0);
        if (!A.first) x[q][u] = *reinterpret_cast<const f4v*>(S.X + (size_t)(r0 + u) * S.ldx + j0);
      }
      if constexpr (kPoints) {
        if (tl < ntiles && r0 + u < S.m)
          cc = points_cost(A.points, *reinterpret_cast<const f4v*>(&dots[stack * U + u][lane * 4]), A.points.xs_sq[r0 + u], ysq);
      }
      if constexpr (CL > 0) {
        if (q < CL) c_lds[q][wave * U + u][lane] = cc;
      }
      if (q >= CL) c[q >= CL ? q - CL : 0][u] = cc;
    }
  }
  for (int e = t; e < kTiles * kSegCols; e += 64 * NW) {
    const int tl = tile0 + e / kSegCols, j = tl / A.ntr * kSegCols + e % kSegCols;
    lds_varphi[e / kSegCols][e % kSegCols] = (tl < ntiles && j < S.n) ? S.varphi[j] : kMaskedOut;
  }
  for (int e = t; e < kTiles * kRows; e += 64 * NW) {
    const int tl = tile0 + e / kRows, i = tl % A.ntr * kRows + e % kRows;
    lds_phi[e / kRows][e % kRows] = (tl < ntiles && i < S.m) ? S.phi[i] : kMaskedOut;
  }
  if (t < 2) failed[t] = 0;
  // the block of eight rows or columns this wave owns (none in the first workgroup, which keeps theta): lane 8 w + i
  // forms the shares w and w + 8 of entry i
  const bool keeper = blockIdx.x == 0;
  const int nblk = A.nblk_m + A.nblk_n;
  const int blk = wave * (gridDim.x - 1) + blockIdx.x - 1;  // (spread over the workgroups first)
  const bool owner = !keeper && blk < nblk, own_rows = blk < A.nblk_m;
  const int bi = own_rows ? blk : blk - A.nblk_m;
  const int entry = bi * kGridBlock + (lane & 7), entries = own_rows ? S.m : S.n;
  const bool entry_exists = owner && entry < entries;
  double state = 0.0, target = 0.0;
  if (entry_exists) {
    state = own_rows ? A.a_in[entry] : A.b_in[entry];
    target = (double)(own_rows ? A.p[entry] : A.q[entry]);
  }
  double theta = vector_load_uniform(A.theta_in);
  double sum_p = vector_load_uniform(A.sum_p);
  if (kTight && t < 2) theta_sum[t] = t == 0 ? theta : sum_p;
  constexpr bool kRecip = U == 8 || TW <= 3;  // (beyond that the registers are worth more)
  const double recip_n = kRecip ? reciprocal_of((double)S.n) : 0.0, recip_m = kRecip ? reciprocal_of((double)S.m) : 0.0;
  auto over = [&](double v, double count, double recip) { return (float)(kRecip ? divide_by(v, count, recip) : v / count); };
  // where the words lie.  Partial sums of the owned block: per round 32 single ones (shares w, w + 8, w + 16, w + 24:
  // 16 k + share) or 16 groups of G; a lane with nothing to fetch asks for a word that somebody else needs
  // (more than 32 partial sums in one round of eight words a lane where registers allow: 2048 x 2048 4.85 -> 4.54 us per
  // iteration, 1500 x 500 3.99 -> 3.68; with three tiles 6.31 and 6.29, with five 9.55 and 9.85)
  constexpr bool kManyAtOnce = G == 1 && TW <= 2;
  constexpr int NP = G == 1 || kPoints ? 4 : 2 * G;
  const bool grouped = G > 1 && !own_rows;  // (row sums never are)
  const int nparts = own_rows ? A.nseg : A.ntr, round_parts = grouped ? 16 * G : 8 * NP;
  const unsigned part_word = (own_rows ? 0u : A.col_word) + (unsigned)(bi * nparts * kGridBlock);
  const unsigned part_lane = (unsigned)min(lane & 7, entries - 1 - bi * kGridBlock);
  // tile totals: the groups e = 64 (wave + NW sb) + lane, + 1024, ..., G words each
  const int ngroups = (A.ntr + G - 1) / G * A.nseg, last_g = (A.ntr - 1) % G;
  auto total_there = [&](int e, int b) { return b <= (e >= ngroups - A.nseg ? last_g : G - 1); };
  // what the wave publishes and what it fetches in hop 2: a quarter of a tile's columns, or its rows and total
  constexpr int kSlots = (5 * kTiles + NW - 1) / NW;
  unsigned pub_base[kSlots], ent_base[kSlots], tot_at[kSlots];  // (wave-uniform)
  int live_lanes[kSlots], slot_lds[kSlots];
  bool slot_rows[kSlots];
#pragma unroll
  for (int k = 0; k < kSlots; ++k) {
    const int s = min(wave + k * NW, 5 * kTiles - 1), lt = s / 5, part = s - lt * 5;
    const int tl = min(tile0 + lt, ntiles - 1), seg = tl / A.ntr, tr = tl - seg * A.ntr;
    slot_rows[k] = part == 4;
    slot_lds[k] = slot_rows[k] ? lt : lt * kSegCols + part * 64;
    const int first = slot_rows[k] ? tr * kRows : seg * kSegCols + part * 64;  // a multiple of eight
    const bool live = wave + k * NW < 5 * kTiles && tile0 + lt < ntiles;
    live_lanes[k] = live ? min(max((slot_rows[k] ? S.m : S.n) - first, 0), slot_rows[k] ? kRows : 64) : 0;
    pub_base[k] = slot_rows[k] ? (unsigned)((first / 8 * A.nseg + seg) * kGridBlock)
                               : A.col_word + (unsigned)((first / 8 * A.ntr + tr) * kGridBlock);
    ent_base[k] = A.ent_word + 2u * (unsigned)(slot_rows[k] ? first : A.nblk_m * kGridBlock + first);
    tot_at[k] = A.tot_word + (unsigned)((tr / G * A.nseg + seg) * G + tr % G);
  }
  int some_live = -1;  // (in the last column segment whole quarters may lie past n)
#pragma unroll
  for (int k = kSlots - 1; k >= 0; --k) some_live = live_lanes[k] > 0 ? k : some_live;
  const unsigned cst_at = A.cst_word + 32u * (blockIdx.x % kGridCopies);
  const unsigned row_lane = (unsigned)((lane >> 3) * A.nseg * kGridBlock + (lane & 7));
  const unsigned col_lane = (unsigned)((lane >> 3) * A.ntr * kGridBlock + (lane & 7));
  __syncthreads();

  auto sweep = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < TW; ++q) {
      const int lt = q * kSide + side;
      const f4v vp = *reinterpret_cast<const f4v*>(&lds_varphi[lt][lane * 4]);
      f4v colacc = {0.f, 0.f, 0.f, 0.f};
      float rs[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float ph = lds_phi[lt][stack * U + u];
        const f4v cc = q < CL ? c_lds[q < CL ? q : 0][wave * U + u][lane] : c[q >= CL ? q - CL : 0][u];
        const f4v v = xbar4(x[q][u], cc, vp + ph, rho) * scale;
        x[q][u] = v;
        colacc += v;
        rs[u] = (v.x + v.y) + (v.z + v.w);
      }
      *reinterpret_cast<f4v*>(&cs[lt][stack][lane * 4]) = colacc;
      const float row = wave_sums<U>(rs, lane);  // lane u: the sum of row u
      if (lane < U) lds_row[lt][stack * U + lane] = row;
      float wave_total = 0.f;
#pragma unroll
      for (int u = 0; u < U; ++u) wave_total += __builtin_bit_cast(float, __builtin_amdgcn_readlane(fbits(row), u));
      if (lane == 0) wt[lt][stack] = wave_total;
      if (TW * U > 8) __builtin_amdgcn_sched_barrier(0);  // (one set of tiles at a time: the registers are full of X and C)
    }
    __syncthreads();
  };
  // Publishes the sums of sweep `it` and brings phi and varphi back.  check_here: with the check that stands behind it
  // (the sweeps without one, nearly all of them, pay no branches for it).
  enum { kGoesOn, kPasses, kGaveUp };
  int nchecks = 0;
  auto exchange = [&, kept_lane = lane](auto check_here, int it) __attribute__((always_inline)) -> int {
    constexpr bool check = decltype(check_here)::value;
    const int lane = kTight ? lane_again() : kept_lane;
    auto part_index = [&](int k0, int b) {  // which partial sum the b-th word of the round from k0 on is
      return k0 + (grouped ? ((lane >> 3) + 8 * (b / G)) * G + b % G : (lane >> 3) + 8 * b);
    };
    // ---- publish the sums of the tiles ----
    const unsigned tag = A.tag0 + (unsigned)it;
    u64* __restrict__ half = A.xchg + (size_t)(tag & 1u) * A.half_words;
#pragma unroll
    for (int k = 0; k < kSlots; ++k) {
      if (live_lanes[k] == 0) continue;
      if (!slot_rows[k]) {
        const float* col = &cs[0][0][0] + (slot_lds[k] / kSegCols) * (NT * kSegCols) + slot_lds[k] % kSegCols + lane;
        float sum = 0.f;
#pragma unroll
        for (int e = 0; e < NT; ++e) sum += col[e * kSegCols];
        if (lane < live_lanes[k]) grid_store(half, pub_base[k] + col_lane, (unsigned)fbits(sum), tag);
      } else {
        float tot = 0.f;
#pragma unroll
        for (int e = 0; e < NT; ++e) tot += wt[slot_lds[k]][e];
        if (lane == 0) grid_store(half, tot_at[k], (unsigned)fbits(tot), tag);
        if (lane < live_lanes[k]) grid_store(half, pub_base[k] + row_lane, (unsigned)fbits(lds_row[slot_lds[k]][lane]), tag);
      }
    }

    // ---- hop 1: the partial sums of the owned entries, and the tile totals ----
    bool lost = false;
    if (owner) {
      double sh[2] = {0.0, 0.0};
      // (one round as a rule; more for large and for oblong problems)
      for (int k0 = 0; kPoints && grouped && k0 < nparts && !lost; k0 += round_parts) {
#pragma unroll 1
        for (int b = 0; b < 2; ++b) {  // (a group, or half of one, at a time: registers)
          float g = 0.f;
          constexpr int kPart = TW <= 3 ? G : 4;  // (1000 x 1000 4.53 us per iteration by halves, 4.03 whole)
#pragma unroll 1
          for (int e0 = 0; e0 < G; e0 += kPart) {
            u64 v[kPart];
            unsigned at[kPart];
#pragma unroll
            for (int e = 0; e < kPart; ++e) at[e] = part_word + part_lane + (unsigned)(min(part_index(k0, b * G + e0 + e), nparts - 1) * kGridBlock);
            grid_gather<kPart, kPause>(half, v, at, tag, A.polls, lost);
#pragma unroll
            for (int e = 0; e < kPart; ++e) g += part_index(k0, b * G + e0 + e) < nparts ? grid_value(v[e]) : 0.f;
          }
          const double add = part_index(k0, b * G) < nparts ? (double)g : 0.0;
          if (b == 0) sh[0] += add;
          else sh[1] += add;
        }
      }
      const bool many = kManyAtOnce && nparts > 8 * NP;
      if (many) {  // (64 partial sums in one round: a second one would be a second trip)
        for (int k0 = 0; k0 < nparts && !lost; k0 += 64) {
          u64 v[8];
          unsigned at[8];
#pragma unroll
          for (int b = 0; b < 8; ++b) at[b] = part_word + part_lane + (unsigned)(min(k0 + (lane >> 3) + 8 * b, nparts - 1) * kGridBlock);
          grid_gather<8, kPause>(half, v, at, tag, A.polls, lost);
#pragma unroll
          for (int b = 0; b < 8; ++b) sh[b & 1] += k0 + (lane >> 3) + 8 * b < nparts ? (double)grid_value(v[b]) : 0.0;
        }
      }
      for (int k0 = 0; !many && !(kPoints && grouped) && k0 < nparts && !lost; k0 += kPoints ? 8 * NP : round_parts) {
        u64 v[NP];
        unsigned at[NP];
#pragma unroll
        for (int b = 0; b < NP; ++b) at[b] = part_word + part_lane + (unsigned)(min(part_index(k0, b), nparts - 1) * kGridBlock);
        grid_gather<NP, kPause>(half, v, at, tag, A.polls, lost);
        if (kPoints || !grouped) {
#pragma unroll
          for (int b = 0; b < NP; ++b) sh[b & 1] += part_index(k0, b) < nparts ? (double)grid_value(v[b]) : 0.0;
        } else if constexpr (!kPoints) {
#pragma unroll
          for (int b = 0; b < 2; ++b) {
            float g = grid_value(v[b * G]);
#pragma unroll
            for (int e = 1; e < G; ++e) g += part_index(k0, b * G + e) < nparts ? grid_value(v[b * G + e]) : 0.f;
            sh[b] += part_index(k0, b * G) < nparts ? (double)g : 0.0;
          }
        }
      }
      // the 16 shares: (w + w+8), then w ^ 4, w ^ 2, w ^ 1: the tree of sum_partials_16
      const double total = add_lane_bit3(add_lane_bit4(add_lane_bit5(sh[0] + sh[1])));
      // eq. (6) up to the constant that is the same for all entries
      const double res = total - target;
      const u64 out = __builtin_bit_cast(u64, state - 2.0 * res);
      state = state - res;
      // (lanes 0 .. 7 the upper halves, lanes 8 .. 15 the lower ones)
      if (entry_exists && lane < 2 * kGridBlock)
        grid_store(half, A.ent_word + (unsigned)((blk * kGridBlock + (lane & 7)) * 2 + (lane >> 3)),
                   lane < kGridBlock ? (unsigned)(out >> 32) : (unsigned)out, tag);
      if (check) {
        // the residual's square over the eight entries, in the order of the first steps of wave_sum_f64
        double sq = entry_exists ? res * res : 0.0;
        sq += dpp_mov_f64<0xB1, 0xF>(sq);
        sq += dpp_mov_f64<0x4E, 0xF>(sq);
        sq += dpp_mov_f64<0x141, 0xF>(sq);
        const u64 w = __builtin_bit_cast(u64, sq);
        const GridArgs& L = late_args();
        if (lane < 2) grid_store(half, L.sq_word + (unsigned)(blk * 2 + lane), lane == 0 ? (unsigned)(w >> 32) : (unsigned)w, tag);
        if (entry_exists && lane < kGridBlock) (own_rows ? L.r : L.s)[kTight ? bi * kGridBlock + lane : entry] = res;
      }
    }
    if (keeper) {
#pragma unroll
      for (int sb = 0; sb < kSB; ++sb) {
        double acc = 0.0;
        for (int e0 = (wave + sb * NW) * 64; e0 < ngroups && !lost; e0 += 1024) {
          const int e = min(e0 + lane, ngroups - 1);
          constexpr int kAtOnce = G > 4 ? 4 : G;
          float g = 0.f;
#pragma unroll 1
          for (int b0 = 0; b0 < G; b0 += kAtOnce) {
            u64 v[kAtOnce];
            unsigned at[kAtOnce];
#pragma unroll
            for (int b = 0; b < kAtOnce; ++b) at[b] = A.tot_word + (unsigned)(e * G + (total_there(e, b0 + b) ? b0 + b : 0));
            grid_gather<kAtOnce, kPause>(half, v, at, tag, A.polls, lost);
#pragma unroll
            for (int b = 0; b < kAtOnce; ++b) g += total_there(e, b0 + b) ? grid_value(v[b]) : 0.f;
          }
          acc += e0 + lane < ngroups ? (double)g : 0.0;
        }
        acc = G == 1 ? butterfly_f64(acc) : wave_sum_f64(acc);
        if (lane == 0) red[wave + sb * NW] = acc;
      }
      if (check) {
        // the squared norms, added up as reduce_kernel, residual_norms_kernel and block_sum_f64 of 1024 threads do: over 64
        // entries first (eight words, in the order of wave_sum_f64)
        const GridArgs& L = late_args();
        for (int side_n = 0; side_n < 2; ++side_n) {
          const int blocks = side_n ? L.nblk_n : L.nblk_m;
          const unsigned word = L.sq_word + (side_n ? 2u * (unsigned)L.nblk_m : 0u);
          for (int b0 = 64 * wave; b0 < blocks && !lost; b0 += 64 * NW) {
            const unsigned w0 = word + 2u * (unsigned)min(b0 + lane, blocks - 1);
            u64 v[2];
            const unsigned at[2] = {w0, w0 + 1};
            grid_gather<2>(half, v, at, tag, A.polls, lost);
            double sq = b0 + lane < blocks ? grid_value(v[0], v[1]) : 0.0;
            sq += dpp_mov_f64<0xB1, 0xF>(sq);
            sq += dpp_mov_f64<0x4E, 0xF>(sq);
            sq += dpp_mov_f64<0x141, 0xF>(sq);
            if ((lane & 7) == 0 && b0 + lane < blocks) sq64[(side_n ? (L.nblk_m + 7) / 8 : 0) + (b0 + lane) / 8] = sq;
          }
        }
      }
      if (lost) failed[0] = 1;
      __syncthreads();
      if (failed[0]) return kGaveUp;
      if (!kTight || wave == 0) {
        int first = 0;
        if (kFull) asm volatile("" : "+v"(first));
        double sum_x = 0.0;
#pragma unroll
        for (int k = 0; k < kShareBlocks; ++k) sum_x += red[first + k];
        if (kTight) {
          theta = theta_sum[0];
          sum_p = theta_sum[1];
        }
        const double eta = (sum_x - sum_p) / ((double)S.m + (double)S.n);
        const u64 cst = __builtin_bit_cast(u64, 2.0 * eta - theta);
        theta = theta - eta;
        static_assert(kGridCopies == 32, "two words per copy, one wave");
        if (wave == 0)
          grid_store(half, A.cst_word + 32u * (unsigned)(lane >> 1) + (unsigned)(lane & 1), (lane & 1) ? (unsigned)cst : (unsigned)(cst >> 32), tag);
        if (kTight && lane == 0) theta_sum[0] = theta;
      }
      if (check) {
        const GridArgs& L = late_args();
        if (wave == 0) {  // (at most 1024 blocks of 64 entries: one to a share)
          double norm2[2];
          for (int side_n = 0; side_n < 2; ++side_n) {
            const int rows64 = (L.nblk_m + 7) / 8, from = side_n ? rows64 : 0, count = side_n ? (L.nblk_n + 7) / 8 : rows64;
            double sum = 0.0;
            for (int k = 0; k < count; k += 64) sum += butterfly_f64(k + lane < count ? sq64[from + k + lane] : 0.0);
            norm2[side_n] = sum;
          }
          bool pass = false;
          if (lane == 0) pass = make_check<kFull>(L.check, nchecks, it, norm2[0], norm2[1]);
          const unsigned word = __builtin_amdgcn_ballot_w64(pass) != 0 ? 1u : 0u;
          if (lane < kGridCopies) grid_store(half, L.cst_word + 32u * (unsigned)lane + 2u, word, tag);
        }
      }
    }

    // ---- hop 2: phi and varphi of the tiles ----
    if (some_live >= 0) {
      u64 v[2 * kSlots + 2];
      unsigned at[2 * kSlots + 2];
      at[2 * kSlots] = cst_at;
      at[2 * kSlots + 1] = cst_at + 1;
#pragma unroll
      for (int k = 0; k < kSlots; ++k) {
        // (a slot without lanes repeats another one's words)
        unsigned from = ent_base[k];
        int last = live_lanes[k] - 1;
#pragma unroll
        for (int e = 0; e < kSlots; ++e)
          if (last < 0 && e == some_live) {
            from = ent_base[e];
            last = live_lanes[e] - 1;
          }
        at[2 * k] = from + 2u * (unsigned)min(lane, last);
        at[2 * k + 1] = at[2 * k] + 1;
      }
      grid_gather<2 * kSlots + 2, kPause>(half, v, at, tag, A.polls, lost);
      const double cst = grid_value(v[2 * kSlots], v[2 * kSlots + 1]);
#pragma unroll
      for (int k = 0; k < kSlots; ++k) {
        const float dual = over(grid_value(v[2 * k], v[2 * k + 1]) + cst, slot_rows[k] ? (double)S.n : (double)S.m, slot_rows[k] ? recip_n : recip_m);
        if (lane < live_lanes[k]) {
          if (slot_rows[k]) lds_phi[slot_lds[k]][lane] = dual;
          else (&lds_varphi[0][0])[slot_lds[k] + lane] = dual;
        }
      }
    }
    int result = kGoesOn;
    if (check) {  // (whether it passes, for everybody; the word comes behind all of the iteration's others)
      u64 v[1];
      const unsigned at[1] = {cst_at + 2u};
      grid_gather<1, 0, true>(half, v, at, tag, A.polls, lost);
      if (!lost && (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)v[0]) != 0) result = kPasses;
    }
    if (lost) failed[1] = 1;
    __syncthreads();
    return failed[1] ? kGaveUp : result;
  };
  int result = kGoesOn, it = 0;
  int upto = A.check.first;  // (the next sweep with a check behind it)
  for (;;) {
    for (; it < upto && result == kGoesOn; ++it) {
      sweep();
      result = exchange(std::false_type{}, it);
    }
    if (result != kGoesOn) break;
    sweep();
    result = exchange(std::true_type{}, it);
    if (result != kGoesOn || it == A.iters - 1) break;
    ++nchecks;
    ++it;
    const GridArgs& L = late_args();
    upto = min(it - 1 + L.check.every, L.iters - 1);
  }
  if (failed[0] || failed[1]) {  // (a workgroup that is not on the chip, or a word lost)
    if (t == 0) {
      A.status->broken = 1;
      __threadfence();
      *A.done = 1;
    }
    return;
  }

  const GridArgs& E = late_args();
  // ---- leave the last sweep's plan and sums, and the state after the last update, in memory ----
  const int lane_now = kFull ? lane_again() : lane;
#pragma unroll
  for (int q = 0; q < TW; ++q) {
    const int tl = tile0 + q * kSide + side;
    const int seg = tl / A.ntr, tr = tl - seg * A.ntr;
    const int j0 = seg * kSegCols + lane_now * 4;
    const int r0 = tr * kRows + stack * U;
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (tl < ntiles && r0 + u < S.m && j0 < S.n_mem) *reinterpret_cast<f4v*>(E.S.X + (size_t)(r0 + u) * E.S.ldx + j0) = x[q][u];
  }
  for (int s = wave; s < 5 * kTiles; s += NW) {
    const int lt = s / 5, part = s - lt * 5;
    const int tl = tile0 + lt;
    if (tl >= ntiles) break;
    const int seg = tl / A.ntr, tr = tl - seg * A.ntr;
    if (part < 4) {
      const int cc = part * 64 + lane_now, j = seg * kSegCols + cc;
      float sum = 0.f;
#pragma unroll
      for (int k = 0; k < NT; ++k) sum += cs[lt][k][cc];
      if (j < S.n) {
        E.S.colpart[(size_t)tr * E.S.np + j] = sum;
        if (tr == 0) E.varphi_out[j] = lds_varphi[lt][cc];
      }
    } else {
      const int i = tr * kRows + lane_now;
      if (lane_now < kRows && i < S.m) {
        E.S.rowpart[(size_t)seg * E.S.mp + i] = lds_row[lt][lane_now];
        if (seg == 0) E.phi_out[i] = lds_phi[lt][lane_now];
      }
      float tot = 0.f;
#pragma unroll
      for (int k = 0; k < NT; ++k) tot += wt[lt][k];
      if (lane_now == 0) E.S.tilesum[(size_t)tr * A.nseg + seg] = tot;
    }
  }
  const bool alt = (it & 1) == 0;  // (behind an odd number of updates)
  if (entry_exists && lane_now < kGridBlock) (own_rows ? (alt ? E.a_alt : E.a_in) : (alt ? E.b_alt : E.b_in))[kTight ? bi * kGridBlock + lane_now : entry] = state;
  if (keeper && wave == 0 && lane_now == 0) *(alt ? E.theta_alt : E.theta_in) = kTight ? theta_sum[0] : theta;
}
