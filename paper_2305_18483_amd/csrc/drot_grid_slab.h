// Grid-resident solver for the group lasso: a whole call in one cooperative launch, the slabs in registers.
// Part of drot.hip (included there, inside its anonymous namespace, in this order); not a stand-alone header.

// ------------------------------------------------------------------------------------------
// The exchange of grid_resident_kernel under the arithmetic of gl_slab_kernel: a workgroup keeps a slab -- the rows of one
// class x 4 CX columns -- of X and C in registers; 32 columns (CX = 8) are the slab of the single launches, 16 (CX = 4) a half of
// one.  Sums of a row over the 32 columns, and totals of a slab, are put together from those of its SUB
// parts in the order in which the lanes of a whole slab add them up, every column is folded by its own threads as there, so
// the results are the same bits.  (But for the norms of the
// residuals where classes lie anywhere, and the stopping test with them: their squares are added up class by class.)
//
// Rows are counted class by class here (`perm`: where the rows of a class are no run), so that a slab's rows lie together in
// the exchange.
//
// What bounds it: the two hops of the exchange, 2.3 us, and the chain of a sweep: two folds over 128 row lanes through LDS
// with a scale of the group between them, five barriers.  Half slabs where the chip holds them all at once halve what a
// workgroup issues per sweep (1500 x 1000, two classes: 6.6 us per iteration with whole slabs, 5.3 with halves; with quarters,
// whose row sums are twice as many words again, 5.5).  Per iteration, in single launches and here, checked every 100: 1500 x 1000,
// two classes, 10.8 and 5.3 us (64 workgroups on 256 compute units there), rows in no order 13.6 and 5.8; 2000 x 1500, five
// classes in no order 13.7 and 7.3; 150 x 300 6.7 and 3.9; two slabs to a workgroup 1203 x 2047, five classes 13.2 and 7.1,
// 2000 x 2500, five in no order 16.8 and 9.9; 1000 x 8000, one class 22.4 and 14.0.
// No kernel here uses scratch memory (a test of the built library holds them to it), and every workgroup holds a slab: the
// planner gives none to the owner waves alone.  (A first version of this, whose workgroups could be owners only and whose
// registers spilled, gave up waiting once, at 700 x 90 with one class; why was not found, nor which of the two had a part in
// it.  The tiles of drot_grid.h have always had workgroups that are owners only.)
// ------------------------------------------------------------------------------------------
struct GridSlabArgs {
  const int* run_start;  // [nruns] first row of every class, counted class by class
  const int* run_len;    // [nruns]
  const int* rows;       // MAPPED: [nruns][row_pitch] the rows of every class
  const int* perm;       // MAPPED: [m] row by count, else null
  int row_pitch;
  int nruns;
  float thr;             // rho * mu
  int butterfly;         // slab totals added up as the fused update does, else as reduce_update_kernel
};

// grid_gather for pairs of words, at[k] and the one behind it (an address each instead of two).
template <int N, int PAUSE = 0>
__device__ __forceinline__ void grid_gather_pairs(const u64* half, u64 (&v)[2 * N], const unsigned (&at)[N], unsigned tag, int limit, bool& lost) {
  for (int polls = 1;; ++polls) {
    bool there = true;
#pragma unroll
    for (int k = 0; k < N; ++k) {
      const u64* p = reinterpret_cast<const u64*>(reinterpret_cast<const char*>(half) + at[k] * 8u);
      v[2 * k] = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      v[2 * k + 1] = __hip_atomic_load(p + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
#pragma unroll
    for (int k = 0; k < 2 * N; ++k) there = there && (unsigned)(v[k] >> 32) == tag;
    if (__builtin_amdgcn_ballot_w64(!there) == 0) return;
    if (polls >= limit) {
      lost = true;
      return;
    }
    if (PAUSE > 0) __builtin_amdgcn_s_sleep(PAUSE);
  }
}

// What a wave does in the exchange besides publishing the sums of its own slab: it owns a block of eight rows or columns,
// or, in the first workgroup, keeps theta (grid_resident_kernel has the same, with its tiles' sums).
template <int NW, int SUB, int PAUSE, bool WIDE>
struct GridOwner {
  static constexpr int kShareBlocks = 1024 / 64, kSB = kShareBlocks / NW;
  static_assert(kShareBlocks % NW == 0, "the slab totals are dealt out to 1024 shares");
  bool keeper, owner, own_rows, entry_exists;
  int blk, at_row, nparts;  // at_row: the owned entry's row (or column) in memory
  unsigned part_word;
  double state, target, theta, sum_p;

  __device__ __forceinline__ void init(const GridArgs& A, const int* perm, int wave, int lane) {
    keeper = blockIdx.x == 0;
    blk = wave * (gridDim.x - 1) + blockIdx.x - 1;  // (spread over the workgroups first)
    owner = !keeper && blk < A.nblk_m + A.nblk_n;
    own_rows = blk < A.nblk_m;
    const int bi = own_rows ? blk : blk - A.nblk_m;
    const int entry = bi * kGridBlock + (lane & 7), entries = own_rows ? A.S.m : A.S.n;
    entry_exists = owner && entry < entries;
    at_row = entry;
    state = target = 0.0;
    if (entry_exists) {
      if (own_rows && perm) at_row = perm[entry];
      state = own_rows ? A.a_in[at_row] : A.b_in[at_row];
      target = (double)(own_rows ? A.p[at_row] : A.q[at_row]);
    }
    theta = vector_load_uniform(A.theta_in);
    sum_p = vector_load_uniform(A.sum_p);
    nparts = own_rows ? A.nseg : A.ntr;
    // (a lane past the last entry asks for the last one's words)
    part_word = (own_rows ? 0u : A.col_word) + (unsigned)(bi * nparts * (own_rows ? SUB : 1) * kGridBlock) +
                (unsigned)min(lane & 7, max(entries - 1 - bi * kGridBlock, 0));
  }

  // The 16 shares of the entry's partial sums, lane 8 w + i those numbered w and w + 8 of entry i; N parts each, added first.
  // W partial sums per lane and round: one round as a rule, each is a trip.
  template <int N, int W>
  __device__ __forceinline__ double gather_parts(const GridArgs& A, const u64* __restrict__ half, unsigned tag, int lane, bool& lost) const {
    double sh[2] = {0.0, 0.0};
    for (int k0 = 0; k0 < nparts && !lost; k0 += 8 * W) {
      u64 v[W * N];
      unsigned at[W * N];
#pragma unroll
      for (int b = 0; b < W; ++b) {
        const int k = min(k0 + (lane >> 3) + 8 * b, nparts - 1);
#pragma unroll
        for (int e = 0; e < N; ++e) at[N * b + e] = part_word + (unsigned)((k * N + e) * kGridBlock);
      }
      grid_gather<W * N, PAUSE>(half, v, at, tag, A.polls, lost);
#pragma unroll
      for (int b = 0; b < W; ++b) {
        float g = grid_value(v[N * b]);
        if constexpr (N == 2) g = grid_value(v[2 * b]) + grid_value(v[2 * b + 1]);
        sh[b & 1] += k0 + (lane >> 3) + 8 * b < nparts ? (double)g : 0.0;
      }
    }
    // the 16 shares: (w + w+8), then w ^ 4, w ^ 2, w ^ 1: the tree of sum_partials_16
    return add_lane_bit3(add_lane_bit4(add_lane_bit5(sh[0] + sh[1])));
  }

  // Hop 1 for an owner wave: the partial sums of its entries, a - 2r and b - 2s published; at a check the squares, too.
  template <bool CHECK>
  __device__ __forceinline__ void own(const GridArgs& A, u64* __restrict__ half, unsigned tag, int lane, bool& lost) {
    const double total = !own_rows ? gather_parts<1, 4>(A, half, tag, lane, lost)
                         : WIDE && nparts > 32 ? gather_parts<SUB, 8>(A, half, tag, lane, lost) : gather_parts<SUB, 4>(A, half, tag, lane, lost);
    const double res = total - target;
    const u64 out = __builtin_bit_cast(u64, state - 2.0 * res);
    state = state - res;
    // (lanes 0 .. 7 the upper halves, lanes 8 .. 15 the lower ones)
    if (entry_exists && lane < 2 * kGridBlock)
      grid_store(half, A.ent_word + (unsigned)((blk * kGridBlock + (lane & 7)) * 2 + (lane >> 3)),
                 lane < kGridBlock ? (unsigned)(out >> 32) : (unsigned)out, tag);
    if constexpr (CHECK) {
      double sq = entry_exists ? res * res : 0.0;
      sq += dpp_mov_f64<0xB1, 0xF>(sq);
      sq += dpp_mov_f64<0x4E, 0xF>(sq);
      sq += dpp_mov_f64<0x141, 0xF>(sq);
      const u64 w = __builtin_bit_cast(u64, sq);
      const GridArgs& L = late_args();
      if (lane < 2) grid_store(half, L.sq_word + (unsigned)(blk * 2 + lane), lane == 0 ? (unsigned)(w >> 32) : (unsigned)w, tag);
      if (entry_exists && lane < kGridBlock) (own_rows ? L.r : L.s)[at_row] = res;
    }
  }

  // Hop 1 for the first workgroup, all its waves: the slab totals, 2 eta - theta published; at a check the test and its
  // answer.  False: a word never came.
  template <bool CHECK>
  __device__ __forceinline__ bool keep(const GridArgs& A, bool butterfly, int slabs, u64* __restrict__ half, unsigned tag, int wave,
                                       int lane, int nchecks, int it, double* red, double* sq64, int* failed) {
    bool lost = false;
    const GridArgs& L = late_args();
#pragma unroll
    for (int sb = 0; sb < kSB; ++sb) {
      double acc = 0.0;
      for (int e0 = (wave + sb * NW) * 64; e0 < slabs && !lost; e0 += 1024) {
        const int e = min(e0 + lane, slabs - 1);
        u64 v[SUB];
        unsigned at[SUB];
#pragma unroll
        for (int b = 0; b < SUB; ++b) at[b] = L.tot_word + (unsigned)(e * SUB + b);
        grid_gather<SUB, PAUSE>(half, v, at, tag, L.polls, lost);
        float g = grid_value(v[0]);
        if constexpr (SUB == 2) g += grid_value(v[1]);
        acc += e0 + lane < slabs ? (double)g : 0.0;
      }
      acc = butterfly ? butterfly_f64(acc) : wave_sum_f64(acc);
      if (lane == 0) red[wave + sb * NW] = acc;
    }
    if constexpr (CHECK) {
      for (int side = 0; side < 2; ++side) {
        const int blocks = side ? L.nblk_n : L.nblk_m;
        const unsigned word = L.sq_word + (side ? 2u * (unsigned)L.nblk_m : 0u);
        for (int b0 = 64 * wave; b0 < blocks && !lost; b0 += 64 * NW) {
          const unsigned w0 = word + 2u * (unsigned)min(b0 + lane, blocks - 1);
          u64 v[2];
          const unsigned at[2] = {w0, w0 + 1};
          grid_gather<2>(half, v, at, tag, L.polls, lost);
          double sq = b0 + lane < blocks ? grid_value(v[0], v[1]) : 0.0;
          sq += dpp_mov_f64<0xB1, 0xF>(sq);
          sq += dpp_mov_f64<0x4E, 0xF>(sq);
          sq += dpp_mov_f64<0x141, 0xF>(sq);
          if ((lane & 7) == 0 && b0 + lane < blocks) sq64[(side ? (L.nblk_m + 7) / 8 : 0) + (b0 + lane) / 8] = sq;
        }
      }
    }
    if (lost) *failed = 1;
    __syncthreads();
    if (*failed) return false;
    double sum_x = 0.0;
#pragma unroll
    for (int k = 0; k < kShareBlocks; ++k) sum_x += red[k];
    const double eta = (sum_x - sum_p) / ((double)L.S.m + (double)L.S.n);
    const u64 cst = __builtin_bit_cast(u64, 2.0 * eta - theta);
    theta = theta - eta;
    static_assert(kGridCopies == 32, "two words per copy, one wave");
    if (wave == 0)
      grid_store(half, L.cst_word + 32u * (unsigned)(lane >> 1) + (unsigned)(lane & 1), (lane & 1) ? (unsigned)cst : (unsigned)(cst >> 32), tag);
    if constexpr (CHECK) {
      if (wave == 0) {
        double norm2[2];
        for (int side = 0; side < 2; ++side) {
          const int rows64 = (L.nblk_m + 7) / 8, from = side ? rows64 : 0, count = side ? (L.nblk_n + 7) / 8 : rows64;
          double sum = 0.0;
          for (int k = 0; k < count; k += 64) sum += butterfly_f64(k + lane < count ? sq64[from + k + lane] : 0.0);
          norm2[side] = sum;
        }
        bool pass = false;
        if (lane == 0) pass = make_check<false>(L.check, nchecks, it, norm2[0], norm2[1]);
        const unsigned word = __builtin_amdgcn_ballot_w64(pass) != 0 ? 1u : 0u;
        if (lane < kGridCopies) grid_store(half, L.cst_word + 32u * (unsigned)lane + 2u, word, tag);
      }
    }
    return true;
  }
};

// CX lanes to a row, 128 row lanes, K rows per thread; TW slabs of a workgroup, one after the other.
template <int K, int CX, int TW, bool MAPPED>
__global__ __launch_bounds__(kSlabRowLanes * CX) void grid_slab_kernel(GridArgs A, GridSlabArgs B) {
  constexpr int COLS = 4 * CX, RL = kSlabRowLanes, NT = RL * CX, NW = NT / 64, SUB = kSlabLanes / CX;
  constexpr int kPos = (RL * K + NT - 1) / NT;  // rows of the class whose phi a thread fetches
  static_assert(SUB == 1 || (SUB == 2 && TW == 1), "halves of a slab go one to a workgroup");
  constexpr bool kCInLds = CX == 8;  // (16 waves of 128 registers hold no more than X)
  // (pauses between the attempts of a wait, in 64 cycles: per iteration without and with one 2000 x 1500, five shuffled classes,
  // 7.35 and 7.26 us, 400 x 3000 6.19 and 6.12; two slabs of runs 7.07 and 7.22, half slabs 5.30 and 5.30)
  constexpr int kPause = CX == 8 && (TW == 1 || MAPPED) ? 4 : 0;
  using Sum = std::conditional_t<MAPPED, double, float>;
  __shared__ f4v c_lds[kCInLds ? TW * K : 1][kCInLds ? NT : 1];
  __shared__ float red[RL][COLS];
  __shared__ Sum part[16][COLS];
  __shared__ float bcast[COLS];
  __shared__ float lds_varphi[TW][COLS];
  __shared__ float lds_phi[TW][RL * K];
  __shared__ double shares[16];
  __shared__ double sq64[kGridSquares<NW>];
  __shared__ int failed[3];
  const SweepArgs& S = A.S;
  if (*A.done) return;
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int cx = t % CX, ry = t / CX;
  const int strips = A.nseg, slabs = strips * B.nruns;  // (of 32 columns; numbered as the single launches' totals are)
  const float rho = S.rho;
  struct SlabAt {
    int run, strip, start, len, col0, cols;  // (cols 0 as well for a part past n: it publishes zeros)
  };
  auto slab_number = [&](int q) -> SlabAt {
    const int part_no = (int)blockIdx.x * TW + q, sl = part_no / SUB;
    SlabAt M{0, 0, 0, 0, 0, 0};
    if (sl < slabs) {
      M.run = sl / strips;
      M.strip = sl - M.run * strips;
      M.start = B.run_start[M.run];
      M.len = B.run_len[M.run];
      M.col0 = M.strip * kSlabCols + (SUB > 1 ? part_no % SUB * COLS : 0);
      M.cols = min(max(S.n - M.col0, 0), COLS);
    }
    return M;
  };
  // (of several slabs: kept in LDS, scalar registers run out as well)
  __shared__ int places[TW][6];
  const SlabAt only = slab_number(0);
  if (TW > 1) {
    for (int q = 0; q < TW; ++q) {
      const SlabAt M = slab_number(q);
      if (t == 0) {
        places[q][0] = M.run;
        places[q][1] = M.strip;
        places[q][2] = M.start;
        places[q][3] = M.len;
        places[q][4] = M.col0;
        places[q][5] = M.cols;
      }
    }
    __syncthreads();
  }
  auto slab_at = [&](int q) __attribute__((always_inline)) -> SlabAt {
    if constexpr (TW == 1) return only;
    auto get = [&](int k) { return __builtin_amdgcn_readfirstlane(places[q][k]); };
    return SlabAt{get(0), get(1), get(2), get(3), get(4), get(5)};
  };
  f4v x[TW][K], c[kCInLds ? 1 : TW][kCInLds ? 1 : K];
#pragma unroll
  for (int q = 0; q < TW; ++q) {
    const SlabAt M = slab_at(q);
    const int nvalid = min(max(M.col0 + M.cols - (M.col0 + cx * 4), 0), 4);
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int pos = ry + RL * k;
      x[q][k] = f4v{0.f, 0.f, 0.f, 0.f};
      f4v cc = {0.f, 0.f, 0.f, 0.f};
      if (pos < M.len) {
        const int row = MAPPED ? B.rows[(size_t)M.run * B.row_pitch + pos] : M.start + pos;
        cc = load4(S.C + (size_t)row * S.ldc + M.col0 + cx * 4, nvalid);
        if (!A.first) x[q][k] = load4(S.X + (size_t)row * S.ldx + M.col0 + cx * 4, nvalid);
      }
      if constexpr (kCInLds) c_lds[q * K + k][t] = cc;
      else c[q][k] = cc;
    }
    // (rows past the class and columns past n: the clamp zeroes them)
#pragma unroll
    for (int e = 0; e < kPos; ++e) {
      const int pos = t + NT * e;
      float ph = kMaskedOut;
      if (pos < M.len) ph = S.phi[MAPPED ? B.rows[(size_t)M.run * B.row_pitch + pos] : M.start + pos];
      if (pos < RL * K) lds_phi[q][pos] = ph;
    }
    if (t < COLS) lds_varphi[q][t] = t < M.cols ? S.varphi[M.col0 + t] : kMaskedOut;
  }
  if (t < 3) failed[t] = 0;
  // (WIDE: more than 32 strips in one round, where that needs no scratch)
  GridOwner<NW, SUB, kPause, CX == 4 || (K == 4 && TW == 1)> own;
  own.init(A, MAPPED ? B.perm : nullptr, wave, lane);
  const unsigned cst_at = A.cst_word + 32u * (blockIdx.x % kGridCopies);
  __syncthreads();

  // column sums of the slab from every thread's four columns, in threads t < COLS: the folds of gl_slab_kernel
  auto fold = [&](f4v mine) __attribute__((always_inline)) -> Sum {
    *reinterpret_cast<f4v*>(&red[ry][cx * 4]) = mine;
    __syncthreads();
    if (t < 16 * COLS) {
      const int col = t % COLS, g = t / COLS;
      float v[RL / 16];
#pragma unroll
      for (int k = 0; k < RL / 16; ++k) v[k] = red[g + 16 * k][col];
      if constexpr (MAPPED) {
#pragma unroll
        for (int h = RL / 32; h > 0; h /= 2)
#pragma unroll
          for (int k = 0; k < h; ++k) v[k] += v[k + h];
        part[g][col] = v[0];
      } else {
        float acc = 0.f;
#pragma unroll
        for (int k = 0; k < RL / 16; ++k) acc += v[k];
        part[g][col] = acc;
      }
    }
    __syncthreads();
    Sum tot = 0;
    if (t < COLS) {
      if constexpr (MAPPED) {
        double v[8];
#pragma unroll
        for (int g = 0; g < 8; ++g) v[g] = part[g][t] + part[g + 8][t];
#pragma unroll
        for (int h = 4; h > 0; h /= 2)
#pragma unroll
          for (int k = 0; k < h; ++k) v[k] += v[k + h];
        tot = v[0];
      } else {
#pragma unroll
        for (int g = 0; g < 16; ++g) tot += part[g][t];
      }
    }
    return tot;
  };

  auto sweep = [&](u64* __restrict__ half, unsigned tag) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < TW; ++q) {
      const SlabAt M = slab_at(q);
      if (M.len == 0) continue;  // (uniform: no slab there)
      const f4v vp = *reinterpret_cast<const f4v*>(&lds_varphi[q][cx * 4]);
      f4v sq = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int k = 0; k < K; ++k) {
        f4v cc;
        if constexpr (kCInLds) cc = c_lds[q * K + k][t];
        else cc = c[q][k];
        x[q][k] = xbar4(x[q][k], cc, vp + lds_phi[q][ry + RL * k], rho);
        sq += x[q][k] * x[q][k];
      }
      const float tsum = (float)fold(sq);
      if (t < COLS) bcast[t] = group_scale(tsum, B.thr, S.scale);
      __syncthreads();
      const f4v sc = *reinterpret_cast<const f4v*>(&bcast[cx * 4]);
      f4v colacc = {0.f, 0.f, 0.f, 0.f};
      // (formed anew in every sweep: kept from one to the next, the words' places would take the registers of the rows)
      int ry_now = ry;
      asm volatile("" : "+v"(ry_now));
      const unsigned row_part = SUB > 1 ? (unsigned)(M.strip * SUB + blockIdx.x % SUB) : (unsigned)M.strip;
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const f4v v = x[q][k] * sc;
        x[q][k] = v;
        float rs = (v.x + v.y) + (v.z + v.w);  // over the CX lanes of the row, as rowlanes_sum adds them
        rs += dpp_mov<0xB1, 0xF>(rs);
        rs += dpp_mov<0x4E, 0xF>(rs);
        if (CX >= 8) rs += dpp_mov<0x141, 0xF>(rs);
        colacc += v;
        const int pos = ry_now + RL * k;
        if (pos < M.len && cx == 0) {
          const unsigned s = (unsigned)(M.start + pos);
          grid_store(half, ((s >> 3) * (unsigned)(strips * SUB) + row_part) * kGridBlock + (s & 7u), (unsigned)fbits(rs), tag);
        }
      }
      const Sum cfold = fold(colacc);  // (the barrier inside orders it after every read of the first fold)
      if (t < 64) {
        const float csum = (float)cfold;
        const float tot = wave_sum(t < COLS ? csum : 0.f);
        if (t < M.cols) {
          const unsigned j = (unsigned)(M.col0 + t);
          const unsigned word = A.col_word + ((j >> 3) * (unsigned)A.ntr + (unsigned)(MAPPED ? 2 * M.run : M.run)) * kGridBlock + (j & 7u);
          grid_store(half, word, (unsigned)fbits(csum), tag);
          if constexpr (MAPPED) grid_store(half, word + kGridBlock, (unsigned)fbits((float)(cfold - (double)csum)), tag);
        }
        if (t == 0) grid_store(half, A.tot_word + (unsigned)(blockIdx.x * TW + q), (unsigned)fbits(tot), tag);
      }
      // (the next slab's fold writes `red` behind this one's last barrier, and `part` behind one of its own; `bcast` was
      // read two barriers ago)
    }
  };

  enum { kGoesOn, kPasses, kGaveUp };
  int nchecks = 0;
  auto exchange = [&](auto check_here, int it) __attribute__((always_inline)) -> int {
    constexpr bool check = decltype(check_here)::value;
    const unsigned tag = A.tag0 + (unsigned)it;
    u64* __restrict__ half = A.xchg + (size_t)(tag & 1u) * A.half_words;
    bool lost = false;
    if (own.owner) own.template own<check>(A, half, tag, lane, lost);
    if (own.keeper && !own.template keep<check>(A, B.butterfly != 0, slabs, half, tag, wave, lane, nchecks, it, shares, sq64, &failed[0]))
      return kGaveUp;
    // ---- hop 2: phi of the class's rows and varphi of the slab's columns ----
    bool wanted = wave == 0;  // (a wave whose threads stand for no row asks for nothing; the first one has the columns)
#pragma unroll
    for (int q = 0; q < TW; ++q) wanted = wanted || wave * 64 < slab_at(q).len;
    if (wanted) {
      int t_now = t;  // (as in the sweep: the places are formed anew)
      asm volatile("" : "+v"(t_now));
#pragma unroll
      for (int q = 0; q < TW; ++q) {  // (one slab after the other: registers; the next one's words have come meanwhile)
        const SlabAt M = slab_at(q);
        if (M.len == 0) continue;
        u64 v[2 * kPos + 4];
        unsigned at[kPos + 2];
#pragma unroll
        for (int p = 0; p < kPos; ++p) at[p] = A.ent_word + 2u * (unsigned)(M.start + min(t_now + NT * p, M.len - 1));
        // (a part past n asks for the last column)
        at[kPos] = A.ent_word + 2u * (unsigned)(A.nblk_m * kGridBlock + min(M.col0 + (t_now & (COLS - 1)), S.n - 1));
        at[kPos + 1] = cst_at;
        grid_gather_pairs<kPos + 2, kPause>(half, v, at, tag, A.polls, lost);
        const double cst = grid_value(v[2 * kPos + 2], v[2 * kPos + 3]);
#pragma unroll
        for (int p = 0; p < kPos; ++p)
          if (t_now + NT * p < M.len) lds_phi[q][t_now + NT * p] = (float)((grid_value(v[2 * p], v[2 * p + 1]) + cst) / (double)S.n);
        if (t_now < M.cols) lds_varphi[q][t_now] = (float)((grid_value(v[2 * kPos], v[2 * kPos + 1]) + cst) / (double)S.m);
      }
    }
    // (one wave asks for all of its workgroup, which waits at the barrier: 1500 x 1000, 500 iterations, 2.62 ms; with every wave asking
    // 2.66, with a rest behind every attempt of theirs 2.71)
    if (check && wave == 0) {
      u64 v[1];
      const unsigned at[1] = {cst_at + 2u};
      grid_gather<1, 0, true>(half, v, at, tag, A.polls, lost);
      if (!lost && (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)v[0]) != 0) failed[2] = 1;
    }
    if (lost) failed[1] = 1;
    __syncthreads();
    return failed[1] ? kGaveUp : check && failed[2] ? kPasses : kGoesOn;
  };

  int result = kGoesOn, it = 0, next_check = A.check.first;
  for (;; ++it) {
    const unsigned tag = A.tag0 + (unsigned)it;
    sweep(A.xchg + (size_t)(tag & 1u) * A.half_words, tag);
    if (it != next_check) {
      result = exchange(std::false_type{}, it);
      if (result != kGoesOn) break;
    } else {
      result = exchange(std::true_type{}, it);
      if (result != kGoesOn || it == A.iters - 1) break;
      ++nchecks;
      const GridArgs& L = late_args();
      next_check = min(it + L.check.every, L.iters - 1);
    }
  }

  if (failed[0] || failed[1]) {  // (a workgroup that is not on the chip, or a word lost)
    if (t == 0) {
      A.status->broken = 1;
      __threadfence();
      *A.done = 1;
    }
    return;
  }

  // ---- leave the plan and the state after the last update in memory (no sums: the planner knows) ----
  const GridArgs& E = late_args();
  int ry_now = ry;
  asm volatile("" : "+v"(ry_now));
#pragma unroll
  for (int q = 0; q < TW; ++q) {
    const SlabAt M = slab_at(q);
    const int nvalid = min(max(M.cols - cx * 4, 0), 4);
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int pos = ry_now + RL * k;
      if (pos < M.len) {
        const int row = MAPPED ? B.rows[(size_t)M.run * B.row_pitch + pos] : M.start + pos;
        store4(E.S.X + (size_t)row * E.S.ldx + M.col0 + cx * 4, x[q][k], nvalid);
      }
    }
    if (M.len > 0 && M.col0 == 0) {
#pragma unroll
      for (int e = 0; e < kPos; ++e) {
        const int pos = t + NT * e;
        if (pos < M.len) E.phi_out[MAPPED ? B.rows[(size_t)M.run * B.row_pitch + pos] : M.start + pos] = lds_phi[q][pos];
      }
    }
    if (M.len > 0 && M.run == 0 && t < M.cols) E.varphi_out[M.col0 + t] = lds_varphi[q][t];
  }
  const bool alt = (it & 1) == 0;  // (behind an odd number of updates)
  if (own.entry_exists && lane < kGridBlock)
    (own.own_rows ? (alt ? E.a_alt : E.a_in) : (alt ? E.b_alt : E.b_in))[own.at_row] = own.state;
  if (own.keeper && t == 0) *(alt ? E.theta_alt : E.theta_in) = own.theta;
}
