// Screened sweeps: the 8-wave tile and the lean one-wave-per-tile kernel.
// Part of drot.hip (included there, inside its anonymous namespace, in this order); not a stand-alone header.

// ------------------------------------------------------------------------------------------
// Screened sweep (large sparse problems).  On top of skipping the all-zero row segments of X, most
// of C need not be read either: a row segment with x = 0 comes out as zero again whenever
// phi_i + varphi_j - rho C_ij <= 0 for its 256 columns, and that can be certified from three numbers.
// A "refresh" sweep, which reads all of C, records for every row segment, with t_j = varphi0_j - rho C_ij
// (varphi0 = the varphi of that sweep),
//     M  = max_j t_j,   j* = a column that attains it,   M2 = max_{j != j*} t_j.
// Later sweeps form, per column segment, the drifts d_j = varphi_j - varphi0_j and delta = max_j d_j.
// Column j* has moved by exactly d_j*, every other column by at most delta, so
//     max_j ( phi_i + varphi_j - rho C_ij )  <=  max( M + d_j*, M2 + delta ) + phi_i  =:  S.
// If S plus a rounding margin is <= 0 and the segment of X is zero, the segment stays zero: its C is
// not read, nothing is computed, its row sum is 0.  The result is the one the plain sweep would
// produce (the margin dominates the handful of fp32 roundings between the two evaluations).  The
// row's own maximiser is what comes close to zero first, and it is tracked exactly; the second
// largest lies far enough below it, as a rule, for the cruder term to stay harmless ten times longer
// than M + delta alone would.  Still, as varphi drifts away from varphi0 fewer segments certify, so the
// bounds are renewed now and then: on the host's schedule while this kernel is in use, on the
// device's own in the lean kernel below.
// Tiles: 8 waves x 8 rows x 256 columns, as the unscreened sweep for sparse plans.
// ------------------------------------------------------------------------------------------
struct ScreenArgs {
  const float* mprime_in;   // [nseg][m] M of the current epoch (screening sweeps)
  float* mprime_out;        // [nseg][m] written by a refresh sweep
  const float* varphi0;     // [n] varphi of the epoch
  int* wave_reads;          // 8-wave tiles, profiling only (else null): [workgroup][wave] row segments of C this wave read
  float* varphi0_out;       // [n] written by a refresh sweep
  int* wg_reads;            // screened point-cloud sweep: [workgroup] row segments whose cost it formed
  unsigned char* lines_out; // [nseg][m] which of the eight 128-byte lines of a row segment of X hold a nonzero, written by a refresh
  // the rest of the bounds: M2 and j* (column within the segment), read and written like mprime
  const float* m2_in;
  float* m2_out;
  const unsigned char* jstar_in;
  unsigned char* jstar_out;
  uint2* codes;             // [nseg][m] the bounds by line, as line_codes packs them (null: neither they nor the line flags are kept)
};

// The lean sweep's arguments: everything kept per row segment is read and written in place.
struct LeanArgs {
  float* X;
  const float* C;
  const float* phi;
  const float* varphi;
  const float* moved;     // [n] varphi_j - varphi0_j
  const float2* drift;    // [n / 32] per line of columns: the largest of those; its magnitude plus the largest |varphi_j|
  const int* done;
  const int* ctl;         // the control words below (kCtlRenew ...): it renews the bounds by itself
  float* rowpart;
  float* m1;              // [nseg][m] M, M2, j*, line bytes, line flags of X
  float* m2;
  unsigned char* jstar;
  uint2* codes;
  unsigned char* lines;
  float* varphi0;         // written by a renewal
  float* colpart;
  float* tilesum;
  int* wg_reads;          // [workgroup] lines of C read (always written)
  int* wg_waste;          // [workgroup] lines read in vain: zero before and after (always written)
  int m, n, ldx, ldc, n_mem, mp, np, ntiles_rows;
  float rho, scale;
  int lines_known;        // the line flags describe X
  int sums_known;         // ... or at least the row-segment sums do
};

// What a refresh records for one row segment from the wave's 256 values t (four per lane): the largest, a
// column that attains it (0 .. 255), and the largest of the others.  All three wave-uniform.
__device__ __forceinline__ void segment_top2(f4v t, int lane, float& M, int& jstar, float& M2) {
  // within the lane: largest, its position, largest of the other three
  const float hi01 = fmaxf(t.x, t.y), lo01 = fminf(t.x, t.y), hi23 = fmaxf(t.z, t.w), lo23 = fminf(t.z, t.w);
  const float m1 = fmaxf(hi01, hi23);
  const int a = m1 == t.x ? 0 : m1 == t.y ? 1 : m1 == t.z ? 2 : 3;
  const float m2l = a < 2 ? fmaxf(lo01, hi23) : fmaxf(hi01, lo23);
  M = wave_max(m1);
  const unsigned long long hit = __builtin_amdgcn_ballot_w64(m1 == M);
  const int L = hit ? (int)__builtin_ctzll(hit) : 0;
  jstar = L * 4 + __builtin_amdgcn_readlane(a, L);
  M2 = wave_max(lane == L ? m2l : m1);  // (a tie between lanes leaves M2 = M)
}

// Largest of the four values of a lane over the eight lanes that hold one line.
__device__ __forceinline__ float line_max(f4v t) {
  float v = fmaxf(fmaxf(t.x, t.y), fmaxf(t.z, t.w));
  v = fmaxf(v, dpp_mov<0xB1, 0xF>(v));
  v = fmaxf(v, dpp_mov<0x4E, 0xF>(v));
  return fmaxf(v, dpp_mov<0x141, 0xF>(v));  // row_half_mirror
}

// The eight bytes of one row segment, packed by the wave that holds its 256 values t (all lanes get them).
__device__ __forceinline__ void line_codes(f4v t, float M, int base, unsigned& lo, unsigned& hi) {
  const int code = (int)line_code(M == -INFINITY ? 0.f : M - line_max(t), base);
  lo = hi = 0;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    lo |= (unsigned)__builtin_amdgcn_readlane(code, 8 * g) << (8 * g);
    hi |= (unsigned)__builtin_amdgcn_readlane(code, 32 + 8 * g) << (8 * g);
  }
}

// The lines of a row segment from the lanes that hold a nonzero: bit g, any of lanes 8g .. 8g+7.
__device__ __forceinline__ unsigned lines_of(unsigned long long lanes) {
  lanes |= lanes >> 4;
  lanes |= lanes >> 2;
  lanes |= lanes >> 1;
  return (unsigned)(((lanes & 0x0101010101010101ull) * 0x0102040810204080ull) >> 56);
}

// The certificate, evaluated by lane l for row l from its record (m1, m2, j) and phi_l; dv: this lane's
// four drifts; delta, mag: their maximum over the wave and the largest |varphi_j| of the segment.  Each of
// the two candidates carries its own margin, 8 units in the last place of its terms (2^-21), which covers
// the roundings of the record, of the drifts, of the sums here and of the sweep's own evaluation (each at
// most half a unit of a term no larger than these); so does the last sum.
__device__ __forceinline__ bool certified_zero(float m1, float m2, unsigned j, f4v dv, float delta, float mag, float ph) {
  constexpr float kEps = 4.76837158e-7f;  // 2^-21
  // the drift of the row's own maximiser: lane j / 4, component j % 4
  const int src = (int)(j >> 2) << 2;
  const float d0 = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(src, fbits(dv.x)));
  const float d1 = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(src, fbits(dv.y)));
  const float d2 = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(src, fbits(dv.z)));
  const float d3 = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(src, fbits(dv.w)));
  const unsigned c = j & 3u;
  const float dstar = c == 0 ? d0 : c == 1 ? d1 : c == 2 ? d2 : d3;
  if (m1 == -INFINITY) return true;  // every pair of the segment is forbidden
  const float s1 = (m1 + dstar) + kEps * (fabsf(m1) + fabsf(dstar));
  const float s2 = m2 == -INFINITY ? -INFINITY : (m2 + delta) + kEps * (fabsf(m2) + fabsf(delta));
  const float bound = fmaxf(s1, s2) + ph;
  return bound + kEps * (fabsf(ph) + mag + fabsf(bound)) <= 0.f;
}

// Control words of the lean sweep's own refresh schedule (device memory; a Renewal, brought up to date by
// reduce_update_kernel after every lean sweep).
constexpr int kCtlRenew = 0, kCtlSince = 1, kCtlPaid = 2;
constexpr int kCtlWords = 4;

constexpr int kScreenRows = 8, kScreenWaves = 8;

template <bool EDGE, bool NT, bool REFRESH>
__device__ __forceinline__ void screened_body(const SweepArgs& A, const ScreenArgs& SC, int lane, int wave, int seg, int tr) {
  constexpr int U = kScreenRows, NW = kScreenWaves;
  const int j0 = seg * kSegCols + lane * 4;
  const int nmem = EDGE ? min(max(A.n_mem - j0, 0), 4) : 4;
  const int r0 = (tr * NW + wave) * U;
  const int nrows = min(max(A.m - r0, 0), U);
  const size_t ldx = (size_t)A.ldx, ldc = (size_t)A.ldc;
  const float* __restrict__ Cp = A.C + (size_t)r0 * ldc + j0;
  float* __restrict__ Xp = A.X + (size_t)r0 * ldx + j0;
  const float rho = A.rho, scale = A.scale;
  const size_t ridx = (size_t)seg * A.mp + r0 + lane;  // this lane's row in the per-row-segment arrays (lane < nrows)

  // lane u: old sum, phi and the bounds of row r0 + u
  const f4v vp = load_varphi_padded(A.varphi, j0);
  float prev = 0.f, ph = kMaskedOut, mpr = 0.f, mpr2 = 0.f;
  unsigned js = 0;
  if (lane < nrows) {
    prev = A.rowpart_prev ? A.rowpart_prev[ridx] : 1.f;
    ph = A.phi[r0 + lane];
    if (!REFRESH) {
      mpr = SC.mprime_in[ridx];
      mpr2 = SC.m2_in[ridx];
      js = SC.jstar_in[ridx];
    }
  }
  bool certified = lane >= nrows;  // rows past the end of the matrix: nothing to do
  if (!REFRESH) {
    const f4v vp0 = load_varphi_padded(SC.varphi0, j0);
    // drift of varphi since the epoch and its magnitude over this wave's columns (columns past n: both
    // carry the same mask value, their difference is 0; they are left out of the magnitude)
    const f4v dv = vp - vp0;
    const float d = fmaxf(fmaxf(dv.x, dv.y), fmaxf(dv.z, dv.w));
    const float a = fmaxf(fmaxf(unmasked_abs(vp.x), unmasked_abs(vp.y)), fmaxf(unmasked_abs(vp.z), unmasked_abs(vp.w)));
    const float delta = wave_max(d), mag = wave_max(a);
    const bool below = certified_zero(mpr, mpr2, js, dv, delta, mag, ph);
    certified = certified || (fbits(prev) == 0 && below);
  }
  const unsigned skipmask = (unsigned)__builtin_amdgcn_ballot_w64(certified) & 0xffu;
  const unsigned nzmask = (unsigned)__builtin_amdgcn_ballot_w64(fbits(prev) != 0) & 0xffu;
  if (REFRESH && tr == 0 && wave == 0) {
    // the first wave of every column segment stores the varphi the new bounds are recorded against
    // (here, behind the stop flag, so that bounds and epoch always belong together; nobody reads
    // varphi0 in a refresh sweep)
    *reinterpret_cast<f4u*>(SC.varphi0_out + j0) = vp;  // (past n both buffers hold the mask value)
  }

  f4v x[U], c[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    x[u] = f4v{0.f, 0.f, 0.f, 0.f};
    c[u] = f4v{0.f, 0.f, 0.f, 0.f};
  }
  if (nrows == U && skipmask == 0) {
    // nothing certified (always so in a refresh sweep, and while the plan is dense): straight-line loads
#pragma unroll
    for (int u = 0; u < U; ++u) c[u] = ld4<EDGE, NT>(Cp + u * ldc, nmem);
  } else {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (!((skipmask >> u) & 1)) c[u] = ld4<EDGE, NT>(Cp + u * ldc, nmem);
  }
  if (nzmask != 0) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if ((nzmask >> u) & 1) x[u] = ld4<EDGE, NT>(Xp + u * ldx, nmem);
  }

  f4v colacc = {0.f, 0.f, 0.f, 0.f};
  float rowkeep = 0.f, mkeep = 0.f, m2keep = 0.f, wave_total = 0.f;
  int jkeep = 0;
  uint2 ckeep = {0u, 0u};
  unsigned lkeep = 0;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    if (!((skipmask >> u) & 1)) {
      const float phu = __builtin_bit_cast(float, __builtin_amdgcn_readlane(fbits(ph), u));
      const f4v v = xbar4(x[u], c[u], vp + phu, rho) * scale;
      const bool nonzero = ((fbits(v.x) | fbits(v.y)) | (fbits(v.z) | fbits(v.w))) != 0;
      if (((nzmask >> u) & 1) || __builtin_amdgcn_ballot_w64(nonzero) != 0) st4<EDGE, NT>(Xp + u * ldx, v, nmem);
      colacc += v;
      const float tot = wave_sum((v.x + v.y) + (v.z + v.w));
      rowkeep = (lane == u) ? tot : rowkeep;
      wave_total += tot;
      if (REFRESH) {  // (columns past n carry the mask value in vp: they never win)
        const f4v t = {fmaf(-rho, c[u].x, vp.x), fmaf(-rho, c[u].y, vp.y), fmaf(-rho, c[u].z, vp.z), fmaf(-rho, c[u].w, vp.w)};
        float mm, mm2;
        int jj;
        segment_top2(t, lane, mm, jj, mm2);
        mkeep = (lane == u) ? mm : mkeep;
        m2keep = (lane == u) ? mm2 : m2keep;
        jkeep = (lane == u) ? jj : jkeep;
        if (SC.codes) {
          unsigned lo, hi;
          line_codes(t, mm, line_code_base(rho), lo, hi);
          ckeep.x = (lane == u) ? lo : ckeep.x;
          ckeep.y = (lane == u) ? hi : ckeep.y;
          const unsigned nl = lines_of(__builtin_amdgcn_ballot_w64(nonzero));
          lkeep = (lane == u) ? nl : lkeep;
        }
      }
    }
  }
  if (lane < nrows) {
    A.rowpart[ridx] = rowkeep;
    if (REFRESH) {
      SC.mprime_out[ridx] = mkeep;
      SC.m2_out[ridx] = m2keep;
      SC.jstar_out[ridx] = (unsigned char)jkeep;
      if (SC.codes) {  // (the lean sweep follows: the lines that hold something)
        SC.codes[ridx] = ckeep;
        SC.lines_out[ridx] = (unsigned char)lkeep;
      }
    }
  }
  if (SC.wave_reads && lane == 0)
    SC.wave_reads[(tr * gridDim.x + seg) * NW + wave] = __builtin_popcount(~skipmask & 0xffu);
  write_col_partials<NW>(colacc, lane, wave, seg, tr, A.n, A.np, A.colpart);
  write_tile_total<NW>(wave_total, lane, wave, seg, tr, A.tilesum);
}

// Profiling: total of `count` per-wave or per-workgroup counters (ints or doubles) into one double.
template <typename T>
__global__ __launch_bounds__(1024) void sum_counts_kernel(const T* __restrict__ counts, int count, double* out) {
  __shared__ double red[1024 / 64];
  double acc = 0.0;
  for (int e = threadIdx.x; e < count; e += 1024) acc += (double)counts[e];
  const double tot = block_sum_f64(acc, red);
  if (threadIdx.x == 0) *out = tot;
}

template <bool NT, bool REFRESH>
__global__ __launch_bounds__(64 * kSweepWaves) void screened_sweep_kernel(SweepArgs A, ScreenArgs SC) {
  if (*A.done) return;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int seg = blockIdx.x, tr = blockIdx.y;
  if ((seg + 1) * kSegCols <= A.n) screened_body<false, NT, REFRESH>(A, SC, lane, wave, seg, tr);
  else screened_body<true, NT, REFRESH>(A, SC, lane, wave, seg, tr);
}

// The screened sweep by lines: one wave owns a whole 64 x 256 tile, lane l holding the line flags, phi and the bounds of
// row l.  It certifies all 64 row segments at once; of the ones left over it looks at the 128-byte lines, eight row
// segments at a time: lane 8 g + k decides whether line g of the k-th of them holds something or may come to.  The eight
// lanes of a line (8 g .. 8 g + 7, one 128-bit access each) then walk through the rows whose line g is left, every line
// at its own pace: a plan has about one nonzero line per nonzero row segment, so a step of the wave takes up to eight
// (row, line) pairs of different rows, and of C and X alike only those lines move.
// The waves of a workgroup work on their own and meet once, at the end (screened_lean_kernel).  The same bits as the
// 8-wave tiles: a row segment's sum is that of its lines' sums in the tree of wave_sum (through LDS; a line left out is
// an exact zero); a column's rows are added in ascending order, the rows of every group of eight first.
//
// Why by lines: a cold start's plan thins out fast (at 20000 x 20000 after 8, 16, 24, 32 sweeps 95 % / 4.8 %, 88 % /
// 0.8 %, 52 % / 0.3 %, 30 % / 0.14 % of the row segments / entries are nonzero), and so do its lines (79 %, 23 %, 8.8 %,
// 4.4 %), while the row segments of 1 KiB hardly do.
// Measured at 20000 x 20000 (quadratic term), us per sweep in row segments (8-wave tiles up to sweep 96, then one wave per
// tile walking row segments) and by lines: sweep 10 822 / 670, 16 765 / 280, 24 470 / 90, 32 270 / 51, 64 150 / 22,
// 96 135 / 20, from 150 on 18 / 18; 500 sweeps of a cold start 42.2 -> 24.6 ms.  In the steady state the kernel reads a
// tenth of the lines it did, and is bound by what a wave waits for: three rounds of waves, each of two trips to memory.
// The lines are fetched and stored cacheable, whatever the size: what is left of a plan is a few megabytes that the next
// sweep fetches again (non-temporal: 25.0 instead of 24.6 ms; 8191 x 8191, 31 % of the lines left: 59 instead of 50 us).
struct LeanTile {
  float total;  // the tile's total, added up as the 8-wave tiles do
  int reads;    // lines of C read
  int waste;    // ... whose line of X was zero before and is zero after (a renewal: is zero after)
};

// Lane u: the lines of row u's segment of X that hold a nonzero (bit g: columns 32g .. 32g+31).  From the flags the
// previous lean sweep, or the sweep that recorded the bounds, left; after any other sweep from the row sums (nonzero
// sum: any line may hold something).
__device__ __forceinline__ unsigned lean_flags(const LeanArgs& A, size_t tile, unsigned ul) {
  if (A.lines_known) return (A.lines + tile)[ul];
  return (!A.sums_known || fbits((A.rowpart + tile)[ul]) != 0) ? 0xffu : 0u;
}

// New bounds (the vector update before this sweep has asked for them): every row segment is processed, four columns to a
// lane, and its M, M2, j* and line bytes are recorded against the varphi of now.
template <bool EDGE>
__device__ __forceinline__ f4v lean_renew(const LeanArgs& A, int lane, int seg, int tr, LeanTile& out) {
  const int j0 = seg * kSegCols + lane * 4;
  const int nmem = EDGE ? min(max(A.n_mem - j0, 0), 4) : 4;
  const int r0 = tr * 64, nrows = min(A.m - r0, 64);
  const size_t ldx = (size_t)A.ldx, ldc = (size_t)A.ldc;
  const float* __restrict__ Cp = A.C + (size_t)r0 * ldc + j0;
  float* __restrict__ Xp = A.X + (size_t)r0 * ldx + j0;
  const float rho = A.rho, scale = A.scale;
  // (the wave's row segments: a scalar place in the arrays plus the lane)
  const size_t tile = (size_t)seg * (size_t)A.mp + (size_t)r0;
  const unsigned ul = (unsigned)lane;
  const f4v vp = load_varphi_padded(A.varphi + seg * kSegCols, 4 * lane);
  float ph = 0.f;
  unsigned oldlines = 0;
  if (lane < nrows) {
    ph = (A.phi + r0)[ul];
    oldlines = lean_flags(A, tile, ul);
  }
  const int base = line_code_base(rho);
  const unsigned myline = (unsigned)lane >> 3;
  float mkeep = 0.f, m2keep = 0.f, rowkeep = 0.f, tile_tot = 0.f, group_tot = 0.f;
  int jkeep = 0;
  uint2 ckeep = {0u, 0u};
  unsigned newlines = 0;
  int nonzero_lines = 0;
  f4v tile_acc = {0.f, 0.f, 0.f, 0.f}, group_acc = {0.f, 0.f, 0.f, 0.f};
  for (int u = 0; u < nrows; ++u) {
    const unsigned ol = (unsigned)__builtin_amdgcn_readlane((int)oldlines, u);
    f4v x = {0.f, 0.f, 0.f, 0.f};
    if ((ol >> myline) & 1) x = ld4<EDGE, false>(Xp + u * ldx, nmem);
    const f4v c = ld4<EDGE, false>(Cp + u * ldc, nmem);
    if ((u & 7) == 0 && u != 0) {
      tile_acc += group_acc;
      tile_tot += group_tot;
      group_acc = f4v{0.f, 0.f, 0.f, 0.f};
      group_tot = 0.f;
    }
    const float phu = __builtin_bit_cast(float, __builtin_amdgcn_readlane(fbits(ph), u));
    const f4v v = xbar4(x, c, vp + phu, rho) * scale;
    const bool nonzero = ((fbits(v.x) | fbits(v.y)) | (fbits(v.z) | fbits(v.w))) != 0;
    const unsigned nl = lines_of(__builtin_amdgcn_ballot_w64(nonzero));
    newlines = (lane == u) ? nl : newlines;
    nonzero_lines += __builtin_popcount(nl);
    group_acc += v;
    const float tot = wave_sum((v.x + v.y) + (v.z + v.w));
    rowkeep = (lane == u) ? tot : rowkeep;
    group_tot += tot;
    const f4v t = {fmaf(-rho, c.x, vp.x), fmaf(-rho, c.y, vp.y), fmaf(-rho, c.z, vp.z), fmaf(-rho, c.w, vp.w)};
    float mm, mm2;
    int jj;
    segment_top2(t, lane, mm, jj, mm2);
    unsigned lo, hi;
    line_codes(t, mm, base, lo, hi);
    mkeep = (lane == u) ? mm : mkeep;
    m2keep = (lane == u) ? mm2 : m2keep;
    jkeep = (lane == u) ? jj : jkeep;
    ckeep.x = (lane == u) ? lo : ckeep.x;
    ckeep.y = (lane == u) ? hi : ckeep.y;
    if (((ol | nl) >> myline) & 1) st4<EDGE, false>(Xp + u * ldx, v, nmem);
  }
  tile_acc += group_acc;
  tile_tot += group_tot;
  if (lane < nrows) {
    (A.rowpart + tile)[ul] = rowkeep;
    (A.lines + tile)[ul] = (unsigned char)newlines;
    (A.m1 + tile)[ul] = mkeep;
    (A.m2 + tile)[ul] = m2keep;
    (A.jstar + tile)[ul] = (unsigned char)jkeep;
    (A.codes + tile)[ul] = ckeep;
  }
  if (tr == 0)  // the first tile of the column segment also stores the epoch's varphi (past n both hold the mask value)
    *reinterpret_cast<f4u*>(A.varphi0 + j0) = vp;
  out.total = tile_tot;
  out.reads = nrows * ((min(A.n - seg * kSegCols, kSegCols) + 31) / 32);
  out.waste = out.reads - nonzero_lines;
  return tile_acc;
}

// In LDS, per wave: the sums of the lines of every row segment, and for the rows left over, in ascending order, what the
// eight lanes that look at their lines need of lane `row`.
struct LeanLds {
  float part[64][8];
  f4v rec[64];         // M, phi, the two words of line bytes
  unsigned row[64];    // row | line flags << 8
};
template <bool EDGE>
__device__ __forceinline__ f4v screened_lean_body(const LeanArgs& A, int lane, int seg, int tr, int& stop, LeanTile& out,
                                                  LeanLds& L) {
  const int j0 = seg * kSegCols + lane * 4;
  const int r0 = tr * 64;
  const int nrows = min(A.m - r0, 64);
  const float rho = A.rho, scale = A.scale;
  // (the wave's row segments: a scalar place in the arrays plus the lane)
  const size_t tile = (size_t)seg * (size_t)A.mp + (size_t)r0;
  const unsigned ul = (unsigned)lane, g = ul >> 3;

  const f4v vp = load_varphi_padded(A.varphi + seg * kSegCols, 4 * lane);
  // (drift and magnitude over the columns of the lane's line, formed by the vector update)
  const float2 dl = (A.drift + seg * (kSegCols / 32))[g];
  const f4v dv = *reinterpret_cast<const f4v*>(A.moved + seg * kSegCols + 4 * lane);
  float ph = kMaskedOut, mpr = 0.f, mpr2 = 0.f;
  unsigned js = 0;
  uint2 codes = {0u, 0u};
  unsigned oldlines = 0;
  if (lane < nrows) {
    ph = (A.phi + r0)[ul];
    mpr = (A.m1 + tile)[ul];
    mpr2 = (A.m2 + tile)[ul];
    js = (A.jstar + tile)[ul];
    codes = (A.codes + tile)[ul];
    oldlines = lean_flags(A, tile, ul);
  }
  // The stop flag and the renewal word travel with the loads above (asked for before them, a wave would
  // sit out their latency with nothing of its own in flight); both are tested before the first store.
  __builtin_amdgcn_sched_barrier(0);
  stop = *A.done;
  const bool renew = A.ctl[kCtlRenew] != 0;
  __builtin_amdgcn_sched_barrier(0);
  // (over the segment: the last three steps of wave_max, the eight lanes of a line agree)
  auto over_lines = [](float v) {
    v = fmaxf(v, dpp_mov<0x140, 0xF>(v));
    v = fmaxf(v, dpp_mov<0x142, 0xA>(v));
    v = fmaxf(v, dpp_mov<0x143, 0xC>(v));
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(fbits(v), 63));
  };
  const float drift = over_lines(dl.x), mag = over_lines(dl.y);
  // the drift of row u's own maximiser, looked up among the segment's 256
  float* __restrict__ lookup = &L.part[0][0];
  *reinterpret_cast<f4v*>(lookup + 4 * lane) = dv;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  const float drift1 = lookup[js];
  // (unchanged: the row segment was all zero and stays so; its sum and its line flags in memory are zeros already)
  const bool unchanged = oldlines == 0 && certified_segment(mpr, mpr2, drift1, drift, mag, ph);
  const bool left = lane < nrows && !unchanged;
  out = LeanTile{0.f, 0, 0};
  if (stop) return f4v{0.f, 0.f, 0.f, 0.f};
  if (renew) return lean_renew<EDGE>(A, lane, seg, tr, out);

  const unsigned long long todo = __builtin_amdgcn_ballot_w64(left);
  const int nleft = __builtin_popcountll(todo);
  if (nleft == 0) {
    if (!A.lines_known && lane < nrows) (A.lines + tile)[ul] = 0;
    return f4v{0.f, 0.f, 0.f, 0.f};
  }
  if (left) {
    const int at = __builtin_popcountll(todo & ((1ull << lane) - 1ull));
    L.rec[at] = f4v{mpr, ph, __builtin_bit_cast(float, (int)codes.x), __builtin_bit_cast(float, (int)codes.y)};
    L.row[at] = (unsigned)lane | oldlines << 8;
    *reinterpret_cast<f4v*>(&L.part[lane][0]) = f4v{0.f, 0.f, 0.f, 0.f};
    *reinterpret_cast<f4v*>(&L.part[lane][4]) = f4v{0.f, 0.f, 0.f, 0.f};
  }
  // (LDS serves a wave's operations in the order it issued them: no barrier, only no reordering by the compiler)
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  const int base = line_code_base(rho);
  const bool line_exists = !EDGE || j0 < A.n_mem;  // (rows are whole lines long in memory)
  const char* __restrict__ Cp = reinterpret_cast<const char*>(A.C + (size_t)r0 * (size_t)A.ldc + (size_t)seg * kSegCols);
  char* __restrict__ Xp = reinterpret_cast<char*>(A.X + (size_t)r0 * (size_t)A.ldx + (size_t)seg * kSegCols);
  const unsigned pitch_c = 4u * (unsigned)A.ldc, pitch_x = 4u * (unsigned)A.ldx;
  int reads = 0, waste = 0;
  f4v tile_acc = {0.f, 0.f, 0.f, 0.f}, group_acc = {0.f, 0.f, 0.f, 0.f};
  int group = 0;
  constexpr int kWalk = 2;  // steps fetched together
  // which lines of the row segments are left, eight at a time: lane 8 g + k decides about line g of the k-th.  Then, bit k
  // of `mine`: the k-th row segment's line g is left, for the eight lanes of line g alike
  unsigned long long mine = 0, xmine = 0;
  for (int k0 = 0; k0 < nleft; k0 += 8) {
    const int kth = k0 + (lane & 7), kc = min(kth, nleft - 1);
    const f4v rec = L.rec[kc];
    const bool held = (L.row[kc] >> (8 + g)) & 1;
    const unsigned code = ((unsigned)fbits(g < 4 ? rec.z : rec.w) >> (8 * (g & 3))) & 0xffu;
    const bool act = kth < nleft && line_exists && (held || !certified_line(rec.x, line_decode(code, base), dl.x, dl.y, rec.y));
    const unsigned long long actb = __builtin_amdgcn_ballot_w64(act), heldb = __builtin_amdgcn_ballot_w64(held);
    reads += __builtin_popcountll(actb);
    mine |= ((actb >> (lane & 56)) & 0xffull) << k0;
    xmine |= ((heldb >> (lane & 56)) & 0xffull) << k0;
  }
  while (__builtin_amdgcn_ballot_w64(mine != 0) != 0) {
    int k[kWalk];
    unsigned row[kWalk];
    float phu[kWalk];
    f4v c[kWalk], x[kWalk];
#pragma unroll
    for (int b = 0; b < kWalk; ++b) {
      k[b] = mine != 0 ? __builtin_ctzll(mine) : -1;
      mine &= mine - 1;
      row[b] = L.row[max(k[b], 0)] & 0xffu;
      phu[b] = L.rec[max(k[b], 0)].y;
    }
#pragma unroll
    for (int b = 0; b < kWalk; ++b) {
      c[b] = f4v{0.f, 0.f, 0.f, 0.f};
      x[b] = f4v{0.f, 0.f, 0.f, 0.f};
      if (k[b] >= 0) {
        c[b] = ld4<false, false>(reinterpret_cast<const float*>(Cp + (row[b] * pitch_c + 16u * (unsigned)lane)), 4);
        if ((xmine >> k[b]) & 1) x[b] = ld4<false, false>(reinterpret_cast<const float*>(Xp + (row[b] * pitch_x + 16u * (unsigned)lane)), 4);
      }
    }
    // (everything fetched has arrived from here on: said once, for all the steps, so that no step's arithmetic and
    // no store below waits again, which on this counter would mean waiting for the stores issued before it)
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    bool put[kWalk];
#pragma unroll
    for (int b = 0; b < kWalk; ++b) {
      const bool on = k[b] >= 0;
      put[b] = false;
      if (__builtin_amdgcn_ballot_w64(on) == 0) break;
      f4v v = xbar4(x[b], c[b], vp + phu[b], rho) * scale;
      if (!on) v = f4v{0.f, 0.f, 0.f, 0.f};
      if (on && (int)(row[b] >> 3) != group) {
        tile_acc += group_acc;
        group_acc = f4v{0.f, 0.f, 0.f, 0.f};
        group = (int)(row[b] >> 3);
      }
      group_acc += v;
      // the line's sum over its eight lanes (X >= 0: zero exactly when the line is); lines with a nonzero now and those
      // that held one before are written, the others are zero in memory and stay so
      float s = (v.x + v.y) + (v.z + v.w);
      s += dpp_mov<0xB1, 0xF>(s);
      s += dpp_mov<0x4E, 0xF>(s);
      s += dpp_mov<0x141, 0xF>(s);
      if (on && (lane & 7) == 0) L.part[row[b]][g] = s;
      const bool held_b = (xmine >> (k[b] & 63)) & 1;
      put[b] = on && (held_b || fbits(s) != 0);
      waste += __builtin_popcountll(__builtin_amdgcn_ballot_w64(on && !put[b] && (lane & 7) == 0));
      x[b] = v;
    }
    // the stores leave together, after the arithmetic of all the steps fetched together: the one counter for loads
    // and stores cannot tell a store still on its way from a load, so a step worked on after another one's store
    // would wait for that store to come back
#pragma unroll
    for (int b = 0; b < kWalk; ++b)
      if (put[b]) st4<false, false>(reinterpret_cast<float*>(Xp + (row[b] * pitch_x + 16u * (unsigned)lane)), x[b], 4);
  }
  tile_acc += group_acc;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  // sums of the row segments from those of their lines, in the order wave_sum adds the lanes
  float rowsum = 0.f;
  unsigned newlines = 0;
  if (left) {
    const f4v lo = *reinterpret_cast<const f4v*>(&L.part[lane][0]), hi = *reinterpret_cast<const f4v*>(&L.part[lane][4]);
    rowsum = ((lo.x + lo.y) + (lo.z + lo.w)) + ((hi.x + hi.y) + (hi.z + hi.w));
    newlines = (fbits(lo.x) != 0 ? 1u : 0u) | (fbits(lo.y) != 0 ? 2u : 0u) | (fbits(lo.z) != 0 ? 4u : 0u) |
               (fbits(lo.w) != 0 ? 8u : 0u) | (fbits(hi.x) != 0 ? 16u : 0u) | (fbits(hi.y) != 0 ? 32u : 0u) |
               (fbits(hi.z) != 0 ? 64u : 0u) | (fbits(hi.w) != 0 ? 128u : 0u);
    // (what is certified unchanged is in memory already, and so are flags that have not changed)
    (A.rowpart + tile)[ul] = rowsum;
  }
  if (lane < nrows && (!A.lines_known || newlines != oldlines)) (A.lines + tile)[ul] = (unsigned char)newlines;
  // the tile's total: the rows of every group of eight in order (lanes 0 and 8 of each row of 16 lanes), the groups in
  // order; of one or two rows, in any order
  float tot = 0.f;
  if (nleft <= 2) {
    tot = wave_sum(rowsum);
  } else {
    float gt = rowsum;
    gt += dpp_mov<0x101, 0xF>(rowsum);  // row_shl:1 .. 7
    gt += dpp_mov<0x102, 0xF>(rowsum);
    gt += dpp_mov<0x103, 0xF>(rowsum);
    gt += dpp_mov<0x104, 0xF>(rowsum);
    gt += dpp_mov<0x105, 0xF>(rowsum);
    gt += dpp_mov<0x106, 0xF>(rowsum);
    gt += dpp_mov<0x107, 0xF>(rowsum);
#pragma unroll
    for (int e = 0; e < 8; ++e) tot += __builtin_bit_cast(float, __builtin_amdgcn_readlane(fbits(gt), 8 * e));
  }
  out.total = tot;
  out.reads = reads;
  out.waste = waste;
  return tile_acc;  // column sums of the tile (columns past n: 0)
}

// Four waves per workgroup, stacked along the rows.  They work independently; each leaves its tile's column sums
// in LDS, counts itself in and ends, and the one that finds itself the last adds the four tiles' sums in the
// order tile 0, 1, 2, 3 (kColGroup in the reduction: the sweeps that store one row of column sums per 64-row
// tile are added up in that order too) and stores them.  No wave waits for another: a wave that has little to
// do gives its place on the SIMD to the next workgroup's at once.  (LDS serves a wave's operations in the order
// it issued them, so a wave's sums are in place before its count is; the count starts at zero behind the one
// barrier at the start, where nobody has anything to wait for yet.)
constexpr int kLeanWaves = 4;
constexpr int kColGroup = kLeanWaves;
static_assert(64 * kLeanWaves == kSegCols, "four columns per lane of the wave that does the final fold");

__global__ __launch_bounds__(64 * kLeanWaves, 8) void screened_lean_kernel(LeanArgs A) {
  __shared__ float fold[kLeanWaves][kSegCols];
  __shared__ float totals[kLeanWaves];
  __shared__ int nreads[kLeanWaves], nwaste[kLeanWaves];
  __shared__ LeanLds lean[kLeanWaves];
  __shared__ int arrived;
  if (threadIdx.x == 0) arrived = 0;
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int seg = blockIdx.x, tr = blockIdx.y * kLeanWaves + wave;
  f4v acc = {0.f, 0.f, 0.f, 0.f};
  LeanTile T{0.f, 0, 0};
  int stop;
  if (tr < A.ntiles_rows) {
    if ((seg + 1) * kSegCols <= A.n) acc = screened_lean_body<false>(A, lane, seg, tr, stop, T, lean[wave]);
    else acc = screened_lean_body<true>(A, lane, seg, tr, stop, T, lean[wave]);
  } else {
    stop = *A.done;
  }
  if (stop) return;
  *reinterpret_cast<f4v*>(&fold[wave][lane * 4]) = acc;
  if (lane == 0) {
    totals[wave] = T.total;
    nreads[wave] = T.reads;
    nwaste[wave] = T.waste;
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  int before = 0;
  if (lane == 0) before = __hip_atomic_fetch_add(&arrived, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  before = __builtin_amdgcn_readfirstlane(before);
  if (before != kLeanWaves - 1) return;  // (somebody is still at work: they will do the rest)
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  const int c0 = lane * 4, j0 = seg * kSegCols + c0;
  const f4v f0 = *reinterpret_cast<const f4v*>(&fold[0][c0]), f1 = *reinterpret_cast<const f4v*>(&fold[1][c0]);
  const f4v f2 = *reinterpret_cast<const f4v*>(&fold[2][c0]), f3 = *reinterpret_cast<const f4v*>(&fold[3][c0]);
  const f4v sum = ((f0 + f1) + f2) + f3;
  float* __restrict__ dst = A.colpart + (size_t)blockIdx.y * A.np + j0;
  if (j0 + 3 < A.n) {
    *reinterpret_cast<f4v*>(dst) = sum;  // (np is a multiple of 64: 16-byte aligned)
  } else {
    if (j0 < A.n) dst[0] = sum.x;
    if (j0 + 1 < A.n) dst[1] = sum.y;
    if (j0 + 2 < A.n) dst[2] = sum.z;
  }
  if (lane == 0) {
    A.tilesum[blockIdx.y * gridDim.x + seg] = ((totals[0] + totals[1]) + totals[2]) + totals[3];
    A.wg_reads[blockIdx.y * gridDim.x + seg] = (nreads[0] + nreads[1]) + (nreads[2] + nreads[3]);
    A.wg_waste[blockIdx.y * gridDim.x + seg] = (nwaste[0] + nwaste[1]) + (nwaste[2] + nwaste[3]);
  }
}
