// Single-workgroup solver for tiny problems.
// Part of drot.hip (included there, inside its anonymous namespace, in this order); not a stand-alone header.

// ------------------------------------------------------------------------------------------
// Resident solver for tiny problems (at most 128 x 256): one workgroup of 16 (or 8) waves keeps X and C in registers
// and runs on through the residual checks in one launch, so an iteration costs two workgroup barriers instead of a kernel
// launch (a launch for every check: 2.27 ms for 2000 iterations of 100 x 100, checked every 100; so 2.03).  The eq. (6) state lives in
// registers of "owner" threads: thread t < m owns row t (a_t, p_t), the column owners follow further
// up (b_j, q_j); phi and varphi travel through LDS.  Per iteration: (A) every wave updates its rows
// (first half of eq. (8) and the quadratic scaling), leaves the row sums and its column partials in
// LDS; barrier; (B) the owners form the residuals, eta, and the new phi, varphi, a, b, theta in fp64;
// barrier.  Arithmetic and precision are those of the multi-launch path (fp32 sweep and
// fp32 sums over at most 256 elements of a row resp. 8 of a column, fp64 above).
// ------------------------------------------------------------------------------------------
struct ResidentArgs {
  float* X;
  const float* C;
  const float* p;
  const float* q;
  VecState V;
  double* a_in;   // a, b before the launch; what they are after an odd number of sweeps goes to the other halves, after an
  double* b_in;   // even number back to where it came from
  double* a_alt;
  double* b_alt;
  int theta_in;   // entry of V.theta to read
  int m, n, ldx, ldc;
  float rho, scale;
  int iters;  // sweeps to run (>= 1)
  int first;  // X_0 = 0: nothing to read
  CheckArgs check;
};

constexpr int kResidentCols = 256, kResidentMaxRows = 128;

// The check behind sweep `it`, by the whole workgroup: the norms as block_sum_f64 forms them, with few registers.
template <int NW, bool HERE>
__device__ __forceinline__ bool resident_check(const ResidentArgs& A, double r2, double s2, int nchecks, int it, double* red, int* passed) {
  const int t = threadIdx.x;
  double norm2[2] = {0.0, 0.0};
#pragma unroll 1
  for (int k = 0; k < 2; ++k) {
    double v = k == 0 ? r2 : s2;
#pragma unroll 1
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    __syncthreads();
    if ((t & 63) == 0) red[t >> 6] = v;
    __syncthreads();
    if (t == 0) {
      double sum = 0.0;
#pragma unroll 1
      for (int w = 0; w < NW; ++w) sum += red[w];
      if (k == 0) norm2[0] = sum;
      else norm2[1] = sum;
    }
  }
  if (t == 0) *passed = make_check<HERE>(A.check, nchecks, it, norm2[0], norm2[1]) ? 1 : 0;
  __syncthreads();
  return *passed != 0;
}

// At most 16 rows: a row to each of 16 waves, CPL columns to a lane (n <= 64 * CPL).
constexpr int kResidentRows = 16;
template <int CPL>
__global__ __launch_bounds__(1024) void resident_kernel(ResidentArgs A) {
  constexpr int NW = kResidentRows;
  static_assert(64 * CPL <= kResidentCols, "layout");
  if (*A.V.done) return;
  __shared__ float lds_phi[kResidentMaxRows];
  __shared__ float lds_varphi[kResidentCols];
  __shared__ float lds_row[kResidentMaxRows];
  __shared__ float lds_col[NW][64 * CPL];
  __shared__ double red[NW];
  __shared__ int passed;
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int j0 = lane * CPL;
  const float rho = A.rho, scale = A.scale;

  float x[CPL], c[CPL];
#pragma unroll
  for (int e = 0; e < CPL; ++e) {
    c[e] = 0.f;
    x[e] = 0.f;
    if (wave < A.m && j0 + e < A.n) {
      c[e] = A.C[(size_t)wave * A.ldc + j0 + e];
      if (!A.first) x[e] = A.X[(size_t)wave * A.ldx + j0 + e];
    }
  }
  const bool row_owner = t < A.m;  // (m <= 128: waves 0 and 1)
  const int jc = t - 256;          // waves 4..7
  const bool col_owner = jc >= 0 && jc < A.n;
  double state = 0.0, target = 0.0;  // a_t and p_t of a row owner, b_j and q_j of a column owner
  if (row_owner) { state = A.a_in[t]; target = (double)A.p[t]; }
  if (col_owner) { state = A.b_in[jc]; target = (double)A.q[jc]; }
  double theta = A.V.theta[A.theta_in];
  const double sum_p = *A.V.sum_p;
  // (divisions by m + n, n and m as multiplications by the fp64 reciprocals: one more rounding of 1e-16)
  const double inv_mn = 1.0 / ((double)A.m + (double)A.n), inv_n = 1.0 / (double)A.n, inv_m = 1.0 / (double)A.m;
  // rows and columns that do not exist get a huge negative dual value: the clamp zeroes them
  if (t < kResidentMaxRows) {
    lds_phi[t] = row_owner ? A.V.phi[t] : kMaskedOut;
    lds_row[t] = 0.f;
  }
  if (jc >= 0 && jc < kResidentCols) lds_varphi[jc] = col_owner ? A.V.varphi[jc] : kMaskedOut;
  __syncthreads();

  const bool owner_wave = wave < 2 || (wave >= 4 && wave < 8);
  double res = 0.0;  // the owner's residual after the latest sweep
  float dual = 0.f;  // the owner's phi_t resp. varphi_j
  // (stretches of sweeps up to a check, or all of them)
  const bool checks = A.check.out != nullptr;
  int nchecks = 0, it = 0, upto = checks ? A.check.first + 1 : A.iters;
  for (;;) {
#pragma unroll 1
  for (; it < upto; ++it) {
    // (A) sweep
    float vp[CPL];
#pragma unroll
    for (int e = 0; e < CPL; ++e) vp[e] = lds_varphi[j0 + e];
    const float ph = lds_phi[wave];
    float rowacc = 0.f;
#pragma unroll
    for (int e = 0; e < CPL; ++e) {
      const float v = fmaxf(x[e] + fmaf(-rho, c[e], vp[e] + ph), 0.f) * scale;
      x[e] = v;
      rowacc += v;
      lds_col[wave][j0 + e] = v;
    }
    const float tot = wave_sum(rowacc);
    if (lane == 0) lds_row[wave] = tot;
    __syncthreads();
    // (B) eq. (6)
    if (owner_wave) {
      // 1^T X 1, the same bits in every owner wave
      const double tot = wave_sum_f64((double)lds_row[lane] + (double)lds_row[lane + 64]);
      const double eta = (tot - sum_p) * inv_mn;
      const double cst = 2.0 * eta - theta;
      theta -= eta;
      if (wave < 2) {
        res = (double)lds_row[t] - target;
        dual = (float)((state - 2.0 * res + cst) * inv_n);
        state -= res;
        if (row_owner) lds_phi[t] = dual;
      } else if (jc < 64 * CPL) {
        double sj = 0.0;
#pragma unroll
        for (int w = 0; w < NW; ++w) sj += (double)lds_col[w][jc];
        res = sj - target;
        dual = (float)((state - 2.0 * res + cst) * inv_m);
        state -= res;
        if (col_owner) lds_varphi[jc] = dual;
      }
    }
    __syncthreads();
  }
  if (!checks) break;
  if (resident_check<NW, false>(A, row_owner ? res * res : 0.0, col_owner ? res * res : 0.0, nchecks, it - 1, red, &passed) || it == A.iters) break;
  ++nchecks;
  upto = min(it + A.check.every, A.iters);
  }
  const bool alt = (it & 1) != 0;

#pragma unroll
  for (int e = 0; e < CPL; ++e)
    if (wave < A.m && j0 + e < A.n) A.X[(size_t)wave * A.ldx + j0 + e] = x[e];
  if (row_owner) {
    A.V.phi[t] = dual;
    (alt ? A.a_alt : A.a_in)[t] = state;
    A.V.r[t] = res;
  }
  if (col_owner) {
    A.V.varphi[jc] = dual;
    (alt ? A.b_alt : A.b_in)[jc] = state;
    A.V.s[jc] = res;
  }
  if (t == 0) A.V.theta[A.theta_in ^ (alt ? 1 : 0)] = theta;
  if (checks) return;  // (the last check has left the norms)
  const double r2 = block_sum_f64(row_owner ? res * res : 0.0, red);
  const double s2 = block_sum_f64(col_owner ? res * res : 0.0, red);
  if (t == 0) {
    A.V.resid[0] = r2;
    A.V.resid[1] = s2;
    A.V.resid[2] = 0.0;
    A.V.resid[3] = -1.0;
  }
}

// The general case: 16 lanes to a row, four rows to a wave at a time, R times.  What bounds an iteration is the issue of
// vector instructions, all waves on one compute unit, and then the fp64 chain of the owners (0.4 us of it all).  With 64
// lanes to a row the sums over the lanes, row after row, were a third of the instructions; over 16 lanes they are four
// steps for four rows, and the columns' sums over the wave's four rows two exchanges that fold two columns at once.
// Columns come in sets of 16 (E of them), so few are idle, and a wave skips a set of rows past m.  The column owners sit
// in waves 2 and up: for n <= 128 not on the SIMDs of the row owners.  Per iteration, 64 lanes to a row and so: 100 x 100
// 1.84 and 1.01 us, 128 x 256 2.95 and 1.81, 64 x 64 1.00 and 0.62, 10 x 10 0.56 and 0.48; without the product with a
// scale of 1 (SCALED) 0.95, 1.65, 0.61 and 0.48.
// SCALED: with a quadratic term; without one the scale is exactly 1 and its product, a seventh of the sweep, left out.
// Lane l, group g = l / 16: rows 4 (wave + NW r) + g, columns 16 e + l % 16.
template <int NW, int R, int E, bool SCALED>
__global__ __launch_bounds__(64 * NW) void resident_wide_kernel(ResidentArgs A) {
  constexpr int EQ = (E + 3) / 4;  // (64 columns to a wave of column owners)
  static_assert(4 * NW * R <= kResidentMaxRows && 16 * E <= kResidentCols && 2 + EQ <= NW, "layout");
  // The check's constants: out of the loop or formed there.  With many columns registers run out (2000 iterations 128 x 256 3.54
  // and 3.42 ms, 65 x 256 2.77 and 2.60); with few it is the schedule that changes: 100 x 16 1.41 and 1.26, 50 x 20 1.32 and
  // 1.16, 40 x 40 1.33 and 1.20, but 100 x 48 1.42 and 1.62, 50 x 80 1.48 and 1.58, 100 x 100 2.02 and 2.01.
  constexpr bool kHere = E > 8 || E == 1 || (R == 1 && E <= 3);
  if (*A.V.done) return;
  __shared__ float lds_phi[kResidentMaxRows];
  __shared__ float lds_varphi[64 * EQ];
  __shared__ float lds_row[kResidentMaxRows];
  __shared__ float lds_col[NW][64 * EQ];
  __shared__ double red[NW];
  __shared__ int passed;
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int col = lane & 15, group = lane >> 4;
  const float rho = A.rho, scale = A.scale;
  float x[R][E], c[R][E];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    // (what lies past the edges: the last row's and column's entry, and then 0)
    const int row = 4 * (wave + NW * r) + group, last_row = min(row, A.m - 1);
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const float v = A.C[last_row * A.ldc + min(16 * e + col, A.n - 1)];
      c[r][e] = row < A.m && 16 * e + col < A.n ? v : 0.f;
      x[r][e] = 0.f;
    }
    if (!A.first) {
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const float v = A.X[last_row * A.ldx + min(16 * e + col, A.n - 1)];
        x[r][e] = row < A.m && 16 * e + col < A.n ? v : 0.f;
      }
    }
  }
  const bool row_owner = t < A.m;  // (m <= 128: waves 0 and 1)
  const int jc = t - 128;          // waves 2..5: not on the row owners' SIMDs while n <= 128
  const bool col_owner = jc >= 0 && jc < A.n;
  double state = 0.0, target = 0.0;  // a_t and p_t of a row owner, b_j and q_j of a column owner
  if (row_owner) { state = A.a_in[t]; target = (double)A.p[t]; }
  if (col_owner) { state = A.b_in[jc]; target = (double)A.q[jc]; }
  double theta = A.V.theta[A.theta_in];
  const double sum_p = *A.V.sum_p;
  const double inv_mn = 1.0 / ((double)A.m + (double)A.n), inv_n = 1.0 / (double)A.n, inv_m = 1.0 / (double)A.m;
  if (t < kResidentMaxRows) {
    lds_phi[t] = row_owner ? A.V.phi[t] : kMaskedOut;
    lds_row[t] = 0.f;
  }
  if (jc >= 0 && jc < 64 * EQ) lds_varphi[jc] = col_owner ? A.V.varphi[jc] : kMaskedOut;
  __syncthreads();

  const bool owner_wave = wave < 2 + EQ;  // (64 columns to a wave)
  // (column of the lane's k-th folded sum: see the exchanges below)
  const int col_at = 16 * (((group & 1) << 1) | (group >> 1)) + col;
  double res = 0.0;  // the owner's residual after the latest sweep
  float dual = 0.f;  // the owner's phi_t resp. varphi_j
  // (stretches of sweeps up to a check, or all of them)
  const bool checks = A.check.out != nullptr;
  int nchecks = 0, it = 0, upto = checks ? A.check.first + 1 : A.iters;
  for (;;) {
#pragma unroll 1
  for (; it < upto; ++it) {
    // (A) sweep
    float vp[E], colacc[4 * EQ];
#pragma unroll
    for (int e = 0; e < E; ++e) vp[e] = lds_varphi[16 * e + col];
#pragma unroll
    for (int e = 0; e < 4 * EQ; ++e) colacc[e] = 0.f;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (4 * (wave + NW * r) < A.m) {  // (the same for the whole wave)
        const int row = 4 * (wave + NW * r) + group;
        const float ph = lds_phi[row];
        float rowacc = 0.f;
#pragma unroll
        for (int e = 0; e < E; ++e) {
          float v = fmaxf(x[r][e] + fmaf(-rho, c[r][e], vp[e] + ph), 0.f);
          if (SCALED) v *= scale;
          x[r][e] = v;
          colacc[e] = r == 0 ? v : colacc[e] + v;
          rowacc = e == 0 ? v : rowacc + v;
        }
        rowacc += dpp_mov<0xB1, 0xF>(rowacc);   // quad_perm [1,0,3,2]
        rowacc += dpp_mov<0x4E, 0xF>(rowacc);   // quad_perm [2,3,0,1]
        rowacc += dpp_mov<0x141, 0xF>(rowacc);  // row_half_mirror
        rowacc += dpp_mov<0x140, 0xF>(rowacc);  // row_mirror
        if (col == 0) lds_row[row] = rowacc;
      }
    }
    // sums over the four groups: of two registers, the lower half of the wave goes on with the first, the upper half with
    // the second; then of two of these the even groups with the first, the odd ones with the second
    float half[2 * EQ];
#pragma unroll
    for (int k = 0; k < 2 * EQ; ++k) {
      if (2 * k < E) {
        const auto h = __builtin_amdgcn_permlane32_swap((unsigned)fbits(colacc[2 * k]), (unsigned)fbits(colacc[2 * k + 1]), false, false);
        half[k] = __builtin_bit_cast(float, (int)h[0]) + __builtin_bit_cast(float, (int)h[1]);
      } else {
        half[k] = 0.f;
      }
    }
#pragma unroll
    for (int k = 0; k < EQ; ++k) {
      const auto h = __builtin_amdgcn_permlane16_swap((unsigned)fbits(half[2 * k]), (unsigned)fbits(half[2 * k + 1]), false, false);
      lds_col[wave][64 * k + col_at] = __builtin_bit_cast(float, (int)h[0]) + __builtin_bit_cast(float, (int)h[1]);
    }
    __syncthreads();
    // (B) eq. (6)
    if (owner_wave) {
      // 1^T X 1, the same bits in every owner wave
      const double tot = wave_sum_f64((double)lds_row[lane] + (double)lds_row[lane + 64]);
      const double eta = (tot - sum_p) * inv_mn;
      const double cst = 2.0 * eta - theta;
      theta -= eta;
      if (wave < 2) {
        res = (double)lds_row[t] - target;
        dual = (float)((state - 2.0 * res + cst) * inv_n);
        state -= res;
        if (row_owner) lds_phi[t] = dual;
      } else {
        double s4[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int w = 0; w < NW; ++w) s4[w & 3] += (double)lds_col[w][jc];
        res = ((s4[0] + s4[1]) + (s4[2] + s4[3])) - target;
        dual = (float)((state - 2.0 * res + cst) * inv_m);
        state -= res;
        if (col_owner) lds_varphi[jc] = dual;
      }
    }
    __syncthreads();
  }
  if (!checks) break;
  if (resident_check<NW, kHere>(A, row_owner ? res * res : 0.0, col_owner ? res * res : 0.0, nchecks, it - 1, red, &passed) || it == A.iters) break;
  ++nchecks;
  upto = min(it + A.check.every, A.iters);
  }
  const bool alt = (it & 1) != 0;

#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int row = 4 * (wave + NW * r) + group;
#pragma unroll
    for (int e = 0; e < E; ++e)
      if (row < A.m && 16 * e + col < A.n) A.X[(size_t)row * A.ldx + 16 * e + col] = x[r][e];
  }
  if (row_owner) {
    A.V.phi[t] = dual;
    (alt ? A.a_alt : A.a_in)[t] = state;
    A.V.r[t] = res;
  }
  if (col_owner) {
    A.V.varphi[jc] = dual;
    (alt ? A.b_alt : A.b_in)[jc] = state;
    A.V.s[jc] = res;
  }
  if (t == 0) A.V.theta[A.theta_in ^ (alt ? 1 : 0)] = theta;
  if (checks) return;  // (the last check has left the norms)
  const double r2 = block_sum_f64(row_owner ? res * res : 0.0, red);
  const double s2 = block_sum_f64(col_owner ? res * res : 0.0, red);
  if (t == 0) {
    A.V.resid[0] = r2;
    A.V.resid[1] = s2;
    A.V.resid[2] = 0.0;
    A.V.resid[3] = -1.0;
  }
}

// A wave for every four rows, sixteen at most, four rows twice beyond 64: at most eight rows of a column are added up in fp32
// (four up to 64 rows), the rest in fp64.  Eight waves with twice the rows each would fold half as many sums (2000 iterations,
// 16 waves and 8: 64 x 64 1.47 and 1.35 ms, 64 x 256 2.44 and 2.29, 128 x 256 3.42 and 3.16, 100 x 200 2.86 and 2.76), but
// twice the rows in fp32; with the two halves of their rows kept apart up to the fp64 sum they are behind (1.68, 2.57, 3.46,
// 3.13).  Up to 32 rows eight waves have four rows each: 10 x 10 1.05 (16 waves) and 0.89, 20 x 30 1.07 and 0.94.
template <int E, bool SCALED>
void launch_resident_wide(const ResidentArgs& RS, hipStream_t stream, hipEvent_t e0, hipEvent_t e1) {
  if (RS.m <= 32) launch_timed((resident_wide_kernel<8, 1, E, SCALED>), dim3(1), dim3(512), stream, e0, e1, RS);
  else if (RS.m <= 64) launch_timed((resident_wide_kernel<16, 1, E, SCALED>), dim3(1), dim3(1024), stream, e0, e1, RS);
  else launch_timed((resident_wide_kernel<16, 2, E, SCALED>), dim3(1), dim3(1024), stream, e0, e1, RS);
}
template <int E>
void launch_resident_wide(const ResidentArgs& RS, hipStream_t stream, hipEvent_t e0, hipEvent_t e1) {
  if (RS.scale != 1.f) launch_resident_wide<E, true>(RS, stream, e0, e1);
  else launch_resident_wide<E, false>(RS, stream, e0, e1);
}

// Few rows and many columns leave most waves without a row of their own there: up to 16 rows of more than 96 columns take
// a wave each.  16 x 256: 0.69 us per iteration, 0.93 the other way; 16 x 128 0.66 and 0.68; 16 x 96 0.66 and 0.65;
// 17 x 200 0.97 (two rows a wave) and 0.93.
// (e0, e1: events that take the kernel's own start and end, or null)
void launch_resident(const ResidentArgs& RS, hipStream_t stream, hipEvent_t e0, hipEvent_t e1) {
  if (RS.m <= kResidentRows && RS.n > 96) {
    if (RS.n <= 128) launch_timed((resident_kernel<2>), dim3(1), dim3(1024), stream, e0, e1, RS);
    else launch_timed((resident_kernel<4>), dim3(1), dim3(1024), stream, e0, e1, RS);
    return;
  }
  switch ((RS.n + 15) / 16) {
    case 1: launch_resident_wide<1>(RS, stream, e0, e1); break;
    case 2: launch_resident_wide<2>(RS, stream, e0, e1); break;
    case 3: launch_resident_wide<3>(RS, stream, e0, e1); break;
    case 4: launch_resident_wide<4>(RS, stream, e0, e1); break;
    case 5: launch_resident_wide<5>(RS, stream, e0, e1); break;
    case 6: launch_resident_wide<6>(RS, stream, e0, e1); break;
    case 7: launch_resident_wide<7>(RS, stream, e0, e1); break;
    case 8: launch_resident_wide<8>(RS, stream, e0, e1); break;
    case 9:
    case 10: launch_resident_wide<10>(RS, stream, e0, e1); break;
    case 11:
    case 12: launch_resident_wide<12>(RS, stream, e0, e1); break;
    case 13:
    case 14: launch_resident_wide<14>(RS, stream, e0, e1); break;
    default: launch_resident_wide<16>(RS, stream, e0, e1); break;
  }
}

// Working copy of the cost for the weighted l1 term: out[i][j] = C[i][j] + W[i][j] (pitch ld; the
// pad columns keep their zeros).  +inf entries of C (forbidden pairs) stay +inf.
__global__ __launch_bounds__(256) void add_weights_kernel(float* __restrict__ out, const float* __restrict__ C,
                                                          const float* __restrict__ W, int m, int n, int ld) {
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (j >= n) return;
  for (int i = blockIdx.y; i < m; i += gridDim.y)
    out[(size_t)i * ld + j] = C[(size_t)i * n + j] + W[(size_t)i * n + j];
}

// S6: r_primal of Appendix C; raises the stop flag at the first check that passes so that every
// later kernel of the solve returns at once.  With gap_tol > 0 a check passes only if objective,
// duality gap and dual residual were evaluated for this very iterate (gap_fresh) and
// |gap| <= gap_tol * |objective|, dual_res <= gap_tol (Section 3, "Stopping criteria").
__global__ void status_kernel(VecState V, int iters, double tol, double gap_tol, int gap_fresh) {
  if (*V.done) return;
  const double r2 = V.resid[0], s2 = V.resid[1];
  V.status->r2 = r2;
  V.status->s2 = s2;
  V.status->nz_segments = V.resid[2];
  V.status->nz_lines = V.resid[3];
  V.status->iters = iters;
  if (gap_fresh) V.status->gap_iters = iters;
  bool pass = tol > 0.0 && r2 <= tol * tol && s2 <= tol * tol;
  if (pass && gap_tol > 0.0) {
    const double objective = V.status->cost + V.status->h;
    pass = gap_fresh && fabs(V.status->gap) <= gap_tol * fabs(objective) && V.status->dual_res <= gap_tol;
  }
  if (pass) {
    V.status->converged = 1;
    __threadfence();
    *V.done = 1;
  }
}
