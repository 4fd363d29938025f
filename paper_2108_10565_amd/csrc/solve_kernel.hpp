// The fused solve of Algorithm 3 (section "Block-wise back-substitution" of
// Wolf et al., arXiv 2108.10565): float64 predictor, float32 chain and
// float32 correction, included by the per-degree object.
//
// What bounds it.  At N = 6 an element needs 1.0 MFLOP on the float64 vector
// pipe (14.6 ns at the measured 70 TFLOP/s) and moves 84 KB (16.8 ns at the
// measured 5 TB/s copy), so neither alone explains the 37 ns it takes (50 ns
// with scalar-loaded Khat and workgroup-wide dark-blue steps): with one or two
// waves per SIMD the time goes to latencies that nothing overlaps (scalar
// loads of Khat, workgroup barriers, LDS round trips of the dark-blue step).
// Of a workgroup's 117,000 cycles (at 39 ns, while the code of the dense star
// rows stood in every mode) the green update took 65,000 (43,000 at the pipe's
// rate), X and its barriers 26,000, the setup 24,000.
// The layout below is chosen to keep those latencies short:
//
// * Columns.  One lane per right-hand-side column (element e, quantity p,
//   time mode u).  A wave holds whole (e, p) groups of T = N + 1 lanes,
//   floor(64 / T) of them (63 of 64 lanes at T = 7), and a coupled quantity
//   shares its wave with its partner (the poroelastic u, v, w <- uf, vf, wf).
//   The dark-blue step and the G coupling therefore exchange data inside one
//   wave, through LDS but without a workgroup barrier; a chunk needs one
//   barrier between its X and the star products that read X of the other
//   quantities, and a second one before the next X where the tile has a single
//   X buffer (SolveCfg).
// * Khat.  The coefficients sit in LDS in usage order; one read brings 16 of
//   them into one register pair (lane l holds coefficient l mod 16) and each
//   multiply-add picks its own with a row broadcast (DPP row_newbcast), at
//   the full float64 rate (measured 76 TFLOP/s against 72 with scalar
//   operands).  Scalar loads, used before, can only be waited for all
//   together, which exposed their latency once per 8 multiply-adds: the
//   green update ran at half the pipe rate.  LDS reads are waited for in
//   order, so two groups stay in flight.
// * Top block.  b = Q0 (S^-1 w) there, so X = Q0 (row of Zinv . S^-1 w) (and
//   the same product with the closure row for a coupled quantity) is one or
//   two products per value, without an exchange.
// * Setup.  Degree 0 has no green update and reads no star matrices (they
//   were staged and scanned: 65,536 elements 92 -> 24 us, 100 elements 7.4 ->
//   5.1).  The columns of a star row are found with one ballot per group, a
//   lane's row of the dark-blue inverse by elimination and back substitution
//   of one right-hand side, and Q0 is read once per group and staged through
//   the group's X blocks (it was read again by each of the T lanes): N = 7,
//   16,384 elements 1.57 -> 1.43 ms, N = 5, 65,536 elements 1.35 -> 1.22 ms.
// * Outputs.  A group's lanes store pairs of consecutive doubles of its own
//   row (16 bytes per lane, T lanes contiguous): no index arithmetic, any
//   chunk size.  Ordinary stores: streaming stores of these 112-byte pieces
//   reach HBM as partial lines (N = 6: 4.08 ms against 2.98 ms).
// * Workgroups are small where the degree's registers allow several per
//   compute unit, so that one group's setup and barriers overlap another's
//   multiply-adds (the tile table of the build).
//
// Inputs outside the fast forms take further code in the same kernel, chosen
// per workgroup.  Where a star row has more than kStarNnz columns, its wave
// runs the green update again with the next ones, as the update is linear in
// them (N = 4, 32,768 elements with one row of 13 columns: 555 us, 320 without;
// 1,588 with the dense rows read from memory for every mode).  A coupled quantity of the closure form (one coupling, to
// a quantity without couplings, and no source of its own) whose partner sits
// in another wave costs two more barriers per chunk (N = 6, 16,384 elements
// with one such coupling: 690 us, 695 without it).  Every other coupled
// quantity is late: its X follows in rounds after the others', one per level
// of the dependency chain and chunk (one late quantity 870 us, twelve levels
// of full rows 2.6 ms); that code stands out of the way of the ordinary case,
// which it cost 3% between the chunks.
#pragma once

// Tile of this degree: waves and elements per workgroup, modes per chunk,
// waves per SIMD the registers are held to, X buffers, and modes per chunk of
// the correction and the residual (always two buffers).
#if !defined(STP_SOLVE_WAVES) || !defined(STP_SOLVE_ELEMS) || !defined(STP_SOLVE_CHUNK) || !defined(STP_SOLVE_OCC) || \
    !defined(STP_SOLVE_BUFS) || !defined(STP_SOLVE_CHUNK2)
#error "compile with the solve tile of the build's table"
#endif

namespace stp {
namespace {

constexpr int kInit = 0;      // b = Q0 (S^-1 w); Q <- X
constexpr int kCorrect = 1;   // b = residual (float workspace); Q <- Q + X
constexpr int kResidual = 2;  // float workspace <- residual of the system for the X in Q

template <int N, int Mode>
struct SolveCfg {
  static constexpr int B = n_modes(N), T = N + 1;
  static constexpr int LN = block_start(N);        // register-resident rows (below the top block)
  static constexpr int LR = LN > 0 ? LN : 1;
  static constexpr int DN = block_size(N);
  static constexpr int kWaves = STP_SOLVE_WAVES, kThreads = 64 * kWaves, kE = STP_SOLVE_ELEMS;
  static constexpr bool kAlone = kWaves == 4 * STP_SOLVE_OCC;  // one workgroup fills the compute unit
  static constexpr int GW = 64 / T;                // groups of T lanes per wave
  static constexpr int kPos = kWaves * GW;         // group positions of the workgroup
  static constexpr int kRows = kE * kNQ;           // (element, quantity) rows
  static_assert(kRows <= kPos, "the elements must fit the workgroup's positions");
  // Modes per chunk and X buffers.  Two buffers: X of the next chunk is
  // written while others still read this one's, one barrier per chunk.  One
  // buffer takes a second barrier, but twice the modes fit, so there are half
  // as many exchanges (N = 3, 262,144 elements: float64 1.21 against 1.24 ms,
  // float32 chain 1.02 against 1.18; N = 5, 262,144: 4.68 against 4.95 with 9
  // modes instead of 3; N = 7 with 13 quantities, 16,384: 1.42 with 6 modes
  // against 1.46 with 4 in two buffers, 1.72 against 1.43 while the code of the
  // dense star rows stood in every mode).
  static constexpr int kBufs = Mode == kInit ? STP_SOLVE_BUFS : 2;
  static constexpr int kChunkTile = Mode == kInit ? STP_SOLVE_CHUNK : STP_SOLVE_CHUNK2;
  static constexpr int kChunk = kChunkTile < DN ? kChunkTile : DN;
  // X buffers: one block of S values per position.  S = T mod 16, so that the
  // address of lane (position, u) is congruent to T position + u: consecutive
  // lanes of a wave fall on consecutive banks.
  static constexpr int stride() {
    int s = kChunk * T;
    while ((s - T) % 16 != 0) ++s;
    return s;
  }
  static constexpr int S = stride();
  static constexpr int kBuf = (kPos + 1) * S;      // + one block for the lanes past the last group
};

// Which row (element * kNQ + quantity) each position holds, and back.  A
// position without a row is -1.  Here the poroelastic rows, grouped by the length
// of their star row, which is uniform over most waves that way: normal
// stresses and pressure (6 columns), then the velocity pairs (4; a pair never
// straddles two waves, a shear row fills the gap), then the shear stresses
// (2).
template <int N>
struct SolveLayout {
  using C = SolveCfg<N, kInit>;
  short row[C::kPos];
  short pos[C::kRows];
  constexpr SolveLayout() : row(), pos() {
    for (int i = 0; i < C::kPos; ++i) row[i] = -1;
    int next = 0;
    const int wide[4] = {0, 1, 2, 9}, shear[3] = {3, 4, 5};
    int filled = 0;  // shear rows placed so far
    for (int k = 0; k < 4; ++k)
      for (int e = 0; e < C::kE; ++e) row[next++] = static_cast<short>(e * kNQ + wide[k]);
    for (int k = 0; k < 3; ++k)
      for (int e = 0; e < C::kE; ++e) {
        if (C::GW > 1 && next % C::GW == C::GW - 1) {
          if (filled < 3 * C::kE) {
            row[next] = static_cast<short>((filled % C::kE) * kNQ + shear[filled / C::kE]);
            ++filled;
          }
          ++next;
        }
        row[next++] = static_cast<short>(e * kNQ + 6 + k);
        row[next++] = static_cast<short>(e * kNQ + 10 + k);
      }
    for (; filled < 3 * C::kE; ++filled)
      row[next++] = static_cast<short>((filled % C::kE) * kNQ + shear[filled / C::kE]);
    for (int i = 0; i < C::kPos; ++i)
      if (row[i] >= 0) pos[row[i]] = static_cast<short>(i);
  }
};
template <int N>
__device__ const SolveLayout<N> kSolveLayout{};

// Row of a position and position of a row.  Any other system's order is
// arithmetic: the table's latency would precede the loads of Q0 (6 quantities,
// N = 2, 65,536 elements: 58 us with a table, 55 without).
template <int N>
__device__ __forceinline__ int layout_row(int pos) {
  using C = SolveCfg<N, kInit>;
  if constexpr (kNQ == kNQPoro) return kSolveLayout<N>.row[pos];
  else return pos < C::kRows ? pos % C::kE * kNQ + pos / C::kE : -1;
}
template <int N>
__device__ __forceinline__ int layout_pos(int row) {
  if constexpr (kNQ == kNQPoro) return kSolveLayout<N>.pos[row];
  else return row % kNQ * SolveCfg<N, kInit>::kE + row / kNQ;
}

template <int N>
constexpr int khat_nnz() {
  using P = stp_gen::KhatPattern<N>;
  int n = 0;
  for (int m = 0; m < n_modes(N); ++m)
    n = P::col_start[m] + P::col_count[m] > n ? P::col_start[m] + P::col_count[m] : n;
  return n;
}

template <int N, typename R, int Mode>
struct SolveShared {
  using C = SolveCfg<N, Mode>;
  static constexpr int kTab = (khat_nnz<N>() + 15) / 16 * 16;
  static constexpr int kCoupled = C::kE * kNQ * (kNQ - 1) / 2;  // entries of E* right of the diagonal
  // where a general E keeps them: after X, or in the residual, whose two X
  // buffers fill the LDS at N = 6, with its output where the rows leave room
  static constexpr int kRes = Mode == kResidual ? (C::kPos + 1) * C::S : 1;
  static constexpr bool kInRows = Mode == kResidual && 8 * kCoupled + 4 * kRes <= 8 * C::kThreads * C::T;
  R khat[kTab > 0 ? kTab : 16];            // Khat in usage order
  union {
    double rows[C::kThreads][C::T];        // per lane: dense row of its dark-blue step
    struct {
      double G[kInRows ? kCoupled : 1];    // as u.c.G
      float res[kRes];                     // residual of the chunk, blocks as in x
    } r;
  };
  double q0[(C::kPos + 1) * C::DN];        // Q0 of the top block
  int pos[C::kRows];
  int row[C::kPos + 1];                    // of a position (the general code's; -1: none)
  int level[C::kRows];                     // level of a row (general E), and its columns (kColumns ..)
  unsigned cols[C::kRows];
  int maxlevel;
  unsigned flags;
  union {
    struct {                               // setup only
      double G[C::kE][kNQ][kNQ];           // E* (lower part zeroed)
      double A[N > 0 ? C::kE : 1][3][kNQ][kNQ];  // -A^{j*}: the green update then adds Khat y
    } s;
    struct {
      R x[C::kBufs * C::kBuf + 2 * C::T * C::T];  // X of the chunks (+ what the last lanes' output reads may run over)
      double G[kInRows ? 1 : kCoupled];    // general E: the entries right of the diagonal, row by row
    } c;
  } u;
  __device__ __forceinline__ double* couplings() {
    if constexpr (kInRows) return r.G;
    else return u.c.G;
  }
  // entry (q, q + 1) of element e; (q, q + 1 + i) is i after it
  __device__ __forceinline__ const double* coupling(int e, int q) {
    return couplings() + e * (kNQ * (kNQ - 1) / 2) + q * (2 * kNQ - 1 - q) / 2;
  }
};

// b += coefficient I of the 16 that the wave's register k holds, times y
// (v_fmac with a row broadcast).  A broadcast needs two wait states after a
// vector write of k, which the compiler does not insert for an asm operand.  k
// comes straight from an LDS read, so there is no such write unless the
// register allocator makes a copy; the build checks in the disassembly that it
// made none (dpp_check.py).
template <int I>
__device__ __forceinline__ void fmac_bcast(double& b, double k, double y) {
  asm("v_fmac_f64_dpp %0, %1, %2 row_newbcast:%c3 row_mask:0xf bank_mask:0xf" : "+v"(b) : "v"(k), "v"(y), "n"(I));
}
template <int I>
__device__ __forceinline__ void fmac_bcast(float& b, float k, float y) {
  asm("v_fmac_f32_dpp %0, %1, %2 row_newbcast:%c3 row_mask:0xf bank_mask:0xf" : "+v"(b) : "v"(k), "v"(y), "n"(I));
}

// The columns of the two-entry rows of Z^-1 (generated) are max(u - 1, 0) and
// min(u + 1, N).
template <int N>
constexpr bool zinv_columns() {
  using ZS = stp_gen::ZinvSparse<N>;
  for (int u = 0; u <= N; ++u) {
    if (ZS::col[2 * u] != (u > 0 ? u - 1 : 0) && ZS::val[2 * u] != 0.0) return false;
    if (ZS::col[2 * u + 1] != (u < N ? u + 1 : N) && ZS::val[2 * u + 1] != 0.0) return false;
  }
  return true;
}

// Row u of (Z - z I)^-1: the solution y of (Z - z I)^T y = e_u by elimination
// without pivoting and back substitution.  For z = dt E_pp < 0.5 (the range
// stp_validate admits) the pivots stay away from zero: over z in [-1e7, 0.5)
// and every degree N <= 7 the smallest is at least 3% of max|Z| + |z| (checked
// numerically).
template <int T>
__device__ __forceinline__ void zinv_row(double z, int u, double (&y)[T]) {
  double m[T][T], inv[T];
#pragma unroll
  for (int r = 0; r < T; ++r) {
#pragma unroll
    for (int c = 0; c < T; ++c) m[r][c] = z_entry(c, r) - (r == c ? z : 0.0);  // transpose
    y[r] = r == u ? 1.0 : 0.0;
  }
#pragma unroll
  for (int k = 0; k < T; ++k) {
    inv[k] = 1.0 / m[k][k];
#pragma unroll
    for (int r = k + 1; r < T; ++r) {
      const double f = m[r][k] * inv[k];
#pragma unroll
      for (int c = k + 1; c < T; ++c) m[r][c] = fma(-f, m[k][c], m[r][c]);
      y[r] = fma(-f, y[k], y[r]);
    }
  }
#pragma unroll
  for (int k = T - 1; k >= 0; --k) {
#pragma unroll
    for (int c = k + 1; c < T; ++c) y[k] = fma(-m[k][c], y[c], y[k]);
    y[k] *= inv[k];
  }
}

// Bit q of the result: f(q) for the lane's group, each lane of the group
// having evaluated it for q = u, u + T, ... only (the lanes of a group would
// all evaluate the same kNQ values otherwise).
template <int T, class F>
__device__ __forceinline__ unsigned group_mask(int grp, int u, F&& f) {
  unsigned mask = 0;
  if constexpr (T == 1) {  // nothing to share
#pragma unroll
    for (int q = 0; q < kNQ; ++q) mask |= f(q) ? 1u << q : 0u;
    return mask;
  }
#pragma unroll
  for (int q0 = 0; q0 < kNQ; q0 += T) {
    const int q = q0 + u < kNQ ? q0 + u : kNQ - 1;
    const unsigned long long bits = __builtin_amdgcn_ballot_w64(q0 + u < kNQ && f(q));
    mask |= (static_cast<unsigned>(bits >> (grp * T)) & ((1u << T) - 1)) << q0;
  }
  return mask;
}

// Orders the LDS accesses of one wave (a wave's LDS operations complete in
// order; this keeps the compiler from reordering them).
__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

typedef double pair_t __attribute__((ext_vector_type(2), aligned(8)));
typedef float quad_t __attribute__((ext_vector_type(4), aligned(4)));

constexpr unsigned kDenseStar = 1u, kGeneralE = 2u, kFarPartner = 4u;
// of SolveShared::cols: the coupled columns, those of the star row above them
// (at kStarShift), and
constexpr unsigned kColumns = (1u << kNQ) - 1, kClosed = 1u << 30, kStiff = 1u << 31;
constexpr int kStarShift = kNQ;
static_assert(2 * kNQ <= 30, "the masks fit below the flags");

// Waves per SIMD the registers are held to.  The residual keeps about 30 more
// than the solve (X of the next chunk, a row of Z), so where the rows of b leave
// no more than 100 it gets one wave less (N = 5) unless its workgroup needs all
// of them (N = 7: 8 waves, 2 per SIMD; it spills there, 232 registers with 13
// quantities and 145 with six, and with the chain and the correction still takes
// 2.3 ms at 8,192 elements with one refinement, against 5.2 ms for the residual
// kernel with one wave per SIMD and no spill).
template <int N, int Mode>
constexpr int solve_occupancy() {
  using C = SolveCfg<N, Mode>;
  return Mode == kResidual && C::kWaves <= 4 && 512 / STP_SOLVE_OCC - 2 * C::LN <= 100 ? STP_SOLVE_OCC - 1 : STP_SOLVE_OCC;
}

// Algorithm 3 over a group of elements in precision R (the dark-blue solves
// are float64 in every mode).  kInit: b = Q0 (S^-1 w), Q <- X.  kCorrect:
// b = the residual in `work` (float), Q <- Q + X.
//
// kResidual: the float64 residual of the full element system for the current
// Q (the matrix-free form of eq:stp-lineq after the multiplication with
// M^-1 S^-1, section "Block-wise back-substitution"):
//   r[p,n,u] = (S^-1 w)_u Q0[p,n] - sum_s Z_us Q[p,n,s] + sum_q E*_pq Q[q,n,u]
//              - sum_j sum_q A^{j*}_pq sum_l Khat^j[n,l] Q[q,l,u],
// written to `work` in float.  Its star and Khat products are the green
// update applied to the known X, chunk by chunk from the top block down, so it
// shares that code; X comes from Q one chunk ahead instead of from the
// dark-blue step, and the local terms of a chunk's rows follow its barrier.
template <int N, typename R, int Mode>
__global__ __launch_bounds__((SolveCfg<N, Mode>::kThreads), (solve_occupancy<N, Mode>())) void solve_kernel(PredictArgs a, float* work) {
  using C = SolveCfg<N, Mode>;
  using P = stp_gen::KhatPattern<N>;
  using ZS = stp_gen::ZinvSparse<N>;
  using LdsR = __attribute__((address_space(3))) R;
  using LdsD = __attribute__((address_space(3))) double;
  constexpr int B = C::B, T = C::T, kE = C::kE, kThreads = C::kThreads, S = C::S, GW = C::GW, DN = C::DN, LN = C::LN;
  static_assert(zinv_columns<N>(), "two-entry rows of Z^-1");
  // Modes of a chunk that the rounds of the late lanes take at a time, and time
  // modes of a dense row in flight: as many as the rows of b leave registers
  // for without a spill or a wave less per SIMD (N = 6, 16,384 elements, one
  // coupling: 1,040 us with 3 modes, 870 with all).
  constexpr bool kRoomy = 512 / STP_SOLVE_OCC - 2 * LN >= 128 && (sizeof(R) == 8 || STP_SOLVE_OCC <= 2);
  constexpr int kPart = kRoomy ? C::kChunk : LN < 60 ? 3 : 2, kStep = !kRoomy ? 1 : sizeof(R) == 8 ? 2 : T;
  __shared__ SolveShared<N, R, Mode> sh;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const int64_t e0 = static_cast<int64_t>(blockIdx.x) * kE;
  const int64_t nloc64 = a.n - e0 < kE ? a.n - e0 : kE;
  const int nloc = static_cast<int>(nloc64);
  const int grp = lane / T, u = lane - grp * T;
  const int pos = grp < GW ? wave * GW + grp : C::kPos;
  const int row = grp < GW ? layout_row<N>(pos) : -1;

  // ---- setup: E, star and Khat to LDS (every load issued before the first
  // LDS store, so the group waits for one memory latency)
  constexpr int kEIt = (kE * kNQ * kNQ + kThreads - 1) / kThreads;
  constexpr int kStar = N > 0 ? 3 * kE * kNQ * kNQ : 0;  // degree 0 has no green update
  constexpr int kAIt = (kStar + kThreads - 1) / kThreads;
  constexpr int nnz = khat_nnz<N>(), kTab = SolveShared<N, R, Mode>::kTab, kKIt = (kTab + kThreads - 1) / kThreads;
  {
    double ev[kEIt], av[kAIt > 0 ? kAIt : 1];
    R kv[kKIt > 0 ? kKIt : 1];
    const R* const ktab = khat_sparse<N, R>();
#pragma unroll
    for (int k = 0; k < kEIt; ++k) {
      const int i = tid + k * kThreads;
      ev[k] = i < nloc * kNQ * kNQ ? a.E[e0 * (kNQ * kNQ) + i] : 0.0;
    }
#pragma unroll
    for (int k = 0; k < kAIt; ++k) {
      const int i = tid + k * kThreads;
      av[k] = i < nloc * 3 * kNQ * kNQ ? a.star[e0 * (3 * kNQ * kNQ) + i] : 0.0;
    }
#pragma unroll
    for (int k = 0; k < kKIt; ++k) {
      const int i = tid + k * kThreads;
      kv[k] = i < nnz ? ktab[i] : R(0);
    }
    unsigned bad = 0;  // input conditions the elimination without pivoting cannot take
#pragma unroll
    for (int k = 0; k < kEIt; ++k) {
      const int i = tid + k * kThreads;
      const int r = (i / kNQ) % kNQ, c = i % kNQ;
      const double v = a.dt * ev[k];
      if (c < r && v != 0.0) bad |= kInputNotUpper;
      if (c == r && v >= 0.5) bad |= kInputSingular;
      if (i < kE * kNQ * kNQ) (&sh.u.s.G[0][0][0])[i] = c >= r ? v : 0.0;
    }
    if (bad && a.status) atomicOr(a.status, bad);
#pragma unroll
    for (int k = 0; k < kAIt; ++k) {
      const int i = tid + k * kThreads;
      if (i < kStar) (&sh.u.s.A[0][0][0][0])[i] = -(a.dt * av[k]);
    }
#pragma unroll
    for (int k = 0; k < kKIt; ++k) {
      const int i = tid + k * kThreads;
      if (i < kTab) sh.khat[i] = kv[k];
    }
  }
  for (int i = tid; i < C::kRows; i += kThreads) sh.pos[i] = layout_pos<N>(i);
  if (u == 0) sh.row[pos] = row;
  if (tid == 0) {
    sh.flags = 0;
    sh.maxlevel = 0;
  }
  const bool valid = row >= 0;  // the lane holds a column (of an element past the end, if not active)
  const int es = valid ? row / kNQ : 0, p = valid ? row - es * kNQ : 0;
  const bool active = valid && es < nloc;
  const int arow = active ? row : 0;
  // uniform bases and 32-bit lane offsets of this lane's row
  const char* const Q0b = reinterpret_cast<const char*>(a.Q0 + e0 * (kNQ * B));
  char* const Qb = reinterpret_cast<char*>(a.Q + e0 * (kNQ * B * T));
  char* const Ib = reinterpret_cast<char*>(a.Qint ? a.Qint + e0 * (kNQ * B) : nullptr);
  char* const Rb = reinterpret_cast<char*>(work ? work + e0 * (kNQ * B * T) : nullptr);
  const unsigned q0off = static_cast<unsigned>(arow * (B * 8));
  const unsigned ioff = q0off + 8 * u;
  const unsigned qoff = static_cast<unsigned>(arow * (B * T * 8) + 16 * u);
  const unsigned roff = static_cast<unsigned>(arow * (B * T * 4) + 4 * u);
  auto load_q0 = [&](int m) __attribute__((always_inline)) {
    return *reinterpret_cast<const double*>(Q0b + q0off + m * 8);
  };
  auto load_r = [&](int m) __attribute__((always_inline)) {
    return *reinterpret_cast<const float*>(Rb + roff + m * (T * 4));
  };
  // Q0 of this group's row, each lane every T-th mode (to LDS below)
  constexpr int kQt = Mode != kCorrect ? (B + T - 1) / T : 0;
  double qt[kQt > 0 ? kQt : 1];
#pragma unroll
  for (int k = 0; k < kQt; ++k)
    qt[k] = k * T + u < B ? *reinterpret_cast<const double*>(Q0b + ioff + k * T * 8) : 0.0;
  __syncthreads();

  // G coupling of this lane's quantity (the first non-zero right of the
  // diagonal and their count), and whether that partner couples further
  const unsigned gmask = group_mask<T>(grp, u, [&](int q) { return valid && q > p && sh.u.s.G[es][p][q] != 0.0; });
  const int gcount = __builtin_popcount(gmask), gp = gmask ? __builtin_ctz(gmask) : p;
  const double gcoef = gmask ? sh.u.s.G[es][p][gp] : 0.0;
  const bool partner_coupled =
      group_mask<T>(grp, u, [&](int q) { return valid && gmask && q > gp && sh.u.s.G[es][gp][q] != 0.0; }) != 0;
  // Row u of (Z - E*_pp I)^-1: two entries of Z^-1 without a diagonal source;
  // otherwise a dense row from an elimination, done only by waves holding
  // such a lane.  xc = row . S^-1 w.
  const double z = valid ? sh.u.s.G[es][p][p] : 0.0;
  const bool wave_stiff = __builtin_amdgcn_ballot_w64(z != 0.0) != 0;
  const bool wave_coupled = __builtin_amdgcn_ballot_w64(gcount != 0) != 0;
  const bool wave_dense = wave_stiff || wave_coupled;
  const int zc0 = ZS::col[2 * u], zc1 = ZS::col[2 * u + 1];
  double zv0 = ZS::val[2 * u], zv1 = ZS::val[2 * u + 1];
  double xc = fma(zv0, sinv_w(zc0), zv1 * sinv_w(zc1)), dc = 0.0;
  if constexpr (Mode != kResidual) {
    double r[T];
#pragma unroll
    for (int v = 0; v < T; ++v) r[v] = (zc0 == v ? zv0 : 0.0) + (zc1 == v ? zv1 : 0.0);
    if (wave_stiff) {
      double zs[T];
      zinv_row<T>(z, u, zs);
      if (z != 0.0) {
        xc = 0.0;
#pragma unroll
        for (int v = 0; v < T; ++v) {
          r[v] = zs[v];
          xc = fma(zs[v], sinv_w(v), xc);
        }
      }
    }
#pragma unroll
    for (int v = 0; v < T; ++v) sh.rows[tid][v] = r[v];
  }
  // sparse row p of the three star matrices: the columns with a non-zero in
  // any direction, in ascending order
  __builtin_amdgcn_sched_barrier(0);  // the elimination's registers are free before these are taken
  unsigned mask = 0;
  if constexpr (N > 0)
    mask = group_mask<T>(grp, u, [&](int q) {
      return valid && (sh.u.s.A[es][0][p][q] != 0.0 || sh.u.s.A[es][1][p][q] != 0.0 || sh.u.s.A[es][2][p][q] != 0.0);
    });
  const unsigned star_mask = mask;
  const int npop = __builtin_popcount(mask);
  // columns the wave's longest row needs (wave-uniform: 2, 4 or 6)
  auto row_length = [](int n) __attribute__((always_inline)) {
    return __builtin_amdgcn_readfirstlane(__builtin_amdgcn_ballot_w64(n > 4)   ? 6
                                          : __builtin_amdgcn_ballot_w64(n > 2) ? 4
                                                                               : 2);
  };
  int ns = row_length(npop);
  R sa0[kStarNnz], sa1[kStarNnz], sa2[kStarNnz];
  LdsR* sp[kStarNnz];
  LdsR* const x0 = (LdsR*)&sh.u.c.x[0];
#pragma unroll
  for (int k = 0; N > 0 && k < kStarNnz; ++k) {
    const bool live = mask != 0;
    const int q = live ? __builtin_ctz(mask) : p;
    mask &= mask - 1;
    const double v0 = sh.u.s.A[es][0][p][q], v1 = sh.u.s.A[es][1][p][q], v2 = sh.u.s.A[es][2][p][q];
    sa0[k] = live ? static_cast<R>(v0) : R(0);
    sa1[k] = live ? static_cast<R>(v1) : R(0);
    sa2[k] = live ? static_cast<R>(v2) : R(0);
    sp[k] = x0 + (live ? sh.pos[es * kNQ + q] : pos) * S + u;
  }
  // A coupled lane is of the closure form (below), or late: its X follows in
  // rounds after the others'.
  const bool closed = gcount == 1 && !partner_coupled && z == 0.0, late = Mode != kResidual && gcount > 0 && !closed;
  const int ppos = gcount > 0 && !late ? sh.pos[es * kNQ + gp] : pos;
  if (u == 0 && valid)
    sh.cols[row] = gmask | (star_mask << kStarShift) | (closed ? kClosed : 0u) | (z != 0.0 ? kStiff : 0u);
  {
    const unsigned f = (active && npop > kStarNnz ? kDenseStar : 0u) |
                       (active && (Mode == kResidual ? gcount > 1 : late) ? kGeneralE : 0u) |
                       (active && Mode != kResidual && ppos / GW != pos / GW ? kFarPartner : 0u);
    if (f) atomicOr(&sh.flags, f);
  }
  __syncthreads();
  const unsigned flags = __builtin_amdgcn_readfirstlane(sh.flags);
  const bool dense_star = (flags & kDenseStar) != 0, closure = (flags & kGeneralE) == 0;
  // some coupled quantity's partner sits in another wave: barriers where the
  // coupled quantities of a wave need only its own order
  const bool far = (flags & kFarPartner) != 0;
  if (__builtin_expect(!closure, 0)) {  // out of the way of the ordinary case, here and below
    // The couplings of a general upper-triangular E move out of the setup's
    // storage, which X takes: reading them from memory once per mode and time
    // made such a workgroup 16 times as slow as an ordinary one (N = 6).
    constexpr int kIt = (SolveShared<N, R, Mode>::kCoupled + kThreads - 1) / kThreads, kTri = kNQ * (kNQ - 1) / 2;
    double gv[kIt];
#pragma unroll
    for (int k = 0; k < kIt; ++k) {
      const int i = tid + k * kThreads, e = i / kTri;
      int q = 0, o = i - e * kTri;  // row q, o places right of the diagonal
#pragma unroll 1
      for (; o >= kNQ - 1 - q; ++q) o -= kNQ - 1 - q;
      gv[k] = e < kE ? sh.u.s.G[e][q][q + 1 + o] : 0.0;
    }
    // dependency levels (longest chain of late quantities down to a quantity),
    // one thread per element
    if (Mode != kResidual && tid < nloc) {
      int lev[kNQ];
      int mx = 0;
#pragma unroll
      for (int o = kNQ - 1; o >= 0; --o) {
        const unsigned m = sh.cols[tid * kNQ + o];
        int l = 0;
#pragma unroll
        for (int q = o + 1; q < kNQ; ++q)
          if ((m >> q & 1u) && lev[q] + 1 > l) l = lev[q] + 1;
        if (m & kClosed) l = 0;
        lev[o] = l;
        sh.level[tid * kNQ + o] = l;
        mx = l > mx ? l : mx;
      }
      atomicMax(&sh.maxlevel, mx);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kIt; ++k) {
      const int i = tid + k * kThreads;
      if (i < SolveShared<N, R, Mode>::kCoupled) sh.couplings()[i] = gv[k];
    }
  }
  if constexpr (Mode != kResidual) {
    // closure row of a coupled lane, X_o = Zinv_o (b_o + g X_p) = zr . b_o + dr . b_p:
    //   dr[w] = g sum_v (row u of Zinv_o)[v] Zinv_p[v][w],
    // the rows Zinv_p[v] being those of the partner's lanes.  After it a
    // lane's dense row is: stiff lanes their row of Zinv (on their own b),
    // closed lanes dr (on the partner's b), the others zero.
    double r[T];
#pragma unroll
    for (int w = 0; w < T; ++w) r[w] = 0.0;
    if (closed) {
      const int plane = ppos / GW * 64 + (ppos - ppos / GW * GW) * T;
#pragma unroll
      for (int w = 0; w < T; ++w) {
        r[w] = gcoef * fma(zv0, sh.rows[plane + zc0][w], zv1 * sh.rows[plane + zc1][w]);
        dc = fma(r[w], sinv_w(w), dc);
      }
    }
    wave_fence();
    if (far) __syncthreads();
    if (wave_dense) {
      if (z == 0.0) {
#pragma unroll
        for (int w = 0; w < T; ++w) sh.rows[tid][w] = r[w];
      } else {
        zv0 = zv1 = 0.0;
      }
    }
    if (late) {  // in the top block the step below then leaves b = Q0 (S^-1 w) in place
      xc = sinv_w(u);
      dc = 0.0;
    }
  }
  // Rows of b below the top block (after the setup: its elimination needs the
  // registers).  b = Q0 (S^-1 w): the group's lanes share one row of Q0, which
  // they loaded together; it goes through the group's own blocks of the X
  // buffers, still unused, instead of T lanes loading the same values (at N = 6
  // that took 3,600 cycles of the compute unit's load path per workgroup).
  // Modes that do not fit the blocks are loaded by every lane.
  LdsR* const xg = x0 + pos * S;            // the group's block
  R b[C::LR];
  const double w_u = sinv_w(u);
  if constexpr (Mode != kCorrect) {
    constexpr int kFit = (S * static_cast<int>(sizeof(R)) - (8 - static_cast<int>(sizeof(R)))) / 8;  // doubles per block
    constexpr int kStaged = LN < C::kBufs * kFit ? LN : C::kBufs * kFit;
    auto aligned = [&](int i) { return (LdsD*)(x0 + (sizeof(R) == 8 ? i : (i + 1) & ~1)); };
    LdsD* const s0 = aligned(pos * S);
    LdsD* const s1 = aligned((C::kBufs - 1) * C::kBuf + pos * S);
#pragma unroll
    for (int k = 0; k < kQt; ++k) {
      const int m = k * T + u;
      if (m >= LN && m < B) sh.q0[pos * DN + m - LN] = qt[k];
      if (m < kFit && m < kStaged) s0[m] = qt[k];
      if (m >= kFit && m < kStaged) s1[m - kFit] = qt[k];
    }
    wave_fence();
#pragma unroll
    for (int n = 0; n < LN; ++n)
      b[n] = static_cast<R>((n < kStaged ? (n < kFit ? s0[n] : s1[n - kFit]) : load_q0(n)) * w_u);
    wave_fence();
    if (far) __syncthreads();  // Q0 of the partners
  } else {
#pragma unroll
    for (int n = 0; n < LN; ++n) b[n] = static_cast<R>(load_r(n));
  }
  LdsR* const xs = x0 + ppos * S;           // what the dense row applies to
  LdsD* const qg = (LdsD*)&sh.q0[0] + pos * DN;
  LdsD* const qp = (LdsD*)&sh.q0[0] + ppos * DN;

  // residual rows of a top-block chunk (kCorrect), loaded one chunk ahead
  constexpr int kTop0 = chunk_size(N, C::kChunk, 0);
  R rtop[Mode == kCorrect ? kTop0 : 1];
  if constexpr (Mode == kCorrect) {
#pragma unroll
    for (int k = 0; k < kTop0; ++k) rtop[k] = static_cast<R>(load_r(LN + k));
  }

  // kResidual: X of the next chunk, as the pairs of the output pass
  constexpr int kPairs = (C::kChunk * T / 2 + T - 1) / T;
  pair_t xpre[Mode == kResidual && kPairs > 0 ? kPairs : 1];
  double xlast = 0.0;
  auto load_chunk = [&](auto gc, auto cic) __attribute__((always_inline)) {
    constexpr int gl = decltype(gc)::value, cil = decltype(cic)::value;
    constexpr int m = chunk_start(gl, C::kChunk, cil), cl = chunk_size(gl, C::kChunk, cil);
    constexpr int npl = cl * T / 2, nl = (npl + T - 1) / T;
#pragma unroll
    for (int j = 0; j < nl; ++j)
      if ((j + 1) * T <= npl || j * T + u < npl)
        xpre[j] = *reinterpret_cast<const pair_t*>(Qb + qoff + (m * T + j * 2 * T) * 8);
    if constexpr ((cl * T) % 2 != 0) {
      if (u == 0) xlast = *reinterpret_cast<const double*>(Qb + qoff + (m * T + cl * T - 1) * 8);
    }
  };
  if constexpr (Mode == kResidual) load_chunk(ic<N>{}, ic<0>{});

  static_for<0, N + 1>([&](auto gi) __attribute__((always_inline)) {
    constexpr int g = N - decltype(gi)::value;
    static_for<0, nchunks(g, C::kChunk)>([&](auto ci) __attribute__((always_inline)) {
      constexpr int cidx = decltype(ci)::value;
      constexpr int m0 = chunk_start(g, C::kChunk, cidx), c = chunk_size(g, C::kChunk, cidx);
      constexpr int CI = chunk_index(N, g, cidx, C::kChunk), xb = (CI & (C::kBufs - 1)) * C::kBuf;
      constexpr int np = c * T / 2, nst = (np + T - 1) / T, nin = (c + T - 1) / T;
      constexpr bool odd = (c * T) % 2 != 0, green = g > 0;
      // the lane's addresses, formed anew for each chunk (an opaque copy of
      // u): held over the multiply-adds they would cost a wave per SIMD
      int uc = u;
      asm volatile("" : "+v"(uc));
      LdsR* const xl = xg + uc;               // the lane's column
      LdsR* const xo = xg + 2 * uc;           // its output pairs
      LdsR* const xi = xg + uc * T;           // its Qint values
      LdsR* const kl = (LdsR*)&sh.khat[0] + (lane & 15);
      // kCorrect: the previous outputs, in flight until they are added to
      pair_t qprev[Mode == kCorrect && nst > 0 ? nst : 1];
      double qlast = 0.0, iprev[Mode == kCorrect ? nin : 1];
      if constexpr (Mode == kCorrect) {
#pragma unroll
        for (int j = 0; j < nst; ++j)
          if ((j + 1) * T <= np || j * T + u < np)
            qprev[j] = *reinterpret_cast<const pair_t*>(Qb + qoff + (m0 * T + j * 2 * T) * 8);
        if constexpr (odd) {
          if (u == 0) qlast = *reinterpret_cast<const double*>(Qb + qoff + (m0 * T + c * T - 1) * 8);
        }
        if (a.Qint) {
#pragma unroll
          for (int k = 0; k < nin; ++k)
            if ((k + 1) * T <= c || k * T + u < c)
              iprev[k] = *reinterpret_cast<const double*>(Ib + ioff + (m0 + k * T) * 8);
        }
      }
      if constexpr (C::kBufs == 1 && CI > 0) __syncthreads();  // the reads of the chunk before
      // ---- X of the chunk: dark-blue blocks and G coupling (float64)
      if constexpr (Mode == kResidual) {
#pragma unroll
        for (int j = 0; j < nst; ++j)
          if ((j + 1) * T <= np || j * T + u < np) {
            xo[xb + j * 2 * T] = xpre[j].x;
            xo[xb + j * 2 * T + 1] = xpre[j].y;
          }
        if constexpr (odd) {
          if (u == 0) xg[xb + c * T - 1] = xlast;
        }
      } else if (Mode == kInit && g == N) {
        if (wave_coupled) {
#pragma unroll
          for (int k = 0; k < c; ++k)
            xl[xb + k * T] = static_cast<R>(fma(xc, qg[m0 - LN + k], dc * qp[m0 - LN + k]));
        } else {
#pragma unroll
          for (int k = 0; k < c; ++k) xl[xb + k * T] = static_cast<R>(xc * qg[m0 - LN + k]);
        }
      } else {
#pragma unroll
        for (int k = 0; k < c; ++k) {
          if constexpr (g < N) xl[xb + k * T] = b[m0 + k];
          else xl[xb + k * T] = rtop[k];
        }
        wave_fence();
        if (far) __syncthreads();
        // columns of the two entries of a row of Z^-1: max(u - 1, 0), min(u + 1, N)
        LdsR* const xz0 = xg + (uc > 0 ? uc - 1 : 0);
        LdsR* const xz1 = xg + (uc < N ? uc + 1 : N);
        double x[c];
#pragma unroll
        for (int k = 0; k < c; ++k)
          x[k] = fma(zv0, static_cast<double>(xz0[xb + k * T]), zv1 * static_cast<double>(xz1[xb + k * T]));
        if (wave_dense) {
          double r[T];
#pragma unroll
          for (int v = 0; v < T; ++v) r[v] = sh.rows[tid][v];
#pragma unroll
          for (int k = 0; k < c; ++k)
#pragma unroll
            for (int v = 0; v < T; ++v) x[k] = fma(r[v], static_cast<double>(xs[xb + k * T + v]), x[k]);
        }
        wave_fence();
        if (far) __syncthreads();
        if (!late) {
#pragma unroll
          for (int k = 0; k < c; ++k) xl[xb + k * T] = static_cast<R>(x[k]);
        }
      }
      if (Mode != kResidual && __builtin_expect(!closure, 0)) {
        // late lanes, level by level: a lane adds the coupled quantities' X to
        // its own value of b, still in its place, then the group's lanes
        // exchange these sums (float64; through the group's block where it
        // holds doubles) and overwrite b with X
        const int row = sh.row[pos], es = row < 0 ? 0 : row / kNQ, p = row < 0 ? 0 : row - es * kNQ;
        const int mine = active ? sh.level[row] : 0;
        const unsigned cols = active ? sh.cols[row] : 0u;
        const int maxlevel = __builtin_amdgcn_readfirstlane(sh.maxlevel);
#pragma unroll 1
        for (int lv = 1; lv <= maxlevel; ++lv) {
          __syncthreads();
          if (mine == lv) {
            const bool dense = __builtin_amdgcn_ballot_w64((cols & kStiff) != 0) != 0;
            static_for<0, (c + kPart - 1) / kPart>([&](auto part) __attribute__((always_inline)) {
              constexpr int k0 = decltype(part)::value * kPart, kn = c - k0 < kPart ? c - k0 : kPart;
              double sum[kn], x[kn];
#pragma unroll
              for (int k = 0; k < kn; ++k) sum[k] = static_cast<double>(xl[xb + (k0 + k) * T]);
              const double* const gq = sh.coupling(es, p);
#pragma unroll 1
              for (unsigned m = cols & kColumns; m != 0; m &= m - 1) {
                const int q = __builtin_ctz(m);
                const double gv = gq[q - p - 1];
                LdsR* const xq = x0 + sh.pos[es * kNQ + q] * S + uc;
#pragma unroll
                for (int k = 0; k < kn; ++k) sum[k] = fma(gv, static_cast<double>(xq[xb + (k0 + k) * T]), sum[k]);
              }
              if constexpr (sizeof(R) == 8) {
#pragma unroll
                for (int k = 0; k < kn; ++k) xl[xb + (k0 + k) * T] = sum[k];
                wave_fence();
              }
              auto sum_of = [&](int k, int v) __attribute__((always_inline)) {  // of the group's lane v
                if constexpr (sizeof(R) == 8) return xg[xb + (k0 + k) * T + v];
                else return __shfl(sum[k], lane - uc + v);
              };
              const int v0 = uc > 0 ? uc - 1 : 0, v1 = uc < N ? uc + 1 : N;
#pragma unroll
              for (int k = 0; k < kn; ++k) x[k] = fma(zv0, sum_of(k, v0), zv1 * sum_of(k, v1));
              if (dense) {
#pragma unroll kStep
                for (int v = 0; v < T; ++v) {
                  const double r = sh.rows[tid][v];
#pragma unroll
                  for (int k = 0; k < kn; ++k) x[k] = fma(r, sum_of(k, v), x[k]);
                }
              }
              wave_fence();
#pragma unroll
              for (int k = 0; k < kn; ++k) xl[xb + (k0 + k) * T] = static_cast<R>(x[k]);
            });
          }
        }
      }
      if constexpr (Mode == kCorrect && g == N && cidx + 1 < nchunks(N, C::kChunk)) {
        constexpr int cn = chunk_size(N, C::kChunk, cidx + 1), mn = chunk_start(N, C::kChunk, cidx + 1);
#pragma unroll
        for (int k = 0; k < cn; ++k) rtop[k] = static_cast<R>(load_r(mn + k));
      }
      wave_fence();
      if constexpr (green || Mode == kResidual) __syncthreads();
      if constexpr (Mode == kResidual) {
        if constexpr (cidx + 1 < nchunks(g, C::kChunk)) load_chunk(ic<g>{}, ic<cidx + 1>{});
        else if constexpr (g > 0) load_chunk(ic<(g > 0 ? g - 1 : 0)>{}, ic<0>{});
        // local terms of the chunk's rows: their residual is now complete
        double zrow[T];  // row u of Z
#pragma unroll
        for (int v = 0; v < T; ++v) zrow[v] = z_entry(uc, v);
        auto store_local = [&](int k, double ex) __attribute__((always_inline)) {  // ex: terms of E
          double base, zx = 0.0;
          if constexpr (g == N) base = qg[m0 - LN + k] * w_u;
          else base = b[m0 + k];
#pragma unroll
          for (int v = 0; v < T; ++v) zx = fma(zrow[v], xg[xb + k * T + v], zx);
          sh.r.res[pos * S + k * T + uc] = static_cast<float>(base - zx + ex);
        };
        if (__builtin_expect(closure, 1)) {
#pragma unroll
          for (int k = 0; k < c; ++k) store_local(k, fma(gcoef, xs[xb + k * T + uc], z * xl[xb + k * T]));
        } else {
          const int row = sh.row[pos], es = row < 0 ? 0 : row / kNQ, p = row < 0 ? 0 : row - es * kNQ;
          double ex[c];
#pragma unroll
          for (int k = 0; k < c; ++k) ex[k] = z * xl[xb + k * T];
          const double* const gq = sh.coupling(es, p);
#pragma unroll 1
          for (unsigned m = active ? sh.cols[row] & kColumns : 0u; m != 0; m &= m - 1) {
            const int q = __builtin_ctz(m);
            const double gv = gq[q - p - 1];
            LdsR* const xq = x0 + sh.pos[es * kNQ + q] * S + uc;
#pragma unroll
            for (int k = 0; k < c; ++k) ex[k] = fma(gv, xq[xb + k * T], ex[k]);
          }
#pragma unroll
          for (int k = 0; k < c; ++k) store_local(k, ex[k]);
        }
        wave_fence();
      }
      // ---- outputs of the chunk from the group's own block: Q <- X or
      // Q <- Q + X, and Qint = dt X[:, :, 0] (only the group writes its block,
      // and not before its next X in the same buffer).  Issued after the green update, where the lane has
      // registers to spare, except where one workgroup fills the compute unit:
      // its waves would all be storing at once there, with no one's
      // multiply-adds to cover it (N = 6: 2.73 ms against 2.67 ms after the
      // first mode; N = 5, several workgroups: 1.22 against 1.25 ms).
      auto store_outputs = [&]() __attribute__((always_inline)) {
        if constexpr (Mode == kResidual) {
          // four consecutive values per lane
          constexpr int n4 = c * T / 4, it4 = (n4 + T - 1) / T, rest = c * T - 4 * n4;
          const float* const rg = sh.r.res + pos * S;
          char* const dst = Rb + roff - 4 * uc + m0 * (T * 4);
          if (active) {
#pragma unroll
            for (int j = 0; j < it4; ++j)
              if ((j + 1) * T <= n4 || j * T + uc < n4) {
                quad_t v;
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = rg[4 * (j * T + uc) + i];
                *reinterpret_cast<quad_t*>(dst + 16 * (j * T + uc)) = v;
              }
            if constexpr (rest > 0) {
#pragma unroll
              for (int i = 0; i < (rest + T - 1) / T; ++i)
                if (i * T + uc < rest) *reinterpret_cast<float*>(dst + 4 * (4 * n4 + i * T + uc)) = rg[4 * n4 + i * T + uc];
            }
          }
          return;
        }
        pair_t v[nst > 0 ? nst : 1];
        double last = 0.0, iv[nin];
#pragma unroll
        for (int j = 0; j < nst; ++j) {
          v[j].x = static_cast<double>(xo[xb + j * 2 * T]);
          v[j].y = static_cast<double>(xo[xb + j * 2 * T + 1]);
        }
        if constexpr (odd) last = static_cast<double>(xg[xb + c * T - 1]);
#pragma unroll
        for (int k = 0; k < nin; ++k) iv[k] = a.dt * static_cast<double>(xi[xb + k * T * T]);
        if constexpr (Mode == kCorrect) {
#pragma unroll
          for (int j = 0; j < nst; ++j) v[j] += qprev[j];
          last += qlast;
#pragma unroll
          for (int k = 0; k < nin; ++k) iv[k] += iprev[k];
        }
        if (active) {
#pragma unroll
          for (int j = 0; j < nst; ++j)
            if ((j + 1) * T <= np || j * T + u < np)
              *reinterpret_cast<pair_t*>(Qb + qoff + (m0 * T + j * 2 * T) * 8) = v[j];
          if constexpr (odd) {
            if (u == 0) *reinterpret_cast<double*>(Qb + qoff + (m0 * T + c * T - 1) * 8) = last;
          }
          if (a.Qint) {
#pragma unroll
            for (int k = 0; k < nin; ++k)
              if ((k + 1) * T <= c || k * T + u < c)
                *reinterpret_cast<double*>(Ib + ioff + (m0 + k * T) * 8) = iv[k];
          }
        }
      };
      // ---- green blocks: y_j = (A^{j*} X)_p of each mode, then the Khat
      // column on the lane's rows.  The X reads of a mode are issued before
      // the multiply-adds of the mode before it.
      if constexpr (green) {
        R xq[kStarNnz], y0 = R(0), y1 = R(0), y2 = R(0);
        auto read_x = [&](auto k) __attribute__((always_inline)) {
          constexpr int off = xb + decltype(k)::value * T;
          xq[0] = sp[0][off];
          xq[1] = sp[1][off];
          if (ns > 2) {
            asm volatile("");  // keep these branches: the rows are 2, 4 or 6 long for a whole wave
            xq[2] = sp[2][off];
            xq[3] = sp[3][off];
          }
          if (ns > 4) {
            asm volatile("");
            xq[4] = sp[4][off];
            xq[5] = sp[5][off];
          }
        };
        auto star = [&](auto k) __attribute__((always_inline)) {
          y0 = sa0[0] * xq[0];
          y1 = sa1[0] * xq[0];
          y2 = sa2[0] * xq[0];
          auto add = [&](int i) __attribute__((always_inline)) {
            y0 = fma(sa0[i], xq[i], y0);
            y1 = fma(sa1[i], xq[i], y1);
            y2 = fma(sa2[i], xq[i], y2);
          };
          add(1);
          if (ns > 2) {
            asm volatile("");
            add(2);
            add(3);
          }
          if (ns > 4) {
            asm volatile("");
            add(4);
            add(5);
          }
        };
        // groups of 16 coefficients [G0, G1) of this chunk, kAhead in flight
        constexpr int kAhead = 2;
        constexpr int first = P::col_start[m0], last = P::col_start[m0 + c - 1] + P::col_count[m0 + c - 1];
        constexpr int G0 = first / 16, G1 = (last + 15) / 16;
        for (int pass = 0;; ++pass) {
          R kc[kAhead + 1];
          read_x(ic<0>{});
          static_for<0, (kAhead < G1 - G0 ? kAhead : G1 - G0)>([&](auto i) __attribute__((always_inline)) {
            kc[(G0 + decltype(i)::value) % (kAhead + 1)] = kl[(G0 + decltype(i)::value) * 16];
          });
          star(ic<0>{});
          static_for<0, c>([&](auto k) __attribute__((always_inline)) {
            constexpr int kk = decltype(k)::value, m = m0 + kk;
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (kk + 1 < c) read_x(ic<kk + 1>{});
            static_for<0, P::col_count[m]>([&](auto i) __attribute__((always_inline)) {
              constexpr int e = P::col_start[m] + decltype(i)::value, G = e / 16;
              if constexpr ((e % 16 == 0 || e == first) && G + kAhead < G1) {
                __builtin_amdgcn_sched_barrier(0);
                kc[(G + kAhead) % (kAhead + 1)] = kl[(G + kAhead) * 16];
                __builtin_amdgcn_sched_barrier(0);
              }
              constexpr int j = P::dir[e];
              fmac_bcast<e % 16>(b[P::row[e]], kc[G % (kAhead + 1)], (j == 0) ? y0 : ((j == 1) ? y1 : y2));
            });
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (kk + 1 < c) star(ic<kk + 1>{});
            if constexpr (C::kAlone && kk == 0) {
              store_outputs();
              __builtin_amdgcn_sched_barrier(0);
            }
          });
          if (kNQ <= kStarNnz || __builtin_expect(!dense_star, 1)) break;
          // A longer star row: the update is linear in the columns, so the same
          // code runs again with the next kStarNnz (as many times as the wave's
          // longest row needs), then the first ones come back for the next chunk.
          int po = pos;
          asm volatile("" : "+v"(po));
          const int row = sh.row[po], es = row < 0 ? 0 : row / kNQ, p = row < 0 ? 0 : row - es * kNQ;
          unsigned cols = active ? sh.cols[row] >> kStarShift & kColumns : 0u;
          const bool again = __builtin_amdgcn_ballot_w64(__builtin_popcount(cols) > (pass + 1) * kStarNnz) != 0;
          constexpr bool kLast = g == 1 && cidx + 1 == nchunks(g, C::kChunk);
          if (!again && (pass == 0 || kLast)) break;
          for (int k = again ? (pass + 1) * kStarNnz : 0; k > 0; --k) cols &= cols - 1;
          ns = row_length(__builtin_popcount(cols));
          const char* const Sb = reinterpret_cast<const char*>(a.star + e0 * (3 * kNQ * kNQ));
          const unsigned soff = active ? 8u * ((es * 3 * kNQ + p) * kNQ) : 0u;
#pragma unroll
          for (int k = 0; k < kStarNnz; ++k) {
            const int q = cols != 0 ? __builtin_ctz(cols) : p;
            const double f = cols != 0 ? -a.dt : 0.0;
            cols &= cols - 1;
            const unsigned off = soff + 8u * q;
            sa0[k] = static_cast<R>(f * *reinterpret_cast<const double*>(Sb + off));
            sa1[k] = static_cast<R>(f * *reinterpret_cast<const double*>(Sb + off + 8 * kNQ * kNQ));
            sa2[k] = static_cast<R>(f * *reinterpret_cast<const double*>(Sb + off + 16 * kNQ * kNQ));
            sp[k] = x0 + (f != 0.0 ? sh.pos[es * kNQ + q] : po) * S + u;
          }
          if (!again) break;
        }
      }
      if constexpr (!green || !C::kAlone) store_outputs();
    });
  });
}

template <int N, typename R, int Mode>
hipError_t launch_solve(const PredictArgs& a, float* work, hipStream_t stream) {
  using C = SolveCfg<N, Mode>;
  const int64_t groups = (a.n + C::kE - 1) / C::kE;
  if (groups > 0x7fffffff) return hipErrorInvalidValue;
  hipLaunchKernelGGL((solve_kernel<N, R, Mode>), dim3(static_cast<unsigned>(groups)), dim3(C::kThreads), 0, stream, a,
                     work);
  return hipGetLastError();
}

}  // namespace
}  // namespace stp
