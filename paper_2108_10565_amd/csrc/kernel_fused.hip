// Register-resident kernels for Algorithm 3 of Wolf et al. (arXiv 2108.10565,
// section "Block-wise back-substitution"), one object per quantity count and
// degree N = STP_DEGREE: the solve and the residual (solve_kernel.hpp), and
// the float32 chain on the matrix cores.
//
// Shared structure.  One lane per column (element e, quantity p, time mode u)
// of the element's right-hand side b_pmu (eq:b_pmu), which keeps b[m] for all
// modes m below the top degree block in registers.  The green-block update
//     b[p, n, u] -= sum_j Khat^j[n, m] (A^{j*} X[:, m, u])_p ,  n < block_start(g)
// is lane-local once the star product y_j = (A^{j*} X[:, m, u])_p is known,
// so the lane applies it as a fully unrolled list of multiply-adds over the
// non-zeros of Khat (compile-time pattern), exactly the zeros the Lemma of
// section "Structure of the system matrix" and the Dubiner structure provide.
//
// Per chunk of modes m of degree block g (g = N .. 0):
//   1. dark-blue blocks and G coupling: X[p, m, s] = row s of
//      (Z - E*_pp I)^-1 times b[p, m, :] (float64).  For E*_pp = 0 that row is
//      a row of Z^-1, which is tridiagonal with a zero diagonal apart from its
//      two corner entries (the Legendre integration recurrence): two entries
//      instead of T.  A quantity o whose row of the strict upper part G of E*
//      holds one coupling G_op to an uncoupled quantity p (the poroelastic
//      u <- uf, v <- vf, w <- wf) uses the closed form
//      X_o = Zinv_o (b_o + G_op X_p) = zr . b_o + dr . b_p,
//      dr = G_op (row of Zinv_o) Zinv_p, so no extra round is needed; any
//      other coupled quantity follows level by level (level = longest
//      coupling chain below it);
//   2. green blocks: every lane reads X[q, m, u] of the quantities in its
//      star row, forms y_1..y_3 with its row of A^{1*}, A^{2*}, A^{3*}, and
//      subtracts Khat^j[n, m] y_j from its registers b[n];
//   3. outputs: X to Q and dt X[:, :, 0] to Qint (the matrix-core chain and a
//      tile that fills the compute unit issue them earlier).
// A^{j*} = dt A^j and E* = dt E are formed in-kernel, so every product runs
// with unit scaling (the paper's libxsmm alpha = 1 remark, section "Roofline
// model").
#include <type_traits>
#include <utility>

#include "common.hpp"
#include "generated/khat_tables.h"

#ifndef STP_DEGREE
#error "compile once per degree with -DSTP_DEGREE=N"
#endif

namespace stp {
namespace {

// Quantities of the system this object is compiled for: 13 (poroelastic) or
// 6 (damped Maxwell, section "Other applications").
#ifndef STP_NQ
#error "compile once per quantity count with -DSTP_NQ=Q"
#endif
constexpr int kNQ = STP_NQ;
static_assert(supported_nq(kNQ), "quantity count without kernels");

// Tile shape of the matrix-core chain: threads per workgroup (upper bound; rounded to
// whole elements and waves) and modes per chunk (degree blocks are split
// evenly).  Both come from the build, which takes them from its tile table.
#if !defined(STP_TILE_THREADS) || !defined(STP_TILE_CHUNK)
#error "compile with -DSTP_TILE_THREADS=T -DSTP_TILE_CHUNK=C (the tile table of the build)"
#endif
constexpr int kTileThreadsN = STP_TILE_THREADS;
constexpr int kChunkMax = STP_TILE_CHUNK;
static_assert(kTileThreadsN >= 64 && kTileThreadsN <= 1024 && kChunkMax >= 1, "tile shape");
constexpr int kMaxElems = 16;
// Non-zero columns kept per lane of a star-matrix row (union over the three
// directions).  The poroelastic Jacobians need at most 6 (normal-stress and
// pressure rows couple to the 6 velocities; velocity rows to 3 stresses and
// the pressure); for a row with more the solve kernel repeats the green update,
// the matrix-core chain reads the dense rows from global memory.
constexpr int kStarNnz = 6;

template <int I>
using ic = std::integral_constant<int, I>;

template <int Begin, class F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(ic<Begin + I>{}), ...);
}
// Calls f(ic<i>) for i = Begin .. End-1 with compile-time i.
template <int Begin, int End, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (End > Begin) static_for_impl<Begin>(f, std::make_integer_sequence<int, End - Begin>{});
}

// Smallest S >= len with nq S = t (mod 16) (nq odd), or the smallest odd
// S >= len (nq even, where no such S exists for odd t).
__host__ __device__ constexpr int stride_for(int len, int t, int nq) {
  for (int s = len; s < len + 32; ++s) {
    if (nq % 2 == 1 ? ((nq * s - t) % 16 + 16) % 16 == 0 : s % 2 == 1) return s;
  }
  return len;
}

template <int N>
struct Cfg {
  static constexpr int B = n_modes(N);
  static constexpr int T = N + 1;
  static constexpr int LN = block_start(N);        // register-resident rows (below the top block)
  static constexpr int LR = LN > 0 ? LN : 1;
  static constexpr int DN = block_size(N);         // modes of the top block (largest block)
  static constexpr int kCols = kNQ * T;            // lanes per element
  static constexpr int kElems =                    // elements per workgroup
      (kTileThreadsN / kCols) < kMaxElems ? (kTileThreadsN / kCols) : kMaxElems;
  static_assert(kElems >= 1, "the tile must hold at least one element");
  static constexpr int kThreads = (kElems * kCols + 63) / 64 * 64;
  static constexpr int kSlots = kElems + 1;        // + one dummy slot for spare lanes
  static constexpr int kChunk = kChunkMax < DN ? kChunkMax : DN;
  // The chunk buffers hold one block of S doubles per (element, quantity) row
  // in the order of the rows in memory (element-major), so a row's block is
  // row * S: the output passes address LDS and memory from the same row
  // index.  S is padded so that kNQ S = T (mod 16) when kNQ is odd: the LDS
  // address of lane (e, p, u) (lanes quantity-major) is then congruent to the
  // lane index modulo 16 doubles, 13 S = 7 making S = 3 = kElems T at N = 6,
  // so 16 consecutive lanes cover one 128-byte span of the banks without a
  // conflict.  One extra block at the end takes the writes of the spare lanes
  // past the last element (their values are never read back).
  static constexpr int kChunkT = kChunk * T;
  static constexpr int S = stride_for(kChunkT, T, kNQ);
  static constexpr int kRows = kElems * kNQ;       // real blocks
  static constexpr int kBufSize = (kRows + 1) * S; // + the spare lanes' block
  // Offset of the block of row `row` = element * kNQ + quantity; rows past
  // the last element (spare lanes, the dummy slot) share the last block.
  static __device__ __forceinline__ int rowblk(int row) { return (row < kRows ? row : kRows) * S; }
  static __device__ __forceinline__ int blk(int e, int q) { return rowblk(e * kNQ + q); }
};

// Degree block g is processed in nchunks(g) chunks of near-equal size.
__host__ __device__ constexpr int nchunks(int g, int cmax) { return (block_size(g) + cmax - 1) / cmax; }
__host__ __device__ constexpr int chunk_size(int g, int cmax, int i) {
  return block_size(g) / nchunks(g, cmax) + (i < block_size(g) % nchunks(g, cmax) ? 1 : 0);
}
__host__ __device__ constexpr int chunk_start(int g, int cmax, int i) {
  return block_start(g) + i * (block_size(g) / nchunks(g, cmax)) +
         (i < block_size(g) % nchunks(g, cmax) ? i : block_size(g) % nchunks(g, cmax));
}

// Lane tid -> (element slot es, quantity p, time mode u), quantity-major:
// the lanes of one quantity are contiguous (kElems * T of them), so the few
// quantities that take the dense dark-blue path (a non-zero diagonal source
// term, or a coupling) occupy few waves and the other waves skip it.  Spare
// lanes past kElems * kCols go to the dummy slot kElems.
template <int N>
struct LaneId {
  int es, p, u;
  __device__ __forceinline__ explicit LaneId(int tid) {
    using C = Cfg<N>;
    constexpr int per_q = C::kElems * C::T;
    if (tid < C::kElems * C::kCols) {
      p = tid / per_q;
      es = (tid % per_q) / C::T;
      u = tid % C::T;
    } else {
      const int i = tid - C::kElems * C::kCols;
      es = C::kElems;
      p = (i / C::T) % kNQ;
      u = i % C::T;
    }
  }
};

template <int N, typename R>
struct Shared {
  using C = Cfg<N>;
  double G[C::kSlots][kNQ][kNQ];            // E* (lower part zeroed)
  double zr[C::kThreads][C::T];             // per lane (e, p, u): row u of (Z - E*_pp I)^-1
  double dr[C::kThreads][C::T];             // per lane: row of Zinv_o G_op Zinv_p (closure coupling)
  int level[C::kSlots][kNQ];
  int maxlevel;
  unsigned flags;
  union {
    double A[C::kSlots][3][kNQ][kNQ];       // setup only: A^{j*} = dt A^j
    struct {
      R bufB[C::kBufSize];                  // b of the chunk: [e][p] blocks of [chunk][T], stride S
      R bufX[C::kBufSize];                  // X of the chunk, same layout
    } c;
  } u;
};

// Solves (Z - z I)^T y = rhs by Gauss-Jordan elimination without pivoting.
// For z = dt E_pp < 0.5 (the range stp_validate admits) the pivots stay away
// from zero: over z in [-1e7, 0.5) and every degree N <= 7 the smallest is at
// least 3% of max|Z| + |z| (checked numerically).  With rhs = e_s, y is row s
// of (Z - z I)^-1.
template <int T>
__device__ __forceinline__ void zt_solve(double z, const double (&rhs)[T], double (&out)[T]) {
  double a[T][T + 1];
#pragma unroll
  for (int r = 0; r < T; ++r) {
#pragma unroll
    for (int c = 0; c < T; ++c) a[r][c] = z_entry(c, r) - (r == c ? z : 0.0);  // transpose
    a[r][T] = rhs[r];
  }
#pragma unroll
  for (int k = 0; k < T; ++k) {
    const double inv = 1.0 / a[k][k];
#pragma unroll
    for (int c = k; c <= T; ++c) a[k][c] *= inv;
#pragma unroll
    for (int r = 0; r < T; ++r) {
      if (r == k) continue;
      const double f = a[r][k];
#pragma unroll
      for (int c = k; c <= T; ++c) a[r][c] -= f * a[k][c];
    }
  }
#pragma unroll
  for (int r = 0; r < T; ++r) out[r] = a[r][T];
}

// The usage-ordered Khat table of degree N in precision R (the solve kernel
// copies it to LDS).
template <int N, typename R>
__device__ __forceinline__ const R* khat_sparse() {
  if constexpr (sizeof(R) == 8) {
    if constexpr (N == 0) return stp_gen::kKhatSparse0;
    else if constexpr (N == 1) return stp_gen::kKhatSparse1;
    else if constexpr (N == 2) return stp_gen::kKhatSparse2;
    else if constexpr (N == 3) return stp_gen::kKhatSparse3;
    else if constexpr (N == 4) return stp_gen::kKhatSparse4;
    else if constexpr (N == 5) return stp_gen::kKhatSparse5;
    else if constexpr (N == 6) return stp_gen::kKhatSparse6;
    else return stp_gen::kKhatSparse7;
  } else {
    if constexpr (N == 0) return stp_gen::kKhatSparseF0;
    else if constexpr (N == 1) return stp_gen::kKhatSparseF1;
    else if constexpr (N == 2) return stp_gen::kKhatSparseF2;
    else if constexpr (N == 3) return stp_gen::kKhatSparseF3;
    else if constexpr (N == 4) return stp_gen::kKhatSparseF4;
    else if constexpr (N == 5) return stp_gen::kKhatSparseF5;
    else if constexpr (N == 6) return stp_gen::kKhatSparseF6;
    else return stp_gen::kKhatSparseF7;
  }
}

// Copies columns [m0 T, m0 T + PER) of the (element, quantity) rows of the
// group (a [n][kNQ][B T] array in memory) into the chunk buffer `buf` (block
// layout of Cfg::blk), converted to R.  Every lane issues all its loads
// before its LDS stores, so the group waits for one memory latency, not one
// per row segment.
template <int N, typename R, int PER, typename Src>
__device__ __forceinline__ void stage_rows(R* buf, const Src* src, int64_t e0, int m0T, int nloc, int tid) {
  using C = Cfg<N>;
  constexpr int kIters = (C::kElems * kNQ * PER + C::kThreads - 1) / C::kThreads;
  const int limit = nloc * kNQ * PER;
  Src v[kIters];
#pragma unroll
  for (int k = 0; k < kIters; ++k) {
    const int i = tid + k * C::kThreads;
    const int row = i / PER, r = i % PER;
    v[k] = i < limit ? src[(e0 * kNQ + row) * (C::B * C::T) + m0T + r] : Src(0);
  }
#pragma unroll
  for (int k = 0; k < kIters; ++k) {
    const int i = tid + k * C::kThreads;
    const int row = i / PER, r = i % PER;
    if (i < limit) buf[C::rowblk(row) + r] = static_cast<R>(v[k]);
  }
}

// Position of chunk ci of degree block g in the chunk order (blocks from N
// down, chunks ascending).
__host__ __device__ constexpr int chunk_index(int N, int g, int ci, int cmax) {
  int s = 0;
  for (int h = N; h > g; --h) s += nchunks(h, cmax);
  return s + ci;
}
}  // namespace
}  // namespace stp

#include "solve_kernel.hpp"

namespace stp {
namespace {

// Per-lane setup of the matrix-core chain: stages E* and
// A^{j*} of the group, then per lane the sparse star row, the G coupling of
// the lane's quantity, row u of (Z - E*_pp I)^-1 (to LDS) and the closure row
// dr (to LDS); the dependency levels of the strict upper part G of E* only
// when some coupling is not of the closure form.
template <int N, typename R>
struct LaneSetup {
  using C = Cfg<N>;
  R sa0[kStarNnz], sa1[kStarNnz], sa2[kStarNnz];
  int sq[kStarNnz];
  int gp, gcount;
  double gcoef;
  bool dense_star, closure;
  int maxlevel, mylevel;

  __device__ __forceinline__ void run(Shared<N, R>& sh, const PredictArgs& a, int64_t e0, int nloc, int tid,
                                      int es, int p, int u, bool active, int cb) {
    constexpr int kThreads = C::kThreads, T = C::T;
    unsigned bad = 0;  // input conditions the elimination without pivoting cannot take
    // E and the star matrices of the group: every load is issued before the
    // first LDS store, so the group waits for one memory latency
    constexpr int kEIt = (C::kSlots * kNQ * kNQ + kThreads - 1) / kThreads;
    constexpr int kAIt = (C::kSlots * 3 * kNQ * kNQ + kThreads - 1) / kThreads;
    double ev[kEIt], av[kAIt];
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
    for (int k = 0; k < kEIt; ++k) {
      const int i = tid + k * kThreads;
      const int r = (i / kNQ) % kNQ, c = i % kNQ;
      const double v = a.dt * ev[k];
      if (c < r && v != 0.0) bad |= kInputNotUpper;
      if (c == r && v >= 0.5) bad |= kInputSingular;
      if (i < C::kSlots * kNQ * kNQ) (&sh.G[0][0][0])[i] = c >= r ? v : 0.0;
    }
    if (bad && a.status) atomicOr(a.status, bad);
#pragma unroll
    for (int k = 0; k < kAIt; ++k) {
      const int i = tid + k * kThreads;
      if (i < C::kSlots * 3 * kNQ * kNQ) (&sh.u.A[0][0][0][0])[i] = a.dt * av[k];
    }
    if (tid == 0) {
      sh.maxlevel = 0;
      sh.flags = 0;
    }
    __syncthreads();
    // G coupling of this lane's quantity (the first non-zero right of the
    // diagonal and their count), and whether that partner couples further
    gcount = 0;
    gp = p;
    gcoef = 0.0;
#pragma unroll
    for (int q = 1; q < kNQ; ++q) {
      const double gq = sh.G[es][p][q];
      if (q > p && gq != 0.0) {
        if (gcount == 0) {
          gcoef = gq;
          gp = q;
        }
        ++gcount;
      }
    }
    bool partner_coupled = false;
#pragma unroll
    for (int q = 1; q < kNQ; ++q)
      partner_coupled = partner_coupled || (q > gp && sh.G[es][gp][q] != 0.0);
    // sparse row p of the three star matrices: the columns with a non-zero
    // in any direction, in ascending order (a bit mask, consumed lowest bit
    // first)
    unsigned mask = 0;
#pragma unroll
    for (int q = 0; q < kNQ; ++q) {
      const double v0 = sh.u.A[es][0][p][q], v1 = sh.u.A[es][1][p][q], v2 = sh.u.A[es][2][p][q];
      if (v0 != 0.0 || v1 != 0.0 || v2 != 0.0) mask |= 1u << q;
    }
    const bool overflow = active && __builtin_popcount(mask) > kStarNnz;
#pragma unroll
    for (int k = 0; k < kStarNnz; ++k) {
      const bool live = mask != 0;
      const int q = live ? __builtin_ctz(mask) : p;
      mask &= mask - 1;
      const double v0 = sh.u.A[es][0][p][q], v1 = sh.u.A[es][1][p][q], v2 = sh.u.A[es][2][p][q];
      sa0[k] = live ? static_cast<R>(v0) : R(0);
      sa1[k] = live ? static_cast<R>(v1) : R(0);
      sa2[k] = live ? static_cast<R>(v2) : R(0);
      sq[k] = (live ? C::blk(es, q) : cb) + u;
    }
    // row u of (Z - E*_pp I)^-1.  Without a diagonal source it is row u of
    // Z^-1, which has two non-zeros (generated table); otherwise it comes from
    // an elimination, done only by waves holding such a lane.
    {
      const double z = sh.G[es][p][p];
      using ZS = stp_gen::ZinvSparse<N>;
      double zr[T];
#pragma unroll
      for (int v = 0; v < T; ++v)
        zr[v] = (ZS::col[2 * u] == v ? ZS::val[2 * u] : 0.0) + (ZS::col[2 * u + 1] == v ? ZS::val[2 * u + 1] : 0.0);
      if (__builtin_amdgcn_ballot_w64(z != 0.0) != 0) {
        double e_u[T], zs[T];
#pragma unroll
        for (int v = 0; v < T; ++v) e_u[v] = (v == u) ? 1.0 : 0.0;
        zt_solve<T>(z, e_u, zs);
        if (z != 0.0) {
#pragma unroll
          for (int v = 0; v < T; ++v) zr[v] = zs[v];
        }
      }
#pragma unroll
      for (int v = 0; v < T; ++v) sh.zr[tid][v] = zr[v];
    }
    // one barrier for the workgroup-uniform flags (scalar branches, no exec
    // masking); it also orders the reads of A before the chunk buffers (which
    // share its storage) are written, and the rows of Zinv before their reads
    // below.  The closure form of the coupling applies when every coupled
    // quantity couples to one quantity that itself is uncoupled (the
    // poroelastic case).
    {
      const unsigned f = (overflow ? 1u : 0u) | ((active && (gcount > 1 || (gcount == 1 && partner_coupled))) ? 2u : 0u);
      if (f) atomicOr(&sh.flags, f);
    }
    __syncthreads();
    const unsigned flags = __builtin_amdgcn_readfirstlane(sh.flags);
    dense_star = (flags & 1u) != 0;
    closure = (flags & 2u) == 0;
    // closure row: X_o = Zinv_o (b_o + g X_p) = zr . b_o + dr . b_p with
    //   dr[w] = g sum_v (row u of Zinv_o)[v] Zinv_p[v][w],
    // the rows Zinv_p[v] being those of the partner's lanes (e, p, v)
    {
      double dr[T];
#pragma unroll
      for (int w = 0; w < T; ++w) dr[w] = 0.0;
      if (gcount == 1 && closure) {
        constexpr int per_q = C::kElems * T;
        double zr[T];
#pragma unroll
        for (int v = 0; v < T; ++v) zr[v] = sh.zr[tid][v];
#pragma unroll
        for (int v = 0; v < T; ++v) {
          const double cv = gcoef * zr[v];
#pragma unroll
          for (int w = 0; w < T; ++w) dr[w] = fma(cv, sh.zr[gp * per_q + es * T + v][w], dr[w]);
        }
      }
#pragma unroll
      for (int v = 0; v < T; ++v) sh.dr[tid][v] = dr[v];
    }
    maxlevel = 0;
    mylevel = 0;
    if (!closure) {
      // dependency levels of a general upper-triangular E (level = longest
      // coupling chain below a quantity), one thread per element
      if (tid < nloc) {
        int lev[kNQ];
        int mx = 0;
#pragma unroll
        for (int o = kNQ - 1; o >= 0; --o) {
          int l = 0;
#pragma unroll
          for (int q = o + 1; q < kNQ; ++q)
            if (sh.G[tid][o][q] != 0.0 && lev[q] + 1 > l) l = lev[q] + 1;
          lev[o] = l;
          sh.level[tid][o] = l;
          mx = l > mx ? l : mx;
        }
        atomicMax(&sh.maxlevel, mx);
      }
      __syncthreads();
      maxlevel = sh.maxlevel;
      mylevel = active ? sh.level[es][p] : 0;
    }
  }

  // y_j = (A^{j*} X[:, m, u])_p for j = 1..3 from the chunk buffer
  template <int kk>
  __device__ __forceinline__ void star(const R* bufX, const PredictArgs& a, int64_t e0, int es, int p, int u,
                                       bool active, R& y0, R& y1, R& y2) const {
    constexpr int T = C::T;
    y0 = y1 = y2 = R(0);
    // opaque per-mode offset: this mode's LDS reads stay here
    int xoff = kk * T;
    asm volatile("" : "+v"(xoff));
    const R* xs = bufX + xoff;
    if (!dense_star) {
#pragma unroll
      for (int k = 0; k < kStarNnz; ++k) {
        const R xq = xs[sq[k]];
        y0 = fma(sa0[k], xq, y0);
        y1 = fma(sa1[k], xq, y1);
        y2 = fma(sa2[k], xq, y2);
      }
    } else {
      const double* st = a.star + (active ? e0 + es : 0) * (3 * kNQ * kNQ) + p * kNQ;
#pragma unroll
      for (int q = 0; q < kNQ; ++q) {
        const R xq = xs[C::blk(es, q) + u];
        y0 = fma(static_cast<R>(a.dt * st[q]), xq, y0);
        y1 = fma(static_cast<R>(a.dt * st[kNQ * kNQ + q]), xq, y1);
        y2 = fma(static_cast<R>(a.dt * st[2 * kNQ * kNQ + q]), xq, y2);
      }
    }
  }
};

// ---------------------------------------------------------------------------
// Float32 chain with the green-block update on the matrix cores.
//
// The green update of a chunk is a product with a shared left operand:
//   b[n, col] -= sum_k Khat(k)[n] Y[k, col],   k = (mode mm of the chunk, direction j),
// Y[k, col] = (A^{j*} X[:, mm, u])_p for column col = (element, quantity p, time
// mode u), n below the block start.  It runs as v_mfma_f32_16x16x4f32 with
// float32 accumulation: wave w keeps the right-hand side rows below the top
// degree block of its own 64 columns (4 column tiles of 16) in accumulator
// tiles of 16 rows; the A operand is a 16-row slice of -Khat read from a
// generated table, the B operand the wave's Y rows, which its lanes compute
// (sparse star rows, vector ALU) into a per-wave LDS buffer.  The dark-blue
// solves stay float64 on the vector ALU, and the matrix-core instructions of a
// chunk overlap the vector work that follows them.  Accumulator layout of
// the 16x16x4 instruction: lane l holds column l % 16, rows 4 (l / 16) + r,
// r = 0..3; A operand A[l % 16][l / 16]; B operand B[l / 16][l % 16].
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int kMG = 4;        // modes per k group: 3 k-blocks of 4 (mode, direction) pairs
constexpr int kYStride = 80;  // floats per k row of a wave's Y buffer: 64 columns, padded against bank conflicts

template <int N>
struct MfmaCfg {
  using C = Cfg<N>;
  static constexpr int kWaves = C::kThreads / 64;
  static constexpr int RN = (C::LN + 15) / 16;  // accumulator row tiles (rows below the top block)
  static constexpr int RA = RN > 0 ? RN : 1;
  static constexpr int kRealCols = C::kElems * C::kCols;
};

template <int N>
struct SharedM {
  Shared<N, float> s;
  float ybuf[MfmaCfg<N>::kWaves][3 * kMG][kYStride];
};

template <int N>
__device__ __forceinline__ const float* khat_mfma() {
  if constexpr (N == 0) return stp_gen::kKhatMfma0;
  else if constexpr (N == 1) return stp_gen::kKhatMfma1;
  else if constexpr (N == 2) return stp_gen::kKhatMfma2;
  else if constexpr (N == 3) return stp_gen::kKhatMfma3;
  else if constexpr (N == 4) return stp_gen::kKhatMfma4;
  else if constexpr (N == 5) return stp_gen::kKhatMfma5;
  else if constexpr (N == 6) return stp_gen::kKhatMfma6;
  else return stp_gen::kKhatMfma7;
}

// Algorithm 3 in float32 with the green update on the matrix cores (dark-blue
// solves in float64).  kInit: b = Q0 (S^-1 w), Q <- X.  kCorrect: b = the
// residual in `rin` (float), Q <- Q + X.
template <int N, int Mode>
__global__ __launch_bounds__(Cfg<N>::kThreads) void mfma_solve_kernel(PredictArgs a, const float* rin) {
  using C = Cfg<N>;
  using MC = MfmaCfg<N>;
  using R = float;
  constexpr int B = C::B, T = C::T, kE = C::kElems, kThreads = C::kThreads;
  __shared__ SharedM<N> shm;
  Shared<N, R>& sh = shm.s;
  R* const bufB = sh.u.c.bufB;
  R* const bufX = sh.u.c.bufX;
  const int tid = threadIdx.x;
  const int lane = tid & 63, lrow = lane >> 4, lcol = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const int64_t e0 = static_cast<int64_t>(blockIdx.x) * kE;
  const int64_t nloc64 = a.n - e0 < kE ? a.n - e0 : kE;
  const int nloc = static_cast<int>(nloc64);
  const LaneId<N> lid(tid);
  const int es = lid.es, p = lid.p, u = lid.u;
  const bool active = es < nloc;
  const int cb = C::blk(es, p);
  float* const yb = &shm.ybuf[wave][0][0];

  // Column tiles of this wave holding real columns (wave-uniform), and the
  // chunk-buffer offset blk(e, p) + u of this lane's column in each tile.
  const int nct = __builtin_amdgcn_readfirstlane(
      (MC::kRealCols - 64 * wave) >= 64 ? 4 : ((MC::kRealCols - 64 * wave) > 0 ? (MC::kRealCols - 64 * wave + 15) / 16 : 0));
  int coff[4];
  v4f acc[4][MC::RA];
  static_for<0, 4>([&](auto ctc) __attribute__((always_inline)) {
    constexpr int ct = decltype(ctc)::value;
    const LaneId<N> cid(64 * wave + 16 * ct + lcol);
    coff[ct] = C::blk(cid.es, cid.p) + cid.u;
    const bool cact = cid.es < nloc;
    const int64_t crow = (cact ? e0 + cid.es : 0) * kNQ + cid.p;
    // accumulators: b rows below the top block
    static_for<0, MC::RA>([&](auto rtc) __attribute__((always_inline)) {
      constexpr int rt = decltype(rtc)::value;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 16 * rt + 4 * lrow + r;
        float v = 0.0f;
        if (cact && row < C::LN) {
          if constexpr (Mode == kInit) v = static_cast<float>(a.Q0[crow * B + row] * sinv_w(cid.u));
          else v = rin[crow * (B * T) + row * T + cid.u];
        }
        acc[ct][rt][r] = v;
      }
    });
  });
  for (int i = lane; i < 3 * kMG * kYStride; i += 64) yb[i] = 0.0f;
  const float* const ktab = khat_mfma<N>();

  constexpr int kFirstC = chunk_size(N, C::kChunk, 0), kFirstM = chunk_start(N, C::kChunk, 0);
  constexpr int kFirstPer = (kE * kNQ * kFirstC + kThreads - 1) / kThreads;
  double q_first[kFirstPer];
  if constexpr (Mode == kInit) {
#pragma unroll
    for (int k = 0; k < kFirstPer; ++k) {
      const int i = tid + k * kThreads;
      const int ee = i / (kNQ * kFirstC), pp = (i / kFirstC) % kNQ, kk = i % kFirstC;
      q_first[k] = (ee < nloc) ? a.Q0[((e0 + ee) * kNQ + pp) * B + kFirstM + kk] : 0.0;
    }
  }
  LaneSetup<N, R> L;
  L.run(sh, a, e0, nloc, tid, es, p, u, active, cb);
  const int pb = C::blk(es, L.gp);
  using ZS = stp_gen::ZinvSparse<N>;
  const int cz0 = cb + ZS::col[2 * u], cz1 = cb + ZS::col[2 * u + 1];
  const double zv0 = ZS::val[2 * u], zv1 = ZS::val[2 * u + 1];
  const bool wave_stiff = __builtin_amdgcn_ballot_w64(sh.G[es][p][p] != 0.0) != 0;
  const bool wave_coupled = __builtin_amdgcn_ballot_w64(L.gcount == 1) != 0;

  static_for<0, N + 1>([&](auto gi) __attribute__((always_inline)) {
    constexpr int g = N - decltype(gi)::value;
    static_for<0, nchunks(g, C::kChunk)>([&](auto ci) __attribute__((always_inline)) {
      constexpr int m0 = chunk_start(g, C::kChunk, decltype(ci)::value);
      constexpr int c = chunk_size(g, C::kChunk, decltype(ci)::value);
      constexpr int kOut = (kE * kNQ * c * T + kThreads - 1) / kThreads;
      // 1. right-hand side of the chunk to LDS
      if constexpr (g == N) {
        if constexpr (Mode == kInit) {
          constexpr int per_thread = (kE * kNQ * c + kThreads - 1) / kThreads;
          double q[per_thread];
          if constexpr (decltype(ci)::value == 0) {
#pragma unroll
            for (int k = 0; k < per_thread; ++k) q[k] = q_first[k];
          } else {
#pragma unroll
            for (int k = 0; k < per_thread; ++k) {
              const int i = tid + k * kThreads;
              const int ee = i / (kNQ * c), pp = (i / c) % kNQ, kk = i % c;
              q[k] = (ee < nloc) ? a.Q0[((e0 + ee) * kNQ + pp) * B + m0 + kk] : 0.0;
            }
          }
#pragma unroll
          for (int k = 0; k < per_thread; ++k) {
            const int i = tid + k * kThreads;
            const int ee = i / (kNQ * c), pp = (i / c) % kNQ, kk = i % c;
            if (ee < nloc) {
#pragma unroll
              for (int uu = 0; uu < T; ++uu) bufB[C::blk(ee, pp) + kk * T + uu] = static_cast<R>(q[k] * sinv_w(uu));
            }
          }
        } else {
          stage_rows<N, R, c * T>(bufB, rin, e0, m0 * T, nloc, tid);
        }
      } else {
        // rows m0 .. m0 + c - 1 leave the accumulators of this wave's columns
        constexpr int rt0 = m0 / 16, rt1 = (m0 + c - 1) / 16;
        static_for<0, 4>([&](auto ctc) __attribute__((always_inline)) {
          constexpr int ct = decltype(ctc)::value;
          if (ct < nct) {
            static_for<rt0, rt1 + 1>([&](auto rtc) __attribute__((always_inline)) {
              constexpr int rt = decltype(rtc)::value;
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                const int mm = 16 * rt + 4 * lrow + r - m0;
                if (mm >= 0 && mm < c) bufB[coff[ct] + mm * T] = acc[ct][rt][r];
              }
            });
          }
        });
      }
      __syncthreads();
      // 2. dark-blue blocks and G coupling (float64)
      if (L.closure) {
        auto dark_blue = [&](auto stiff_c, auto coupled_c) __attribute__((always_inline)) {
          constexpr bool kStiff = decltype(stiff_c)::value, kCoupled = decltype(coupled_c)::value;
          double zr[T], drr[T];
          if constexpr (kStiff) {
#pragma unroll
            for (int v = 0; v < T; ++v) zr[v] = sh.zr[tid][v];
          }
          if constexpr (kCoupled) {
#pragma unroll
            for (int v = 0; v < T; ++v) drr[v] = sh.dr[tid][v];
          }
          static_for<0, c>([&](auto k) __attribute__((always_inline)) {
            constexpr int kk = decltype(k)::value;
            double x;
            if constexpr (kStiff) {
              x = 0.0;
#pragma unroll
              for (int v = 0; v < T; ++v) x = fma(zr[v], static_cast<double>(bufB[cb + kk * T + v]), x);
            } else {
              x = fma(zv0, static_cast<double>(bufB[cz0 + kk * T]), zv1 * static_cast<double>(bufB[cz1 + kk * T]));
            }
            if constexpr (kCoupled) {
#pragma unroll
              for (int v = 0; v < T; ++v) x = fma(drr[v], static_cast<double>(bufB[pb + kk * T + v]), x);
            }
            bufX[cb + kk * T + u] = static_cast<R>(x);
          });
        };
        using yes = std::true_type;
        using no = std::false_type;
        if (wave_stiff) {
          if (wave_coupled) dark_blue(yes{}, yes{});
          else dark_blue(yes{}, no{});
        } else {
          if (wave_coupled) dark_blue(no{}, yes{});
          else dark_blue(no{}, no{});
        }
      } else {
        double zr[T];
#pragma unroll
        for (int v = 0; v < T; ++v) zr[v] = sh.zr[tid][v];
        static_for<0, c>([&](auto k) __attribute__((always_inline)) {
          constexpr int kk = decltype(k)::value;
          double x = 0.0;
#pragma unroll
          for (int v = 0; v < T; ++v) x = fma(zr[v], static_cast<double>(bufB[cb + kk * T + v]), x);
          bufX[cb + kk * T + u] = static_cast<R>(x);
        });
        for (int r = 1; r <= L.maxlevel; ++r) {
          __syncthreads();
          if (L.mylevel == r) {
            static_for<0, c>([&](auto k) __attribute__((always_inline)) {
              constexpr int kk = decltype(k)::value;
              double accd[T];
#pragma unroll
              for (int v = 0; v < T; ++v) accd[v] = static_cast<double>(bufB[cb + kk * T + v]);
              for (int q = p + 1; q < kNQ; ++q) {
                const double gq = sh.G[es][p][q];
                if (gq != 0.0) {
                  const int qb = C::blk(es, q) + kk * T;
#pragma unroll
                  for (int v = 0; v < T; ++v) accd[v] = fma(gq, static_cast<double>(bufX[qb + v]), accd[v]);
                }
              }
              double x = 0.0;
#pragma unroll
              for (int v = 0; v < T; ++v) x = fma(zr[v], accd[v], x);
              bufX[cb + kk * T + u] = static_cast<R>(x);
            });
          }
        }
      }
      __syncthreads();
      // 3. outputs of the chunk: Q <- X (kInit) or Q <- Q + X (kCorrect) in a
      //    rolled loop of groups of three values per lane, contiguous runs,
      //    streaming stores; then Qint
      {
        constexpr int per = c * T;
        const int limit = nloc * kNQ * per;
        double* Qg = a.Q + e0 * (kNQ * B * T) + m0 * T;
        auto lds_index = [&](int i) __attribute__((always_inline)) { return C::rowblk(i / per) + i % per; };
        {
          constexpr int kOutGroup = 3;
          constexpr int nOut = (kOut + kOutGroup - 1) / kOutGroup;
#pragma unroll 1
          for (int gi = 0; gi < nOut; ++gi) {
            double xv[kOutGroup], qv[kOutGroup];
#pragma unroll
            for (int k = 0; k < kOutGroup; ++k) {
              const int i = tid + (gi * kOutGroup + k) * kThreads;
              qv[k] = (Mode == kCorrect && i < limit) ? Qg[(i / per) * (B * T) + i % per] : 0.0;
              xv[k] = static_cast<double>(bufX[lds_index(i)]);
            }
#pragma unroll
            for (int k = 0; k < kOutGroup; ++k) {
              const int i = tid + (gi * kOutGroup + k) * kThreads;
              if (i < limit) __builtin_nontemporal_store(xv[k] + qv[k], &Qg[(i / per) * (B * T) + i % per]);
            }
          }
        }
        if (a.Qint) {
          double* Ig = a.Qint + e0 * (kNQ * B);
          constexpr int kInt = (kE * kNQ * c + kThreads - 1) / kThreads;
          const int ilimit = nloc * kNQ * c;
#pragma unroll
          for (int k = 0; k < kInt; ++k) {
            const int j = tid + k * kThreads;
            const int row = j / c, kk = j % c;
            double v = a.dt * static_cast<double>(bufX[C::rowblk(row) + kk * T]);
            if constexpr (Mode == kCorrect) v += j < ilimit ? Ig[row * B + m0 + kk] : 0.0;
            if (j < ilimit) __builtin_nontemporal_store(v, &Ig[row * B + m0 + kk]);
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      // 4. green blocks on the matrix cores, in groups of kMG modes
      if constexpr (g > 0) {
        constexpr int RG = (block_start(g) + 15) / 16;   // row tiles holding rows below block g
        static_for<0, (c + kMG - 1) / kMG>([&](auto grc) __attribute__((always_inline)) {
          constexpr int mg0 = decltype(grc)::value * kMG;
          constexpr int gm = (c - mg0) < kMG ? (c - mg0) : kMG;
          constexpr int nkb = (3 * gm + 3) / 4;
          // A = -Khat rows 16 rt + l % 16 of (mode, direction) k = 4 kb + l / 16,
          // loaded first so that the loads overlap the star products
          constexpr int base = stp_gen::KhatMfma<N>::off[m0 + mg0];
          float av[RG][nkb];
#pragma unroll
          for (int kb = 0; kb < nkb; ++kb) {
            // k past the group's 3 gm pairs pads the last k-block: A = 0 there
            // (the load address is clamped to the group's first pair)
            const int k = 4 * kb + lrow;
            const bool live = k < 3 * gm;
            const int kc = live ? k : 0;
            const int mm = kc / 3, j = kc - 3 * mm;
#pragma unroll
            for (int rt = 0; rt < RG; ++rt) {
              const float v = ktab[base + mm * (RG * 48) + (rt * 3 + j) * 16 + lcol];
              av[rt][kb] = live ? v : 0.0f;
            }
          }
          // star products of the group's modes -> Y rows k = 3 mm + j of this wave
          static_for<0, gm>([&](auto mmc) __attribute__((always_inline)) {
            constexpr int mm = decltype(mmc)::value;
            R y0, y1, y2;
            L.template star<mg0 + mm>(bufX, a, e0, es, p, u, active, y0, y1, y2);
            yb[(3 * mm + 0) * kYStride + lane] = y0;
            yb[(3 * mm + 1) * kYStride + lane] = y1;
            yb[(3 * mm + 2) * kYStride + lane] = y2;
          });
          // B = Y (k = 4 kb + l / 16, column l % 16 of tile ct)
          float bv[4][nkb];
          static_for<0, 4>([&](auto ctc) __attribute__((always_inline)) {
            constexpr int ct = decltype(ctc)::value;
#pragma unroll
            for (int kb = 0; kb < nkb; ++kb) bv[ct][kb] = yb[(4 * kb + lrow) * kYStride + 16 * ct + lcol];
          });
          // k-blocks outermost: consecutive instructions update different
          // accumulator tiles, so none waits on the previous one's result
#pragma unroll
          for (int kb = 0; kb < nkb; ++kb) {
            static_for<0, 4>([&](auto ctc) __attribute__((always_inline)) {
              constexpr int ct = decltype(ctc)::value;
              if (ct < nct) {
                static_for<0, RG>([&](auto rtc) __attribute__((always_inline)) {
                  constexpr int rt = decltype(rtc)::value;
                  acc[ct][rt] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[rt][kb], bv[ct][kb], acc[ct][rt], 0, 0, 0);
                });
              }
            });
          }
        });
      }
    });
  });
}

}  // namespace

template <>
hipError_t launch_fused<STP_NQ, STP_DEGREE>(const PredictArgs& a, int precision, int refine_steps,
                                            float* workspace, bool valu_float_chain, hipStream_t stream) {
  constexpr int N = STP_DEGREE;
  using C = Cfg<N>;
  const int64_t groups = (a.n + C::kElems - 1) / C::kElems;
  if (groups > 0x7fffffff) return hipErrorInvalidValue;
  const dim3 grid(static_cast<unsigned>(groups)), block(C::kThreads);
  if (precision == 0) {
    return launch_solve<N, double, kInit>(a, nullptr, stream);
  }
  hipError_t err;
  if (valu_float_chain) {
    err = launch_solve<N, float, kInit>(a, nullptr, stream);
  } else {
    hipLaunchKernelGGL((mfma_solve_kernel<N, kInit>), grid, block, 0, stream, a, nullptr);
    err = hipGetLastError();
  }
  for (int k = 0; k < refine_steps && err == hipSuccess; ++k) {
    err = launch_solve<N, double, kResidual>(a, workspace, stream);
    if (err != hipSuccess) break;
    if (valu_float_chain) {
      err = launch_solve<N, float, kCorrect>(a, workspace, stream);
    } else {
      hipLaunchKernelGGL((mfma_solve_kernel<N, kCorrect>), grid, block, 0, stream, a,
                         static_cast<const float*>(workspace));
      err = hipGetLastError();
    }
  }
  return err;
}

}  // namespace stp
