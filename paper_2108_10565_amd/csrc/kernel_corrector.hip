// Corrector of one ADER-DG time step (section "ADER-DG discretisation": the
// semi-discrete system eq:semi_discrete integrated over the step, with the
// predictor's time-integrated DOFs Qint = int Q dt in place of the solution):
//
//   Q <- Q + sum_j A^j Qint V^j + E Qint
//          - sum_f ( Gp_f Qint Fl_f + Gm_f Qint_nb(f) Fn_{f, j(f), h(f)} )
//
// V^j, Fl, Fn: reference volume / own-face / neighbour-face tables divided by
// the mass of the test function; Gp_f, Gm_f: the Godunov split of the face's
// normal Jacobian, scaled by 2 |S_f| / |J| (host-built per face).  The volume
// term is the integrated-by-parts flux form of A q_x + B q_y + C q_z, the face
// term Godunov's upwind flux An^+ q^- + An^- q^+ across each face.
//
// Every term is a product G X T (quantities x quantities, quantities x modes,
// modes x modes) and both products run on the float64 matrix cores
// (v_mfma_f64_16x16x4f64), one wave per element and range of output tiles,
// without LDS and without barriers: W^T = X^T G^T is formed tile by tile (16
// modes x 16 quantities, 4 instructions), and its accumulator registers are,
// as they stand, the A operand of W T: register r of lane l holds quantity
// l % 16 of mode 4 r + l / 16 of the tile, exactly what step r needs.  X^T, G^T
// and the tables are read straight from memory (Qint and the operators once
// per element, the tables from the caches, prefetched one term ahead).
#include "common.hpp"

namespace stp {
namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

__device__ __forceinline__ v4d mfma(double a, double b, v4d c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Operand layout of v_mfma_f64_16x16x4f64 (checked on gfx950 with an in-bounds
// probe of one wave): lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16];
// accumulator register r of lane l is row l / 16 + 4 r, column l % 16.
//
// TPW: output tiles (16 modes) per wave; an element takes
// ceil(NT / TPW) waves.
template <int NQ, int N, int TPW>
__global__ __launch_bounds__(256, TPW > 1 ? 2 : 3) void corrector_kernel(CorrectArgs a) {
  constexpr int B = n_modes(N), QB = NQ * B, Q2 = NQ * NQ;
  constexpr int NT = (B + 15) / 16, kParts = (NT + TPW - 1) / TPW, QS = (NQ + 3) / 4;
  constexpr size_t BB = static_cast<size_t>(B) * B;
  const int lane = threadIdx.x % 64, col = lane % 16, kq = lane / 16;
  const int64_t unit =
      static_cast<int64_t>(blockIdx.x) * 4 + __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / 64);
  const int64_t e = unit / kParts;
  if (e >= a.n) return;
  const int c0 = static_cast<int>(unit % kParts) * TPW;  // first output tile of this wave
  const double* const Vt = a.tables;           // [3][B][B]
  const double* const Fl = a.tables + 3 * BB;  // [4][B][B]
  const double* const Fn = a.tables + 7 * BB;  // [4][4][6][B][B]

  // lane offsets of the output columns: tile c0 + c, clamped to the table
  // (columns past B - 1 are computed from the last one and not stored)
  int coff[TPW];
#pragma unroll
  for (int c = 0; c < TPW; ++c) {
    const int j = 16 * (c0 + c) + col;
    coff[c] = j < B ? j : B - 1;
  }
  // X^T tile t of a Qint block: mode 16 t + col, quantities 4 s + kq (zero past the end)
  auto load_x = [&](const double* X, int t, double (&x)[QS]) __attribute__((always_inline)) {
    const int l = 16 * t + col;
#pragma unroll
    for (int s = 0; s < QS; ++s) {
      const int q = 4 * s + kq;
      x[s] = (l < B && q < NQ) ? X[q * B + l] : 0.0;
    }
  };
  // G^T: quantities 4 s + kq (rows) to quantity col (zero past the end)
  auto load_g = [&](const double* G, double sign, double (&g)[QS]) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < QS; ++s) {
      const int q = 4 * s + kq;
      g[s] = (col < NQ && q < NQ) ? sign * G[col * NQ + q] : 0.0;
    }
  };
  // the four table rows of each inner step of tile t (clamped: W is zero there)
  auto load_t = [&](const double* T, int t, double (&b)[4][TPW]) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int l = 16 * t + 4 * r + kq;
      const double* row = T + (l < B ? l : B - 1) * B;
#pragma unroll
      for (int c = 0; c < TPW; ++c) b[r][c] = row[coff[c]];
    }
  };
  v4d acc[TPW];
#pragma unroll
  for (int c = 0; c < TPW; ++c) acc[c] = v4d{0.0, 0.0, 0.0, 0.0};
  // acc += (G X)_tile t . T rows; upper: the table has zeros on and below the
  // diagonal blocks (V: degree l < degree k), so tiles left of t add nothing
  auto term = [&](const double (&x)[QS], const double (&g)[QS], const double (&b)[4][TPW], int t,
                  bool upper) __attribute__((always_inline)) {
    v4d w = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < QS; ++s) w = mfma(x[s], g[s], w);
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (16 * t + 4 * r < B) {
#pragma unroll
        for (int c = 0; c < TPW; ++c)
          if (!upper || c0 + c >= t) acc[c] = mfma(w[r], b[r][c], acc[c]);
      }
  };

  // ---- own block: E, the three volume terms and the four own-face terms
  const double* const Xo = a.Qint + e * QB;
  {
    double g[7][QS];
#pragma unroll
    for (int m = 0; m < 7; ++m) load_g(m < 3 ? a.star + (e * 3 + m) * Q2 : a.Gp + (e * 4 + (m - 3)) * Q2, m < 3 ? 1.0 : -1.0, g[m]);
    double x[QS], b[2][4][TPW];
    load_x(Xo, 0, x);
    load_t(Vt, 0, b[0]);
#pragma unroll 1
    for (int t = 0; t < NT; ++t) {
      double xn[QS];
      load_x(Xo, t + 1 < NT ? t + 1 : t, xn);
#pragma unroll
      for (int m = 0; m < 7; ++m) {
        // the next term's rows in flight during this one's products
        if (m < 6) load_t(m + 1 < 3 ? Vt + (m + 1) * BB : Fl + (m - 2) * BB, t, b[(m + 1) % 2]);
        else load_t(Vt, t + 1 < NT ? t + 1 : t, b[(m + 1) % 2]);
        term(x, g[m], b[m % 2], t, m < 3);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int c = 0; c < TPW; ++c) b[0][i][c] = b[1][i][c];
#pragma unroll
      for (int s = 0; s < QS; ++s) x[s] = xn[s];
    }
  }
  // ---- neighbours
#pragma unroll 1
  for (int f = 0; f < 4; ++f) {
    const int nb = __builtin_amdgcn_readfirstlane(a.neighbor[e * 4 + f]);
    const int code = __builtin_amdgcn_readfirstlane(a.nb_code[e * 4 + f]);
    const double* const X = a.Qint + static_cast<int64_t>(nb) * QB;
    const double* const T = Fn + (static_cast<size_t>(f) * 24 + code) * BB;
    double g[QS], x[QS], b[4][TPW];
    load_g(a.Gm + (e * 4 + f) * Q2, -1.0, g);
    load_x(X, 0, x);
    load_t(T, 0, b);
#pragma unroll 1
    for (int t = 0; t < NT; ++t) {
      double xn[QS], bn[4][TPW];
      const int tn = t + 1 < NT ? t + 1 : t;
      load_x(X, tn, xn);
      load_t(T, tn, bn);
      term(x, g, b, t, false);
#pragma unroll
      for (int s = 0; s < QS; ++s) x[s] = xn[s];
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < TPW; ++c) b[r][c] = bn[r][c];
    }
  }
  // ---- + E Qint (A operand: rows of E, B operand: rows of Qint), then Q += the update
  double ge[QS];
  {
    const double* const E = a.E + e * Q2;
#pragma unroll
    for (int s = 0; s < QS; ++s) {
      const int q = 4 * s + kq;
      ge[s] = (col < NQ && q < NQ) ? E[col * NQ + q] : 0.0;
    }
  }
#pragma unroll
  for (int c = 0; c < TPW; ++c) {
    const int j = 16 * (c0 + c) + col;
    double x[QS];
#pragma unroll
    for (int s = 0; s < QS; ++s) {
      const int q = 4 * s + kq;
      x[s] = (j < B && q < NQ) ? Xo[q * B + j] : 0.0;
    }
#pragma unroll
    for (int s = 0; s < QS; ++s) acc[c] = mfma(ge[s], x[s], acc[c]);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = kq + 4 * r;
      if (i < NQ && j < B) a.Q[e * QB + i * B + j] += acc[c][r];
    }
  }
}

template <int NQ, int N, int TPW>
hipError_t launch_tiles(const CorrectArgs& a, hipStream_t stream) {
  constexpr int NT = (n_modes(N) + 15) / 16, kParts = (NT + TPW - 1) / TPW;
  const int64_t blocks = (a.n * kParts + 3) / 4;
  if (blocks > 0x7fffffff) return hipErrorInvalidValue;
  hipLaunchKernelGGL((corrector_kernel<NQ, N, TPW>), dim3(static_cast<unsigned>(blocks)), dim3(256), 0, stream, a);
  return hipGetLastError();
}

// Output tiles per wave.  Fewer tiles per wave form W more often (4
// instructions per tile of W against 4 per output tile of it), more of them
// leave the chip idle while there are fewer waves than SIMDs (1,024).
// Measured, microseconds (13 quantities):
//   N = 6, 5,000 elements: 6 tiles 436, 3 tiles 418, 2 tiles 454;
//          1,080: 167 / 134 / 132;  320: 88 / 56 / 50
//   N = 7, 8,640 elements: 8 tiles 1,266, 4 tiles 1,107, 3 tiles 1,334
//   N = 4, 20,480 elements: 3 tiles 495, 2 tiles 646, 1 tile 692;  320: 34 / 29 / 24
// so degrees of four tiles and more take half of an element per wave (also
// the registers of two waves per SIMD), the others a whole element, and below
// one element per SIMD the tiles are spread further.
template <int NQ, int N>
hipError_t launch_one(const CorrectArgs& a, hipStream_t stream) {
  constexpr int NT = (n_modes(N) + 15) / 16;
  const bool few = a.n <= 1024;
  if constexpr (NT >= 4) {
    if (few) return launch_tiles<NQ, N, (NT + 2) / 3>(a, stream);
    return launch_tiles<NQ, N, (NT + 1) / 2>(a, stream);
  } else {
    if constexpr (NT >= 2) {
      if (few) return launch_tiles<NQ, N, 1>(a, stream);
    }
    return launch_tiles<NQ, N, NT>(a, stream);
  }
}

template <int NQ>
hipError_t launch_nq(const CorrectArgs& a, hipStream_t stream) {
  switch (a.B) {
    case n_modes(0): return launch_one<NQ, 0>(a, stream);
    case n_modes(1): return launch_one<NQ, 1>(a, stream);
    case n_modes(2): return launch_one<NQ, 2>(a, stream);
    case n_modes(3): return launch_one<NQ, 3>(a, stream);
    case n_modes(4): return launch_one<NQ, 4>(a, stream);
    case n_modes(5): return launch_one<NQ, 5>(a, stream);
    case n_modes(6): return launch_one<NQ, 6>(a, stream);
    case n_modes(7): return launch_one<NQ, 7>(a, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

bool corrector_fits(int nq, int B) {
  if (!supported_nq(nq)) return false;
  for (int N = 0; N <= kMaxDegree; ++N)
    if (n_modes(N) == B) return true;
  return false;
}

hipError_t launch_corrector(const CorrectArgs& a, hipStream_t stream) {
  if (a.n <= 0) return hipSuccess;
  if (a.nq == kNQPoro) return launch_nq<kNQPoro>(a, stream);
  if (a.nq == kNQMaxwell) return launch_nq<kNQMaxwell>(a, stream);
  return hipErrorInvalidValue;
}

}  // namespace stp
