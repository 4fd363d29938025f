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
// per element, the tables from the caches).
//
// What bounds it: the float64 matrix pipe (77 TFLOP/s, blocks of 16 modes: at
// N = 4 0.87 MFLOP per element = 11 ns, at N = 6 3.1 = 40 ns) where the chip is
// full, and before that the latency of the operands, so the 11 terms and their
// tiles are one unrolled sequence that always has the next step's loads in
// flight, also across terms and faces: a loop over the faces that waited for
// its neighbour's index, then for its blocks, and that moved prefetched
// registers, took 511 us at N = 4, 20,480 elements (now 367; 6 quantities N = 5,
// 13,720 elements 440 -> 311; N = 6, 5,000 elements 430 -> 320).
#include <utility>

#include "common.hpp"
#include "launch_slices.hpp"

namespace stp {
namespace {

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

typedef double v4d __attribute__((ext_vector_type(4)));

__device__ __forceinline__ v4d mfma(double a, double b, v4d c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Operand layout of v_mfma_f64_16x16x4f64 (checked on gfx950 with an in-bounds
// probe of one wave): lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16];
// accumulator register r of lane l is row l / 16 + 4 r, column l % 16.
//
// TPW: output tiles (16 modes) per wave; an element takes
// ceil(NT / TPW) waves.  block0: first workgroup of this launch's slice.
template <int NQ, int N, int TPW>
__global__ __launch_bounds__(256, 2) void corrector_kernel(CorrectArgs a, int64_t block0) {
  constexpr int B = n_modes(N), QB = NQ * B, Q2 = NQ * NQ, BB = B * B;
  constexpr int NT = (B + 15) / 16, kParts = (NT + TPW - 1) / TPW, QS = (NQ + 3) / 4, kTerms = 11;
  const int lane = threadIdx.x % 64, col = lane % 16, kq = lane / 16;
  const int64_t unit =
      (block0 + blockIdx.x) * 4 + __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / 64);
  const int64_t e = unit / kParts;
  if (e >= a.n) return;
  const int c0 = kParts > 1 ? static_cast<int>(unit % kParts) * TPW : 0;  // first output tile of this wave

  // the neighbours of all four faces, before anything waits
  int nb[4], code[4];
#pragma unroll
  for (int f = 0; f < 4; ++f) {
    nb[f] = __builtin_amdgcn_readfirstlane(a.neighbor[e * 4 + f]);
    code[f] = __builtin_amdgcn_readfirstlane(a.nb_code[e * 4 + f]);
  }
  // operands of term m: 0-2 volume, 3-6 own faces, 7-10 neighbours
  const double* const Xo = a.Qint + e * QB;
  auto x_of = [&](auto mc) __attribute__((always_inline)) {
    constexpr int m = decltype(mc)::value;
    if constexpr (m < 7) {
      // opaque: the tiles are read again in each term (from the caches), held
      // over the seven terms they would take 14 registers each
      const double* p = Xo;
      if constexpr (NT > 4) asm volatile("" : "+s"(p));
      return p;
    } else return a.Qint + static_cast<int64_t>(nb[m - 7]) * QB;
  };
  auto g_of = [&](auto mc) __attribute__((always_inline)) {
    constexpr int m = decltype(mc)::value;
    if constexpr (m < 3) return a.star + (e * 3 + m) * Q2;
    else if constexpr (m < 7) return a.Gp + (e * 4 + (m - 3)) * Q2;
    else return a.Gm + (e * 4 + (m - 7)) * Q2;
  };
  // tables: V [3][B][B], Fl [4][B][B], Fn [4][4][6][B][B]
  auto t_of = [&](auto mc) __attribute__((always_inline)) {
    constexpr int m = decltype(mc)::value;
    if constexpr (m < 7) return a.tables + m * BB;
    else return a.tables + 7 * BB + ((m - 7) * 24 + code[m - 7]) * BB;
  };

  // Lane offsets in bytes, clamped into the block they address: row kq (or, in
  // the last step of a ragged count, the last valid row instead), column col.
  // Everything else of an address is a constant or wave-uniform.
  constexpr int kQr = 4 * (QS - 1), kLr = 16 * (NT - 1), kTr = 4 * ((B - 1) / 4);  // first of the last step
  const int kql = kQr + kq < NQ ? kq : NQ - 1 - kQr, coll = kLr + col < B ? col : B - 1 - kLr;
  const int ktl = kTr + kq < B ? kq : B - 1 - kTr;
  unsigned xoff[2][2], toff[2][TPW], qoff[2][TPW], goff[2];
  goff[0] = 8 * ((col < NQ ? col : NQ - 1) * NQ + kq);
  goff[1] = goff[0] + 8 * (kql - kq);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int k = 0; k < 2; ++k) xoff[i][k] = 8 * ((i ? kql : kq) * B + (k ? coll : col));
#pragma unroll
  for (int c = 0; c < TPW; ++c) {
    const int j = 16 * (c0 + c) + col, jc = j < B ? j : B - 1;
    toff[0][c] = 8 * (kq * B + jc);
    toff[1][c] = 8 * (ktl * B + jc);
    qoff[0][c] = toff[0][c];
    qoff[1][c] = 8 * (kql * B + jc);
  }
  auto at = [](const double* p, int k, unsigned off) __attribute__((always_inline)) {
    return *reinterpret_cast<const double*>(reinterpret_cast<const char*>(p + k) + off);
  };
  // X^T tile t of a Qint block: mode 16 t + col, quantities 4 s + kq (zero past the end)
  auto load_x = [&](const double* X, auto tc, double (&x)[QS]) __attribute__((always_inline)) {
    constexpr int t = decltype(tc)::value;
#pragma unroll
    for (int s = 0; s < QS; ++s) x[s] = at(X, 4 * s * B + 16 * t, xoff[s == QS - 1][t == NT - 1]);
  };
  auto mask_x = [&](auto tc, double (&x)[QS]) __attribute__((always_inline)) {
    constexpr int t = decltype(tc)::value;
#pragma unroll
    for (int s = 0; s < QS; ++s)
      if (4 * s + 4 > NQ || 16 * t + 16 > B) x[s] = (4 * s + kq < NQ && 16 * t + col < B) ? x[s] : 0.0;
  };
  // G^T: quantities 4 s + kq (rows, zero past the end) to quantity col
  auto load_g = [&](const double* G, double (&g)[QS]) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < QS; ++s) g[s] = at(G, 4 * s, goff[s == QS - 1]);
  };
  auto mask_g = [&](bool negate, double (&g)[QS]) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < QS; ++s) {
      const double v = negate ? -g[s] : g[s];
      g[s] = 4 * s + 4 > NQ ? (4 * s + kq < NQ ? v : 0.0) : v;
    }
  };
  // the four table rows of each inner step of tile t (clamped: W is zero there)
  auto load_t = [&](const double* T, auto tc, double (&b)[4][TPW]) __attribute__((always_inline)) {
    constexpr int t = decltype(tc)::value;
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (16 * t + 4 * r < B) {
#pragma unroll
        for (int c = 0; c < TPW; ++c) b[r][c] = at(T, (16 * t + 4 * r) * B, toff[16 * t + 4 * r == kTr][c]);
      }
  };
  v4d acc[TPW];
#pragma unroll
  for (int c = 0; c < TPW; ++c) acc[c] = v4d{0.0, 0.0, 0.0, 0.0};

  // Terms and their tiles t as one straight sequence of steps, the loads of
  // the next step (also of the next term, X of the next face) in flight
  // during the products of this one.
  double x[2][QS], g[2][QS], b[2][4][TPW];
  load_g(g_of(ic<0>{}), g[0]);
  load_x(x_of(ic<0>{}), ic<0>{}, x[0]);
  load_t(t_of(ic<0>{}), ic<0>{}, b[0]);
  double xe[TPW][QS];
  static_for<0, kTerms>([&](auto mc) __attribute__((always_inline)) {
    constexpr int m = decltype(mc)::value;
    mask_g(m >= 3, g[m % 2]);
    static_for<0, NT>([&](auto tc) __attribute__((always_inline)) {
      constexpr int t = decltype(tc)::value, i = m * NT + t;
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (t == 0 && m + 1 < kTerms) load_g(g_of(ic<m + 1>{}), g[(m + 1) % 2]);
      if constexpr (t == 0 && m + 1 == kTerms) load_g(a.E + e * Q2, g[(m + 1) % 2]);
      if constexpr (t + 1 < NT) {
        load_x(x_of(mc), ic<t + 1>{}, x[(i + 1) % 2]);
        load_t(t_of(mc), ic<t + 1>{}, b[(i + 1) % 2]);
      } else if constexpr (m + 1 < kTerms) {
        load_x(x_of(ic<m + 1>{}), ic<0>{}, x[(i + 1) % 2]);
        load_t(t_of(ic<m + 1>{}), ic<0>{}, b[(i + 1) % 2]);
      } else {
        // for + E Qint: rows of Qint at the output columns
#pragma unroll
        for (int c = 0; c < TPW; ++c)
#pragma unroll
          for (int s = 0; s < QS; ++s) xe[c][s] = at(x_of(ic<0>{}), 4 * s * B, qoff[s == QS - 1][c]);
      }
      __builtin_amdgcn_sched_barrier(0);
      // acc += (G X)_tile t . T rows.  The volume tables have zeros on and
      // below the diagonal blocks (degree l < degree k): tiles left of t add nothing.
      mask_x(tc, x[i % 2]);
      v4d w = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int s = 0; s < QS; ++s) w = mfma(x[i % 2][s], g[m % 2][s], w);
      int cw = c0;  // opaque: the compiler would build a copy of the kernel per value
      if constexpr (m < 3 && kParts > 1) asm volatile("" : "+s"(cw));
#pragma unroll
      for (int c = 0; c < TPW; ++c)
        if (m >= 3 || cw + c >= t) {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (16 * t + 4 * r < B) acc[c] = mfma(w[r], b[i % 2][r][c], acc[c]);
        }
    });
  });
  // ---- + E Qint (A operand: rows of E, B operand: rows of Qint), then Q += the update
  constexpr int ge = kTerms % 2;
  double qv[TPW][4];
  double* const Qe = a.Q + e * QB;
#pragma unroll
  for (int c = 0; c < TPW; ++c)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (4 * r < NQ) qv[c][r] = at(Qe, 4 * r * B, qoff[r == QS - 1][c]);
  mask_g(false, g[ge]);
#pragma unroll
  for (int c = 0; c < TPW; ++c) {
    const int j = 16 * (c0 + c) + col;
#pragma unroll
    for (int s = 0; s < QS; ++s) acc[c] = mfma(g[ge][s], 4 * s + kq < NQ ? xe[c][s] : 0.0, acc[c]);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = kq + 4 * r;
      if (4 * r < NQ && i < NQ && j < B) Qe[i * B + j] = qv[c][r] + acc[c][r];
    }
  }
}

template <int NQ, int N, int TPW>
hipError_t launch_tiles(const CorrectArgs& a, hipStream_t stream) {
  constexpr int NT = (n_modes(N) + 15) / 16, kParts = (NT + TPW - 1) / TPW;
  const int64_t blocks = (a.n * kParts + 3) / 4;
  return for_slices(blocks, 256, hipSuccess, [&](int64_t first, unsigned count) {
    hipLaunchKernelGGL((corrector_kernel<NQ, N, TPW>), dim3(count), dim3(256), 0, stream, a, first);
    return hipGetLastError();
  });
}

// Output tiles per wave.  W is formed once per wave and term (4 instructions
// per tile against 4 per output tile of it), so a wave that takes the whole
// element does the least work; with fewer waves than SIMDs (1,024) that leaves
// the chip idle and the tiles are spread.  Measured, microseconds (13
// quantities; whole element / half / third of its tiles per wave):
//   N = 3, 40,000 elements: 404 / 647;   320: 17.4 / 16.6
//   N = 4, 20,480: 367 / 551;   1,080: 43 / 51;   320: 26 / 24
//   N = 5, 2,560: 94 / 106 / 106;   1,080: 64 / 65 / 64;   320: 38 / 30 / 29
//   N = 6, 5,000: 320 / 383 / 416;   2,560: 189 / 200 / 233;
//          1,080: 122 / 120 / 122;   320: 71 / 51 / 45
//   N = 7, 8,640: 995 / 1,057 / 1,246;   2,560: 356 / 334 / 404;
//          1,080: 229 / 203 / 213;   320: 133 / 81 / 71
template <int NQ, int N>
hipError_t launch_one(const CorrectArgs& a, hipStream_t stream) {
  constexpr int NT = (n_modes(N) + 15) / 16;
  if constexpr (NT >= 4) {
    if (a.n <= 1024) return launch_tiles<NQ, N, (NT + 2) / 3>(a, stream);
    if constexpr (NT >= 8) {
      if (a.n <= 4096) return launch_tiles<NQ, N, NT / 2>(a, stream);
    }
  } else if constexpr (NT >= 2) {
    if (a.n <= 1024) return launch_tiles<NQ, N, (NT + 1) / 2>(a, stream);
  }
  return launch_tiles<NQ, N, NT>(a, stream);
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
