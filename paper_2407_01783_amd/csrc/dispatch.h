// Compile-time dispatch of the launchers: value widths, (dim, right-hand
// sides), lanes per row, and the operator values of a working precision.
#pragma once

#include <algorithm>
#include <string>
#include <type_traits>

#include "kernels.h"
#include "ops.h"

namespace stokes {
namespace ops {

template <int V>
using IC = std::integral_constant<int, V>;

// W in {1,2,3,4,6,8,12,16,24}
template <class F>
void dispatch_w(int W, F&& f) {
  switch (W) {
    case 1: f(IC<1>{}); break;
    case 2: f(IC<2>{}); break;
    case 3: f(IC<3>{}); break;
    case 4: f(IC<4>{}); break;
    case 6: f(IC<6>{}); break;
    case 8: f(IC<8>{}); break;
    case 12: f(IC<12>{}); break;
    case 16: f(IC<16>{}); break;
    case 24: f(IC<24>{}); break;
    default: throw Error(STOKES_ERR_UNSUPPORTED, "unsupported vector width " + std::to_string(W));
  }
}

// dim in {2,3}, nrb in {1,2,4,8}
template <class F>
void dispatch_dn(int D, int NRB, F&& f) {
  auto inner = [&](auto Dc) {
    switch (NRB) {
      case 1: f(Dc, IC<1>{}); break;
      case 2: f(Dc, IC<2>{}); break;
      case 4: f(Dc, IC<4>{}); break;
      case 8: f(Dc, IC<8>{}); break;
      default: throw Error(STOKES_ERR_UNSUPPORTED, "unsupported batch " + std::to_string(NRB));
    }
  };
  if (D == 3) inner(IC<3>{});
  else if (D == 2) inner(IC<2>{});
  else throw Error(STOKES_ERR_UNSUPPORTED, "dim");
}

inline double* partials(stokes_ctx* c) { return c->red.partials.as<double>(); }
// the sums of a CG iteration that outlive the kernel after theirs
inline double* rr_partials(stokes_ctx* c) { return partials(c) + size_t(kMaxBlocks) * 2 * kMaxSys; }
inline double* sig_partials(stokes_ctx* c) { return rr_partials(c) + size_t(kMaxBlocks) * kMaxSys; }
inline double* rho_partials(stokes_ctx* c) { return sig_partials(c) + size_t(kMaxBlocks) * kFoldWidth; }
inline CgSums cg_sums(stokes_ctx* c, const CgPlan& pl) {
  return {rho_partials(c), rr_partials(c), sig_partials(c), pl.nrho, pl.nrr, pl.nsig};
}

// Workgroups that cover `rows` rows in one pass of the XCD partition, G lanes
// per row or 2^lg wavefronts per slice.
inline int grid_rows(int64_t rows, int G, int lg) {
  const int64_t xn = ((rows + 7) / 8 + 63) / 64 * 64, per = (kBlock / G) >> lg;
  return static_cast<int>(8 * std::max<int64_t>(1, (xn + per - 1) / per));
}

// log2 of the wavefronts that share a slice in a product over `rows` rows with
// G lanes per row and wg values per lane (rows_split in kernels.h).  Only the
// widths 1 and 3: the others can be run by 2, 4 or 8 lanes per row, a choice
// that is timed per context and must not change the sums.  The lines lie where
// the card stops being short of wavefronts (2^14 fill it, at 64 rows each), by
// the time of one product at lg = 0 / 1 / 2, in us:
//   width 1, rows of 24 slots or more (two-ring levels, P2 pressure levels):
//             two-ring P1 in 3D (65), FP64 product 36 k 8.5 / 8.0 / 6.8; 69 k
//             14.0 / 12.2 / 10.4; 91 k 15.4 / 13.8 / 12.9; 118 k 17.1 / 16.8 /
//             16.1; 185 k 23.9 / 22.8 / 23.3; FP32 118 k 8.0 / 8.3 / 8.3;
//             P2 level in 3D (200), half, 118 k: 51 / 49 / 45
//   width 1, short rows, 3D (M_Q, L_Q and their levels: 15): FP32 first and
//             later step 36 k 5.6 / 5.4 / 4.8; 55 k 4.8 / 4.4 / 4.4, 4.4 / 4.2 /
//             4.3; 74 k 5.1 / 4.8 / 5.8, 4.6 / 4.5 / 4.6; 97 k 5.1 / 4.9 / 6.2,
//             4.5 / 4.5 / 4.9; 125 k 5.0 / 5.0 / 6.4, 4.6 / 4.8 / 5.6; FP64 later
//             step 55 k 4.9 / 4.9 / 4.8; 74 k 5.7 / 6.4 / 6.5; 97 k 5.5 / 5.9 /
//             6.8; 125 k 6.4 / 6.6 / 7.7
//   width 1, short rows, 2D: L_Q (7), FP64 later step 33 k 3.9 / 4.2 / 4.4,
//             49 k 3.9 / 4.2 / 4.4; first step 26 k 5.1 / 4.3 / 4.5; two-ring
//             (19), FP64 first step 26 k 6.2 / 5.4 / 5.0; 40 k 6.2 / 6.1 / 5.8;
//             49 k 5.5 / 5.5 / 5.4, later 4.6 / 4.9 / 5.0; 103 k 8.8 / 9.6 / 11.0
//   width 3   68 k rows FP32 step best at 2; 104 k: bfloat16 step
//             12.1 / 8.5 / 8.9, first step 11.7 / 8.4 / 8.3, K_gamma product
//             11.6 / 9.1 / 9.0, B^T 7.8 / 6.8 / 6.4; 251 k: 14.2 / 12.7 /
//             16.6, 13.6 / 12.9 / 14.6, 15.1 / 13.8 / 14.4, 10.1 / 10.4 /
//             10.2; 493 k: 22.1 / 20.2 / 26.1, 20.5 / 20.8 / 23.4, 23.0 /
//             22.3 / 23.7, 15.3 / 14.7 / 16.5; 2.05 M: 56 / 58 / 79,
//             62 / 65 / 81, 72 / 71 / 73, 47 / 46 / 57
inline int split_rows(int64_t rows, int wg) {
  if (rows < (int64_t(1) << 17) && rows * wg < (int64_t(1) << 18)) return 2;
  return wg > 1 && rows < (int64_t(1) << 19) ? 1 : 0;
}
inline int split_lg(stokes_ctx* c, const Sell& S, int G, int wg) {
  if (G != 1 || !split_width(wg)) return 0;
  const int64_t rows = S.nrows;
  if (wg > 1 || S.nnz_pad >= 24 * rows) return split_rows(rows, wg);
  if (c->dim == 2 && S.nnz_pad < 10 * rows) return rows < 7 * (int64_t(1) << 12) ? 2 : 0;
  if (rows < 3 * (int64_t(1) << 14)) return 2;
  return c->dim == 3 && rows < (int64_t(1) << 16) ? 1 : 0;
}

// Partial sums (workgroups times width) up to which the kernels that use a CG
// scalar add them up themselves (cg_plan in cg.hip): every wavefront reads all
// of them.  90,601 rows in 2D, FP32: the update with 2,816 sums to read takes
// 7.3 us, with 1,424 of them 6.2 us, with none 4.9 us, and a launch that adds
// them up 3.4 us and the gaps around it.
constexpr int64_t kFoldMax = 1536;

// The same for a product that ends in a sum over all rows (one partial per
// workgroup, kMaxBlocks of them; fewer wavefronts per slice where that keeps
// the sums within kFoldMax).
inline int dot_rows(int64_t rows, int W, int lg) {
  int lo = lg;
  while (lo > 0 && grid_rows(rows, 1, lo) * int64_t(W) > kFoldMax) --lo;
  if ((lo ? grid_rows(rows, 1, lo) : grid_for(rows)) * int64_t(W) <= kFoldMax) return lo;
  while (lg > 0 && grid_rows(rows, 1, lg) > kMaxBlocks) --lg;
  return lg;
}
inline int split_lg_dot(stokes_ctx* c, const Sell& S, int G, int wg) {
  return dot_rows(S.nrows, G * wg, split_lg(c, S, G, wg));
}

// Workgroups (and lg) of a Chebyshev step that ends in a sum.
inline int cheb_dot_grid(stokes_ctx* c, const Sell& S, int G, int W, int& lg) {
  lg = split_lg_dot(c, S, G, W / G);
  return lg ? grid_rows(S.nrows, G, lg) : grid_for(S.nrows * G);
}

// f(SP): the shared-slice variant of a kernel where lg > 0.
template <int G, int WG, class F>
void with_split(int lg, F&& f) {
  if constexpr (G == 1 && split_width(WG)) {
    if (lg > 0) return f(std::true_type{});
  }
  (void)lg;
  f(std::false_type{});
}

// Lanes per row that a request of G gives at width W: the largest of 8, 4, 2
// not above it that divides W, else 1.  The lanes_* functions below return
// such numbers, so that a launch and the sums read from its workgroups count
// the same lanes.
inline int compiled_lanes(int W, int G) {
  for (int g : {8, 4, 2})
    if (G >= g && W % g == 0) return g;
  return 1;
}

// f(lanes per row) with a number from compiled_lanes as a constant
template <int WW, class F>
void with_g(int G, F&& f) {
  if constexpr (WW % 8 == 0) {
    if (G >= 8) return f(IC<8>{});
  }
  if constexpr (WW % 4 == 0) {
    if (G >= 4) return f(IC<4>{});
  }
  if constexpr (WW % 2 == 0) {
    if (G >= 2) return f(IC<2>{});
  }
  f(IC<1>{});
}

// Entry-split lanes E of a scalar operator (Sell::es, set per multigrid
// level); compiled for the pressure widths W in {1, 2, 4, 8} and, with values
// in the working precision (PLAIN) and E = 4, 8, for the 3D velocity widths 3
// and 6.  Returns false (nothing launched) for other E or W.
template <int WW, bool PLAIN, class F>
bool with_e(int E, F&& f) {
  if constexpr (WW == 1 || WW == 2 || WW == 4 || WW == 8) {
    switch (E) {
      case 2: f(IC<2>{}); return true;
      case 4: f(IC<4>{}); return true;
      case 8: f(IC<8>{}); return true;
      case 16: f(IC<16>{}); return true;
      default: return false;
    }
  } else if constexpr (PLAIN && (WW == 3 || WW == 6)) {
    switch (E) {
      case 4: f(IC<4>{}); return true;
      case 8: f(IC<8>{}); return true;
      default: return false;
    }
  } else {
    (void)E;
    (void)f;
    return false;
  }
}

// Index of the interleaved copies of the velocity pattern (iw slots per group).
inline SellIdx vel_il_idx(stokes_ctx* c, int W, int iw) {
  SellIdx ix = c->sA.idx(W);
  ix.cdel = (iw == 8 ? c->cdel_i8 : c->cdel_i).as<const uint8_t>();
  ix.cols = (iw == 8 ? c->cols_i8 : c->cols_i).as<const int32_t>();
  if (!c->vel_af) ix.cmeta = nullptr;  // read the packed offsets of affine slots too
  return ix;
}

// Before tuning: the largest G leaving each lane at least 3 components.
inline int heuristic_lanes(int W) {
  for (int g : {8, 4, 2})
    if (W % g == 0 && W / g >= 3) return g;
  return 1;
}

inline int lanes_w(stokes_ctx* c, int W, bool f32) {
  if (c->force_lanes > 0) return compiled_lanes(W, c->force_lanes);
  const auto it = c->lanes.find(W * 2 + (f32 ? 1 : 0));
  return it != c->lanes.end() ? compiled_lanes(W, it->second) : heuristic_lanes(W);
}

// B^T rows have their own tuned G (key offset kBtKey)
constexpr int kBtKey = 1 << 20;
inline int lanes_bt(stokes_ctx* c, int W, bool f32) {
  if (c->force_lanes > 0) return compiled_lanes(W, c->force_lanes);
  const auto it = c->lanes.find(kBtKey + W * 2 + (f32 ? 1 : 0));
  return it != c->lanes.end() ? compiled_lanes(W, it->second) : lanes_w(c, W, f32);
}

// the bfloat16-direction Chebyshev kernels too (key offset kQbKey)
constexpr int kQbKey = 2 << 20;
inline int lanes_qb(stokes_ctx* c, int W) {
  if (c->force_lanes > 0) return compiled_lanes(W, c->force_lanes);
  const auto it = c->lanes.find(kQbKey + W * 2 + 1);
  return it != c->lanes.end() ? compiled_lanes(W, it->second) : lanes_w(c, W, true);
}

// velocity-row operators use the tuned G; the pressure operators one lane per row
inline int lanes_op(stokes_ctx* c, const Sell* S, int W, bool f32) {
  if (S == &c->sBt) return lanes_bt(c, W, f32);
  return S == &c->sA ? lanes_w(c, W, f32) : 1;
}

inline int lanes_rows(stokes_ctx* c, int64_t nrows, int W, bool f32) {
  return nrows == c->n_int ? lanes_w(c, W, f32) : 1;
}

template <int NS>
void finish_n(stokes_ctx* c, int nblocks, int kind, int W, Scalars* sc, int cps, int nsys, int first, double* res) {
  hipLaunchKernelGGL((k_finish<NS>), dim3(1), dim3(kBlock), 0, c->stream, (const double*)partials(c), nblocks, kind, W,
                     sc, cps, nsys, first, res);
}
template <int NS>
void finish(stokes_ctx* c, int64_t rows, int kind, int W, Scalars* sc, int cps, int nsys, int first, double* res) {
  finish_n<NS>(c, grid_for(rows), kind, W, sc, cps, nsys, first, res);
}

template <class T> const DevBuf& btvals(stokes_ctx* c);
template <> inline const DevBuf& btvals<double>(stokes_ctx* c) { return c->Bt64; }
template <> inline const DevBuf& btvals<float>(stokes_ctx* c) { return c->Bt32; }
template <class T> const DevBuf& avals(stokes_ctx* c);
template <> inline const DevBuf& avals<double>(stokes_ctx* c) { return c->A64; }
template <> inline const DevBuf& avals<float>(stokes_ctx* c) { return c->A32; }

}  // namespace ops
}  // namespace stokes
