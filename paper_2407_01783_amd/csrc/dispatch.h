// Compile-time dispatch of the launchers: value widths, (dim, right-hand
// sides), lanes per row, and the operator values of a working precision.
#pragma once

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

// Lanes per row G of the velocity-row kernels: the largest of 8, 4, 2 not
// above the request that divides W (the compiled variants).
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
  if (c->force_lanes > 0) return c->force_lanes;
  const auto it = c->lanes.find(W * 2 + (f32 ? 1 : 0));
  return it != c->lanes.end() ? it->second : heuristic_lanes(W);
}

// B^T rows have their own tuned G (key offset kBtKey)
constexpr int kBtKey = 1 << 20;
inline int lanes_bt(stokes_ctx* c, int W, bool f32) {
  if (c->force_lanes > 0) return c->force_lanes;
  const auto it = c->lanes.find(kBtKey + W * 2 + (f32 ? 1 : 0));
  return it != c->lanes.end() ? it->second : lanes_w(c, W, f32);
}

// the bfloat16-direction Chebyshev kernels too (key offset kQbKey)
constexpr int kQbKey = 2 << 20;
inline int lanes_qb(stokes_ctx* c, int W) {
  if (c->force_lanes > 0) return c->force_lanes;
  const auto it = c->lanes.find(kQbKey + W * 2 + 1);
  return it != c->lanes.end() ? it->second : lanes_w(c, W, true);
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
void finish(stokes_ctx* c, int64_t rows, int kind, int W, Scalars* sc, int cps, int nsys, int first, double* res) {
  hipLaunchKernelGGL((k_finish<NS>), dim3(1), dim3(kBlock), 0, c->stream, (const double*)partials(c), grid_for(rows),
                     kind, W, sc, cps, nsys, first, res);
}

template <class T> const DevBuf& btvals(stokes_ctx* c);
template <> inline const DevBuf& btvals<double>(stokes_ctx* c) { return c->Bt64; }
template <> inline const DevBuf& btvals<float>(stokes_ctx* c) { return c->Bt32; }
template <class T> const DevBuf& avals(stokes_ctx* c);
template <> inline const DevBuf& avals<double>(stokes_ctx* c) { return c->A64; }
template <> inline const DevBuf& avals<float>(stokes_ctx* c) { return c->A32; }

}  // namespace ops
}  // namespace stokes
