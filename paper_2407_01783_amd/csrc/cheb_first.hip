// Launchers of the first Chebyshev step (kernels.h).
#include "dispatch.h"

namespace stokes {
namespace ops {

namespace {
template <class T, class TM>
void cheb_first_impl(stokes_ctx* c, const Sell& S, const TM* vals, T ms, const TM* scaled, int W, const T* r,
                     const T* dinv, T theta_inv, T* d1, T* res, T* z, T c1, T c2, int accumulate) {
  const int G = lanes_op(c, &S, W, std::is_same<T, float>::value);
  dispatch_w(W, [&](auto Wc) {
    constexpr int WW = decltype(Wc)::value;
    if (S.es > 1 && (!scaled || !std::is_same<T, TM>::value) && with_e<WW, std::is_same<T, TM>::value>(S.es, [&](auto Ec) {
          constexpr int EE = decltype(Ec)::value;
          auto kern = accumulate ? k_cheb_first_es<T, WW, 1, EE, 0, TM> : k_cheb_first_es<T, WW, 0, EE, 0, TM>;
          if constexpr (!std::is_same<T, TM>::value)
            if (scaled)
              kern = accumulate ? k_cheb_first_es<T, WW, 1, EE, 1, TM> : k_cheb_first_es<T, WW, 0, EE, 1, TM>;
          const TM* v = scaled ? scaled : vals;
          hipLaunchKernelGGL(kern, dim3(grid_full(S.nrows * EE)), dim3(kBlock), 0, c->stream, S.nrows, S.idx(WW), v,
                             v == scaled ? (T)1 : ms, r, dinv, theta_inv, d1, res, z, c1, c2);
        }))
      return;
    with_g<WW>(G, [&](auto Gc) {
      constexpr int GG = decltype(Gc)::value;
      const int lg = split_lg(c, S, GG, WW / GG);
      const int nb = grid_rows(S.nrows, GG, lg);
      with_split<GG, WW / GG>(lg, [&](auto SPc) {
        constexpr bool SP = decltype(SPc)::value;
        auto go = [&](auto kern, const TM* v) {
          hipLaunchKernelGGL(kern, dim3(nb), dim3(kBlock), 0, c->stream, S.nrows, S.idx(WW), v,
                             v == scaled ? (T)1 : ms, r, dinv, theta_inv, d1, res, z, c1, c2, lg);
        };
        if (scaled) {
          if (accumulate) go(k_cheb_first<T, WW, 1, GG, 1, TM, SP>, scaled);
          else go(k_cheb_first<T, WW, 0, GG, 1, TM, SP>, scaled);
        } else {
          if (accumulate) go(k_cheb_first<T, WW, 1, GG, 0, TM, SP>, vals);
          else go(k_cheb_first<T, WW, 0, GG, 0, TM, SP>, vals);
        }
      });
    });
  });
  check_launch();
  // operator, r gathered (and dinv with the unscaled one), dinv read; res, d1, z written (z read)
  count_bytes(c, op_bytes(S, sizeof(TM)) + double(S.ncols) * (W * sizeof(T) + (scaled ? 0 : sizeof(T))) +
                     double(S.nrows) * (sizeof(T) + W * sizeof(T) * (3 + (accumulate ? 1 : 0))));
}
}  // namespace

template <class T>
void cheb_first(stokes_ctx* c, const Sell& S, const T* vals, int W, const T* r, const T* dinv, T theta_inv, T* d1,
                T* res, T* z, T c1, T c2, int accumulate) {
  // the velocity operator has a column-scaled copy S D^{-1}
  const T* scaled = (&S == &c->sA && vals == avals<T>(c).template as<T>()) ? pick<T>(c->AD64, c->AD32) : nullptr;
  cheb_first_impl<T, T>(c, S, vals, (T)1, scaled, W, r, dinv, theta_inv, d1, res, z, c1, c2, accumulate);
}

void cheb_first_hs(stokes_ctx* c, const Sell& S, const _Float16* vals, float ms, const _Float16* scaled, int W,
                   const float* r, const float* dinv, float theta_inv, float* d1, float* res, float* z, float c1,
                   float c2, int accumulate) {
  cheb_first_impl<float, _Float16>(c, S, vals, ms, scaled, W, r, dinv, theta_inv, d1, res, z, c1, c2, accumulate);
}

void cheb_first_h(stokes_ctx* c, int W, const float* r, const float* dinv, float theta_inv, float* q1, float* res,
                  float* z, float c1, float c2) {
  const Sell& S = c->sA;
  const int G = lanes_op(c, &S, W, true);
  dispatch_w(W, [&](auto Wc) {
    constexpr int WW = decltype(Wc)::value;
    with_g<WW>(G, [&](auto Gc) {
      constexpr int GG = decltype(Gc)::value;
      hipLaunchKernelGGL((k_cheb_first_q<float, _Float16, WW, 0, GG, 8>), dim3(grid_full(S.nrows * GG)), dim3(kBlock), 0,
                         c->stream, S.nrows, S.idx(WW),
                         (const _Float16*)c->AD16.as<_Float16>(), r, dinv, theta_inv, q1, res, z, c1, c2);
    });
  });
  check_launch();
  // half values, r gathered, dinv read; q1, res, z written
  count_bytes(c, op_bytes(S, 2) + double(S.nrows) * 4.0 * (4.0 * W + 1.0));
}

void cheb_first_hb(stokes_ctx* c, int W, const float* r, const float* dinv, float theta_inv, uint16_t* q1,
                   float* res, float* z, float c1, float c2, bool zw) {
  const Sell& S = c->sA;
  const int G = lanes_qb(c, W);
  int wp = W;
  bool il = false;
  dispatch_w(W, [&](auto Wc) {
    constexpr int WW = decltype(Wc)::value;
    wp = bf_width<WW>();
    with_g<WW>(G, [&](auto Gc) {
      constexpr int GG = decltype(Gc)::value;
      const int lg = split_lg(c, S, GG, WW / GG);
      const int nb = grid_rows(S.nrows, GG, lg);
      il = c->vel_il && c->AD16i.p;  // the eight-slot interleaved copies
      with_split<GG, WW / GG>(lg, [&](auto SPc) {
        constexpr bool SP = decltype(SPc)::value;
        auto kern = il ? (zw ? k_cheb_first_qb<_Float16, WW, 0, GG, 8, true, SP>
                             : k_cheb_first_qb<_Float16, WW, 2, GG, 8, true, SP>)
                       : (zw ? k_cheb_first_qb<_Float16, WW, 0, GG, 8, false, SP>
                             : k_cheb_first_qb<_Float16, WW, 2, GG, 8, false, SP>);
        hipLaunchKernelGGL(kern, dim3(nb), dim3(kBlock), 0, c->stream, S.nrows,
                           il ? vel_il_idx(c, WW, il_width<_Float16>()) : S.idx(WW),
                           (const _Float16*)(il ? c->AD16i : c->AD16).template as<_Float16>(), r, dinv, theta_inv, q1, res,
                           z, c1, c2, lg);
      });
    });
  });
  check_launch();
  // half values, r gathered; res (floats) and q1 (bfloat16) written; dinv
  // read and z written unless deferred
  count_bytes(c, op_bytes(S, 2, !il || c->vel_af) +
                     double(S.nrows) * (4.0 * (2.0 * W) + 2.0 * wp + (zw ? 4.0 * (W + 1.0) : 0.0)));
}

template void cheb_first<double>(stokes_ctx*, const Sell&, const double*, int, const double*, const double*, double, double*, double*, double*, double, double, int);
template void cheb_first<float>(stokes_ctx*, const Sell&, const float*, int, const float*, const float*, float, float*, float*, float*, float, float, int);

}  // namespace ops
}  // namespace stokes
