// Launchers of the conjugate-gradient kernels (kernels.h).
#include "dispatch.h"

namespace stokes {
namespace ops {

template <class T>
void cg_spmv(stokes_ctx* c, int64_t nrows, const Sell* S, const T* vals, int W, const T* z, const T* extra, T* q,
             T* p, Scalars* sc, int cps, int nsys) {
  const int G = S ? lanes_op(c, S, W, std::is_same<T, float>::value) : 1;
  dispatch_w(W, [&](auto Wc) {
    constexpr int WW = decltype(Wc)::value;
    with_g<WW>(G, [&](auto Gc) {
      constexpr int GG = decltype(Gc)::value;
      const int lg = S ? split_lg_dot(nrows, GG, WW / GG) : 0;
      const int nb = lg ? grid_rows(nrows, GG, lg) : grid_for(nrows * GG);
      with_split<GG, WW / GG>(lg, [&](auto SPc) {
        hipLaunchKernelGGL((k_cg_spmv<T, WW, GG, decltype(SPc)::value>), dim3(nb), dim3(kBlock), 0, c->stream, nrows,
                           S ? S->idx(WW) : SellIdx{}, vals, z, extra, q, p, sc, cps, nsys, partials(c), lg);
      });
      finish_n<WW>(c, nb, FIN_ALPHA, WW, sc, cps, nsys, 0, nullptr);
    });
  });
  check_launch();
  // operator and z gathered (z streamed without one), q and p read and written (extra read)
  count_bytes(c, (S ? op_bytes(*S, sizeof(T)) + double(S->ncols) * W * sizeof(T) : 0) +
                     double(nrows) * W * sizeof(T) * (4 + (extra ? 1 : 0) + (S ? 0 : 1)));
}

template <class T>
void cg_update(stokes_ctx* c, int64_t nrows, int W, int prec, T* x, T* r, const T* p, const T* q, const T* dinv,
               T theta_inv, T* d0, T* z, Scalars* sc, int cps, int nsys) {
  const int G = lanes_rows(c, nrows, W, std::is_same<T, float>::value);
  dispatch_w(W, [&](auto Wc) {
    constexpr int WW = decltype(Wc)::value;
    with_g<WW>(G, [&](auto Gc) {
      constexpr int GG = decltype(Gc)::value;
      const int nb = grid_for(nrows * GG);
      if (prec == 2) {
        hipLaunchKernelGGL((k_cg_update<T, WW, 2, GG>), dim3(nb), dim3(kBlock), 0, c->stream, nrows, x, r, p, q, dinv,
                           theta_inv, d0, z, sc, cps, nsys, partials(c));
        finish<WW>(c, nrows * GG, FIN_RR, WW, sc, cps, nsys, 0, nullptr);
      } else if (prec == 0) {
        hipLaunchKernelGGL((k_cg_update<T, WW, 0, GG>), dim3(nb), dim3(kBlock), 0, c->stream, nrows, x, r, p, q, dinv,
                           theta_inv, d0, z, sc, cps, nsys, partials(c));
        finish<WW>(c, nrows * GG, FIN_RR, WW, sc, cps, nsys, 0, nullptr);
      } else {
        hipLaunchKernelGGL((k_cg_update<T, WW, 1, GG>), dim3(nb), dim3(kBlock), 0, c->stream, nrows, x, r, p, q, dinv,
                           theta_inv, d0, z, sc, cps, nsys, partials(c));
        finish<2 * WW>(c, nrows * GG, FIN_RR_RHO, WW, sc, cps, nsys, 0, nullptr);
      }
    });
  });
  check_launch();
  // x, r read and written, p, q read; dinv; d0 and z (or z) written
  count_bytes(c, double(nrows) * (W * sizeof(T) * (6 + (prec == 0 ? 2 : prec == 1 ? 1 : 0)) +
                                  (prec == 2 ? 0 : sizeof(T))));
}

template <class T>
void cheb_init(stokes_ctx* c, int64_t nrows, int W, const T* r, const T* dinv, T theta_inv, T* d0, T* z) {
  const int G = lanes_rows(c, nrows, W, std::is_same<T, float>::value);
  dispatch_w(W, [&](auto Wc) {
    constexpr int WW = decltype(Wc)::value;
    with_g<WW>(G, [&](auto Gc) {
      constexpr int GG = decltype(Gc)::value;
      hipLaunchKernelGGL((k_cheb_init<T, WW, GG>), dim3(grid_for(nrows * GG)), dim3(kBlock), 0, c->stream, nrows, r,
                         dinv, theta_inv, d0, z);
    });
  });
  check_launch();
  count_bytes(c, double(nrows) * (W * sizeof(T) * 3 + sizeof(T)));
}

template void cg_spmv<double>(stokes_ctx*, int64_t, const Sell*, const double*, int, const double*, const double*, double*, double*, Scalars*, int,  int);
template void cg_update<double>(stokes_ctx*, int64_t, int, int, double*, double*, const double*, const double*, const double*, double, double*, double*,        Scalars*, int, int);
template void cheb_init<double>(stokes_ctx*, int64_t, int, const double*, const double*, double, double*, double*);
template void cg_spmv<float>(stokes_ctx*, int64_t, const Sell*, const float*, int, const float*, const float*, float*, float*, Scalars*, int,  int);
template void cg_update<float>(stokes_ctx*, int64_t, int, int, float*, float*, const float*, const float*, const float*, float, float*, float*,        Scalars*, int, int);
template void cheb_init<float>(stokes_ctx*, int64_t, int, const float*, const float*, float, float*, float*);

}  // namespace ops
}  // namespace stokes
