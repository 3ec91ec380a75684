// Launchers of the conjugate-gradient kernels (kernels.h).
#include "dispatch.h"

namespace stokes {
namespace ops {

namespace {

// wavefronts per slice and workgroups of the product
template <class T>
void spmv_grid(stokes_ctx* c, int64_t nrows, const Sell* S, bool blocks, int W, int& G, int& lg, int& nb) {
  G = S && !blocks ? lanes_op(c, S, W, std::is_same<T, float>::value) : 1;
  if (blocks) {  // one lane per row in any case: the widths need not be those of split_lg
    lg = W <= 3 ? dot_rows(nrows, W, split_rows(nrows, W)) : 0;
  } else {
    lg = S ? split_lg_dot(c, *S, G, W / G) : 0;
  }
  nb = lg ? grid_rows(nrows, G, lg) : grid_for(nrows * G);
}

}  // namespace

template <class T>
CgPlan cg_plan(stokes_ctx* c, int64_t nrows, const Sell* S, bool blocks, const Sell& pcS, int W) {
  constexpr bool f32 = std::is_same<T, float>::value;
  CgPlan p;
  int G, lg;
  spmv_grid<T>(c, nrows, S, blocks, W, G, lg, p.nsig);
  p.nrr = grid_for(nrows * lanes_rows(c, nrows, W, f32));
  p.nrho = cheb_dot_grid(c, pcS, lanes_op(c, &pcS, W, f32), W, lg);
  p.fold = W <= kFoldWidth && int64_t(std::max(std::max(p.nsig, p.nrr), p.nrho)) * W <= kFoldMax;
  return p;
}

template <class T>
void cg_state(stokes_ctx* c, const CgPlan& pl, int W, Scalars* sc, int cps, int nsys) {
  dispatch_w(W, [&](auto Wc) {
    constexpr int WW = decltype(Wc)::value;
    if constexpr (WW <= kFoldWidth)
      hipLaunchKernelGGL((k_cg_state<WW>), dim3(1), dim3(64), 0, c->stream, sc, cg_sums(c, pl), cps, nsys);
  });
  check_launch();
}

template <class T>
void cg_spmv(stokes_ctx* c, const CgPlan& pl, int64_t nrows, const Sell* S, const T* vals, bool blocks, int W,
             const T* z, const T* extra, T* q, T* p, Scalars* sc, int cps, int nsys) {
  int G, lg, nb;
  spmv_grid<T>(c, nrows, S, blocks, W, G, lg, nb);
  dispatch_w(W, [&](auto Wc) {
    constexpr int WW = decltype(Wc)::value;
    auto launch = [&](auto kern) {
      hipLaunchKernelGGL(kern, dim3(nb), dim3(kBlock), 0, c->stream, nrows, S ? S->idx(WW) : SellIdx{}, vals, z, extra,
                         q, p, sc, cps, nsys, pl.fold ? sig_partials(c) : partials(c), lg, cg_sums(c, pl));
      if (!pl.fold) finish_n<WW>(c, nb, FIN_ALPHA, WW, sc, cps, nsys, 0, nullptr);
    };
    auto go = [&](auto Gc, auto SPc, auto BDc) {
      constexpr int GG = decltype(Gc)::value, BD = decltype(BDc)::value;
      constexpr bool SP = decltype(SPc)::value;
      if constexpr (WW <= kFoldWidth)
        if (pl.fold) return launch(k_cg_spmv<T, WW, GG, SP, BD, true>);
      launch(k_cg_spmv<T, WW, GG, SP, BD, false>);
    };
    auto go_blocks = [&](auto BDc) {
      if constexpr (WW <= 3)
        if (lg > 0) return go(IC<1>{}, std::true_type{}, BDc);
      go(IC<1>{}, std::false_type{}, BDc);
    };
    if (blocks) {
      if constexpr (WW > 1) go_blocks(IC<WW % 3 == 0 ? 3 : 2>{});  // W = dim x 1, 2, 4 or 8
      return;
    }
    with_g<WW>(G, [&](auto Gc) {
      with_split<decltype(Gc)::value, WW / decltype(Gc)::value>(lg, [&](auto SPc) { go(Gc, SPc, IC<0>{}); });
    });
  });
  check_launch();
  // operator and z gathered (z streamed without one), q and p read and written (extra read)
  const double entries = blocks ? 0.5 * c->dim * (c->dim + 1) : 1.0;
  count_bytes(c, (S ? op_bytes(*S, sizeof(T) * entries) + double(S->ncols) * W * sizeof(T) : 0) +
                     double(nrows) * W * sizeof(T) * (4 + (extra ? 1 : 0) + (S ? 0 : 1)));
}

template <class T>
void cg_update(stokes_ctx* c, const CgPlan& pl, int64_t nrows, int W, int prec, T* x, T* r, const T* p, const T* q,
               const T* dinv, T theta_inv, T* d0, T* z, Scalars* sc, int cps, int nsys) {
  const int G = lanes_rows(c, nrows, W, std::is_same<T, float>::value);
  dispatch_w(W, [&](auto Wc) {
    constexpr int WW = decltype(Wc)::value;
    with_g<WW>(G, [&](auto Gc) {
      constexpr int GG = decltype(Gc)::value;
      const int nb = grid_for(nrows * GG);
      auto go = [&](auto kern, double* sums) {
        hipLaunchKernelGGL(kern, dim3(nb), dim3(kBlock), 0, c->stream, nrows, x, r, p, q, dinv, theta_inv, d0, z, sc,
                           cps, nsys, sums, cg_sums(c, pl));
      };
      if (prec == 2) {
        go(k_cg_update<T, WW, 2, GG>, partials(c));
        finish_n<WW>(c, nb, FIN_RR, WW, sc, cps, nsys, 0, nullptr);
      } else if (prec == 0) {  // the sum of r.r is added up with that of r.z
        if constexpr (WW <= kFoldWidth)
          if (pl.fold) return go(k_cg_update<T, WW, 0, GG, true>, rr_partials(c));
        go(k_cg_update<T, WW, 0, GG>, rr_partials(c));
      } else {
        go(k_cg_update<T, WW, 1, GG>, partials(c));
        finish_n<2 * WW>(c, nb, FIN_RR_RHO, WW, sc, cps, nsys, 0, nullptr);
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

#define INST(T)                                                                                                       \
  template CgPlan cg_plan<T>(stokes_ctx*, int64_t, const Sell*, bool, const Sell&, int);                              \
  template void cg_state<T>(stokes_ctx*, const CgPlan&, int, Scalars*, int, int);                                     \
  template void cg_spmv<T>(stokes_ctx*, const CgPlan&, int64_t, const Sell*, const T*, bool, int, const T*, const T*, \
                           T*, T*, Scalars*, int, int);                                                               \
  template void cg_update<T>(stokes_ctx*, const CgPlan&, int64_t, int, int, T*, T*, const T*, const T*, const T*, T,  \
                             T*, T*, Scalars*, int, int);                                                             \
  template void cheb_init<T>(stokes_ctx*, int64_t, int, const T*, const T*, T, T*, T*);
INST(double)
INST(float)

}  // namespace ops
}  // namespace stokes
