// Launchers of the later Chebyshev steps (kernels.h).
#include "dispatch.h"

namespace stokes {
namespace ops {

void cheb_step_hb(stokes_ctx* c, int W, const uint16_t* q, uint16_t* qn, const float* res_in, float* res_out,
                  float* z, const float* dinv, float c1, float c2, const QSum* fin, bool zw) {
  const Sell& S = c->sA;
  // the timed launches: the steps that carry the iterate (deferred or not), not the closing one
  const bool timed = fin == nullptr && prof_begin(c, &S, nullptr, nullptr);
  const int zm = fin ? 2 : zw ? 0 : 1;
  QSum fa{};
  if (fin) {
    if (fin->n < 0 || fin->n > kQSumMax) throw Error(STOKES_ERR_ARG, "deferred Chebyshev sum too long");
    fa = *fin;
  }
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
      with_split<GG, WW / GG>(lg, [&](auto SPc) {
        constexpr bool SP = decltype(SPc)::value;
        if constexpr (BfRaw<bf_width<WW>(), WW / GG>::kOn) {
          if (c->vel_il && c->AD16i.p) {  // the eight-slot interleaved copies
            auto kern = zm == 0   ? k_cheb_step_qb<_Float16, WW, GG, 8, true, 0, SP>
                        : zm == 1 ? k_cheb_step_qb<_Float16, WW, GG, 8, true, 1, SP>
                                  : k_cheb_step_qb<_Float16, WW, GG, 8, true, 2, SP>;
            hipLaunchKernelGGL(kern, dim3(nb), dim3(kBlock), 0, c->stream, S.nrows,
                               vel_il_idx(c, WW, il_width<_Float16>()), (const _Float16*)c->AD16i.as<_Float16>(), q, qn,
                               res_in, res_out, z, dinv, c1, c2, fa, lg);
            il = true;
            return;
          }
        }
        auto kern = zm == 0   ? k_cheb_step_qb<_Float16, WW, GG, 8, false, 0, SP>
                    : zm == 1 ? k_cheb_step_qb<_Float16, WW, GG, 8, false, 1, SP>
                              : k_cheb_step_qb<_Float16, WW, GG, 8, false, 2, SP>;
        hipLaunchKernelGGL(kern, dim3(nb), dim3(kBlock), 0, c->stream, S.nrows, S.idx(WW),
                           (const _Float16*)c->AD16.as<_Float16>(), q, qn, res_in, res_out, z, dinv, c1, c2, fa, lg);
      });
    });
  });
  check_launch();
  // algorithmic bytes: the stored operator once (half values of every padded
  // entry, the column-index structure it reads: slot words alone for the
  // affine slices of the interleaved copy); q read once (gathered and own
  // row, WP bfloat16); res_in read (W floats); then
  //   carrying z:  res_out and z written, z and dinv read, qn written;
  //   deferred:    res_out and qn written;
  //   closing:     r and the n earlier directions read, dinv read, z written
  const double vec = zm == 0   ? 4.0 * (W * 4.0 + 1.0) + 2.0 * 2.0 * wp
                     : zm == 1 ? 4.0 * (W * 2.0) + 2.0 * 2.0 * wp
                               : 4.0 * (W * 3.0 + 1.0) + 2.0 * wp * (1.0 + fa.n);
  const double bytes = op_bytes(S, 2, !il || c->vel_af) + double(S.nrows) * vec;
  count_bytes(c, bytes);
  if (timed) prof_end(c, bytes);
}

void cheb_step_h(stokes_ctx* c, int W, const float* q, float* qn, const float* res_in, float* res_out, float* z,
                 const float* dinv, float c1, float c2) {
  const Sell& S = c->sA;
  const bool timed = prof_begin(c, &S, nullptr, nullptr);
  const int G = lanes_op(c, &S, W, true);
  dispatch_w(W, [&](auto Wc) {
    constexpr int WW = decltype(Wc)::value;
    with_g<WW>(G, [&](auto Gc) {
      constexpr int GG = decltype(Gc)::value;
      auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(grid_full(S.nrows * GG)), dim3(kBlock), 0, c->stream, S.nrows, S.idx(WW),
                           (const _Float16*)c->AD16.as<_Float16>(), q, qn, res_in, res_out, z, dinv, c1, c2);
      };
      go(k_cheb_step_q<float, _Float16, WW, GG, 8>);
    });
  });
  check_launch();
  // algorithmic bytes: the stored operator once (half values of every padded
  // entry, the column-index structure); q gathered once; res_in, q, z read;
  // res_out, qn, z written (W floats each); dinv read
  const double bytes = op_bytes(S, 2) + double(S.nrows) * 4.0 * (W * 6.0 + 1.0);
  count_bytes(c, bytes);
  if (timed) prof_end(c, bytes);
}

void cheb_step_hs(stokes_ctx* c, const Sell& S, const _Float16* vals, float ms, int W, const float* d, float* dn,
                  const float* res_in, float* res_out, float* z, const float* dinv, float c1, float c2) {
  const int G = lanes_op(c, &S, W, true);
  dispatch_w(W, [&](auto Wc) {
    constexpr int WW = decltype(Wc)::value;
    if (S.es > 1 && with_e<WW, false>(S.es, [&](auto Ec) {
          constexpr int EE = decltype(Ec)::value;
          hipLaunchKernelGGL((k_cheb_step_es<float, WW, EE, _Float16>), dim3(grid_full(S.nrows * EE)), dim3(kBlock),
                             0, c->stream, S.nrows, S.idx(WW), vals, ms, d, dn, res_in, res_out, z, dinv, c1, c2);
        }))
      return;
    with_g<WW>(G, [&](auto Gc) {
      constexpr int GG = decltype(Gc)::value;
      const int lg = split_lg(c, S, GG, WW / GG);
      with_split<GG, WW / GG>(lg, [&](auto SPc) {
        hipLaunchKernelGGL((k_cheb_step<float, WW, 0, GG, _Float16, decltype(SPc)::value>),
                           dim3(grid_rows(S.nrows, GG, lg)), dim3(kBlock), 0, c->stream, S.nrows, S.idx(WW), vals, ms, d,
                           dn, res_in, res_out, z, dinv, c1, c2, (const float*)nullptr, (Scalars*)nullptr, 1, 0, 0,
                           partials(c), lg);
      });
    });
  });
  check_launch();
  // half values, d gathered; res_in, z, dinv read; res_out, dn, z written
  count_bytes(c, op_bytes(S, 2) + double(S.ncols) * W * 4.0 + double(S.nrows) * 4.0 * (W * 5.0 + 1.0));
}

template <class T>
void cheb_step(stokes_ctx* c, const Sell& S, const T* vals, int W, const T* d, T* dn, const T* res_in, T* res_out,
               T* z, const T* dinv, T c1, T c2, const T* rvec, Scalars* sc, int cps, int nsys, int rho_mode) {
  // the timed kernel is the plain Chebyshev step (no fused dot) on the velocity block
  const bool timed = rvec == nullptr && prof_begin(c, &S, (const void*)vals, (const void*)avals<T>(c).template as<T>());
  const int G = lanes_op(c, &S, W, std::is_same<T, float>::value);
  dispatch_w(W, [&](auto Wc) {
    constexpr int WW = decltype(Wc)::value;
    if (!rvec && S.es > 1 && with_e<WW, true>(S.es, [&](auto Ec) {
          constexpr int EE = decltype(Ec)::value;
          hipLaunchKernelGGL((k_cheb_step_es<T, WW, EE>), dim3(grid_full(S.nrows * EE)), dim3(kBlock), 0, c->stream,
                             S.nrows, S.idx(WW), vals, (T)1, d, dn, res_in, res_out, z, dinv, c1, c2);
        }))
      return;
    with_g<WW>(G, [&](auto Gc) {
      constexpr int GG = decltype(Gc)::value;
      int lg = split_lg(c, S, GG, WW / GG);
      const int nb = rvec ? cheb_dot_grid(c, S, GG, WW, lg) : grid_rows(S.nrows, GG, lg);
      double* sums = rvec && rho_mode == RHO_FOLDED ? rho_partials(c) : partials(c);
      with_split<GG, WW / GG>(lg, [&](auto SPc) {
        constexpr bool SP = decltype(SPc)::value;
        auto kern = rvec ? k_cheb_step<T, WW, 1, GG, T, SP> : k_cheb_step<T, WW, 0, GG, T, SP>;
        hipLaunchKernelGGL(kern, dim3(nb), dim3(kBlock), 0, c->stream, S.nrows, S.idx(WW), vals, (T)1, d, dn, res_in,
                           res_out, z, dinv, c1, c2, rvec, sc, cps, nsys, 0, sums, lg);
      });
      if (!rvec) return;
      if (rho_mode == RHO_FIRST) finish_n<WW>(c, nb, FIN_RHO, WW, sc, cps, nsys, 1, nullptr);
      if (rho_mode == RHO_AND_RR)
        hipLaunchKernelGGL((k_finish_rr_rho<WW>), dim3(1), dim3(kBlock), 0, c->stream, (const double*)rr_partials(c),
                           grid_for(S.nrows * lanes_rows(c, S.nrows, WW, std::is_same<T, float>::value)),
                           (const double*)sums, nb, sc, cps, nsys);
    });
  });
  check_launch();
  // algorithmic bytes: the stored operator once (values of every padded
  // entry, the column-index structure); d gathered once; res_in, z, dinv
  // (and rvec) read; res_out, dn, z written
  const double bytes = op_bytes(S, sizeof(T)) + double(S.ncols) * W * sizeof(T) +
                       double(S.nrows) * sizeof(T) * (W * (rvec ? 6.0 : 5.0) + 1.0);
  count_bytes(c, bytes);
  if (timed) prof_end(c, bytes);
}

template void cheb_step<double>(stokes_ctx*, const Sell&, const double*, int, const double*, double*, const double*, double*, double*, const double*, double,   double, const double*, Scalars*, int, int, int);
template void cheb_step<float>(stokes_ctx*, const Sell&, const float*, int, const float*, float*, const float*, float*, float*, const float*, float,   float, const float*, Scalars*, int, int, int);

}  // namespace ops
}  // namespace stokes
