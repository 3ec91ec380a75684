// Launcher of the divergence product B u (k_B in kernels.h).
#include <algorithm>

#include "dispatch.h"

namespace stokes {
namespace ops {

namespace {

// Lanes per pressure row: the fewest of 1, 2, 4, 8 that give the chip about
// 7 * 2^14 lanes (7 wavefronts per CU).  Timed on 3D meshes of 9 to 64 cells:
// at 35,937 rows E = 1 / 2 / 4 / 8 takes 17.0 / 15.1 / 14.6 / 16.2 us, at
// 68,921 rows 21.8 / 20.2 / 21.8 / 22.2 us and at 117,649 rows 23.9 / 27.6 /
// 30.9 / 32.0 us (FP32), where split rows only fragment the slot loads.
// Eight FP64 right-hand sides gather 192-byte segments and take four lanes on
// any mesh (274,625 rows: 669 us with one lane, 473 with two, 463 with four).
int b_lanes(const Sell& S, int nrb, bool f64) {
  int e = 1;
  while (e < 8 && S.nrows * e < 7 * (int64_t(1) << 14)) e *= 2;
  return f64 && nrb == 8 ? std::max(e, 4) : e;
}

}  // namespace

template <class T>
void Bmul(stokes_ctx* c, int nrb, const T* u, T* p, T a, const T* pin, T b) {
  const Sell& S = c->sB;
  const T* vals = pick<T>(c->B64, c->B32);
  const int lanes = b_lanes(S, nrb, std::is_same<T, double>::value);
  dispatch_dn(c->dim, nrb, [&](auto Dc, auto Nc) {
    constexpr int D = decltype(Dc)::value, N = decltype(Nc)::value;
    auto go = [&](auto Ec) {
      constexpr int E = decltype(Ec)::value;
      hipLaunchKernelGGL((k_B<T, D, N, E>), dim3(grid_full(S.nrows * E)), dim3(kBlock), 0, c->stream, S.nrows, S.idx(),
                         vals, u, p, a, pin, b);
    };
    switch (lanes) {
      case 8: go(IC<8>{}); break;
      case 4: go(IC<4>{}); break;
      case 2: go(IC<2>{}); break;
      default: go(IC<1>{});
    }
  });
  check_launch();
  // B (dim planes), u gathered, p written (and pin read)
  count_bytes(c, op_bytes(S, sizeof(T)) + double(S.ncols) * c->dim * nrb * sizeof(T) +
                     double(S.nrows) * nrb * sizeof(T) * (pin ? 2 : 1));
}

template void Bmul<float>(stokes_ctx*, int, const float*, float*, float, const float*, float);
template void Bmul<double>(stokes_ctx*, int, const double*, double*, double, const double*, double);

}  // namespace ops
}  // namespace stokes
