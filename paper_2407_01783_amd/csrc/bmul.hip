// Launcher of the divergence product B u (k_B in kernels.h).
#include <algorithm>

#include "dispatch.h"

namespace stokes {
namespace ops {

namespace {

// Lanes per pressure row: the fewest of 1, 2, 4, 8 that give the chip about
// 6 * 2^14 lanes (6 wavefronts per CU).  E = 1 / 2 / 4 / 8 in us, P2/P1 in 3D,
// one right-hand side:
//   35,937 rows FP32 26 / 15 / 15 / 16, FP64 30 / 27 / 25 / 28
//   50,653 rows      27 / 16 / 18 / 18       32 / 30 / 32 / 33
//   91,125 rows      32 / 22 / 25 / 27       53 / 46 / 47 / 53
//   117,649 rows     35 / 29 / 32 / 33       57 / 57 / 59 / 65
// Wider rows of u, gathered in pieces of 24 D bytes and more, differ:
//   * eight FP64 right-hand sides take four lanes on any mesh, two on P3/P2
//     pairs (P2/P1, 274,625 rows 668 / 472 / 463 / 471; P3/P2, 50,653 rows 174 /
//     145 / 203 / 170, 117,649 rows 393 / 368 / 388 / 351);
//   * 32 bytes per component (eight FP32, four FP64) take eight in 3D below
//     5 * 2^14 rows (35,937 rows 37 / 42 / 37 / 32 and 43 / 52 / 42 / 39,
//     68,921 rows 73 / 68 / 59 / 54 and 95 / 79 / 68 / 68; against them 50,653
//     rows 40 / 44 / 47 / 42 and 48 / 54 / 55 / 53), one in 2D from 2^16 on
//     (66,049 rows 14 / 16 / 15 / 17 and 15 / 17 / 15 / 17).
int b_lanes(const Sell& S, int dim, bool p3, int nrb, size_t size) {
  const int64_t rows = S.nrows;
  int e = 1;
  while (e < 8 && rows * e < 6 * (int64_t(1) << 14)) e *= 2;
  if (nrb * size == 64) return std::max(e, p3 ? 2 : 4);
  if (nrb * size == 32 && dim == 3 && rows < 5 * (int64_t(1) << 14)) return 8;
  if (nrb * size == 32 && dim == 2 && rows >= (int64_t(1) << 16)) return 1;
  return e;
}

}  // namespace

template <class T>
void Bmul(stokes_ctx* c, int nrb, const T* u, T* p, T a, const T* pin, T b) {
  const Sell& S = c->sB;
  const T* vals = pick<T>(c->B64, c->B32);
  const int lanes = b_lanes(S, c->dim, c->mesh.order == 3, nrb, sizeof(T));
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
