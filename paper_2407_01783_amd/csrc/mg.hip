// Geometric multigrid V-cycle for the P1 pressure operator eps M_Q + L_Q
// (eps = 1), the operator the paper uses to precondition the Schur-complement
// approximations B M^{-1} B^T / B Lambda^{-1} B^T (Sec. 4.2).  The paper
// applies two algebraic-multigrid V-cycles (Table 1, BoomerAMG); on the
// structured Kuhn mesh a geometric hierarchy is available instead:
//
//   * level l+1 has n / 2^(l+1) cells per side; its vertices are the level-0
//     vertices whose grid indices are multiples of 2^(l+1) (jittered
//     positions kept), its simplices the Kuhn split of the coarse grid, and
//     its operator M_Q + L_Q is re-assembled on that mesh;
//   * a level-l vertex with grid index f is the midpoint of the coarse Kuhn
//     edge (f - s, f + s) with s = f mod 2 (componentwise), so P1
//     interpolation averages those two coarse values; restriction is its
//     transpose;
//   * smoothing: Chebyshev-Jacobi on the upper part of each level's spectrum,
//     the same polynomial before and after the coarse correction, so the
//     cycle is symmetric and can precondition CG (but for the flexible form
//     of FP32 cycles, mg_vcycle in ops.h);
//   * coarsest level: an exact dense inverse where that is cheaper than what
//     it replaces (build_mg), else a Chebyshev polynomial over its whole
//     spectrum.
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <memory>
#include <type_traits>

#include "kernels.h"
#include "ops.h"

namespace stokes {

namespace {

template <int V>
using IC = std::integral_constant<int, V>;

template <class F>
void dispatch_dn(int D, int NRB, F&& f) {
  auto inner = [&](auto Dc) {
    switch (NRB) {
      case 1: f(Dc, IC<1>{}); break;
      case 2: f(Dc, IC<2>{}); break;
      case 4: f(Dc, IC<4>{}); break;
      case 8: f(Dc, IC<8>{}); break;
      default: throw Error(STOKES_ERR_UNSUPPORTED, "batch");
    }
  };
  if (D == 3) inner(IC<3>{});
  else inner(IC<2>{});
}

// restriction: coarse vertex C gathers fine vertices 2C (weight 1) and
// 2C + s, 2C - s (weight 1/2) for every nonzero s in {0,1}^D
template <typename T, int D, int NRB>
__global__ __launch_bounds__(kBlock) void k_restrict(int nf, int nc, const T* __restrict__ rf, T* __restrict__ rc) {
  const int64_t ncv = (int64_t)ipow_dev(nc + 1, D);
  GRID_STRIDE_ROWS(C, ncv) {
    int cg[3] = {0, 0, 0};
    int64_t rem = C;
    for (int d = 0; d < D; ++d) {
      cg[d] = (int)(rem % (nc + 1));
      rem /= (nc + 1);
    }
    T acc[NRB];
    auto fid = [&](const int* g) {
      int64_t id = 0, st = 1;
      for (int d = 0; d < D; ++d, st *= (nf + 1)) id += g[d] * st;
      return id;
    };
    {
      int g[3];
      for (int d = 0; d < D; ++d) g[d] = 2 * cg[d];
      const int64_t f = fid(g);
#pragma unroll
      for (int r = 0; r < NRB; ++r) acc[r] = rf[f * NRB + r];
    }
    for (int s = 1; s < (1 << D); ++s) {
      for (int sg = -1; sg <= 1; sg += 2) {
        int g[3];
        bool ok = true;
        for (int d = 0; d < D; ++d) {
          g[d] = 2 * cg[d] + sg * ((s >> d) & 1);
          ok = ok && g[d] >= 0 && g[d] <= nf;
        }
        if (!ok) continue;
        const int64_t f = fid(g);
#pragma unroll
        for (int r = 0; r < NRB; ++r) acc[r] += T(0.5) * rf[f * NRB + r];
      }
    }
#pragma unroll
    for (int r = 0; r < NRB; ++r) rc[C * NRB + r] = acc[r];
  }
}

// interpolation, added to the fine vector: ef[f] += (ec[(f-s)/2] + ec[(f+s)/2]) / 2
template <typename T, int D, int NRB>
__global__ __launch_bounds__(kBlock) void k_prolong_add(int nf, int nc, const T* __restrict__ ec, T* __restrict__ ef) {
  const int64_t nfv = (int64_t)ipow_dev(nf + 1, D);
  GRID_STRIDE_ROWS(f, nfv) {
    int fg[3] = {0, 0, 0};
    int64_t rem = f;
    for (int d = 0; d < D; ++d) {
      fg[d] = (int)(rem % (nf + 1));
      rem /= (nf + 1);
    }
    int64_t a = 0, b = 0, st = 1;
    for (int d = 0; d < D; ++d, st *= (nc + 1)) {
      const int s = fg[d] & 1;
      a += ((fg[d] - s) / 2) * st;
      b += ((fg[d] + s) / 2) * st;
    }
#pragma unroll
    for (int r = 0; r < NRB; ++r) ef[f * NRB + r] += T(0.5) * (ec[a * NRB + r] + ec[b * NRB + r]);
  }
}

struct Cheb {
  double theta_inv;
  std::vector<double> c1, c2;
};

Cheb coef(const Bounds& b, int degree) {
  Cheb k;
  const double theta = 0.5 * (b.hi + b.lo), delta = 0.5 * (b.hi - b.lo);
  k.theta_inv = 1.0 / theta;
  const double sigma1 = theta / delta;
  double rho = 1.0 / sigma1;
  for (int j = 1; j < degree; ++j) {
    const double rn = 1.0 / (2.0 * sigma1 - rho);
    k.c1.push_back(rn * rho);
    k.c2.push_back(2.0 * rn / delta);
    rho = rn;
  }
  return k;
}

template <class T>
T* wsp(stokes_ctx* c, const std::string& name, int64_t n) {
  return static_cast<T*>(c->workspace(name + (std::is_same<T, float>::value ? "_f" : "_d"), n * sizeof(T)));
}


// y[row][w] (+)= sum_k vals[k] x[cols[k]][w] over CSR rows (grid transfers
// of the velocity multigrid, W interleaved components per node), E lanes per
// row: they read consecutive entries and add their sums by lane exchanges.
// Restriction rows have some 30-100 entries and there are few of them (16
// lanes: 29,791 rows 43 -> 8.7 us, 343 rows 30 -> 5.8 us, FP32), prolongation
// rows up to ten (2 lanes: 250,047 rows 7.8 -> 7.0 us).
template <typename T, int W, int ACC, int E>
__global__ __launch_bounds__(kBlock) void k_csr_w(int64_t nrows, const int32_t* __restrict__ rp,
                                                  const int32_t* __restrict__ cols, const T* __restrict__ vals,
                                                  const T* __restrict__ x, T* __restrict__ y) {
  GRID_STRIDE_ROWS_G(row, sub, nrows, E) {
    T acc[W];
#pragma unroll
    for (int w = 0; w < W; ++w) acc[w] = 0;
    const int32_t end = rp[row + 1];
    for (int32_t k = rp[row] + sub; k < end; k += E) {
      const T v = vals[k];
      const T* xp = x + (int64_t)cols[k] * W;
#pragma unroll
      for (int w = 0; w < W; ++w) acc[w] = fma(v, xp[w], acc[w]);
    }
    if constexpr (E > 1) {
#pragma unroll
      for (int o = E / 2; o >= 1; o /= 2)
#pragma unroll
        for (int w = 0; w < W; ++w) acc[w] += __shfl_xor(acc[w], o);
    }
#pragma unroll
    for (int w = 0; w < W; ++w)
      if (w % E == sub) y[row * W + w] = ACC ? y[row * W + w] + acc[w] : acc[w];
  }
}

template <class F>
void dispatch_w_mg(int W, F&& f) {
  switch (W) {
    case 2: f(IC<2>{}); break;
    case 3: f(IC<3>{}); break;
    case 4: f(IC<4>{}); break;
    case 6: f(IC<6>{}); break;
    case 8: f(IC<8>{}); break;
    case 12: f(IC<12>{}); break;
    case 16: f(IC<16>{}); break;
    case 24: f(IC<24>{}); break;
    default: throw Error(STOKES_ERR_UNSUPPORTED, "velocity multigrid width");
  }
}

}  // namespace

// Rows of a level that is solved by its dense inverse where it cannot coarsen.
static int64_t dense_rows(stokes_ctx* c, int64_t nrows) { return nrows <= c->mg_dense_last ? nrows : 0; }

// Eight FP64 right-hand sides: from some 4,000 rows on the cycle below the
// dense level is the faster one.
template <class T>
static bool mg_deep(const MgHier& H, int nrb) {
  return nrb * sizeof(T) >= 64 && H.dlv + 1 < static_cast<int>(H.lv.size()) && H.dense.n > 4000;
}

// Choose the dense level of a built hierarchy: the first one within
// mg_dense_max (a P2 pressure level: mg_dense_low) rows, or the last one.
static void dense_levels(stokes_ctx* c, MgHier& H) {
  const int nlev = static_cast<int>(H.lv.size());
  H.dlv = -1;
  H.dense.reset(0);
  H.last.reset(0);
  for (int l = 0; l < nlev && H.dlv < 0; ++l) {
    const int64_t nr = H.lv[l].S->nrows;
    const bool p2 = c->mesh.order == 3 && l == 0;
    if (l == nlev - 1 ? dense_rows(c, nr) > 0 : nr <= (p2 ? c->mg_dense_low : c->mg_dense_max)) H.dlv = l;
  }
  if (H.dlv >= 0) H.dense.reset(H.lv[H.dlv].S->nrows);
  if (H.dlv >= 0 && H.dlv < nlev - 1) H.last.reset(dense_rows(c, H.lv[nlev - 1].S->nrows));
}

template <class T>
void mg_ready(stokes_ctx* c, MgHier& H, int nrb) {
  if (H.dlv < 0) return;
  const MgHier::View &V = H.lv[H.dlv], &L = H.lv.back();
  if (!mg_deep<T>(H, nrb)) {
    dense_ready<T>(c, *V.S, V.v64->as<const double>(), H.dense);
    if (dense_has<T>(H.dense)) return;
  }
  dense_ready<T>(c, *L.S, L.v64->as<const double>(), H.last);
}
template void mg_ready<double>(stokes_ctx*, MgHier&, int);
template void mg_ready<float>(stokes_ctx*, MgHier&, int);

// Entry-split lanes per level (Sell::es).  The coarse levels have a few
// thousand rows of a two-ring stencil, where one lane per row leaves the chip
// idle.  mg_es = 1 (default): 8 lanes per row on levels below 2^14 rows, one
// lane above -- a fixed rule, so that every context sums the same way and
// solves are reproducible bit for bit; -1: time the level product in the form
// the FP32 V-cycle uses (half values when present) for E = 1, 2, 4, 8, 16
// and keep the fastest; 0: one lane per row; 2, 4, 8, 16: that E everywhere.
namespace {
void tune_levels(stokes_ctx* c, MgHier& H) {
  if (c->mg_es == 0) return;
  if (c->mg_es == 1) {
    for (auto& L : H.own) L->S.es = L->S.nrows < (int64_t(1) << 14) ? 8 : 1;
    return;
  }
  if (c->mg_es > 1) {  // a fixed E on every level
    for (auto& L : H.own) L->S.es = c->mg_es;
    return;
  }
  hipEvent_t e0, e1;
  HIP_CHECK(hipEventCreate(&e0));
  HIP_CHECK(hipEventCreate(&e1));
  for (auto& L : H.own) {
    Sell& S = L->S;
    if (S.nrows == 0) continue;
    DevBuf x, y;
    x.alloc(S.nrows * sizeof(float));
    y.alloc(S.nrows * sizeof(float));
    HIP_CHECK(hipMemsetAsync(x.p, 0, S.nrows * sizeof(float), c->stream));
    const bool half = c->pmg_half && L->v16.p;
    auto run = [&]() {
      if (half)
        ops::spmv_hs(c, S, L->v16.as<_Float16>(), L->s16, 1, x.as<float>(), y.as<float>(), 1.0f, nullptr, 0.0f);
      else
        ops::spmv<float>(c, S, L->v32.as<float>(), 1, x.as<float>(), y.as<float>(), 1.0f, nullptr, 0.0f);
    };
    int best = 1;
    float best_ms = 1e30f;
    for (int e : {1, 2, 4, 8, 16}) {
      S.es = e;
      run();  // warm-up
      HIP_CHECK(hipEventRecord(e0, c->stream));
      for (int rep = 0; rep < 5; ++rep) run();
      HIP_CHECK(hipEventRecord(e1, c->stream));
      HIP_CHECK(hipEventSynchronize(e1));
      float ms = 0;
      HIP_CHECK(hipEventElapsedTime(&ms, e0, e1));
      if (const char* ev = std::getenv("STOKES_LOG"); ev && std::atoi(ev) >= 1)
        std::fprintf(stderr, "[stokes] mg level n=%d rows=%lld E=%d: %.1f us per product\n", L->n,
                     (long long)S.nrows, e, 1e3 * ms / 5);
      if (ms < best_ms) {
        best_ms = ms;
        best = e;
      }
    }
    S.es = best;
  }
  HIP_CHECK(hipEventDestroy(e0));
  HIP_CHECK(hipEventDestroy(e1));
}
}  // namespace

// Build both hierarchies (called once per context after assembly).  Level
// 0 is the pressure space: the (n+1)^dim vertices of the mesh for P2/P1, the
// (2n+1)^dim P2 nodes for P3/P2.  The P2 nodes of the mesh with n cells sit
// where the vertices of the mesh with 2n cells would, and a P1 function of
// the mesh is a P2 function with the nodal values that the Kuhn P1
// interpolation from n to 2n gives (vertex values kept, edge midpoints the
// mean of the two ends): so the P2 level is level "2n" of the same
// hierarchy, and its first coarse level is the P1 space of the mesh itself.
void build_mg(stokes_ctx* c) {
  MgHier& H = c->mgq;
  H.lv.clear();
  H.own.clear();
  const HostMesh& fm = c->mesh;
  const int D = fm.dim;
  int n = fm.order == 3 ? 2 * fm.n : fm.n;  // lattice intervals per side of the pressure nodes
  H.lv.push_back({&c->sQ, &c->XQ64, &c->XQ32, &c->dXQ64, &c->dXQ32, &c->bXQ_smooth, &c->bXQ, n});
  while (n % 2 == 0 && n > 2 && ipow(n + 1, D) > c->mg_dense_low) {
    n /= 2;
    const int stride = fm.n / n;  // mesh vertices per coarse cell side
    auto L = std::make_unique<MgLevel>();
    L->n = n;
    HostMesh m;
    build_mesh(D, n, 0, 0.0, m);
    // coordinates: the level-0 vertex at stride * (grid index)
    const int64_t nf1 = fm.n + 1;
    for (int64_t g = 0; g < m.n_p1; ++g) {
      int64_t rem = g, fid = 0, st = 1;
      for (int d = 0; d < D; ++d, st *= nf1) {
        fid += (rem % (n + 1)) * stride * st;
        rem /= (n + 1);
      }
      for (int d = 0; d < D; ++d) m.vcoords[g * D + d] = fm.vcoords[fid * D + d];
    }
    L->nrows = m.n_p1;
    assemble_p1(c, m, *L);
    H.lv.push_back({&L->S, &L->v64, &L->v32, &L->d64, &L->d32, &L->bs, &L->bf, n});
    H.own.push_back(std::move(L));
  }
  dense_levels(c, H);
  // The Galerkin hierarchy of B_I Lambda_V^-1 B_I^T + M_Q.  On the P2
  // pressure of a P3/P2 pair that operator is close to the P2 mass matrix,
  // whose low-energy modes include non-smooth ones (vertex and edge values
  // coupled through negative entries) that the P1 coarse space does not
  // hold and that the smoothing interval leaves out, so its V-cycle
  // contracts more slowly there (about 0.72 per cycle on a 3D mesh), yet it
  // stays symmetric positive definite and is the better preconditioner.
  c->mgx.lv.clear();
  c->mgx.own.clear();
  if (fm.order != 3 || c->mgx_p3) {
    assemble_galerkin(c, c->mgx);
  }
  dense_levels(c, c->mgx);
  tune_levels(c, c->mgq);
  tune_levels(c, c->mgx);
}

template <class T>
void mg_vcycle(stokes_ctx* c, const MgHier& H, int nrb, const T* r, T* e, bool flexible, int lv) {
  const int nlev = static_cast<int>(H.lv.size());
  if (lv >= nlev) throw Error(STOKES_ERR_STATE, "pressure multigrid hierarchy not built");
  const MgHier::View& V = H.lv[lv];
  const Sell& S = *V.S;
  const T* vals = ops::pick<T>(*V.v64, *V.v32);
  const T* dinv = ops::pick<T>(*V.d64, *V.d32);
  const Bounds& bs = *V.bs;
  const Bounds& bf = *V.bf;
  const int64_t nr = S.nrows, n = nr * nrb;
  const std::string tag = "mg" + std::to_string(lv);
  T* d0 = wsp<T>(c, tag + "_d0", n);
  T* d1 = wsp<T>(c, tag + "_d1", n);
  T* res = wsp<T>(c, tag + "_res", n);
  // FP32 cycles read the half-precision level values (X = s16 x stored)
  const _Float16* v16 = nullptr;
  if constexpr (std::is_same<T, float>::value)
    if (c->pmg_half && V.v16 && V.v16->p) v16 = V.v16->as<_Float16>();
  // t = r - X e
  auto residual = [&](const T* e_, const T* r_, T* t_) {
    if constexpr (std::is_same<T, float>::value) {
      if (v16) return ops::spmv_hs(c, S, v16, V.s16, nrb, e_, t_, -1.0f, r_, 1.0f);
    }
    ops::spmv<T>(c, S, vals, nrb, e_, t_, (T)-1, r_, (T)1);
  };
  // z (+)= p(D^{-1} X) D^{-1} rin ; accumulate into z when acc != 0 (degree >= 2)
  auto cheb = [&](const Bounds& b, int degree, const T* rin, T* z, int acc) {
    const Cheb k = coef(b, degree);
    if (degree == 1) {
      ops::cheb_init<T>(c, nr, nrb, rin, dinv, (T)k.theta_inv, d0, z);
      return;
    }
    if constexpr (std::is_same<T, float>::value) {
      if (v16) {
        // X D^-1 rounded entry by entry is not D^-1-symmetric (by half
        // roundings, some 1e-4): only where the caller's method bears that
        const _Float16* vd16 = flexible && V.vd16 && V.vd16->p ? V.vd16->as<_Float16>() : nullptr;
        ops::cheb_first_hs(c, S, v16, V.s16, vd16, nrb, rin, dinv, (float)k.theta_inv, d0, res, z, (float)k.c1[0],
                           (float)k.c2[0], acc);
        float* da = d0;
        float* db = d1;
        for (int j = 2; j < degree; ++j) {
          ops::cheb_step_hs(c, S, v16, V.s16, nrb, da, db, res, res, z, dinv, (float)k.c1[j - 1], (float)k.c2[j - 1]);
          std::swap(da, db);
        }
        return;
      }
    }
    ops::cheb_first<T>(c, S, vals, nrb, rin, dinv, (T)k.theta_inv, d0, res, z, (T)k.c1[0], (T)k.c2[0], acc);
    T* da = d0;
    T* db = d1;
    for (int j = 2; j < degree; ++j) {
      ops::cheb_step<T>(c, S, vals, nrb, da, db, res, res, z, dinv, (T)k.c1[j - 1], (T)k.c2[j - 1], nullptr, nullptr,
                        1, 0, 0);
      std::swap(da, db);
    }
  };
  if (lv == H.dlv && !mg_deep<T>(H, nrb) && dense_has<T>(H.dense)) {
    dense_solve<T>(c, H.dense, nrb, r, e);
    return;
  }
  if (lv == nlev - 1) {  // dense inverse, or a polynomial over the whole spectrum
    if (dense_has<T>(H.last)) {
      dense_solve<T>(c, H.last, nrb, r, e);
    } else {
      cheb(bf, c->mg_coarse_degree, r, e, 0);
    }
    return;
  }
  const int nu = V.nu > 0 ? V.nu : c->mg_smooth_degree;
  T* t = wsp<T>(c, tag + "_t", n);
  const MgHier::View& C = H.lv[lv + 1];
  const int nf = V.n;
  const int64_t ncn = C.S->nrows * nrb;
  T* rc = wsp<T>(c, "mg" + std::to_string(lv + 1) + "_rc", ncn);
  T* ec = wsp<T>(c, "mg" + std::to_string(lv + 1) + "_ec", ncn);
  cheb(bs, nu, r, e, 0);                                                // pre-smoothing from zero
  residual(e, r, t);                                                    // t = r - X e
  dispatch_dn(c->dim, nrb, [&](auto Dc, auto Nc) {
    constexpr int DD = decltype(Dc)::value, N = decltype(Nc)::value;
    hipLaunchKernelGGL((k_restrict<T, DD, N>), dim3(ops::grid_for(C.S->nrows)), dim3(kBlock), 0, c->stream, nf, C.n,
                       (const T*)t, rc);
  });
  ops::check_launch();
  ops::count_bytes(c, double(n + ncn) * sizeof(T));  // fine residual read, coarse one written
  mg_vcycle<T>(c, H, nrb, rc, ec, flexible, lv + 1);
  dispatch_dn(c->dim, nrb, [&](auto Dc, auto Nc) {
    constexpr int DD = decltype(Dc)::value, N = decltype(Nc)::value;
    hipLaunchKernelGGL((k_prolong_add<T, DD, N>), dim3(ops::grid_for(nr)), dim3(kBlock), 0, c->stream, nf, C.n,
                       (const T*)ec, e);
  });
  ops::check_launch();
  ops::count_bytes(c, double(ncn + 2 * n) * sizeof(T));  // coarse correction read, e read and written
  residual(e, r, t);                                                    // t = r - X e
  if (nu >= 2) {
    cheb(bs, nu, t, e, 1);                                              // post-smoothing, e += p(.) t
  } else {
    T* dz = wsp<T>(c, tag + "_dz", n);
    cheb(bs, nu, t, dz, 0);
    ops::axpby<T>(c, n, (T)1, dz, (T)1, e);
  }
}

template void mg_vcycle<double>(stokes_ctx*, const MgHier&, int, const double*, double*, bool, int);
template void mg_vcycle<float>(stokes_ctx*, const MgHier&, int, const float*, float*, bool, int);

// ======================================================= velocity multigrid
//
// Geometric multigrid for the scalar velocity block alpha M + mu L (the
// A~_{lambda,3} preconditioner of Sec. 3.2) on the nested Kuhn meshes n, n/2,
// ...: the counterpart of the paper's fixed number of AMG V-cycles (Sec. 3.3).
//   * level 0 is the assembled interior operator (internal row order), the
//     coarse levels rediscretise alpha M + mu L on the coarse meshes (their
//     vertices keep the fine jittered positions);
//   * interpolation is P2 interpolation of the coarse basis at the fine P2
//     nodes (exact for the nested unjittered meshes), restriction its
//     transpose, coarse Dirichlet nodes dropped;
//   * Chebyshev-Jacobi smoothing on the upper spectrum, the same polynomial
//     before and after the correction, so the cycle is symmetric positive
//     definite; a coarsest level of at most mg_dense_last rows is solved densely.

void build_vmg(stokes_ctx* c) {
  c->vmg_built = false;
  c->vmg.clear();
  c->vmg_dense.reset(0);
  const HostMesh& fm = c->mesh;
  const int D = fm.dim;
  int nf = fm.n, stride = 1;
  std::vector<int32_t> fine_nat = c->h_int2nat;
  auto rows_of = [&](int n) { return ipow(2 * int64_t(n) - 1, D); };
  while (nf % 2 == 0 && nf >= 4 && rows_of(nf) > c->mg_dense_max) {
    const int nc = nf / 2;
    stride *= 2;
    auto L = std::make_unique<VmgLevel>();
    L->n = nc;
    HostMesh m;
    build_mesh(D, nc, 0, 0.0, m);
    const int64_t nf1 = fm.n + 1;
    for (int64_t g = 0; g < m.n_p1; ++g) {
      int64_t rem = g, fid = 0, st = 1;
      for (int d = 0; d < D; ++d, st *= nf1) {
        fid += (rem % (nc + 1)) * stride * st;
        rem /= (nc + 1);
      }
      for (int d = 0; d < D; ++d) m.vcoords[g * D + d] = fm.vcoords[fid * D + d];
    }
    assemble_p2_level(c, m, *L);
    // lanes per row: coarse levels have at most an eighth of the fine rows, too
    // few to hide a row's chain of gathers behind other rows.  FP32, 3D, one
    // right-hand side, one lane (a slice not shared) / 4 / 8 per row: 29,791 rows
    // 13.2 / 8.5 / 11.3 us per product, 3,375 rows 12.2 / 6.2 / 5.5 us.  Kernels
    // of a whole cycle with one lane (slices shared where the width allows it)
    // / 4 / 8 on every coarse level, FP32: 3D 32 cells 181 / 189 / 209 us, 64 cells
    // 828 / 897 / 988, with two right-hand sides 313 / 269 / 284 and 1,417 / 1,393 /
    // 1,474; 2D 128 cells 104 / 97 / 94, 256 cells 173 / 163 / 189.
    L->S.es = L->S.nrows < (int64_t(1) << 14) ? 8 : 4;
    HostCsr P, R;
    std::vector<double> pv;
    p2_prolongation(D, nf, fine_nat, P, pv);
    std::vector<int64_t> tsrc;
    transpose_pattern(P, R, tsrc);
    std::vector<double> rv(tsrc.size());
    for (size_t k = 0; k < tsrc.size(); ++k) rv[k] = pv[tsrc[k]];
    auto up = [&](const HostCsr& h, const std::vector<double>& v, DevCsr& d, DevBuf& v64, DevBuf& v32) {
      std::vector<int32_t> rp(h.rowptr.begin(), h.rowptr.end());
      d.nrows = h.nrows;
      d.nnz = h.rowptr.back();
      upload(d.rowptr, rp);
      upload(d.cols, h.cols);
      upload(v64, v);
      std::vector<float> f(v.begin(), v.end());
      upload(v32, f);
    };
    up(P, pv, L->P, L->pv64, L->pv32);
    up(R, rv, L->R, L->rv64, L->rv32);
    // natural ids of the coarse interior nodes, the rows of the next level
    fine_nat.clear();
    for (int64_t v = 0; v < m.n_p2; ++v)
      if (!m.p2_bnd[v]) fine_nat.push_back(static_cast<int32_t>(v));
    c->vmg.push_back(std::move(L));
    nf = nc;
  }
  c->vmg_dense.reset(dense_rows(c, c->vmg.empty() ? c->sA.nrows : c->vmg.back()->nrows));
  HIP_CHECK(hipStreamSynchronize(c->stream));
  c->vmg_mu = c->prob.mu;
  c->vmg_built = true;
}

template <class T>
void vmg_ready(stokes_ctx* c) {
  const Sell& S = c->vmg.empty() ? c->sA : c->vmg.back()->S;
  const DevBuf& v = c->vmg.empty() ? c->A64 : c->vmg.back()->v64;
  dense_ready<T>(c, S, v.as<const double>(), c->vmg_dense);
}
template void vmg_ready<double>(stokes_ctx*);
template void vmg_ready<float>(stokes_ctx*);

template <class T>
void vel_vcycle(stokes_ctx* c, int W, const T* r, T* e, int lv) {
  const int nlev = static_cast<int>(c->vmg.size()) + 1;
  const bool fine = lv == 0;
  const VmgLevel* L = fine ? nullptr : c->vmg[lv - 1].get();
  const Sell& S = fine ? c->sA : L->S;
  const T* vals = fine ? ops::pick<T>(c->A64, c->A32) : ops::pick<T>(L->v64, L->v32);
  const T* dinv = fine ? ops::pick<T>(c->dA64, c->dA32) : ops::pick<T>(L->d64, L->d32);
  const Bounds bf = fine ? c->bA : L->bf;
  const Bounds bs = fine ? Bounds{c->bA.hi / c->mg_smooth_ratio, c->bA.hi} : L->bs;
  const int64_t nr = S.nrows, n = nr * W;
  const std::string tag = "vmg" + std::to_string(lv);
  T* d0 = wsp<T>(c, tag + "_d0", n);
  T* d1 = wsp<T>(c, tag + "_d1", n);
  T* res = wsp<T>(c, tag + "_res", n);
  auto cheb = [&](const Bounds& b, int degree, const T* rin, T* z, int acc) {
    const Cheb k = coef(b, degree);
    ops::cheb_first<T>(c, S, vals, W, rin, dinv, (T)k.theta_inv, d0, res, z, (T)k.c1[0], (T)k.c2[0], acc);
    T* da = d0;
    T* db = d1;
    for (int j = 2; j < degree; ++j) {
      ops::cheb_step<T>(c, S, vals, W, da, db, res, res, z, dinv, (T)k.c1[j - 1], (T)k.c2[j - 1], nullptr, nullptr, 1,
                        0, 0);
      std::swap(da, db);
    }
  };
  if (lv == nlev - 1) {  // coarsest
    if (dense_has<T>(c->vmg_dense)) {
      dense_solve<T>(c, c->vmg_dense, W, r, e);
    } else {
      cheb(bf, c->mg_coarse_degree, r, e, 0);
    }
    return;
  }
  const VmgLevel& C = *c->vmg[lv];
  const int nu = std::max(2, c->vmg_smooth_degree);
  T* t = wsp<T>(c, tag + "_t", n);
  const int64_t ncn = C.nrows * W;
  T* rc = wsp<T>(c, "vmg" + std::to_string(lv + 1) + "_rc", ncn);
  T* ec = wsp<T>(c, "vmg" + std::to_string(lv + 1) + "_ec", ncn);
  cheb(bs, nu, r, e, 0);                                 // pre-smoothing from zero
  ops::spmv<T>(c, S, vals, W, e, t, (T)-1, r, (T)1);     // t = r - A e
  dispatch_w_mg(W, [&](auto Wc) {
    constexpr int WW = decltype(Wc)::value;
    hipLaunchKernelGGL((k_csr_w<T, WW, 0, 16>), dim3(ops::grid_full(C.nrows * 16)), dim3(kBlock), 0, c->stream, C.nrows,
                       C.R.rowptr.as<int32_t>(), C.R.cols.as<int32_t>(), ops::pick<T>(C.rv64, C.rv32), (const T*)t, rc);
  });
  ops::check_launch();
  // CSR restriction: row pointers, columns and values, fine residual gathered, coarse written
  ops::count_bytes(c, double(C.nrows + 1) * 4.0 + double(C.R.nnz) * (4.0 + sizeof(T)) + double(n + ncn) * sizeof(T));
  vel_vcycle<T>(c, W, rc, ec, lv + 1);
  dispatch_w_mg(W, [&](auto Wc) {
    constexpr int WW = decltype(Wc)::value;
    hipLaunchKernelGGL((k_csr_w<T, WW, 1, 2>), dim3(ops::grid_full(nr * 2)), dim3(kBlock), 0, c->stream, nr,
                       C.P.rowptr.as<int32_t>(), C.P.cols.as<int32_t>(), ops::pick<T>(C.pv64, C.pv32), (const T*)ec, e);
  });
  ops::check_launch();
  ops::count_bytes(c, double(nr + 1) * 4.0 + double(C.P.nnz) * (4.0 + sizeof(T)) + double(ncn + 2 * n) * sizeof(T));
  ops::spmv<T>(c, S, vals, W, e, t, (T)-1, r, (T)1);     // t = r - A e
  cheb(bs, nu, t, e, 1);                                 // post-smoothing, e += p(.) t
}

template void vel_vcycle<double>(stokes_ctx*, int, const double*, double*, int);
template void vel_vcycle<float>(stokes_ctx*, int, const float*, float*, int);

}  // namespace stokes
