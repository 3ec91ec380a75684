// A whole preconditioned CG solve of a small velocity system in one launch.
//
// A CG iteration with a degree-k Chebyshev-Jacobi preconditioner is k + 1
// products and three sums, which take 7-9 launches; on the few thousand rows
// of a small mesh each of them is 2-6 us of latency, and the host looks at
// the residual every other iteration.  One workgroup of 16 wavefronts does
// the solve instead: the two vectors that are gathered live in LDS, every
// thread owns rows (64-row slices dealt to the wavefronts in turn) whose other
// vectors only it touches, the sums cross the workgroup through LDS, and the
// matrix is kept in the LDS too or streams from the L2 (12 bytes per FP64
// entry).  What bounds it is one compute unit's LDS and L2 rate, and on the
// smallest systems the chain of barriers and dependent reads: an iteration
// with a 4-step polynomial takes 10 us on 225 rows, 17 us on 961, 35 us on
// 2,209, where the launches took 50-55 us.  The arithmetic of an iteration is
// that of k_cg_spmv, k_cg_update and k_cheb_step.
#include <algorithm>
#include <type_traits>

#include "kernels.h"
#include "ops.h"

namespace stokes {
namespace ops {

namespace {

constexpr int kSmallBlock = 1024;
constexpr int kSmallWaves = kSmallBlock / 64;

template <typename T>
struct SmallArgs {
  int64_t nrows;
  int nslices, nnz;  // nnz: entries of the operator
  const int64_t* sp;
  const int32_t* cols;
  const T* vals;   // A~ (preconditioner, and the operator unless blk)
  const T* blk;    // symmetric blocks of the strain operator (null: vals)
  const T* dinv;
  const T* b;
  T* x;
  T *r, *p, *q, *res, *z;
  Scalars* sc;
  int cps, degree, maxit;
  double rtol2;
  T thinv;
  T c1[16], c2[16];
};

// Barrier for the LDS alone.  Only LDS data crosses threads here (a row's
// global vectors are read and written by the thread that owns the row), so
// the barrier does not wait for outstanding global stores as __syncthreads
// does: with those waits an iteration took 15 us on 225 rows.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Sum over the 16 lanes of a row of the wavefront by rotations (every lane of
// the row ends with the same bits), without LDS traffic.
template <int ROR>
__device__ __forceinline__ double row_rotate(double x) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, 0x120 + ROR, 0xF, 0xF, true);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), 0x120 + ROR, 0xF, 0xF, true);
  return __builtin_bit_cast(double, (uint64_t(hi) << 32) | lo);
}
__device__ __forceinline__ double row_sum(double x) {
  x += row_rotate<8>(x);
  x += row_rotate<4>(x);
  x += row_rotate<2>(x);
  x += row_rotate<1>(x);
  return x;
}
__device__ __forceinline__ double lane_value(double x, int lane) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)u, lane);
  const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
  return __builtin_bit_cast(double, (uint64_t(hi) << 32) | lo);
}

// acc += sum_j v_j g[c_j][0..W), eight entries at a time; the last group of
// four is masked instead of cut into single entries, each a round trip to the
// matrix of its own.
template <typename T, int W>
__device__ __forceinline__ void small_row(const int32_t* __restrict__ cols, const T* __restrict__ vals, int64_t beg,
                                          int width, const T* g, T (&acc)[W]) {
  auto group = [&](auto Uc, int j) {
    constexpr int U = decltype(Uc)::value;
    int32_t c[U];
    T v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t e = beg + 64 * (U == 8 ? j + u : min(j + u, width - 1));
      c[u] = cols[e];
      v[u] = vals[e];
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (U == 8 || j + u < width) {
#pragma unroll
        for (int w = 0; w < W; ++w) acc[w] = fma(v[u], g[c[u] * W + w], acc[w]);
      }
  };
  int j = 0;
  for (; j + 8 <= width; j += 8) group(std::integral_constant<int, 8>{}, j);
  for (; j < width; j += 4) group(std::integral_constant<int, 4>{}, j);
}

// the same with the symmetric D x D blocks of the strain operator (k_spmv_blk)
template <typename T, int D, int W>
__device__ __forceinline__ void small_row_blk(const int32_t* __restrict__ cols, const T* __restrict__ vals,
                                              int64_t beg, int lane, int width, const T* g, T (&acc)[W]) {
  constexpr int DD = D * (D + 1) / 2, U = D == 2 ? 4 : 2;
  const T* __restrict__ vrow = vals + (beg - lane) * DD + lane;
  for (int j = 0; j < width; j += U) {
    int32_t c[U];
    T v[U][DD];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t k = min(j + u, width - 1);
      c[u] = cols[beg + 64 * k];
#pragma unroll
      for (int e = 0; e < DD; ++e) v[u][e] = vrow[k * 64 * DD + 64 * e];
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (j + u < width) {
#pragma unroll
        for (int r = 0; r < W / D; ++r)
#pragma unroll
          for (int a = 0; a < D; ++a)
#pragma unroll
            for (int d = 0; d < D; ++d)
              acc[r * D + a] = fma(v[u][sym_index<D>(a, d)], g[c[u] * W + r * D + d], acc[r * D + a]);
      }
  }
}

// The vectors of one row that its thread alone uses.
template <typename T, int W>
struct SmallRow {
  T x[W], r[W], p[W], q[W], res[W], z[W];
};
enum { ROW_X = 1, ROW_R = 2, ROW_P = 4, ROW_Q = 8, ROW_RES = 16, ROW_Z = 32 };

// RES: at most kSmallBlock rows, one per thread, whose vectors stay in
// registers, and a matrix that fits in the LDS beside the gathered vectors
// (packed row by row, with 16-bit columns): the iterations then touch no
// global memory at all (but for the strain operator's blocks).  Otherwise a thread has several
// rows, its vectors are in global memory and the matrix streams.
template <typename T, int D, int W, bool RES>
__global__ __launch_bounds__(kSmallBlock) void k_pcg_small(SmallArgs<T> a) {
  extern __shared__ double lds[];
  double(*red)[kSmallWaves][W] = reinterpret_cast<double(*)[kSmallWaves][W]>(lds);  // [4]
  double* tol2 = lds + 4 * kSmallWaves * W;  // [W]
  T* gA = reinterpret_cast<T*>(tol2 + W);
  T* gB = gA + a.nrows * W;
  int* sp = reinterpret_cast<int*>(gB + a.nrows * W);  // [nslices + 1] first slot of a slice
  T* mv = reinterpret_cast<T*>(reinterpret_cast<double*>(gB + a.nrows * W) + (a.nslices + 2) / 2);  // RES: values
  uint16_t* mc = reinterpret_cast<uint16_t*>(mv + a.nnz);                                          // RES: columns
  for (int i = threadIdx.x; i <= a.nslices; i += kSmallBlock) sp[i] = (int)(a.sp[i] >> 6);
  lds_barrier();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // RES: the thread's row, its nonzero entries from `first` on
  int first = 0, len = 0;
  if constexpr (RES) {
    const bool has = (int)threadIdx.x < a.nrows;
    const int64_t beg = has ? (int64_t)sp[wave] * 64 + lane : 0;
    const int width = has ? sp[wave + 1] - sp[wave] : 0;
    for (int j = 0; j < width; ++j) len += a.vals[beg + 64 * j] != T(0);
    int scan = len;
    for (int o = 1; o < 64; o *= 2) {
      const int t = __shfl_up(scan, o, 64);
      if (lane >= o) scan += t;
    }
    int* wsum = reinterpret_cast<int*>(red);
    if (lane == 63) wsum[wave] = scan;
    lds_barrier();
    for (int w = 0; w < wave; ++w) first += wsum[w];
    first += scan - len;
    for (int j = 0, e = first; j < width; ++j) {
      const T v = a.vals[beg + 64 * j];
      if (v == T(0)) continue;
      mv[e] = v;
      mc[e++] = (uint16_t)a.cols[beg + 64 * j];
    }
    lds_barrier();
  }
  // slot totals over the workgroup, the same bits in every thread; slots of
  // one system carry the system's total.  buf: one of four staging areas, so
  // that one barrier is enough.
  auto total = [&](double (&v)[W], int buf) {
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const double t = row_sum(v[w]);
      const double u = (lane_value(t, 0) + lane_value(t, 16)) + (lane_value(t, 32) + lane_value(t, 48));
      if (lane == 0) red[buf][wave][w] = u;
    }
    lds_barrier();
    static_assert(kSmallWaves == 16, "one wavefront's sum per lane of a row");
#pragma unroll
    for (int w = 0; w < W; ++w) v[w] = lane_value(row_sum(red[buf][lane & 15][w]), 0);
    if (a.cps > 1) {  // cps = D: one system per right-hand side
#pragma unroll
      for (int r = 0; r < W / D; ++r) {
        double t = 0;
#pragma unroll
        for (int d = 0; d < D; ++d) t += v[r * D + d];
#pragma unroll
        for (int d = 0; d < D; ++d) v[r * D + d] = t;
      }
    }
  };
  auto slice = [&](int s, int64_t& beg, int& width) {
    beg = (int64_t)sp[s] * 64 + lane;
    width = sp[s + 1] - sp[s];
  };
  // RES: the thread's row
  SmallRow<T, W> own;
  T di_own = 0;
  if constexpr (RES) {
    if ((int)threadIdx.x < a.nrows) di_own = a.dinv[threadIdx.x];
  }
  // f(slice, row, dinv, vectors) over the thread's rows; L, S: the vectors it
  // reads and writes
  auto rows = [&](auto L, auto S, auto&& f) {
    constexpr int ld = decltype(L)::value, st = decltype(S)::value;
    if constexpr (RES) {
      const int64_t row = (int64_t)wave * 64 + lane;
      if (row < a.nrows) f(wave, row, di_own, own);
    } else {
      for (int s = wave; s < a.nslices; s += kSmallWaves) {
        const int64_t row = (int64_t)s * 64 + lane;
        if (row >= a.nrows) continue;
        SmallRow<T, W> v;
        const T di = a.dinv[row];
#pragma unroll
        for (int w = 0; w < W; ++w) {
          const int64_t i = row * W + w;
          if (ld & ROW_X) v.x[w] = a.x[i];
          if (ld & ROW_R) v.r[w] = a.r[i];
          if (ld & ROW_P) v.p[w] = a.p[i];
          if (ld & ROW_Q) v.q[w] = a.q[i];
          if (ld & ROW_RES) v.res[w] = a.res[i];
          if (ld & ROW_Z) v.z[w] = a.z[i];
        }
        f(s, row, di, v);
#pragma unroll
        for (int w = 0; w < W; ++w) {
          const int64_t i = row * W + w;
          if (st & ROW_X) a.x[i] = v.x[w];
          if (st & ROW_R) a.r[i] = v.r[w];
          if (st & ROW_P) a.p[i] = v.p[w];
          if (st & ROW_Q) a.q[i] = v.q[w];
          if (st & ROW_RES) a.res[i] = v.res[w];
          if (st & ROW_Z) a.z[i] = v.z[w];
        }
      }
    }
  };
  // acc = the row of A~ times the gathered vector g
  auto product = [&](int s, const T* g, T (&acc)[W]) {
#pragma unroll
    for (int w = 0; w < W; ++w) acc[w] = 0;
    if constexpr (RES) {
      // four entries at a time: the loop is bound by LDS reads, and wider
      // groups mask off more of them (961 rows: 350 us a solve of 20
      // iterations with four, 400 with ten)
      for (int j = 0; j < len; j += 4) {
        int c[4];
        T v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int e = first + min(j + u, len - 1);
          c[u] = mc[e];
          v[u] = mv[e];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (j + u < len) {
#pragma unroll
            for (int w = 0; w < W; ++w) acc[w] = fma(v[u], g[c[u] * W + w], acc[w]);
          }
      }
    } else {
      int64_t beg;
      int width;
      slice(s, beg, width);
      small_row<T, W>(a.cols, a.vals, beg, width, g, acc);
    }
  };
  using std::integral_constant;
  double rho[W], part[W], pz[W];
  bool act[W];
  T alpha[W], beta[W];
  bool bad = false;
  T* zb = gA;  // holds z between iterations
  auto new_rho = [&](bool first) {
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const double rn = part[w];
      beta[w] = (!first && act[w] && rho[w] != 0) ? (T)(rn / rho[w]) : T(0);
      if (act[w] && !(rn > 0)) bad = true;
      rho[w] = rn;
    }
  };
  // z = p_k(D^-1 A) D^-1 r, rho = r . z; d0 = thinv D^-1 r was left in gA (and
  // in z) by the update of r, whose r . d0 is in pz
  auto precondition = [&](bool first) {
    if (a.degree == 1) {
      zb = gA;
#pragma unroll
      for (int w = 0; w < W; ++w) part[w] = pz[w];
      total(part, 2);
      new_rho(first);
      return;
    }
    T *src = gA, *dst = gB;
    for (int j = 1; j < a.degree; ++j) {
      const bool last = j == a.degree - 1;
      const T c1 = a.c1[j - 1], c2 = a.c2[j - 1];
#pragma unroll
      for (int w = 0; w < W; ++w) part[w] = 0;
      rows(integral_constant<int, ROW_R | ROW_RES | ROW_Z>{}, integral_constant<int, ROW_RES | ROW_Z>{},
           [&](int s, int64_t row, T di, SmallRow<T, W>& v) {
             T acc[W];
             product(s, src, acc);
#pragma unroll
             for (int w = 0; w < W; ++w) {
               const int64_t i = row * W + w;
               const T rs = (j == 1 ? v.r[w] : v.res[w]) - acc[w];
               const T dn = fma(c1, src[i], (c2 * di) * rs);
               v.res[w] = rs;
               v.z[w] += dn;
               dst[i] = last ? v.z[w] : dn;
               if (last) part[w] += (double)v.r[w] * (double)v.z[w];
             }
           });
      if (!last) lds_barrier();
      T* t = src;
      src = dst;
      dst = t;
    }
    zb = src;
    total(part, 2);
    new_rho(first);
  };
  // r = b, x = p = q = 0
#pragma unroll
  for (int w = 0; w < W; ++w) part[w] = pz[w] = 0;
  rows(integral_constant<int, 0>{}, integral_constant<int, 63>{}, [&](int, int64_t row, T di, SmallRow<T, W>& v) {
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const int64_t i = row * W + w;
      v.x[w] = v.p[w] = v.q[w] = v.res[w] = T(0);
      v.r[w] = a.b[i];
      v.z[w] = v.r[w] * (di * a.thinv);
      gA[i] = v.z[w];
      part[w] += (double)v.r[w] * (double)v.r[w];
      pz[w] += (double)v.r[w] * (double)v.z[w];
    }
  });
  total(part, 3);
#pragma unroll
  for (int w = 0; w < W; ++w) {
    if (threadIdx.x == 0) {
      tol2[w] = a.rtol2 * part[w];
      if (w % a.cps == 0) a.sc->bb[w / a.cps] = a.sc->rr[w / a.cps] = part[w];
    }
    act[w] = part[w] > 0;
    rho[w] = 0;
  }
  auto any = [&]() {
    bool x = false;
#pragma unroll
    for (int w = 0; w < W; ++w) x = x || act[w];
    return x;
  };
  int it = 0;
  while (it < a.maxit && any()) {
    precondition(it == 0);
    if (bad) break;
    ++it;
    // q = A z + beta q, p = z + beta p, sigma = p . q
#pragma unroll
    for (int w = 0; w < W; ++w) part[w] = 0;
    rows(integral_constant<int, ROW_P | ROW_Q>{}, integral_constant<int, ROW_P | ROW_Q>{},
         [&](int s, int64_t row, T, SmallRow<T, W>& v) {
           T acc[W];
           if (a.blk) {
             int64_t beg;
             int width;
             slice(s, beg, width);
#pragma unroll
             for (int w = 0; w < W; ++w) acc[w] = 0;
             small_row_blk<T, D, W>(a.cols, a.blk, beg, lane, width, zb, acc);
           } else {
             product(s, zb, acc);
           }
#pragma unroll
           for (int w = 0; w < W; ++w) {
             v.q[w] = fma(beta[w], v.q[w], acc[w]);
             v.p[w] = fma(beta[w], v.p[w], zb[row * W + w]);
             part[w] += (double)v.p[w] * (double)v.q[w];
           }
         });
    total(part, 0);
#pragma unroll
    for (int w = 0; w < W; ++w) {
      alpha[w] = 0;
      if (act[w]) {
        if (part[w] > 0) alpha[w] = (T)(rho[w] / part[w]);
        else bad = true;
      }
      if (threadIdx.x == 0 && w % a.cps == 0) a.sc->sigma[w / a.cps] = part[w];
      part[w] = 0;
      pz[w] = 0;
    }
    // x += alpha p, r -= alpha q, rr = r . r; d0
    rows(integral_constant<int, ROW_X | ROW_R | ROW_P | ROW_Q>{}, integral_constant<int, ROW_X | ROW_R | ROW_Z>{},
         [&](int, int64_t row, T di, SmallRow<T, W>& v) {
#pragma unroll
           for (int w = 0; w < W; ++w) {
             v.x[w] = fma(alpha[w], v.p[w], v.x[w]);
             const T rn = fma(-alpha[w], v.q[w], v.r[w]);
             v.r[w] = rn;
             part[w] += (double)rn * (double)rn;
             v.z[w] = a.degree > 1 ? rn * di * a.thinv : rn * di;
             gA[row * W + w] = v.z[w];
             pz[w] += (double)rn * (double)v.z[w];
           }
         });
    total(part, 1);
#pragma unroll
    for (int w = 0; w < W; ++w) {
      if (act[w] && !(part[w] > tol2[w])) act[w] = false;
      if (threadIdx.x == 0 && w % a.cps == 0) a.sc->rr[w / a.cps] = part[w];
    }
    if (bad) break;
  }
  if constexpr (RES) {
    const int64_t row = (int64_t)wave * 64 + lane;
    if (row < a.nrows)
#pragma unroll
      for (int w = 0; w < W; ++w) a.x[row * W + w] = own.x[w];
  }
  if (threadIdx.x == 0) {
    a.sc->iters = it;
    a.sc->breakdown = bad ? 1 : 0;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      if (w % a.cps) continue;
      const int s = w / a.cps;
      a.sc->rho[s] = rho[w];
      a.sc->active[s] = act[w] ? 1 : 0;
    }
  }
}

template <typename T>
size_t small_lds(const Sell& S, int W) {
  return size_t(4 * kSmallWaves + 1) * W * sizeof(double) + size_t(2) * S.nrows * W * sizeof(T) +
         size_t(S.nslices + 2) / 2 * sizeof(double);
}
// the matrix beside them
template <typename T>
bool small_resident(const Sell& S, int W, size_t lds) {
  return S.nrows <= kSmallBlock && small_lds<T>(S, W) + size_t(S.nnz) * (sizeof(T) + 2) <= lds;
}

}  // namespace

// Which systems run in one launch: those whose matrix stays in the LDS, and
// those that stream at most 1.5 MB per iteration (one compute unit draws some
// 60 bytes a cycle from the L2; a 4-step preconditioner and the operator) and
// whose gathered vectors fit.  Whole solves, FP64 / FP32, launches with their
// scalars formed where they are used and one launch: 225 rows 25 -> 11 / 25 ->
// 11 ms, 961 rows 48 -> 24 / 50 -> 21, 2,209 rows (1.2 MB) 63 -> 53 / 66 -> 39,
// FP32 3,025 rows 78 -> 53; 3D 343 rows 21 -> 15, FP32 729 rows 23 -> 17.  Past
// the line, when it was drawn: FP64 2,197 rows in 3D (2.7 MB) 25 -> 27, FP32
// 9,025 rows (3.2 MB) 22 -> 26 ms.
template <class T>
bool pcg_small_fits(stokes_ctx* c, int W, int degree) {
  const Sell& S = c->sA;
  if (!c->pcg_small || W != c->dim) return false;  // one right-hand side
  if (small_lds<T>(S, W) > c->lds_bytes) return false;
  const double step = double(S.nnz_pad) * (sizeof(T) + 4.0);
  const double op = c->strain ? double(S.nnz_pad) * (sizeof(T) * W * (W + 1) / 2 + 4.0) : step;
  if (small_resident<T>(S, W, c->lds_bytes)) return !c->strain || op <= 1.5e6;
  return (degree - 1) * step + op <= 1.5e6;
}

template <class T>
void pcg_small(stokes_ctx* c, int W, int cps, int degree, T thinv, const double* c1, const double* c2, double rtol,
               int maxit, const T* b, T* x, T* r, T* p, T* q, T* res, T* z, Scalars* sc) {
  const Sell& S = c->sA;
  SmallArgs<T> a{};
  a.nrows = S.nrows;
  a.nslices = (int)S.nslices;
  a.nnz = (int)S.nnz;
  a.sp = S.slice_ptr.as<const int64_t>();
  a.cols = S.cols.as<const int32_t>();
  a.vals = pick<T>(c->A64, c->A32);
  a.blk = c->strain ? pick<T>(c->AB64, c->AB32) : nullptr;
  a.dinv = pick<T>(c->dA64, c->dA32);
  a.b = b;
  a.x = x;
  a.r = r;
  a.p = p;
  a.q = q;
  a.res = res;
  a.z = z;
  a.sc = sc;
  a.cps = cps;
  a.degree = degree;
  a.maxit = maxit;
  a.rtol2 = rtol * rtol;
  a.thinv = thinv;
  for (int j = 0; j + 1 < degree && j < 16; ++j) {
    a.c1[j] = (T)c1[j];
    a.c2[j] = (T)c2[j];
  }
  const bool one = small_resident<T>(S, W, c->lds_bytes);
  const size_t lds = small_lds<T>(S, W) + (one ? size_t(S.nnz) * (sizeof(T) + 2) : 0);
  auto go = [&](auto kern) {
    HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)c->lds_bytes));
    hipLaunchKernelGGL(kern, dim3(1), dim3(kSmallBlock), lds, c->stream, a);
  };
  if (c->dim == 2 && W == 2) one ? go(k_pcg_small<T, 2, 2, true>) : go(k_pcg_small<T, 2, 2, false>);
  else if (c->dim == 3 && W == 3) one ? go(k_pcg_small<T, 3, 3, true>) : go(k_pcg_small<T, 3, 3, false>);
  else throw Error(STOKES_ERR_UNSUPPORTED, "single-launch CG width " + std::to_string(W));
  check_launch();
}

#define INST(T)                                                                                                  \
  template bool pcg_small_fits<T>(stokes_ctx*, int, int);                                                        \
  template void pcg_small<T>(stokes_ctx*, int, int, int, T, const double*, const double*, double, int, const T*, \
                             T*, T*, T*, T*, T*, T*, Scalars*);
INST(float)
INST(double)

}  // namespace ops
}  // namespace stokes
