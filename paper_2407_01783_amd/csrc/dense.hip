// Dense inverse of a small sliced-ELL operator (the coarsest level of a
// multigrid hierarchy) and the product with it.
//
// The inverse is formed on the device by the block sweep operator: for every
// 64-row pivot block k of the symmetric matrix,
//     A_kk <- -A_kk^-1,   A_ik <- A_ik A_kk^-1,   A_ij <- A_ij - A_ik A_kk^-1 A_kj,
// which keeps the matrix symmetric, so only its lower block triangle is
// stored and updated; once every block is swept the matrix holds -A^-1.  Each
// step reads and writes that triangle once (N^2 / 2 values twice) for N^2 64
// flops: it is bound by memory and LDS alike at this block size.  The whole
// inverse takes about N^3 flops (2,744 rows 4 ms, 4,913 rows 10.4 ms, 8,836 rows
// 45 ms, once per hierarchy and precision in use); a host Cholesky
// factorisation of 1,331 rows took over two seconds.
#include <type_traits>

#include "kernels.h"
#include "ops.h"

namespace stokes {

namespace {

constexpr int kTile = 64;

// dense entries of the rows (pads of the sliced-ELL rows hold 0 and are skipped)
__global__ __launch_bounds__(kBlock) void k_sell_to_dense(int64_t n, const int64_t* __restrict__ sp,
                                                          const int32_t* __restrict__ cols,
                                                          const double* __restrict__ vals, int64_t N,
                                                          double* __restrict__ A) {
  GRID_STRIDE_ROWS(r, n) {
    for (int64_t k = sp[r >> 6] + (r & 63); k < sp[(r >> 6) + 1]; k += 64) {
      const double v = vals[k];
      if (v != 0.0) A[r * N + cols[k]] = v;
    }
  }
}

// unit diagonal on the padding rows n .. N-1
__global__ __launch_bounds__(kBlock) void k_pad_diag(int64_t n, int64_t N, double* __restrict__ A) {
  GRID_STRIDE_ROWS(q, N - n) A[(n + q) * N + (n + q)] = 1.0;
}

// P = A_kk^-1 by Gauss-Jordan (one workgroup; a serial chain of 64 steps).
// Four lanes hold a row, 16 values each, in registers: a step broadcasts the
// pivot row through LDS (two buffers, so one barrier per step) and takes the
// row's pivot-column value from the lane that holds it.  With the tile in LDS
// instead it took 110 us.  bad |= a pivot is not positive.
__global__ __launch_bounds__(kBlock) void k_sweep_pivot(int64_t N, int64_t k, const double* __restrict__ A,
                                                        double* __restrict__ P, int* __restrict__ bad) {
  __shared__ double prow[2][kTile];
  const int t = threadIdx.x, r = t / 4, c0 = (t % 4) * 16;
  double v[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    // the lower triangle of the tile, mirrored
    const int i = r > c0 + q ? r : c0 + q, j = r > c0 + q ? c0 + q : r;
    v[q] = A[(k * kTile + i) * N + k * kTile + j];
  }
  for (int pb = 0; pb < 4; ++pb) {
#pragma unroll
    for (int pq = 0; pq < 16; ++pq) {
      const int p = 16 * pb + pq;
      double* row = prow[p & 1];
      if (r == p) {
#pragma unroll
        for (int q = 0; q < 16; ++q) row[c0 + q] = v[q];
      }
      __syncthreads();
      const double d = row[p];
      if (t == 0 && !(d > 0)) *bad = 1;
      const double inv = 1.0 / d;
      const double f = __shfl(v[pq], (t & 63 & ~3) + pb, 64);
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const double x = row[c0 + q] * inv;
        const bool piv = pb * 16 == c0 && q == pq;
        if (r == p) v[q] = piv ? inv : x;
        else v[q] = piv ? -f * inv : v[q] - f * x;
      }
    }
  }
#pragma unroll
  for (int q = 0; q < 16; ++q) P[r * kTile + c0 + q] = v[q];
}

// acc[a][b] += sum_k L[k][4 ty + a] R[k][4 tx + b] over the staged tiles
__device__ __forceinline__ void tile_fma(const double (*L)[kTile], const double (*R)[kTile], int ty, int tx,
                                         double (&acc)[4][4]) {
#pragma unroll 4
  for (int k = 0; k < kTile; ++k) {
    double a[4], b[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) a[q] = L[k][4 * ty + q];
#pragma unroll
    for (int q = 0; q < 4; ++q) b[q] = R[k][4 * tx + q];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = fma(a[i], b[j], acc[i][j]);
  }
}

// Column panel of the sweep: T_I = A_Ik (old), Q_I = T_I P, and the panel
// itself becomes Q (A_kk becomes -P).  T and Q are stored transposed per
// 64-row tile ([I][k][row]), the order in which the update stages them.
__global__ __launch_bounds__(kBlock) void k_sweep_panel(int64_t N, int64_t k, double* __restrict__ A,
                                                        const double* __restrict__ P, double* __restrict__ T,
                                                        double* __restrict__ Q) {
  __shared__ double st[kTile][kTile], sp[kTile][kTile];
  const int64_t I = blockIdx.x;
  const int t = threadIdx.x, r = t / 4, c0 = (t % 4) * 16;
  if (I == k) {
#pragma unroll
    for (int q = 0; q < 16; ++q) A[(k * kTile + r) * N + k * kTile + c0 + q] = -P[r * kTile + c0 + q];
    return;
  }
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int c = c0 + q;
    // st[kk][row] = A_Ik[row][kk]
    if (I > k) st[c][r] = A[(I * kTile + r) * N + k * kTile + c];
    else st[r][c] = A[(k * kTile + r) * N + I * kTile + c];
    sp[r][c] = P[r * kTile + c];
  }
  __syncthreads();
  const int ty = t / 16, tx = t % 16;
  double acc[4][4] = {};
  tile_fma(st, sp, ty, tx, acc);
  __syncthreads();
  // sp[kk][row] = Q_I[row][kk]
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) sp[4 * tx + j][4 * ty + i] = acc[i][j];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int c = c0 + q;
    T[(I * kTile + r) * kTile + c] = st[r][c];
    Q[(I * kTile + r) * kTile + c] = sp[r][c];
    if (I > k) A[(I * kTile + r) * N + k * kTile + c] = sp[c][r];
    else A[(k * kTile + r) * N + I * kTile + c] = sp[r][c];
  }
}

// Trailing tiles of the lower triangle: A_IJ -= Q_I T_J^T (I, J != k)
__global__ __launch_bounds__(kBlock) void k_sweep_update(int64_t N, int64_t k, double* __restrict__ A,
                                                         const double* __restrict__ T, const double* __restrict__ Q) {
  const int64_t I = blockIdx.y, J = blockIdx.x;
  if (J > I || I == k || J == k) return;
  __shared__ double sq[kTile][kTile], st[kTile][kTile];
  const int t = threadIdx.x, r = t / 4, c0 = (t % 4) * 16;
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    sq[r][c0 + q] = Q[(I * kTile + r) * kTile + c0 + q];
    st[r][c0 + q] = T[(J * kTile + r) * kTile + c0 + q];
  }
  __syncthreads();
  const int ty = t / 16, tx = t % 16;
  double acc[4][4] = {};
  tile_fma(sq, st, ty, tx, acc);
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) A[(I * kTile + 4 * ty + i) * N + J * kTile + 4 * tx + j] -= acc[i][j];
}

// The inverse in full (rows of ld values, pads 0)
template <typename T>
__global__ __launch_bounds__(kBlock) void k_sweep_out(int64_t n, int64_t ld, int64_t N, const double* __restrict__ A,
                                                      T* __restrict__ inv) {
  const int64_t i = blockIdx.x;
  for (int64_t j = threadIdx.x; j < ld; j += blockDim.x) {
    double v = 0;
    if (j < n) v = -(i >= j ? A[i * N + j] : A[j * N + i]);
    inv[i * ld + j] = (T)v;
  }
}

// y[i][r] = sum_j Cinv[i][j] x[j][r]: RW rows per wavefront, 16 bytes of the
// matrix per lane and load.  The product streams the matrix once (non-temporal,
// or the up to 100 MB of it push the next level's rows out of the caches: its
// 36 k-row products right after took 10.3 and 11 us, now 9.3 and 9.3), but
// every wavefront reads all of x, NRB values per matrix entry, from the L2:
// with one row per wavefront that is what four and more right-hand sides wait
// for, while several rows leave a small matrix short of wavefronts (dense_rw).
// One to three right-hand sides keep one row (4,096 rows RW = 1 / 2 / 4, FP32:
// one 13.0 / 13.2 / 12.8 us, two 14.8 / 18.6 / 16.4).
// ld: row pitch, a multiple of 4.
template <typename T, int NRB, int RW>
__global__ __launch_bounds__(kBlock) void k_dense_mv(int64_t n, int64_t ld, const T* __restrict__ Ci,
                                                     const T* __restrict__ x, T* __restrict__ y) {
  constexpr int V = 16 / sizeof(T), U = NRB <= 4 ? 4 : 1;
  typedef T vec_t __attribute__((ext_vector_type(V)));
  const int lane = threadIdx.x & 63;
  const int64_t row = ((int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6)) * RW;
  if (row >= n) return;  // whole wavefronts exit together
  const T* ci[RW];  // past the last row: the last row again
#pragma unroll
  for (int q = 0; q < RW; ++q) ci[q] = Ci + (row + q < n ? row + q : n - 1) * ld;
  double acc[RW][NRB];
#pragma unroll
  for (int q = 0; q < RW; ++q)
#pragma unroll
    for (int r = 0; r < NRB; ++r) acc[q][r] = 0;
  auto chunk = [&](auto Uc, int64_t j) {
    constexpr int UU = decltype(Uc)::value;
    vec_t a[UU][RW];
#pragma unroll
    for (int u = 0; u < UU; ++u)
#pragma unroll
      for (int q = 0; q < RW; ++q)
        a[u][q] = __builtin_nontemporal_load(reinterpret_cast<const vec_t*>(ci[q] + j + u * 64 * V));
#pragma unroll
    for (int u = 0; u < UU; ++u)
#pragma unroll
      for (int v = 0; v < V; ++v)
#pragma unroll
        for (int r = 0; r < NRB; ++r) {
          const double xv = (double)x[(j + u * 64 * V + v) * NRB + r];
#pragma unroll
          for (int q = 0; q < RW; ++q) acc[q][r] += (double)a[u][q][v] * xv;
        }
  };
  int64_t j = lane * V;
  for (; j + ((U - 1) * 64 + 1) * V <= n; j += U * 64 * V) chunk(std::integral_constant<int, U>{}, j);
  for (; j + V <= n; j += 64 * V) chunk(std::integral_constant<int, 1>{}, j);
  for (int64_t k = j; k < n && k < j + V; ++k)  // the columns past the last whole 16 bytes
#pragma unroll
    for (int q = 0; q < RW; ++q)
#pragma unroll
      for (int r = 0; r < NRB; ++r) acc[q][r] += (double)ci[q][k] * (double)x[k * NRB + r];
#pragma unroll
  for (int q = 0; q < RW; ++q)
#pragma unroll
    for (int r = 0; r < NRB; ++r) {
      acc[q][r] = wave_sum(acc[q][r]);
      if (lane == 0 && row + q < n) y[(row + q) * NRB + r] = (T)acc[q][r];
    }
}

}  // namespace

namespace {

template <class T>
void form_inverse(stokes_ctx* c, const Sell& S, const double* v64, const DenseInv& D, DevBuf& out) {
  const int64_t n = S.nrows, nt = (n + kTile - 1) / kTile, N = nt * kTile;
  DevBuf A, P, T_, Q, bad;
  A.alloc(N * N * sizeof(double));
  P.alloc(kTile * kTile * sizeof(double));
  T_.alloc(N * kTile * sizeof(double));
  Q.alloc(N * kTile * sizeof(double));
  bad.alloc(sizeof(int));
  out.alloc(n * D.ld * sizeof(T));
  HIP_CHECK(hipMemsetAsync(A.p, 0, N * N * sizeof(double), c->stream));
  HIP_CHECK(hipMemsetAsync(bad.p, 0, sizeof(int), c->stream));
  hipLaunchKernelGGL(k_sell_to_dense, dim3(ops::grid_for(n)), dim3(kBlock), 0, c->stream, n,
                     S.slice_ptr.as<const int64_t>(), S.cols.as<const int32_t>(), v64, N, A.as<double>());
  if (N > n)
    hipLaunchKernelGGL(k_pad_diag, dim3(1), dim3(kBlock), 0, c->stream, n, N, A.as<double>());
  for (int64_t k = 0; k < nt; ++k) {
    hipLaunchKernelGGL(k_sweep_pivot, dim3(1), dim3(kBlock), 0, c->stream, N, k, A.as<const double>(), P.as<double>(),
                       bad.as<int>());
    hipLaunchKernelGGL(k_sweep_panel, dim3(nt), dim3(kBlock), 0, c->stream, N, k, A.as<double>(), P.as<const double>(),
                       T_.as<double>(), Q.as<double>());
    hipLaunchKernelGGL(k_sweep_update, dim3(nt, nt), dim3(kBlock), 0, c->stream, N, k, A.as<double>(),
                       T_.as<const double>(), Q.as<const double>());
  }
  hipLaunchKernelGGL(k_sweep_out<T>, dim3(n), dim3(kBlock), 0, c->stream, n, D.ld, N, A.as<const double>(),
                     out.as<T>());
  ops::check_launch();
  int hbad = 0;
  HIP_CHECK(hipMemcpyAsync(&hbad, bad.p, sizeof(int), hipMemcpyDeviceToHost, c->stream));
  HIP_CHECK(hipStreamSynchronize(c->stream));
  if (hbad) {
    out.release();
    throw Error(STOKES_ERR_BREAKDOWN, "coarsest multigrid operator is not positive definite");
  }
}

}  // namespace

template <class T>
void dense_ready(stokes_ctx* c, const Sell& S, const double* v64, DenseInv& D) {
  constexpr bool f32 = std::is_same<T, float>::value;
  bool& tried = f32 ? D.tried32 : D.tried64;
  if (D.n == 0 || tried) return;
  const size_t need = (size_t(D.n + kTile) * (D.n + kTile) + size_t(2 * kTile) * (D.n + kTile)) * sizeof(double) +
                      size_t(D.n) * D.ld * sizeof(T);
  size_t cap = size_t(c->dense_bytes);
  if (c->dense_bytes < 0) {
    size_t free_b = 0, total = 0;
    HIP_CHECK(hipMemGetInfo(&free_b, &total));
    cap = free_b / 2;
  }
  DevBuf& out = f32 ? D.i32 : D.i64;
  if (need <= cap) {
    try {
      form_inverse<T>(c, S, v64, D, out);
    } catch (const Error& e) {
      out.release();
      if (e.code != STOKES_ERR_ALLOC) throw;
    }
  }
  tried = true;
}
template void dense_ready<float>(stokes_ctx*, const Sell&, const double*, DenseInv&);
template void dense_ready<double>(stokes_ctx*, const Sell&, const double*, DenseInv&);

template <class T>
bool dense_has(const DenseInv& D) {
  return D.n > 0 && ops::pick<T>(D.i64, D.i32) != nullptr;
}
template bool dense_has<float>(const DenseInv&);
template bool dense_has<double>(const DenseInv&);

// Matrix rows per wavefront from 4 values per row on, by the time of the
// product, RW = 1 / 2 / 4 in us:
//   rows    FP32, four     FP32, eight    FP64, four     FP64, eight
//   1,000   6 / 7 / 10     8 / 10 / 15    7 / 8 / 12     12 / 15 / 19
//   1,331   7 / 7 / 11     15 / 14 / 18   10 / 10 / 12   24 / 19 / 23
//   2,744   15 / 14 / 18   35 / 27 / 30   23 / 23 / 25   64 / 54 / 41
//   4,096   27 / 19 / 27   65 / 38 / 39   48 / 34 / 39   121 / 77 / 56
//   5,832   47 / 33 / 45   140 / 73 / 87  108 / 59 / 66  269 / 155 / 131
//   8,000   123 / 57 / 67  254 / 145 / 117  197 / 107 / 93  487 / 262 / 178
// and of the velocity, 3D 3,375 rows: FP32 12 values 61 / 35 / 48, 24 values
// 162 / 89 / 72, FP64 120 / 62 / 62, 297 / 166 / 108; 2D 2,601 rows, 16 values:
// FP32 65 / 50 / 48, FP64 119 / 92 / 57.
static int dense_rw(int64_t n, int W, size_t size) {
  if (n < 1200) return 1;
  return int64_t(n * W * size) >= (W * size >= 64 ? 130000 : 200000) ? 4 : 2;
}

template <class T>
void dense_solve(stokes_ctx* c, const DenseInv& D, int W, const T* x, T* y) {
  const T* Ci = ops::pick<T>(D.i64, D.i32);
  auto go = [&](auto Wc) {
    constexpr int WW = decltype(Wc)::value;
    auto launch = [&](auto Rc) {
      constexpr int RW = decltype(Rc)::value, rows = RW * kBlock / 64;
      hipLaunchKernelGGL((k_dense_mv<T, WW, RW>), dim3((D.n + rows - 1) / rows), dim3(kBlock), 0, c->stream, D.n,
                         D.ld, Ci, x, y);
    };
    if constexpr (WW >= 4) {
      const int rw = dense_rw(D.n, WW, sizeof(T));
      if (rw == 4) return launch(std::integral_constant<int, 4>{});
      if (rw == 2) return launch(std::integral_constant<int, 2>{});
    }
    launch(std::integral_constant<int, 1>{});
  };
  switch (W) {
    case 1: go(std::integral_constant<int, 1>{}); break;
    case 2: go(std::integral_constant<int, 2>{}); break;
    case 3: go(std::integral_constant<int, 3>{}); break;
    case 4: go(std::integral_constant<int, 4>{}); break;
    case 6: go(std::integral_constant<int, 6>{}); break;
    case 8: go(std::integral_constant<int, 8>{}); break;
    case 12: go(std::integral_constant<int, 12>{}); break;
    case 16: go(std::integral_constant<int, 16>{}); break;
    case 24: go(std::integral_constant<int, 24>{}); break;
    default: throw Error(STOKES_ERR_UNSUPPORTED, "dense solve width " + std::to_string(W));
  }
  ops::check_launch();
  ops::count_bytes(c, double(D.n) * D.ld * sizeof(T) + 2.0 * D.n * W * sizeof(T));  // the inverse, x, y
}
template void dense_solve<float>(stokes_ctx*, const DenseInv&, int, const float*, float*);
template void dense_solve<double>(stokes_ctx*, const DenseInv&, int, const double*, double*);

}  // namespace stokes
