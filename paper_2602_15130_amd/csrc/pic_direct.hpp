// Direct Poisson solve: one correction in the full discrete Fourier basis.
//
// The periodic operator A = -L_h (7-point or trilinear elements) is diagonal
// in the products of the 1-D modes 1, cos(2 pi k i / n), sin(2 pi k i / n) and,
// for even n, (-1)^i; pic_lowmode.hpp solves the lowest of them before the CG,
// and here all n modes of every axis are taken, so that the residual r_0 = -b -
// A x_0 of the warm start (formed with the right-hand side) is solved away at
// once; the constant mode is left alone, x keeps its zero mean.  Three 1-D
// transforms each way, as matrix products with the n x n table of an axis:
// 12 n^4 operations on an n^3 mesh, on the FP64 matrix cores.
//
// k_direct_check then forms the true residual of the corrected x and E = -grad
// phi.  The CG kernel is launched as before: each of its workgroups sums the
// check's partials and leaves if ||r|| <= tol ||b||, else the CG runs from x
// (and rebuilds E).  Rounding leaves ||r|| / ||b|| near 2e-18 n^2 (9e-15 at 64^3,
// 4e-14 at 128^3), so at the usual 1e-12 the CG does not run.
//
// Bound: launch latency and the products' load chains on small meshes, the
// matrix cores from 128^3 on.
//
// Every sum has a fixed order, so results do not depend on scheduling.
#pragma once

#include "pic_kernels.hpp"

namespace pic {

struct DirectArgs {
  const double* f[3];  // [n][n] per axis: row a, mode a at nodes 0 .. n - 1
  const double* t[3];  // its transpose: row i, all modes at node i
  const double* lam;   // [3][nmax] 1-D eigenvalues
  int nmax;
  double *u, *w;       // two mesh-sized buffers; w holds the residual at the start
  double* x;
  const double* part;  // block sums of b
  int nparts;
  double* mean;        // their total over the node count, for k_direct_check
};

__device__ inline DirectArgs member_view(const SimConst& K, DirectArgs d) {
  for (int a = 0; a < 3; ++a) {
    d.f[a] = mem(K, d.f[a]);
    d.t[a] = mem(K, d.t[a]);
  }
  d.lam = mem(K, d.lam);
  d.u = mem(K, d.u);
  d.w = mem(K, d.w);
  d.x = mem(K, d.x);
  d.part = mem(K, d.part);
  d.mean = mem(K, d.mean);
  return d;
}

// Doubles of the tables of a mesh.
inline int64_t direct_table_doubles(const int nc[3]) {
  int64_t s = 0, nmax = 0;
  for (int d = 0; d < 3; ++d) {
    s += 2 * (int64_t)nc[d] * nc[d];
    nmax = nc[d] > nmax ? nc[d] : nmax;
  }
  return s + 3 * nmax;
}

__global__ void __launch_bounds__(kBlock) k_direct_tables(SimConst K, double* base, int nmax) {
  base = mem(K, base);
  const int64_t at = blockIdx.x * (int64_t)kBlock + threadIdx.x;
  int64_t t = at;
  double* f = base;
  for (int d = 0; d < 3; ++d) {
    const int n = K.nc[d];
    const int64_t sq = (int64_t)n * n;
    if (t < 2 * sq) {
      // row a of the table, row i of its transpose (angles reduced exactly in integers)
      const int r = (int)((t % sq) / n), q = (int)((t % sq) % n);
      const int a = t < sq ? r : q, i = t < sq ? q : r, k = (a + 1) / 2;
      const double arg = (double)((2 * (int64_t)k * i) % (2 * n)) / (double)n;
      f[t] = a == 0 ? 1.0 : ((a & 1) ? cospi(arg) : sinpi(arg));
      return;
    }
    t -= 2 * sq;
    f += 2 * sq;
  }
  if (t < 3 * nmax) {
    const int d = (int)(t / nmax), a = (int)(t % nmax);
    const double s = a < K.nc[d] ? sinpi((double)((a + 1) / 2) / (double)K.nc[d]) : 0.0;
    f[t] = 4.0 * s * s * K.ih2[d];
  }
}

// 1 / (eigenvalue times squared norm) of mode (a, b, c); 0 for the constant.
__device__ inline double direct_scale(const SimConst& K, const DirectArgs& D, int a, int b, int c) {
  const double ma = D.lam[a], mb = D.lam[D.nmax + b], mc = D.lam[2 * D.nmax + c];
  double lam = ma + mb + mc;
  if (K.poisson_op == 1) {  // Q1: mu_d times the 1-D mass eigenvalues 1 - mu h^2 / 6 of the others
    const double sa = 1.0 - ma / (6.0 * K.ih2[0]), sb = 1.0 - mb / (6.0 * K.ih2[1]),
                 sc = 1.0 - mc / (6.0 * K.ih2[2]);
    lam = ma * sb * sc + sa * mb * sc + sa * sb * mc;
  }
  auto half = [&](int m, int n) { return m == 0 || 2 * ((m + 1) / 2) == n ? 1.0 : 0.5; };
  const double nrm = half(a, K.nc[0]) * half(b, K.nc[1]) * half(c, K.nc[2]) * (double)K.nn;
  return a + b + c > 0 ? 1.0 / (lam * nrm) : 0.0;
}

// Mean of b from the block sums, by one workgroup of NT threads (for the check).
template <int NT>
__device__ inline void direct_mean(const SimConst& K, const DirectArgs& D, double* sh) {
  double acc = 0.0;
  for (int i = threadIdx.x; i < D.nparts; i += NT) acc += D.part[i];
  acc = block_sum_t<NT>(acc, sh);
  if (threadIdx.x == 0) *D.mean = acc / (double)K.nn;
}

// v_mfma_f64_16x16x4f64: lane l gives A[l % 16][l / 16] and B[l / 16][l % 16];
// its four results are C[4 v + l / 16][l % 16], v = 0 .. 3.
typedef double f64x4 __attribute__((ext_vector_type(4)));
__device__ inline f64x4 mfma_f64(double a, double b, f64x4 c) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
#else
  return c;
#endif
}

// The six transforms one by one, C = A B with A row-major in k and B row-major in n:
//   0  x forward   rows (k, j), A = w (the residual), B = transposed table -> u
//   1  y forward   per z plane, A = table, B = u's plane             -> w
//   2  z forward   A = table, B = w as [nz][nx ny], scaled           -> u
//   3  z backward  A = transposed table, B = u                       -> w
//   4  y backward  per z plane, A = transposed table, B = w's plane  -> u
//   5  x backward  A = u, B = table                                  -> added to x
// A workgroup of four waves makes a T x T tile of C, a wave T/2 x T/2 of it;
// k in chunks of 32 staged through LDS, the next chunk's loads in flight
// during the products.  T = 64 where that gives every CU a tile, else 32.
constexpr int kDirectK = 32;

template <int MODE, int T>
__global__ void __launch_bounds__(256) k_direct_axis(SimConst K, DirectArgs D) {
  D = member_view(K, D);
  constexpr int S = T / 32;          // 16 x 16 products of a wave along each side
  constexpr int PA = T * kDirectK / 256;  // elements of A (and of B) a thread stages
  __shared__ double As[T][kDirectK + 1], Bs[kDirectK][T + 1];
  __shared__ double sh[4];
  const int nx = K.nc[0], ny = K.nc[1], nz = K.nc[2], plane = nx * ny;
  constexpr bool X = MODE == 0 || MODE == 5, Y = MODE == 1 || MODE == 4;
  const int M = X ? ny * nz : (Y ? ny : nz), N = Y || X ? nx : plane, KK = X ? nx : (Y ? ny : nz);
  const int mt = (M + T - 1) / T;
  const int batch = blockIdx.x / mt, m0 = (blockIdx.x - batch * mt) * T, n0 = blockIdx.y * T;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r = lane & 15, g = lane >> 4;
  const int wm = (wave & 1) * (T / 2), wn = (wave >> 1) * (T / 2);
  if (MODE == 0 && blockIdx.x == 0 && blockIdx.y == 0) direct_mean<256>(K, D, sh);
  const double* src = MODE == 1 || MODE == 3 || MODE == 5 ? D.u : D.w;
  double* dst = MODE == 0 || MODE == 2 || MODE == 4 ? D.u : D.w;
  const int64_t at = Y ? (int64_t)batch * plane : 0;
  auto load_a = [&](int m, int k) -> double {
    if (m >= M || k >= KK) return 0.0;
    if (MODE == 1) return D.f[1][(int64_t)m * ny + k];
    if (MODE == 2) return D.f[2][(int64_t)m * nz + k];
    if (MODE == 3) return D.t[2][(int64_t)m * nz + k];
    if (MODE == 4) return D.t[1][(int64_t)m * ny + k];
    return src[(int64_t)m * nx + k];
  };
  auto load_b = [&](int k, int n) -> double {
    if (k >= KK || n >= N) return 0.0;
    if (MODE == 0) return D.t[0][(int64_t)k * nx + n];
    if (MODE == 5) return D.f[0][(int64_t)k * nx + n];
    return src[at + (int64_t)k * N + n];
  };
  double ra[PA], rb[PA];
  auto fetch = [&](int k0) {
#pragma unroll
    for (int q = 0; q < PA; ++q) {
      ra[q] = load_a(m0 + tid / kDirectK + q * (256 / kDirectK), k0 + tid % kDirectK);
      rb[q] = load_b(k0 + tid / T + q * (256 / T), n0 + tid % T);
    }
  };
  f64x4 acc[S][S];
#pragma unroll
  for (int i = 0; i < S; ++i)
#pragma unroll
    for (int j = 0; j < S; ++j) acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};
  fetch(0);
  for (int k0 = 0; k0 < KK; k0 += kDirectK) {
    __syncthreads();  // the last chunk is consumed
#pragma unroll
    for (int q = 0; q < PA; ++q) {
      As[tid / kDirectK + q * (256 / kDirectK)][tid % kDirectK] = ra[q];
      Bs[tid / T + q * (256 / T)][tid % T] = rb[q];
    }
    __syncthreads();
    if (k0 + kDirectK < KK) fetch(k0 + kDirectK);
#pragma unroll
    for (int k = 0; k < kDirectK; k += 4) {
      double a[S], b[S];
#pragma unroll
      for (int i = 0; i < S; ++i) {
        a[i] = As[wm + 16 * i + r][k + g];
        b[i] = Bs[k + g][wn + 16 * i + r];
      }
#pragma unroll
      for (int i = 0; i < S; ++i)
#pragma unroll
        for (int j = 0; j < S; ++j) acc[i][j] = mfma_f64(a[i], b[j], acc[i][j]);
    }
  }
#pragma unroll
  for (int j = 0; j < S; ++j) {
    const int n = n0 + wn + 16 * j + r;
    if (n >= N) continue;
#pragma unroll
    for (int i = 0; i < S; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int m = m0 + wm + 16 * i + 4 * v + g;
        if (m >= M) continue;
        const int64_t o = at + (int64_t)m * N + n;
        if (MODE == 2) dst[o] = acc[i][j][v] * direct_scale(K, D, n % nx, n / nx, m);
        else if (MODE == 5) D.x[o] += acc[i][j][v];
        else dst[o] = acc[i][j][v];
      }
  }
}

// C = A B over all 16 x 16 tiles of M x N by the NW waves of a workgroup, operands
// from LDS: A(m, k), B(k, n), and store(m, n, value); k up to a multiple of four,
// where one of the operands (a table) is zero beyond KK.
template <int NW, class FA, class FB, class FS>
__device__ inline void direct_product(int M, int N, int KK, FA A, FB B, FS store) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 15, g = lane >> 4;
  const int tm = (M + 15) / 16, tn = (N + 15) / 16;
  for (int t = wave; t < tm * tn; t += NW) {
    const int m0 = (t / tn) * 16, n0 = (t % tn) * 16;
    const int ma = min(m0 + r, M - 1), nb = min(n0 + r, N - 1);
    f64x4 c = {0.0, 0.0, 0.0, 0.0};
    int k = 0;
    for (; k + 16 <= KK; k += 16) {
      double a[4], b[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        a[q] = A(ma, k + 4 * q + g);
        b[q] = B(k + 4 * q + g, nb);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) c = mfma_f64(a[q], b[q], c);
    }
    for (; k < KK; k += 4) c = mfma_f64(A(ma, k + g), B(k + g, nb), c);
    if (n0 + r < N)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (m0 + 4 * v + g < M) store(m0 + 4 * v + g, n0 + r, c[v]);
  }
  __syncthreads();
}

// A table in LDS, rows of stride direct_pitch(n), zero beyond n.
__host__ __device__ inline int direct_pitch(int n) { return ((n + 3) / 4 * 4) | 1; }
__host__ __device__ inline int direct_table_lds(int n) { return (n + 3) / 4 * 4 * direct_pitch(n); }
template <int NT>
__device__ inline void direct_stage_table(const double* f, int n, double* p) {
  const int n4 = (n + 3) / 4 * 4, lp = direct_pitch(n);
  for (int t0 = threadIdx.x; t0 < n4 * n4; t0 += 4 * NT) {  // (four loads in flight)
    double v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int t = t0 + q * NT, a = t / n4, i = t - a * n4;
      v[q] = a < n && i < n ? f[a * n + i] : 0.0;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int t = t0 + q * NT, a = t / n4, i = t - a * n4;
      if (a < n4) p[a * lp + i] = v[q];
    }
  }
}

// Meshes whose planes fit LDS twice, with the tables of x and y, and whose z table
// does: three launches instead of six, the transforms of x and y in one
// (DIR 0 forward, w -> u; 1 backward, w -> added to x), a workgroup of 16 waves
// per plane, and those of z both ways in the other (u -> w), a workgroup of eight
// waves per 16 columns.  Bound by launches and by the loads of the tables; a launch
// per axis is 4 to 7 us for 1 us of products.  Six launches against three: 28
// and 19 us at 32^3, 35 and 36 at 64^3, where the three gaps between launches
// that are gone decide (a step 0.8 % faster).
constexpr int kDirectPlaneThreads = 1024;
inline size_t direct_plane_lds(const int nc[3]) {
  return (2 * (size_t)nc[1] * (nc[0] | 1) + direct_table_lds(nc[0]) + direct_table_lds(nc[1])) *
         sizeof(double);
}
constexpr int kDirectColumns = 16, kDirectColumnThreads = 512;
inline size_t direct_column_lds(const int nc[3]) {
  return (2 * (size_t)nc[2] * (kDirectColumns + 1) + direct_table_lds(nc[2])) * sizeof(double);
}

template <int DIR>
__global__ void __launch_bounds__(kDirectPlaneThreads) k_direct_plane(SimConst K, DirectArgs D) {
  D = member_view(K, D);
  extern __shared__ double lds[];
  __shared__ double sh[kDirectPlaneThreads / 64];
  const int nx = K.nc[0], ny = K.nc[1], ld = nx | 1, lx = direct_pitch(nx), ly = direct_pitch(ny);
  double* P = lds;
  double* Q = P + ny * ld;
  double* tx = Q + ny * ld;
  double* ty = tx + direct_table_lds(nx);
  const int64_t at = (int64_t)blockIdx.x * nx * ny;
  if (DIR == 0 && blockIdx.x == 0) direct_mean<kDirectPlaneThreads>(K, D, sh);
  direct_stage_table<kDirectPlaneThreads>(D.f[0], nx, tx);
  direct_stage_table<kDirectPlaneThreads>(D.f[1], ny, ty);
  for (int t0 = threadIdx.x; t0 < nx * ny; t0 += 4 * kDirectPlaneThreads) {
    double v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int t = t0 + q * kDirectPlaneThreads;
      v[q] = t < nx * ny ? D.w[at + t] : 0.0;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int t = t0 + q * kDirectPlaneThreads, j = t / nx;
      if (t < nx * ny) P[j * ld + t - j * nx] = v[q];
    }
  }
  __syncthreads();
  constexpr int NW = kDirectPlaneThreads / 64;
  if constexpr (DIR == 0) {
    direct_product<NW>(ny, nx, nx, [&](int m, int k) { return P[m * ld + min(k, nx - 1)]; },
                       [&](int k, int n) { return tx[n * lx + k]; },
                       [&](int m, int n, double v) { Q[m * ld + n] = v; });
    direct_product<NW>(ny, nx, ny, [&](int m, int k) { return ty[m * ly + k]; },
                       [&](int k, int n) { return Q[min(k, ny - 1) * ld + n]; },
                       [&](int m, int n, double v) { D.u[at + m * nx + n] = v; });
  } else {
    direct_product<NW>(ny, nx, ny, [&](int m, int k) { return ty[k * ly + m]; },
                       [&](int k, int n) { return P[min(k, ny - 1) * ld + n]; },
                       [&](int m, int n, double v) { Q[m * ld + n] = v; });
    direct_product<NW>(ny, nx, nx, [&](int m, int k) { return Q[m * ld + min(k, nx - 1)]; },
                       [&](int k, int n) { return tx[k * lx + n]; },
                       [&](int m, int n, double v) { D.x[at + m * nx + n] += v; });
  }
}

__global__ void __launch_bounds__(kDirectColumnThreads) k_direct_columns(SimConst K, DirectArgs D) {
  D = member_view(K, D);
  extern __shared__ double lds[];
  const int nx = K.nc[0], nz = K.nc[2], plane = nx * K.nc[1], lz = direct_pitch(nz);
  constexpr int ld = kDirectColumns + 1;
  double* P = lds;
  double* Q = P + nz * ld;
  double* tz = Q + nz * ld;
  const int c0 = blockIdx.x * kDirectColumns, nc = min(kDirectColumns, plane - c0);
  direct_stage_table<kDirectColumnThreads>(D.f[2], nz, tz);
  for (int t0 = threadIdx.x; t0 < nz * kDirectColumns; t0 += 4 * kDirectColumnThreads) {
    double v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int t = t0 + q * kDirectColumnThreads, k = t / kDirectColumns, i = t % kDirectColumns;
      v[q] = k < nz && i < nc ? D.u[(int64_t)k * plane + c0 + i] : 0.0;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int t = t0 + q * kDirectColumnThreads, k = t / kDirectColumns;
      if (k < nz) P[k * ld + t % kDirectColumns] = v[q];
    }
  }
  __syncthreads();
  constexpr int NW = kDirectColumnThreads / 64;
  direct_product<NW>(nz, nc, nz, [&](int m, int k) { return tz[m * lz + k]; },
                     [&](int k, int n) { return P[min(k, nz - 1) * ld + n]; },
                     [&](int m, int n, double v) {
                       Q[m * ld + n] = v * direct_scale(K, D, (c0 + n) % nx, (c0 + n) / nx, m);
                     });
  direct_product<NW>(nz, nc, nz, [&](int m, int k) { return tz[k * lz + m]; },
                     [&](int k, int n) { return Q[min(k, nz - 1) * ld + n]; },
                     [&](int m, int n, double v) { D.w[(int64_t)m * plane + c0 + n] = v; });
}

// A mesh that fits one workgroup's LDS twice: all six transforms in one launch,
// one workgroup of 16 waves per member, so that a small solve costs one launch's
// latency instead of six.  Rows along x have an odd stride (bank spread).
constexpr int kDirectSmallThreads = 1024;
inline size_t direct_small_lds(const int nc[3]) {
  const size_t ld = nc[0] | 1, buf = (size_t)nc[2] * nc[1] * ld;
  size_t tab = 0;
  for (int d = 0; d < 3; ++d) tab += direct_table_lds(nc[d]);
  return (2 * buf + tab) * sizeof(double);
}

__global__ void __launch_bounds__(kDirectSmallThreads) k_direct_small(SimConst K, DirectArgs D) {
  D = member_view(K, D);
  extern __shared__ double lds[];
  __shared__ double sh[kDirectSmallThreads / 64];
  const int nx = K.nc[0], ny = K.nc[1], nz = K.nc[2];
  const int ld = nx | 1, pl = ny * ld;  // row and plane stride
  double* P = lds;
  double* Q = P + nz * pl;
  const int tid = threadIdx.x;
  direct_mean<kDirectSmallThreads>(K, D, sh);
  const double* tab[3];
  int lp[3];
  {
    double* p = Q + nz * pl;
    for (int d = 0; d < 3; ++d) {
      direct_stage_table<kDirectSmallThreads>(D.f[d], K.nc[d], p);
      tab[d] = p;
      lp[d] = direct_pitch(K.nc[d]);
      p += direct_table_lds(K.nc[d]);
    }
  }
  for (int t = tid; t < nz * pl; t += kDirectSmallThreads) {
    const int i = t % ld, row = t / ld;
    P[t] = i < nx ? D.w[row * nx + i] : 0.0;
    Q[t] = 0.0;
  }
  __syncthreads();
  auto product = [&](int M, int N, int KK, auto A, auto B, auto store) {
    direct_product<kDirectSmallThreads / 64>(M, N, KK, A, B, store);
  };
  // (beyond an axis the table is zero; the other operand repeats its last row)
  const int rows = ny * nz;
  product(rows, nx, nx, [&](int m, int k) { return P[m * ld + min(k, nx - 1)]; },
          [&](int k, int n) { return tab[0][n * lp[0] + k]; },
          [&](int m, int n, double v) { Q[m * ld + n] = v; });
  for (int dir = 0; dir < 2; ++dir) {
    // y of every plane: columns (k, a), rows of the table forward, columns backward
    auto ytab = [&](int m, int k) { return dir ? tab[1][k * lp[1] + m] : tab[1][m * lp[1] + k]; };
    const double* from = dir ? P : Q;
    double* to = dir ? Q : P;
    product(ny, nz * nx, ny, ytab,
            [&](int k, int n) { return from[(n / nx) * pl + min(k, ny - 1) * ld + n % nx]; },
            [&](int m, int n, double v) { to[(n / nx) * pl + m * ld + n % nx] = v; });
    if (dir) break;
    product(nz, pl, nz, [&](int m, int k) { return tab[2][m * lp[2] + k]; },
            [&](int k, int n) { return P[min(k, nz - 1) * pl + n]; },
            [&](int m, int n, double v) {
              const int a = n % ld;
              Q[m * pl + n] = a < nx ? v * direct_scale(K, D, a, n / ld, m) : 0.0;
            });
    product(nz, pl, nz, [&](int m, int k) { return tab[2][k * lp[2] + m]; },
            [&](int k, int n) { return Q[min(k, nz - 1) * pl + n]; },
            [&](int m, int n, double v) { P[m * pl + n] = v; });
  }
  product(rows, nx, nx, [&](int m, int k) { return Q[m * ld + min(k, nx - 1)]; },
          [&](int k, int n) { return tab[0][k * lp[0] + n]; },
          [&](int m, int n, double v) { D.x[m * nx + n] += v; });
}

// The corrected potential's residual (block sums of r^2 and of b^2, b's mean
// removed from here on) and E = -grad phi with its FP32 copy; also zeroes the
// CG's barrier words (nbar of them).
constexpr int kCheckBlocks = 1024;
__global__ void __launch_bounds__(kBlock) k_direct_check(SimConst K, double* b, const double* x,
                                                         const double* mean, double* check,
                                                         double* E, float* E32, unsigned* bar,
                                                         int nbar) {
  b = mem(K, b);
  x = mem(K, x);
  mean = mem(K, mean);
  check = mem(K, check);
  E = mem(K, E);
  E32 = mem(K, E32);
  bar = mem(K, bar);
  __shared__ double sh[3 * kWaves];
  const int stride = gridDim.x * kBlock;
  for (int t = blockIdx.x * kBlock + threadIdx.x; t < nbar; t += stride) bar[t] = 0u;
  const double mb = *mean;
  double v[3] = {0.0, 0.0, 0.0};
  for (int n = blockIdx.x * kBlock + threadIdx.x; n < K.nn; n += stride) {
    int i, j, k;
    node_coords(K, n, i, j, k);
    const double bv = b[n] - mb;
    const double rv = -bv - neg_lap(K, i, j, k, [&](int m) { return x[m]; });
    b[n] = bv;
    v[0] += rv * rv;
    v[1] += bv * bv;
    node_field(K, x, n, i, j, k, E, E32);
  }
  block_sum3_t<kBlock>(v, 2, sh);
  if (threadIdx.x == 0) {
    check[blockIdx.x] = v[0];
    check[gridDim.x + blockIdx.x] = v[1];
  }
}

}  // namespace pic
