// Diagnostics of a march that read a field once and reduce it: the
// horizontal power spectrum of Eq. 12 and the 2-D power spectrum whose
// strongest modes make the 90 %-power reconstruction of App. B.  Kept apart from the stepping
// kernels; launched through rt_diag.h by the C ABI.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "rt_diag.h"

namespace rtk {
namespace {

constexpr int kSpecThreads = 256;

// DFTs of n <= kSplitMax points in two stages, n = n1 n2 with n1 the largest
// divisor up to sqrt(n):
//   Y[b][j] = sum_a f[a n2 + b] w^{a j n2},  j < n1, b < n2
//   F[k]    = sum_b Y[b][k mod n1] w^{b k}
// with w = e^{-2 pi i / n}: n1 + n2 products per coefficient instead of n.
// Twiddles and Y in LDS; every twiddle is sincospi of its own angle.  The
// direct kernels below, n products per coefficient, take prime n (n1 = 1),
// longer lines, whose tables and Y exceed the default LDS limit of 64 KB, and
// those of a large prime factor where that is faster (row_split, col_split).
// 256x256: rows 13.5 -> 5.0 us, columns 39.7 -> 5.6, one row's spectrum 11.3 ->
// 3.4; bound by the LDS reads of the twiddles (two per product).
constexpr int kSplitMax = 2048;

int split_of(int n) {
  int n1 = 1;
  for (int d = 2; d * d <= n; ++d)
    if (n % d == 0) n1 = d;
  return n1;
}

bool splits(int n) { return n <= kSplitMax && split_of(n) > 1; }

// Stages or not, for lines that can be split.  One block does all of a split
// line, where the direct kernels give 256 coefficients to each block, so with
// n2 a large prime the split block's chain of products is the longer one and
// pays only if the chip is full.  A launch takes ns per product of a block's
// chain, times share per block on a CU once that exceeds 1 (fitted on 64x2042 to
// 2018x2018, batches of 1 to 16; the direct columns wait for strided loads).
// Direct and split, us: 2042x64 98.6 and 197, 2042x2 85 and 191, 64x2042 279 and
// 384, but 8 x 64x2042 787 and 647, 16x1006 143 and 100, 300x302 65 and 25.
int chunks(int n) { return (n + kSpecThreads - 1) / kSpecThreads; }
double chain_ns(long blocks, long chain, double ns, double share) {
  constexpr long kCus = 256;
  return ns * (double)chain * std::max(1.0, share * (double)((blocks + kCus - 1) / kCus));
}
bool row_split(int nx, int ny, int nb) {
  if (!splits(nx)) return false;
  const int nk = nx / 2 + 1, n1 = split_of(nx);
  return chain_ns((long)ny * nb, chunks(nx) * n1 + chunks(nk) * (nx / n1), 46.0, 0.9) <
         chain_ns((long)chunks(nk) * ny * nb, nx, 45.0, 0.58);
}
bool col_split(int ny, int nk, int nb) {
  if (!splits(ny)) return false;
  const int n1 = split_of(ny);
  return chain_ns((long)nk * nb, chunks(ny) * (n1 + ny / n1), 48.0, 0.8) <
         chain_ns((long)chunks(ny) * nk * nb, ny, 140.0, 0.33);
}

__device__ __forceinline__ void twiddles(int n, double* tw) {  // [0, n): cos(2 pi k / n), [n, 2 n): sin
  for (int k = threadIdx.x; k < n; k += kSpecThreads) {
    double sn, cs;
    sincospi(2.0 * k / n, &sn, &cs);
    tw[k] = cs;
    tw[n + k] = sn;
  }
}

// Stage 2 for coefficient k of a line's Y ([n2][n1] (re, im) pairs).
__device__ __forceinline__ void stage2(int n, int n1, int n2, const double* tw, const double* Y, int k, double& re,
                                       double& im) {
  re = 0.0;
  im = 0.0;
  int idx = 0;
  const double* y = Y + 2 * (k % n1);
  for (int b = 0; b < n2; ++b) {
    const double cr = y[2 * b * n1], ci = y[2 * b * n1 + 1], c = tw[idx], s = tw[n + idx];
    re += cr * c + ci * s;  // (cr + i ci)(c - i s)
    im += ci * c - cr * s;
    idx += k;
    if (idx >= n) idx -= n;
  }
}

// Stage 1 of a row of real values into Y.
__device__ __forceinline__ void stage1_real(int n, int n1, int n2, const double* tw, const double* f, double* Y) {
  for (int o = threadIdx.x; o < n; o += kSpecThreads) {
    const int b = o / n1, step = (o - b * n1) * n2;
    double re = 0.0, im = 0.0;
    int idx = 0;
    for (int a = 0; a < n1; ++a) {
      const double v = f[a * n2 + b];
      re += v * tw[idx];
      im -= v * tw[n + idx];
      idx += step;
      if (idx >= n) idx -= n;
    }
    Y[2 * o] = re;
    Y[2 * o + 1] = im;
  }
}

// C[b][y][k], k = 0 .. nx/2, of every row; one block per row and member.
__global__ __launch_bounds__(kSpecThreads) void k_dft_rows_split(int nx, int ny, int n1, const double* f,
                                                                 long long mstride, int nk, double* C) {
  extern __shared__ double lds[];  // twiddles 2 nx, Y 2 nx
  const int y = blockIdx.x, b = blockIdx.y;
  twiddles(nx, lds);
  __syncthreads();
  stage1_real(nx, n1, nx / n1, lds, f + (long long)b * mstride + (size_t)y * nx, lds + 2 * nx);
  __syncthreads();
  double* c = C + ((size_t)b * ny + y) * nk * 2;
  for (int k = threadIdx.x; k < nk; k += kSpecThreads) {
    double re, im;
    stage2(nx, n1, nx / n1, lds, lds + 2 * nx, k, re, im);
    c[2 * k] = re;
    c[2 * k + 1] = im;
  }
}

// E[b][q][k] = |sum_y C[b][y][k] e^{-2 pi i q y / ny}|^2; one block per column
// and member.
__global__ __launch_bounds__(kSpecThreads) void k_dft_cols_split(int ny, int n1, int nk, const double* C, double* E) {
  extern __shared__ double lds[];  // twiddles 2 ny, Y 2 ny
  const int k = blockIdx.x, b = blockIdx.y, n2 = ny / n1;
  double* Y = lds + 2 * ny;
  twiddles(ny, lds);
  __syncthreads();
  const double* cb = C + ((size_t)b * ny * nk + k) * 2;
  for (int o = threadIdx.x; o < ny; o += kSpecThreads) {
    const int r = o / n1, step = (o - r * n1) * n2;
    double re = 0.0, im = 0.0;
    int idx = 0;
    for (int a = 0; a < n1; ++a) {
      const double* v = cb + (size_t)(a * n2 + r) * nk * 2;
      const double cr = v[0], ci = v[1], c = lds[idx], s = lds[ny + idx];
      re += cr * c + ci * s;
      im += ci * c - cr * s;
      idx += step;
      if (idx >= ny) idx -= ny;
    }
    Y[2 * o] = re;
    Y[2 * o + 1] = im;
  }
  __syncthreads();
  for (int q = threadIdx.x; q < ny; q += kSpecThreads) {
    double re, im;
    stage2(ny, n1, n2, lds, Y, q, re, im);
    E[((size_t)b * ny + q) * nk + k] = re * re + im * im;
  }
}

// E[b][k] = |F[k]|^2 of one row; one block per member.
__global__ __launch_bounds__(kSpecThreads) void k_one_row_spectrum(int nx, int n1, const double* f, long long mstride,
                                                                   int nbins, double* E) {
  extern __shared__ double lds[];
  const int b = blockIdx.x;
  twiddles(nx, lds);
  __syncthreads();
  stage1_real(nx, n1, nx / n1, lds, f + (long long)b * mstride, lds + 2 * nx);
  __syncthreads();
  for (int k = threadIdx.x; k < nbins; k += kSpecThreads) {
    double re, im;
    stage2(nx, n1, nx / n1, lds, lds + 2 * nx, k, re, im);
    E[(size_t)b * nbins + k] = re * re + im * im;
  }
}

// All rows, or one that is not split.  One block per (mode n, member b): each
// thread takes whole rows of the selection, forms the row's Fourier
// coefficient at n with the twiddles exp(-2 pi i k / nx) held in LDS (index
// n x mod nx, advanced by n per column), and accumulates its squared modulus;
// a fixed-order tree sums the threads.
__global__ __launch_bounds__(kSpecThreads) void k_row_spectrum(int nx, int ny, const double* f, long long mstride,
                                                               int row, int nbins, double* E) {
  extern __shared__ double tw[];  // [0, nx): cos(2 pi k / nx), [nx, 2 nx): sin
  __shared__ double red[kSpecThreads];
  const int n = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
  for (int k = tid; k < nx; k += kSpecThreads) {
    double s, c;
    sincospi(2.0 * k / nx, &s, &c);
    tw[k] = c;
    tw[nx + k] = s;
  }
  __syncthreads();
  const double* fb = f + (long long)b * mstride;
  const int j0 = row < 0 ? 0 : row, j1 = row < 0 ? ny : row + 1;
  double acc = 0.0;
  for (int j = j0 + tid; j < j1; j += kSpecThreads) {
    const double* fr = fb + (size_t)j * nx;
    double re = 0.0, im = 0.0;
    int idx = 0;
    for (int x = 0; x < nx; ++x) {
      const double v = fr[x];
      re += v * tw[idx];
      im -= v * tw[nx + idx];
      idx += n;
      if (idx >= nx) idx -= nx;
    }
    acc += re * re + im * im;
  }
  red[tid] = acc;
  __syncthreads();
  for (int s = kSpecThreads / 2; s > 0; s >>= 1) {
    if (tid < s) red[tid] += red[tid + s];
    __syncthreads();
  }
  if (tid == 0) E[(size_t)b * nbins + n] = red[0];
}

// 2-D DFT of lines that are not split, pass 1: C[b][y][k] = sum_x f_b(y, x)
// e^{-2 pi i k x / nx} for k = 0 .. nx/2, as (re, im) pairs.  One thread per coefficient, threads of
// a block along k for one row (the row's values are read by every thread:
// broadcast), twiddles in LDS.
__global__ __launch_bounds__(kSpecThreads) void k_dft_rows(int nx, int ny, const double* f, long long mstride,
                                                           int nk, double* C) {
  extern __shared__ double tw[];  // [0, nx): cos(2 pi k / nx), [nx, 2 nx): sin
  const int y = blockIdx.y, b = blockIdx.z, tid = threadIdx.x;
  for (int k = tid; k < nx; k += kSpecThreads) {
    double sn, cs;
    sincospi(2.0 * k / nx, &sn, &cs);
    tw[k] = cs;
    tw[nx + k] = sn;
  }
  __syncthreads();
  const int k = blockIdx.x * kSpecThreads + tid;
  if (k >= nk) return;
  const double* fr = f + (long long)b * mstride + (size_t)y * nx;
  double re = 0.0, im = 0.0;
  int idx = 0;
  for (int x = 0; x < nx; ++x) {
    const double v = fr[x];
    re += v * tw[idx];
    im -= v * tw[nx + idx];
    idx += k;
    if (idx >= nx) idx -= nx;
  }
  double* c = C + (((size_t)b * ny + y) * nk + k) * 2;
  c[0] = re;
  c[1] = im;
}

// Pass 2: F[b][q][k] = sum_y C[b][y][k] e^{-2 pi i q y / ny} for q = 0 ..
// ny - 1, and E = |F|^2.  One thread per (q, k), threads of a block along q
// for one k (each C[y][k] is read by every thread: broadcast).
__global__ __launch_bounds__(kSpecThreads) void k_dft_cols_power(int ny, int nk, const double* C, double* E) {
  extern __shared__ double tw[];  // [0, ny): cos(2 pi q / ny), [ny, 2 ny): sin
  const int k = blockIdx.y, b = blockIdx.z, tid = threadIdx.x;
  for (int q = tid; q < ny; q += kSpecThreads) {
    double sn, cs;
    sincospi(2.0 * q / ny, &sn, &cs);
    tw[q] = cs;
    tw[ny + q] = sn;
  }
  __syncthreads();
  const int q = blockIdx.x * kSpecThreads + tid;
  if (q >= ny) return;
  const double* cb = C + (size_t)b * ny * nk * 2 + (size_t)k * 2;
  double re = 0.0, im = 0.0;
  int idx = 0;
  for (int y = 0; y < ny; ++y) {
    const double cr = cb[(size_t)y * nk * 2], ci = cb[(size_t)y * nk * 2 + 1];
    const double c = tw[idx], s = tw[ny + idx];
    // (cr + i ci)(c - i s)
    re += cr * c + ci * s;
    im += ci * c - cr * s;
    idx += q;
    if (idx >= ny) idx -= ny;
  }
  E[((size_t)b * ny + q) * nk + k] = re * re + im * im;
}

}  // namespace

hipError_t launch_power_spectrum_2d(int nx, int ny, int nb, const double* f, long long member_stride, double* C,
                                    double* E, hipStream_t s) {
  if (nx < 1 || nx > kSpecMaxNx || ny < 1 || ny > kSpecMaxNx || nb < 1) return hipErrorInvalidValue;
  const int nk = nx / 2 + 1;
  if (row_split(nx, ny, nb))
    hipLaunchKernelGGL(k_dft_rows_split, dim3(ny, nb), dim3(kSpecThreads), 4 * (size_t)nx * sizeof(double), s, nx, ny,
                       split_of(nx), f, member_stride, nk, C);
  else
    hipLaunchKernelGGL(k_dft_rows, dim3((nk + kSpecThreads - 1) / kSpecThreads, ny, nb), dim3(kSpecThreads),
                       2 * (size_t)nx * sizeof(double), s, nx, ny, f, member_stride, nk, C);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (col_split(ny, nk, nb))
    hipLaunchKernelGGL(k_dft_cols_split, dim3(nk, nb), dim3(kSpecThreads), 4 * (size_t)ny * sizeof(double), s, ny,
                       split_of(ny), nk, C, E);
  else
    hipLaunchKernelGGL(k_dft_cols_power, dim3((ny + kSpecThreads - 1) / kSpecThreads, nk, nb), dim3(kSpecThreads),
                       2 * (size_t)ny * sizeof(double), s, ny, nk, C, E);
  return hipGetLastError();
}

hipError_t launch_row_spectrum(int nx, int ny, int nb, const double* f, long long member_stride, int row, double* E,
                               hipStream_t s) {
  if (nx < 1 || nx > kSpecMaxNx || ny < 1 || nb < 1 || row < -1 || row >= ny) return hipErrorInvalidValue;
  const int nbins = nx / 2 + 1;
  // One block per member does both stages in turn, where the direct kernel
  // has a block per mode: split only while the block's chain is the shorter.
  const int n1 = split_of(nx);
  if (row >= 0 && splits(nx) && chunks(nx) * n1 + chunks(nbins) * (nx / n1) < nx) {
    hipLaunchKernelGGL(k_one_row_spectrum, dim3(nb), dim3(kSpecThreads), 4 * (size_t)nx * sizeof(double), s, nx,
                       n1, f + (size_t)row * nx, member_stride, nbins, E);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_row_spectrum, dim3(nbins, nb), dim3(kSpecThreads), 2 * (size_t)nx * sizeof(double), s, nx,
                     ny, f, member_stride, row, nbins, E);
  return hipGetLastError();
}

}  // namespace rtk
