// Device helpers shared by the tile kernels (rt_kernels.hip) and the column
// kernels (rt_columns.hip): addressing, wavefront reductions and the order
// in which the chip's eight XCDs take a launch's work.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace rtk {

// Periodic column index.  The tile halos reach at most TX + 2 columns past
// the domain, so for every grid wider than that one conditional add or
// subtract does; narrower grids take the loop.
__device__ __forceinline__ int wrapx(int i, int nx) {
  i = i < 0 ? i + nx : (i >= nx ? i - nx : i);
  if ((unsigned)i >= (unsigned)nx) {
    while (i < 0) i += nx;
    while (i >= nx) i -= nx;
  }
  return i;
}

// Element i of an array of doubles (or int32) addressed as a uniform base
// plus a 32-bit byte offset, which maps onto the scalar-base / 32-bit
// vector-offset form of the global memory instructions.  Every plane of a
// state holds fewer than 2^28 cells (checked when a context is created).
__device__ __forceinline__ double ldg(const double* base, uint32_t i) {
  return *reinterpret_cast<const double*>(reinterpret_cast<const char*>(base) + i * 8u);
}
__device__ __forceinline__ void stg(double* base, uint32_t i, double v) {
  *reinterpret_cast<double*>(reinterpret_cast<char*>(base) + i * 8u) = v;
}
__device__ __forceinline__ int32_t ldg(const int32_t* base, uint32_t i) {
  return *reinterpret_cast<const int32_t*>(reinterpret_cast<const char*>(base) + i * 4u);
}
__device__ __forceinline__ void stg(int32_t* base, uint32_t i, int32_t v) {
  *reinterpret_cast<int32_t*>(reinterpret_cast<char*>(base) + i * 4u) = v;
}

// Wavefront reductions with DPP lane permutations inside each row of 16
// lanes (swap neighbours, swap pairs, mirror half-rows, mirror rows: after
// the four steps every lane holds its row's result, the same in every lane
// because each step combines a lane with its partner in both orders), then
// the four rows' results read from lanes 0, 16, 32, 48 and combined in a
// fixed order.  Called with the whole wavefront active; `id` fills lanes
// whose source is inactive.
template <int CTRL>
__device__ __forceinline__ double dpp_perm(double v, double id) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const unsigned long long o = (unsigned long long)__double_as_longlong(id);
  const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp((int)(unsigned)o, (int)(unsigned)b, CTRL, 0xf, 0xf, false);
  const unsigned hi =
      (unsigned)__builtin_amdgcn_update_dpp((int)(unsigned)(o >> 32), (int)(unsigned)(b >> 32), CTRL, 0xf, 0xf, false);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

__device__ __forceinline__ double read_lane(double v, int lane) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, lane);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), lane);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

constexpr int kDppQuadSwap1 = 0xB1;  // quad_perm [1, 0, 3, 2]
constexpr int kDppQuadSwap2 = 0x4E;  // quad_perm [2, 3, 0, 1]
constexpr int kDppHalfMirror = 0x141;
constexpr int kDppMirror = 0x140;

__device__ __forceinline__ double wave_max(double v) {
  const double id = -__builtin_inf();
  v = fmax(v, dpp_perm<kDppQuadSwap1>(v, id));
  v = fmax(v, dpp_perm<kDppQuadSwap2>(v, id));
  v = fmax(v, dpp_perm<kDppHalfMirror>(v, id));
  v = fmax(v, dpp_perm<kDppMirror>(v, id));
  return fmax(fmax(read_lane(v, 0), read_lane(v, 16)), fmax(read_lane(v, 32), read_lane(v, 48)));
}

__device__ __forceinline__ double wave_sum(double v) {
  v += dpp_perm<kDppQuadSwap1>(v, 0.0);
  v += dpp_perm<kDppQuadSwap2>(v, 0.0);
  v += dpp_perm<kDppHalfMirror>(v, 0.0);
  v += dpp_perm<kDppMirror>(v, 0.0);
  return (read_lane(v, 0) + read_lane(v, 16)) + (read_lane(v, 32) + read_lane(v, 48));
}

template <int NT>
__device__ double block_max(double v, double* red) {
  v = wave_max(v);
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  __syncthreads();
  if (l == 0) red[w] = v;
  __syncthreads();
  double m = red[0];
#pragma unroll
  for (int k = 1; k < NT / 64; ++k) m = fmax(m, red[k]);
  return m;
}

template <int NT>
__device__ double block_sum(double v, double* red) {
  v = wave_sum(v);
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  __syncthreads();
  if (l == 0) red[w] = v;
  __syncthreads();
  double s = red[0];
#pragma unroll
  for (int k = 1; k < NT / 64; ++k) s += red[k];
  return s;
}

// Largest s over the block with the smallest i among equal s (a total
// order, so the result does not depend on the order of combination).
__device__ __forceinline__ void argmax_merge(double& s, int& i, double s2, int i2) {
  if (s2 > s || (s2 == s && i2 < i)) {
    s = s2;
    i = i2;
  }
}

template <int NT>
__device__ void block_argmax(double& s, int& i, double* rs, int* ri) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) argmax_merge(s, i, __shfl_xor(s, o, 64), __shfl_xor(i, o, 64));
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  __syncthreads();
  if (l == 0) {
    rs[w] = s;
    ri[w] = i;
  }
  __syncthreads();
  s = rs[0];
  i = ri[0];
#pragma unroll
  for (int k = 1; k < NT / 64; ++k) argmax_merge(s, i, rs[k], ri[k]);
}

// Workgroups are dispatched round-robin over the 8 XCDs of the chip (linear
// id mod 8), and each XCD has its own L2.  With tiles in raster order,
// horizontally adjacent tiles would sit on different XCDs and each L2 would
// fetch the halo cache lines they share.  Instead, the workgroups of XCD k
// take the k-th contiguous band of tiles (in raster order within the band):
// horizontal neighbours share an L2, and vertical neighbours follow one
// tile row later in the same L2.  A bijection of [0, T) for any T.
constexpr int kXcds = 8;

__device__ __forceinline__ int xcd_band(int L, int T) {
  const int per = (T + kXcds - 1) / kXcds;  // items of each of the first `tall` XCDs
  const int tall = T - (per - 1) * kXcds;   // 1..8 XCDs with `per` items, the rest per - 1
  const int xcd = L % kXcds, local = L / kXcds;
  return xcd < tall ? xcd * per + local : tall * per + (xcd - tall) * (per - 1) + local;
}

__device__ __forceinline__ void tile_of_block(int& bx, int& by) {
  const int nbx = (int)gridDim.x;
  const int t = xcd_band((int)blockIdx.x + nbx * (int)blockIdx.y, nbx * (int)gridDim.y);
  bx = t % nbx;
  by = t / nbx;
}

}  // namespace rtk
