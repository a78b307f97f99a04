// Column kernels: one wavefront marches a strip of columns upward, one cell
// per lane and one row per iteration, with the rows a stencil needs in
// registers and x neighbours taken from the next lane (a lane shift of the
// whole wavefront).  No LDS and no barriers; what the tile kernels compute
// again for every tile's halo (primitives 1.58 and predictor 1.28 times per
// cell on 16x15 tiles) is computed once but for the outer lanes of a strip
// (4 of 64) and two rows around a segment.  The expressions are those of the
// tile kernels, so the results are the same to the bit.
//
// k_step_cols is bound by VALU issue: about 490 instructions per row and
// wavefront at a given dt (530 in the march) where the 16x15 tiles take 845
// per 64 cells plus their barriers.  Two rows per loop turn save 3-6 % (what
// a row hands to the next changes registers by name, not by moves).  Tiles
// against columns, us: 8 x 1024x2048 550 -> 320 given dt and 590 -> 348 in
// the march; 8 x 512x1024 153 -> 84 and 172 -> 94; 64 x 128x256 79 -> 58 and
// 95 -> 63; 1024x2048 68 -> 47 and 77 -> 51.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "rt_kernels.h"
#include "rt_wave.h"

namespace rtk {

namespace {

constexpr int kColWaves = 4;                 // wavefronts per block (they share nothing)
constexpr int kStepHalo = 2;                 // columns to each side a step needs
constexpr int kStepOwn = 64 - 2 * kStepHalo; // columns a wavefront of the step writes

// The value of the lane to the right / to the left (whole wavefront active;
// lane 63 / lane 0 get zero).
__device__ __forceinline__ double from_right(double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)b, 0x130, 0xf, 0xf, true);  // wave_shl:1
  const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), 0x130, 0xf, 0xf, true);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ double from_left(double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)b, 0x138, 0xf, 0xf, true);  // wave_shr:1
  const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), 0x138, 0xf, 0xf, true);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

struct Raw {
  double r, mx, my, E;
};

// Row gy of one member's state (clamped into the domain) at this lane's column.
__device__ __forceinline__ Raw load_row(const Params& P, const double* U, size_t N, int gy, uint32_t col) {
  const int sy = gy < 0 ? 0 : (gy >= P.ny ? P.ny - 1 : gy);
  const double* p = U + (size_t)sy * P.nx;
  return Raw{ldg(p, col), ldg(p + N, col), ldg(p + 2 * N, col), ldg(p + 3 * N, col)};
}

// Primitives of row gy, wall ghosts below row 0 and above row ny - 1.
__device__ __forceinline__ W4 row_prims(const Params& P, const Raw& q, int gy) {
  W4 w = cons_to_prim(P, q.r, q.mx, q.my, q.E);
  if (gy < 0) w = ghost_bottom(P, w);
  else if (gy >= P.ny) w = ghost_top(P, w);
  return w;
}

struct D4 {
  double r, u, v, p;
};
__device__ __forceinline__ D4 diff(const W4& a, const W4& b) { return D4{a.r - b.r, a.u - b.u, a.v - b.v, a.p - b.p}; }

template <bool BAL>
__global__ __launch_bounds__(64 * kColWaves) void k_step_cols(Params P, StepArgs a, int strips, int segs) {
  const int lane = threadIdx.x & 63;
  const int per = strips * segs;
  const int w = __builtin_amdgcn_readfirstlane(xcd_band((int)blockIdx.x, (int)gridDim.x) * kColWaves + (int)(threadIdx.x >> 6));
  if (w >= per * P.nb) return;
  const int b = w / per, t = w - b * per;
  const int seg = t / strips, strip = t - seg * strips;
  const int nx = P.nx, ny = P.ny;
  const size_t N = (size_t)nx * ny;
  const int ys = (int)((long)ny * seg / segs), ye = (int)((long)ny * (seg + 1) / segs);
  const int x0 = strip * kStepOwn;
  const uint32_t col = (uint32_t)wrapx(x0 - kStepHalo + lane, nx);
  const bool own = lane >= kStepHalo && lane < 64 - kStepHalo && x0 - kStepHalo + lane < nx;
  const bool first = t == 0;
  const double* U = a.U + (size_t)b * 4 * N;
  double* Un = a.Un + (size_t)b * 4 * N;

  // the rows below the segment and its first row, in flight while the time
  // step is formed
  const Raw qm = load_row(P, U, N, ys - 2, col);
  Raw uc = load_row(P, U, N, ys - 1, col);
  Raw un = load_row(P, U, N, ys, col);

  double dt = 0.0;
  int nstep = 0;
  bool last = false;
  const Ctl* cin = nullptr;
  Ctl* cout = nullptr;
  double t_in = 0.0, T_in = 0.0;
  if (a.ctl) {
    const int L = a.launch;
    cin = a.ctl + (size_t)(L & 1) * P.nb + b;
    cout = a.ctl + (size_t)((L + 1) & 1) * P.nb + b;
    if (cin->done) {
      if (first && lane == 0) *cout = *cin;
      return;
    }
    t_in = cin->t;
    T_in = cin->T;
    nstep = cin->nsteps;
    const uint64_t* row = a.acc + ((size_t)(L % 3) * P.nb + b) * kAccRow;
    double ms = 0.0;
    if (lane < kAccSlots) ms = __longlong_as_double((long long)row[lane * kAccStride]);
    ms = wave_max(ms);
    const double rem = T_in - t_in;
    dt = P.cfl / ms;
    if (dt >= rem) {
      dt = rem;
      last = true;
    }
  } else {
    if (a.nsteps_limit && a.dt_index >= a.nsteps_limit[b]) return;
    dt = a.dt[(size_t)b * a.dt_stride + a.dt_index];
  }
  double* snap = nullptr;
  bool unphys = false, no_slot = false;
  if (a.pool && (nstep % a.snap_interval) == 0) {
    const int slot = nstep / a.snap_interval;
    if (slot < a.snap_slots) snap = a.pool + ((size_t)slot * P.nb + b) * 4 * N;
    else no_slot = true;  // snapshot beyond the pool, reported below
  }

  const double hx = 0.5 * dt * P.inv_dx, hy = 0.5 * dt * P.inv_dy, hg = 0.5 * dt * P.g_y;
  const double ax = dt * P.inv_dx, ay = dt * P.inv_dy, dtg = dt * P.g_y;
  const bool need_speed = a.ctl != nullptr || a.acc_out != nullptr;
  double smax = 0.0;

  // Carried from row j - 1 to row j: its upper face state (r, n = v, t = u,
  // p), the flux through its lower face, its conserved values after the x
  // fluxes and its density; and the primitives and raw values of row j with
  // the differences across its lower face.
  FS top{1.0, 0.0, 0.0, 1.0};
  double Gb[4] = {0, 0, 0, 0}, part[4] = {0, 0, 0, 0}, r0 = 0.0;
  W4 wc = row_prims(P, uc, ys - 1);
  D4 da = diff(wc, row_prims(P, qm, ys - 2));

  // Update of row j (flux G through its upper face) and its signal speed.
  auto finish = [&](int j, const double G[4]) {
    double n0 = part[0] - ay * (G[0] - Gb[0]);
    double n1 = part[1] - ay * (G[1] - Gb[1]);
    double n2 = part[2] - ay * (G[2] - Gb[2]);
    double n3 = part[3] - ay * (G[3] - Gb[3]);
    n2 = n2 + dtg * 0.5 * (r0 + n0);
    n3 = n3 + dtg * 0.5 * (Gb[0] + G[0]);
    if (own) {
      double* o = Un + (size_t)j * nx;
      stg(o, col, n0);
      stg(o + N, col, n1);
      stg(o + 2 * N, col, n2);
      stg(o + 3 * N, col, n3);
    }
    if (need_speed) {
      const W4 q = cons_to_prim(P, n0, n1, n2, n3);
      unphys |= unphysical(q);
      const double cs = sqrt_fast(P.gamma * q.p * q.ri);
      const double sx = (fabs(q.u) + cs) * P.inv_dx, sy = (fabs(q.v) + cs) * P.inv_dy;
      const double s = sx > sy ? sx : sy;
      smax = own && s > smax ? s : smax;
    }
  };

  const int jend = ye < ny ? ye : ny - 1;  // the row above the segment, or its last row below the top wall
  auto row = [&](int j) __attribute__((always_inline)) {
    if (j >= ys && j == 0) {
      // the bottom wall's row: the loop starts at row 0 with ghosts below
      da = diff(row_prims(P, un, 0), ghost_bottom(P, row_prims(P, un, 0)));
      wc = row_prims(P, un, 0);
      uc = un;
      un = load_row(P, U, N, 1, col);
    }
    const Raw u2 = load_row(P, U, N, j + 2, col);
    const W4 wn = row_prims(P, un, j + 1);
    const D4 db = diff(wn, wc);
    D4 xb = D4{from_right(wc.r) - wc.r, from_right(wc.u) - wc.u, from_right(wc.v) - wc.v, from_right(wc.p) - wc.p};
    D4 xa = D4{from_left(xb.r), from_left(xb.u), from_left(xb.v), from_left(xb.p)};
    int code;
    const W4 sx = mc4_diff<false>(P, wc, xa.r, xa.u, xa.v, xa.p, xb.r, xb.u, xb.v, xb.p, code);
    W4 sy = mc4_diff<false>(P, wc, da.r, da.u, da.v, da.p, db.r, db.u, db.v, db.p, code);
    if constexpr (BAL) mc_p_balanced_diff<false>(P, wc, da.p, db.p, sy, code);
    const W4 q = predict(P, wc, sx, sy, hx, hy, hg);
    if (j >= ys) {
      const FS bot{q.r - 0.5 * sy.r, q.v - 0.5 * sy.v, q.u - 0.5 * sy.u, q.p - 0.5 * sy.p};
      double G[4];
      if (j == 0) {
        G[0] = 0.0;
        G[1] = 0.0;
        G[2] = wall_pressure(P, bot, false);
        G[3] = 0.0;
      } else {
        double f[4];
        hllc(P, top, bot, f);
        G[0] = f[0];
        G[1] = f[2];
        G[2] = f[1];
        G[3] = f[3];
      }
      if (j > ys) finish(j - 1, G);
      if (j < ye) {
        const FS L{q.r + 0.5 * sx.r, q.u + 0.5 * sx.u, q.v + 0.5 * sx.v, q.p + 0.5 * sx.p};
        const FS R{from_right(q.r - 0.5 * sx.r), from_right(q.u - 0.5 * sx.u), from_right(q.v - 0.5 * sx.v),
                   from_right(q.p - 0.5 * sx.p)};
        double F[4];
        hllc(P, L, R, F);
        part[0] = uc.r - ax * (F[0] - from_left(F[0]));
        part[1] = uc.mx - ax * (F[1] - from_left(F[1]));
        part[2] = uc.my - ax * (F[2] - from_left(F[2]));
        part[3] = uc.E - ax * (F[3] - from_left(F[3]));
        r0 = uc.r;
        if (snap && own) {
          double* o = snap + (size_t)j * nx;
          stg(o, col, uc.r);
          stg(o + N, col, uc.mx);
          stg(o + 2 * N, col, uc.my);
          stg(o + 3 * N, col, uc.E);
        }
        const double hr = 0.5 * fabs(sx.r), hp = 0.5 * fabs(sx.p), vr = 0.5 * fabs(sy.r), vp = 0.5 * fabs(sy.p);
        unphys |= unphysical(wc) | !(q.r - hr > 0.0) | !(q.p - hp > 0.0) | !(q.r - vr > 0.0) | !(q.p - vp > 0.0);
      }
      Gb[0] = G[0];
      Gb[1] = G[1];
      Gb[2] = G[2];
      Gb[3] = G[3];
    }
    top = FS{q.r + 0.5 * sy.r, q.v + 0.5 * sy.v, q.u + 0.5 * sy.u, q.p + 0.5 * sy.p};
    da = db;
    wc = wn;
    uc = un;
    un = u2;
  };
  // two rows per turn, so that what a row hands to the next changes
  // registers by name instead of by moves
  for (int j = ys > 0 ? ys - 1 : 0;;) {
    row(j);
    if (++j > jend) break;
    row(j);
    if (++j > jend) break;
  }
  if (ye == ny) {
    const double G[4] = {0.0, 0.0, wall_pressure(P, top, true), 0.0};
    finish(ny - 1, G);
  }

  if (own && no_slot) atomicOr(&a.flags->snap_overflow, 1);
  if (own && unphys) atomicOr(&a.flags->err_unphys, 1);
  if (!need_speed) return;
  const double bm = wave_max(smax);
  if (a.ctl == nullptr) {
    if (lane == 0) atomicMax((unsigned long long*)(a.acc_out + b), (unsigned long long)__double_as_longlong(bm));
    return;
  }
  const int L = a.launch;
  if (first && lane < kAccSlots) a.acc[((size_t)((L + 2) % 3) * P.nb + b) * kAccRow + lane * kAccStride] = 0ull;
  if (lane != 0) return;
  atomicMax((unsigned long long*)(a.acc + ((size_t)((L + 1) % 3) * P.nb + b) * kAccRow + (t % kAccSlots) * kAccStride),
            (unsigned long long)__double_as_longlong(bm));
  if (!first) return;
  if (a.dt_log) {
    if (nstep < a.dt_log_cap) a.dt_log[(size_t)b * a.dt_log_cap + nstep] = dt;
    else atomicOr(&a.flags->err_overflow, 1);
  }
  Ctl o;
  o.T = T_in;
  o.t = last ? T_in : t_in + dt;
  o.dt_last = dt;
  o.nsteps = nstep + 1;
  o.done = last ? 1 : 0;
  *cout = o;
  if (last) atomicSub(&a.flags->n_active, 1);
}

// Row segments of a launch: k wavefronts per SIMD, k = 1, 2 or 3 (the most
// that fit at their register count), the k with the least of
// c_k (rows per segment + 2.3).  That is the measured time of a launch less
// a constant 3 us: a segment costs its rows and the 2.3 rows' worth below and
// above it, and a row 1.23, 2.10, 3.03 us with 1, 2, 3 wavefronts on a SIMD
// (512x1024 x 4 and x 8 given dt: 51.2 and 95.9 us with one, 46.8 and 85.2
// with two, 46.3 and 83.7 with three; 512x1024: 17.7, 17.1, 16.9).
constexpr int kSimds = 1024;
int row_segments(int ny, int strips, int nb) {
  constexpr double c[3] = {1.23, 2.10, 3.03};
  int best = 1;
  double cost = 1e300;
  for (int k = 1; k <= 3; ++k) {
    const int segs = std::min(ny, std::max(1, (int)((long)k * kSimds / ((long)strips * nb))));
    const double t = c[k - 1] * ((ny + segs - 1) / segs + 2.3);
    if (t < cost) {
      cost = t;
      best = segs;
    }
  }
  return best;
}

}  // namespace

hipError_t launch_step_cols(const Params& P, const StepArgs& a, hipStream_t s) {
  const int strips = (P.nx + kStepOwn - 1) / kStepOwn;
  const int segs = row_segments(P.ny, strips, P.nb);
  const long waves = (long)strips * segs * P.nb;
  const dim3 grid((unsigned)((waves + kColWaves - 1) / kColWaves));
  if (P.recon == 1)
    hipLaunchKernelGGL((k_step_cols<true>), grid, dim3(64 * kColWaves), 0, s, P, a, strips, segs);
  else
    hipLaunchKernelGGL((k_step_cols<false>), grid, dim3(64 * kColWaves), 0, s, P, a, strips, segs);
  return hipGetLastError();
}

}  // namespace rtk
