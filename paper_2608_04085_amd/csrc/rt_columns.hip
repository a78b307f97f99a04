// Column kernels: one wavefront marches a strip of columns upward, one cell
// per lane and one row per iteration, with the rows a stencil needs in
// registers and x neighbours taken from the next lane (a lane shift of the
// whole wavefront).  No barriers; what the tile kernels compute
// again for every tile's halo (primitives 1.58 and predictor 1.28 times per
// cell on 16x15 tiles) is computed once but for the outer lanes of a strip
// (4 of 64) and two rows around a segment.  The expressions are those of the
// tile kernels, so the results are the same to the bit.
//
// k_step_cols is bound by VALU issue: 494 instructions per row and wavefront
// at a given dt (532 in the march), 567 (610) per 64 cells with the lanes
// beside the strips, where the 16x15 tiles take 845 plus their barriers.  Two
// rows per loop turn save 3-6 % (what a row hands to the next changes registers
// by name, not by moves), and 4 % more come from wavefronts that keep pace
// (below).  Tiles against columns, us, of 50 launches in a row: 8 x 1024x2048 529
// -> 309 given dt and 588 -> 334 in the march; 8 x 512x1024 131 -> 78 and 147 ->
// 85; 64 x 128x256 72 -> 52 and 80 -> 58; 1024x2048 69 -> 43 and 77 -> 48 (noisy
// states, which part the lanes' branches, up to 7 % more by columns; under a long
// load the clock falls to 1.8 GHz, 8 x 1024x2048 to 365 and 390).
//
// k_adj_cols is the whole adjoint of a step in one launch: about 940 VALU
// instructions per row and wavefront, and no intermediates in memory (the
// tile pair moves 1294 MiB per launch at 8 x 512x1024, most of it between its
// two kernels).  It is bound by registers and latency: 220 registers per lane
// leave two wavefronts per SIMD, so what a row hands to the next waits in LDS
// (40 doubles per lane), is read again by each phase that needs it, and the
// limiter cases are formed at once (left to the end of the row they keep the
// 8 slopes' differences in registers: 256 and spills, 227 us against 201 at
// 8 x 512x1024; with all of it in registers 398).  The cases travel as binary
// exponents, so that a weight costs one ldexp, and the HLLC adjoint scatters
// its upwind side by exact products (1100 -> 990 instructions, 201 -> 194).
// Two rows per loop turn and even pace: 194 -> 181.  (Reading a phase's LDS
// values a phase ahead is worth nothing.)  Tiles against columns, us: 8 x
// 1024x2048 1512 -> 656, 8 x 512x1024 392 -> 180, 64 x 128x256 190 -> 123,
// 512x1024 45 -> 36.
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
// lane 63 / lane 0 get zero, or with ROT those of lane 0 / lane 63).
template <int CTRL>
__device__ __forceinline__ double lane_move(double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, 0xf, 0xf, true);
  const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xf, 0xf, true);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
template <bool ROT>
__device__ __forceinline__ double lane_right(double v) {
  return lane_move<ROT ? 0x134 : 0x130>(v);  // wave_rol:1, wave_shl:1
}
template <bool ROT>
__device__ __forceinline__ double lane_left(double v) {
  return lane_move<ROT ? 0x13c : 0x138>(v);  // wave_ror:1, wave_shr:1
}

// A row of exactly 64 cells fills a wavefront and is periodic by rotation: no
// columns beside the strip, and one strip where 60 (58) columns each take two.
// 256 x 64x128, us: step 77 -> 43, in the march 89 -> 50, adjoint 160 -> 92; 16
// x 64x128 step 10.0 -> 7.3 (tiles 8.2).
inline bool row_is_wavefront(const Params& P) { return P.nx == 64; }

// A value that is the same in every lane, in scalar registers.
__device__ __forceinline__ double uniform(double v) { return read_lane(v, 0); }

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

// A SIMD issues its oldest wavefront first, so wavefronts with the same work
// end one after the other and the last runs alone, at its own latency (3 per
// SIMD were resident for 66 % of the launch on average, 2 for 78 %).  Priority
// falls with the rows still to come: whoever is ahead fills the others' gaps,
// and they end together.  8 x 512x1024, us: step 102 -> 97, adjoint 200 -> 192.
// Not with one wavefront per SIMD, whose priority would only hold up another
// stream's blocks (32 x 64x128 gradient 9.2 ms, with it 9.4).  One call per two
// rows.
__device__ __forceinline__ void pace(int left, int rows) {
  if (16 * left <= rows) __builtin_amdgcn_s_setprio(0);
  else if (4 * left <= rows) __builtin_amdgcn_s_setprio(1);
  else if (2 * left <= rows) __builtin_amdgcn_s_setprio(2);
  else __builtin_amdgcn_s_setprio(3);
}

struct D4 {
  double r, u, v, p;
};
__device__ __forceinline__ D4 diff(const W4& a, const W4& b) { return D4{a.r - b.r, a.u - b.u, a.v - b.v, a.p - b.p}; }

template <bool BAL, bool ROT>
__global__ __launch_bounds__(64 * kColWaves) void k_step_cols(Params P, StepArgs a, int strips, int segs, int paced) {
  constexpr int halo = ROT ? 0 : kStepHalo;
  auto from_right = [](double v) __attribute__((always_inline)) { return lane_right<ROT>(v); };
  auto from_left = [](double v) __attribute__((always_inline)) { return lane_left<ROT>(v); };
  const int lane = threadIdx.x & 63;
  const int per = strips * segs;
  const int w = __builtin_amdgcn_readfirstlane(xcd_band((int)blockIdx.x, (int)gridDim.x) * kColWaves + (int)(threadIdx.x >> 6));
  if (w >= per * P.nb) return;
  const int b = w / per, t = w - b * per;
  const int seg = t / strips, strip = t - seg * strips;
  const int nx = P.nx, ny = P.ny;
  const size_t N = (size_t)nx * ny;
  const int ys = (int)((long)ny * seg / segs), ye = (int)((long)ny * (seg + 1) / segs);
  const int x0 = strip * (64 - 2 * halo);
  const uint32_t col = (uint32_t)wrapx(x0 - halo + lane, nx);
  const bool own = lane >= halo && lane < 64 - halo && x0 - halo + lane < nx;
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
  const bool need_speed = a.ctl != nullptr || a.speeds != nullptr;
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
    const W4 sx = mc4_diff<false, true>(P, wc, xa.r, xa.u, xa.v, xa.p, xb.r, xb.u, xb.v, xb.p, code);
    W4 sy = mc4_diff<false, true>(P, wc, da.r, da.u, da.v, da.p, db.r, db.u, db.v, db.p, code);
    if constexpr (BAL) mc_p_balanced_diff<false, true>(P, wc, da.p, db.p, sy, code);
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
  const int j0 = ys > 0 ? ys - 1 : 0;
  for (int j = j0;;) {
    if (paced) pace(jend + 1 - j, jend + 1 - j0);
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
    if (lane == 0) a.speeds[w] = bm;  // (b * per + t)
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

// Adjoint of one step.  lambda^n of a cell needs the slope cotangents of the
// cell and its four neighbours, these the cotangents of their faces, these
// the predicted states across the faces: three columns and three rows to
// each side in all.
constexpr int kAdjHalo = 3, kAdjOwn = 64 - 2 * kAdjHalo;

struct Lam {
  double v[4];
};
__device__ __forceinline__ Lam load_lam(const Params& P, const double* Lm, size_t N, int gy, uint32_t col) {
  const int sy = gy < 0 ? 0 : (gy >= P.ny ? P.ny - 1 : gy);
  const double* p = Lm + (size_t)sy * P.nx;
  return Lam{{ldg(p, col), ldg(p + N, col), ldg(p + 2 * N, col), ldg(p + 3 * N, col)}};
}

// What a row hands on through LDS, each lane its own (registers bound the
// wavefronts in flight).  Row k = m - 1: slopes, primitives, lambda^{n+1} and
// the cotangent its lower face gives it.  Row g = m - 2: slope terms so far,
// direct part, forward products of the y slopes and (u, v, 1/rho).
enum { kSx = 0, kSy = 4, kPrim = 8, kLam = 13, kYb = 17, kAcc = 21, kDir = 25, kFwd = 29, kVel = 33, kAdjKept = 36 };

// Between the phases of a row: what the next phase needs from LDS is read
// again there instead of staying in registers.
__device__ __forceinline__ void phase() { asm volatile("" ::: "memory"); }

template <bool BAL, bool ROT>
__global__ __launch_bounds__(64 * kColWaves, 2) void k_adj_cols(Params P, AdjArgs a, int strips, int segs, int paced) {
  __shared__ double sRow[kColWaves][kAdjKept][64];
  __shared__ int sCase[kColWaves][8][64];  // row k's limiter cases, x slopes then y slopes (mc_exponents)
  constexpr int halo = ROT ? 0 : kAdjHalo;
  auto from_right = [](double v) __attribute__((always_inline)) { return lane_right<ROT>(v); };
  auto from_left = [](double v) __attribute__((always_inline)) { return lane_left<ROT>(v); };
  const int lane = threadIdx.x & 63;
  const int per = strips * segs;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int w = xcd_band((int)blockIdx.x, (int)gridDim.x) * kColWaves + wave;
  if (w >= per * P.nb) return;
  const int b = w / per, t = w - b * per;
  const int seg = t / strips, strip = t - seg * strips;
  const int nx = P.nx, ny = P.ny;
  const size_t N = (size_t)nx * ny;
  const int ys = (int)((long)ny * seg / segs), ye = (int)((long)ny * (seg + 1) / segs);
  const int x0 = strip * (64 - 2 * halo);
  const uint32_t col = (uint32_t)wrapx(x0 - halo + lane, nx);
  const bool own = lane >= halo && lane < 64 - halo && x0 - halo + lane < nx;
  const double* U = a.U + (size_t)b * 4 * N;
  const double* Lm = a.lam_next + (size_t)b * 4 * N;
  double* Lo = a.lam + (size_t)b * 4 * N;
  if (a.nsteps_limit && a.dt_index >= a.nsteps_limit[b]) {
    // the member finished before step n: lambda^n = lambda^{n+1}
    for (int j = ys; j < ye; ++j) {
      const Lam l = load_lam(P, Lm, N, j, col);
      if (own) {
        double* o = Lo + (size_t)j * nx;
#pragma unroll
        for (int v = 0; v < 4; ++v) stg(o + v * N, col, l.v[v]);
      }
    }
    return;
  }
  const int m0 = ys >= 2 ? ys - 2 : 0, m1 = ye + 1 < ny ? ye + 1 : ny;
  const Raw qm = load_row(P, U, N, m0 - 1, col);
  const Raw qc = load_row(P, U, N, m0, col);
  Raw un = load_row(P, U, N, m0 + 1, col);
  Lam lm = load_lam(P, Lm, N, m0, col);
  const double dt = uniform(a.dt[(size_t)b * a.dt_stride + a.dt_index]);
  const double hg = uniform(0.5 * dt * P.g_y), hdtg = hg;
  const double hx = uniform(0.5 * dt * P.inv_dx), hy = uniform(0.5 * dt * P.inv_dy);
  const double ax = uniform(dt * P.inv_dx), ay = uniform(dt * P.inv_dy);

  auto kept = [&](int q) __attribute__((always_inline)) -> double& { return sRow[wave][q][lane]; };
  auto keep4 = [&](int q, const W4& w) __attribute__((always_inline)) {
    kept(q) = w.r;
    kept(q + 1) = w.u;
    kept(q + 2) = w.v;
    kept(q + 3) = w.p;
  };
  auto kept4 = [&](int q) __attribute__((always_inline)) {
    return W4{kept(q), kept(q + 1), kept(q + 2), kept(q + 3), 0.0};
  };

  // row m: primitives and the differences across its lower face
  W4 wc = row_prims(P, qc, m0);
  D4 da = diff(wc, row_prims(P, qm, m0 - 1));
  W4 qk{1, 0, 0, 1, 0};  // predicted state of row k
  bool unphys = false;

  // lambda^n of row g from its slope terms (the walls' ghosts last; row 0's
  // backward products wait in its place of lambda^n)
  auto finish = [&](int g, double acc[4]) __attribute__((always_inline)) {
    double* o = Lo + (size_t)g * nx;
    if (g == 0 || g == ny - 1) {
      double gb[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) gb[v] = g == 0 && own ? -ldg(o + v * N, col) : 0.0;
      if (g == ny - 1) {
#pragma unroll
        for (int v = 0; v < 4; ++v) gb[v] += kept(kFwd + v);
      }
      const double sgn = g == 0 ? -1.0 : 1.0;
      acc[0] += gb[0] + sgn * P.g_y * P.dy * gb[3];
      acc[1] += gb[1];
      acc[2] -= gb[2];
      acc[3] += gb[3];
    }
    double ub[4];
    prim_adj(P, W4{1.0, kept(kVel), kept(kVel + 1), 1.0, kept(kVel + 2)}, W4{acc[0], acc[1], acc[2], acc[3]}, ub);
    if (own) {
#pragma unroll
      for (int v = 0; v < 4; ++v) stg(o + v * N, col, kept(kDir + v) + ub[v]);
    }
  };

  auto row = [&](int m) __attribute__((always_inline)) {
    const int k = m - 1;
    const bool complete = m > m0 && k >= ys - 1;
    // the right face of row k
    W4 xl{0, 0, 0, 0, 0}, xr{0, 0, 0, 0, 0};
    if (complete) {
      const double l2 = kept(kLam + 2);
      const double lL[4] = {kept(kLam) + hdtg * l2, kept(kLam + 1), l2, kept(kLam + 3)};
      const double Fb[4] = {ax * (from_right(lL[0]) - lL[0]), ax * (from_right(lL[1]) - lL[1]),
                            ax * (from_right(lL[2]) - lL[2]), ax * (from_right(lL[3]) - lL[3])};
      const W4 sxk = kept4(kSx);
      FS Lb{0, 0, 0, 0}, Rb{0, 0, 0, 0};
      hllc_adj(P, FS{qk.r + 0.5 * sxk.r, qk.u + 0.5 * sxk.u, qk.v + 0.5 * sxk.v, qk.p + 0.5 * sxk.p},
               FS{from_right(qk.r - 0.5 * sxk.r), from_right(qk.u - 0.5 * sxk.u), from_right(qk.v - 0.5 * sxk.v),
                  from_right(qk.p - 0.5 * sxk.p)},
               Fb, Lb, Rb);
      xl = W4{from_left(Rb.r), from_left(Rb.n), from_left(Rb.t), from_left(Rb.p), 0.0};
      xr = W4{Lb.r, Lb.n, Lb.t, Lb.p, 0.0};
    }
    phase();
    // row m's slopes and predicted state
    const W4 wn = row_prims(P, un, m + 1);
    const D4 db = diff(wn, wc);
    const D4 xb = D4{from_right(wc.r) - wc.r, from_right(wc.u) - wc.u, from_right(wc.v) - wc.v, from_right(wc.p) - wc.p};
    const D4 xa = D4{from_left(xb.r), from_left(xb.u), from_left(xb.v), from_left(xb.p)};
    int code, cases[8];
    const W4 sx = mc4_diff<false, true>(P, wc, xa.r, xa.u, xa.v, xa.p, xb.r, xb.u, xb.v, xb.p, code, cases);
    W4 sy = mc4_diff<false, true>(P, wc, da.r, da.u, da.v, da.p, db.r, db.u, db.v, db.p, code, cases + 4);
    if constexpr (BAL) mc_p_balanced_diff<false, true>(P, wc, da.p, db.p, sy, code, cases + 4);
#pragma unroll
    for (int v = 0; v < 8; ++v) asm volatile("" : "+v"(cases[v]));  // here, while the differences are at hand
    const W4 q = predict(P, wc, sx, sy, hx, hy, hg);
    if (m >= ys && m < ye) {
      const double hr = 0.5 * fabs(sx.r), hp = 0.5 * fabs(sx.p), vr = 0.5 * fabs(sy.r), vp = 0.5 * fabs(sy.p);
      unphys |= unphysical(wc) | !(q.r - hr > 0.0) | !(q.p - hp > 0.0) | !(q.r - vr > 0.0) | !(q.p - vp > 0.0);
    }
    phase();
    // the face between rows k and m
    W4 yt{0, 0, 0, 0, 0}, yb{0, 0, 0, 0, 0};  // what it gives rows k and m
    const FS above{q.r - 0.5 * sy.r, q.v - 0.5 * sy.v, q.u - 0.5 * sy.u, q.p - 0.5 * sy.p};
    if (m == 0) {
      FS T{0, 0, 0, 0};
      wall_pressure_adj(P, above, false, ay * lm.v[2], T);
      yb = W4{T.r, T.t, T.n, T.p, 0.0};
    }
    if (m > m0) {
      FS Bb{0, 0, 0, 0}, Tb{0, 0, 0, 0};
      const W4 syk = kept4(kSy);
      const FS below{qk.r + 0.5 * syk.r, qk.v + 0.5 * syk.v, qk.u + 0.5 * syk.u, qk.p + 0.5 * syk.p};
      if (m == ny) {
        wall_pressure_adj(P, below, true, -ay * kept(kLam + 2), Bb);
      } else {
        const double l2 = kept(kLam + 2);
        const double lB[4] = {kept(kLam) + hdtg * l2, kept(kLam + 1), l2, kept(kLam + 3)};
        const double lT[4] = {lm.v[0] + hdtg * lm.v[2], lm.v[1], lm.v[2], lm.v[3]};
        const double g0 = ay * (lT[0] - lB[0]) + hdtg * (lT[3] + lB[3]);
        const double g1 = ay * (lT[1] - lB[1]);
        const double g2 = ay * (lT[2] - lB[2]);
        const double g3 = ay * (lT[3] - lB[3]);
        const double Fb[4] = {g0, g2, g1, g3};
        hllc_adj(P, below, above, Fb, Bb, Tb);
        yb = W4{Tb.r, Tb.t, Tb.n, Tb.p, 0.0};
      }
      yt = W4{Bb.r, Bb.t, Bb.n, Bb.p, 0.0};
    }
    phase();
    // the next row's loads, in flight until its slopes
    const Raw u2 = load_row(P, U, N, m + 2, col);
    const Lam ln = load_lam(P, Lm, N, m + 1, col);
    if (complete) {
      // all that row k's four faces give it
      const W4 ybk = kept4(kYb), sxk = kept4(kSx), syk = kept4(kSy);
      W4 wk = kept4(kPrim);
      wk.ri = kept(kPrim + 4);
      const W4 qx{xl.r + xr.r, xl.u + xr.u, xl.v + xr.v, xl.p + xr.p, 0.0};
      W4 sxb{0.5 * (xr.r - xl.r), 0.5 * (xr.u - xl.u), 0.5 * (xr.v - xl.v), 0.5 * (xr.p - xl.p), 0.0};
      const W4 qb{qx.r + ybk.r + yt.r, qx.u + ybk.u + yt.u, qx.v + ybk.v + yt.v, qx.p + ybk.p + yt.p, 0.0};
      W4 syb{0.5 * (yt.r - ybk.r), 0.5 * (yt.u - ybk.u), 0.5 * (yt.v - ybk.v), 0.5 * (yt.p - ybk.p), 0.0};
      W4 wb{0.0, 0.0, 0.0, 0.0, 0.0};
      predict_adj(P, wk, sxk, syk, hx, hy, qb, wb, sxb, syb);
      double pa[4], pb[4], ya[4], yf[4];
      // (the weights are 0, 1/2 or 2: adding these exact products is what a
      // fused multiply-add of weight and cotangent gives)
      const double sxv[4] = {sxb.r, sxb.u, sxb.v, sxb.p}, syv[4] = {syb.r, syb.u, syb.v, syb.p};
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int cx = sCase[wave][v][lane], cy = sCase[wave][4 + v][lane];
        pa[v] = weighted_a(sxv[v], cx);
        pb[v] = weighted_b(sxv[v], cx);
        ya[v] = weighted_a(syv[v], cy);
        yf[v] = weighted_b(syv[v], cy);
      }
      double acc[4];
      if (k > ys) {
        // row g = k - 1 takes its last term, the backward part of row k
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[v] = kept(kAcc + v) - ya[v];
        finish(k - 1, acc);
      }
      if (k == 0 && ys == 0 && own) {
#pragma unroll
        for (int v = 0; v < 4; ++v) stg(Lo + v * N, col, ya[v]);
      }
      // row k's terms in the order of the gather: the x slopes of its
      // left neighbour, its own, its right neighbour, then its own y
      // slopes and those of the row below
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        double s = from_left(pb[v]);
        s += pa[v] - pb[v];
        s -= from_right(pa[v]);
        s += ya[v] - yf[v];
        acc[v] = s;
      }
      if constexpr (BAL) {
        const int cp = sCase[wave][7][lane];
        acc[0] += P.g_y * P.dy * (1.0 - weighted_a(1.0, cp) - weighted_b(1.0, cp)) * syb.p;
      }
      if (k > 0 && k > ys - 1) {
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[v] += kept(kFwd + v);
      }
      double ud[4];
      prim_adj(P, wk, wb, ud);
      const double l2 = kept(kLam + 2);
      kept(kDir) = ud[0] + kept(kLam) + dt * P.g_y * l2;
      kept(kDir + 1) = ud[1] + kept(kLam + 1);
      kept(kDir + 2) = ud[2] + l2;
      kept(kDir + 3) = ud[3] + kept(kLam + 3);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        kept(kAcc + v) = acc[v];
        kept(kFwd + v) = yf[v];
      }
      kept(kVel) = wk.u;
      kept(kVel + 1) = wk.v;
      kept(kVel + 2) = wk.ri;
    }
    // row m becomes row k
    keep4(kSx, sx);
    keep4(kSy, sy);
    keep4(kPrim, wc);
    kept(kPrim + 4) = wc.ri;
    keep4(kYb, yb);
#pragma unroll
    for (int v = 0; v < 4; ++v) kept(kLam + v) = lm.v[v];
    qk = q;
#pragma unroll
    for (int v = 0; v < 8; ++v) sCase[wave][v][lane] = cases[v];
    wc = wn;
    da = db;
    un = u2;
    lm = ln;
  };
  for (int m = m0;;) {
    if (paced) pace(m1 + 1 - m, m1 + 1 - m0);
    row(m);
    if (++m > m1) break;
    row(m);
    if (++m > m1) break;
  }
  if (ye == ny) {
    double acc[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[v] = kept(kAcc + v);
    finish(ny - 1, acc);
  }
  if (own && unphys) atomicOr(&a.flags->err_unphys, 1);
}

// Row segments of a launch: k wavefronts per SIMD, 1 up to the most that fit
// at the kernel's registers, the k with the least of c_k (rows per segment +
// over).  That is the measured time of a launch in us less a constant 3: a
// row costs c_k with k wavefronts on a SIMD, and a segment `over` rows' worth
// below and above it (a whole column kOverWhole).  Strips of many members may
// be more than fit: each further wavefront of a SIMD then adds `full` per row.
// That many are by the number of strips, so narrow grids get there with the
// lanes beyond their width idle: 5x248 x 1095 members, one segment each, step
// 484 us and adjoint 954 where 16x15 tiles take 155 and 258.  A launch beside
// another one (beside) takes one wavefront per SIMD and leaves the other its
// own.
constexpr int kSimds = 1024;
constexpr double kOverWhole = 1.2;
template <int K>
int row_segments(int ny, int strips, int nb, const double (&c)[K], double full, double over, bool beside,
                 double* us = nullptr) {
  int best = 1;
  double cost = 1e300;
  for (int k = 1; k <= (beside ? 1 : K); ++k) {
    const int segs = std::min(ny, std::max(1, (int)((long)k * kSimds / ((long)strips * nb))));
    const long w = ((long)strips * segs * nb + kSimds - 1) / kSimds;  // wavefronts per SIMD
    const double t = (w <= K ? c[w - 1] : full * (double)w) * ((ny + segs - 1) / segs + (segs > 1 ? over : kOverWhole));
    if (t < cost) {
      cost = t;
      best = segs;
    }
  }
  if (us) *us = cost + 3.0;
  return best;
}
// Step, noisy states, launch included, with one, two and three wavefronts per
// SIMD: 512x1024 19.9, 18.7, 18.6; x 4 members 58.8, 51.6, 52.4; x 8 106, 93.0,
// 91.3; 64 x 128x256 76.2, 67.8, 62.9; 8 x 1024x2048 382, 348, 345.  Beyond: 3x10
// x 39250 402, 5x4 x 28130 137, 3x158 x 5817 878.
constexpr double kStepRow[3] = {1.23, 2.12, 3.03}, kStepFull = 0.92, kStepOver = 2.3;
// Adjoint, the same with one and two: 512x512 25.9, 29.1; 512x1024 39.6, 38.4;
// x 4 118, 99.8; x 8 224, 189; 64 x 128x256 163, 135.  Beyond: 3x10 x 39250 888,
// 5x4 x 28130 299, 3x158 x 5817 1902.
constexpr double kAdjRow[2] = {2.9, 4.6}, kAdjFull = 2.0, kAdjOver = 2.7;

int step_strips(const Params& P) { return row_is_wavefront(P) ? 1 : (P.nx + kStepOwn - 1) / kStepOwn; }
int adj_strips(const Params& P) { return row_is_wavefront(P) ? 1 : (P.nx + kAdjOwn - 1) / kAdjOwn; }

}  // namespace

double step_cols_us(const Params& P) {
  // a little less than the fit's constant below a few rows: 300x300 7.6,
  // 256x512 9.0, 384x512 10.5
  double us;
  (void)row_segments(P.ny, step_strips(P), P.nb, kStepRow, kStepFull, kStepOver, false, &us);
  return us - 0.6;
}

int step_cols_parts(const Params& P) {
  const int strips = step_strips(P);
  return strips * row_segments(P.ny, strips, P.nb, kStepRow, kStepFull, kStepOver, false);
}

hipError_t launch_step_cols(const Params& P, const StepArgs& a, hipStream_t s) {
  if (a.speeds && a.beside) return hipErrorInvalidValue;  // (other segments than step_cols_parts counts)
  const int strips = step_strips(P);
  const int segs = row_segments(P.ny, strips, P.nb, kStepRow, kStepFull, kStepOver, a.beside);
  const long waves = (long)strips * segs * P.nb;
  const int paced = a.beside || waves > kSimds;
  const dim3 grid((unsigned)((waves + kColWaves - 1) / kColWaves));
  const dim3 block(64 * kColWaves);
  const bool rot = row_is_wavefront(P);
  if (P.recon == 1 && rot) hipLaunchKernelGGL((k_step_cols<true, true>), grid, block, 0, s, P, a, strips, segs, paced);
  else if (P.recon == 1) hipLaunchKernelGGL((k_step_cols<true, false>), grid, block, 0, s, P, a, strips, segs, paced);
  else if (rot) hipLaunchKernelGGL((k_step_cols<false, true>), grid, block, 0, s, P, a, strips, segs, paced);
  else hipLaunchKernelGGL((k_step_cols<false, false>), grid, block, 0, s, P, a, strips, segs, paced);
  return hipGetLastError();
}

double adj_cols_us(const Params& P) {
  double us;
  (void)row_segments(P.ny, adj_strips(P), P.nb, kAdjRow, kAdjFull, kAdjOver, false, &us);
  return us;
}

hipError_t launch_adj_cols(const Params& P, const AdjArgs& a, hipStream_t s) {
  if (a.fold.Z != nullptr || a.dtd.mu != nullptr) return hipErrorInvalidValue;
  const int strips = adj_strips(P);
  const int segs = row_segments(P.ny, strips, P.nb, kAdjRow, kAdjFull, kAdjOver, a.beside);
  const long waves = (long)strips * segs * P.nb;
  const int paced = a.beside || waves > kSimds;
  const dim3 grid((unsigned)((waves + kColWaves - 1) / kColWaves));
  const dim3 block(64 * kColWaves);
  const bool rot = row_is_wavefront(P);
  if (P.recon == 1 && rot) hipLaunchKernelGGL((k_adj_cols<true, true>), grid, block, 0, s, P, a, strips, segs, paced);
  else if (P.recon == 1) hipLaunchKernelGGL((k_adj_cols<true, false>), grid, block, 0, s, P, a, strips, segs, paced);
  else if (rot) hipLaunchKernelGGL((k_adj_cols<false, true>), grid, block, 0, s, P, a, strips, segs, paced);
  else hipLaunchKernelGGL((k_adj_cols<false, false>), grid, block, 0, s, P, a, strips, segs, paced);
  return hipGetLastError();
}

}  // namespace rtk
