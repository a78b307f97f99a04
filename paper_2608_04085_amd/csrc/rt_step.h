// The step kernel's tile: LDS helpers shared with the adjoint's tile kernels
// (rt_kernels.hip) and the body of the fused step, which runs as a kernel of
// its own and beside the fused adjoint (rt_fused.hip).
#pragma once
#include "rt_kernels.h"
#include "rt_wave.h"

namespace rtk {

// ----------------------------------------------------------------- LDS tile helpers
// Phase A: primitives of the tile + halo 2.  Returns nonzero on an
// unphysical interior state.  A thread's cells are addressed first and all
// their loads issued before any is used, so the memory latencies of its
// passes overlap instead of adding up; halo rows beyond the wall ghosts load
// a clamped in-range cell that is never used.
template <int TX, int TY, int NT, class LDS>
__device__ int tile_prims(const Params& P, const double* U, size_t N, int x0, int y0, LDS& S) {
  constexpr int AX = TX + 4, AY = TY + 4, IT = (AX * AY + NT - 1) / NT;
  int bad = 0;
  uint32_t c[IT];
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int k = (int)threadIdx.x + it * NT;
    const int kk = k < AX * AY ? k : AX * AY - 1;
    const int lx = kk % AX, ly = kk / AX;
    const int gx = wrapx(x0 - 2 + lx, P.nx);
    const int gy = y0 - 2 + ly;
    const int sy = gy < 0 ? 0 : (gy >= P.ny ? P.ny - 1 : gy);
    c[it] = (uint32_t)(sy * P.nx + gx);
  }
  double r[IT], mx[IT], my[IT], E[IT];
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    r[it] = ldg(U, c[it]);
    mx[it] = ldg(U + N, c[it]);
    my[it] = ldg(U + 2 * N, c[it]);
    E[it] = ldg(U + 3 * N, c[it]);
  }
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int k = (int)threadIdx.x + it * NT;
    if (k >= AX * AY) break;
    const int lx = k % AX, ly = k / AX;
    const int gy = y0 - 2 + ly;
    W4 w{1.0, 0.0, 0.0, 1.0, 1.0};
    if (gy >= -1 && gy <= P.ny) {
      w = cons_to_prim(P, r[it], mx[it], my[it], E[it]);
      if (gy >= 0 && gy < P.ny) bad |= unphysical(w);
      if (gy < 0) w = ghost_bottom(P, w);
      else if (gy >= P.ny) w = ghost_top(P, w);
    }
    S.W[0][ly][lx] = w.r;
    S.W[1][ly][lx] = w.u;
    S.W[2][ly][lx] = w.v;
    S.W[3][ly][lx] = w.p;
    S.W[4][ly][lx] = w.ri;
  }
  return bad;
}

template <class LDS>
__device__ __forceinline__ W4 ldW(const LDS& S, int x, int y) {
  return W4{S.W[0][y][x], S.W[1][y][x], S.W[2][y][x], S.W[3][y][x], S.W[4][y][x]};
}
template <class LDS>
__device__ __forceinline__ W4 ldQ(const LDS& S, int k, int x, int y) {
  return W4{S.Q[4 * k + 0][y][x], S.Q[4 * k + 1][y][x], S.Q[4 * k + 2][y][x], S.Q[4 * k + 3][y][x], 0.0};
}

// Phase B: slopes and predictor on the cross-shaped halo-1 region.  BAL:
// the well-balanced pressure slopes in y (mc_p_balanced).  CODES: the MC
// cases of the tile cells go to codes_out.
//
// One position k of the halo-1 region, computed without branches: a corner,
// a row outside the domain or an index past the region is computed from
// in-range LDS values (k clamped) and reported as not valid, so the caller
// stores nothing for it.
template <int TX, int TY, bool BAL, bool CODES, class LDS>
__device__ __forceinline__ bool predict_at(const Params& P, const LDS& S, int k, int y0, double hx, double hy,
                                           double hg, W4& q, W4& sx, W4& sy, int& cx, int& cy) {
  constexpr int QX = TX + 2, QY = TY + 2;
  const int kc = k < QX * QY ? k : QX * QY - 1;
  const int lx = kc % QX, ly = kc / QX;
  const int gy = y0 - 1 + ly;
  const bool valid = k < QX * QY && !((lx == 0 || lx == QX - 1) && (ly == 0 || ly == QY - 1)) && gy >= 0 &&
                     gy < P.ny;
  const W4 wc = ldW(S, lx + 1, ly + 1);
  sx = mc4<CODES>(P, ldW(S, lx, ly + 1), wc, ldW(S, lx + 2, ly + 1), cx);
  sy = mc4<CODES>(P, ldW(S, lx + 1, ly), wc, ldW(S, lx + 1, ly + 2), cy);
  if constexpr (BAL) mc_p_balanced<CODES>(P, ldW(S, lx + 1, ly), wc, ldW(S, lx + 1, ly + 2), sy, cy);
  q = predict(P, wc, sx, sy, hx, hy, hg);
  return valid;
}

// Stores one position's predicted state and slopes (and its MC cases for a
// tile cell); returns nonzero if a face state would be unphysical.
template <int TX, int TY, bool CODES, class LDS>
__device__ __forceinline__ int predict_store(const Params& P, LDS& S, int k, int x0, int y0, const W4& q,
                                             const W4& sx, const W4& sy, int cx, int cy, int32_t* codes_out) {
  constexpr int QX = TX + 2;
  const int lx = k % QX, ly = k / QX;
  S.Q[0][ly][lx] = q.r;
  S.Q[1][ly][lx] = q.u;
  S.Q[2][ly][lx] = q.v;
  S.Q[3][ly][lx] = q.p;
  S.Q[4][ly][lx] = sx.r;
  S.Q[5][ly][lx] = sx.u;
  S.Q[6][ly][lx] = sx.v;
  S.Q[7][ly][lx] = sx.p;
  S.Q[8][ly][lx] = sy.r;
  S.Q[9][ly][lx] = sy.u;
  S.Q[10][ly][lx] = sy.v;
  S.Q[11][ly][lx] = sy.p;
  if constexpr (CODES) {
    if (lx >= 1 && lx <= TX && ly >= 1 && ly <= TY) {
      const int gx = x0 - 1 + lx;
      if (gx < P.nx) stg(codes_out, (uint32_t)((y0 - 1 + ly) * P.nx + gx), cx | (cy << 8));
    }
  }
  const double hr = 0.5 * fabs(sx.r), hp = 0.5 * fabs(sx.p), vr = 0.5 * fabs(sy.r), vp = 0.5 * fabs(sy.p);
  return !(q.r - hr > 0.0) || !(q.p - hp > 0.0) || !(q.r - vr > 0.0) || !(q.p - vp > 0.0);
}

// The region has more positions than the block has threads for the 256-
// thread tiles, so some wavefronts take two.  With PAIR those compute both
// positions in one branch-free stretch (their instruction streams
// interleave and hide each other's latency) instead of one after the
// other; whether a wavefront has a second position is uniform across it.
// PAIR costs registers: the step kernel has them to spare, the adjoint
// kernel would drop to two wavefronts per SIMD.
//
// ALIAS: the predicted states overwrite the primitive tile they are computed
// from (one LDS region serves both): every thread computes its positions
// (two at most) into registers, the block waits until all have read the
// primitives, then the results are stored.
template <int TX, int TY, int NT, bool BAL, bool CODES, bool PAIR, bool ALIAS = false, class LDS>
__device__ int tile_predict(const Params& P, double dt, int x0, int y0, LDS& S, int32_t* codes_out) {
  constexpr int QN = (TX + 2) * (TY + 2);
  const double hx = 0.5 * dt * P.inv_dx, hy = 0.5 * dt * P.inv_dy, hg = 0.5 * dt * P.g_y;
  int bad = 0;
  if constexpr (ALIAS) {
    static_assert(PAIR && !CODES && QN <= 2 * NT, "one pass of at most two positions per thread");
    const int k = threadIdx.x;
    const int wave_first = k - (int)(threadIdx.x & 63);
    W4 q, sx, sy, q2 = W4{}, sx2 = W4{}, sy2 = W4{};
    int cx = 0, cy = 0, cx2 = 0, cy2 = 0;
    const bool v1 = predict_at<TX, TY, BAL, CODES>(P, S, k, y0, hx, hy, hg, q, sx, sy, cx, cy);
    bool v2 = false;
    if (wave_first + NT < QN) v2 = predict_at<TX, TY, BAL, CODES>(P, S, k + NT, y0, hx, hy, hg, q2, sx2, sy2, cx2, cy2);
    __syncthreads();  // the primitives are read: their space takes the predicted states
    if (v1) bad |= predict_store<TX, TY, CODES>(P, S, k, x0, y0, q, sx, sy, cx, cy, codes_out);
    if (v2) bad |= predict_store<TX, TY, CODES>(P, S, k + NT, x0, y0, q2, sx2, sy2, cx2, cy2, codes_out);
    return bad;
  }
  for (int k = threadIdx.x; k < QN; k += (PAIR ? 2 : 1) * NT) {
    const int wave_first = k - (int)(threadIdx.x & 63);
    W4 q, sx, sy;
    int cx = 0, cy = 0;
    if (PAIR && wave_first + NT < QN) {
      W4 q2, sx2, sy2;
      int cx2 = 0, cy2 = 0;
      const bool v1 = predict_at<TX, TY, BAL, CODES>(P, S, k, y0, hx, hy, hg, q, sx, sy, cx, cy);
      const bool v2 = predict_at<TX, TY, BAL, CODES>(P, S, k + NT, y0, hx, hy, hg, q2, sx2, sy2, cx2, cy2);
      if (v1) bad |= predict_store<TX, TY, CODES>(P, S, k, x0, y0, q, sx, sy, cx, cy, codes_out);
      if (v2) bad |= predict_store<TX, TY, CODES>(P, S, k + NT, x0, y0, q2, sx2, sy2, cx2, cy2, codes_out);
    } else {
      if (predict_at<TX, TY, BAL, CODES>(P, S, k, y0, hx, hy, hg, q, sx, sy, cx, cy))
        bad |= predict_store<TX, TY, CODES>(P, S, k, x0, y0, q, sx, sy, cx, cy, codes_out);
    }
  }
  return bad;
}

// Face states from the predictor region: x faces in (r, n = u, t = v, p),
// y faces in (r, n = v, t = u, p).
template <class LDS>
__device__ __forceinline__ FS xface_right_of(const LDS& S, int x, int y) {  // state at the cell's right face
  return FS{S.Q[0][y][x] + 0.5 * S.Q[4][y][x], S.Q[1][y][x] + 0.5 * S.Q[5][y][x], S.Q[2][y][x] + 0.5 * S.Q[6][y][x],
            S.Q[3][y][x] + 0.5 * S.Q[7][y][x]};
}
template <class LDS>
__device__ __forceinline__ FS xface_left_of(const LDS& S, int x, int y) {
  return FS{S.Q[0][y][x] - 0.5 * S.Q[4][y][x], S.Q[1][y][x] - 0.5 * S.Q[5][y][x], S.Q[2][y][x] - 0.5 * S.Q[6][y][x],
            S.Q[3][y][x] - 0.5 * S.Q[7][y][x]};
}
template <class LDS>
__device__ __forceinline__ FS yface_top_of(const LDS& S, int x, int y) {
  return FS{S.Q[0][y][x] + 0.5 * S.Q[8][y][x], S.Q[2][y][x] + 0.5 * S.Q[10][y][x], S.Q[1][y][x] + 0.5 * S.Q[9][y][x],
            S.Q[3][y][x] + 0.5 * S.Q[11][y][x]};
}
template <class LDS>
__device__ __forceinline__ FS yface_bottom_of(const LDS& S, int x, int y) {
  return FS{S.Q[0][y][x] - 0.5 * S.Q[8][y][x], S.Q[2][y][x] - 0.5 * S.Q[10][y][x], S.Q[1][y][x] - 0.5 * S.Q[9][y][x],
            S.Q[3][y][x] - 0.5 * S.Q[11][y][x]};
}

// Phase C's face items: k < NXF are the x faces (TX + 1 per tile row, TY
// rows), the next NYF the y faces (TX per face row, TY + 1 rows), with no
// gap, so a wavefront may hold both kinds.  Both kinds run one instruction
// stream: the face's two predicted states are read through per-lane LDS
// offsets (which planes hold the normal and the tangential velocity and
// their slopes, and whether the right state is the next column or the next
// row), and the flux comes back in face-normal order.  Only y faces on a
// wall branch off.
template <int TX, int TY>
struct FaceItems {
  static constexpr int QX = TX + 2, PS = (TX + 2) * (TY + 2);
  static constexpr int NXF = (TX + 1) * TY, NYF = TX * (TY + 1), N = NXF + NYF;
};

// Flux of face item k in face-normal order; returns 1 for an x face, 2 for a
// y face, 0 past the items or for a face outside the domain.  Every lane
// runs the same instructions (an item past the end reads the last item's
// states, a face outside the domain reads whatever its rows hold, and a
// wall face's HLLC result is replaced), so a wavefront never takes two
// paths except for the wall faces of the first and last tile rows.
template <int TX, int TY, class LDS>
__device__ __forceinline__ int step_face_flux(const Params& P, const LDS& S, int k, int y0, double f[4]) {
  using FI = FaceItems<TX, TY>;
  const int kc = k < FI::N ? k : FI::N - 1;
  const bool xf = kc < FI::NXF;
  const int kk = kc - FI::NXF;
  const int fy = xf ? kc / (TX + 1) : kk / TX;
  const int fx = xf ? kc - (kc / (TX + 1)) * (TX + 1) : kk % TX;
  const int j = y0 + fy;
  // left state: the right face of cell (fx, fy + 1) or the top face of
  // cell (fx + 1, fy) of the predictor region; right state one column or
  // one row further
  const int l = xf ? (fy + 1) * FI::QX + fx : fy * FI::QX + fx + 1;
  const int r = l + (xf ? 1 : FI::QX);
  const int pn = xf ? FI::PS : 2 * FI::PS, pt = xf ? 2 * FI::PS : FI::PS;  // velocity planes
  const int sb = xf ? 4 * FI::PS : 8 * FI::PS;                             // slope planes
  const double* q = &S.Q[0][0][0];
  const FS L{q[l] + 0.5 * q[sb + l], q[pn + l] + 0.5 * q[sb + pn + l], q[pt + l] + 0.5 * q[sb + pt + l],
             q[3 * FI::PS + l] + 0.5 * q[sb + 3 * FI::PS + l]};
  const FS R{q[r] - 0.5 * q[sb + r], q[pn + r] - 0.5 * q[sb + pn + r], q[pt + r] - 0.5 * q[sb + pt + r],
             q[3 * FI::PS + r] - 0.5 * q[sb + 3 * FI::PS + r]};
  hllc(P, L, R, f);
  if (!xf && (j == 0 || j == P.ny)) {
    f[1] = j == 0 ? wall_pressure(P, R, false) : wall_pressure(P, L, true);
    f[0] = 0.0;
    f[2] = 0.0;
    f[3] = 0.0;
  }
  const bool inside = k < FI::N && (xf ? j < P.ny : j <= P.ny);
  return inside ? (xf ? 1 : 2) : 0;
}

// Stores the flux of face item k (kind from step_face_flux) into F or G.
template <int TX, int TY, class LDS>
__device__ __forceinline__ void step_face_store(LDS& S, int k, int kind, const double f[4]) {
  using FI = FaceItems<TX, TY>;
  if (kind == 1) {
    const int fx = k % (TX + 1), fy = k / (TX + 1);
    S.fg.F[0][fy][fx] = f[0];
    S.fg.F[1][fy][fx] = f[1];
    S.fg.F[2][fy][fx] = f[2];
    S.fg.F[3][fy][fx] = f[3];
  } else if (kind == 2) {
    const int kk = k - FI::NXF, fx = kk % TX, fy = kk / TX;
    S.fg.G[0][fy][fx] = f[0];
    S.fg.G[1][fy][fx] = f[2];
    S.fg.G[2][fy][fx] = f[1];
    S.fg.G[3][fy][fx] = f[3];
  }
}

// ----------------------------------------------------------------- step
// LDS of the step kernel: the flux arrays reuse the primitive tile, which is
// dead once the predictor has run.
template <int TX, int TY, bool ALIAS = false>
struct StepLDS {
  static constexpr int AX = TX + 4, AY = TY + 4;
  static constexpr int QX = TX + 2, QY = TY + 2;
  union {
    double W[5][AY][AX];  // rho, u, v, p, 1/rho
    struct {
      double F[4][TY][TX + 1];
      double G[4][TY + 1][TX];
    } fg;
  };
  double Q[12][QY][QX];
};
// ALIAS: one region by phase (primitives, then predicted states and slopes,
// then fluxes), for a fourth resident block per CU on large grids.
template <int TX, int TY>
struct StepLDS<TX, TY, true> {
  static constexpr int AX = TX + 4, AY = TY + 4;
  static constexpr int QX = TX + 2, QY = TY + 2;
  union {
    double W[5][AY][AX];
    double Q[12][QY][QX];
    struct {
      double F[4][TY][TX + 1];
      double G[4][TY + 1][TX];
    } fg;
  };
};

// One tile (tbx, tby) of member b.
template <int TX, int TY, int NT, bool BAL, bool ALIAS>
__device__ __forceinline__ void step_tile_body(const Params& P, const StepArgs& a, StepLDS<TX, TY, ALIAS>& S,
                                               double* sRed, int b, int tbx, int tby) {
  static_assert(NT >= TX * TY && NT % 64 == 0, "one thread per tile cell at least");
  const int x0 = tbx * TX, y0 = tby * TY;
  const int tid = threadIdx.x;
  const int nx = P.nx, ny = P.ny;
  const size_t N = (size_t)nx * ny;
  const double* U = a.U + (size_t)b * 4 * N;
  const bool first_block = blockIdx.x == 0 && blockIdx.y == 0;

  // time step of this member.  In the march the control record and the
  // signal-speed slots are loaded here but used only after phase A, which
  // does not depend on them, so their latency overlaps it.
  double dt = 0.0;
  int nstep = 0;
  bool last = false;
  const Ctl* cin = nullptr;
  Ctl* cout = nullptr;
  int done = 0;
  double t_in = 0.0, T_in = 0.0, ms_lane = 0.0;
  if (a.ctl) {
    const int L = a.launch;
    cin = a.ctl + (size_t)(L & 1) * P.nb + b;
    cout = a.ctl + (size_t)((L + 1) & 1) * P.nb + b;
    done = cin->done;
    t_in = cin->t;
    T_in = cin->T;
    nstep = cin->nsteps;
    // a few slots per lane; the max across the wave is taken after phase A
    const uint64_t* row = a.acc + ((size_t)(L % 3) * P.nb + b) * kAccRow;
    const int lane = tid & 63;
#pragma unroll
    for (int k = lane; k < kAccSlots; k += 64)
      ms_lane = fmax(ms_lane, __longlong_as_double((long long)row[k * kAccStride]));
  } else {
    if (a.nsteps_limit && a.dt_index >= a.nsteps_limit[b]) return;
    dt = a.dt[(size_t)b * a.dt_stride + a.dt_index];
  }

  // prefetch this thread's own cell for the update
  const int tx = tid % TX, ty = tid / TX;
  const int gx = x0 + tx, gy = y0 + ty;
  const bool own = tid < TX * TY && gx < nx && gy < ny;
  const uint32_t c = own ? (uint32_t)(gy * nx + gx) : 0u;
  double u0 = 0.0, u1 = 0.0, u2 = 0.0, u3 = 0.0;
  if (own) {
    u0 = ldg(U, c);
    u1 = ldg(U + N, c);
    u2 = ldg(U + 2 * N, c);
    u3 = ldg(U + 3 * N, c);
  }

  // phase A: primitives of the tile + halo 2
  int bad = tile_prims<TX, TY, NT>(P, U, N, x0, y0, S);
  if (a.ctl) {
    // the same member for the whole block, so the return is uniform
    if (done) {
      if (first_block && tid == 0) *cout = *cin;
      return;
    }
    const double ms = wave_max(ms_lane);
    const double rem = T_in - t_in;
    dt = P.cfl / ms;
    if (dt >= rem) {
      dt = rem;
      last = true;
    }
  }
  __syncthreads();

  // phase B: slopes and predictor on the cross-shaped halo-1 region
  bad |= tile_predict<TX, TY, NT, BAL, false, true, ALIAS>(P, dt, x0, y0, S, nullptr);
  __syncthreads();

  // phase C: every face of the tile once
  constexpr int NF = FaceItems<TX, TY>::N;
  if constexpr (ALIAS) {
    // the fluxes overwrite the predicted states: all faces of this thread
    // first, then the stores once every thread has read its states
    constexpr int FMAX = (NF + NT - 1) / NT;
    double fl[FMAX][4];
    int kind[FMAX];
#pragma unroll
    for (int it = 0; it < FMAX; ++it) {
      kind[it] = 0;
      if ((tid & ~63) + it * NT < NF) kind[it] = step_face_flux<TX, TY>(P, S, tid + it * NT, y0, fl[it]);
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < FMAX; ++it) step_face_store<TX, TY>(S, tid + it * NT, kind[it], fl[it]);
  } else {
    for (int k = tid; (k & ~63) < NF; k += NT) {
      double f[4];
      const int kind = step_face_flux<TX, TY>(P, S, k, y0, f);
      step_face_store<TX, TY>(S, k, kind, f);
    }
  }
  __syncthreads();

  // phase D: update with the gravity source
  const bool need_speed = a.ctl != nullptr || a.speeds != nullptr;
  double smax = 0.0;
  if (own) {
    const double ax = dt * P.inv_dx, ay = dt * P.inv_dy;
    double n0 = u0 - ax * (S.fg.F[0][ty][tx + 1] - S.fg.F[0][ty][tx]) - ay * (S.fg.G[0][ty + 1][tx] - S.fg.G[0][ty][tx]);
    double n1 = u1 - ax * (S.fg.F[1][ty][tx + 1] - S.fg.F[1][ty][tx]) - ay * (S.fg.G[1][ty + 1][tx] - S.fg.G[1][ty][tx]);
    double n2 = u2 - ax * (S.fg.F[2][ty][tx + 1] - S.fg.F[2][ty][tx]) - ay * (S.fg.G[2][ty + 1][tx] - S.fg.G[2][ty][tx]);
    double n3 = u3 - ax * (S.fg.F[3][ty][tx + 1] - S.fg.F[3][ty][tx]) - ay * (S.fg.G[3][ty + 1][tx] - S.fg.G[3][ty][tx]);
    const double dtg = dt * P.g_y;
    n2 = n2 + dtg * 0.5 * (u0 + n0);
    n3 = n3 + dtg * 0.5 * (S.fg.G[0][ty][tx] + S.fg.G[0][ty + 1][tx]);
    double* Un = a.Un + (size_t)b * 4 * N;
    stg(Un, c, n0);
    stg(Un + N, c, n1);
    stg(Un + 2 * N, c, n2);
    stg(Un + 3 * N, c, n3);
    if (a.pool && (nstep % a.snap_interval) == 0) {
      const int slot = nstep / a.snap_interval;
      if (slot < a.snap_slots) {
        double* sp = a.pool + ((size_t)slot * P.nb + b) * 4 * N;
        stg(sp, c, u0);
        stg(sp + N, c, u1);
        stg(sp + 2 * N, c, u2);
        stg(sp + 3 * N, c, u3);
      } else {
        bad |= 4;  // snapshot beyond the pool, reported below
      }
    }
    if (need_speed) {
      const W4 w = cons_to_prim(P, n0, n1, n2, n3);
      bad |= unphysical(w);
      const double cs = sqrt_fast(P.gamma * w.p * w.ri);
      const double sx = (fabs(w.u) + cs) * P.inv_dx, sy = (fabs(w.v) + cs) * P.inv_dy;
      smax = sx > sy ? sx : sy;
    }
  }
  if (bad & 4) atomicOr(&a.flags->snap_overflow, 1);
  if (bad & 1) atomicOr(&a.flags->err_unphys, 1);
  if (!need_speed) return;

  // epilogue: the block's largest signal speed of U^{n+1}; in the march
  // folded into the member's accumulator (non-negative doubles order like
  // their bits)
  const double bm = block_max<NT>(smax, sRed);
  if (a.ctl == nullptr) {
    if (tid == 0) a.speeds[((size_t)b * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x] = bm;
    return;
  }
  const int L = a.launch;
  if (first_block) {
    // clear the slots of launch L + 1's target, one per thread
    uint64_t* clr = a.acc + ((size_t)((L + 2) % 3) * P.nb + b) * kAccRow;
    for (int k = tid; k < kAccSlots; k += NT) clr[k * kAccStride] = 0ull;
  }
  if (tid != 0) return;
  const int slot = (int)((blockIdx.x + (size_t)gridDim.x * blockIdx.y) % kAccSlots);
  atomicMax((unsigned long long*)(a.acc + ((size_t)((L + 1) % 3) * P.nb + b) * kAccRow + slot * kAccStride),
            (unsigned long long)__double_as_longlong(bm));
  if (!first_block) return;
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

}  // namespace rtk
