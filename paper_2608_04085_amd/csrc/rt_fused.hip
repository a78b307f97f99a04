// Adjoint of one step in one launch: kernels A and B of the tile pair on one
// tile, with the tile's halo wide enough (three cells of primitives, two of
// predicted states, one of slope cotangents) that nothing has to go through
// memory.  For grids that a few rounds of blocks cover, where a launch
// lasts as long as its blocks' chains of loads, barriers and arithmetic:
// one launch instead of two, every phase one pass of the block, and a cell's
// two faces of its own in one phase.  The expressions are those of the other
// adjoint kernels, so the results are the same to the bit.  Tile pair (or, in
// parentheses, the folded sweep) against this kernel, us: 64x128 9.3 (7.4) ->
// 6.5, 128x256 11.0 (9.4) -> 6.9, 256x256 13.8 -> 9.1, 256x512 18.2 -> 11.6,
// 512x512 28.0 -> 22.0.
#include <hip/hip_runtime.h>

#include "rt_kernels.h"
#include "rt_step.h"
#include "rt_wave.h"

namespace rtk {

namespace {

template <int TX, int TY>
struct FusedLDS {
  static constexpr int PX = TX + 6, PY = TY + 6;  // primitives
  static constexpr int QX = TX + 4, QY = TY + 4;  // predicted states, slopes, lambda^{n+1}
  static constexpr int ZX = TX + 2, ZY = TY + 2;  // face cotangents, then slope cotangents
  union {
    double W[5][PY][PX];
    // cell (x, y): first the cotangents its left and its bottom face give it,
    // then, in the same place, those of its x and y slopes
    struct {
      double X[4][ZY][ZX];
      double Y[4][ZY][ZX];
    } z;
  };
  double Q[12][QY][QX];
  double L[4][QY][QX];
  int32_t C[QY][QX];  // limiter cases, x slopes then y slopes
};

// One tile (tbx, tby) of member b.
template <int TX, int TY, int NT, bool DTD, bool BAL>
__device__ __forceinline__ void adj_tile_body(const Params& P, const AdjArgs& a, FusedLDS<TX, TY>& S, int b, int tbx,
                                              int tby) {
  using LDS = FusedLDS<TX, TY>;
  constexpr int PX = LDS::PX, PY = LDS::PY, QX = LDS::QX, QY = LDS::QY, ZX = LDS::ZX, ZY = LDS::ZY;
  constexpr int EX = ZX > ZY ? ZX : ZY;  // threads beside the cells': first faces of rows and columns
  static_assert(NT >= ZX * ZY + EX && NT >= PX * PY && NT % 64 == 0, "one pass per phase");
  const int x0 = tbx * TX, y0 = tby * TY;
  const int tid = threadIdx.x;
  const int nx = P.nx, ny = P.ny;
  const size_t N = (size_t)nx * ny;
  const double* U = a.U + (size_t)b * 4 * N;
  const double* Lm = a.lam_next + (size_t)b * 4 * N;
  double* Lo = a.lam + (size_t)b * 4 * N;

  // this thread's cell (the tile and one cell around it, no corners)
  const int zx = tid % ZX, zy = tid / ZX;
  const bool in_z = tid < ZX * ZY;
  const bool corner = (zx == 0 || zx == ZX - 1) && (zy == 0 || zy == ZY - 1);
  const int gx = x0 - 1 + zx, gy = y0 - 1 + zy;
  const bool cell = in_z && !corner && gy >= 0 && gy < ny;
  const bool own = cell && zx >= 1 && zx <= TX && zy >= 1 && zy <= TY && gx < nx;
  const uint32_t c = cell ? (uint32_t)(gy * nx + wrapx(gx, nx)) : 0u;
  if (a.nsteps_limit && a.dt_index >= a.nsteps_limit[b]) {
    // the member finished before step n: lambda^n = lambda^{n+1}
    if (own) {
#pragma unroll
      for (int v = 0; v < 4; ++v) stg(Lo + v * N, c, ldg(Lm + v * N, c));
    }
    return;
  }
  const double dt = a.dt[(size_t)b * a.dt_stride + a.dt_index];
  const double hdtg = 0.5 * dt * P.g_y;
  int bad = 0;
  // DTD: step n + 1's sum of mu and its cell of largest speed, as
  // launch_dt_correct forms them (its 256 threads are this block's first), in
  // the shadow of the loads below: 3 x 127x130 gradient 2.61 -> 2.28 ms
  __shared__ double cm[4], cs[4];
  __shared__ int ci[4], ct[4];
  bool corrects = false;
  if constexpr (DTD) {
    corrects = a.dtd.before.mu != nullptr && a.dt_index + 1 < a.nsteps_limit[b];
    if (corrects && tid < 256) {
      const size_t o = (size_t)b * a.dtd.stride;
      double m = 0.0, sp = -1.0;
      int ix = 0x7fffffff, tile = 0;
      auto merge = [&](double s2, int i2, int t2) {
        if (s2 > sp || (s2 == sp && i2 < ix)) {
          sp = s2;
          ix = i2;
          tile = t2;
        }
      };
      for (int k = tid; k < a.dtd.count; k += 256) {
        m += a.dtd.before.mu[o + k];
        merge(a.dtd.before.smax[o + k], a.dtd.before.imax[o + k], k);
      }
      m = wave_sum(m);
#pragma unroll
      for (int d = 32; d > 0; d >>= 1) merge(__shfl_xor(sp, d, 64), __shfl_xor(ix, d, 64), __shfl_xor(tile, d, 64));
      if ((tid & 63) == 0) {
        cm[tid >> 6] = m;
        cs[tid >> 6] = sp;
        ci[tid >> 6] = ix;
        ct[tid >> 6] = tile;
      }
    }
  }

  // primitives of the tile + 3 and lambda^{n+1} of the tile + 2
  {
    constexpr int IT = (PX * PY + NT - 1) / NT;
    double r[IT], mx[IT], my[IT], E[IT];
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int k = tid + it * NT, kk = k < PX * PY ? k : PX * PY - 1;
      const int j = y0 - 3 + kk / PX, sy = j < 0 ? 0 : (j >= ny ? ny - 1 : j);
      const uint32_t o = (uint32_t)(sy * nx + wrapx(x0 - 3 + kk % PX, nx));
      r[it] = ldg(U, o);
      mx[it] = ldg(U + N, o);
      my[it] = ldg(U + 2 * N, o);
      E[it] = ldg(U + 3 * N, o);
    }
    constexpr int IL = (QX * QY + NT - 1) / NT;
    double l[IL][4];
#pragma unroll
    for (int it = 0; it < IL; ++it) {
      const int k = tid + it * NT, kk = k < QX * QY ? k : QX * QY - 1;
      const int j = y0 - 2 + kk / QX, sy = j < 0 ? 0 : (j >= ny ? ny - 1 : j);
      const uint32_t o = (uint32_t)(sy * nx + wrapx(x0 - 2 + kk % QX, nx));
#pragma unroll
      for (int v = 0; v < 4; ++v) l[it][v] = ldg(Lm + v * N, o);
    }
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int k = tid + it * NT;
      if (k >= PX * PY) break;
      const int lx = k % PX, ly = k / PX, j = y0 - 3 + ly;
      W4 w{1.0, 0.0, 0.0, 1.0, 1.0};
      if (j >= -1 && j <= ny) {
        w = cons_to_prim(P, r[it], mx[it], my[it], E[it]);
        if (j >= 0 && j < ny) bad |= unphysical(w);
        if (j < 0) w = ghost_bottom(P, w);
        else if (j >= ny) w = ghost_top(P, w);
      }
      S.W[0][ly][lx] = w.r;
      S.W[1][ly][lx] = w.u;
      S.W[2][ly][lx] = w.v;
      S.W[3][ly][lx] = w.p;
      S.W[4][ly][lx] = w.ri;
    }
#pragma unroll
    for (int it = 0; it < IL; ++it) {
      const int k = tid + it * NT;
      if (k >= QX * QY) break;
#pragma unroll
      for (int v = 0; v < 4; ++v) S.L[v][k / QX][k % QX] = l[it][v];
    }
  }
  __syncthreads();
  if constexpr (DTD) {
    if (corrects) {
      // wherever this tile holds the cell (its lambda is read after the next
      // barrier)
      int w = 0;
#pragma unroll
      for (int k = 1; k < 4; ++k)
        if (cs[k] > cs[w] || (cs[k] == cs[w] && ci[k] < ci[w])) w = k;
      const int ix = ci[w];
      const double m = ((cm[0] + cm[1]) + cm[2]) + cm[3];
      const bool last = a.dt_index + 2 == a.nsteps_limit[b];  // step n + 1 was the member's last: its mu is kept
      if (last && tid == 0 && tbx == 0 && tby == 0) a.dtd.mu_last[b] = m;
      for (int k = tid; k < QX * QY; k += NT) {
        const int j = y0 - 2 + k / QX, sy = j < 0 ? 0 : (j >= ny ? ny - 1 : j);
        if (last || sy * nx + wrapx(x0 - 2 + k % QX, nx) != ix) continue;
        const double* u = a.dtd.before.u + ((size_t)b * a.dtd.stride + ct[w]) * 4;
        double d[4];
        const double Sm = signal_speed_grad(P, u[0], u[1], u[2], u[3], d);
        const double coef = (m - a.dtd.mu_last[b]) * (-P.cfl / (Sm * Sm));
#pragma unroll
        for (int v = 0; v < 4; ++v) S.L[v][k / QX][k % QX] += coef * d[v];
      }
    }
  }

  // slopes, their cases and the predicted states of the tile + 2 (but for the
  // three cells of each corner that no face needs)
  const double hx = 0.5 * dt * P.inv_dx, hy = 0.5 * dt * P.inv_dy, hg = 0.5 * dt * P.g_y;
  auto ldW = [&](int x, int y) { return W4{S.W[0][y][x], S.W[1][y][x], S.W[2][y][x], S.W[3][y][x], S.W[4][y][x]}; };
  for (int k = tid; k < QX * QY; k += NT) {
    const int lx = k % QX, ly = k / QX, j = y0 - 2 + ly;
    const int ex = lx < QX - 1 - lx ? lx : QX - 1 - lx, ey = ly < QY - 1 - ly ? ly : QY - 1 - ly;
    if (j < 0 || j >= ny || ex + ey < 2) continue;
    const W4 wc = ldW(lx + 1, ly + 1), wb = ldW(lx + 1, ly), wt = ldW(lx + 1, ly + 2);
    int cx, cy;
    const W4 sx = mc4<true>(P, ldW(lx, ly + 1), wc, ldW(lx + 2, ly + 1), cx);
    W4 sy = mc4<true>(P, wb, wc, wt, cy);
    if constexpr (BAL) mc_p_balanced<true>(P, wb, wc, wt, sy, cy);
    const W4 q = predict(P, wc, sx, sy, hx, hy, hg);
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
    S.C[ly][lx] = cx | (cy << 8);
    const double hr = 0.5 * fabs(sx.r), hp = 0.5 * fabs(sx.p), vr = 0.5 * fabs(sy.r), vp = 0.5 * fabs(sy.p);
    bad |= !(q.r - hr > 0.0) | !(q.p - hp > 0.0) | !(q.r - vr > 0.0) | !(q.p - vp > 0.0);
  }
  __syncthreads();

  // faces, in the coordinates of Q (cell (zx, zy) of Z is (zx + 1, zy + 1))
  const double ax = dt * P.inv_dx, ay = dt * P.inv_dy;
  double mu = 0.0;  // DTD: this thread's share of d<lambda^{n+1}, U^{n+1}>/d dt, each face once
  auto lam = [&](int x, int y, double l[4]) {
    const double l2 = S.L[2][y][x];
    l[0] = S.L[0][y][x] + hdtg * l2;
    l[1] = S.L[1][y][x];
    l[2] = l2;
    l[3] = S.L[3][y][x];
  };
  auto side = [&](int s, int n, int t, double h, int x, int y) {  // state at distance h slopes from a cell's centre
    return FS{S.Q[0][y][x] + h * S.Q[s][y][x], S.Q[n][y][x] + h * S.Q[s + n][y][x], S.Q[t][y][x] + h * S.Q[s + t][y][x],
              S.Q[3][y][x] + h * S.Q[s + 3][y][x]};
  };
  // right face of cell (x, y); count: DTD counts it here
  auto xface = [&](int x, int y, bool count, FS& Lb, FS& Rb) {
    double lL[4], lR[4];
    lam(x, y, lL);
    lam(x + 1, y, lR);
    const double Fb[4] = {ax * (lR[0] - lL[0]), ax * (lR[1] - lL[1]), ax * (lR[2] - lL[2]), ax * (lR[3] - lL[3])};
    double F[4];
    hllc_adj(P, side(4, 1, 2, 0.5, x, y), side(4, 1, 2, -0.5, x + 1, y), Fb, Lb, Rb, DTD ? F : nullptr);
    if constexpr (DTD)
      if (count)
        mu += P.inv_dx * ((lR[0] - lL[0]) * F[0] + (lR[1] - lL[1]) * F[1] + (lR[2] - lL[2]) * F[2] +
                          (lR[3] - lL[3]) * F[3] + hdtg * (lR[2] - lL[2]) * F[0]);
  };
  // top face of cell (x, y), row j of faces
  auto yface = [&](int x, int y, int j, bool count, FS& Bb, FS& Tb) {
    if (j == 0) {
      double lT[4];
      lam(x, y + 1, lT);
      const FS T = side(8, 2, 1, -0.5, x, y + 1);
      wall_pressure_adj(P, T, false, ay * lT[2], Tb);
      if constexpr (DTD)
        if (count) mu += P.inv_dy * lT[2] * wall_pressure(P, T, false);
    } else if (j == ny) {
      double lB[4];
      lam(x, y, lB);
      const FS B = side(8, 2, 1, 0.5, x, y);
      wall_pressure_adj(P, B, true, -ay * lB[2], Bb);
      if constexpr (DTD)
        if (count) mu -= P.inv_dy * lB[2] * wall_pressure(P, B, true);
    } else if (j > 0 && j < ny) {
      double lB[4], lT[4];
      lam(x, y, lB);
      lam(x, y + 1, lT);
      const double g0 = ay * (lT[0] - lB[0]) + hdtg * (lT[3] + lB[3]);
      const double g1 = ay * (lT[1] - lB[1]);
      const double g2 = ay * (lT[2] - lB[2]);
      const double g3 = ay * (lT[3] - lB[3]);
      const double Fb[4] = {g0, g2, g1, g3};
      double F[4];
      hllc_adj(P, side(8, 2, 1, 0.5, x, y), side(8, 2, 1, -0.5, x, y + 1), Fb, Bb, Tb, DTD ? F : nullptr);
      if constexpr (DTD)
        if (count)
          mu += P.inv_dy * ((lT[0] - lB[0]) * F[0] + (lT[1] - lB[1]) * F[2] + (lT[2] - lB[2]) * F[1] +
                            (lT[3] - lB[3]) * F[3] + hdtg * (lT[2] - lB[2]) * F[0]) +
                0.5 * P.g_y * (lT[3] + lB[3]) * F[0];
    }
  };
  // a cell's thread takes its right and its top face; spare thread e the left
  // face of row e's first cell and the bottom face of column e's first cell
  FS Lb{0, 0, 0, 0}, Bb{0, 0, 0, 0};
  {
    const int e = tid - ZX * ZY;
    const bool halo_row = e == 0 || e == ZY - 1, halo_col = e == 0 || e == ZX - 1;
    // cell to the left of the face, in Z coordinates
    const int fx = in_z ? zx : (halo_row ? 0 : -1), fy = in_z ? zy : e;
    const int jr = y0 - 1 + fy;
    if (in_z ? cell : (e >= 0 && e < ZY && jr >= 0 && jr < ny)) {
      FS Rb{0, 0, 0, 0};
      xface(fx + 1, fy + 1, own, Lb, Rb);
      if (fx + 1 < ZX) {
        S.z.X[0][fy][fx + 1] = Rb.r;
        S.z.X[1][fy][fx + 1] = Rb.n;
        S.z.X[2][fy][fx + 1] = Rb.t;
        S.z.X[3][fy][fx + 1] = Rb.p;
      }
    }
    // cell below the face
    const int hx_ = in_z ? zx : e, hy_ = in_z ? zy : (halo_col ? 0 : -1);
    const int j = y0 + hy_;  // row of faces
    if ((in_z ? !corner : (e >= 0 && e < ZX)) && j >= 0 && j <= ny) {
      FS Tb{0, 0, 0, 0};
      const bool wall_below = in_z && zy == 0 && j == 0 && zx >= 1 && zx <= TX && gx < nx;
      yface(hx_ + 1, hy_ + 1, j, own || wall_below, Bb, Tb);
      if (hy_ + 1 < ZY) {
        S.z.Y[0][hy_ + 1][hx_] = Tb.r;
        S.z.Y[1][hy_ + 1][hx_] = Tb.t;
        S.z.Y[2][hy_ + 1][hx_] = Tb.n;
        S.z.Y[3][hy_ + 1][hx_] = Tb.p;
      }
    }
  }
  // the cell's own state again, for the predictor's and the primitive map's
  // adjoint
  double u0 = 1.0, u1 = 0.0, u2 = 0.0, u3 = 1.0;
  if (cell) {
    u0 = ldg(U, c);
    u1 = ldg(U + N, c);
    u2 = ldg(U + 2 * N, c);
    u3 = ldg(U + 3 * N, c);
  }
  __syncthreads();

  // cells: slope cotangents and the direct part of lambda^n
  double dir[4] = {0, 0, 0, 0};
  W4 w{1, 0, 0, 1, 1}, sxb{0, 0, 0, 0, 0}, syb{0, 0, 0, 0, 0};
  if (cell) {
    const int qx_ = zx + 1, qy_ = zy + 1;
    const W4 xl{S.z.X[0][zy][zx], S.z.X[1][zy][zx], S.z.X[2][zy][zx], S.z.X[3][zy][zx], 0.0};
    const W4 yb{S.z.Y[0][zy][zx], S.z.Y[1][zy][zx], S.z.Y[2][zy][zx], S.z.Y[3][zy][zx], 0.0};
    const W4 xr{Lb.r, Lb.n, Lb.t, Lb.p, 0.0}, yt{Bb.r, Bb.t, Bb.n, Bb.p, 0.0};
    const W4 qx{xl.r + xr.r, xl.u + xr.u, xl.v + xr.v, xl.p + xr.p, 0.0};
    sxb = W4{0.5 * (xr.r - xl.r), 0.5 * (xr.u - xl.u), 0.5 * (xr.v - xl.v), 0.5 * (xr.p - xl.p), 0.0};
    const W4 qb{qx.r + yb.r + yt.r, qx.u + yb.u + yt.u, qx.v + yb.v + yt.v, qx.p + yb.p + yt.p, 0.0};
    syb = W4{0.5 * (yt.r - yb.r), 0.5 * (yt.u - yb.u), 0.5 * (yt.v - yb.v), 0.5 * (yt.p - yb.p), 0.0};
    W4 wb{0, 0, 0, 0, 0};
    w = cons_to_prim(P, u0, u1, u2, u3);
    const W4 sx{S.Q[4][qy_][qx_], S.Q[5][qy_][qx_], S.Q[6][qy_][qx_], S.Q[7][qy_][qx_], 0.0};
    const W4 sy{S.Q[8][qy_][qx_], S.Q[9][qy_][qx_], S.Q[10][qy_][qx_], S.Q[11][qy_][qx_], 0.0};
    predict_adj(P, w, sx, sy, hx, hy, qb, wb, sxb, syb);
    const double ln[4] = {S.L[0][qy_][qx_], S.L[1][qy_][qx_], S.L[2][qy_][qx_], S.L[3][qy_][qx_]};
    if constexpr (DTD)
      if (own) {
        const double ri = w.ri;
        const double axr = w.u * sx.r + w.r * sx.u, axu = w.u * sx.u + sx.p * ri, axv = w.u * sx.v,
                     axp = P.gamma * w.p * sx.u + w.u * sx.p;
        const double ayr = w.v * sy.r + w.r * sy.v, ayu = w.v * sy.u, ayv = w.v * sy.v + sy.p * ri,
                     ayp = P.gamma * w.p * sy.v + w.v * sy.p;
        mu += P.g_y * ln[2] * u0 - 0.5 * P.inv_dx * (qb.r * axr + qb.u * axu + qb.v * axv + qb.p * axp) -
              0.5 * P.inv_dy * (qb.r * ayr + qb.u * ayu + qb.v * ayv + qb.p * ayp) + 0.5 * P.g_y * qb.v;
      }
    double ud[4];
    prim_adj(P, w, wb, ud);
    dir[0] = ud[0] + ln[0] + dt * P.g_y * ln[2];
    dir[1] = ud[1] + ln[1];
    dir[2] = ud[2] + ln[2];
    dir[3] = ud[3] + ln[3];
    // (only this thread has read these places)
    S.z.X[0][zy][zx] = sxb.r;
    S.z.X[1][zy][zx] = sxb.u;
    S.z.X[2][zy][zx] = sxb.v;
    S.z.X[3][zy][zx] = sxb.p;
    S.z.Y[0][zy][zx] = syb.r;
    S.z.Y[1][zy][zx] = syb.u;
    S.z.Y[2][zy][zx] = syb.v;
    S.z.Y[3][zy][zx] = syb.p;
  }
  __syncthreads();

  // gather of the limiter adjoints, as kernel B's
  if (own) {
    double wb[4] = {0.0, 0.0, 0.0, 0.0};
    auto add = [&](const double (&Z)[4][ZY][ZX], int x, int y, int code, double sa, double sb, double out[4]) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        double ca, cb;
        mc_weights((code >> (2 * v)) & 3, ca, cb);
        out[v] += (sa * ca + sb * cb) * Z[v][y][x];
      }
    };
    const int cc = S.C[zy + 1][zx + 1], c0 = cc >> 8;
    add(S.z.X, zx - 1, zy, S.C[zy + 1][zx] & 0xff, 0.0, 1.0, wb);
    add(S.z.X, zx, zy, cc & 0xff, 1.0, -1.0, wb);
    add(S.z.X, zx + 1, zy, S.C[zy + 1][zx + 2] & 0xff, -1.0, 0.0, wb);
    add(S.z.Y, zx, zy, c0, 1.0, -1.0, wb);
    if constexpr (BAL) {
      double wa, wbb;
      mc_weights((c0 >> 6) & 3, wa, wbb);
      wb[0] += P.g_y * P.dy * (1.0 - wa - wbb) * syb.p;
    }
    if (gy > 0) add(S.z.Y, zx, zy - 1, S.C[zy][zx + 1] >> 8, 0.0, 1.0, wb);
    if (gy < ny - 1) add(S.z.Y, zx, zy + 1, S.C[zy + 2][zx + 1] >> 8, -1.0, 0.0, wb);
    if (gy == 0 || gy == ny - 1) {
      double gb[4] = {0.0, 0.0, 0.0, 0.0};
      if (gy == 0) add(S.z.Y, zx, zy, c0, -1.0, 0.0, gb);
      if (gy == ny - 1) add(S.z.Y, zx, zy, c0, 0.0, 1.0, gb);
      const double sgn = gy == 0 ? -1.0 : 1.0;
      wb[0] += gb[0] + sgn * P.g_y * P.dy * gb[3];
      wb[1] += gb[1];
      wb[2] -= gb[2];
      wb[3] += gb[3];
    }
    double ub[4];
    prim_adj(P, w, W4{wb[0], wb[1], wb[2], wb[3], 0.0}, ub);
#pragma unroll
    for (int v = 0; v < 4; ++v) stg(Lo + v * N, c, dir[v] + ub[v]);
  }
  if (bad) atomicOr(&a.flags->err_unphys, 1);
  if constexpr (DTD) {
    __shared__ double rmu[NT / 64], rsp[NT / 64];
    __shared__ int rix[NT / 64];
    double sp = -1.0;
    int ix = 0x7fffffff;
    if (own) {
      sp = signal_speed(P, u0, u1, u2, u3);
      ix = (int)c;
    }
    const double m = block_sum<NT>(mu, rmu);
    block_argmax<NT>(sp, ix, rsp, rix);
    const size_t o = (size_t)b * a.dtd.stride + (size_t)tby * gridDim.x + tbx;
    if (own && (int)c == ix) {
      double* u = a.dtd.u + o * 4;
      u[0] = u0;
      u[1] = u1;
      u[2] = u2;
      u[3] = u3;
    }
    if (tid == 0) {
      a.dtd.mu[o] = m;
      a.dtd.smax[o] = sp;
      a.dtd.imax[o] = ix;
    }
  }
}

// (DTD: 128 registers, where 130 would leave three blocks of 256 threads per CU)
template <int TX, int TY, int NT, bool DTD, bool BAL>
__global__ __launch_bounds__(NT, DTD && NT <= 512 ? 4 : 1) void k_adj_fused(Params P, AdjArgs a) {
  __shared__ FusedLDS<TX, TY> S;
  int tbx, tby;
  tile_of_block(tbx, tby);
  adj_tile_body<TX, TY, NT, DTD, BAL>(P, a, S, blockIdx.z, tbx, tby);
}

// The adjoint of one step and, in the second half of the grid, a step at a
// given dt of other states (the reverse sweep's re-computation of the segment
// before): both are a chain of phases that leaves most of the chip idle on
// small grids, so side by side they take little more than the longer one, and
// the sweep needs no second stream and no events.
template <int TX, int TY, int NT, bool DTD, bool BAL>
__global__ __launch_bounds__(NT, DTD ? 4 : 1) void k_adj_fused_and_step(Params P, AdjArgs a, StepArgs st) {
  __shared__ union {
    FusedLDS<TX, TY> adj;
    StepLDS<TX, TY, false> step;
  } S;
  int tbx, tby;
  tile_of_block(tbx, tby);
  const int b = blockIdx.z;
  if (b < P.nb) adj_tile_body<TX, TY, NT, DTD, BAL>(P, a, S.adj, b, tbx, tby);
  else step_tile_body<TX, TY, NT, BAL, false>(P, st, S.step, nullptr, b - P.nb, tbx, tby);
}

template <int TX, int TY, int NT, bool DTD, bool BAL>
hipError_t launch_pair(const Params& P, const AdjArgs& a, const StepArgs& st, hipStream_t s) {
  const dim3 grid((P.nx + TX - 1) / TX, (P.ny + TY - 1) / TY, 2 * P.nb);
  if (DTD && (a.dtd.count != (int)(grid.x * grid.y) || a.dtd.stride < a.dtd.count || !a.dtd.u || !a.nsteps_limit))
    return hipErrorInvalidValue;
  hipLaunchKernelGGL((k_adj_fused_and_step<TX, TY, NT, DTD, BAL>), grid, dim3(NT), 0, s, P, a, st);
  return hipGetLastError();
}
template <int TX, int TY, int NT>
hipError_t launch_pair_t(const Params& P, const AdjArgs& a, const StepArgs& st, hipStream_t s) {
  if (a.dtd.mu != nullptr)
    return P.recon == 1 ? launch_pair<TX, TY, NT, true, true>(P, a, st, s) : launch_pair<TX, TY, NT, true, false>(P, a, st, s);
  return P.recon == 1 ? launch_pair<TX, TY, NT, false, true>(P, a, st, s) : launch_pair<TX, TY, NT, false, false>(P, a, st, s);
}

template <int TX, int TY, int NT>
hipError_t launch_t(const Params& P, const AdjArgs& a, hipStream_t s) {
  const dim3 grid((P.nx + TX - 1) / TX, (P.ny + TY - 1) / TY, P.nb);
  const bool bal = P.recon == 1;
  if (a.dtd.mu != nullptr) {
    if (a.dtd.count != (int)(grid.x * grid.y) || a.dtd.stride < a.dtd.count || !a.dtd.u || !a.nsteps_limit)
      return hipErrorInvalidValue;
    if (bal)
      hipLaunchKernelGGL((k_adj_fused<TX, TY, NT, true, true>), grid, dim3(NT), 0, s, P, a);
    else
      hipLaunchKernelGGL((k_adj_fused<TX, TY, NT, true, false>), grid, dim3(NT), 0, s, P, a);
  } else if (bal) {
    hipLaunchKernelGGL((k_adj_fused<TX, TY, NT, false, true>), grid, dim3(NT), 0, s, P, a);
  } else {
    hipLaunchKernelGGL((k_adj_fused<TX, TY, NT, false, false>), grid, dim3(NT), 0, s, P, a);
  }
  return hipGetLastError();
}

}  // namespace

namespace {

// The shapes: threads for one pass over the primitives (the widest phase) and
// the time of a launch, fixed + per_round * rounds, a round being one block per
// CU.  With at most one block per CU a launch lasts as long as one block's
// chain of phases, and the smallest tile that still covers the grid in one
// round wins; beyond that larger tiles compute less halo again.  Measured, us:
// 8x8 6.5 (64x128), 8.3, 11.4 (256x256), 19.7 (256x512); 16x8 6.9 (128x256),
// 9.6, 18.0; 16x16 8.7-9.2 (256x256), 13.2 (256x512), 18.8, 23.5; 24x16 9.4-9.9
// (300x300), 18.4 (384x512); 32x16 10.9-11.6 (256x512), 22.0 (512x512), 32.7.
struct Shape {
  int tx, ty;
  double fixed, per_round;
};
constexpr Shape kShapes[] = {{8, 8, 4.2, 2.0}, {16, 8, 3.6, 3.4}, {16, 16, 4.2, 4.85}, {24, 16, 1.0, 8.7}, {32, 16, 1.0, 10.7}};
constexpr int kCus = 256;

long shape_blocks(const Params& P, const Shape& h) {
  return (long)((P.nx + h.tx - 1) / h.tx) * ((P.ny + h.ty - 1) / h.ty);
}

int pick_shape(const Params& P, int nb, double* us) {
  int best = 0;
  double t = 1e300;
  for (int k = 0; k < (int)(sizeof kShapes / sizeof kShapes[0]); ++k) {
    const long rounds = (shape_blocks(P, kShapes[k]) * nb + kCus - 1) / kCus;
    const double u = kShapes[k].fixed + kShapes[k].per_round * (double)rounds;
    if (u < t) {
      t = u;
      best = k;
    }
  }
  if (us) *us = t;
  return best;
}

}  // namespace

int adj_fused_blocks(const Params& P, int nb) { return (int)shape_blocks(P, kShapes[pick_shape(P, nb, nullptr)]); }

double adj_fused_us(const Params& P) {
  double us;
  (void)pick_shape(P, P.nb, &us);
  return us;
}

hipError_t launch_adj_fused(const Params& P, const AdjArgs& a, hipStream_t s) {
  if (a.fold.Z != nullptr) return hipErrorInvalidValue;
  switch (pick_shape(P, a.dtd.mu ? a.dtd.batch : P.nb, nullptr)) {
    case 0: return launch_t<8, 8, 256>(P, a, s);
    case 1: return launch_t<16, 8, 320>(P, a, s);
    case 2: return launch_t<16, 16, 512>(P, a, s);
    case 3: return launch_t<24, 16, 704>(P, a, s);
    default: return launch_t<32, 16, 1024>(P, a, s);
  }
}

// Whether the small shapes, those with a paired kernel, are the ones that run,
// and the pair's grid holds both halves of the batch.
bool adj_fused_pairs(const Params& P) { return P.nb <= 32767 && pick_shape(P, P.nb, nullptr) <= 2; }

hipError_t launch_adj_fused_and_step(const Params& P, const AdjArgs& a, const StepArgs& st, hipStream_t s) {
  if (a.fold.Z != nullptr || st.ctl != nullptr || st.speeds != nullptr) return hipErrorInvalidValue;
  switch (pick_shape(P, P.nb, nullptr)) {
    case 0: return launch_pair_t<8, 8, 256>(P, a, st, s);
    case 1: return launch_pair_t<16, 8, 320>(P, a, st, s);
    case 2: return launch_pair_t<16, 16, 512>(P, a, st, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace rtk
