// lc_fused2d.h -- the single pass (lc_fused.h) on two-dimensional grids: one
// launch per step, one block per tile, every stage on a rectangle that
// shrinks by one site.
//
// A step of a grid with at most one tile per CU is bound by the serial chain
// of its stages, not by bandwidth or issue (256^2 in FP64: 2.0 us of launch,
// then loads, stress, moments and collision, predictor and corrector, each
// waiting for the one before), so the block takes off that chain what the
// next stage does not need:
//  - every global load is issued before the first stage;
//  - the moment sums of the populations and the division by the density run
//    beside the stress, on the waves that have no stress point;
//  - the collision and its stores run beside the predictor, on the waves
//    that have no predictor point.
// To that end the points of the moment stage are dealt to the block's waves
// from the last one down and those of the other stages from the first one up.
#pragma once

#include "lc_fused.h"

namespace lc {

// Shapes of the single pass on two-dimensional grids: tiles of TX x TY
// sites, all with 1024 threads.  A step of a small grid is a chain of stages
// with a barrier between them, and a CU that holds one block spends the chain
// once; so the runtime takes the smallest tile with which the grid has at
// most one tile per CU (16x8 up to 32x20, whose radius-3 rectangle of 38x26
// points still has one thread per point).  Measured per step in the mixed
// form on 301x419 sites: 15.4 us with 530 tiles of 32x8 sites and 512 threads
// (two rounds of blocks), 9.7 us with 210 tiles of 32x20; on 256^2 sites (32x8
// tiles) 7.4 -> 7.1 us in FP64 and 5.9 -> 5.6 us in FP32, on 128x16 (16x8)
// 6.0 -> 4.9 us in FP64, against the same tiles without the overlap above.
constexpr int FUSED2D_NTHR = 1024;
constexpr int FUSED2D_CUS = 256;  // compute units of the chip
constexpr int FUSED2D_NV = 5;
__host__ __device__ constexpr int fused2d_tx(int v) { return v == 0 ? 16 : 32; }
__host__ __device__ constexpr int fused2d_ty(int v) { return v < 2 ? 8 : (v == 2 ? 12 : (v == 3 ? 16 : 20)); }

// ST: the difference stencils (lc_staged.h).  With the isotropic ones the
// whole stress of the radius-3 rectangle, corners included, is in LDS for the
// body force, and the stencils of Q, u and Q^P come from the pairs of opposite
// velocities, with the arithmetic of the two sweeps.
// REC: record what the reverse step of the step needs (at the tile's sites):
// the velocity, the density and body force, and the predictor.
struct StepRecord {
  double *u, *rho_f, *qp;  // 2, 1 + 2 and 5 components
};

template <typename S, bool DEV, int TX, int TY, bool MRT, typename QT, bool SR, int ST, bool REC>
__device__ __forceinline__ void fused2d_body(const QT* __restrict__ Qin, const S* __restrict__ fin,
                                             S* __restrict__ fout, QT* __restrict__ Qout, const GridDims& g,
                                             const Coef<S>& c, const Coef<QT>& cq, int bx, int by, uint32_t srkey,
                                             const StepRecord& rec) {
  using L = Lattice<0>;
  constexpr int NTHR = FUSED2D_NTHR, NT = TX * TY;
  using R4 = Rect<TX, TY, 4>;
  using R3 = Rect<TX, TY, 3>;
  using R2 = Rect<TX, TY, 2>;
  using R1 = Rect<TX, TY, 1>;
  static_assert(R3::N <= NTHR, "one point per thread in every stage");
  // stress columns kept: tau_{a x} at x-range of radius 3 and y-range of
  // radius 2 (for d_x at the radius-2 sites), tau_{a y} the other way round
  constexpr int WX = R3::W, NXA = R3::W * R2::H;
  constexpr int WY = R2::W, NYA = R2::W * R3::H;
  constexpr bool ISO = ST == STENCIL_ISO;
  __shared__ QT sQ[5][R4::N];
  __shared__ QT sTx[2][ISO ? 1 : NXA];
  __shared__ QT sTy[2][ISO ? 1 : NYA];
  __shared__ QT sTi[ISO ? 2 : 1][ISO ? 2 : 1][ISO ? R3::N : 1];  // isotropic: tau_ab on the radius-3 rectangle
  __shared__ QT sU[2][R2::N];
  __shared__ QT sP[5][R1::N];

  const int tid = threadIdx.x, wave = tid / 64;
  const int x0 = bx * TX, y0 = by * TY;
  const int64_t N = g.N;
  const uint32_t sy = uint32_t(g.nx);
  // the thread's point of the moment stage (waves in reverse), tile sites first
  const int kl = (NTHR / 64 - 1 - wave) * 64 + tid % 64;
  const bool lb = kl < R2::N;
  int i2 = 0, j2 = 0;
  if (lb) tile_first<TX, TY, 2>(kl, i2, j2);
  // its collision runs beside the predictor where its wave has no point of it
  const bool beside = wave * 64 >= R1::N;

  // site indices (periodic) of the thread's points of the radius-4 rectangle
  // (Q loads), and the pull of its populations: f_i(x) = buf_i(x - c_i)
  constexpr int P4 = (R4::N + NTHR - 1) / NTHR;
  QT qv[P4][5];
  S f[L::q];
  uint32_t site = 0;
  auto load = [&](auto wrap) {
#pragma unroll
    for (int n = 0; n < P4; n++) {
      const int k = tid + n * NTHR;
      if (k < R4::N) {
        const uint32_t s = uint32_t(wrap(x0 - 4 + k % R4::W, g.nx)) + sy * uint32_t(wrap(y0 - 4 + k / R4::W, g.ny));
#pragma unroll
        for (int q = 0; q < 5; q++) qv[n][q] = Qin[size_t(q) * size_t(N) + s];
      }
    }
    if (lb) {
      const int gx = wrap(x0 - 2 + i2, g.nx), gy = wrap(y0 - 2 + j2, g.ny);
      site = uint32_t(gx) + sy * uint32_t(gy);
      const uint32_t xp = (gx + 1 == g.nx) ? 0u - uint32_t(g.nx - 1) : 1u;
      const uint32_t xm = (gx == 0) ? uint32_t(g.nx - 1) : 0u - 1u;
      const uint32_t yp = (gy + 1 == g.ny) ? 0u - uint32_t(g.ny - 1) * sy : sy;
      const uint32_t ym = (gy == 0) ? uint32_t(g.ny - 1) * sy : 0u - sy;
#pragma unroll
      for (int i = 0; i < L::q; i++) {
        uint32_t d = site;
        if (L::cx(i) == 1) d += xm;
        if (L::cx(i) == -1) d += xp;
        if (L::cy(i) == 1) d += ym;
        if (L::cy(i) == -1) d += yp;
        f[i] = fin[size_t(i) * size_t(N) + d];
      }
    }
  };
  // without a division where the rectangle wraps at most once
  if (g.nx >= R4::W && g.ny >= R4::H)
    load([](int v, int n) { return wrap_near(v, n); });
  else
    load([](int v, int n) { return wrapi(v, n); });
#pragma unroll
  for (int n = 0; n < P4; n++) {
    const int k = tid + n * NTHR;
    if (k < R4::N) {
#pragma unroll
      for (int q = 0; q < 5; q++) sQ[q][k] = qv[n][q];
    }
  }
  __syncthreads();

  // stress on the radius-3 rectangle (compact: without its corners, which
  // neither d_x nor d_y needs)
  if (tid < R3::N) {
    const int i3 = tid % R3::W, j3 = tid / R3::W;
    const int k4 = (i3 + 1) + R4::W * (j3 + 1);
    Sym<QT> q, Lq, d[3];
    QT t[3][3];
    if constexpr (ISO) {
      stencil_lds_iso2<QT, R4::W, R4::N>(sQ, k4, q, d, Lq);
      const Sym<QT> H = molecular_field(q, Lq, cq);
      stress(q, H, d, cq, t);
#pragma unroll
      for (int a = 0; a < 2; a++)
#pragma unroll
        for (int b = 0; b < 2; b++) sTi[a][b][tid] = t[a][b];
    } else {
      const bool xin = i3 >= 1 && i3 < R3::W - 1, yin = j3 >= 1 && j3 < R3::H - 1;
      if (xin || yin) {
        stencil_lds<QT, 2, R4::W, R4::N>(sQ, sQ, sQ, k4, q, d, Lq);
        const Sym<QT> H = molecular_field(q, Lq, cq);
        stress(q, H, d, cq, t);
        if (yin) {
          const int kx = i3 + WX * (j3 - 1);
#pragma unroll
          for (int a = 0; a < 2; a++) sTx[a][kx] = t[a][0];
        }
        if (xin) {
          const int ky = (i3 - 1) + WY * j3;
#pragma unroll
          for (int a = 0; a < 2; a++) sTy[a][ky] = t[a][1];
        }
      }
    }
  }
  S rho = S(1), mass = S(0), j[3] = {S(0), S(0), S(0)}, inv = S(1);
  if (lb) moment_sums<0, S, DEV>(f, rho, mass, j, inv);
  __syncthreads();

  // body force and velocity on the radius-2 rectangle
  S F[3] = {S(0), S(0), S(0)}, u[3] = {S(0), S(0), S(0)};
  auto collide_store = [&]() {
    if (!(kl < NT && x0 + i2 - 2 < g.nx && y0 + j2 - 2 < g.ny)) return;
    if constexpr (REC) {
      rec.rho_f[site] = rho;
#pragma unroll
      for (int a = 0; a < 2; a++) {
        rec.u[a * size_t(N) + site] = u[a];
        rec.rho_f[(a + 1) * size_t(N) + site] = F[a];
      }
    }
    if constexpr (MRT)
      collide_mrt<0, S, DEV>(f, rho, mass, u, F, c);
    else
      collide_pairs<0, S, DEV>(f, rho, mass, u, F, c);
#pragma unroll
    for (int i = 0; i < L::q; i++) store_out(&(fout + size_t(i) * size_t(N))[site], f[i]);
  };
  if (lb) {
    if constexpr (ISO) {  // F_a = 3 sum_i w_i sum_b c_ib tau_ab(x + c_i), over pairs
      const int k3 = (i2 + 1) + R3::W * (j2 + 1);
#pragma unroll
      for (int a = 0; a < 2; a++) {
        QT acc = QT(0);
#pragma unroll
        for (int i = 1; i < L::q; i++) {
          if (L::opp(i) < i) continue;
          const int o = L::cx(i) + R3::W * L::cy(i);
          QT dsum = QT(0);
#pragma unroll
          for (int b = 0; b < 2; b++) {
            const int cb = b == 0 ? L::cx(i) : L::cy(i);
            if (cb == 0) continue;
            const QT dt = sTi[a][b][k3 + o] - sTi[a][b][k3 - o];
            dsum += cb > 0 ? dt : -dt;
          }
          acc += QT(3.0 * L::w(i)) * dsum;
        }
        F[a] = S(acc);
      }
    } else {
      const int kx = (i2 + 1) + WX * j2, ky = i2 + WY * (j2 + 1);
#pragma unroll
      for (int a = 0; a < 2; a++) {
        const QT acc = (sTx[a][kx + 1] - sTx[a][kx - 1]) + (sTy[a][ky + WY] - sTy[a][ky - WY]);
        F[a] = S(QT(0.5) * acc);
      }
    }
    velocity<0, S>(j, F, inv, u);
    const int k2 = i2 + R2::W * j2;
    sU[0][k2] = QT(u[0]);
    sU[1][k2] = QT(u[1]);
    if (!beside) collide_store();
  }
  __syncthreads();

  // predictor on the radius-1 rectangle; a tile site keeps what its corrector
  // needs (as the two-sweep Q update does)
  if (beside) collide_store();
  Flow<QT, 2> fl;
  Sym<QT> r, q;
  if (tid < R1::N) {
    int i1, j1;
    tile_first<TX, TY, 1>(tid, i1, j1);
    const int k4 = (i1 + 3) + R4::W * (j1 + 3);
    const int k2 = (i1 + 1) + R2::W * (j1 + 1);
    Sym<QT> Lq, d[3];
    if constexpr (ISO)
      stencil_lds_iso2<QT, R4::W, R4::N, false>(sQ, k4, q, d, Lq);
    else
      stencil_lds<QT, 2, R4::W, R4::N, false>(sQ, sQ, sQ, k4, q, d, Lq);
    const Sym<QT> H = SR ? molecular_field_exact(q, Lq, cq) : molecular_field(q, Lq, cq);
    QT up[3] = {QT(0), QT(0), QT(0)}, G[3][3];
#pragma unroll
    for (int a = 0; a < 3; a++)
#pragma unroll
      for (int b = 0; b < 3; b++) G[a][b] = QT(0);
#pragma unroll
    for (int a = 0; a < 2; a++) {
      up[a] = sU[a][k2] * QT(0.5);
      if constexpr (ISO) {  // undivided: 6 sum_i w_i c_ib u_a(x + c_i), over pairs
        QT g0 = QT(0), g1 = QT(0);
#pragma unroll
        for (int i = 1; i < L::q; i++) {
          if (L::opp(i) < i) continue;
          const int o = L::cx(i) + R2::W * L::cy(i);
          const QT dif = sU[a][k2 + o] - sU[a][k2 - o];
          const QT w6 = QT(6.0 * L::w(i));
          if (L::cx(i) != 0) g0 += (L::cx(i) > 0 ? w6 : -w6) * dif;
          if (L::cy(i) != 0) g1 += (L::cy(i) > 0 ? w6 : -w6) * dif;
        }
        G[a][0] = g0;
        G[a][1] = g1;
      } else {
        G[a][0] = sU[a][k2 + 1] - sU[a][k2 - 1];
        G[a][1] = sU[a][k2 + R2::W] - sU[a][k2 - R2::W];
      }
    }
    fl = flow_terms<QT, true, 2>(up, G, cq);
    r = be_rate_flow<QT, true, 2>(q, H, d, fl, cq);
    const int k1 = i1 + R1::W * j1;
    sP[0][k1] = q.xx + r.xx;
    sP[1][k1] = q.xy + r.xy;
    sP[2][k1] = q.xz + r.xz;
    sP[3][k1] = q.yy + r.yy;
    sP[4][k1] = q.yz + r.yz;
  }
  __syncthreads();

  // corrector at the tile's sites
  const int tx = tid % TX, ty = tid / TX;
  if (tid < NT && x0 + tx < g.nx && y0 + ty < g.ny) {
    const int k1 = (tx + 1) + R1::W * (ty + 1);
    Sym<QT> p, Lp, d[3];
    if constexpr (ISO)
      stencil_lds_iso2<QT, R1::W, R1::N, false>(sP, k1, p, d, Lp);
    else
      stencil_lds<QT, 2, R1::W, R1::N, false>(sP, sP, sP, k1, p, d, Lp);
    const Sym<QT> H = SR ? molecular_field_exact(p, Lp, cq) : molecular_field(p, Lp, cq);
    const Sym<QT> Rp = be_rate_flow<QT, true, 2>(p, H, d, fl, cq);
    const int64_t s = int64_t(uint32_t(x0 + tx) + sy * uint32_t(y0 + ty));
    if constexpr (REC) store_sym(rec.qp, N, s, p);
    store_q_update<QT, SR>(Qout, N, s, q, r, Rp, srkey);
  }
}

template <typename S, bool DEV, int TX, int TY, bool MRT, typename QT, bool SR, int ST = STENCIL_COMPACT,
          bool REC = false>
__global__ void __launch_bounds__(FUSED2D_NTHR)
    fused2d_step(const QT* __restrict__ Qin, const S* __restrict__ fin, S* __restrict__ fout, QT* __restrict__ Qout,
                 GridDims g, Coef<S> c, Coef<QT> cq, uint32_t srkey, StepRecord rec) {
  const int t = xcd_remap(blockIdx.x + gridDim.x * blockIdx.y, gridDim.x * gridDim.y);
  fused2d_body<S, DEV, TX, TY, MRT, QT, SR, ST, REC>(Qin, fin, fout, Qout, g, c, cq, t % gridDim.x, t / gridDim.x,
                                                     srkey, rec);
}

}  // namespace lc
