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
#include "lc_launch.h"

namespace lc {

// Rectangles of a tile and the LDS its stages take (values of the order-tensor
// type): Q on radius 4, the stress, the velocity on radius 2, Q^P on radius 1.
template <int TX, int TY, bool ISO>
struct Fused2d {
  using R4 = Rect<TX, TY, 4>;
  using R3 = Rect<TX, TY, 3>;
  using R2 = Rect<TX, TY, 2>;
  using R1 = Rect<TX, TY, 1>;
  static constexpr int NTHR = FUSED2D_NTHR, NT = TX * TY;
  static_assert(R3::N <= NTHR, "one point per thread in every stage");
  // stress columns kept: tau_{a x} at x-range of radius 3 and y-range of
  // radius 2 (for d_x at the radius-2 sites), tau_{a y} the other way round;
  // isotropic: tau_ab on the whole radius-3 rectangle
  static constexpr int WX = R3::W, NXA = R3::W * R2::H;
  static constexpr int WY = R2::W, NYA = R2::W * R3::H;
  static constexpr int NQ = 5 * R4::N, NTAU = ISO ? 4 * R3::N : 2 * (NXA + NYA), NU = 2 * R2::N, NP = 5 * R1::N;
  // the thread's point of the moment stage (waves in reverse), tile sites first
  struct Moment {
    int kl, i2, j2;
    __device__ __forceinline__ Moment()
        : kl((NTHR / 64 - 1 - int(threadIdx.x) / 64) * 64 + threadIdx.x % 64), i2(0), j2(0) {
      if (any()) tile_first<TX, TY, 2>(kl, i2, j2);
    }
    __device__ __forceinline__ bool any() const { return kl < R2::N; }
  };
};

// The stages of one step on a tile, from Q on radius 4 in LDS (mQ, complete) and
// the pulled populations f of the thread's moment point.  put_f(i, j, f, rho,
// mass, u, F) takes the moments of tile site (i, j), for its collision;
// put_q(i, j, q, r, Rp, p) the Q, rate, corrector rate and predictor.  mT, mU
// and mP are the LDS of the stress, velocity and predictor.
// ST: the difference stencils (lc_staged.h).  With the isotropic ones the
// whole stress of the radius-3 rectangle, corners included, is in LDS for the
// body force, and the stencils of Q, u and Q^P come from the pairs of opposite
// velocities, with the arithmetic of the two sweeps.
template <typename S, bool DEV, int TX, int TY, typename QT, bool SR, int ST, typename PUTF, typename PUTQ>
__device__ __forceinline__ void fused2d_stages(QT* mQ, QT* mT, QT* mU, QT* mP,
                                               const typename Fused2d<TX, TY, ST == STENCIL_ISO>::Moment& m,
                                               S (&f)[9], const Coef<QT>& cq, PUTF put_f, PUTQ put_q) {
  using L = Lattice<0>;
  constexpr bool ISO = ST == STENCIL_ISO;
  using C = Fused2d<TX, TY, ISO>;
  using R4 = typename C::R4;
  using R3 = typename C::R3;
  using R2 = typename C::R2;
  using R1 = typename C::R1;
  constexpr int NT = C::NT, WX = C::WX, WY = C::WY;
  auto sQ = reinterpret_cast<QT(*)[R4::N]>(mQ);
  auto sTx = reinterpret_cast<QT(*)[C::NXA]>(mT);
  auto sTy = reinterpret_cast<QT(*)[C::NYA]>(mT + 2 * C::NXA);
  auto sTi = reinterpret_cast<QT(*)[2][R3::N]>(mT);
  auto sU = reinterpret_cast<QT(*)[R2::N]>(mU);
  auto sP = reinterpret_cast<QT(*)[R1::N]>(mP);
  const int tid = threadIdx.x, wave = tid / 64;
  const int kl = m.kl, i2 = m.i2, j2 = m.j2;
  const bool lb = m.any();
  // its collision runs beside the predictor where its wave has no point of it
  const bool beside = wave * 64 >= R1::N;

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
    if (!beside && kl < NT) put_f(i2 - 2, j2 - 2, f, rho, mass, u, F);
  }
  __syncthreads();

  // predictor on the radius-1 rectangle; a tile site keeps what its corrector
  // needs (as the two-sweep Q update does)
  if (beside && kl < NT) put_f(i2 - 2, j2 - 2, f, rho, mass, u, F);
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
  if (tid < NT) {
    const int tx = tid % TX, ty = tid / TX;
    const int k1 = (tx + 1) + R1::W * (ty + 1);
    Sym<QT> p, Lp, d[3];
    if constexpr (ISO)
      stencil_lds_iso2<QT, R1::W, R1::N, false>(sP, k1, p, d, Lp);
    else
      stencil_lds<QT, 2, R1::W, R1::N, false>(sP, sP, sP, k1, p, d, Lp);
    const Sym<QT> H = SR ? molecular_field_exact(p, Lp, cq) : molecular_field(p, Lp, cq);
    put_q(tx, ty, q, r, be_rate_flow<QT, true, 2>(p, H, d, fl, cq), p);
  }
}

// Collision in place on f.
template <typename S, bool DEV, bool MRT>
__device__ __forceinline__ void collide2d(S (&f)[9], S rho, S mass, const S (&u)[3], const S (&F)[3],
                                          const Coef<S>& c) {
  if constexpr (MRT)
    collide_mrt<0, S, DEV>(f, rho, mass, u, F, c);
  else
    collide_pairs<0, S, DEV>(f, rho, mass, u, F, c);
}

// Q on radius 4 of a tile from memory into LDS, and the pulled populations
// f_i(x) = buf_i(x - c_i) of the thread's moment point, every load issued
// before the first value is stored.
template <int TX, int TY, bool ISO, typename S, typename QT>
__device__ __forceinline__ void fused2d_load(const QT* __restrict__ Qin, const S* __restrict__ fin, QT* mQ,
                                             const typename Fused2d<TX, TY, ISO>::Moment& m, S (&f)[9],
                                             const TileDims& g, int x0, int y0) {
  using L = Lattice<0>;
  using C = Fused2d<TX, TY, ISO>;
  using R4 = typename C::R4;
  auto sQ = reinterpret_cast<QT(*)[R4::N]>(mQ);
  const int tid = threadIdx.x;
  const size_t N = size_t(g.N);
  const uint32_t sy = uint32_t(g.nx);
  constexpr int P4 = (R4::N + C::NTHR - 1) / C::NTHR;
  QT qv[P4][5];
  auto load = [&](auto wrap) {
#pragma unroll
    for (int n = 0; n < P4; n++) {
      const int k = tid + n * C::NTHR;
      if (k < R4::N) {
        const uint32_t s = uint32_t(wrap(x0 - 4 + k % R4::W, g.nx)) + sy * uint32_t(wrap(y0 - 4 + k / R4::W, g.ny));
#pragma unroll
        for (int q = 0; q < 5; q++) qv[n][q] = (Qin + size_t(q) * N)[s];
      }
    }
    if (m.any()) {
      const int gx = wrap(x0 - 2 + m.i2, g.nx), gy = wrap(y0 - 2 + m.j2, g.ny);
      const uint32_t site = uint32_t(gx) + sy * uint32_t(gy);
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
        f[i] = (fin + size_t(i) * N)[d];
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
    const int k = tid + n * C::NTHR;
    if (k < R4::N) {
#pragma unroll
      for (int q = 0; q < 5; q++) sQ[q][k] = qv[n][q];
    }
  }
}

// REC: record what the reverse step of the step needs (at the tile's sites):
// the velocity, the density and body force, and the predictor.
struct StepRecord {
  double *u, *rho_f, *qp;  // 2, 1 + 2 and 5 components
};

// What a tile's last step of a launch does with its sites: collide and store,
// update Q and store.
template <typename S, bool DEV, bool MRT, typename QT, bool SR, bool REC>
struct Fused2dOut {
  S* fout;
  QT* Qout;
  const TileDims& g;
  const Coef<S>& c;
  int x0, y0;
  uint32_t srkey;
  const StepRecord& rec;
  __device__ __forceinline__ bool site(int i, int j, uint32_t& s) const {
    s = uint32_t(x0 + i) + uint32_t(g.nx) * uint32_t(y0 + j);
    return x0 + i < g.nx && y0 + j < g.ny;
  }
  __device__ __forceinline__ void put_f(int i, int j, S (&f)[9], S rho, S mass, const S (&u)[3],
                                        const S (&F)[3]) const {
    uint32_t s;
    if (!site(i, j, s)) return;
    const size_t N = size_t(g.N);
    if constexpr (REC) {
      rec.rho_f[s] = rho;
#pragma unroll
      for (int a = 0; a < 2; a++) {
        rec.u[a * N + s] = u[a];
        rec.rho_f[(a + 1) * N + s] = F[a];
      }
    }
    collide2d<S, DEV, MRT>(f, rho, mass, u, F, c);
#pragma unroll
    for (int k = 0; k < 9; k++) store_out(&(fout + size_t(k) * N)[s], f[k]);
  }
  __device__ __forceinline__ void put_q(int i, int j, const Sym<QT>& q, const Sym<QT>& r, const Sym<QT>& Rp,
                                        const Sym<QT>& p) const {
    uint32_t s;
    if (!site(i, j, s)) return;
    if constexpr (REC) store_sym(rec.qp, g.N, int64_t(s), p);
    store_q_update<QT, SR>(Qout, g.N, int64_t(s), q, r, Rp, srkey);
  }
};

template <typename S, bool DEV, int TX, int TY, bool MRT, typename QT, bool SR, int ST = STENCIL_COMPACT,
          bool REC = false>
__global__ void __launch_bounds__(FUSED2D_NTHR)
    fused2d_step(const QT* __restrict__ Qin, const S* __restrict__ fin, S* __restrict__ fout, QT* __restrict__ Qout,
                 TileDims g, Coef<S> c, Coef<QT> cq, uint32_t srkey, StepRecord rec) {
  constexpr bool ISO = ST == STENCIL_ISO;
  using C = Fused2d<TX, TY, ISO>;
  __shared__ QT mQ[C::NQ], mT[C::NTAU], mU[C::NU], mP[C::NP];
  const int t = xcd_remap(blockIdx.x + gridDim.x * blockIdx.y, gridDim.x * gridDim.y);
  const int x0 = g.xb + (t % gridDim.x) * TX, y0 = (t / gridDim.x) * TY;
  const typename C::Moment m;
  S f[9];
  fused2d_load<TX, TY, ISO>(Qin, fin, mQ, m, f, g, x0, y0);
  __syncthreads();
  const Fused2dOut<S, DEV, MRT, QT, SR, REC> out{fout, Qout, g, c, x0, y0, srkey, rec};
  fused2d_stages<S, DEV, TX, TY, QT, SR, ST>(
      mQ, mT, mU, mP, m, f, cq, [&](auto&&... a) { out.put_f(a...); }, [&](auto&&... a) { out.put_q(a...); });
}

// Two steps in one launch, for grids whose tiles of 16x8 sites each have a CU:
// the first on the tile extended by four sites on every side, whose outcome
// stays in LDS, the second on the tile.  A launch and the wait for memory are
// a third of such a step (1.8 and 0.5 to 0.9 us), and the larger first step
// still has one point per thread in every stage.  Measured per step, one -> two
// steps per launch: 4.6 -> 4.1 us on 64^2 and 4.7 -> 4.2 us on 128^2 sites in
// FP32; 5.2 -> 4.9 us on 64^2 and 5.6 -> 5.2 us on 100^2 (MRT) in FP64, whose
// larger first step costs more of what the launch saves.
template <typename S, bool DEV, bool MRT, typename QT, bool SR, int ST = STENCIL_COMPACT>
__global__ void __launch_bounds__(FUSED2D_NTHR)
    fused2d_pair(const QT* __restrict__ Qin, const S* __restrict__ fin, S* __restrict__ fout, QT* __restrict__ Qout,
                 TileDims g, Coef<S> c, Coef<QT> cq, uint32_t srkey0, uint32_t srkey1) {
  using L = Lattice<0>;
  constexpr int TX = FUSED2D_PAIR_TX, TY = FUSED2D_PAIR_TY, EX = TX + 8, EY = TY + 8;
  constexpr bool ISO = ST == STENCIL_ISO;
  using E = Fused2d<EX, EY, ISO>;  // the extended tile: its sites are the tile's radius-4 rectangle
  using C = Fused2d<TX, TY, ISO>;
  static_assert(E::NT == C::R4::N, "the first step leaves what the second starts from");
  __shared__ QT mQ[E::NQ], mT[E::NTAU], mU[E::NU], mP[E::NP];
  __shared__ S sF[9][E::NT];  // post-collision populations of the first step
  const int t = xcd_remap(blockIdx.x + gridDim.x * blockIdx.y, gridDim.x * gridDim.y);
  const int x0 = (t % gridDim.x) * TX, y0 = (t / gridDim.x) * TY;
  const typename E::Moment me;
  S f[9];
  fused2d_load<EX, EY, ISO>(Qin, fin, mQ, me, f, g, x0 - 4, y0 - 4);
  __syncthreads();
  // Q on the extended tile replaces that of the radius-4 rectangle around it,
  // which is last read by the predictor
  auto sQ = reinterpret_cast<QT(*)[E::NT]>(mQ);
  fused2d_stages<S, DEV, EX, EY, QT, SR, ST>(
      mQ, mT, mU, mP, me, f, cq,
      [&](int i, int j, S(&fc)[9], S rho, S mass, const S(&u)[3], const S(&F)[3]) {
        collide2d<S, DEV, MRT>(fc, rho, mass, u, F, c);
#pragma unroll
        for (int k = 0; k < 9; k++) sF[k][i + EX * j] = fc[k];
      },
      [&](int i, int j, const Sym<QT>& q, const Sym<QT>& r, const Sym<QT>& Rp, const Sym<QT>&) {
        const uint32_t s = SR ? uint32_t(wrapi(x0 - 4 + i, g.nx)) + uint32_t(g.nx) * uint32_t(wrapi(y0 - 4 + j, g.ny))
                              : 0u;
        q_update<QT, SR>(s, q, r, Rp, srkey0, [&](int k, QT v) { sQ[k][i + EX * j] = v; });
      });
  __syncthreads();
  const typename C::Moment m;
  if (m.any()) {
#pragma unroll
    for (int k = 0; k < 9; k++) f[k] = sF[k][(m.i2 + 2 - L::cx(k)) + EX * (m.j2 + 2 - L::cy(k))];
  }
  const StepRecord none{};
  const Fused2dOut<S, DEV, MRT, QT, SR, false> out{fout, Qout, g, c, x0, y0, srkey1, none};
  fused2d_stages<S, DEV, TX, TY, QT, SR, ST>(
      mQ, mT, mU, mP, m, f, cq, [&](auto&&... a) { out.put_f(a...); }, [&](auto&&... a) { out.put_q(a...); });
}

}  // namespace lc
