// lc_vjp.h -- one reverse-mode step of the hybrid scheme (D2Q9, double).
//
// Given the forward quantities of step n (Q, the predictor Q^P, density,
// body force and force-corrected velocity) and the adjoint (adj_f, adj_Q) of
// the state at step n+1, vjp_step forms the adjoint of the state at step n and
// accumulates the derivatives with respect to gamma, K and Gamma:
//   streaming and collision -> corrector rate at Q^P (and its H, Laplacian
//   and gradient stencils) -> predictor rate at Q -> velocity gradient and
//   force-corrected velocity -> body force and stress -> molecular field.
// Stencil adjoints are applied as gathers: the compact Laplacian is
// self-adjoint and the central difference D has adjoint -D on a periodic
// grid.
//
// One launch per reverse step, one block of 768 threads per tile of 16x16
// sites (40x4 on grids of few rows, rev_shape).  As in the single pass of the forward step, the stages run on rectangles that
// shrink by one site per gather (both rates on radius 3, collision and
// force-corrected velocity on 2, stress and molecular field on 1, the
// order-tensor adjoint on the tile) and hand their fields on in LDS, so a site
// reads 15 forward and 14 adjoint values and writes 14.  The corrector leaves
// its neighbours nothing that they cannot form themselves: with R^P's adjoint
// Rb = adj_Q/2, the adjoints of the Laplacian and the gradients at Q^P are
// K Gamma Rb and -u Rb, so only the adjoint and the velocity are shared and
// the two rates need no barrier between them.  As three kernels that passed
// about a hundred doubles per site through memory a reverse step of 256^2
// sites took 32.3 us, against 15.0 us in one.  The collision runs beside the
// rates, on waves of its own.  The adjoint is read and written in different
// buffers, since neighbouring tiles read each other's sites.
#pragma once

#include "lc_adjoint.h"
#include "lc_aux.h"
#include "lc_fused.h"

namespace lc {

// Scratch fields of the reverse step (double, N values per component): the
// forward recompute of a single step and the second adjoint buffers.
struct VjpFields {
  double *tau, *rho, *u, *F, *qp, *r;
  double *adj_f, *adj_q;
  double* part;  // [nblocks][3] parameter partials
  int64_t nblocks;
};
constexpr int VJP_COMPS = 4 + 1 + 2 + 2 + 5 + 5 + 9 + 5;

__device__ __forceinline__ void block_reduce3(double (&v)[3], double* __restrict__ dst) {
  __shared__ double part[16][3];
  const int tid = threadIdx.x + blockDim.x * (threadIdx.y + blockDim.y * threadIdx.z);
  const int lane = tid & 63, wid = tid >> 6;
  const int nw = (blockDim.x * blockDim.y * blockDim.z + 63) >> 6;
#pragma unroll
  for (int k = 0; k < 3; k++) v[k] = wave_sum(v[k]);
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < 3; k++) part[wid][k] = v[k];
  }
  __syncthreads();
  if (tid < 3) {
    double acc = part[0][tid];
    for (int w = 1; w < nw; w++) acc += part[w][tid];
    dst[tid] = acc;
  }
}

// zero the per-block parameter partials before a reverse call
__global__ void __launch_bounds__(256) vjp_zero(double* __restrict__ part, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    part[i] = 0.0;
}

#define LC_SITE_2D                                                       \
  const int x = blockIdx.x * blockDim.x + threadIdx.x;                   \
  const int y = blockIdx.y * blockDim.y + threadIdx.y;                   \
  const bool in = x < g.nx && y < g.ny;                                  \
  const int64_t N = g.N;                                                 \
  const int64_t s = in ? x + (int64_t)g.nx * y : 0;                      \
  const Nbr nb = neighbours(in ? x : 0, in ? y : 0, 0, g.nx, g.ny, 1);

// density, force-corrected velocity and body force from f and tau; f is
// either logical (pull == 0) or a population buffer in pull form
__global__ void __launch_bounds__(256) vjp_fwd_moments(const double* __restrict__ f, int pull,
                                                       const double* __restrict__ tau, VjpFields v, GridDims g) {
  LC_SITE_2D
  if (!in) return;
  double F[3];
  body_force<0, double>(tau, N, s, nb, F);
  double ff[9];
  if (pull) {
    gather_f<0, double>(f, N, s, nb, ff);
  } else {
#pragma unroll
    for (int i = 0; i < 9; i++) ff[i] = f[i * N + s];
  }
  double rho, u[3];
  moments<0, double, false>(ff, F, rho, u);
  v.rho[s] = rho;
  v.u[s] = u[0];
  v.u[N + s] = u[1];
  v.F[s] = F[0];
  v.F[N + s] = F[1];
}

// base + Laplacian of the first and minus the divergence of the other two of
// three five-component fields at a point, from their values at the point and
// its neighbours: at(f, c, o), field f (0: Laplacian adjoint, 1 and 2: adjoints
// of the x and y gradients), component c, o = 0 the point, 1..4 the neighbours
// x + 1, x - 1, y + 1, y - 1.
template <typename AT>
__device__ __forceinline__ Sym<double> gather_adj(const Sym<double>& base, AT at) {
  const double b[5] = {base.xx, base.xy, base.xz, base.yy, base.yz};
  double v[5];
#pragma unroll
  for (int c = 0; c < 5; c++) {
    const double lap = (at(0, c, 1) + at(0, c, 2)) + (at(0, c, 3) + at(0, c, 4)) - 4.0 * at(0, c, 0);
    const double div = -0.5 * ((at(1, c, 1) - at(1, c, 2)) + (at(2, c, 3) - at(2, c, 4)));
    v[c] = (b[c] + lap) + div;
  }
  return Sym<double>{v[0], v[1], v[2], v[3], v[4]};
}

// Velocity and its gradient at LDS point k.
template <int W, int RN>
__device__ __forceinline__ void velgrad_lds(const double (*u)[RN], int k, double (&G)[3][3], double (&uc)[3]) {
#pragma unroll
  for (int a = 0; a < 3; a++) {
    uc[a] = a < 2 ? u[a < 2 ? a : 0][k] : 0.0;
    G[a][0] = a < 2 ? 0.5 * (u[a < 2 ? a : 0][k + 1] - u[a < 2 ? a : 0][k - 1]) : 0.0;
    G[a][1] = a < 2 ? 0.5 * (u[a < 2 ? a : 0][k + W] - u[a < 2 ? a : 0][k - W]) : 0.0;
    G[a][2] = 0.0;
  }
}

// One reverse step.  adj_f, adj_q: the adjoint of the state at step n+1;
// out_f, out_q: that of step n.  Q, qp, rho, u, F: the forward quantities of
// step n.  The launch takes the tiles of the columns from g.xb on; the parameter
// partials of a block's own sites are added to part[block].
template <int TX, int TY>
__global__ void __launch_bounds__(REV_NTHR)
    vjp_step(const double* __restrict__ adj_f, const double* __restrict__ adj_q, double* __restrict__ out_f,
             double* __restrict__ out_q, const double* __restrict__ Q, const double* __restrict__ qp,
             const double* __restrict__ rho, const double* __restrict__ u, const double* __restrict__ F,
             double* __restrict__ part, TileDims g, Coef<double> c) {
  using L = Lattice<0>;
  using R4 = Rect<TX, TY, 4>;
  using R3 = Rect<TX, TY, 3>;
  using R2 = Rect<TX, TY, 2>;
  using R1 = Rect<TX, TY, 1>;
  // waves of the two roles
  constexpr int RATE_WAVES = (R3::N + 63) / 64, COLL_THR = REV_NTHR - RATE_WAVES * 64;
  constexpr int COLL_PTS = (R2::N + COLL_THR - 1) / COLL_THR;  // points per thread
  static_assert(R4::N <= REV_NTHR && COLL_THR > 0, "one point per thread and stage");
  __shared__ double sU[2][R4::N], sQ[5][R4::N];
  // Q^P and the order-tensor adjoint on radius 4, until the rates are taken;
  // then the molecular field's and stress's Laplacian and gradient adjoints on
  // radius 1
  __shared__ double sW[15 * R1::N > 10 * R4::N ? 15 * R1::N : 10 * R4::N];
  __shared__ double sG[4][R3::N];   // velocity-gradient adjoint
  __shared__ double sUb[2][R2::N];  // velocity adjoint
  __shared__ double sFb[2][R2::N];  // body-force adjoint
  __shared__ double sD[3][RATE_WAVES];  // parameter partials of the waves
  auto sP = reinterpret_cast<double(*)[R4::N]>(sW);
  auto sA = reinterpret_cast<double(*)[R4::N]>(sW + 5 * R4::N);
  auto sL = reinterpret_cast<double(*)[R1::N]>(sW);

  const int tid = threadIdx.x, wave = tid / 64;
  const int blk = xcd_remap(blockIdx.x + gridDim.x * blockIdx.y, gridDim.x * gridDim.y);
  const int x0 = g.xb + (blk % gridDim.x) * TX, y0 = (blk / gridDim.x) * TY;
  const size_t N = size_t(g.N);
  const bool near = g.nx >= R4::W && g.ny >= R4::H;  // the rectangle wraps at most once
  auto wrap = [&](int v, int n) { return near ? wrap_near(v, n) : wrapi(v, n); };

  // Q^P, u, Q and the adjoint on radius 4, one point per thread
  if (tid < R4::N) {
    const uint32_t s =
        uint32_t(wrap(x0 - 4 + tid % R4::W, g.nx)) + uint32_t(g.nx) * uint32_t(wrap(y0 - 4 + tid / R4::W, g.ny));
    double v[17];
#pragma unroll
    for (int k = 0; k < 5; k++) {
      v[k] = qp[k * N + s];
      v[5 + k] = adj_q[k * N + s];
      v[10 + k] = Q[k * N + s];
    }
    v[15] = u[s];
    v[16] = u[N + s];
#pragma unroll
    for (int k = 0; k < 5; k++) {
      sP[k][tid] = v[k];
      sA[k][tid] = v[5 + k];
      sQ[k][tid] = v[10 + k];
    }
    sU[0][tid] = v[15];
    sU[1][tid] = v[16];
  }

  // The two roles run on waves of their own and meet at the barriers, of which
  // both pass the same number; apart, neither holds registers for the other.
  if (wave >= RATE_WAVES) {
    // collision and force-corrected velocity at points of radius 2
    double fb[COLL_PTS][9], rhob[COLL_PTS], rh[COLL_PTS], u3[COLL_PTS][3], ubc[COLL_PTS][3];
    uint32_t s[COLL_PTS];
#pragma unroll
    for (int n = 0; n < COLL_PTS; n++) {
      const int kl = tid - RATE_WAVES * 64 + n * COLL_THR;
      if (kl >= R2::N) break;
      const int gx = wrap(x0 - 2 + kl % R2::W, g.nx), gy = wrap(y0 - 2 + kl / R2::W, g.ny);
      s[n] = uint32_t(gx) + uint32_t(g.nx) * uint32_t(gy);
      double fbs[9], F3[3] = {0, 0, 0}, Fb[3] = {0, 0, 0};
#pragma unroll
      for (int i = 0; i < 9; i++) {  // f'_i(x + c_i) = f*_i(x)
        const int tx = gx + L::cx(i), ty = gy + L::cy(i);
        const uint32_t t = uint32_t(tx < 0 ? g.nx - 1 : (tx == g.nx ? 0 : tx)) +
                           uint32_t(g.nx) * uint32_t(ty < 0 ? g.ny - 1 : (ty == g.ny ? 0 : ty));
        fbs[i] = adj_f[i * N + t];
        fb[n][i] = 0.0;
      }
      rh[n] = rho[s[n]];
      rhob[n] = 0.0;
#pragma unroll
      for (int a = 0; a < 3; a++) {
        u3[n][a] = a < 2 ? u[a * N + s[n]] : 0.0;
        if (a < 2) F3[a] = F[a * N + s[n]];
        ubc[n][a] = 0.0;
      }
      collide_vjp<0, double>(fbs, rh[n], u3[n], F3, c, fb[n], rhob[n], ubc[n], Fb);
      sFb[0][kl] = Fb[0];
      sFb[1][kl] = Fb[1];
    }
    // three threads add the block's parameter partials up at the end
    const int kd = tid - RATE_WAVES * 64;
    const double before = kd < 3 ? part[int64_t(blk) * 3 + kd] : 0.0;
    __syncthreads();  // 1
    __syncthreads();  // 2
    // adjoint of the force-corrected momentum: the velocity adjoint with the
    // velocity-gradient gather applied, over rho; the populations of the tile
    // and the body force (which enters u with weight 1/2)
#pragma unroll
    for (int n = 0; n < COLL_PTS; n++) {
      const int kl = tid - RATE_WAVES * 64 + n * COLL_THR;
      if (kl >= R2::N) break;
      const int i2 = kl % R2::W, j2 = kl / R2::W;
      const int k3 = (i2 + 1) + R3::W * (j2 + 1);
      double ubt[2], jb[2];
#pragma unroll
      for (int a = 0; a < 2; a++) {
        ubt[a] = (ubc[n][a] + sUb[a][kl]) - 0.5 * ((sG[2 * a][k3 + 1] - sG[2 * a][k3 - 1]) +
                                                   (sG[2 * a + 1][k3 + R3::W] - sG[2 * a + 1][k3 - R3::W]));
        jb[a] = ubt[a] / rh[n];
        sFb[a][kl] += 0.5 * jb[a];
      }
      if (i2 >= 2 && i2 < TX + 2 && j2 >= 2 && j2 < TY + 2 && x0 + i2 - 2 < g.nx && y0 + j2 - 2 < g.ny) {
        const double rb = rhob[n] - (ubt[0] * u3[n][0] + ubt[1] * u3[n][1]) / rh[n];
#pragma unroll
        for (int i = 0; i < 9; i++) out_f[i * N + s[n]] = fb[n][i] + rb + L::cx(i) * jb[0] + L::cy(i) * jb[1];
      }
    }
    __syncthreads();  // 3
    __syncthreads();  // 4
    if (kd < 3) {
      double acc = sD[kd][0];
#pragma unroll
      for (int w = 1; w < RATE_WAVES; w++) acc += sD[kd][w];
      part[int64_t(blk) * 3 + kd] = before + acc;
    }
  } else {
    // the order tensor at a point of radius 3
    const int i3 = tid % R3::W, j3 = tid / R3::W;
    auto within = [&](int r) {
      return tid < R3::N && i3 >= 3 - r && i3 < TX + 3 + r && j3 >= 3 - r && j3 < TY + 3 + r;
    };
    const bool own = within(0) && x0 + i3 - 3 < g.nx && y0 + j3 - 3 < g.ny;
    const int k4 = (i3 + 1) + R4::W * (j3 + 1);
    __syncthreads();  // 1

    // corrector Q' = Q + (R + R^P)/2 and predictor rate on radius 3
    Sym<double> qb = sym_zero<double>(), Rb = sym_zero<double>();
    double d[3] = {0.0, 0.0, 0.0};
    if (within(3)) {
      double ub[3] = {0, 0, 0}, Gb[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};
      Sym<double> Pb = sym_zero<double>();
      auto aq_at = [&]() { return Sym<double>{sA[0][k4], sA[1][k4], sA[2][k4], sA[3][k4], sA[4][k4]}; };
      {
        const Sym<double> aq = aq_at();
        const Sym<double> Rpb{0.5 * aq.xx, 0.5 * aq.xy, 0.5 * aq.xz, 0.5 * aq.yy, 0.5 * aq.yz};
        double G[3][3], uc[3];
        velgrad_lds<R4::W, R4::N>(sU, k4, G, uc);
        Sym<double> P, dP[3], LP, HPb = sym_zero<double>(), LPb;
        Sym<double> dPb[3] = {sym_zero<double>(), sym_zero<double>(), sym_zero<double>()};
        stencil_lds<double, 2, R4::W, R4::N>(sP, sP, sP, k4, P, dP, LP);
        const Sym<double> HP = molecular_field(P, LP, c);
        be_rate_vjp<2>(P, HP, dP, uc, G, Rpb, c, Pb, HPb, dPb, ub, Gb, d);
        molecular_field_vjp(P, LP, HPb, c, Pb, LPb, d);
      }
      // what both rates read is read from LDS again rather than held: the
      // operands of the two do not fit the registers together
      asm volatile("" ::: "memory");
      {
        const Sym<double> aq = aq_at();
        const int off[5] = {k4, k4 + 1, k4 - 1, k4 + R4::W, k4 - R4::W};
        const Sym<double> qpb = gather_adj(Pb, [&](int f, int k, int o) {
          const double rp = 0.5 * sA[k][off[o]];
          return f == 0 ? c.K * (c.Gam * rp) : -sU[f - 1][off[o]] * rp;
        });
        Rb = Sym<double>{0.5 * aq.xx + qpb.xx, 0.5 * aq.xy + qpb.xy, 0.5 * aq.xz + qpb.xz, 0.5 * aq.yy + qpb.yy,
                         0.5 * aq.yz + qpb.yz};
        qb = Sym<double>{aq.xx + qpb.xx, aq.xy + qpb.xy, aq.xz + qpb.xz, aq.yy + qpb.yy, aq.yz + qpb.yz};
      }
      asm volatile("" ::: "memory");
      {
        double G[3][3], uc[3];
        velgrad_lds<R4::W, R4::N>(sU, k4, G, uc);
        Sym<double> q, dq[3], Lq, Hb = sym_zero<double>();
        Sym<double> dqb[3] = {sym_zero<double>(), sym_zero<double>(), sym_zero<double>()};
        stencil_lds<double, 2, R4::W, R4::N>(sQ, sQ, sQ, k4, q, dq, Lq);
        const Sym<double> H = molecular_field(q, Lq, c);
        be_rate_vjp<2>(q, H, dq, uc, G, Rb, c, qb, Hb, dqb, ub, Gb, d);
      }
      sG[0][tid] = Gb[0][0];
      sG[1][tid] = Gb[0][1];
      sG[2][tid] = Gb[1][0];
      sG[3][tid] = Gb[1][1];
      if (within(2)) {
        const int k2 = (i3 - 1) + R2::W * (j3 - 1);
        sUb[0][k2] = ub[0];
        sUb[1][k2] = ub[1];
      }
    }
    __syncthreads();  // 2
    __syncthreads();  // 3

    // body force, stress and molecular field on radius 1
    if (within(1)) {
      const int k2 = (i3 - 1) + R2::W * (j3 - 1);
      double tb[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};
#pragma unroll
      for (int a = 0; a < 2; a++) {
        tb[a][0] = -0.5 * (sFb[a][k2 + 1] - sFb[a][k2 - 1]);
        tb[a][1] = -0.5 * (sFb[a][k2 + R2::W] - sFb[a][k2 - R2::W]);
      }
      const double ux = sU[0][k4], uy = sU[1][k4];
      // the rate's adjoints of H and of the gradients
      Sym<double> Hb{c.Gam * Rb.xx, c.Gam * Rb.xy, c.Gam * Rb.xz, c.Gam * Rb.yy, c.Gam * Rb.yz};
      Sym<double> dqb[3] = {Sym<double>{-ux * Rb.xx, -ux * Rb.xy, -ux * Rb.xz, -ux * Rb.yy, -ux * Rb.yz},
                            Sym<double>{-uy * Rb.xx, -uy * Rb.xy, -uy * Rb.xz, -uy * Rb.yy, -uy * Rb.yz},
                            sym_zero<double>()};
      Sym<double> q, dq[3], Lq, Lb;
      stencil_lds<double, 2, R4::W, R4::N>(sQ, sQ, sQ, k4, q, dq, Lq);
      const Sym<double> H = molecular_field(q, Lq, c);
      stress_vjp<2>(q, H, dq, tb, c, qb, Hb, dqb, d);
      const int k1 = (i3 - 2) + R1::W * (j3 - 2);
#pragma unroll
      for (int n = 0; n < 2; n++) {
        sL[5 * n + 5][k1] = dqb[n].xx;
        sL[5 * n + 6][k1] = dqb[n].xy;
        sL[5 * n + 7][k1] = dqb[n].xz;
        sL[5 * n + 8][k1] = dqb[n].yy;
        sL[5 * n + 9][k1] = dqb[n].yz;
      }
      molecular_field_vjp(q, Lq, Hb, c, qb, Lb, d);
      sL[0][k1] = Lb.xx;
      sL[1][k1] = Lb.xy;
      sL[2][k1] = Lb.xz;
      sL[3][k1] = Lb.yy;
      sL[4][k1] = Lb.yz;
    }
    // the parameter derivatives count at the block's own sites
#pragma unroll
    for (int k = 0; k < 3; k++) {
      const double sum = wave_sum(own ? d[k] : 0.0);
      if (tid % 64 == 0) sD[k][wave] = sum;
    }
    __syncthreads();  // 4
    if (own) {
      const int k1 = (i3 - 2) + R1::W * (j3 - 2);
      const int off[5] = {k1, k1 + 1, k1 - 1, k1 + R1::W, k1 - R1::W};
      const Sym<double> o = gather_adj(qb, [&](int f, int k, int n) { return sL[5 * f + k][off[n]]; });
      store_sym(out_q, int64_t(N), int64_t(x0 + i3 - 3) + int64_t(g.nx) * (y0 + j3 - 3), o);
    }
  }
}

// adjoint back into the caller's buffers (9 and 5 components)
__global__ void __launch_bounds__(256) vjp_copy(const double* __restrict__ f, const double* __restrict__ q,
                                                double* __restrict__ fo, double* __restrict__ qo, int64_t N) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < 9 * N; i += (int64_t)gridDim.x * blockDim.x) {
    fo[i] = f[i];
    if (i < 5 * N) qo[i] = q[i];
  }
}

// parameter partials of the blocks, added to dparams: each thread
// sums a fixed strided subset, then a fixed-order block reduction
// (deterministic for a fixed launch shape).
__global__ void __launch_bounds__(256) vjp_params(const double* __restrict__ part, int64_t nblocks,
                                                  double* __restrict__ dparams) {
  double v[3] = {0.0, 0.0, 0.0};
  for (int64_t b = threadIdx.x; b < nblocks; b += blockDim.x) {
#pragma unroll
    for (int k = 0; k < 3; k++) v[k] += part[b * 3 + k];
  }
  __shared__ double tot[3];
  block_reduce3(v, tot);
  __syncthreads();
  if (threadIdx.x < 3) dparams[threadIdx.x] += tot[threadIdx.x];
}

}  // namespace lc
