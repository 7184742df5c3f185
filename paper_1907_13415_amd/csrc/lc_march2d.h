// lc_march2d.h -- the step of a large two-dimensional grid in one pass, one
// wave per strip.
//
// A wave owns a strip of 56 columns (one column per lane, four more lanes of
// halo on either side) and marches along y through a chunk of rows.  The
// stages run on lagged rows of the march: with Q row p newest, the stress of
// row p-1, the body force, moments and collision of row p-2, the predictor of
// row p-3 and the corrector of row p-4 (Sec. 1.2.2).  Neighbours in x are the
// neighbouring lanes (DPP wave shifts, an operand of the instruction that uses
// them), neighbours in y the lane's own registers of earlier rows, so there is
// no barrier and no block: every stage is evaluated once per site, but for the
// halo lanes (64 for 56) and the rows a chunk repeats (six of stress down to
// none of the corrector).  f and Q are read once and written once.
//
// The arithmetic is that of the two sweeps and of the tiled single pass, in
// the same order (bit-identical); the gradient, Laplacian and molecular field
// of Q that the stress needs are kept (in LDS, each lane its own) for the
// predictor, which needs the same.
#pragma once

#include "lc_launch.h"
#include "lc_split.h"

namespace lc {

// Value of the lane to the right (D = 1) or left (D = -1); zero beyond the wave.
template <int D>
__device__ __forceinline__ int lane_shift_bits(int v) {
  static_assert(D == 1 || D == -1, "one lane");
  // wave_shl:1 takes the value of the next lane, wave_shr:1 of the one before
  return __builtin_amdgcn_update_dpp(0, v, D == 1 ? 0x130 : 0x138, 0xf, 0xf, true);
}
template <int D>
__device__ __forceinline__ float lane_shift(float v) {
  return __int_as_float(lane_shift_bits<D>(__float_as_int(v)));
}
template <int D>
__device__ __forceinline__ double lane_shift(double v) {
  return __hiloint2double(lane_shift_bits<D>(__double2hiint(v)), lane_shift_bits<D>(__double2loint(v)));
}

// v(x + cx) of a value held per lane.
template <typename S>
__device__ __forceinline__ S lane_at(S v, int cx) {
  return cx > 0 ? lane_shift<1>(v) : (cx < 0 ? lane_shift<-1>(v) : v);
}

// Gradients (undivided: times two) and Laplacian of NC components from three
// rows held per lane, with the sums of stencil_lds and stencil_lds_iso2.
template <typename S, int ST, int NC>
__device__ __forceinline__ void row_stencil(const S (&ym)[NC], const S (&c)[NC], const S (&yp)[NC], S (&dx)[NC],
                                            S (&dy)[NC], S (&lap)[NC]) {
  using L = Lattice<0>;
#pragma unroll
  for (int q = 0; q < NC; q++) {
    if constexpr (ST == STENCIL_ISO) {
      S gx = S(0), gy = S(0), l = S(0);
#pragma unroll
      for (int i = 1; i < L::q; i++) {
        if (L::opp(i) < i) continue;
        const int cx = L::cx(i), cy = L::cy(i);
        const S vp = lane_at(cy > 0 ? yp[q] : (cy < 0 ? ym[q] : c[q]), cx);
        const S vm = lane_at(cy > 0 ? ym[q] : (cy < 0 ? yp[q] : c[q]), -cx);
        const S wg = S(6.0 * L::w(i)), wl = S(6.0 * L::w(i));
        const S dif = vp - vm, sum = vp + vm;
        if (cx != 0) gx += (cx > 0 ? wg : -wg) * dif;
        if (cy != 0) gy += (cy > 0 ? wg : -wg) * dif;
        l += wl * sum;
      }
      dx[q] = gx;
      dy[q] = gy;
      lap[q] = l - S(6.0 * (1.0 - L::w(0))) * c[q];
    } else {
      const S xp = lane_shift<1>(c[q]), xm = lane_shift<-1>(c[q]);
      dx[q] = xp - xm;
      dy[q] = yp[q] - ym[q];
      const S l = (xp + xm) + (yp[q] + ym[q]);
      lap[q] = l - S(4) * c[q];
    }
  }
}

template <typename S>
__device__ __forceinline__ Sym<S> as_sym(const S (&v)[5]) {
  return Sym<S>{v[0], v[1], v[2], v[3], v[4]};
}

// The strip of columns from x0 on, rows yb .. ye-1 (ye <= ny).
template <typename S, bool DEV, bool MRT, typename QT, bool SR, int ST>
__device__ __forceinline__ void march2d_body(const QT* __restrict__ Qin, const S* __restrict__ fin,
                                             S* __restrict__ fout, QT* __restrict__ Qout, const GridDims& g,
                                             const Coef<S>& c, const Coef<QT>& cq, int x0, int yb, int ye,
                                             uint32_t srkey) {
  using L = Lattice<0>;
  constexpr bool ISO = ST == STENCIL_ISO;
  const int lane = threadIdx.x;
  const int x = x0 - MARCH_HALO + lane;
  const bool own = lane >= MARCH_HALO && lane < MARCH_HALO + MARCH_COLS && x < g.nx;
  // Byte offsets of the lane's column and its two neighbours, and the arrays'
  // component bases: an access is a uniform base and one 32-bit offset per lane
  // that carries the row as well (rows of a grid of at most 2^32 bytes a
  // component), so it needs no address arithmetic of its own.
  const size_t N = size_t(g.N);
  const int xc = wrapi(x, g.nx);
  const uint32_t qx = uint32_t(xc) * uint32_t(sizeof(QT)), qrow = uint32_t(g.nx) * uint32_t(sizeof(QT));
  const uint32_t frow = uint32_t(g.nx) * uint32_t(sizeof(S));
  const uint32_t fx[3] = {uint32_t(xc == 0 ? g.nx - 1 : xc - 1) * uint32_t(sizeof(S)),
                          uint32_t(xc) * uint32_t(sizeof(S)),
                          uint32_t(xc + 1 == g.nx ? 0 : xc + 1) * uint32_t(sizeof(S))};
  auto in_bytes = [](const auto* base, uint32_t off) {
    return *reinterpret_cast<decltype(base)>(reinterpret_cast<const char*>(base) + off);
  };
  // periodic index of the row after periodic row y
  auto after = [&](int y) { return y + 1 == g.ny ? 0 : y + 1; };

  struct Rows {
    QT v[5];
  };
  // What the stress of a row leaves for its predictor two iterations later,
  // in the lane's own LDS words: the undivided gradients, Q and H (or the
  // Laplacian, where the predictor's H is summed in double).  Held in registers
  // it would cost 40 of them.
  constexpr int PV = 16 / sizeof(QT), NPACK = 20 / PV;
  struct alignas(16) Pack {
    QT v[PV];
  };
  __shared__ Pack kept[3][NPACK][64];
  auto keep = [&](int slot, const QT (&v)[20]) {
#pragma unroll
    for (int n = 0; n < NPACK; n++) {
      Pack p;
#pragma unroll
      for (int k = 0; k < PV; k++) p.v[k] = v[n * PV + k];
      kept[slot][n][lane] = p;
    }
  };
  auto recall = [&](int slot, QT (&v)[20]) {
#pragma unroll
    for (int n = 0; n < NPACK; n++) {
      const Pack p = kept[slot][n][lane];
#pragma unroll
      for (int k = 0; k < PV; k++) v[n * PV + k] = p.v[k];
    }
  };
  struct Stash {  // what the corrector takes over from the predictor
    Sym<QT> r, q;
    Flow<QT, 2> fl;
  };
  auto fetch_q = [&](int y, Rows& r) {
    const uint32_t off = qx + qrow * uint32_t(y);
#pragma unroll
    for (int q = 0; q < 5; q++) r.v[q] = in_bytes(Qin + size_t(q) * N, off);
  };
  // populations of a row, given it and the rows around it: f_i(x) = buf_i(x - c_i)
  auto fetch_f = [&](int below, int y, int above, S (&f)[L::q]) {
    const uint32_t at[3] = {frow * uint32_t(below), frow * uint32_t(y), frow * uint32_t(above)};
#pragma unroll
    for (int i = 0; i < L::q; i++) f[i] = in_bytes(fin + size_t(i) * N, at[1 - L::cy(i)] + fx[1 - L::cx(i)]);
  };

  // undivided gradients enter the elastic stress squared: K/4 there
  Coef<QT> c4 = cq;
  c4.K = cq.K * QT(0.25);

  // Rows in rings of three, indexed by the row modulo 3 (counted from the
  // march's start): slot K is that of rows p and p-3, K+1 of p-2 and p-5, K+2
  // of p-1 and p-4.
  Rows Q[3], P[3];
  QT t[3][2][2], u[3][2];
  Stash st[3];
  // Rows in flight, AHEAD iterations before their use: a load returns only
  // after the stores issued before it, and one iteration (about 2 us) is not
  // always enough.  2048^2 sites: FP32 142 us with one, 126 with two and 127
  // with three; FP64, whose one wave per SIMD has nothing beside it, 258 with
  // two and 238 with three; 1024^2 in the mixed form 41.7 with two and 43.7
  // with three.
  constexpr int AHEAD = sizeof(S) == 8 ? 3 : 2;
  Rows qn[3];
  S f[3][L::q];
  // periodic indices of rows p-3+AHEAD .. p-1+AHEAD (of populations) and
  // p+AHEAD (of Q)
  int wq = wrapi(yb - 4, g.ny);
  fetch_q(wq, Q[1]);
  fetch_q(wq = after(wq), Q[2]);
#pragma unroll
  for (int n = 0; n < AHEAD; n++) fetch_q(wq = after(wq), qn[n]);
  wq = after(wq);
  int w0 = wrapi(yb - 3, g.ny), w1 = after(w0), w2 = after(w1);
  if constexpr (AHEAD == 3) {
    fetch_f(w0, w1, w2, f[0]);
    w0 = w1;
    w1 = w2;
    w2 = after(w2);
  }

  auto iteration = [&](auto slot, int p) {
    constexpr int K0 = decltype(slot)::value, K1 = (K0 + 1) % 3, K2 = (K0 + 2) % 3;
    Q[K0] = qn[K0];
    S fc[L::q];
#pragma unroll
    for (int i = 0; i < L::q; i++) fc[i] = f[K1][i];
    if (p + AHEAD <= ye + 3) fetch_q(wq, qn[AHEAD == 3 ? K0 : K2]);
    if (p + AHEAD <= ye + 3) fetch_f(w0, w1, w2, f[AHEAD == 3 ? K1 : K0]);
    wq = after(wq);
    w0 = w1;
    w1 = w2;
    w2 = after(w2);

    // stress of row p-1
    {
      QT dx[5], dy[5], lap[5];
      row_stencil<QT, ST, 5>(Q[K1].v, Q[K2].v, Q[K0].v, dx, dy, lap);
      const Sym<QT> q = as_sym(Q[K2].v), Lq = as_sym(lap);
      const Sym<QT> H = molecular_field(q, Lq, cq);
      const Sym<QT> d[3] = {as_sym(dx), as_sym(dy), sym_zero<QT>()};
      QT tau[3][3];
      stress(q, H, d, c4, tau);
#pragma unroll
      for (int a = 0; a < 2; a++)
#pragma unroll
        for (int b = 0; b < 2; b++) t[K2][a][b] = tau[a][b];
      const Sym<QT> h = SR ? Lq : H;
      keep(K2, {dx[0], dx[1], dx[2], dx[3], dx[4], dy[0], dy[1], dy[2], dy[3], dy[4], q.xx, q.xy, q.xz, q.yy, q.yz,
                h.xx, h.xy, h.xz, h.yy, h.yz});
    }
    // body force, moments and collision of row p-2
    if (p >= yb) {
      S F[3] = {S(0), S(0), S(0)};
#pragma unroll
      for (int a = 0; a < 2; a++) {
        if constexpr (ISO) {  // F_a = 3 sum_i w_i sum_b c_ib tau_ab(x + c_i), over pairs
          QT acc = QT(0);
#pragma unroll
          for (int i = 1; i < L::q; i++) {
            if (L::opp(i) < i) continue;
            const int cx = L::cx(i), cy = L::cy(i);
            QT dsum = QT(0);
#pragma unroll
            for (int b = 0; b < 2; b++) {
              const int cb = b == 0 ? cx : cy;
              if (cb == 0) continue;
              const QT dt = lane_at(t[cy > 0 ? K2 : (cy < 0 ? K0 : K1)][a][b], cx) -
                            lane_at(t[cy > 0 ? K0 : (cy < 0 ? K2 : K1)][a][b], -cx);
              dsum += cb > 0 ? dt : -dt;
            }
            acc += QT(3.0 * L::w(i)) * dsum;
          }
          F[a] = S(acc);
        } else {
          const QT acc = (lane_shift<1>(t[K1][a][0]) - lane_shift<-1>(t[K1][a][0])) + (t[K2][a][1] - t[K0][a][1]);
          F[a] = S(QT(0.5) * acc);
        }
      }
      S rho, mass, us[3];
      moments<0, S, DEV>(fc, F, rho, us, mass);
      u[K1][0] = QT(us[0]);
      u[K1][1] = QT(us[1]);
      if (p - 2 >= yb && p - 2 < ye) {
        if constexpr (MRT)
          collide_mrt<0, S, DEV>(fc, rho, mass, us, F, c);
        else
          collide_pairs<0, S, DEV>(fc, rho, mass, us, F, c);
        if (own) {
          const uint32_t off = fx[1] + frow * uint32_t(p - 2);
#pragma unroll
          for (int i = 0; i < L::q; i++)
            *reinterpret_cast<S*>(reinterpret_cast<char*>(fout + size_t(i) * N) + off) = fc[i];
        }
      }
    }
    // predictor of row p-3
    if (p >= yb + 2) {
      QT k[20];
      recall(K0, k);
      const Sym<QT> q{k[10], k[11], k[12], k[13], k[14]}, h{k[15], k[16], k[17], k[18], k[19]};
      const Sym<QT> H = SR ? molecular_field_exact(q, h, cq) : h;
      const Sym<QT> d[3] = {Sym<QT>{k[0], k[1], k[2], k[3], k[4]}, Sym<QT>{k[5], k[6], k[7], k[8], k[9]},
                            sym_zero<QT>()};
      QT gx[2], gy[2], G[3][3];
      if constexpr (ISO) {  // undivided: 6 sum_i w_i c_ib u_a(x + c_i), over pairs
        QT lap[2];
        row_stencil<QT, ST, 2>(u[K2], u[K0], u[K1], gx, gy, lap);
      } else {
#pragma unroll
        for (int a = 0; a < 2; a++) {
          gx[a] = lane_shift<1>(u[K0][a]) - lane_shift<-1>(u[K0][a]);
          gy[a] = u[K1][a] - u[K2][a];
        }
      }
#pragma unroll
      for (int a = 0; a < 3; a++) {
        G[a][0] = a < 2 ? gx[a < 2 ? a : 0] : QT(0);
        G[a][1] = a < 2 ? gy[a < 2 ? a : 0] : QT(0);
        G[a][2] = QT(0);
      }
      const QT uh[3] = {u[K0][0] * QT(0.5), u[K0][1] * QT(0.5), QT(0)};
      Stash& s = st[K0];
      s.fl = flow_terms<QT, true, 2>(uh, G, cq);
      s.r = be_rate_flow<QT, true, 2>(q, H, d, s.fl, cq);
      s.q = q;
      P[K0] = Rows{{q.xx + s.r.xx, q.xy + s.r.xy, q.xz + s.r.xz, q.yy + s.r.yy, q.yz + s.r.yz}};
    }
    // corrector of row p-4
    if (p >= yb + 4) {
      const Stash& s = st[K2];
      QT dx[5], dy[5], lap[5];
      row_stencil<QT, ST, 5>(P[K1].v, P[K2].v, P[K0].v, dx, dy, lap);
      const Sym<QT> pc = as_sym(P[K2].v), Lp = as_sym(lap);
      const Sym<QT> H = SR ? molecular_field_exact(pc, Lp, cq) : molecular_field(pc, Lp, cq);
      const Sym<QT> d[3] = {as_sym(dx), as_sym(dy), sym_zero<QT>()};
      const Sym<QT> Rp = be_rate_flow<QT, true, 2>(pc, H, d, s.fl, cq);
      if (own) store_q_update<QT, SR, false>(Qout, g.N, uint32_t(x) + uint32_t(g.nx) * uint32_t(p - 4), s.q, s.r, Rp, srkey);
    }
  };
  for (int p = yb - 2; p <= ye + 3; p += 3) {
    iteration(std::integral_constant<int, 0>{}, p);
    if (p + 1 <= ye + 3) iteration(std::integral_constant<int, 1>{}, p + 1);
    if (p + 2 <= ye + 3) iteration(std::integral_constant<int, 2>{}, p + 2);
  }
}

template <typename S, bool DEV, bool MRT, typename QT, bool SR, int ST = STENCIL_COMPACT>
__global__ void __launch_bounds__(64)
    march2d_step(const QT* __restrict__ Qin, const S* __restrict__ fin, S* __restrict__ fout, QT* __restrict__ Qout,
                 GridDims g, Coef<S> c, Coef<QT> cq, int cols, int rows, uint32_t srkey) {
  const int t = xcd_remap(blockIdx.x, gridDim.x);
  const int yb = (t / cols) * rows;
  march2d_body<S, DEV, MRT, QT, SR, ST>(Qin, fin, fout, Qout, g, c, cq, (t % cols) * MARCH_COLS, yb,
                                        min(yb + rows, g.ny), srkey);
}

}  // namespace lc
