// One RK stage with one thread per cell: the passes of the z-march
// (mhd_zmarch.hip, mhd_zfinal.hip) for contexts too small to fill the device
// with marching workgroups.
//
// A march is a serial chain: every plane costs a workgroup two or three
// barriers and as many trips to memory (2.5 us a plane), and each chunk
// recomputes some planes of lead-in, 8 launches a stage.  While the
// arrays fit in the caches, the same quantities are cheaper read by every
// cell from its neighbours: 7 launches without a barrier.  Each expression is
// the march's own, in its order (z divergences summed over planes k-3..k+3
// as the march scatters them), so both paths give the same bits.
#include <hip/hip_runtime.h>

#include "mhd_cell.hpp"
#include "mhd_zmarch.hpp"
#include "mhd_zstage.hpp"

namespace smhd {
namespace {

template <class T> struct CK {
  const BoxDev* boxes;
  const Blk* tab;
  int nblk;
  CP8<T> f;
  ZWork<T> ws;
  Phys<T> ph;
  const T* zt;
  const T* lnavg;
  int stretched;            // some box is: pass F scales by the planes' Jacobians
  CPart* cpart;             // per block, or null
  P8<T> du;
  int du_mode;
  P8<T> f_out;
  T alpha;
  double beta;
  const double* dt_dev;
  double dt_host;
};

#define CELL_BEGIN                                                                     \
  const int per_ = (K.nblk + 7) >> 3;                                                  \
  const int bi_ = (int)(blockIdx.x & 7u) * per_ + (int)(blockIdx.x >> 3);              \
  if (bi_ >= K.nblk) return;                                                           \
  const Blk tb_ = K.tab[bi_];                                                          \
  const BoxDev& b = K.boxes[tb_.box];                                                  \
  const bool own = (int)threadIdx.x < tb_.n;                                           \
  const Cell<T, W> c(b, (unsigned)tb_.start + (own ? threadIdx.x : 0u), K.zt);         \
  auto A = [&](int id) -> T* { return K.ws.arr(id) + b.off; };                         \
  auto F = [&](int v) -> const T* { return K.f.p[v] + b.off; };                        \
  const Phys<T>& ph = K.ph;                                                            \
  const unsigned tm = ph.terms;                                                        \
  const bool inside = !c.walled() || (c.k >= b.g0 && c.k < b.g1);                      \
  (void)A; (void)F; (void)tm; (void)own; (void)inside;

#define CELL_KERNEL template <class T, bool W> __global__ __launch_bounds__(kBlock) void

// Face velocities, x and y face densities, e_m and its log.
CELL_KERNEL k_cprim(CK<T> K) {
  CELL_BEGIN
  if (!own) return;
  const T* rho = F(0);
  const T rx = c.template dn<X>(rho), ry = c.template dn<Y>(rho), rz = c.template dn<Z>(rho);
  c.st(A(WC_RX), rx);
  c.st(A(WC_RY), ry);
  c.st(A(WC_UX), c.ld(F(1)) / rx);
  c.st(A(WC_UY), c.ld(F(2)) / ry);
  c.st(A(WS_UZ), c.ld(F(3)) / rz);
  const T em = c.ld(F(4)) / c.ld(rho);
  c.st(A(WC_EM), em);
  c.st(A(WC_LEM), log(em));
}

// div u and the speed-like viscosity (pass A1), with the block's largest
// wave speed.
CELL_KERNEL k_cnus(CK<T> K) {
  __shared__ double sh[kBlock];
  CELL_BEGIN
  const T ubx = c.template up<X>(A(WC_UX)), uby = c.template up<Y>(A(WC_UY)), ubz = c.template up<Z>(A(WS_UZ));
  const T dxy = c.template dup<X>(A(WC_UX)) + c.template dup<Y>(A(WC_UY));
  const T dzz = c.template dup<Z>(A(WS_UZ));
  const T bbx = c.template up<X>(F(5)), bby = c.template up<Y>(F(6)), bbz = c.template up<Z>(F(7));
  const T rq = c.ld(F(0)), eq = c.ld(F(4));
  const T D = dxy + dzz;
  const T P = ph.gamma1 * eq;
  const T cs = sqrt(ph.gamma * P / rq);
  const T bb = norm3(bbx, bby, bbz);
  const T ca = bb / sqrt(ph.mu * rq);
  T nus;
  if (ph.nu_const > T(0)) {
    nus = ph.nu_const / T(b.hmin);
  } else {
    const T relu = -D > T(0) ? -D : T(0);
    nus = ph.nu1 * norm3(ubx, uby, ubz) + ph.nu3 * (cs + ca) + ph.nu2 * c.plane(ZJ_H) * relu;
  }
  if (own) {
    c.st(A(WS_NUS), nus);
    c.st(A(WS_D), D);
    if (tm & T_DIVB)
      c.st(A(WS_DIVB), (c.template dup<X>(F(5)) + c.template dup<Y>(F(6))) + c.template dup<Z>(F(7)));
  }
  if (!K.cpart) return;
  double cmax = 0.0;
  if (own && inside) {
    const double ux_ = ubx, uy_ = uby, uz_ = ubz;
    const double bx_ = bbx, by_ = bby, bz_ = bbz, bbd = bb;
    const double udotb = bbd > 0.0 ? (ux_ * bx_ + uy_ * by_ + uz_ * bz_) / bbd : 0.0;
    const double uu = ux_ * ux_ + uy_ * uy_ + uz_ * uz_;
    const double up = sqrt(fmax(uu - udotb * udotb, 0.0));
    cmax = fmax(cmax, (double)cs + (double)ca + up);
  }
  const double m = block_max<kBlock>(cmax, sh);
  if (threadIdx.x == 0) K.cpart[bi_].cmax = m;
}

// Pass A2: the maximum over 3x3x3 (or, H = 2, 5x5x5) cells, then the
// three-cell means, the floor and ln, with the block's largest viscosity.
template <class T, bool W, int H> __global__ __launch_bounds__(kBlock) void k_cmax(CK<T> K) {
  CELL_BEGIN
  if (!own) return;
  const T* a = A(WS_NUS);
  T m = c.ld(a);
#pragma unroll
  for (int z = -H; z <= H; ++z) {
    if (!c.has(z)) continue;
#pragma unroll
    for (int y = -H; y <= H; ++y)
#pragma unroll
      for (int x = -H; x <= H; ++x) m = fmax(m, c.ld(a, c.d[X][x + 3] + c.d[Y][y + 3] + c.d[Z][z + 3]));
  }
  c.st(A(WC_M), m);
}
CELL_KERNEL k_cmean(CK<T> K) {
  __shared__ double sh[kBlock];
  CELL_BEGIN
  const T* a = A(WC_M);
  auto plane = [&](unsigned o) {
    T sx[3];
#pragma unroll
    for (int y = -1; y <= 1; ++y) {
      const unsigned f = o + c.d[Y][y + 3];
      sx[y + 1] = (c.ld(a, f + c.d[X][2]) + c.ld(a, f) + c.ld(a, f + c.d[X][4])) / T(3);
    }
    return (sx[0] + sx[1] + sx[2]) / T(3);
  };
  T s = plane(0u);
  int cnt = 1;
  if (c.has(-1)) { s = plane(c.d[Z][2]) + s; cnt = 2; }
  if (c.has(1)) { s = s + plane(c.d[Z][4]); ++cnt; }
  T v = s / T(cnt);
  v = v > T(1e-30) ? v : T(1e-30);
  if (own) {
    const T l = log(v);
    c.st(A(WS_LNT), l);
    c.st(A(WC_NU), exp(l));
  }
  if (!K.cpart) return;
  const double m = block_max<kBlock>(own && inside ? (double)v : 0.0, sh);
  if (threadIdx.x == 0) K.cpart[bi_].numax = m;
}
CELL_KERNEL k_clines(CK<T> K) {
  CELL_BEGIN
  if (!own) return;
  c.st(A(WC_XL), c.template dn<X>(A(WS_LNT)));
  c.st(A(WC_YL), c.template dn<Y>(A(WS_LNT)));
}

// Pass Q, the edge along y (AX = X: with the x-derivatives) or along x (AX =
// Y); the outputs of both in QOUT order.
template <int AX, class T, bool W, class FA, class FF>
__device__ __forceinline__ void zedge_pair(const Cell<T, W>& c, const CK<T>& K, const FA& A, const FF& F) {
  const Phys<T>& ph = K.ph;
  const unsigned tm = ph.terms;
  const bool visc = tm & T_VISC, res = tm & T_RESIST, ind = tm & T_INDUCT, lor = tm & T_LORENTZ,
             adv = tm & T_ADV;
  const bool need_nu = visc || (res && !(ph.eta_const > T(0)));
  const T inv_mu = ph.inv_mu;
  const int U = AX == X ? WC_UX : WC_UY, R = AX == X ? WC_RX : WC_RY, L = AX == X ? WC_XL : WC_YL;
  const T zR = c.template dn<Z>(A(R));
  const T zP = c.template dn<Z>(F(1 + AX));
  const T zU = c.template dn<Z>(A(U));
  const T dzU = c.template ddn<Z>(A(U));
  const T zB = c.template dn<Z>(F(5 + AX));
  const T dzB = c.template ddn<Z>(F(5 + AX));
  const T aU = c.template dn<AX>(A(WS_UZ));
  const T daU = c.template ddn<AX>(A(WS_UZ));
  const T aB = c.template dn<AX>(F(7));
  const T daB = c.template ddn<AX>(F(7));
  const T aP = c.template dn<AX>(F(3));
  T n = T(0), t = T(0), s = T(0);
  if (need_nu) n = c.plane(AX == X ? ZJ_LXZ : ZJ_LYZ) * exp(c.template dn<Z>(A(L)));
  if (visc) {
    s = T(0.5) * (dzU + daU);
    t = zR * n * s;
  }
  const T eta = ph.eta_const > T(0) ? ph.eta_const : ph.nuB * n;
  T j, e = T(0);
  if constexpr (AX == X) {
    j = dzB - daB;
    if (ind) e = e - (aU * zB - zU * aB);
  } else {
    j = daB - dzB;
    if (ind) e = e - (zU * aB - aU * zB);
  }
  if (res) e = e + eta * j;
  T ga = t, gz = t;
  if (adv) {
    ga = ga - zP * aU;
    gz = gz - aP * zU;
  }
  T q = visc ? T(2) * t * s : T(0);
  if (res) q = q + eta * j * j * inv_mu;
  const int o = WS_Q0 + (AX == X ? QOUT_GXZ : QOUT_GYZ);
  c.st(A(o), ga);
  c.st(A(o + 1), gz);
  c.st(A(o + 2), e);
  c.st(A(o + 3), lor ? j * aB : T(0));
  c.st(A(o + 4), lor ? j * zB : T(0));
  c.st(A(o + 5), q);
}

// Passes Q and P, one group of outputs per blockIdx.y.
CELL_KERNEL k_cedges(CK<T> K) {
  CELL_BEGIN
  if (!own) return;
  const bool lnp = (tm & T_PRES) && (tm & T_LNP);
  const T* pav = K.ws.lnpav + b.poff;
  const T lpa = lnp ? pav[c.k] : T(0);
  auto in = [&](const T* a, int x, int y) { return c.ld(a, c.d[X][x + 3] + c.d[Y][y + 3]); };
  auto S = [&](int q, int x, int y) -> T {
    switch (q) {
      case DQ_PX: return in(F(1), x, y);
      case DQ_PY: return in(F(2), x, y);
      case DQ_E: return in(F(4), x, y);
      case DQ_BX: return in(F(5), x, y);
      case DQ_BY: return in(F(6), x, y);
      case DQ_UX: return in(A(WC_UX), x, y);
      case DQ_UY: return in(A(WC_UY), x, y);
      case DQ_NU: return in(A(WC_NU), x, y);
      case DQ_EM: return in(A(WC_EM), x, y);
      case DQ_LEM: return in(A(WC_LEM), x, y);
      case DQ_RXD: return in(A(WC_RX), x, y);
      case DQ_RYD: return in(A(WC_RY), x, y);
      case DQ_XL: return in(A(WC_XL), x, y);
      case DQ_RHO: return c.ld(F(0));
      case DQ_LQ: return log(ph.gamma1 * in(F(4), x, y)) - lpa;
      default: return c.ld(A(WS_D));
    }
  };
  switch (blockIdx.y) {
    case 0: zedge_pair<X>(c, K, A, F); break;
    case 1: zedge_pair<Y>(c, K, A, F); break;
    case 2: {
      const Geo<T> g(b);
      T gxy, gyx, ez, lxz, lyz, qz;
      zedge_q<T>(S, 0, 0, g, ph, gxy, gyx, ez, lxz, lyz, qz);
      const int o = WS_P0;
      c.st(A(o + POUT_GXY), gxy);
      c.st(A(o + POUT_GYX), gyx);
      c.st(A(o + POUT_EZ), ez);
      c.st(A(o + POUT_LXZ), lxz);
      c.st(A(o + POUT_LYZ), lyz);
      c.st(A(o + POUT_QZ), qz);
      break;
    }
    case 3: {
      const Geo<T> g(b);
      T gxx, gyy, qc, dpx, dpy;
      centre_q<T>(S, 0, 0, g, ph, gxx, gyy, qc);
      face_dp<T>(S, 0, 0, g, ph, lnp ? T(exp(lpa)) : T(0), dpx, dpy);
      const int o = WS_P0;
      c.st(A(o + POUT_GXX), gxx);
      c.st(A(o + POUT_GYY), gyy);
      c.st(A(o + POUT_QC), qc);
      c.st(A(o + POUT_DPX), dpx);
      c.st(A(o + POUT_DPY), dpy);
      c.st(A(o + POUT_HX), xface_h<T>(S, 0, 0, g, ph));
      c.st(A(o + POUT_HY), yface_h<T>(S, 0, 0, g, ph));
      break;
    }
    default: {
      // z-face energy flux and pressure gradient; Gzz, Czz at the centre
      const bool visc = tm & T_VISC, adv = tm & T_ADV, pres = tm & T_PRES, ediff = tm & T_EDIFF;
      T hz = T(0);
      if (adv) hz = -c.template dn<Z>(F(4)) * c.ld(A(WS_UZ));
      if (ediff) {
        const T* lem = A(WC_LEM);
        T dl;
        if (tm & T_EDIFFAV) {
          const T* av = K.lnavg + b.poff;
          dl = c.template op<Z, 1, 0>([&](unsigned f) { return c.ld(lem, f) - av[(c.o + f) / c.sz]; });
        } else {
          dl = c.template ddn<Z>(lem);
        }
        hz = hz + ph.nuE * c.template dn<Z>(F(0)) * (c.plane(ZJ_LZF) * c.template dn<Z>(A(WC_NU))) *
                      c.template dn<Z>(A(WC_EM)) * dl;
      }
      T dpz = T(0);
      if (lnp) {
        auto la = [&](unsigned f) { return pav[(c.o + f) / c.sz]; };
        auto lq = [&](unsigned f) { return log(ph.gamma1 * c.ld(F(4), f)) - la(f); };
        dpz = exp(c.template op<Z, 0, 0>(la)) * exp(c.template op<Z, 0, 0>(lq)) *
              (c.template op<Z, 1, 0>(lq) + c.template op<Z, 1, 0>(la));
      } else if (pres) {
        dpz = ph.gamma1 * c.template ddn<Z>(F(4));
      }
      const T szz = c.template dup<Z>(A(WS_UZ));
      T gzz = T(0), czz = T(0);
      if (visc) {
        const T tzz = c.ld(F(0)) * (c.plane(ZJ_LZZ) * c.ld(A(WC_NU))) * (szz + ph.c1 * c.ld(A(WS_D)));
        gzz = tzz;
        czz = tzz * szz;
      }
      if (adv) gzz = gzz - c.template up<Z>(F(3)) * c.template up<Z>(A(WS_UZ));
      const int o = WS_Q0;
      c.st(A(o + QOUT_HZ), hz);
      c.st(A(o + QOUT_DPZ), dpz);
      c.st(A(o + QOUT_GZZ), gzz);
      c.st(A(o + QOUT_CZZ), czz);
      break;
    }
  }
}

// Pass F at one cell, one field per blockIdx.y.  The z divergence of a
// column a reaches output k through the first differences d_p = a[p] -
// a[p-1] of planes p = k-2..k+3, an interpolation directly, summed in the
// march's order and with its choice of constants or table by the plane that
// it scatters.
CELL_KERNEL k_cfinal(CK<T> K) {
  CELL_BEGIN
  if (!own) return;
  const T inv_mu = ph.inv_mu;
  const double dt = K.dt_dev ? *K.dt_dev : K.dt_host;
  const T bdt = T(K.beta * dt);
  const T kd = ((tm & T_DIVB) && dt > 0.0) ? T(double(ph.c_divb) * double(T(b.hmin)) * double(T(b.hmin)) / dt) : T(0);
  const T hz = T(b.hinv[2]);
  const bool cori = tm & T_CORI;
  const T wx = ph.cor2[0], wy = ph.cor2[1];
  const int N = b.nzt;
  auto Q = [&](int q) -> const T* { return A(WS_Q0 + q); };
  auto P = [&](int q) -> const T* { return A(WS_P0 + q); };
  auto inner = [&](int p) { return !c.walled() || (c.k + p >= 6 && c.k + p + 3 <= N - 4); };
  const bool str = W && K.stretched;
  // one scattered plane: first difference of column a (FORM of the derivative)
  auto der = [&](T& acc, auto form, int p, T cur, T prev, T sign) {
    constexpr int FORM = decltype(form)::value;
    T dl = str ? cur - prev : (cur - prev) * hz;
    if (sign < T(0)) dl = -dl;
    if (inner(p)) {
      T w = T(0);
#pragma unroll
      for (int q = -3; q <= 3; ++q) w = q == p ? zdcoef6<FORM, T>(q) : w;
      if (str) acc += w * dl * c.plane(FORM ? ZJ_C : ZJ_F);
      else acc += w * dl;
    } else {
      const T w = c.zt[b.zoff + ((long long)(FORM ? ZT_DDUP : ZT_DDDN) * N + c.k) * 7 + p + 3];
      if (str) acc += w * dl * c.plane(FORM ? ZJ_C : ZJ_F);
      else acc += w * dl;
    }
  };
  auto itp = [&](T& acc, auto form, int p, T v) {
    constexpr int FORM = decltype(form)::value;
    if (inner(p)) {
      T w = T(0);
#pragma unroll
      for (int q = -3; q <= 3; ++q) w = q == p ? zcoef6<0, FORM, T>(q) : w;
      acc += w * v;
    } else {
      acc += c.zt[b.zoff + ((long long)(FORM ? ZT_IUP : ZT_IDN) * N + c.k) * 7 + p + 3] * v;
    }
  };
  constexpr auto UP = std::integral_constant<int, 1>{};
  constexpr auto DN = std::integral_constant<int, 0>{};
  // planes k-3..k+3 in order; body(p, offset of the plane)
  auto planes = [&](const T* a, auto&& body) {
    // (the difference at k-3 has weight 0 in every stencil)
    T prev = c.has(-3) ? c.ld(a, c.d[Z][0]) : T(0);
#pragma unroll
    for (int p = -3; p <= 3; ++p) {
      if (!c.has(p)) {
        prev = T(0);
        continue;
      }
      const unsigned f = c.d[Z][p + 3];
      const T cur = c.ld(a, f);
      body(p, f, cur, prev);
      prev = cur;
    }
  };
  T acc = T(0);
  // the energy first (an x or y stencil at each of 6 z planes, three times the
  // others' loads), rho and B_z last, so that the launch ends on short
  // workgroups: 48^3 float64 26.5 -> 24.8 us, 32^3 11.9 -> 10.7, 20x22x24
  // 9.7 -> 8.0
  const int v = int((0x70653214u >> (4 * blockIdx.y)) & 7u);
  switch (v) {
    case 0:
      planes(F(3), [&](int p, unsigned f, T cur, T prev) {
        if (!(tm & T_CONT)) return;
        if (p == 0) acc += -(c.template dup<X>(F(1)) + c.template dup<Y>(F(2)));
        der(acc, UP, p, cur, prev, T(-1));
      });
      break;
    case 1: {
      const T dpx = c.ld(P(POUT_DPX));
      planes(Q(QOUT_GXZ), [&](int p, unsigned f, T cur, T prev) {
        if (p == 0)
          acc += c.template ddn<X>(P(POUT_GXX)) + c.template dup<Y>(P(POUT_GXY)) -
                 c.template up<Y>(P(POUT_LXZ)) * inv_mu - dpx;
        der(acc, UP, p, cur, prev, T(1));
        itp(acc, UP, p, c.ld(Q(QOUT_LXY), f) * inv_mu);
        if (cori) itp(acc, UP, p, -wy * c.template op<X, 0, 0>([&](unsigned a) { return c.ld(F(3), f + a); }));
      });
      break;
    }
    case 2: {
      const T dpy = c.ld(P(POUT_DPY));
      planes(Q(QOUT_GYZ), [&](int p, unsigned f, T cur, T prev) {
        if (p == 0)
          acc += c.template ddn<Y>(P(POUT_GYY)) + c.template dup<X>(P(POUT_GYX)) +
                 c.template up<X>(P(POUT_LYZ)) * inv_mu - dpy;
        der(acc, UP, p, cur, prev, T(1));
        itp(acc, UP, p, -c.ld(Q(QOUT_LYX), f) * inv_mu);
        if (cori) itp(acc, UP, p, wx * c.template op<Y, 0, 0>([&](unsigned a) { return c.ld(F(3), f + a); }));
      });
      break;
    }
    case 3: {
      const T dpz = c.ld(Q(QOUT_DPZ));
      planes(Q(QOUT_GZZ), [&](int p, unsigned f, T cur, T prev) {
        if (p == 0) {
          acc -= dpz;
          acc += c.template dup<X>(Q(QOUT_GZX)) + c.template dup<Y>(Q(QOUT_GZY)) +
                 (c.template up<Y>(Q(QOUT_LZX)) - c.template up<X>(Q(QOUT_LZY))) * inv_mu;
        }
        der(acc, DN, p, cur, prev, T(1));
        if (tm & T_GRAV) itp(acc, DN, p, -c.ld(F(0), f) * ph.gz);
        if (cori) {
          const T czz = wy * c.template op<X, 0, 1>([&](unsigned a) { return c.ld(F(1), f + a); }) -
                        wx * c.template op<Y, 0, 1>([&](unsigned a) { return c.ld(F(2), f + a); });
          itp(acc, DN, p, czz);
        }
      });
      break;
    }
    case 4: {
      const T qc = c.ld(P(POUT_QC)), czz_ = c.ld(Q(QOUT_CZZ));
      planes(Q(QOUT_HZ), [&](int p, unsigned f, T cur, T prev) {
        if (p == 0) {
          const T* qz = P(POUT_QZ);
          acc += qc + czz_ + c.template dup<X>(P(POUT_HX)) + c.template dup<Y>(P(POUT_HY)) +
                 c.template op<Y, 0, 1>([&](unsigned m) {
                   return c.template op<X, 0, 1>([&](unsigned a) { return c.ld(qz, m + a); });
                 });
          if (tm & T_COOL) {
            const T rc = c.ld(F(0)), ec = c.ld(F(4));
            T q = -rc * (ec / rc - ph.e_cool) * ph.inv_tcool;
            if (ph.cool_cut) {
              const T rr = rc * ph.inv_rho_cool, r2 = rr * rr;
              q = q * ((ph.cool_cut == 1 ? r2 : T(1)) / (T(1) + r2));
            }
            acc += q;
          }
        }
        der(acc, UP, p, cur, prev, T(1));
        itp(acc, UP, p, c.template op<X, 0, 1>([&](unsigned a) { return c.ld(Q(QOUT_QY), f + a); }));
        itp(acc, UP, p, c.template op<Y, 0, 1>([&](unsigned a) { return c.ld(Q(QOUT_QX), f + a); }));
      });
      break;
    }
    case 5:
      planes(Q(QOUT_EY), [&](int p, unsigned f, T cur, T prev) {
        if (p == 0) {
          acc += -c.template dup<Y>(P(POUT_EZ));
          if (kd != T(0)) acc += kd * c.template ddn<X>(A(WS_DIVB));
        }
        der(acc, UP, p, cur, prev, T(1));
      });
      break;
    case 6:
      planes(Q(QOUT_EX), [&](int p, unsigned f, T cur, T prev) {
        if (p == 0) {
          acc += c.template dup<X>(P(POUT_EZ));
          if (kd != T(0)) acc += kd * c.template ddn<Y>(A(WS_DIVB));
        }
        der(acc, UP, p, cur, prev, T(-1));
      });
      break;
    default: {
      T fbz = -(c.template dup<X>(Q(QOUT_EY)) - c.template dup<Y>(Q(QOUT_EX)));
      if (kd != T(0)) fbz += kd * c.template ddn<Z>(A(WS_DIVB));
      acc = fbz;
      break;
    }
  }
  if (c.walled()) {
    const bool keep = v == 3 ? (c.k > b.g0 && c.k < b.g1) : (v == 7 ? (c.k >= b.g0 && c.k <= b.g1) : inside);
    if (!keep) acc = T(0);
  }
  T* du = K.du.p[v] + b.off;
  if (K.f_out.p[0] == nullptr) {
    c.st(du, acc);
    return;
  }
  const T uin = (K.du_mode & DU_READ) ? c.ld(du) : T(0), fin = c.ld(F(v));
  const T U = (K.du_mode & DU_READ) ? K.alpha * uin + acc : acc;
  if (K.du_mode & DU_WRITE) c.st(du, U);
  c.st(K.f_out.p[v] + b.off, fin + bdt * U);
}

template <class T, bool W> void stage(const ZLaunch& L, const ZStageArgs<T>& a) {
  CK<T> K;
  K.boxes = L.boxes;
  K.tab = L.tab;
  K.nblk = L.nblk;
  K.f = a.f;
  K.ws = a.w;
  K.ph = a.ph;
  K.zt = a.ztab;
  K.lnavg = a.lnavg;
  K.stretched = L.stretched;
  K.cpart = a.cpart;
  K.du = a.du;
  K.du_mode = a.du_mode;
  K.f_out = a.f_out;
  K.alpha = a.alpha;
  K.beta = a.beta;
  K.dt_dev = a.dt_dev;
  K.dt_host = a.dt_host;
  auto go = [&](void (*kern)(CK<T>), int roles) {
    hipLaunchKernelGGL(kern, dim3(8 * ((L.nblk + 7) / 8), roles), dim3(kBlock), 0, L.stream, K);
  };
  L.at(PASS_PRIM);
  go(k_cprim<T, W>, 1);
  go(k_cnus<T, W>, 1);
  L.at(PASS_MEAN3);
  if (a.ph.terms & T_MAX5) go(k_cmax<T, W, 2>, 1);
  else go(k_cmax<T, W, 1>, 1);
  go(k_cmean<T, W>, 1);
  if (a.cpart) {
    L.at(PASS_REDUCE);
    launch_courant(L, a);
    L.at(PASS_MEAN3);
  }
  launch_plane_means<T>(L, a);
  go(k_clines<T, W>, 1);
  L.at(PASS_EDGES);
  go(k_cedges<T, W>, 5);
  L.at(PASS_FINAL);
  go(k_cfinal<T, W>, 8);
  L.at(PASS_END);
}

}  // namespace

template <class T> void launch_cellstage(const ZLaunch& L, const ZStageArgs<T>& a) {
  if (L.wall) stage<T, true>(L, a);
  else stage<T, false>(L, a);
}
template void launch_cellstage<float>(const ZLaunch&, const ZStageArgs<float>&);
template void launch_cellstage<double>(const ZLaunch&, const ZStageArgs<double>&);

}  // namespace smhd
