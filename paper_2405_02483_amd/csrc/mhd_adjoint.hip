// (dF/df)^T w of the right-hand side F (eqs. mass, mom, ien, indu with
// itv, ohm, vdiss, RMnu, nuij, ediffuse and the optional terms), in
// hand-fused passes over the cells of all boxes.
//
// The passes follow the right-hand side backwards.  Every flux, edge
// quantity and heating term of F is differenced or interpolated once more
// before it reaches an output, so its cotangent at its own position is a
// stencil of w and is formed there, in registers.  What is stored are the
// cotangents of the interpolated and differenced inputs at each position
// (10 per cell edge, 6 per face, 4 per axis at the centre); the next pass
// gathers their transposed stencils into velocities, momenta, B, energy and
// density.  On a periodic axis the transpose of an interpolation is the
// interpolation of the opposite stagger, that of a derivative minus the
// derivative of the opposite stagger; near the ends of a wall-bounded z
// axis the gather runs over the columns of the box's coefficient table.
//
// One thread per cell; a workgroup takes 256 consecutive cells, and
// consecutive workgroups of an XCD take consecutive cells, so that the
// stencils' repeated reads hit in L1 (x, y) and in that XCD's L2 (z).
//
// With the core terms 88 arrays, some 190 reads and writes per cell and
// stage, against 1700 of an operation-by-operation program, which this
// replaced (each operation a pass over 2 to 5 arrays, 160 launches a stage).
// The pointwise passes are bound by those bytes, the edges' and vectors'
// gathers (half the time) by the caches' latency, at 2.9 TB/s.  One step's
// adjoint:
// 128^3 float32 23.06 -> 3.14 ms, 64^3 float32 with walls and every
// optional term 14.37 -> 2.35 ms; a 6-step float64 rollout of 48^3 with its
// gradient 63.2 -> 6.5 ms.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "mhd_adjoint.hpp"
#include "mhd_cell.hpp"

namespace smhd {
namespace {

// Workspace arrays.  Vectors take three (x, y, z); edge quantities 10 per
// edge direction (EdgeQ), edge c running along axis c between the axes
// a = c + 1 and b = c + 2 (cyclic).
enum VArr : int {
  VA_U = 0,                 // face velocities
  VA_R = VA_U + 3,          // face densities dn_a(rho)
  VA_EM = VA_R + 3, VA_LEM, // e / rho and its log
  VA_XWE, VA_YWE,           // x and y transposes of w_e's centre interpolation
  VA_NT, VA_LNT,            // <nu> (floored) and its log
  VA_XL, VA_YL,             // dn_x, dn_y of ln <nu>
  VA_EDGE,                  // 30
  VA_XE = VA_EDGE + 30,     // cotangents of dn_a(e), dn_a(nu), dn_a(e_m), ddn_a(ln e_m)
  VA_XNT = VA_XE + 3, VA_XEM = VA_XNT + 3, VA_DLEM = VA_XEM + 3,
  VA_RF = VA_DLEM + 3,      // of the face densities, from the energy diffusion
  VA_UF = VA_RF + 3,        // of the face velocities, from the energy flux
  VA_XLB = VA_UF + 3, VA_YLB,   // of dn_x, dn_y of ln <nu>
  VA_NTB,                   // of <nu>
  VA_MB0, VA_MB1,           // of the maxima, in turn
  VA_CP, VA_CU = VA_CP + 3, VA_SD = VA_CU + 3, VA_CB = VA_SD + 3,   // of up_a(p_a, u_a), dup_a(u_a), up_a(B_a)
  VA_RHOB = VA_CB + 3, VA_EB,   // pointwise parts of rho and e
  VA_RB,                    // of the face densities
  VA_MX = VA_RB + 3,        // speed-like viscosity and its maxima so far
  VA_CORE = VA_MX + 4,
  VA_MX5 = VA_CORE,         // three more with T_MAX5
  VA_LNP = VA_MX5 + 3,      // T_LNP: ln P, cotangents of dn_a, ddn_a of it
  VA_QI = VA_LNP + 1, VA_QD = VA_QI + 3,
  VA_DVB = VA_QD + 3,       // T_DIVB: of div B
  VA_EDX,                   // T_EDIFFAV: of the plane mean's log, cell by cell
  VA_SE,                    // T_SMAG: shear on the edges, then its centre value and cotangent
  VA_SC = VA_SE + 3,
  VA_RGH = VA_SC + 3,       // T_ORDER2: rough cells, flags, second-order parts of the strain's cotangents
  VA_RGF, VA_HS2, VA_SD2 = VA_HS2 + 3,
  VA_TAU = VA_SD2 + 3,      // T_QUENCH: raw stress, q, its maxima, cotangents (6 each)
  VA_QQ = VA_TAU + 6, VA_Q1 = VA_QQ + 6, VA_Q2 = VA_Q1 + 6, VA_Q3 = VA_Q2 + 6, VA_TB = VA_Q3 + 6,
  VA_QB0 = VA_TB + 6, VA_QB1 = VA_QB0 + 6,
  VA_COUNT = VA_QB1 + 6
};
enum EdgeQ : int { EQ_UAB = 0, EQ_UBA, EQ_HS, EQ_PAB, EQ_PBA, EQ_BAB, EQ_BBA, EQ_J, EQ_RHO, EQ_LNU, EQ_COUNT };

constexpr int kFillTmp = 6;   // arrays that vjp_fill takes of the workspace
constexpr unsigned kCoreTerms = T_CONT | T_ADV | T_PRES | T_VISC | T_LORENTZ | T_INDUCT | T_RESIST | T_EDIFF;

// What a set of terms takes of the transpose: the workspace arrays, the
// launches and, within a launch, the operands.
struct Need {
  unsigned tm;
  bool cst, etac;           // constant viscosity, constant resistivity
  template <class T>
  __host__ __device__ __forceinline__ explicit Need(const Phys<T>& ph)
      : tm(ph.terms), cst(ph.nu_const > T(0)), etac(ph.eta_const > T(0)) {}
  __host__ __device__ __forceinline__ bool any(unsigned t) const { return tm & t; }
  __host__ __device__ __forceinline__ bool heat() const { return any(T_VISC | T_RESIST); }
  // the viscosity on the edges; anywhere; as the maximum of the speed-like one
  __host__ __device__ __forceinline__ bool enu() const { return any(T_VISC) || (any(T_RESIST) && !etac); }
  __host__ __device__ __forceinline__ bool nu() const { return enu() || any(T_EDIFF); }
  __host__ __device__ __forceinline__ bool chain() const { return nu() && !cst; }
  __host__ __device__ __forceinline__ bool smag() const { return any(T_SMAG) && chain(); }
  __host__ __device__ __forceinline__ bool quench() const { return any(T_QUENCH) && any(T_VISC); }
  __host__ __device__ __forceinline__ bool order2() const { return any(T_ORDER2) && any(T_VISC); }
  __host__ __device__ __forceinline__ bool lnp() const { return any(T_LNP) && any(T_PRES); }
  __host__ __device__ __forceinline__ bool ediffav() const { return any(T_EDIFFAV) && any(T_EDIFF); }
  // face velocities and densities, edges, the faces' fluxes, the centre
  __host__ __device__ __forceinline__ bool faces() const {
    return any(T_ADV | T_VISC | T_INDUCT | T_PRES | T_EDIFF) || chain();
  }
  __host__ __device__ __forceinline__ bool edges() const {
    return any(T_ADV | T_VISC | T_INDUCT | T_RESIST | T_LORENTZ) || smag();
  }
  __host__ __device__ __forceinline__ bool fluxes() const { return any(T_ADV | T_EDIFF) || lnp(); }
  __host__ __device__ __forceinline__ bool strain() const { return any(T_VISC | T_PRES) || chain(); }
  __host__ __device__ __forceinline__ bool centre() const { return strain() || any(T_ADV | T_COOL); }
  __host__ __device__ __forceinline__ bool shear() const { return any(T_VISC) || smag(); }
  __host__ __device__ __forceinline__ bool cu() const { return any(T_ADV) || chain(); }
  __host__ __device__ __forceinline__ bool rhob() const { return any(T_VISC | T_COOL) || chain(); }
  __host__ __device__ __forceinline__ bool eb() const { return any(T_PRES | T_COOL) || chain(); }
};

// A set of terms that needs more than kLeanArrays of the 88 core arrays, and
// leaves at most kFullSpare of the full layout unused, runs with every array
// (ALL): its kernels know where they lie and branch less.  Others take only
// what they need, through a table.  Measured, us of one transpose, every
// array against what is needed: 128^3 float32 continuity alone 614 / 106,
// viscous stress (44 arrays) 641 / 513, ideal MHD (46) 656 / 491, Lorentz force
// 608 / 192; but constant coefficients without energy diffusion (64) 553 / 640,
// without energy diffusion (74) 697 / 795, hydrodynamics (79) 736 / 771, and
// the core terms through the table 752 / 1088 (the gathers' 40 and more base
// pointers fill the scalar registers).  The spare of 40 keeps every set below
// the workspace that an operation-by-operation program took for it.
constexpr int kLeanArrays = 50, kFullSpare = 40;

// Where each array lies in the workspace (at[id], in arrays; all: at[id] =
// id); returns the number of arrays (none with the continuity alone, 44 with
// the viscous stress alone, 88 with the core terms).
int layout(const Need& nd, unsigned char (&at)[VA_COUNT], bool& all) {
  int n = 0;
  auto take = [&](bool need, int id, int count) {
    for (int q = 0; need && q < count; ++q) at[id + q] = (unsigned char)n++;
  };
  for (unsigned char& a : at) a = 0;
  take(nd.faces(), VA_U, 6);           // with VA_R
  take(nd.any(T_EDIFF), VA_EM, 1);
  take(nd.any(T_EDIFF) || nd.order2(), VA_LEM, 1);
  take(nd.heat(), VA_XWE, 2);
  take(nd.nu(), VA_NT, 1);
  take(nd.enu(), VA_LNT, 3);           // with VA_XL, VA_YL
  const bool eq[EQ_COUNT] = {nd.any(T_ADV | T_INDUCT), nd.any(T_ADV | T_INDUCT), nd.shear(), nd.any(T_ADV),
                             nd.any(T_ADV), nd.any(T_INDUCT | T_LORENTZ), nd.any(T_INDUCT | T_LORENTZ),
                             nd.any(T_RESIST | T_LORENTZ), nd.any(T_VISC), nd.enu()};
  for (int e = 0; e < 3; ++e)
    for (int q = 0; q < EQ_COUNT; ++q) take(eq[q], VA_EDGE + e * EQ_COUNT + q, 1);
  take(nd.any(T_ADV), VA_XE, 3);
  take(nd.any(T_EDIFF), VA_XNT, 12);   // with VA_XEM, VA_DLEM, VA_RF
  take(nd.any(T_ADV), VA_UF, 3);
  take(nd.enu(), VA_XLB, 2);
  take(nd.chain(), VA_NTB, 3);         // with VA_MB0, VA_MB1
  take(nd.any(T_ADV), VA_CP, 3);
  take(nd.cu(), VA_CU, 3);
  take(nd.strain(), VA_SD, 3);
  take(nd.chain(), VA_CB, 3);
  take(nd.rhob(), VA_RHOB, 1);
  take(nd.eb(), VA_EB, 1);
  take(nd.faces(), VA_RB, 3);
  take(nd.chain(), VA_MX, 4);
  const bool most = n > kLeanArrays;
  take(nd.chain() && nd.any(T_MAX5), VA_MX5, 3);
  take(nd.lnp(), VA_LNP, 7);           // with VA_QI, VA_QD
  take(nd.any(T_DIVB), VA_DVB, 1);
  take(nd.ediffav(), VA_EDX, 1);
  take(nd.smag(), VA_SE, 6);           // with VA_SC
  take(nd.order2(), VA_RGH, VA_TAU - VA_RGH);
  take(nd.quench(), VA_TAU, VA_COUNT - VA_TAU);
  const int full = nd.quench() ? VA_COUNT : nd.order2() ? VA_TAU : nd.any(T_SMAG) ? VA_RGH : nd.ediffav() ? VA_SE :
                   nd.any(T_DIVB) ? VA_EDX : nd.lnp() ? VA_DVB : nd.any(T_MAX5) ? VA_LNP : VA_CORE;
  all = most && full <= n + kFullSpare;
  if (!all) return n;
  for (int q = 0; q < VA_COUNT; ++q) at[q] = (unsigned char)q;
  return full;
}

template <class T> struct VArgs {
  const BoxDev* boxes;
  const Blk* tab;
  int nblk;
  CP8<T> s, w;
  P8<T> g;
  T* base;
  long long stride;
  const T* zt;
  const double* pm;
  int nplanes;
  Phys<T> ph;
  double nu2, c_smag, dt;
  double c_divb;
  int acc;
  int nmax;                 // maxima in the chain (3, or 6 with T_MAX5)
};
// (with every array the table stays out of the launches' arguments)
template <class T, bool ALL> struct VK : VArgs<T> {
  __host__ __device__ __forceinline__ int slot(int id) const { return id; }
};
template <class T> struct VK<T, false> : VArgs<T> {
  unsigned char at[VA_COUNT];   // layout()
  __host__ __device__ __forceinline__ int slot(int id) const { return at[id]; }
};

// ALL: every core term's arrays are kept, at addresses known to the compiler,
// and read and written without a look at the terms.
#define VJP_CELL                                                             \
  const int per_ = (K.nblk + 7) >> 3;                                        \
  const int bi_ = (int)(blockIdx.x & 7u) * per_ + (int)(blockIdx.x >> 3);    \
  if (bi_ >= K.nblk) return;                                                 \
  const Blk tb_ = K.tab[bi_];                                                \
  if ((int)threadIdx.x >= tb_.n) return;                                     \
  const BoxDev& b = K.boxes[tb_.box];                                        \
  const Cell<T, W> c(b, (unsigned)tb_.start + threadIdx.x, K.zt);            \
  auto An = [&](int slot) -> T* { return K.base + (long long)slot * K.stride + b.off; };   \
  auto A = [&](int id) -> T* { return An(K.slot(id)); };                      \
  auto Am = [&](int id, int m) -> T* { return An(K.slot(id) + m); };   \
  auto S = [&](int v) -> const T* { return K.s.p[v] + b.off; };              \
  auto Wt = [&](int v) -> const T* { return K.w.p[v] + b.off; };             \
  const unsigned tm = K.ph.terms;                                            \
  const Need nd(K.ph);                                                       \
  (void)A; (void)An; (void)Am; (void)S; (void)Wt; (void)tm; (void)nd;

#define VJP_KERNEL template <class T, bool W, bool ALL> __global__ __launch_bounds__(kBlock) void

// The same with at least `f32` waves a SIMD in float32.  The kernels that
// gather most wait for the caches; left alone the compiler hoists loads until
// 98 to 113 registers hold them and 4 waves fit.  128^3 float32: edges and
// faces 266 us at 4 waves, 254 at 5, 270 at 6 (spilling); vectors 217 at 4,
// 192 at 5, 176 at 6, 185 at 8; centre 74 at 4, 70 at 5, 84 at 6.  In float64
// every such bound spills (edges and faces 25 -> 41 us at 48^3), so there the
// compiler's choice stands.
#define VJP_KERNEL_WAVES(f32)                                    \
  template <class T, bool W, bool ALL>                           \
  __global__ __launch_bounds__(kBlock)                           \
      __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? f32 : 1))) void

template <class T> __device__ __forceinline__ T vnorm3(T x, T y, T z) {
  const T s = x * x + y * y + z * z;
  return s > T(0) ? sqrt(s) : T(0);
}

// Viscosity length of the centre component a, and of edge e's component.
template <class T, bool W> __device__ __forceinline__ T len_c(const Cell<T, W>& c, int a) {
  return (W && a == Z && c.b.stretched) ? c.plane(ZJ_LZZ) : T(c.b.lv[a]);
}
template <class T, bool W> __device__ __forceinline__ T len_e(const Cell<T, W>& c, int e) {
  if (W && e != Z && c.b.stretched) return c.plane(e == X ? ZJ_LYZ : ZJ_LXZ);
  return T(c.b.le[2 - e]);     // le: xy, xz, yz; edge z, y, x
}
template <class T, bool W> __device__ __forceinline__ double h_shock(const Cell<T, W>& c) {
  return (W && c.b.stretched) ? double(c.plane(ZJ_H)) : c.b.hmin;
}

// ---------------------------------------------------------------------------
// Face densities and velocities, e_m, ln e_m, and w_e's x and y transposes.
VJP_KERNEL k_prim(VK<T, ALL> K) {
  VJP_CELL
  const T* rho = S(0);
  const bool faces = ALL || nd.faces(), diff = ALL || nd.any(T_EDIFF), logs = diff || nd.order2();
  const T rx = faces ? c.template dn<X>(rho) : T(1), ry = faces ? c.template dn<Y>(rho) : T(1),
          rz = faces ? c.template dn<Z>(rho) : T(1);
  const T em = logs ? c.ld(S(4)) / c.ld(rho) : T(1);
  if (faces) {
    c.st(A(VA_R), rx);
    c.st(A(VA_R + 1), ry);
    c.st(A(VA_R + 2), rz);
    c.st(A(VA_U), c.ld(S(1)) / rx);
    c.st(A(VA_U + 1), c.ld(S(2)) / ry);
    c.st(A(VA_U + 2), c.ld(S(3)) / rz);
  }
  if (diff) c.st(A(VA_EM), em);
  if (logs) c.st(A(VA_LEM), log(em));
  if (ALL || nd.heat()) {
    c.st(A(VA_XWE), c.template upT<X>(Wt(4)));
    c.st(A(VA_YWE), c.template upT<Y>(Wt(4)));
  }
  if (nd.lnp()) c.st(A(VA_LNP), log(K.ph.gamma1 * c.ld(S(4))));
}

// Second-order switch: rough cells, then the flags of the positions a rough
// cell touches (bit 0 the centre, 1 + c the edge along axis c).
VJP_KERNEL k_rough(VK<T, ALL> K) {
  VJP_CELL
  const T* rho = S(0);
  const T* le = A(VA_LEM);
  auto lr = [&](unsigned f) { return log(c.ld(rho, f)); };
  auto lm = [&](unsigned f) { return c.ld(le, f); };
  T m = T(0);
  auto axis = [&](const auto& f, int ax) {
    m = fmax(m, fabs(f(c.d[ax][4]) - T(2) * f(0u) + f(c.d[ax][2])));
  };
  axis(lr, X);
  axis(lr, Y);
  axis(lm, X);
  axis(lm, Y);
  if (c.has(-1) && c.has(1)) {
    axis(lr, Z);
    axis(lm, Z);
  }
  c.st(A(VA_RGH), m > K.ph.d2_lim ? T(1) : T(0));
}
VJP_KERNEL k_rough_flags(VK<T, ALL> K) {
  VJP_CELL
  const T* r = A(VA_RGH);
  auto at = [&](int x, int y, int z) {
    if (z && !c.has(-1)) return false;
    return c.ld(r, c.d[X][3 - x] + c.d[Y][3 - y] + c.d[Z][3 - z]) > T(0.5);
  };
  unsigned f = at(0, 0, 0) ? 1u : 0u;
  if (at(0, 0, 0) || at(0, 1, 0) || at(0, 0, 1) || at(0, 1, 1)) f |= 2u;
  if (at(0, 0, 0) || at(1, 0, 0) || at(0, 0, 1) || at(1, 0, 1)) f |= 4u;
  if (at(0, 0, 0) || at(1, 0, 0) || at(0, 1, 0) || at(1, 1, 0)) f |= 8u;
  c.st(A(VA_RGF), T(f));
}

template <class T> __device__ __forceinline__ bool order2(const VArgs<T>& K) {
  return (K.ph.terms & T_ORDER2) && (K.ph.terms & T_VISC);
}
template <class T> __device__ __forceinline__ bool quenched(const VArgs<T>& K) {
  return (K.ph.terms & T_QUENCH) && (K.ph.terms & T_VISC);
}
template <class T> __device__ __forceinline__ bool smag(const VArgs<T>& K) {
  return (K.ph.terms & T_SMAG) && !(K.ph.nu_const > T(0));
}

// Shear on the edge along axis C (eq. itv): sixth order, or second (O2).
template <int C, bool O2, class T, bool W, class F>
__device__ __forceinline__ T shear(const Cell<T, W>& c, const F& A) {
  constexpr int P = (C + 1) % 3, Q = (C + 2) % 3;
  if constexpr (O2) return T(0.5) * (c.template d2n<Q>(A(VA_U + P)) + c.template d2n<P>(A(VA_U + Q)));
  else return T(0.5) * (c.template ddn<Q>(A(VA_U + P)) + c.template ddn<P>(A(VA_U + Q)));
}
// The strain that the stress takes: second order where flagged.
template <int C, class T, bool W, class F>
__device__ __forceinline__ T strain_e(const Cell<T, W>& c, const VArgs<T>& K, const F& A) {
  if (order2(K) && ((unsigned)c.ld(A(VA_RGF)) & (2u << C))) return shear<C, true>(c, A);
  return shear<C, false>(c, A);
}

// T_SMAG: the shear on the edges (blockIdx.y: edge direction).
VJP_KERNEL k_shear(VK<T, ALL> K) {
  VJP_CELL
  const int e = (int)blockIdx.y;
  c.st(Am(VA_SE, e), e == X ? shear<X, false>(c, A) : (e == Y ? shear<Y, false>(c, A) : shear<Z, false>(c, A)));
}

// The speed-like viscosity (eq. RMnu, eq. nusmag).  Each product and sum is
// rounded on its own, whatever the surrounding expression, so that ties and
// signs (max, relu) fall the same way wherever this is evaluated.
VJP_KERNEL k_nus(VK<T, ALL> K) {
  VJP_CELL
  const Phys<T>& ph = K.ph;
  const T sxx = c.template dup<X>(A(VA_U)), syy = c.template dup<Y>(A(VA_U + 1)), szz = c.template dup<Z>(A(VA_U + 2));
  const T sxy_ = sxx + syy;
  const T D = sxy_ + szz;
  const T ub = vnorm3(c.template up<X>(A(VA_U)), c.template up<Y>(A(VA_U + 1)), c.template up<Z>(A(VA_U + 2)));
  const T bb = vnorm3(c.template up<X>(S(5)), c.template up<Y>(S(6)), c.template up<Z>(S(7)));
  const T rho = c.ld(S(0));
  const T P = ph.gamma1 * c.ld(S(4));
  const T gp = ph.gamma * P;
  const T cs = sqrt(gp / rho);
  const T mr = ph.mu * rho;
  const T ca = bb / sqrt(mr);
  const T v1 = ph.nu1 * ub;
  const T cc = cs + ca;
  const T v2 = ph.nu3 * cc;
  const T relu = -D > T(0) ? -D : T(0);
  const T v3 = T(K.nu2 * h_shock(c)) * relu;
  const T v12 = v1 + v2;
  T nus = v12 + v3;
  if (smag(K)) {
    // centre values of the shear, kept for the transpose
    const T cyz = c.template ii<Z, 1, Y, 1>(A(VA_SE)), cxz = c.template ii<Z, 1, X, 1>(A(VA_SE + 1)),
            cxy = c.template ii<Y, 1, X, 1>(A(VA_SE + 2));
    c.st(A(VA_SC), cyz);
    c.st(A(VA_SC + 1), cxz);
    c.st(A(VA_SC + 2), cxy);
    const T s2 = T(2) * (sxx * sxx + syy * syy + szz * szz - D * D * T(1.0 / 3.0) +
                         T(2) * (cxy * cxy + cxz * cxz + cyz * cyz));
    const T v4 = T(K.c_smag * h_shock(c)) * (s2 > T(0) ? sqrt(s2) : T(0));
    nus = nus + v4;
  }
  c.st(A(VA_MX), nus);
}

// Id of the m-th array of the maximum chain (0: the viscosity itself).
__host__ __device__ __forceinline__ int mx_id(int m) { return m < 4 ? VA_MX + m : VA_MX5 + (m - 4); }

// Maximum over three cells along x, y, z in turn: the three stages.
VJP_KERNEL k_max3(VK<T, ALL> K) {
  VJP_CELL
  const T* a = A(VA_MX);
  auto mx = [&](unsigned f) {
    return fmax(fmax(c.ld(a, f + c.d[X][2]), c.ld(a, f)), c.ld(a, f + c.d[X][4]));
  };
  auto my = [&](unsigned f, T own) { return fmax(fmax(mx(f + c.d[Y][2]), own), mx(f + c.d[Y][4])); };
  const T m1 = mx(0u);
  const T m2 = my(0u, m1);
  T m3 = m2;
  if (c.has(-1)) m3 = fmax(m3, my(c.d[Z][2], mx(c.d[Z][2])));
  if (c.has(1)) m3 = fmax(m3, my(c.d[Z][4], mx(c.d[Z][4])));
  c.st(A(VA_MX + 1), m1);
  c.st(A(VA_MX + 2), m2);
  c.st(A(VA_MX + 3), m3);
}
// One stage (five cells: each axis twice).
template <class T, bool W, bool ALL, int AX> __global__ __launch_bounds__(kBlock) void k_max1(VK<T, ALL> K, int src, int dst) {
  VJP_CELL
  c.st(An(dst), c.template max3<AX>(An(src)));
}
// Transpose of one stage; blockIdx.y: component (quenching).
template <class T, bool W, bool ALL, int AX>
__global__ __launch_bounds__(kBlock) void k_max1T(VK<T, ALL> K, int prim, int yb, int dst) {
  VJP_CELL
  const int m = (int)blockIdx.y;
  c.st(An(dst + m), c.template max3T<AX>(An(prim + m), An(yb + m)));
}

// <nu>: the mean over three cells along each axis (the available ones at
// the ends of a wall axis), the floor, and ln.  nu_const: the constant.
VJP_KERNEL k_mean(VK<T, ALL> K, int mx) {
  VJP_CELL
  T v;
  if (K.ph.nu_const > T(0)) {
    v = T(double(K.ph.nu_const) / b.hmin);
  } else {
    const T* a = An(mx);
    auto row = [&](unsigned f) { return (c.ld(a, f + c.d[X][2]) + c.ld(a, f) + c.ld(a, f + c.d[X][4])) / T(3); };
    auto pl = [&](unsigned f) { return (row(f + c.d[Y][2]) + row(f) + row(f + c.d[Y][4])) / T(3); };
    const bool lo = c.has(-1), hi = c.has(1);
    T s = pl(0u);
    if (lo) s = pl(c.d[Z][2]) + s;
    if (hi) s = s + pl(c.d[Z][4]);
    v = s / T(1 + (lo ? 1 : 0) + (hi ? 1 : 0));
  }
  v = v > T(1e-30) ? v : T(1e-30);
  c.st(A(VA_NT), v);
  if (ALL || nd.enu()) c.st(A(VA_LNT), log(v));
}
VJP_KERNEL k_lines(VK<T, ALL> K) {
  VJP_CELL
  c.st(A(VA_XL), c.template dn<X>(A(VA_LNT)));
  c.st(A(VA_YL), c.template dn<Y>(A(VA_LNT)));
}

// Density, viscosity and w_e's heating cotangent on the edge along C.
template <bool ALL, int C, class T, bool W, class F> struct EdgeBase {
  T rho = T(0), nu = T(0), Qb = T(0);
  __device__ __forceinline__ EdgeBase(const Cell<T, W>& c, const F& A, const Need& nd) {
    constexpr int Q = C == Z ? Y : Z;                    // the second axis
    constexpr int first = C == X ? 1 : 0;                // interpolated along y (edge x) or x first
    if (ALL || nd.any(T_VISC)) rho = c.template dn<Q>(A(VA_R + first));
    if (ALL || nd.enu()) nu = len_e(c, C) * exp(c.template dn<Q>(A(C == X ? VA_YL : VA_XL)));
    if (ALL || nd.heat()) Qb = c.template upT<Q>(A(C == X ? VA_YWE : VA_XWE));
  }
};

// T_QUENCH: raw stress (roles 0..2 the edges, 3..5 the centre), q, the
// maxima over 3x3x3 cells.
template <int C, class T, bool W, class F>
__device__ __forceinline__ T raw_edge(const Cell<T, W>& c, const VArgs<T>& K, const F& A) {
  const EdgeBase<true, C, T, W, F> E(c, A, Need(K.ph));   // (with T_VISC)
  return E.rho * E.nu * strain_e<C>(c, K, A);
}
// Strain and div u at the centre as the stress takes them (vs, vD), and the
// sixth-order ones (s, D).
template <class T, bool W, class F> struct Centre {
  T s[3] = {}, D = T(0), vs[3] = {}, vD = T(0);
  bool rough = false;
  // (need false: nothing takes them)
  __device__ __forceinline__ Centre(const Cell<T, W>& c, const VArgs<T>& K, const F& A, bool need = true) {
    if (!need) return;
    s[0] = c.template dup<X>(A(VA_U));
    s[1] = c.template dup<Y>(A(VA_U + 1));
    s[2] = c.template dup<Z>(A(VA_U + 2));
    const T xy = s[0] + s[1];
    D = xy + s[2];
    rough = order2(K) && ((unsigned)c.ld(A(VA_RGF)) & 1u);
    vD = D;
#pragma unroll
    for (int a = 0; a < 3; ++a) vs[a] = s[a];
    if (rough) {
      vs[0] = c.template d2u<X>(A(VA_U));
      vs[1] = c.template d2u<Y>(A(VA_U + 1));
      vs[2] = c.template d2u<Z>(A(VA_U + 2));
      vD = vs[0] + vs[1] + vs[2];
    }
  }
};
VJP_KERNEL k_tau(VK<T, ALL> K) {
  VJP_CELL
  const int m = (int)blockIdx.y;
  T t;
  if (m < 3) {
    t = m == X ? raw_edge<X>(c, K, A) : (m == Y ? raw_edge<Y>(c, K, A) : raw_edge<Z>(c, K, A));
    c.st(Am(VA_TAU, m), t);
  } else if (m == 3) {
    const Centre<T, W, decltype(A)> E(c, K, A);
    const T r = c.ld(S(0)), nt = c.ld(A(VA_NT));
#pragma unroll
    for (int a = 0; a < 3; ++a)
      c.st(A(VA_TAU + 3 + a), r * (len_c(c, a) * nt) * (E.vs[a] + K.ph.c1 * E.vD));
  }
}
VJP_KERNEL k_quench(VK<T, ALL> K) {
  VJP_CELL
  const int m = (int)blockIdx.y;
  const T* t = Am(VA_TAU, m);
  const T s = fabs(c.template second<X>(t)) + fabs(c.template second<Y>(t)) + fabs(c.template second<Z>(t));
  const T den = fabs(c.ld(t)) + s / K.ph.q_max;
  c.st(Am(VA_QQ, m), den > T(0) ? s / den : T(0));
}
VJP_KERNEL k_quench_max(VK<T, ALL> K) {
  VJP_CELL
  const int m = (int)blockIdx.y;
  const T* a = Am(VA_QQ, m);
  auto mx = [&](unsigned f) {
    return fmax(fmax(c.ld(a, f + c.d[X][2]), c.ld(a, f)), c.ld(a, f + c.d[X][4]));
  };
  auto my = [&](unsigned f, T own) { return fmax(fmax(mx(f + c.d[Y][2]), own), mx(f + c.d[Y][4])); };
  const T m1 = mx(0u);
  const T m2 = my(0u, m1);
  T m3 = m2;
  if (c.has(-1)) m3 = fmax(m3, my(c.d[Z][2], mx(c.d[Z][2])));
  if (c.has(1)) m3 = fmax(m3, my(c.d[Z][4], mx(c.d[Z][4])));
  c.st(Am(VA_Q1, m), m1);
  c.st(Am(VA_Q2, m), m2);
  c.st(Am(VA_Q3, m), m3);
}
// The factor of component m at the cell.
template <class T, bool W, class F>
__device__ __forceinline__ T qfac(const Cell<T, W>& c, const VArgs<T>& K, const F& A, int m) {
  const T q = c.ld(A(VA_Q3) + (long long)m * K.stride);
  return q < K.ph.q_lim ? q : K.ph.q_lim;
}

// Cotangents of the momentum fluxes on the edge along C (between the axes P
// and Q): the flux of p_P enters dp_P through dup_Q, that of p_Q dp_Q
// through dup_P.
template <int C, class T, bool W, class F>
__device__ __forceinline__ void flux_cot(const Cell<T, W>& c, const F& Wt, T& g1, T& g2) {
  constexpr int P = (C + 1) % 3, Q = (C + 2) % 3;
  g1 = c.template dupT<Q>(Wt(1 + P));
  g2 = c.template dupT<P>(Wt(1 + Q));
}
// The quenched stress's cotangent, and through the cap that of the maximum
// of q.
template <int C, class T, bool W, class F, class G>
__device__ __forceinline__ T taub_edge(const Cell<T, W>& c, const VArgs<T>& K, const F& A, const G& Wt) {
  const EdgeBase<true, C, T, W, F> E(c, A, Need(K.ph));   // (with T_VISC)
  T g1, g2;
  flux_cot<C>(c, Wt, g1, g2);
  return g1 + g2 + T(2) * strain_e<C>(c, K, A) * E.Qb;
}
VJP_KERNEL k_taub(VK<T, ALL> K) {
  VJP_CELL
  const int m = (int)blockIdx.y;
  auto put = [&](int q, T tb) {
    const T x = c.ld(Am(VA_Q3, q));
    c.st(Am(VA_TB, q), tb);
    c.st(Am(VA_QB0, q), x < K.ph.q_lim ? c.ld(Am(VA_TAU, q)) * tb : T(0));
  };
  if (m < 3) {
    put(m, m == X ? taub_edge<X>(c, K, A, Wt) : (m == Y ? taub_edge<Y>(c, K, A, Wt) : taub_edge<Z>(c, K, A, Wt)));
  } else if (m == 3) {
    const Centre<T, W, decltype(A)> E(c, K, A);
    const T we = c.ld(Wt(4));
    put(3, c.template ddnT<X>(Wt(1)) + E.vs[0] * we);
    put(4, c.template ddnT<Y>(Wt(2)) + E.vs[1] * we);
    put(5, c.template ddnT<Z>(Wt(3)) + E.vs[2] * we);
  }
}
// From the cotangent of q: that of D2 (into QB0), and the stress's own
// through |tau| and the factor (into TB).
VJP_KERNEL k_quenchT(VK<T, ALL> K) {
  VJP_CELL
  const int m = (int)blockIdx.y;
  const T* t = Am(VA_TAU, m);
  const T qb = c.template max3T<X>(Am(VA_QQ, m), Am(VA_QB0, m));
  const T s = fabs(c.template second<X>(t)) + fabs(c.template second<Y>(t)) + fabs(c.template second<Z>(t));
  const T tv = c.ld(t);
  const T den = fabs(tv) + s / K.ph.q_max;
  const T q = c.ld(Am(VA_QQ, m));
  const T sb = den > T(0) ? qb / den : T(0);
  const T db = den > T(0) ? -(qb * q / den) : T(0);
  c.st(Am(VA_QB1, m), sb + db / K.ph.q_max);
  T tb = c.ld(Am(VA_TB, m)) * qfac(c, K, A, m);
  tb += tv > T(0) ? db : (tv < T(0) ? -db : T(0));
  c.st(Am(VA_TB, m), tb);
}
// The second differences' transposes, added to the stress's cotangent.
VJP_KERNEL k_quenchT2(VK<T, ALL> K) {
  VJP_CELL
  const int m = (int)blockIdx.y;
  const T* t = Am(VA_TAU, m);
  const T* sb = Am(VA_QB1, m);
  T tb = c.ld(Am(VA_TB, m));
  auto axis = [&](auto ax) {
    constexpr int AX = decltype(ax)::value;
    auto z = [&](int q) {
      if (!c.template hasax<AX>(q)) return T(0);
      const T d = c.template second<AX>(t, q);
      const T v = c.ld(sb, c.d[AX][q + 3]);
      return d > T(0) ? v : (d < T(0) ? -v : T(0));
    };
    // outputs on the end planes of a wall axis are 0 whatever the stress
    const bool wz = AX == Z && c.walled();
    const int N = b.nzt;
    T r = T(0);
    if (!wz || (c.k >= 1 && c.k <= N - 2)) r += T(-2) * z(0);
    if (!wz || c.k - 1 >= 1) r += z(-1);
    if (!wz || c.k + 1 <= N - 2) r += z(1);
    tb += r;
  };
  axis(std::integral_constant<int, X>{});
  axis(std::integral_constant<int, Y>{});
  axis(std::integral_constant<int, Z>{});
  c.st(Am(VA_TB, m), tb);
}

// ---------------------------------------------------------------------------
// Edge along C, between the axes P and Q: stress, E_C, the Lorentz products
// and the heating, backwards.  With u_P, p_P, B_P interpolated along Q and
// u_Q, p_Q, B_Q along P:
//   E = -(uP bQ - uQ bP) + eta J,  J = dd_P(B_Q) - dd_Q(B_P);
//   dp_P += dup_Q(tau - pP uQ) - up_Q(J bQ) / mu,
//   dp_Q += dup_P(tau - pQ uP) + up_P(J bP) / mu,
//   dB_P -= dup_Q(E), dB_Q += dup_P(E), de += up_P up_Q(2 tau S + eta J^2 / mu).
template <bool ALL, int C, class T, bool W, class F, class G, class H>
__device__ __forceinline__ void edge_back(const Cell<T, W>& c, const VArgs<T>& K, const Need& nd, const F& A, const G& Wt,
                                          const H& S) {
  constexpr int P = (C + 1) % 3, Q = (C + 2) % 3;
  const Phys<T>& ph = K.ph;
  const unsigned tm = nd.tm;
  const bool visc = tm & T_VISC, res = tm & T_RESIST, ind = tm & T_INDUCT, lor = tm & T_LORENTZ,
             adv = tm & T_ADV;
  const EdgeBase<ALL, C, T, W, F> E(c, A, nd);
  T uP = T(0), uQ = T(0), bP = T(0), bQ = T(0), J = T(0), g1 = T(0), g2 = T(0);
  if (ALL || nd.any(T_ADV | T_INDUCT)) {
    uP = c.template dn<Q>(A(VA_U + P));
    uQ = c.template dn<P>(A(VA_U + Q));
  }
  if (ALL || nd.any(T_INDUCT | T_LORENTZ)) {
    bP = c.template dn<Q>(S(5 + P));
    bQ = c.template dn<P>(S(5 + Q));
  }
  if (ALL || nd.any(T_RESIST | T_LORENTZ)) J = c.template ddn<P>(S(5 + Q)) - c.template ddn<Q>(S(5 + P));
  if (ALL || nd.any(T_VISC | T_ADV)) flux_cot<C>(c, Wt, g1, g2);
  T uPb = T(0), uQb = T(0), pPb = T(0), pQb = T(0), bPb = T(0), bQb = T(0), Jb = T(0), Sb = T(0), rb = T(0),
    nb = T(0);
  if (visc) {
    const T st = strain_e<C>(c, K, A);
    const T raw = E.rho * E.nu * st;
    T tb = g1 + g2 + T(2) * st * E.Qb, tau = raw;
    if (quenched(K)) {
      tau = raw * qfac(c, K, A, C);
      tb = c.ld(A(VA_TB + C));
    }
    Sb = T(2) * tau * E.Qb + E.rho * E.nu * tb;
    rb = E.nu * st * tb;
    nb = E.rho * st * tb;
  }
  if (adv) {
    const T pP = c.template dn<Q>(S(1 + P)), pQ = c.template dn<P>(S(1 + Q));
    pPb = -uQ * g1;
    uQb = -pP * g1;
    pQb = -uP * g2;
    uPb = -pQ * g2;
  }
  T Eb = T(0);
  if (ALL || nd.any(T_INDUCT | T_RESIST)) Eb = c.template dupT<P>(Wt(5 + Q)) - c.template dupT<Q>(Wt(5 + P));
  if (ind) {
    uPb -= bQ * Eb;
    bQb -= uP * Eb;
    uQb += bP * Eb;
    bPb += uQ * Eb;
  }
  if (res) {
    const T eta = ph.eta_const > T(0) ? ph.eta_const : ph.nuB * E.nu;
    const T jq = J * E.Qb * ph.inv_mu;
    Jb += eta * (Eb + T(2) * jq);
    if (!(ph.eta_const > T(0))) nb += ph.nuB * (J * (Eb + jq));
  }
  if (lor) {
    const T l1 = -(c.template upT<Q>(Wt(1 + P)) * ph.inv_mu), l2 = c.template upT<P>(Wt(1 + Q)) * ph.inv_mu;
    Jb += bQ * l1 + bP * l2;
    bQb += J * l1;
    bPb += J * l2;
  }
  auto put = [&](int q, T v) { c.st(A(VA_EDGE + C * EQ_COUNT + q), v); };
  if (ALL || nd.any(T_ADV | T_INDUCT)) {
    put(EQ_UAB, uPb);
    put(EQ_UBA, uQb);
  }
  if (ALL || nd.any(T_ADV)) {
    put(EQ_PAB, pPb);
    put(EQ_PBA, pQb);
  }
  if (ALL || nd.any(T_INDUCT | T_LORENTZ)) {
    put(EQ_BAB, bPb);
    put(EQ_BBA, bQb);
  }
  if (ALL || nd.any(T_RESIST | T_LORENTZ)) put(EQ_J, Jb);
  if (ALL || nd.any(T_VISC)) put(EQ_RHO, rb);
  if (ALL || nd.enu()) put(EQ_LNU, E.nu * nb);
  if (!(ALL || nd.shear())) return;
  const T hs = T(0.5) * Sb;
  if (order2(K)) {
    const bool r = (unsigned)c.ld(A(VA_RGF)) & (2u << C);
    put(EQ_HS, r ? T(0) : hs);
    c.st(A(VA_HS2 + C), r ? hs : T(0));
  } else {
    put(EQ_HS, hs);
  }
}

// Face normal to a: the energy flux H = -dn_a(e) u_a + nuE dn_a(rho) l
// dn_a(nu) dn_a(e_m) ddn_a(ln e_m), backwards; with T_LNP the pressure
// gradient exp(dn_a ln P) ddn_a ln P too (the plane mean of eq. pressure
// drops out of the product and of its derivative).
template <bool ALL, int AX, class T, bool W, class F, class G, class H>
__device__ __forceinline__ void face_back(const Cell<T, W>& c, const VArgs<T>& K, const Need& nd, const F& A, const G& Wt,
                                          const H& S) {
  const Phys<T>& ph = K.ph;
  const T Hb = c.template dupT<AX>(Wt(4));
  T xe = T(0), uf = T(0), rf = T(0), xn = T(0), xm = T(0), dl = T(0);
  if (nd.tm & T_ADV) {
    xe = -(c.ld(A(VA_U + AX)) * Hb);
    uf = -(c.template dn<AX>(S(4)) * Hb);
  }
  if (nd.tm & T_EDIFF) {
    const T l = (W && AX == Z && c.b.stretched) ? c.plane(ZJ_LZF) : T(c.b.lv[AX]);
    const T kr = ph.nuE * c.ld(A(VA_R + AX));
    const T ln = l * c.template dn<AX>(A(VA_NT));
    const T em = c.template dn<AX>(A(VA_EM));
    T dv = c.template ddn<AX>(A(VA_LEM));
    if (AX == Z && (nd.tm & T_EDIFFAV)) {
      // ln <e_m> of the offset's plane
      const double* pm = K.pm + c.b.poff;
      dv -= c.template op<Z, 1, 0>([&](unsigned f) { return T(log(T(pm[(c.o + f) / c.sz]))); });
    }
    rf = ph.nuE * ln * em * dv * Hb;
    xn = kr * l * em * dv * Hb;
    xm = kr * ln * dv * Hb;
    dl = kr * ln * em * Hb;
  }
  if (ALL || nd.any(T_ADV)) {
    c.st(A(VA_XE + AX), xe);
    c.st(A(VA_UF + AX), uf);
  }
  if (ALL || nd.any(T_EDIFF)) {
    c.st(A(VA_RF + AX), rf);
    c.st(A(VA_XNT + AX), xn);
    c.st(A(VA_XEM + AX), xm);
    c.st(A(VA_DLEM + AX), dl);
  }
  if (nd.lnp()) {
    const T gb = -c.ld(Wt(1 + AX)) * exp(c.template dn<AX>(A(VA_LNP)));
    c.st(A(VA_QI + AX), gb * c.template ddn<AX>(A(VA_LNP)));
    c.st(A(VA_QD + AX), gb);
  }
}

// Edges (roles 0..2, the direction) and faces (3..5, the normal); the launch
// takes the roles from `role` on.
VJP_KERNEL_WAVES(5) k_edge_face(VK<T, ALL> K, int role) {
  VJP_CELL
  switch ((ALL ? 0 : role) + (int)blockIdx.y) {
    case 0: edge_back<ALL, X>(c, K, nd, A, Wt, S); break;
    case 1: edge_back<ALL, Y>(c, K, nd, A, Wt, S); break;
    case 2: edge_back<ALL, Z>(c, K, nd, A, Wt, S); break;
    case 3: face_back<ALL, X>(c, K, nd, A, Wt, S); break;
    case 4: face_back<ALL, Y>(c, K, nd, A, Wt, S); break;
    default: face_back<ALL, Z>(c, K, nd, A, Wt, S); break;
  }
}

// The edges' ln nu gathered along their second axis, and with the optional
// terms the cotangents of div B and of the plane means' log.
VJP_KERNEL k_lines_back(VK<T, ALL> K) {
  VJP_CELL
  auto Eq = [&](int e, int q) { return A(VA_EDGE + e * EQ_COUNT + q); };
  if (ALL || nd.enu()) {
    c.st(A(VA_XLB), c.template dnT<Y>(Eq(Z, EQ_LNU)) + c.template dnT<Z>(Eq(Y, EQ_LNU)));
    c.st(A(VA_YLB), c.template dnT<Z>(Eq(X, EQ_LNU)));
  }
  if ((tm & T_DIVB) && K.dt > 0.0) {
    const T kd = T(K.c_divb / K.dt * b.hmin) * T(b.hmin);
    c.st(A(VA_DVB), kd * (c.template ddnT<X>(Wt(5)) + c.template ddnT<Y>(Wt(6)) + c.template ddnT<Z>(Wt(7))));
  }
  if (nd.ediffav()) c.st(A(VA_EDX), c.template ddnT<Z>(A(VA_DLEM + Z)));
}

// Cotangent of a centre stress component: momentum flux and heating, or the
// quenching's transpose.
template <int AX, class T, bool W, class F, class G>
__device__ __forceinline__ T taub_centre(const Cell<T, W>& c, const VArgs<T>& K, const F& A, const G& Wt, T vs, T we) {
  if (quenched(K)) return c.ld(A(VA_TB + 3 + AX));
  return c.template ddnT<AX>(Wt(1 + AX)) + vs * we;
}

// <nu>: from the centre stress, the faces and the edges' logs.
VJP_KERNEL k_nu_back(VK<T, ALL> K) {
  VJP_CELL
  const T nt = c.ld(A(VA_NT));
  T nb = T(0);
  if (tm & T_VISC) {
    const Centre<T, W, decltype(A)> E(c, K, A);
    const T we = c.ld(Wt(4)), rho = c.ld(S(0));
    const T tb[3] = {taub_centre<X>(c, K, A, Wt, E.vs[0], we), taub_centre<Y>(c, K, A, Wt, E.vs[1], we),
                     taub_centre<Z>(c, K, A, Wt, E.vs[2], we)};
#pragma unroll
    for (int a = 0; a < 3; ++a) nb += rho * len_c(c, a) * (E.vs[a] + K.ph.c1 * E.vD) * tb[a];
  }
  if (ALL || nd.any(T_EDIFF))
    nb += c.template dnT<X>(A(VA_XNT)) + c.template dnT<Y>(A(VA_XNT + 1)) + c.template dnT<Z>(A(VA_XNT + 2));
  if (ALL || nd.enu()) nb += (c.template dnT<X>(A(VA_XLB)) + c.template dnT<Y>(A(VA_YLB))) / nt;
  c.st(A(VA_NTB), nt > T(1e-30) ? nb : T(0));
}

// Transpose of the three-cell means: on a wall axis output q averages over
// 2 cells at an end, else 3.
VJP_KERNEL k_mean_back(VK<T, ALL> K) {
  VJP_CELL
  const T* a = A(VA_NTB);
  const int N = b.nzt;
  auto zc = [&](unsigned f) {
    auto cnt = [&](int q) { return T(c.walled() && (q == 0 || q == N - 1) ? 2 : 3); };
    T s = c.ld(a, f) / cnt(c.k);
    if (c.has(-1)) s += c.ld(a, f + c.d[Z][2]) / cnt(c.k - 1);
    if (c.has(1)) s += c.ld(a, f + c.d[Z][4]) / cnt(c.k + 1);
    return s;
  };
  auto yc = [&](unsigned f) { return (zc(f + c.d[Y][2]) + zc(f) + zc(f + c.d[Y][4])) / T(3); };
  c.st(A(VA_MB0), (yc(c.d[X][2]) + yc(0u) + yc(c.d[X][4])) / T(3));
}

// Centre: the stress, the diagonal momentum fluxes, -P div u and the
// speed-like viscosity (mb: the cotangent of its first maximum), backwards.
VJP_KERNEL_WAVES(5) k_centre_back(VK<T, ALL> K, int mb) {
  VJP_CELL
  const Phys<T>& ph = K.ph;
  const Centre<T, W, decltype(A)> E(c, K, A, ALL || nd.strain());
  const T rho = c.ld(S(0)), e = c.ld(S(4)), nt = ALL || nd.any(T_VISC) ? c.ld(A(VA_NT)) : T(0), we = c.ld(Wt(4));
  const T P = ph.gamma1 * e;
  T Db = T(0), vDb = T(0), rb = T(0), Pb = T(0);
  T vsb[3] = {}, sb[3] = {}, cp[3] = {}, cu[3] = {}, cb[3] = {};
  const bool vel = ALL || nd.cu(), flux = ALL || nd.any(T_VISC | T_ADV);
  const T uc[3] = {vel ? c.template up<X>(A(VA_U)) : T(0), vel ? c.template up<Y>(A(VA_U + 1)) : T(0),
                   vel ? c.template up<Z>(A(VA_U + 2)) : T(0)};
  const T gf[3] = {flux ? c.template ddnT<X>(Wt(1)) : T(0), flux ? c.template ddnT<Y>(Wt(2)) : T(0),
                   flux ? c.template ddnT<Z>(Wt(3)) : T(0)};
  if (tm & T_VISC) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const T rn = rho * (len_c(c, a) * nt), m = E.vs[a] + ph.c1 * E.vD;
      T tb, t = rn * m;
      if (quenched(K)) {
        t = t * qfac(c, K, A, 3 + a);
        tb = c.ld(A(VA_TB + 3 + a));
      } else {
        tb = gf[a] + E.vs[a] * we;
      }
      vsb[a] = t * we + rn * tb;
      vDb += ph.c1 * rn * tb;
      rb += len_c(c, a) * nt * m * tb;
    }
  }
  if (tm & T_ADV) {
    const T pc[3] = {c.template up<X>(S(1)), c.template up<Y>(S(2)), c.template up<Z>(S(3))};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      cp[a] = -(uc[a] * gf[a]);
      cu[a] = -(pc[a] * gf[a]);
    }
  }
  if (tm & T_PRES) {
    Pb -= E.D * we;
    Db -= P * we;
  }
  if (ALL ? !nd.cst : nd.chain()) {
    const T nb = c.template max3T<X>(A(VA_MX), An(mb));
    const T ub = vnorm3(uc[0], uc[1], uc[2]);
    const T wu = ub > T(0) ? ph.nu1 * nb / ub : T(0);
    const T bc[3] = {c.template up<X>(S(5)), c.template up<Y>(S(6)), c.template up<Z>(S(7))};
    const T bb = vnorm3(bc[0], bc[1], bc[2]);
    const T v3 = ph.nu3 * nb;
    const T sr = sqrt(ph.mu * rho), ca = bb / sr, bbb = v3 / sr;
    rb -= ph.mu * (v3 * ca / sr) / (T(2) * sr);
    const T arg = ph.gamma * P / rho, cs = sqrt(arg);
    const T ab = cs > T(0) ? v3 / (T(2) * cs) : T(0);
    Pb += ph.gamma * (ab / rho);
    rb -= ab * arg / rho;
    const T wb = bb > T(0) ? bbb / bb : T(0);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      cu[a] += wu * uc[a];
      cb[a] = wb * bc[a];
    }
    if (-E.D > T(0)) Db -= T(K.nu2 * h_shock(c)) * nb;
    if (smag(K)) {
      const T q[3] = {c.ld(A(VA_SC)), c.ld(A(VA_SC + 1)), c.ld(A(VA_SC + 2))};
      const T s2 = T(2) * (E.s[0] * E.s[0] + E.s[1] * E.s[1] + E.s[2] * E.s[2] - E.D * E.D * T(1.0 / 3.0) +
                           T(2) * (q[0] * q[0] + q[1] * q[1] + q[2] * q[2]));
      const T s2b = s2 > T(0) ? T(K.c_smag * h_shock(c)) * nb / (T(2) * sqrt(s2)) : T(0);
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        sb[a] = T(4) * E.s[a] * s2b;
        c.st(A(VA_SC + a), T(8) * q[a] * s2b);
      }
      Db -= T(4.0 / 3.0) * E.D * s2b;
    }
  }
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    T v6 = sb[a] + Db, v2 = vsb[a] + vDb;
    if (!E.rough) {
      v6 += v2;
      v2 = T(0);
    }
    if (ALL || nd.strain()) c.st(A(VA_SD + a), v6);
    if (order2(K)) c.st(A(VA_SD2 + a), v2);
    if (ALL || nd.any(T_ADV)) c.st(A(VA_CP + a), cp[a]);
    if (ALL || nd.cu()) c.st(A(VA_CU + a), cu[a]);
    if (ALL || nd.chain()) c.st(A(VA_CB + a), cb[a]);
  }
  T eb = ph.gamma1 * Pb;
  // Newtonian cooling (eq. NewtonCool, eq. rhocool): -(e - rho e_cool) / t
  // times r2 / (1 + r2) or 1 / (1 + r2)
  if (tm & T_COOL) {
    T fac = T(1), dfac = T(0);
    if (ph.cool_cut) {
      const T r = rho * ph.inv_rho_cool, r2 = r * r, d = T(1) / (T(1) + r2);
      fac = (ph.cool_cut == 1 ? r2 : T(1)) * d;
      dfac = (ph.cool_cut == 1 ? T(2) : T(-2)) * r * d * d * ph.inv_rho_cool;
    }
    eb -= ph.inv_tcool * fac * we;
    rb += (ph.e_cool * fac - (e - rho * ph.e_cool) * dfac) * ph.inv_tcool * we;
  }
  if (ALL || nd.rhob()) c.st(A(VA_RHOB), rb);
  if (ALL || nd.eb()) c.st(A(VA_EB), eb);
}

// T_SMAG: the centre shear's cotangents back on the edges.
VJP_KERNEL k_smag_back(VK<T, ALL> K) {
  VJP_CELL
  const int e = (int)blockIdx.y;
  const T v = e == X ? c.template iiT<Y, 1, Z, 1>(A(VA_SC))
                     : (e == Y ? c.template iiT<X, 1, Z, 1>(A(VA_SC + 1)) : c.template iiT<X, 1, Y, 1>(A(VA_SC + 2)));
  auto hs = [&](int edge) { return A(VA_EDGE + edge * EQ_COUNT + EQ_HS); };
  T* h = e == X ? hs(X) : (e == Y ? hs(Y) : hs(Z));
  c.st(h, c.ld(h) + T(0.5) * v);
}

template <class T, bool W>
__device__ __forceinline__ void add_to(const Cell<T, W>& c, const VArgs<T>& K, int v, T x) {
  T* g = K.g.p[v] + c.b.off;
  c.st(g, K.acc ? c.ld(g) + x : x);
}

// Component a of the velocity: every gather, then the momentum and the face
// density it came from.
template <bool ALL, int AX, class T, bool W, class F, class G>
__device__ __forceinline__ void vel_back(const Cell<T, W>& c, const VArgs<T>& K, const Need& nd, const F& A, const G& Wt) {
  constexpr int B1 = (AX + 1) % 3, A2 = (AX + 2) % 3;   // edges along A2 (as P) and along B1 (as Q)
  auto Eq = [&](int e, int q) { return A(VA_EDGE + e * EQ_COUNT + q); };
  T ub = T(0), pb = T(0), rf = T(0);
  const bool ui = ALL || nd.any(T_ADV | T_INDUCT);
  if (ALL || nd.any(T_ADV)) ub += c.ld(A(VA_UF + AX));
  if (ui) ub += c.template dnT<B1>(Eq(A2, EQ_UAB));
  if (ALL || nd.shear()) ub += c.template ddnT<B1>(Eq(A2, EQ_HS));
  if (ui) ub += c.template dnT<A2>(Eq(B1, EQ_UBA));
  if (ALL || nd.shear()) ub += c.template ddnT<A2>(Eq(B1, EQ_HS));
  if (ALL || nd.cu()) ub += c.template upT<AX>(A(VA_CU + AX));
  if (ALL || nd.strain()) ub += c.template dupT<AX>(A(VA_SD + AX));
  if (order2(K))
    ub += c.template d2nT<B1>(A(VA_HS2 + A2)) + c.template d2nT<A2>(A(VA_HS2 + B1)) +
          c.template d2uT<AX>(A(VA_SD2 + AX));
  if (ALL || nd.any(T_ADV))
    pb += c.template dnT<B1>(Eq(A2, EQ_PAB)) + c.template dnT<A2>(Eq(B1, EQ_PBA)) + c.template upT<AX>(A(VA_CP + AX));
  if (nd.tm & T_CONT) pb -= c.template dupT<AX>(Wt(0));
  if (nd.tm & T_CORI) {
    // p_AX drives dp_P and dp_Q (P, Q the next axes): -2 Omega x p
    pb += K.ph.cor2[A2] * c.template iiT<AX, 1, B1, 0>(Wt(1 + B1)) * T(-1);
    pb += K.ph.cor2[B1] * c.template iiT<AX, 1, A2, 0>(Wt(1 + A2));
  }
  if (ALL || nd.faces()) {
    const T r = c.ld(A(VA_R + AX));
    const T q = ub / r;
    if (ALL || nd.any(T_EDIFF)) rf = c.ld(A(VA_RF + AX));
    T rb = rf - q * c.ld(A(VA_U + AX));
    if (ALL || nd.any(T_VISC)) {
      if constexpr (AX == X) rb += c.template dnT<Y>(Eq(Z, EQ_RHO)) + c.template dnT<Z>(Eq(Y, EQ_RHO));
      if constexpr (AX == Y) rb += c.template dnT<Z>(Eq(X, EQ_RHO));
    }
    c.st(A(VA_RB + AX), rb);
    pb += q;
  }
  add_to(c, K, 1 + AX, pb);
}
template <bool ALL, int AX, class T, bool W, class F>
__device__ __forceinline__ void field_back(const Cell<T, W>& c, const VArgs<T>& K, const Need& nd, const F& A) {
  constexpr int B1 = (AX + 1) % 3, A2 = (AX + 2) % 3;
  auto Eq = [&](int e, int q) { return A(VA_EDGE + e * EQ_COUNT + q); };
  T v = T(0);
  const bool bq = ALL || nd.any(T_INDUCT | T_LORENTZ), jq = ALL || nd.any(T_RESIST | T_LORENTZ);
  if (bq) v += c.template dnT<B1>(Eq(A2, EQ_BAB));
  if (jq) v -= c.template ddnT<B1>(Eq(A2, EQ_J));
  if (bq) v += c.template dnT<A2>(Eq(B1, EQ_BBA));
  if (jq) v += c.template ddnT<A2>(Eq(B1, EQ_J));
  if (ALL || nd.chain()) v += c.template upT<AX>(A(VA_CB + AX));
  if ((K.ph.terms & T_DIVB) && K.dt > 0.0) v += c.template dupT<AX>(A(VA_DVB));
  add_to(c, K, 5 + AX, v);
}
// blockIdx.y 0..2 the velocities, 3..5 the magnetic field.
VJP_KERNEL_WAVES(6) k_vector_back(VK<T, ALL> K) {
  VJP_CELL
  switch (blockIdx.y) {
    case 0: vel_back<ALL, X>(c, K, nd, A, Wt); break;
    case 1: vel_back<ALL, Y>(c, K, nd, A, Wt); break;
    case 2: vel_back<ALL, Z>(c, K, nd, A, Wt); break;
    case 3: field_back<ALL, X>(c, K, nd, A); break;
    case 4: field_back<ALL, Y>(c, K, nd, A); break;
    default: field_back<ALL, Z>(c, K, nd, A); break;
  }
}

// e_m, the pressure gradient and gravity, then e and rho.
VJP_KERNEL k_scalar_back(VK<T, ALL> K) {
  VJP_CELL
  const Phys<T>& ph = K.ph;
  T eb = T(0), rb = T(0), rho = T(1), em = T(1);
  if (ALL || nd.any(T_EDIFF)) {
    rho = c.ld(S(0));
    em = c.ld(A(VA_EM));
  }
  if (ALL || nd.eb()) eb += c.ld(A(VA_EB));
  if (ALL || nd.any(T_ADV))
    eb = eb + c.template dnT<X>(A(VA_XE)) + c.template dnT<Y>(A(VA_XE + 1)) + c.template dnT<Z>(A(VA_XE + 2));
  if (tm & T_PRES) {
    if (tm & T_LNP)
      eb += (c.template dnT<X>(A(VA_QI)) + c.template ddnT<X>(A(VA_QD)) + c.template dnT<Y>(A(VA_QI + 1)) +
             c.template ddnT<Y>(A(VA_QD + 1)) + c.template dnT<Z>(A(VA_QI + 2)) + c.template ddnT<Z>(A(VA_QD + 2))) /
            c.ld(S(4));
    else
      eb -= ph.gamma1 * (c.template ddnT<X>(Wt(1)) + c.template ddnT<Y>(Wt(2)) + c.template ddnT<Z>(Wt(3)));
  }
  if (ALL || nd.rhob()) rb += c.ld(A(VA_RHOB));
  if (ALL || nd.faces())
    rb = rb + c.template dnT<X>(A(VA_RB)) + c.template dnT<Y>(A(VA_RB + 1)) + c.template dnT<Z>(A(VA_RB + 2));
  if (tm & T_GRAV) rb -= ph.gz * c.template dnT<Z>(Wt(3));
  if (tm & T_EDIFF) {
    T mb = c.template dnT<X>(A(VA_XEM)) + c.template dnT<Y>(A(VA_XEM + 1)) + c.template dnT<Z>(A(VA_XEM + 2)) +
           (c.template ddnT<X>(A(VA_DLEM)) + c.template ddnT<Y>(A(VA_DLEM + 1)) + c.template ddnT<Z>(A(VA_DLEM + 2))) /
               em;
    if (tm & T_EDIFFAV)   // the plane mean's log: its cells' cotangents summed over the plane
      mb -= T(K.pm[K.nplanes + b.poff + c.k]) / T(K.pm[b.poff + c.k]);
    const T q = mb / rho;
    eb += q;
    rb -= q * em;
  }
  add_to(c, K, 4, eb);
  add_to(c, K, 0, rb);
}

// The mean of src over each z plane of every box, in float64 and a fixed
// order (one workgroup per plane).
constexpr int kPlaneBlock = 256;
template <class T>
__global__ __launch_bounds__(kPlaneBlock) void k_plane_mean(const BoxDev* __restrict__ boxes, int nbox,
                                                           const T* __restrict__ src, double* __restrict__ pm) {
  __shared__ double sh[kPlaneBlock];
  const int P = (int)blockIdx.x;
  int bi = 0;
  while (bi + 1 < nbox && boxes[bi + 1].poff <= P) ++bi;
  const BoxDev& b = boxes[bi];
  const int n = b.nx * b.ny;
  const T* __restrict__ s = src + b.off + (long long)(P - b.poff) * n;
  double acc = 0.0;
  for (int i = threadIdx.x; i < n; i += kPlaneBlock) acc += (double)s[i];
  sh[threadIdx.x] = acc;
  __syncthreads();
  for (int w = kPlaneBlock / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) pm[P] = sh[0] / (double)n;
}

template <class T>
__global__ __launch_bounds__(kBlock) void k_axpby8(const BoxDev* boxes, const Blk* tab, P8<T> y, CP8<T> x, T a, T bx,
                                                   int mask) {
  const Blk t = tab[blockIdx.x];
  if ((int)threadIdx.x >= t.n) return;
  const BoxDev& b = boxes[t.box];
  const unsigned q = (unsigned)t.start + threadIdx.x;
  const long long o = b.off + q;
  const int k = (int)(q / ((unsigned)b.nx * (unsigned)b.ny));
  const bool cen = !mask || !b.wall || (k >= b.g0 && k < b.g1);
  T yv[8], xv[8];
#pragma unroll
  for (int v = 0; v < 8; ++v) {
    yv[v] = a == T(0) ? T(0) : a * y.p[v][o];
    xv[v] = bx * x.p[v][o];
  }
#pragma unroll
  for (int v = 0; v < 8; ++v) {
    bool keep = cen;
    if (mask && b.wall && v == 3) keep = k > b.g0 && k < b.g1;
    if (mask && b.wall && v == 7) keep = k >= b.g0 && k <= b.g1;
    y.p[v][o] = keep ? yv[v] + xv[v] : T(0);
  }
}

template <class T, bool W, bool ALL>
void run(const VjpLaunch& L, const VK<T, ALL>& K) {
  const int g = 8 * ((L.nblk + 7) / 8);
  const dim3 blk(kBlock);
  auto go = [&](auto* kern, int roles, auto... args) {
    hipLaunchKernelGGL(kern, dim3(g, roles), blk, 0, L.stream, K, args...);
  };
  auto slot = [&](int id) { return K.slot(id); };
  auto max1 = [&](int ax, int src, int dst) {
    auto* kern = ax == X ? k_max1<T, W, ALL, X> : (ax == Y ? k_max1<T, W, ALL, Y> : k_max1<T, W, ALL, Z>);
    go(kern, 1, slot(src), slot(dst));
  };
  auto max1T = [&](int ax, int prim, int yb, int dst, int comps) {
    auto* kern = ax == X ? k_max1T<T, W, ALL, X> : (ax == Y ? k_max1T<T, W, ALL, Y> : k_max1T<T, W, ALL, Z>);
    go(kern, comps, slot(prim), slot(yb), slot(dst));
  };
  auto plane_mean = [&](int id, double* pm) {
    hipLaunchKernelGGL(k_plane_mean<T>, dim3(L.nplanes), dim3(kPlaneBlock), 0, L.stream, L.boxes, L.nbox,
                       (const T*)(K.base + (long long)slot(id) * K.stride), pm);
  };
  const Need nd(K.ph);
  const bool chain = ALL ? !nd.cst : nd.chain(), smag = chain && nd.any(T_SMAG);
  const bool edges = ALL || nd.edges(), fluxes = ALL || nd.fluxes();
  if (ALL || nd.faces() || nd.heat()) go(k_prim<T, W, ALL>, 1);
  if (nd.ediffav()) plane_mean(VA_EM, L.pm);
  if (nd.order2()) {
    go(k_rough<T, W, ALL>, 1);
    go(k_rough_flags<T, W, ALL>, 1);
  }
  if (chain) {
    if (smag) go(k_shear<T, W, ALL>, 3);
    go(k_nus<T, W, ALL>, 1);
    if (K.nmax == 6)
      for (int m = 0; m < 6; ++m) max1(m / 2, mx_id(m), mx_id(m + 1));
    else
      go(k_max3<T, W, ALL>, 1);
  }
  if (ALL || nd.nu()) go(k_mean<T, W, ALL>, 1, slot(mx_id(K.nmax)));
  if (ALL || nd.enu()) go(k_lines<T, W, ALL>, 1);
  if (nd.quench()) {
    go(k_tau<T, W, ALL>, 4);
    go(k_quench<T, W, ALL>, 6);
    go(k_quench_max<T, W, ALL>, 6);
    go(k_taub<T, W, ALL>, 4);
    max1T(Z, VA_Q2, VA_QB0, VA_QB1, 6);
    max1T(Y, VA_Q1, VA_QB1, VA_QB0, 6);
    go(k_quenchT<T, W, ALL>, 6);
    go(k_quenchT2<T, W, ALL>, 6);
  }
  if (edges || fluxes) go(k_edge_face<T, W, ALL>, edges && fluxes ? 6 : 3, edges ? 0 : 3);
  if (ALL || nd.enu() || nd.ediffav() || (nd.any(T_DIVB) && K.dt > 0.0)) go(k_lines_back<T, W, ALL>, 1);
  if (nd.ediffav()) plane_mean(VA_EDX, L.pm + L.nplanes);
  int mb = VA_MB0;
  if (chain) {
    go(k_nu_back<T, W, ALL>, 1);
    go(k_mean_back<T, W, ALL>, 1);
    // back through the maxima but the first, which the centre pass takes
    for (int m = K.nmax - 1; m > 0; --m) {
      const int to = mb == VA_MB0 ? VA_MB1 : VA_MB0;
      max1T(K.nmax == 6 ? m / 2 : m, mx_id(m), mb, to, 1);
      mb = to;
    }
  }
  if (ALL || nd.centre()) go(k_centre_back<T, W, ALL>, 1, slot(mb));
  if (smag) go(k_smag_back<T, W, ALL>, 3);
  go(k_vector_back<T, W, ALL>, 6);
  go(k_scalar_back<T, W, ALL>, 1);
}

}  // namespace

template <class T> int vjp_arrays(const Phys<T>& ph) {
  unsigned char at[VA_COUNT];
  bool all;
  return std::max(layout(Need(ph), at, all), kFillTmp);
}
template int vjp_arrays<float>(const Phys<float>&);
template int vjp_arrays<double>(const Phys<double>&);

template <class T>
void vjp_rhs(const VjpLaunch& L, const Phys<T>& ph, double nu2, double c_smag, double c_divb, CP8<T> s, CP8<T> w,
             P8<T> g, bool acc, T* base, long long stride, double dt) {
  auto set = [&](VArgs<T>& K) {
    K.boxes = L.boxes;
    K.tab = L.tab;
    K.nblk = L.nblk;
    K.s = s;
    K.w = w;
    K.g = g;
    K.base = base;
    K.stride = stride;
    K.zt = static_cast<const T*>(L.ztab);
    K.pm = L.pm;
    K.nplanes = L.nplanes;
    K.ph = ph;
    K.nu2 = nu2;
    K.c_smag = c_smag;
    K.c_divb = c_divb;
    K.dt = dt;
    K.acc = acc ? 1 : 0;
    K.nmax = (ph.terms & T_MAX5) ? 6 : 3;
  };
  VK<T, true> every;
  VK<T, false> lean;
  bool all;
  (void)layout(Need(ph), lean.at, all);
  if (all) {
    set(every);
    L.wall ? run<T, true, true>(L, every) : run<T, false, true>(L, every);
  } else {
    set(lean);
    L.wall ? run<T, true, false>(L, lean) : run<T, false, false>(L, lean);
  }
}

template <class T> void vjp_axpby8(const VjpLaunch& L, P8<T> y, CP8<T> x, double a, double b, bool mask) {
  hipLaunchKernelGGL(k_axpby8<T>, dim3(L.nblk), dim3(kBlock), 0, L.stream, L.boxes, L.tab, y, x, T(a), T(b),
                     mask ? 1 : 0);
}

// ---------------------------------------------------------------------------
// Transpose of the closed-wall ghost fill (Section 10 "Closed"), linearised
// at the filled state s.  The fill sets, on ghost plane k at distance d from
// the wall, from interior planes a0 (next to the wall) and a1:
//   rho_k = exp(L_r), L_r = (1 + d) ln rho_a0 - d ln rho_a1,
//   e_k = rho_k exp(L_m), L_m the same of ln(e / rho),
//   p_x,k = X_k p_x,m / X_m with X = xdn(rho) on planes k and m (the mirror
//   across the wall; p_y with ydn), B_x,k = -B_x,m, B_y,k = -B_y,m,
//   p_z and B_z beyond the wall face mirrored (- and +), p_z = 0 on both
//   wall faces.
// One thread per ghost cell of one side (lower side 0, upper 1; the sides
// run apart, since their mirror planes can meet in a shallow box), in three
// launches: (1) the cotangents of X_k and X_m of each ghost p_x, p_y cell
// into tmp 0..3 and the mirror contributions to p_x, p_y, B and p_z; (2) the
// cotangent of the ghost density (through X_k and e_k), of L_r and L_m into
// tmp 4, 5, and that of the mirror density through X_m; (3) per column the
// sums over the side's ghost planes into rho and e at a0 and a1, and the
// ghost cotangents cleared.
namespace {
struct GhostCell {
  int i, j, k, m, d, a0, a1;
  bool lower;
};
__device__ __forceinline__ bool ghost_cell(const BoxDev& b, const Blk& t, int side, GhostCell& c) {
  long long q = t.start + threadIdx.x;   // over nx * ny * (2 ngz)
  c.i = (int)(q % b.nx);
  q /= b.nx;
  c.j = (int)(q % b.ny);
  const int s = (int)(q / b.ny);
  c.lower = s < b.ngz;
  if (c.lower != (side == 0)) return false;
  c.k = c.lower ? s : b.g1 + (s - b.ngz);
  c.d = c.lower ? b.g0 - c.k : c.k - b.g1 + 1;
  c.m = c.lower ? 2 * b.g0 - 1 - c.k : 2 * b.g1 - 1 - c.k;
  c.a0 = c.lower ? b.g0 : b.g1 - 1;
  c.a1 = c.lower ? b.g0 + 1 : b.g1 - 2;
  return true;
}
}  // namespace

template <class T>
__global__ __launch_bounds__(kBlock) void k_fill_vjp1(const BoxDev* boxes, const Blk* gtab, int side, CP8<T> s,
                                                      P8<T> g, T* t0, T* t1, T* t2, T* t3) {
  const Blk t = gtab[blockIdx.x];
  if ((int)threadIdx.x >= t.n) return;
  const BoxDev& b = boxes[t.box];
  GhostCell c;
  if (!ghost_cell(b, t, side, c)) return;
  const Geo<T> G(b);
  const int i = c.i, j = c.j, k = c.k, m = c.m;
  const long long o = G.at(i, j, k), om = G.at(i, j, m);
  const T* rho = s.p[0];
  const T xk = op6<0, 0, T>([&](int l) { return rho[G.at(i + l, j, k)]; }, T(0));
  const T xm = op6<0, 0, T>([&](int l) { return rho[G.at(i + l, j, m)]; }, T(0));
  const T yk = op6<0, 0, T>([&](int l) { return rho[G.at(i, j + l, k)]; }, T(0));
  const T ym = op6<0, 0, T>([&](int l) { return rho[G.at(i, j + l, m)]; }, T(0));
  const T gpx = g.p[1][o], gpy = g.p[2][o];
  const T pxm = s.p[1][om], pym = s.p[2][om];
  t0[o] = gpx * (pxm / xm);
  t1[o] = gpy * (pym / ym);
  t2[o] = -(gpx * (xk * pxm / xm) / xm);
  t3[o] = -(gpy * (yk * pym / ym) / ym);
  g.p[1][om] += gpx * (xk / xm);
  g.p[2][om] += gpy * (yk / ym);
  g.p[5][om] -= g.p[5][o];
  g.p[6][om] -= g.p[6][o];
  // z-faces beyond the wall face mirror the faces inside it
  if (c.lower || k != b.g1) {
    const long long of = G.at(i, j, c.lower ? 2 * b.g0 - k : 2 * b.g1 - k);
    g.p[3][of] -= g.p[3][o];
    g.p[7][of] += g.p[7][o];
  }
}

template <class T>
__global__ __launch_bounds__(kBlock) void k_fill_vjp2(const BoxDev* boxes, const Blk* gtab, int side, CP8<T> s,
                                                      P8<T> g, const T* t0, const T* t1, const T* t2,
                                                      const T* t3, T* t4, T* t5) {
  const Blk t = gtab[blockIdx.x];
  if ((int)threadIdx.x >= t.n) return;
  const BoxDev& b = boxes[t.box];
  GhostCell c;
  if (!ghost_cell(b, t, side, c)) return;
  const Geo<T> G(b);
  const int i = c.i, j = c.j, k = c.k;
  const long long o = G.at(i, j, k), om = G.at(i, j, c.m);
  // transposes of xdn, ydn on a periodic axis: xup, yup
  const T rk = g.p[0][o] + op6<0, 1, T>([&](int l) { return t0[G.at(i + l, j, k)]; }, T(0)) +
               op6<0, 1, T>([&](int l) { return t1[G.at(i, j + l, k)]; }, T(0));
  const T rn = s.p[0][o], en = s.p[4][o], ge = g.p[4][o];
  t4[o] = (rk + ge * (en / rn)) * rn;
  t5[o] = ge * en;
  g.p[0][om] += op6<0, 1, T>([&](int l) { return t2[G.at(i + l, j, k)]; }, T(0)) +
                op6<0, 1, T>([&](int l) { return t3[G.at(i, j + l, k)]; }, T(0));
}

template <class T>
__global__ __launch_bounds__(kBlock) void k_fill_vjp3(const BoxDev* boxes, const Blk* gtab, int side, CP8<T> s,
                                                      P8<T> g, const T* t4, const T* t5) {
  const Blk t = gtab[blockIdx.x];
  if ((int)threadIdx.x >= t.n) return;
  const BoxDev& b = boxes[t.box];
  GhostCell c;
  if (!ghost_cell(b, t, side, c)) return;
  const Geo<T> G(b);
  const int i = c.i, j = c.j, k = c.k;
  const long long o = G.at(i, j, k);
  if (c.d == 1) {
    // L_r and L_m of every ghost plane of this side, into ln rho, ln e_m at a0, a1
    T lr0 = T(0), lr1 = T(0), lm0 = T(0), lm1 = T(0);
    for (int dd = 1; dd <= b.ngz; ++dd) {
      const long long oq = G.at(i, j, c.lower ? b.g0 - dd : b.g1 - 1 + dd);
      lr0 += T(1 + dd) * t4[oq];
      lr1 -= T(dd) * t4[oq];
      lm0 += T(1 + dd) * t5[oq];
      lm1 -= T(dd) * t5[oq];
    }
    const long long o0 = G.at(i, j, c.a0), o1 = G.at(i, j, c.a1);
    // ln e_m = ln e - ln rho
    g.p[0][o0] += (lr0 - lm0) / s.p[0][o0];
    g.p[4][o0] += lm0 / s.p[4][o0];
    g.p[0][o1] += (lr1 - lm1) / s.p[0][o1];
    g.p[4][o1] += lm1 / s.p[4][o1];
    if (c.lower) g.p[3][G.at(i, j, b.g0)] = T(0);   // p_z on the lower wall face
  }
  // the fill overwrites every ghost value except B_z on the upper wall face
#pragma unroll
  for (int v = 0; v < 8; ++v)
    if (!(v == 7 && k == b.g1)) g.p[v][o] = T(0);
}

template <class T> void vjp_fill(const VjpLaunch& L, CP8<T> s, P8<T> g, T* tmp, long long stride) {
  if (L.nghost_blk == 0) return;
  T* t[6];
  for (int q = 0; q < 6; ++q) t[q] = tmp + (long long)q * stride;
  for (int side = 0; side < 2; ++side) {
    hipLaunchKernelGGL(k_fill_vjp1<T>, dim3(L.nghost_blk), dim3(kBlock), 0, L.stream, L.boxes, L.gtab, side, s,
                       g, t[0], t[1], t[2], t[3]);
    hipLaunchKernelGGL(k_fill_vjp2<T>, dim3(L.nghost_blk), dim3(kBlock), 0, L.stream, L.boxes, L.gtab, side, s,
                       g, (const T*)t[0], (const T*)t[1], (const T*)t[2], (const T*)t[3], t[4], t[5]);
    hipLaunchKernelGGL(k_fill_vjp3<T>, dim3(L.nghost_blk), dim3(kBlock), 0, L.stream, L.boxes, L.gtab, side, s,
                       g, (const T*)t[4], (const T*)t[5]);
  }
}

template void vjp_rhs<float>(const VjpLaunch&, const Phys<float>&, double, double, double, CP8<float>, CP8<float>,
                            P8<float>, bool, float*, long long, double);
template void vjp_rhs<double>(const VjpLaunch&, const Phys<double>&, double, double, double, CP8<double>,
                             CP8<double>, P8<double>, bool, double*, long long, double);
template void vjp_axpby8<float>(const VjpLaunch&, P8<float>, CP8<float>, double, double, bool);
template void vjp_axpby8<double>(const VjpLaunch&, P8<double>, CP8<double>, double, double, bool);
template void vjp_fill<float>(const VjpLaunch&, CP8<float>, P8<float>, float*, long long);
template void vjp_fill<double>(const VjpLaunch&, CP8<double>, P8<double>, double*, long long);

}  // namespace smhd
