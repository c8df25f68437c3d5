// Building blocks of the cell-parallel kernels (one thread per cell, operands
// read through the caches): a cell with its neighbours' offsets, the staggered
// operators on operands given by offset, their transposes, and the maximum
// over three cells.
#pragma once

#include "mhd_kernels.hpp"

namespace smhd {

constexpr int X = 0, Y = 1, Z = 2;

// The factor of a z derivative at output plane k of a wall-bounded axis: the
// Jacobian of an up (centre) or down (face) output, end copy built in (1/dz
// on a uniform axis).
template <class T>
__device__ __forceinline__ T zjac(const T* zt, const BoxDev& b, int form, int k) {
  return zt[b.joff + (long long)k * ZJ_COUNT + (form ? ZJ_C : ZJ_F)];
}

// Coefficient of input plane p in output plane k of a z operator on a
// wall-bounded axis, before the 1/h of a derivative: fam 0, 1 from the box's
// table (reduced orders at the ends, the end output no stencil reaches
// copying its neighbour's); fam 2 the second-order pair, whose end output
// copies its neighbour's in the same way.
template <class T>
__device__ __forceinline__ T zw_coef(const T* zt, const BoxDev& b, int fam, int form, int k, int p) {
  const int N = b.nzt;
  if (fam == 2) {
    const int c = form ? (k + 1 < N ? k + 1 : N - 1) : (k > 0 ? k : 1);
    return p == c ? T(1) : (p == c - 1 ? T(-1) : T(0));
  }
  const int type = fam == 0 ? (form ? ZT_IUP : ZT_IDN) : (form ? ZT_DUP : ZT_DDN);
  return zt[b.zoff + ((long long)type * N + k) * 7 + (p - k) + 3];
}

// Which of (lo, mid, hi) is the first maximal one: 0, 1 or 2.
template <class T> __device__ __forceinline__ int first_max(T lo, T mid, T hi) {
  int s = 0;
  T v = lo;
  if (mid > v) { v = mid; s = 1; }
  if (hi > v) s = 2;
  return s;
}

// One cell with its neighbours' byte offsets (periodic wrap applied; planes
// past a wall take the cell itself and are never used).  Offsets are 32-bit
// within the box, so that a load is a scalar base plus one register; a box
// of 2^32 bytes or more would need a workspace beyond the device's memory.
// W: some box has walls.
template <class T, bool W> struct Cell {
  const BoxDev& b;
  const T* zt;
  unsigned o, sz;
  int k;
  unsigned d[3][7];
  __device__ __forceinline__ Cell(const BoxDev& b_, unsigned q, const T* zt_) : b(b_), zt(zt_) {
    const unsigned nx = (unsigned)b.nx, ny = (unsigned)b.ny;
    const unsigned qx = q / nx, qy = qx / ny;
    const int i = (int)(q - qx * nx), j = (int)(qx - qy * ny);
    k = (int)qy;
    o = q * (unsigned)sizeof(T);
    sz = nx * ny * (unsigned)sizeof(T);
#pragma unroll
    for (int m = -3; m <= 3; ++m) {
      const int x = i + m, y = j + m, z = k + m, N = b.nzt;
      const int dx = x < 0 ? m + b.nx : (x >= b.nx ? m - b.nx : m);
      const int dy = y < 0 ? m + b.ny : (y >= b.ny ? m - b.ny : m);
      int dz = z < 0 ? m + N : (z >= N ? m - N : m);
      if (W && b.wall && (z < 0 || z >= N)) dz = 0;
      d[X][m + 3] = (unsigned)dx * (unsigned)sizeof(T);
      d[Y][m + 3] = (unsigned)dy * nx * (unsigned)sizeof(T);
      d[Z][m + 3] = (unsigned)dz * sz;
    }
  }
  __device__ __forceinline__ T ld(const T* a, unsigned off = 0u) const {
    return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(a) + (o + off));
  }
  __device__ __forceinline__ void st(T* a, T v) const {
    *reinterpret_cast<T*>(reinterpret_cast<char*>(a) + o) = v;
  }
  __device__ __forceinline__ bool walled() const { return W && b.wall; }
  // a z neighbour that exists
  __device__ __forceinline__ bool has(int m) const { return !walled() || (k + m >= 0 && k + m < b.nzt); }
  template <int AX> __device__ __forceinline__ bool hasax(int m) const { return AX != Z || has(m); }
  __device__ __forceinline__ T plane(int e) const { return zt[b.joff + (long long)k * ZJ_COUNT + e]; }
  __device__ __forceinline__ unsigned zoffs(int p) const { return (unsigned)(p - k) * sz; }

  // S_AX of f, f(offset) the operand at a byte offset from the cell.  FAM 0
  // interpolation, 1 derivative, 2 second-order derivative; FORM 0 dn, 1 up.
  template <int AX, int FAM, int FORM, class F> __device__ __forceinline__ T op(const F& f) const {
    T h = T(b.hinv[AX]);
    if constexpr (W && AX == Z) {
      if (b.wall) {
        if (k < 3 || k > b.nzt - 4) {
          T acc = T(0);
          const int p0 = k - 3 > 0 ? k - 3 : 0, p1 = k + 3 < b.nzt - 1 ? k + 3 : b.nzt - 1;
#pragma unroll 1
          for (int p = p0; p <= p1; ++p) acc += zw_coef(zt, b, FAM, FORM, k, p) * f(zoffs(p));
          return FAM ? acc * (b.stretched ? zjac(zt, b, FORM, k) : h) : acc;
        }
        if (FAM && b.stretched) h = zjac(zt, b, FORM, k);
      }
    }
    auto at = [&](int m) { return f(d[AX][m + 3]); };
    if constexpr (FAM == 2) return FORM ? (at(1) - at(0)) * h : (at(0) - at(-1)) * h;
    else return op6<FAM, FORM, T>(at, h);
  }
  // Its transpose at this cell, applied to the outputs' cotangent f.
  template <int AX, int FAM, int FORM, class F> __device__ __forceinline__ T opT(const F& f) const {
    const T h = T(b.hinv[AX]);
    if constexpr (W && AX == Z) {
      if (b.wall) {
        if (k < 6 || k >= b.nzt - 6) {
          T acc = T(0);
          const int k0 = k - 3 > 0 ? k - 3 : 0, k1 = k + 3 < b.nzt - 1 ? k + 3 : b.nzt - 1;
#pragma unroll 1
          for (int q = k0; q <= k1; ++q) {
            T c = zw_coef(zt, b, FAM, FORM, q, k);
            if (FAM && b.stretched) c *= zjac(zt, b, FORM, q);
            acc += c * f(zoffs(q));
          }
          return FAM && !b.stretched ? acc * h : acc;
        }
        if (FAM && b.stretched) {
          auto at = [&](int m) { return f(d[AX][m + 3]) * zjac(zt, b, FORM, k + m); };
          if constexpr (FAM == 2) return FORM ? at(-1) - at(0) : at(0) - at(1);
          else return -op6<1, 1 - FORM, T>(at, T(1));
        }
      }
    }
    auto at = [&](int m) { return f(d[AX][m + 3]); };
    if constexpr (FAM == 2) return FORM ? (at(-1) - at(0)) * h : (at(0) - at(1)) * h;
    else {
      const T v = op6<FAM, 1 - FORM, T>(at, h);
      return FAM ? -v : v;
    }
  }
#define CELL_OP(name, FAM, FORM)                                                                          \
  template <int AX> __device__ __forceinline__ T name(const T* a) const {                                \
    return op<AX, FAM, FORM>([&](unsigned f) { return ld(a, f); });                                      \
  }                                                                                                      \
  template <int AX> __device__ __forceinline__ T name##T(const T* a) const {                             \
    return opT<AX, FAM, FORM>([&](unsigned f) { return ld(a, f); });                                     \
  }
  CELL_OP(dn, 0, 0)
  CELL_OP(up, 0, 1)
  CELL_OP(ddn, 1, 0)
  CELL_OP(dup, 1, 1)
  CELL_OP(d2n, 2, 0)
  CELL_OP(d2u, 2, 1)
#undef CELL_OP
  // interpolation (dn or up, forward or transposed) along A of that along B
  template <int A, int FA, int B, int FB> __device__ __forceinline__ T ii(const T* a) const {
    return op<A, 0, FA>([&](unsigned f) { return op<B, 0, FB>([&](unsigned g) { return ld(a, f + g); }); });
  }
  template <int A, int FA, int B, int FB> __device__ __forceinline__ T iiT(const T* a) const {
    return opT<A, 0, FA>([&](unsigned f) { return opT<B, 0, FB>([&](unsigned g) { return ld(a, f + g); }); });
  }
  // value at offset m along AX, or -inf past a wall (never a maximum)
  template <int AX> __device__ __forceinline__ T orninf(const T* a, int m) const {
    return hasax<AX>(m) ? ld(a, d[AX][m + 3]) : T(-INFINITY);
  }
  template <int AX> __device__ __forceinline__ T max3(const T* a) const {
    const T lo = orninf<AX>(a, -1), mid = ld(a), hi = orninf<AX>(a, 1);
    const int s = first_max(lo, mid, hi);
    return s == 0 ? lo : (s == 1 ? mid : hi);
  }
  // transpose of the maximum of a over three cells: the cell is the hi
  // neighbour of the one below, the middle of its own, the lo of the one above
  template <int AX> __device__ __forceinline__ T max3T(const T* a, const T* yb) const {
    const T v2 = orninf<AX>(a, -2), v1 = orninf<AX>(a, -1), v0 = ld(a), p1 = orninf<AX>(a, 1),
            p2 = orninf<AX>(a, 2);
    const T w1 = ld(yb, d[AX][2]), w0 = ld(yb), wp = ld(yb, d[AX][4]);
    T sum = T(0);
    if (hasax<AX>(-1) && first_max(v2, v1, v0) == 2) sum += w1;
    if (first_max(v1, v0, p1) == 1) sum += w0;
    if (hasax<AX>(1) && first_max(v0, p1, p2) == 0) sum += wp;
    return sum;
  }
  // second difference (0 on the end planes of a wall axis), at offset m
  template <int AX> __device__ __forceinline__ T second(const T* a, int m = 0) const {
    if (AX == Z && walled() && (k + m <= 0 || k + m >= b.nzt - 1)) return T(0);
    return ld(a, d[AX][m + 4]) - T(2) * ld(a, d[AX][m + 3]) + ld(a, d[AX][m + 2]);
  }
};

}  // namespace smhd
