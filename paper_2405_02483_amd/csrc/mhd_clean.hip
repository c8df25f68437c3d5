// div B cleaning in Fourier space (Section 3, eq. clean1, eq. clean2) for
// periodic boxes: the potential phi solves the staggered Laplacian
// ddxup(ddxdn(phi)) + ddyup(ddydn(phi)) + ddzup(ddzdn(phi)) = div B, with
// div B = ddxup(B_x) + ddyup(B_y) + ddzup(B_z) at the centres; on a Fourier
// mode the Laplacian is multiplication by -(K_x^2 + K_y^2 + K_z^2), K the
// sixth-order derivative symbol, zero only for the mean mode (whose phi is
// 0).  Then B_a -= ddadn(phi) on the faces, which leaves a discretely
// solenoidal field.
//
// Boxes whose edges factor into small primes take the transforms below
// (with odd factors up to kCleanMixed cells), the others rocFFT's
// real-to-complex and back.
#include <hip/hip_runtime.h>
#include <rocfft/rocfft.h>

#include <algorithm>
#include <cmath>
#include <mutex>

#include "mhd_clean.hpp"
#include "mhd_zmarch.hpp"

namespace smhd {

namespace {

constexpr int kCleanBlock = 256;

// Cell coordinates of box-local index q in 32-bit arithmetic (boxes hold
// fewer than 2^31 cells; 64-bit division is emulated and slow).
__device__ __forceinline__ void clean_coords(unsigned q, unsigned nx, unsigned ny, int& i, int& j, int& k) {
  const unsigned qx = q / nx, qy = qx / ny;
  i = (int)(q - qx * nx);
  j = (int)(qx - qy * ny);
  k = (int)qy;
}

// The stencil kernels march along z: one thread per (x, y) column and
// chunk of kCleanZ planes, the z operand in a register window of six
// planes.  A workgroup covers kCleanTX x kCleanTY columns, so the rows of a y
// stencil are mostly shared within it.  Short chunks: the window's five
// warm-up planes hit in the caches that the neighbouring chunk fills, and a
// march costs a trip to memory a plane.  us per call with chunks of 32, 16, 8
// and 4 planes: float32 64^3 60 / 51 / 47 / 45, 128^3 108 / 93 / 90 / 87,
// 256^3 422 / 413 / 410 / 403; float64 64^3 72 / 55 / 47 / 43, 128^3 147 /
// 122 / 113 / 116, 256^3 788 / 762 / 760 / 757.
constexpr int kCleanZ = 4;
constexpr int kCleanTX = 64, kCleanTY = kCleanBlock / kCleanTX;

__device__ __forceinline__ int wrapz(int k, int n) { return k < 0 ? k + n : (k >= n ? k - n : k); }

// div B at the centres of one box (box-local output index).
template <class T>
__global__ __launch_bounds__(kCleanBlock) void k_clean_div(BoxDev b, const T* __restrict__ bx,
                                                           const T* __restrict__ by,
                                                           const T* __restrict__ bz, T* __restrict__ div, int zc) {
  const int i = (int)(blockIdx.x * kCleanTX + threadIdx.x % kCleanTX);
  const int j = (int)(blockIdx.y * kCleanTY + threadIdx.x / kCleanTX);
  if (i >= b.nx || j >= b.ny) return;
  const unsigned nxy = (unsigned)b.nx * (unsigned)b.ny;
  const unsigned q = (unsigned)j * (unsigned)b.nx + (unsigned)i;
  const int z0 = (int)blockIdx.z * zc, z1 = min(z0 + zc, b.nzt);
  const Geo<T> g(b);
  // window of bz at planes k-2 .. k+3 (the up derivative's samples)
  T w[6];
#pragma unroll
  for (int m = 0; m < 5; ++m) w[m] = bz[g.at(i, j, wrapz(z0 - 2 + m, b.nzt))];
  for (int k = z0; k < z1; ++k) {
    w[5] = bz[g.at(i, j, wrapz(k + 3, b.nzt))];
    div[(long long)k * nxy + q] = op6<1, 1, T>([&](int m) { return bx[g.at(i + m, j, k)]; }, g.hxi) +
                                  op6<1, 1, T>([&](int m) { return by[g.at(i, j + m, k)]; }, g.hyi) +
                                  op6<1, 1, T>([&](int m) { return w[m + 2]; }, g.hzi);
#pragma unroll
    for (int m = 0; m < 5; ++m) w[m] = w[m + 1];
  }
}

// phi^ = -div^ / (K_x^2 + K_y^2 + K_z^2) times `scale` (the 1/N of the
// unnormalised inverse transform); the mean mode's phi is 0.  F holds
// (nx/2 + 1) x ny x nz complex values, x fastest.
template <class T, class C>
__global__ __launch_bounds__(kCleanBlock) void k_clean_solve(C* __restrict__ F, const T* __restrict__ k2x,
                                                             const T* __restrict__ k2y,
                                                             const T* __restrict__ k2z, int nxh, int ny, int nz,
                                                             T scale) {
  const unsigned q = blockIdx.x * kCleanBlock + threadIdx.x;
  if ((long long)q >= (long long)nxh * ny * nz) return;
  int i, j, k;
  clean_coords(q, (unsigned)nxh, (unsigned)ny, i, j, k);
  const T L = k2x[i] + k2y[j] + k2z[k];
  C v = F[q];
  const T s = L > T(0) ? -scale / L : T(0);
  v.x *= s;
  v.y *= s;
  F[q] = v;
}

// B_a -= ddadn(phi) on the faces of one box (phi box-local).
template <class T>
__global__ __launch_bounds__(kCleanBlock) void k_clean_apply(BoxDev b, const T* __restrict__ phi,
                                                             T* __restrict__ bx, T* __restrict__ by,
                                                             T* __restrict__ bz, int zc) {
  const int i = (int)(blockIdx.x * kCleanTX + threadIdx.x % kCleanTX);
  const int j = (int)(blockIdx.y * kCleanTY + threadIdx.x / kCleanTX);
  if (i >= b.nx || j >= b.ny) return;
  const unsigned nxy = (unsigned)b.nx * (unsigned)b.ny;
  const unsigned q = (unsigned)j * (unsigned)b.nx + (unsigned)i;
  const int z0 = (int)blockIdx.z * zc, z1 = min(z0 + zc, b.nzt);
  const Geo<T> g(b);
  auto at = [&](int x, int y, int z) {
    x = x < 0 ? x + b.nx : (x >= b.nx ? x - b.nx : x);
    y = y < 0 ? y + b.ny : (y >= b.ny ? y - b.ny : y);
    return phi[(long long)z * nxy + (long long)y * b.nx + x];
  };
  // window of phi at planes k-3 .. k+2 (the down derivative's samples)
  T w[6];
#pragma unroll
  for (int m = 0; m < 5; ++m) w[m] = at(i, j, wrapz(z0 - 3 + m, b.nzt));
  for (int k = z0; k < z1; ++k) {
    w[5] = at(i, j, wrapz(k + 2, b.nzt));
    const long long o = b.off + (long long)k * nxy + q;
    bx[o] -= op6<1, 0, T>([&](int m) { return at(i + m, j, k); }, g.hxi);
    by[o] -= op6<1, 0, T>([&](int m) { return at(i, j + m, k); }, g.hyi);
    bz[o] -= op6<1, 0, T>([&](int m) { return w[m + 3]; }, g.hzi);
#pragma unroll
    for (int m = 0; m < 5; ++m) w[m] = w[m + 1];
  }
}

// K(theta_m)^2 of the sixth-order staggered derivative (eq. deriv) for
// modes m = 0..count-1 of a periodic axis of n cells and spacing h.
void symbol_sq(int n, int count, double h, std::vector<double>& out) {
  const double d[3] = {75.0 / 64.0, -25.0 / 384.0, 3.0 / 640.0};
  for (int m = 0; m < count; ++m) {
    const double th = 2.0 * M_PI * m / n;
    double K = 0.0;
    for (int p = 1; p <= 3; ++p) K += d[p - 1] * std::sin((2 * p - 1) * th / 2.0);
    K *= 2.0 / h;
    out.push_back(K * K);
  }
}

// ---------------------------------------------------------------------------
// Fourier transforms in LDS: div B -> [x] -> [y] -> [z, solve, z inverse] ->
// [y inverse] -> [x inverse] -> phi.  The z transform, the division by the
// symbol and the inverse share one load and one store of the spectrum.  A
// workgroup transforms `cols` lines at once (x: pairs of real rows as one
// complex line each; y, z: neighbouring kx, up to a cache line of them and
// more where they are short) in
// place, in Stockham passes of radix 8, 4, 2, 3, 5, 7, 11, 13 whose
// elements wait in registers across a barrier.  The kernels come in three
// classes of radices: with 11 and 13 in the same kernel as the powers of two
// its registers (244) would leave 2 waves a SIMD.  us per call, these
// transforms against rocFFT with kernels of their own for div B and the
// solve (and 32-plane stencils): float32 24^3 33 / 55, 64^3 36 / 65,
// 100x100x200 112 / 129, 128^3 83 / 113, 256^3 389 / 504, 1000x40x50 100 / 112,
// 500x20x20 41 / 53; float64 64^3 39 / 108, 96^3 79 / 157, 128^3 114 / 182, 256^3
// 750 / 912.  Behind it: 16x256x256 float32 95 / 87 and 12x400x400 float64
// 336 / 305 (a cache line of kx holds 9 and 7), 1000x12x12 float32 45 / 42.
// The first call of a context: 0.3-1 ms against 1.2-1.8 s in a new process
// (3.5 ms after that).
//
// Boxes with odd factors take them up to kCleanMixed cells: every box measured
// below it but the three above is faster than before; above, with everything
// else equal, float32 144^3 127 / 137 and 150^3 144 / 156 but 160^3 168 / 147,
// 18x512x512 281 / 237, 200^3 255 / 254; float64 150^3 203 / 193, 160^3 217 / 202,
// 216x220x208 562 / 589.
constexpr int kFftThreads = 256, kFftPasses = 12;
constexpr long long kCleanMixed = 2000000;
// bytes of the lines of a workgroup, and elements a thread holds
template <int CL> constexpr size_t kFftLine = CL < 2 ? 32 * 1024 : 16 * 1024;

struct FftAxis {
  int n, np, cols;           // length, passes, lines per workgroup (a power of two)
  int tw;                    // first twiddle in the table: exp(-2 pi i m / n), m < n
  int cl;                    // class of its radices: 0 a power of two, 1 up to 7, 2 up to 13
  unsigned char radix[kFftPasses];
};

template <class T> struct Cx { T x, y; };
template <class T> __device__ __forceinline__ Cx<T> operator+(Cx<T> a, Cx<T> b) { return {a.x + b.x, a.y + b.y}; }
template <class T> __device__ __forceinline__ Cx<T> operator-(Cx<T> a, Cx<T> b) { return {a.x - b.x, a.y - b.y}; }
template <class T> __device__ __forceinline__ Cx<T> mul(Cx<T> a, Cx<T> w) {
  return {a.x * w.x - a.y * w.y, a.x * w.y + a.y * w.x};
}
// -i a (forward) or +i a (inverse)
template <bool INV, class T> __device__ __forceinline__ Cx<T> rot(Cx<T> a) {
  return INV ? Cx<T>{-a.y, a.x} : Cx<T>{a.y, -a.x};
}

// cos and sin of 2 pi m / R, m < R, of the odd radices, by their power series
// (constants of the kernels: read from the twiddle table in LDS and with
// integer divisions below, float32 96x192x108 took 119 us against 93).
template <int R> struct Root { double c[R], s[R]; };
constexpr double kPi = 3.14159265358979323846;
constexpr double series_cos(double x) {   // |x| <= pi / 2
  double t = 1.0, v = 1.0;
  for (int k = 1; k <= 14; ++k) {
    t *= -x * x / ((2 * k - 1) * (2 * k));
    v += t;
  }
  return v;
}
constexpr double series_sin(double x) {
  double t = x, v = x;
  for (int k = 1; k <= 14; ++k) {
    t *= -x * x / ((2 * k) * (2 * k + 1));
    v += t;
  }
  return v;
}
template <int R> constexpr Root<R> roots() {
  Root<R> r{};
  r.c[0] = 1.0;
  r.s[0] = 0.0;
  for (int m = 1; m <= R / 2; ++m) {
    // (4 m < R: an angle up to pi / 2; above, from its supplement)
    const bool low = 4 * m < R;
    const double x = low ? 2.0 * kPi * m / R : kPi * (R - 2 * m) / R;
    r.c[m] = low ? series_cos(x) : -series_cos(x);
    r.s[m] = series_sin(x);
    r.c[R - m] = r.c[m];
    r.s[R - m] = -r.s[m];
  }
  return r;
}

template <int R, bool INV, class T> __device__ __forceinline__ void dft(Cx<T> (&v)[R]) {
  if constexpr (R == 2) {
    const Cx<T> a = v[0], b = v[1];
    v[0] = a + b;
    v[1] = a - b;
  } else if constexpr (R == 4) {
    const Cx<T> a = v[0] + v[2], b = v[0] - v[2], c = v[1] + v[3], d = rot<INV>(v[1] - v[3]);
    v[0] = a + c;
    v[1] = b + d;
    v[2] = a - c;
    v[3] = b - d;
  } else if constexpr (R == 8) {
    Cx<T> e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
    dft<4, INV, T>(e);
    dft<4, INV, T>(o);
    const T h = T(0.70710678118654752440);
    const Cx<T> r1 = rot<INV>(o[1]), r3 = rot<INV>(o[3]);
    o[1] = {h * (o[1].x + r1.x), h * (o[1].y + r1.y)};
    o[2] = rot<INV>(o[2]);
    o[3] = {h * (r3.x - o[3].x), h * (r3.y - o[3].y)};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      v[q] = e[q] + o[q];
      v[q + 4] = e[q] - o[q];
    }
  } else {
    // odd prime: sums and differences of the pairs (r, R - r)
    constexpr int H = (R - 1) / 2;
    Cx<T> a[H], b[H], out[R];
    out[0] = v[0];
#pragma unroll
    for (int r = 0; r < H; ++r) {
      a[r] = v[r + 1] + v[R - 1 - r];
      b[r] = v[r + 1] - v[R - 1 - r];
      out[0] = out[0] + a[r];
    }
    constexpr Root<R> W = roots<R>();
#pragma unroll
    for (int q = 1; q <= H; ++q) {
      Cx<T> s = v[0], d = {T(0), T(0)};
#pragma unroll
      for (int r = 1; r <= H; ++r) {
        const T wc = T(W.c[r * q % R]), ws = T(W.s[r * q % R]);
        s = {s.x + wc * a[r - 1].x, s.y + wc * a[r - 1].y};
        d = {d.x + ws * b[r - 1].x, d.y + ws * b[r - 1].y};
      }
      const Cx<T> t = rot<INV>(d);
      out[q] = s + t;
      out[R - q] = s - t;
    }
#pragma unroll
    for (int q = 0; q < R; ++q) v[q] = out[q];
  }
}

// t / n for t < 2^16, n < 2^16 (inv_of(n), the same in every thread, once).
__device__ __forceinline__ unsigned inv_of(int n) { return 0xffffffffu / (unsigned)n + 1u; }
__device__ __forceinline__ int div_by(int t, unsigned inv) { return (int)__umulhi((unsigned)t, inv); }

// One Stockham pass over `cols` lines, element (i, c) at i * cp + c, in
// place: every thread holds its butterflies in registers across the barrier.
template <int R, bool INV, int CL, class T>
__device__ __forceinline__ void fft_pass(Cx<T>* __restrict__ l, const Cx<T>* __restrict__ tw, int n, int ns, int lc,
                                         int cp) {
  constexpr int E = (int)(kFftLine<CL> / sizeof(Cx<T>)) / kFftThreads;   // elements per thread
  constexpr int U = (E + R - 1) / R;
  const int nb = n / R, step = nb / ns, cnt = nb << lc;
  const unsigned ins = CL == 0 ? 0u : inv_of(ns);
  Cx<T> v[U][R];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int t = (int)threadIdx.x + u * kFftThreads;
    if (t < cnt) {
      const int c = t & ((1 << lc) - 1), j = t >> lc;
#pragma unroll
      for (int r = 0; r < R; ++r) v[u][r] = l[(j + r * nb) * cp + c];
    }
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int t = (int)threadIdx.x + u * kFftThreads;
    if (t >= cnt) continue;
    const int c = t & ((1 << lc) - 1), j = t >> lc;
    const int q = CL == 0 ? j >> __builtin_ctz((unsigned)ns) : (ns == 1 ? j : div_by(j, ins)), k = j - q * ns;
    if (ns > 1) {
#pragma unroll
      for (int r = 1; r < R; ++r) {
        Cx<T> w = tw[r * k * step];
        if (INV) w.y = -w.y;
        v[u][r] = mul(v[u][r], w);
      }
    }
    dft<R, INV, T>(v[u]);
    const int o = q * ns * R + k;
#pragma unroll
    for (int r = 0; r < R; ++r) l[(o + r * ns) * cp + c] = v[u][r];
  }
  __syncthreads();
}

// The whole transform of the lines in l.  All threads call; the lines are
// visible on entry and on return.
template <bool INV, int CL, class T>
__device__ __forceinline__ void fft_lines(Cx<T>* l, const Cx<T>* tw, const FftAxis& A, int lc, int cp) {
  int ns = 1;
  for (int p = 0; p < A.np; ++p) {
    const int R = A.radix[p];
    if constexpr (CL == 0) {
      if (R == 8) fft_pass<8, INV, CL>(l, tw, A.n, ns, lc, cp);
      else if (R == 4) fft_pass<4, INV, CL>(l, tw, A.n, ns, lc, cp);
      else fft_pass<2, INV, CL>(l, tw, A.n, ns, lc, cp);
    } else if (CL == 2 && R >= 11) {
      if constexpr (CL == 2) {
        if (R == 11) fft_pass<11, INV, CL>(l, tw, A.n, ns, lc, cp);
        else fft_pass<13, INV, CL>(l, tw, A.n, ns, lc, cp);
      }
    } else switch (R) {
      case 8: fft_pass<8, INV, CL>(l, tw, A.n, ns, lc, cp); break;
      case 4: fft_pass<4, INV, CL>(l, tw, A.n, ns, lc, cp); break;
      case 2: fft_pass<2, INV, CL>(l, tw, A.n, ns, lc, cp); break;
      case 3: fft_pass<3, INV, CL>(l, tw, A.n, ns, lc, cp); break;
      case 5: fft_pass<5, INV, CL>(l, tw, A.n, ns, lc, cp); break;
      default: fft_pass<7, INV, CL>(l, tw, A.n, ns, lc, cp); break;
    }
    ns *= R;
  }
}

// div B at the centre (x, row), the rows of all planes numbered through.
template <class T>
__device__ __forceinline__ T div_at(const BoxDev& b, const T* bx, const T* by, const T* bz, int x, int row) {
  const int z = row / b.ny, y = row - z * b.ny;
  auto wrap = [](int i, int m) { return i < 0 ? i + m : (i >= m ? i - m : i); };
  auto at = [&](const T* f, int i, int j, int k) { return f[b.off + ((long long)k * b.ny + j) * b.nx + i]; };
  return op6<1, 1, T>([&](int m) { return at(bx, wrap(x + m, b.nx), y, z); }, T(b.hinv[0])) +
         op6<1, 1, T>([&](int m) { return at(by, x, wrap(y + m, b.ny), z); }, T(b.hinv[1])) +
         op6<1, 1, T>([&](int m) { return at(bz, x, y, wrap(z + m, b.nzt)); }, T(b.hinv[2]));
}

// x transforms.  Forward: two rows of div B per line in, half spectra of both
// out (pitch kx apart).  Inverse: half spectra in, rows of phi out.
// DIV: div B is formed as the rows are loaded (small boxes: a launch less;
// on large ones its stencils stall the few workgroups that fit).
template <class T, bool INV, int CL, bool DIV>
__global__ __launch_bounds__(kFftThreads) void k_fft_x(FftAxis A, BoxDev b, const T* __restrict__ bx,
                                                      const T* __restrict__ by, const T* __restrict__ bz, int rows, const Cx<T>* __restrict__ tws,
                                                      T* __restrict__ real, Cx<T>* __restrict__ spec, int pitch) {
  extern __shared__ __align__(16) unsigned char lds_[];
  const int n = A.n, cp = A.cols + 1, lc = __builtin_ctz((unsigned)A.cols);
  Cx<T>* tw = reinterpret_cast<Cx<T>*>(lds_);
  Cx<T>* l = tw + n;
  const int row0 = (int)blockIdx.x * A.cols * 2, nh = n / 2 + 1;
  const unsigned in = CL == 0 ? 0u : inv_of(n), inh = inv_of(nh);
  auto line = [&](int t) { return CL == 0 ? t >> __builtin_ctz((unsigned)n) : div_by(t, in); };
  for (int t = (int)threadIdx.x; t < n; t += kFftThreads) tw[t] = tws[A.tw + t];
  if (!INV) {
    for (int t = (int)threadIdx.x; t < (n << lc); t += kFftThreads) {
      const int p = line(t), x = t - p * n, r = row0 + 2 * p;
      if constexpr (DIV) {
        l[x * cp + p] = {r < rows ? div_at(b, bx, by, bz, x, r) : T(0),
                         r + 1 < rows ? div_at(b, bx, by, bz, x, r + 1) : T(0)};
      } else {
        const T* __restrict__ s = real + (long long)r * n + x;
        l[x * cp + p] = {r < rows ? s[0] : T(0), r + 1 < rows ? s[n] : T(0)};
      }
    }
  } else {
    for (int t = (int)threadIdx.x; t < (nh << lc); t += kFftThreads) {
      const int p = div_by(t, inh), k = t - p * nh, r = row0 + 2 * p;
      const Cx<T> zero = {T(0), T(0)};
      Cx<T> u = r < rows ? spec[(long long)r * pitch + k] : zero;
      Cx<T> v = r + 1 < rows ? spec[(long long)(r + 1) * pitch + k] : zero;
      // the modes that are their own mirror are real
      if (k == 0 || 2 * k == n) u.y = v.y = T(0);
      l[k * cp + p] = {u.x - v.y, u.y + v.x};
      if (k > 0 && 2 * k < n) l[(n - k) * cp + p] = {u.x + v.y, v.x - u.y};
    }
  }
  __syncthreads();
  fft_lines<INV, CL>(l, tw, A, lc, cp);
  if (!INV) {
    for (int t = (int)threadIdx.x; t < (nh << lc); t += kFftThreads) {
      const int p = div_by(t, inh), k = t - p * nh, r = row0 + 2 * p;
      const Cx<T> a = l[k * cp + p], c = l[(k == 0 ? 0 : n - k) * cp + p];
      if (r < rows) spec[(long long)r * pitch + k] = {T(0.5) * (a.x + c.x), T(0.5) * (a.y - c.y)};
      if (r + 1 < rows) spec[(long long)(r + 1) * pitch + k] = {T(0.5) * (a.y + c.y), T(0.5) * (c.x - a.x)};
    }
  } else {
    for (int t = (int)threadIdx.x; t < (n << lc); t += kFftThreads) {
      const int p = line(t), x = t - p * n, r = row0 + 2 * p;
      const Cx<T> a = l[x * cp + p];
      if (r < rows) real[(long long)r * n + x] = a.x;
      if (r + 1 < rows) real[(long long)(r + 1) * n + x] = a.y;
    }
  }
}

// y transforms (in place), and the z transform with the solve and its
// inverse.  blockIdx.x: tile of kx, blockIdx.y: z (or y); line element i
// lies i * stride from the tile's first.
// SOLVE: phi^ = -div^ / (K_x^2 + K_y^2 + K_z^2) times `scale` (the 1/N of
// the unnormalised inverse); the mean mode's phi is 0.
template <class T, bool INV, bool SOLVE, int CL>
__global__ __launch_bounds__(kFftThreads) void k_fft_yz(FftAxis A, const Cx<T>* __restrict__ tws,
                                                       Cx<T>* __restrict__ spec, int nxh, long long outer,
                                                       long long stride, const T* __restrict__ k2x,
                                                       const T* __restrict__ k2y, const T* __restrict__ k2z,
                                                       T scale) {
  extern __shared__ __align__(16) unsigned char lds_[];
  const int n = A.n, cp = A.cols, lc = __builtin_ctz((unsigned)A.cols);
  Cx<T>* tw = reinterpret_cast<Cx<T>*>(lds_);
  Cx<T>* l = tw + n;
  for (int t = (int)threadIdx.x; t < n; t += kFftThreads) tw[t] = tws[A.tw + t];
  const int kx0 = (int)blockIdx.x << lc;
  Cx<T>* base = spec + blockIdx.y * outer + kx0;
  for (int t = (int)threadIdx.x; t < (n << lc); t += kFftThreads) {
    const int c = t & (A.cols - 1), i = t >> lc;
    l[t] = kx0 + c < nxh ? base[i * stride + c] : Cx<T>{T(0), T(0)};
  }
  __syncthreads();
  fft_lines<INV, CL>(l, tw, A, lc, cp);
  if constexpr (SOLVE) {
    const T ky = k2y[blockIdx.y];
    for (int t = (int)threadIdx.x; t < (n << lc); t += kFftThreads) {
      const int c = t & (A.cols - 1), i = t >> lc;
      if (kx0 + c >= nxh) continue;
      const T L = k2x[kx0 + c] + ky + k2z[i];
      const T s = L > T(0) ? -scale / L : T(0);
      l[t] = {l[t].x * s, l[t].y * s};
    }
    __syncthreads();
    fft_lines<true, CL>(l, tw, A, lc, cp);
  }
  for (int t = (int)threadIdx.x; t < (n << lc); t += kFftThreads) {
    const int c = t & (A.cols - 1), i = t >> lc;
    if (kx0 + c < nxh) base[i * stride + c] = l[t];
  }
}

// Whether a workgroup holds `cols` lines of the axis (fft_pass).
bool fft_holds(const FftAxis& A, int cols, size_t csize) {
  return (size_t)A.n * cols * csize <= (A.cl < 2 ? kFftLine<0> : kFftLine<2>);
}

// The passes of an axis of n cells, or false: a prime above 13, or longer
// than the LDS buffers hold four lines of.
bool fft_axis(int n, size_t csize, FftAxis& A) {
  A.n = n;
  A.np = 0;
  int m = n;
  for (int R : {8, 4, 2, 3, 5, 7, 11, 13})
    while (m % R == 0 && A.np < kFftPasses) {
      A.radix[A.np++] = (unsigned char)R;
      m /= R;
    }
  if (m != 1) return false;
  const int top = A.radix[A.np - 1];   // (the largest prime comes last)
  A.cl = (n & (n - 1)) == 0 ? 0 : (top <= 7 ? 1 : 2);
  A.cols = 128 / (int)csize;   // a cache line of kx
  while (A.cols > 1 && !fft_holds(A, A.cols, csize)) A.cols /= 2;
  return A.cols >= 4;
}

// Lines a workgroup by the box (fft_axis: what the LDS buffers hold, a cache
// line of kx at most).  Fewer while the workgroups do not fill the device,
// down to an element a thread: us per call before and after, float32
// 500x20x20 91 / 41, 512x32x32 83 / 45, 250x80x100 121 / 110, 64^3 45 / 36 (x);
// 60x60x512 109 / 104, 20x500x20 63 / 54 (y, z; 4 lines at least).  The powers
// of two gain up to 768 workgroups (1024x64x64 135 / 129), odd factors lose
// beyond 256 (400x60x80 127 / 134).  More for short lines while enough
// workgroups remain: a workgroup of 16 lines of 16 holds one element a
// thread, 512x512x16 153 / 129, float64 239 / 196.
void fft_cols(FftAxis (&ax)[3], int nx, int ny, int nz, size_t csize) {
  const long long rows = (long long)ny * nz;
  const int nxh = nx / 2 + 1;
  while (ax[0].cols > 1 && ax[0].n * ax[0].cols >= 512 && rows < 2LL * ax[0].cols * (ax[0].cl == 0 ? 768 : 256)) ax[0].cols /= 2;
  for (int a = 1; a < 3; ++a) {
    FftAxis& A = ax[a];
    auto groups = [&](int cols) { return (long long)((nxh + cols - 1) / cols) * (a == 1 ? nz : ny); };
    while (A.cols > 4 && A.n * A.cols >= 512 && groups(A.cols) <= 256) A.cols /= 2;
    while (A.n * A.cols < 1024 && nxh > A.cols && groups(2 * A.cols) >= 1024 && fft_holds(A, 2 * A.cols, csize))
      A.cols *= 2;
  }
}

std::once_flag g_rocfft_once;
rocfft_status g_rocfft_setup = rocfft_status_success;

}  // namespace

struct CleanState {
  struct Plan {
    int nx, ny, nz;
    bool own = false;           // the transforms of this file
    FftAxis ax[3];
    rocfft_plan fwd = nullptr, inv = nullptr;
  };
  std::vector<Plan> plans;
  int dtype = -1;
  void* real = nullptr;   // div B, then phi: the largest box's cells
  void* cplx = nullptr;   // its transform
  void* work = nullptr;   // rocFFT's work buffer, the largest the plans ask
  void* ktab = nullptr;   // K^2 per axis and box
  void* twid = nullptr;   // twiddles of this file's transforms
  size_t work_bytes = 0;
  std::vector<long long> koff;   // per box: offset of its x, y, z tables in ktab
  rocfft_execution_info info = nullptr;
};

void clean_free(CleanState* s) {
  if (!s) return;
  for (auto& p : s->plans) {
    if (p.fwd) (void)rocfft_plan_destroy(p.fwd);
    if (p.inv) (void)rocfft_plan_destroy(p.inv);
  }
  if (s->info) (void)rocfft_execution_info_destroy(s->info);
  (void)hipFree(s->real);
  (void)hipFree(s->cplx);
  (void)hipFree(s->work);
  (void)hipFree(s->ktab);
  (void)hipFree(s->twid);
  delete s;
}

// Cells up to which div B is formed in the x transform.
static constexpr long long kCleanFuse = 1000000;

// Row pitch of a box's half spectrum: rows start on a cache line.
template <class T> static int spec_pitch(const BoxDev& b) {
  const int line = 128 / (2 * (int)sizeof(T));
  return (b.nx / 2 + 1 + line - 1) / line * line;
}

// div B of the box (in real, or up to kCleanFuse cells formed on the way)
// through the transforms and the solve, to phi.
template <class T>
static void own_transforms(const BoxDev& b, P8<T> f, const FftAxis (&ax)[3], const Cx<T>* tw, Cx<T>* spec, T* real,
                           const T* k2, hipStream_t stream) {
  const int nxh = b.nx / 2 + 1, pitch = spec_pitch<T>(b);
  const int rows = b.ny * b.nzt;
  const dim3 gx((rows + 2 * ax[0].cols - 1) / (2 * ax[0].cols)), blk(kFftThreads);
  const dim3 gy((nxh + ax[1].cols - 1) / ax[1].cols, b.nzt), gz((nxh + ax[2].cols - 1) / ax[2].cols, b.ny);
  auto lds = [](const FftAxis& A, int pad) { return (size_t)A.n * (A.cols + pad + 1) * sizeof(Cx<T>); };
  const T *kx = k2, *ky = kx + nxh, *kz = ky + b.ny;
  const long long plane = (long long)pitch * b.ny;
  // the kernel of an axis's class
  auto pick = [](int cl, auto* k0, auto* k1, auto* k2) { return cl == 0 ? k0 : (cl == 1 ? k1 : k2); };
  auto x = [&](auto inv, auto div) {
    constexpr bool INV = decltype(inv)::value, DIV = decltype(div)::value;
    auto* kern = pick(ax[0].cl, k_fft_x<T, INV, 0, DIV>, k_fft_x<T, INV, 1, DIV>, k_fft_x<T, INV, 2, DIV>);
    hipLaunchKernelGGL(kern, gx, blk, lds(ax[0], 1), stream, ax[0], b, (const T*)f.p[5], (const T*)f.p[6],
                       (const T*)f.p[7], rows, tw, real, spec, pitch);
  };
  auto y = [&](auto inv) {
    constexpr bool INV = decltype(inv)::value;
    auto* kern = pick(ax[1].cl, k_fft_yz<T, INV, false, 0>, k_fft_yz<T, INV, false, 1>, k_fft_yz<T, INV, false, 2>);
    hipLaunchKernelGGL(kern, gy, blk, lds(ax[1], 0), stream, ax[1], tw, spec, nxh, plane, (long long)pitch, kx, ky,
                       kz, T(0));
  };
  if (b.ncell <= kCleanFuse) x(std::false_type{}, std::true_type{});
  else x(std::false_type{}, std::false_type{});
  y(std::false_type{});
  auto* solve = pick(ax[2].cl, k_fft_yz<T, false, true, 0>, k_fft_yz<T, false, true, 1>, k_fft_yz<T, false, true, 2>);
  hipLaunchKernelGGL(solve, gz, blk, lds(ax[2], 0), stream, ax[2], tw, spec, nxh, (long long)pitch, plane, kx, ky, kz,
                     T(1.0 / (double)b.ncell));
  y(std::true_type{});
  x(std::true_type{}, std::false_type{});
}

template <class T>
int clean_boxes(CleanState** sp, const std::vector<BoxDev>& boxes, P8<T> f, hipStream_t stream,
                std::string& err) {
  using C = typename std::conditional<sizeof(T) == 4, float2, double2>::type;
  const rocfft_precision prec = sizeof(T) == 4 ? rocfft_precision_single : rocfft_precision_double;
  if (!*sp) {
    CleanState* s = new CleanState;
    s->dtype = sizeof(T);
    // one plan pair per distinct box shape, buffers for the largest box
    long long ncell = 0, ncplx = 0;
    std::vector<double> k2;
    std::vector<C> tw;
    for (const BoxDev& b : boxes) {
      ncell = std::max(ncell, b.ncell);
      ncplx = std::max(ncplx, (long long)spec_pitch<T>(b) * b.ny * b.nzt);
      s->koff.push_back((long long)k2.size());
      symbol_sq(b.nx, b.nx / 2 + 1, b.dx, k2);
      symbol_sq(b.ny, b.ny, b.dy, k2);
      symbol_sq(b.nzt, b.nzt, b.dz, k2);
      bool have = false;
      for (const auto& p : s->plans) have |= p.nx == b.nx && p.ny == b.ny && p.nz == b.nzt;
      if (have) continue;
      CleanState::Plan p;
      p.nx = b.nx;
      p.ny = b.ny;
      p.nz = b.nzt;
      const int edge[3] = {b.nx, b.ny, b.nzt};
      p.own = true;
      for (int a = 0; a < 3; ++a) p.own = p.own && fft_axis(edge[a], sizeof(C), p.ax[a]);
      p.own = p.own && (b.ncell <= kCleanMixed || p.ax[0].cl + p.ax[1].cl + p.ax[2].cl == 0);
      if (p.own) {
        fft_cols(p.ax, b.nx, b.ny, b.nzt, sizeof(C));
        for (FftAxis& A : p.ax) {
          A.tw = (int)tw.size();
          for (int m = 0; m < A.n; ++m) {
            const double th = 2.0 * M_PI * m / A.n;
            tw.push_back(C{T(std::cos(th)), T(-std::sin(th))});
          }
        }
        s->plans.push_back(p);
        continue;
      }
      std::call_once(g_rocfft_once, [] { g_rocfft_setup = rocfft_setup(); });
      if (g_rocfft_setup != rocfft_status_success) {
        clean_free(s);
        err = "rocfft_setup failed";
        return 1;
      }
      if (!s->info && rocfft_execution_info_create(&s->info) != rocfft_status_success) {
        clean_free(s);
        err = "rocfft execution info";
        return 1;
      }
      const size_t len[3] = {(size_t)b.nx, (size_t)b.ny, (size_t)b.nzt};   // fastest first
      if (rocfft_plan_create(&p.fwd, rocfft_placement_notinplace, rocfft_transform_type_real_forward, prec, 3,
                             len, 1, nullptr) != rocfft_status_success ||
          rocfft_plan_create(&p.inv, rocfft_placement_notinplace, rocfft_transform_type_real_inverse, prec, 3,
                             len, 1, nullptr) != rocfft_status_success) {
        s->plans.push_back(p);
        clean_free(s);
        err = "rocfft_plan_create failed";
        return 1;
      }
      size_t w1 = 0, w2 = 0;
      (void)rocfft_plan_get_work_buffer_size(p.fwd, &w1);
      (void)rocfft_plan_get_work_buffer_size(p.inv, &w2);
      s->work_bytes = std::max(s->work_bytes, std::max(w1, w2));
      s->plans.push_back(p);
    }
    std::vector<T> kt(k2.begin(), k2.end());
    if (hipMalloc(&s->real, sizeof(T) * ncell) != hipSuccess ||
        hipMalloc(&s->cplx, sizeof(C) * ncplx) != hipSuccess ||
        (s->work_bytes && hipMalloc(&s->work, s->work_bytes) != hipSuccess) ||
        hipMalloc(&s->ktab, sizeof(T) * kt.size()) != hipSuccess ||
        hipMemcpy(s->ktab, kt.data(), sizeof(T) * kt.size(), hipMemcpyHostToDevice) != hipSuccess ||
        (!tw.empty() &&
         (hipMalloc(&s->twid, sizeof(C) * tw.size()) != hipSuccess ||
          hipMemcpy(s->twid, tw.data(), sizeof(C) * tw.size(), hipMemcpyHostToDevice) != hipSuccess))) {
      clean_free(s);
      err = "allocation failed";
      return 2;
    }
    *sp = s;
  }
  CleanState* s = *sp;
  if (s->info && (rocfft_execution_info_set_stream(s->info, stream) != rocfft_status_success ||
      (s->work && rocfft_execution_info_set_work_buffer(s->info, s->work, s->work_bytes) != rocfft_status_success))) {
    err = "rocfft execution info";
    return 1;
  }
  T* real = static_cast<T*>(s->real);
  C* cplx = static_cast<C*>(s->cplx);
  const T* kt = static_cast<const T*>(s->ktab);
  for (size_t bi = 0; bi < boxes.size(); ++bi) {
    const BoxDev& b = boxes[bi];
    const CleanState::Plan* p = nullptr;
    for (const auto& q : s->plans)
      if (q.nx == b.nx && q.ny == b.ny && q.nz == b.nzt) p = &q;
    const int nxh = b.nx / 2 + 1;
    const int zc = std::max(kCleanZ, (b.nzt + 65534) / 65535);   // the grid's limit
    const dim3 gc((unsigned)((b.nx + kCleanTX - 1) / kCleanTX), (unsigned)((b.ny + kCleanTY - 1) / kCleanTY),
                  (unsigned)((b.nzt + zc - 1) / zc));
    const long long nc = (long long)nxh * b.ny * b.nzt;
    const dim3 gk((unsigned)((nc + kCleanBlock - 1) / kCleanBlock));
    if (!p->own || b.ncell > kCleanFuse)
      hipLaunchKernelGGL(k_clean_div<T>, gc, dim3(kCleanBlock), 0, stream, b, f.p[5], f.p[6], f.p[7], real,
                         zc);
    if (p->own) {
      own_transforms<T>(b, f, p->ax, reinterpret_cast<const Cx<T>*>(s->twid), reinterpret_cast<Cx<T>*>(cplx), real,
                        kt + s->koff[bi], stream);
      hipLaunchKernelGGL(k_clean_apply<T>, gc, dim3(kCleanBlock), 0, stream, b, (const T*)real, f.p[5], f.p[6],
                         f.p[7], zc);
      continue;
    }
    void* in1[1] = {real};
    void* out1[1] = {cplx};
    if (rocfft_execute(p->fwd, in1, out1, s->info) != rocfft_status_success) {
      err = "rocfft forward transform failed";
      return 1;
    }
    const T* kx = kt + s->koff[bi];
    hipLaunchKernelGGL((k_clean_solve<T, C>), gk, dim3(kCleanBlock), 0, stream, cplx, kx, kx + nxh,
                       kx + nxh + b.ny, nxh, b.ny, b.nzt, T(1.0 / (double)b.ncell));
    void* in2[1] = {cplx};
    void* out2[1] = {real};
    if (rocfft_execute(p->inv, in2, out2, s->info) != rocfft_status_success) {
      err = "rocfft inverse transform failed";
      return 1;
    }
    hipLaunchKernelGGL(k_clean_apply<T>, gc, dim3(kCleanBlock), 0, stream, b, (const T*)real, f.p[5], f.p[6],
                       f.p[7], zc);
  }
  return 0;
}

template int clean_boxes<float>(CleanState**, const std::vector<BoxDev>&, P8<float>, hipStream_t, std::string&);
template int clean_boxes<double>(CleanState**, const std::vector<BoxDev>&, P8<double>, hipStream_t,
                                 std::string&);

}  // namespace smhd
