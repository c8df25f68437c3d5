// Transpose of the right-hand side's Jacobian, (dF/df)^T w at a state f, in
// hand-fused passes (mhd_adjoint.hip).  The forward intermediates that the
// transposes need are recomputed from the state; the cotangents of the
// right-hand side's outputs are never stored per flux but formed where they
// are used, as stencils of w.
#pragma once

#include "mhd_kernels.hpp"

namespace smhd {

struct VjpLaunch {
  const BoxDev* boxes;    // device
  const Blk* tab;         // device, blocks over every cell
  int nblk;
  hipStream_t stream;
  int nbox, nplanes;      // boxes; z planes of all boxes (BoxDev::poff)
  int wall;               // some box has closed walls
  double* pm;             // 2 * nplanes values: plane means (T_EDIFFAV)
  const void* ztab;       // z-coefficient tables of wall boxes, compute type
  const Blk* gtab;        // blocks over the ghost planes of wall boxes
  int nghost_blk;
};

// Workspace arrays (of the packed field size) that vjp_rhs needs with the
// terms and constant coefficients of ph (6 at least, for vjp_fill).
template <class T> int vjp_arrays(const Phys<T>& ph);

// g[v] (+)= (dF/df_v)^T w at the state s (acc: added, else overwritten).  s,
// w and g are packed field arrays, none overlapping another; base holds
// vjp_arrays(ph) arrays `stride` elements apart.  dt: the step's (the
// div B diffusion's coefficient; 0 leaves that term out).  nu2, c_smag: the
// coefficients before rounding to T (the lengths multiply them first).
template <class T>
void vjp_rhs(const VjpLaunch& L, const Phys<T>& ph, double nu2, double c_smag, double c_divb, CP8<T> s, CP8<T> w,
             P8<T> g, bool acc, T* base, long long stride, double dt);

// y[v] = a * y[v] + b * x[v] for the 8 fields (a == 0: y is not read).  With
// mask, zero where the right-hand side itself is zeroed on a wall box (ghost
// planes; p_z on the wall faces).
template <class T> void vjp_axpby8(const VjpLaunch& L, P8<T> y, CP8<T> x, double a, double b, bool mask);

// Closed walls (Section 10): the transpose of the ghost fill at the filled
// state s, in place: g holds the cotangent of the filled state on entry and
// that of the state before the fill on exit (zero in the ghost planes and on
// the two wall faces of p_z, which the fill overwrites).  tmp: 6 arrays of
// the packed field size (only their ghost cells are used).
template <class T> void vjp_fill(const VjpLaunch& L, CP8<T> s, P8<T> g, T* tmp, long long stride);

}  // namespace smhd
