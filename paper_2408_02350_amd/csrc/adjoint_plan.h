// Launch plan of the reverse transport (host and device code of the
// reverse step include this; the forward kernels do not).
#ifndef BGK_ADJOINT_PLAN_H
#define BGK_ADJOINT_PLAN_H

#include <hip/hip_runtime.h>

#include <cstdint>

#include "bgk.h"

namespace bgk {

struct Ctx;

// A forward step's state that the reverse step reads (f-tilde's interior
// rows, f^{n+1}, and the moments of n+1), when the caller kept it from the
// forward pass instead of having the reverse step recompute it.
struct AdjState {
  const void* ft;
  const void* f1;
  const double* rho1;
  const double* U1;
  const double* T1;
};
hipError_t launch_adjoint_step_kept(const Ctx& c, const void* f_n, const double* U_n,
                                    const AdjState& s, const void* lam_f1, const double* lam_U1,
                                    const double* lam_rho1, const double* lam_T1, void* lam_f,
                                    double* lam_U, double* dJ_dlid);

// R velocities per lane for the interior patches, stepping along z in 3D
// and x in 2D.  FP32 storage: 4 when 4 divides nv, else 2, and in 3D 5 when 5
// divides nv (the increments of a line start at its multiples of R, so another
// R would round differently).  FP64: any R up to D + 2, the last group of a
// line overlapping where R does not divide nv, at the least tiles * (R + 2):
// an edge costs about as much set-up as two velocities (nv = 14, 3D: R = 5
// 2.30 ms, 3 2.41, 4 2.68, 2 2.85; nv = 24, 2D: 3 223 us, 4 271, 2 278); above
// D + 2 the registers leave one wave per SIMD (3D R = 7 2.79 ms).  P = 4 or 3
// particles per patch, at half the row loads, are slower for the same reason
// (2.7 - 3.5 ms), P = 1 in 2D too (280 us).  Rw for the per-particle
// wall kernel (4 when 4 divides nv, else 2: at 5 its register footprint
// halves its waves), interior patches of P = 2 particles, and the 64-lane
// tiles of R (Rw) velocities the grid needs: one wavefront per (patch or
// wall particle, tile), each tile holding its part of lam_U per particle.
// Blocks of several wavefronts sharing one derivation of the edge records
// were slower in both precisions (the waves of a block then wait on the
// derivation together).
struct AdjPlan {
  int R, Rw, P, tiles, tiles_w;
};
inline AdjPlan adj_plan(const bgk_config& cfg) {
  int64_t nvel = 1;
  for (int a = 0; a < cfg.dim; ++a) nvel *= cfg.nv;
  AdjPlan p{};
  p.Rw = (cfg.nv % 4 == 0) ? 4 : 2;
  p.P = 2;
  auto tiles = [&](int R) { return (nvel / cfg.nv * ((cfg.nv + R - 1) / R) + 63) / 64; };
  if (cfg.precision == BGK_FP64) {
    p.R = 2;
    for (int R = 3; R <= cfg.dim + 2 && R <= cfg.nv; ++R)
      if (tiles(R) * (R + 2) < tiles(p.R) * (p.R + 2)) p.R = R;
  } else {
    p.R = (cfg.dim == 3 && cfg.nv % 5 == 0) ? 5 : p.Rw;
  }
  p.tiles = static_cast<int>(tiles(p.R));
  p.tiles_w = static_cast<int>((nvel / p.Rw + 63) / 64);
  return p;
}

}  // namespace bgk

#endif  // BGK_ADJOINT_PLAN_H
