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
// R would round differently).  FP64: 2 to 4 in 2D and 2 or 4 to 7 in 3D, the last
// group of a line overlapping where R does not divide nv, at the least
// tiles * (R + 2): an edge costs about as much set-up as two velocities (2D
// nv = 24: 3 223 us, 4 271, 2 278; 3D nv = 12: 6 1.17 ms, 4 1.41; nv = 18: 6
// 3.96, 5 4.78).  R = 7 leaves 2 waves per SIMD for 3 and is weighed 1.1 (nv =
// 20: 5 5.36 ms, 7 5.57; nv = 14, two groups of 7 a line: 2.10).  P particles
// per patch: 2 in 2D (FP64 222 us, 1 236, 3 252, 4 334), 1 in 3D, where the
// second particle's registers cost more waves than its shared rows save loads
// (FP64 nv = 16: 3.23 -> 2.78 ms; FP32 nv = 20 22.7 -> 22.3, P = 3 and 4 25.3).
// An entry's order in the sum over a particle's neighbours does not depend on
// P (ascending).  Rw for the per-particle
// wall kernel (4 when 4 divides nv, else 2: at 5 its register footprint
// halves its waves), and the 64-lane
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
  p.P = cfg.dim == 3 ? 1 : 2;
  auto tiles = [&](int R) { return (nvel / cfg.nv * ((cfg.nv + R - 1) / R) + 63) / 64; };
  if (cfg.precision == BGK_FP64) {
    auto cost = [&](int R) { return tiles(R) * (R + 2) * (R == 7 ? 11 : 10); };
    p.R = 2;
    for (int R = cfg.dim + 1; R <= (cfg.dim == 3 ? 7 : 4) && R <= cfg.nv; ++R)
      if (cost(R) < cost(p.R)) p.R = R;
  } else {
    p.R = (cfg.dim == 3 && cfg.nv % 5 == 0) ? 5 : p.Rw;
  }
  p.tiles = static_cast<int>(tiles(p.R));
  p.tiles_w = static_cast<int>((nvel / p.Rw + 63) / 64);
  return p;
}

}  // namespace bgk

#endif  // BGK_ADJOINT_PLAN_H
