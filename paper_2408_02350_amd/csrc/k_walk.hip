// S4 in 3D FP64 for velocity grids that one block of the fused kernel cannot
// hold: f-tilde of the interior particles,
//   ft = f_i (1 + dt sum_j c_ij) - dt sum_j c_ij f_j,
//   c_ij = g.w - |P.w| - |Q.w| - |R.w|,  w = v - U_i,
// written to memory and relaxed by k_collide.
//
// One wavefront owns (a patch of 4 interior particles, a slab of 64 lanes x R
// velocities); the slabs are the outer order, so that the waves of an XCD
// read the same slab of neighbouring rows and find them in its L2.  A lane's
// R velocities step along z (R.w is constant along it), the last group of a
// column overlapping the one before where R does not divide nv (its stores
// leave the overlap out).  The wave walks the sorted union of its particles'
// neighbour lists with two rows in flight, and stages the edge records of 16
// entries at a time in LDS, one (entry, particle) per lane.
//
// Against the fused kernel that walks the tiles in one 1024-lane block per CU
// (f-tilde in 128 KB of LDS): no barrier, so no phase of a patch leaves the CU
// idle, fewer rows fetched from beyond the L2 (60 instead of 90-100 GB at
// 48^3 x 20^3) and R free of nv's divisors, for one write and one read of
// f-tilde.  With the relaxation, us: 48^3 x 20^3 17630 -> 16653; 30^3 x 20^3 at
// h = 3.1 dx 10597 -> 8718; 26^3 x 14^3 1193 -> 976, x 22^3 4330 -> 3583, x
// 24^3 4962 -> 4220; 10^3 x 20^3 151 -> 106.  Where one tile holds the grid
// the fused kernel stays ahead (32^3 x 16^3 2223 against 2512 at R = 4, 26^3 x
// 12^3 549 against 631).  The walk at 48^3 x 20^3 (14.1 ms) is bound by FP64
// VALU issue (0.68 of the cycles, at 1.84 GHz under this load); without its row
// loads it takes 11.2 ms, with every row in L2 12.9.
#include "device_common.h"

namespace bgk {

struct WalkArgs {
  int N, NV, nv, cap, Ni, npatch, ucap, groups;  // groups: R-velocity groups of the grid
  double vmax, dt, dvs;
  const double* f;
  double* ft;
  const double* U;
  const double* ops;
  const int32_t* plist;
  const int32_t* ucount;
  const int32_t* uj;
  const uint32_t* ue;
};

constexpr int kWalkChunk = 16;   // union entries whose records are staged at a time
constexpr int kWalkP = 4;        // particles per patch
constexpr int kWalkRec = 12;     // see the staging below

template <int R, int WPE>
__global__ __launch_bounds__(64, WPE) void k_walk(const WalkArgs a) {
  constexpr int TP = kWalkP, CH = kWalkChunk, REC = kWalkRec;
  // record: rows P, Q, R with the z column in velocity steps (the increment of
  // each projection) and, in R's z slot (b has no z component), the increment
  // of g.w; then the three a_k.U
  __shared__ __align__(16) double lrec[CH][TP][REC];
  const int lane = threadIdx.x;
  const int lb = xcd_logical_block(blockIdx.x, gridDim.x);
  const int tile = lb / a.npatch, patch = lb - tile * a.npatch;
  const double* __restrict__ f = a.f;
  const size_t NVs = static_cast<size_t>(a.NV);
  const int zs = a.nv * a.nv;
  const uint32_t zsb = static_cast<uint32_t>(zs) * sizeof(double);
  const int nu = a.ucount[patch];
  const int32_t* __restrict__ ujp = a.uj + static_cast<size_t>(patch) * a.ucap;
  const uint32_t* __restrict__ uep = a.ue + static_cast<size_t>(patch) * a.ucap;
  // staging: lane l forms the record of (entry l / 4 of the chunk, particle l % 4)
  const int st = lane & 3;
  const int sg = patch * TP + st;
  const int si = sg < a.Ni ? a.plist[sg] : -1;
  double sU[3];
#pragma unroll
  for (int m = 0; m < 3; ++m) sU[m] = si >= 0 ? a.U[static_cast<size_t>(m) * a.N + si] : 0.0;
  const double* __restrict__ sops = a.ops + static_cast<size_t>(max(si, 0)) * a.cap * 9;
  // this lane's velocities
  const int L = tile * 64 + lane;
  const bool on = L < a.groups;
  const int col = on ? L % zs : 0, zg = on ? L / zs : 0;
  const int z0 = min(zg * R, a.nv - R);
  const int skip = zg * R - z0;  // velocities that the group before holds
  const uint32_t qoff = static_cast<uint32_t>(z0 * zs + col) * sizeof(double);
  const double v0[3] = {vnode(col % a.nv, a.nv, a.vmax), vnode(col / a.nv, a.nv, a.vmax),
                        static_cast<double>(z0) - 0.5 * (a.nv - 1)};  // (z in steps, exact)

  double acc[TP][R], csum[TP][R];
#pragma unroll
  for (int t = 0; t < TP; ++t)
#pragma unroll
    for (int r = 0; r < R; ++r) acc[t][r] = csum[t][r] = 0.0;

  for (int b0 = 0; b0 < nu; b0 += 64) {
    const int bn = min(64, nu - b0), last = bn - 1;
    // the next 64 union entries, one per lane: row index << 4 | slot mask
    uint32_t pe = 0xFFFFFFFFu, vju = 0;
    if (lane < bn) {
      pe = uep[b0 + lane];
      uint32_t m = 0;
#pragma unroll
      for (int t = 0; t < TP; ++t)
        if (((pe >> (8 * t)) & 0xFFu) != 0xFFu) m |= 1u << t;
      vju = (static_cast<uint32_t>(ujp[b0 + lane]) << 4) | m;
    }
    double ra[R], rb[R];
    auto load_row = [&](int u, double (&buf)[R]) {
      const int j = static_cast<int>(static_cast<uint32_t>(__builtin_amdgcn_readlane(vju, u)) >> 4);
      load_rz<double, R>(f + static_cast<size_t>(j) * NVs, qoff, zsb, buf);
      asm volatile("" ::: "memory");  // (kept where it is issued)
    };
    auto process = [&](int u, const double (&fj)[R]) {
      // one wait for the row, before the branches
#pragma unroll
      for (int r = 0; r < R; ++r) asm volatile("" ::"v"(fj[r]));
      const uint32_t mask = static_cast<uint32_t>(__builtin_amdgcn_readlane(vju, u)) & 15u;
#pragma unroll
      for (int t = 0; t < TP; ++t) {
        if (mask & (1u << t)) {
          typedef double V __attribute__((ext_vector_type(2)));
          const V* rp = reinterpret_cast<const V*>(__builtin_assume_aligned(lrec[u & (CH - 1)][t], 16));
          double rv[REC];
#pragma unroll
          for (int i = 0; i < REC / 2; ++i) {
            const V x = rp[i];
            rv[2 * i] = x[0];
            rv[2 * i + 1] = x[1];
          }
          double p0 = fma(rv[2], v0[2], fma(rv[1], v0[1], fma(rv[0], v0[0], -rv[9])));
          double p1 = fma(rv[5], v0[2], fma(rv[4], v0[1], fma(rv[3], v0[0], -rv[10])));
          const double p2 = fma(rv[7], v0[1], fma(rv[6], v0[0], -rv[11]));
          double gw = ((p0 + p1) + p2) - fabs(p2);
#pragma unroll
          for (int r = 0; r < R; ++r) {
            if (r > 0) {
              p0 = p0 + rv[2];
              p1 = p1 + rv[5];
              gw = gw + rv[8];
            }
            const double c = (gw - fabs(p0)) - fabs(p1);
            csum[t][r] = csum[t][r] + c;
            acc[t][r] = fma(c, fj[r], acc[t][r]);
          }
        }
      }
    };
    load_row(0, ra);
    load_row(min(1, last), rb);
    for (int u = 0; u < bn; u += 2) {
      if ((u & (CH - 1)) == 0) {
        const int w = u + (lane >> 2);
        const uint32_t e =
            (static_cast<uint32_t>(__shfl(static_cast<int>(pe), w, 64)) >> (8 * st)) & 0xFFu;
        __syncthreads();  // (one wave: the chunk before is consumed)
        if (w < bn && e != 0xFFu) {
          const double* o = sops + e * 9;
          double av[9];
#pragma unroll
          for (int k = 0; k < 9; ++k) av[k] = o[k];
          double* rec = lrec[lane >> 2][st];
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            double b = 0.0;
#pragma unroll
            for (int m = 0; m < 3; ++m) b = fma(av[k * 3 + m], sU[m], b);
            rec[9 + k] = b;
            rec[k * 3] = av[k * 3];
            rec[k * 3 + 1] = av[k * 3 + 1];
          }
          const double s0 = av[2] * a.dvs, s1 = av[5] * a.dvs;
          rec[2] = s0;
          rec[5] = s1;
          rec[8] = (s0 + s1) + av[8] * a.dvs;
        }
        __syncthreads();
      }
      process(u, ra);
      load_row(min(u + 2, last), ra);
      if (u + 1 < bn) process(u + 1, rb);
      load_row(min(u + 3, last), rb);
    }
  }

#pragma unroll
  for (int t = 0; t < TP; ++t) {
    const int i = __builtin_amdgcn_readlane(si, t);
    if (i < 0) continue;
    double o[R];
    load_rz<double, R>(f + static_cast<size_t>(i) * NVs, qoff, zsb, o);
#pragma unroll
    for (int r = 0; r < R; ++r) o[r] = fma(o[r], fma(a.dt, csum[t][r], 1.0), -(a.dt * acc[t][r]));
    double* row = a.ft + static_cast<size_t>(i) * NVs;
    if (on && skip == 0) {
      store_rz<double, R>(row, qoff, zsb, o);
    } else if (on) {
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (r >= skip) row[(z0 + r) * zs + col] = o[r];
    }
  }
}

template <int R, int WPE>
static hipError_t launch_walk_r(const Ctx& c, WalkArgs a) {
  a.groups = c.cfg.nv * c.cfg.nv * ((c.cfg.nv + R - 1) / R);
  const int64_t nb = static_cast<int64_t>(c.npatch) * ((a.groups + 63) / 64);
  if (nb > INT32_MAX) return hipErrorInvalidValue;
  hipLaunchKernelGGL((k_walk<R, WPE>), dim3(static_cast<unsigned>(nb)), dim3(64), 0, c.stream, a);
  return hipGetLastError();
}

// (such clouds have patches of kWalkP, and a grid of several tiles has nv >= 14)
bool walk_supported(const Ctx& c) { return c.D == 3 && c.cfg.precision == BGK_FP64; }

// R: of 5 (three waves per SIMD) and 6 to 8 (two), the least waves x (R + 1.6),
// an edge's set-up being worth about 1.6 velocities, with 8% against the
// widths of two waves per SIMD.  us with the relaxation: 20^3 grid R 5 2260, 7
// 2364, 4 2415, 6 2656; 14^3 R 7 976, 5 995; 18^3 R 6 1807, 5 1935; 24^3 R 8
// 4220, 6 4411, 5 4416 (26^3 particles); 30^3 R 5 3712, 6 3847, 8 3868 (20^3).
hipError_t launch_walk(const Ctx& c, const void* f_in, void* ft, const double* U) {
  if (c.npatch == 0) return hipSuccess;
  WalkArgs a{c.N, c.NV, c.cfg.nv, c.cap, c.Ni, c.npatch, c.ucap, 0, c.cfg.vmax, c.cfg.dt,
             2.0 * c.cfg.vmax / (c.cfg.nv - 1), static_cast<const double*>(f_in),
             static_cast<double*>(ft), U, c.d.ops64, c.d.cperm, c.d.ucount, c.d.uj, c.d.ue};
  int best = 5;
  double cost = 0.0;
  for (int R = 5; R <= 8; ++R) {
    const int64_t groups = static_cast<int64_t>(c.cfg.nv) * c.cfg.nv * ((c.cfg.nv + R - 1) / R);
    const double w = (groups + 63) / 64 * (R + 1.6) * (R == 5 ? 1.0 : 1.08);
    if (R == 5 || w < cost) {
      best = R;
      cost = w;
    }
  }
  switch (best) {
    case 5: return launch_walk_r<5, 3>(c, a);
    case 6: return launch_walk_r<6, 2>(c, a);
    case 7: return launch_walk_r<7, 2>(c, a);
    default: return launch_walk_r<8, 2>(c, a);
  }
}

}  // namespace bgk
