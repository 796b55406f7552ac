// One four-edge-class obstacle evaluated by a quad of lanes, lane j <-> edge
// slot j (slots past the obstacle's edges repeat its last edge), equal bit
// for bit to obstacle_sd<MF, 4> on the same obstacle: each lane takes its
// edge against every robot vertex and the obstacle point(s) of its slot
// against every robot edge with the same operations, the minima and maxima
// are then reduced across the quad (the order of a minimum does not matter),
// and the soft-min's sum adds the obstacle axes' terms in slot order after
// the robot axes', as obstacle_sd does.
#pragma once

#include <hip/hip_runtime.h>

#include "psdf_device.hpp"
#include "psdf_winner.hpp"

namespace psdf {

template <int C>
__device__ __forceinline__ float quad_dpp(float x) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), C, 0xf, 0xf, false));
}
__device__ __forceinline__ float quad_min(float x) {
  x = fminf(x, quad_dpp<kDppXor1>(x));
  return fminf(x, quad_dpp<kDppXor2>(x));
}
__device__ __forceinline__ float quad_max(float x) {
  x = fmaxf(x, quad_dpp<kDppXor1>(x));
  return fmaxf(x, quad_dpp<kDppXor2>(x));
}

// What lane j of the quad holds of the obstacle.
struct QuadEdge {
  float tax, tay;   // A_j - p
  float tbx, tby;   // B_j - p (read only when open)
  float ux, uy;     // (B_j - A_j) / (|B_j - A_j| + eps)
  float len;        // |B_j - A_j|
  int mi;           // edge count of the obstacle
  bool closed, bad;
};

// own(lo, hi) gives lane j's obstacle interval on its own axis n'_j
// (own_intervals); it is called by whole quads only, and only where no robot
// axis separates.  Every lane of the quad must be active; all four return
// the sd.
template <int MF, class Own>
__device__ __forceinline__ float quad_eval(const FpConst& F, const QuadEdge& q, const float4* rf,
                                           Own own) {
  const float ca = fmaf(q.tax, q.ux, q.tay * q.uy);
  const float cb = fmaf(q.tay, q.ux, -(q.tax * q.uy));

  // robot vertices against edge j; the robot's interval on n'_j
  float dv2 = __builtin_huge_valf(), rlo = __builtin_huge_valf(), rhi = -__builtin_huge_valf();
#pragma unroll
  for (int l = 0; l < MF; ++l) {
    const float4 r = rf[l];
    const float a = fmaf(r.x, q.ux, fmaf(r.y, q.uy, -ca));
    const float b = fmaf(r.y, q.ux, fmaf(-r.x, q.uy, -cb));
    rlo = fminf(rlo, b);
    rhi = fmaxf(rhi, b);
    dv2 = fminf(dv2, frame_d2(a, b, q.len));
  }
  // obstacle point(s) of slot j against the robot edges
  float ra_lo[MF], ra_hi[MF], de2 = __builtin_huge_valf();
#pragma unroll
  for (int l = 0; l < MF; ++l) { ra_lo[l] = __builtin_huge_valf(); ra_hi[l] = -__builtin_huge_valf(); }
  auto visit = [&](float wx, float wy) {
#pragma unroll
    for (int l = 0; l < MF; ++l) {
      const float4 r = rf[l];
      const float a = fmaf(wx, r.z, fmaf(wy, r.w, -F.cu[l]));
      const float b = fmaf(wx, r.w, fmaf(-wy, r.z, -F.cn[l]));
      ra_lo[l] = fminf(ra_lo[l], b);
      ra_hi[l] = fmaxf(ra_hi[l], b);
      de2 = fminf(de2, frame_d2(a, b, F.len[l]));
    }
  };
  visit(q.tax, q.tay);
  if (!q.closed) visit(q.tbx, q.tby);

  // across the quad
  dv2 = quad_min(dv2);
  de2 = quad_min(de2);
  float dl[MF];
  bool sep = false;
#pragma unroll
  for (int l = 0; l < MF; ++l) {
    ra_lo[l] = quad_min(ra_lo[l]);
    ra_hi[l] = quad_max(ra_hi[l]);
    dl[l] = fminf(ra_hi[l] - F.oa[l], F.ob[l] - ra_lo[l]);
    sep = sep || (dl[l] < -F.eps_sat);
  }
  float dlo = 0.f;   // obstacle axis j
  if (!sep) {        // the same in all four lanes
    float olo, ohi;
    own(olo, ohi);
    dlo = fminf(ohi - rlo, rhi - olo);
    sep = quad_max((dlo < -F.eps_sat) ? 1.f : 0.f) > 0.f;
  }

  float sd = sqrtf(fminf(dv2, de2));
  if (!sep) {
    float mu = __builtin_huge_valf();
#pragma unroll
    for (int l = 0; l < MF; ++l) mu = fminf(mu, fmaxf(dl[l], 0.0f));
    mu = fminf(mu, quad_min(fmaxf(dlo, 0.0f)));
    float depth = mu;
    if (!F.hard) {
      float acc = 0.0f;
#pragma unroll
      for (int l = 0; l < MF; ++l)
        if (l < F.m) acc += expf(-F.eta * (fmaxf(dl[l], 0.0f) - mu));
      const float ej = expf(-F.eta * (fmaxf(dlo, 0.0f) - mu));
      const float e0 = quad_dpp<0x00>(ej), e1 = quad_dpp<0x55>(ej);
      const float e2 = quad_dpp<0xAA>(ej), e3 = quad_dpp<0xFF>(ej);
      if (0 < q.mi) acc += e0;
      if (1 < q.mi) acc += e1;
      if (2 < q.mi) acc += e2;
      if (3 < q.mi) acc += e3;
      depth = mu - logf(acc) / F.eta;
    }
    sd = -depth;
  }
  if (q.bad) sd = __builtin_nanf("");
  return sd;
}

// Lane j's edge of an obstacle with edges [e0, e0 + mi), 1 <= mi <= 4, read
// from the edge arrays, with the constants load_obstacle derives (act false:
// no load, the zero edge).  (ax, ay) and (bx, by) get A_j and B_j.
__device__ __forceinline__ void quad_load(QuadEdge& q, const float* __restrict__ gax,
                                          const float* __restrict__ gay,
                                          const float* __restrict__ gbx,
                                          const float* __restrict__ gby, int e0, int mi,
                                          bool closed, bool act, float eps, float px, float py,
                                          float& ax, float& ay, float& bx, float& by) {
  const int j = threadIdx.x & 3;
  ax = ay = bx = by = 0.f;
  if (act) {
    const int e = e0 + min(j, mi - 1);
    ax = gax[e]; ay = gay[e]; bx = gbx[e]; by = gby[e];
  }
  const float dx = bx - ax, dy = by - ay;
  float iv2, il;
  edge_consts(dx, dy, eps, iv2, il);
  q.ux = dx * il;
  q.uy = dy * il;
  q.len = __builtin_amdgcn_sqrtf(fmaf(dx, dx, dy * dy));
  q.tax = ax - px; q.tay = ay - py;
  q.tbx = bx - px; q.tby = by - py;
  q.mi = mi;
  q.closed = closed;
  q.bad = false;
}

// Lane j's own-axis interval from the quad's edges (own_intervals).
__device__ __forceinline__ void quad_own(const QuadEdge& q, float ax, float ay, float bx, float by,
                                         float& lo, float& hi) {
  lo = __builtin_huge_valf();
  hi = -__builtin_huge_valf();
  auto point = [&](float wx, float wy) {
    const float p = fmaf(wy - ay, q.ux, -((wx - ax) * q.uy));
    lo = fminf(lo, p);
    hi = fmaxf(hi, p);
  };
  point(quad_dpp<0x00>(ax), quad_dpp<0x00>(ay));
  point(quad_dpp<0x55>(ax), quad_dpp<0x55>(ay));
  point(quad_dpp<0xAA>(ax), quad_dpp<0xAA>(ay));
  point(quad_dpp<0xFF>(ax), quad_dpp<0xFF>(ay));
  if (!q.closed) {
    point(quad_dpp<0x00>(bx), quad_dpp<0x00>(by));
    point(quad_dpp<0x55>(bx), quad_dpp<0x55>(by));
    point(quad_dpp<0xAA>(bx), quad_dpp<0xAA>(by));
    point(quad_dpp<0xFF>(bx), quad_dpp<0xFF>(by));
  }
}

}  // namespace psdf
