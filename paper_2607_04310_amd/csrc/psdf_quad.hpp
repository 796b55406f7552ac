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

// ---- an obstacle of at most G = 4, 8 or 16 edges per group of G lanes, the
// footprint's slots in a loop over a table in LDS: the same value again, bit
// for bit, with no footprint size in the code and few registers (which is
// what a chain of dependent loads needs: waves to hide it behind).

// Slot l of the footprint at a stage: the rotated vertex and direction
// (rotated_slot), and the constants of robot edge l.
struct FpSlot {
  float4 r;                     // R v_l, R u_l
  float cu, cn, len, oa, ob;
};

template <int G>
__device__ __forceinline__ float group_min(float x) {
  x = fminf(x, quad_dpp<kDppXor1>(x));
  x = fminf(x, quad_dpp<kDppXor2>(x));
  if (G > 4) x = fminf(x, quad_dpp<kDppHalfMirror>(x));
  if (G > 8) x = fminf(x, quad_dpp<kDppMirror>(x));
  return x;
}
template <int G>
__device__ __forceinline__ float group_max(float x) {
  x = fmaxf(x, quad_dpp<kDppXor1>(x));
  x = fmaxf(x, quad_dpp<kDppXor2>(x));
  if (G > 4) x = fmaxf(x, quad_dpp<kDppHalfMirror>(x));
  if (G > 8) x = fmaxf(x, quad_dpp<kDppMirror>(x));
  return x;
}
template <int G>
__device__ __forceinline__ uint32_t group_min_u32(uint32_t x) {
  x = min(x, dpp_u32<kDppXor1>(x));
  x = min(x, dpp_u32<kDppXor2>(x));
  if (G > 4) x = min(x, dpp_u32<kDppHalfMirror>(x));
  if (G > 8) x = min(x, dpp_u32<kDppMirror>(x));
  return x;
}
// Lane k of the group's value (k a constant after unrolling).
template <int G>
__device__ __forceinline__ float group_lane(float x, int k) {
  if constexpr (G == 4) {
    switch (k) {
      case 0: return quad_dpp<0x00>(x);
      case 1: return quad_dpp<0x55>(x);
      case 2: return quad_dpp<0xAA>(x);
      default: return quad_dpp<0xFF>(x);
    }
  }
  return __shfl(x, ((threadIdx.x & 63) & ~(G - 1)) + k);
}

// sd of an obstacle of mi edges, 1 <= mi <= G, at a stage at (px, py); lane j
// of the group has its edge min(j, mi - 1), A = (ax, ay), B = (bx, by)
// (act; without it the value is meaningless).  dls holds 64 / G x kMaxFp
// floats of the wave.  Every lane of the wave is active.
template <int G>
__device__ __forceinline__ float group_sd(const FpConst& F, const FpSlot* fs, float* dls,
                                          float ax, float ay, float bx, float by, int mi,
                                          bool closed, bool act, float px, float py) {
  const int lane = threadIdx.x & 63, j = lane & (G - 1), m = F.m;
  float* dl = dls + (lane / G) * kMaxFp;
  const float dx = bx - ax, dy = by - ay;
  float iv2, il;
  edge_consts(dx, dy, F.eps, iv2, il);
  const float ux = dx * il, uy = dy * il;
  const float len = __builtin_amdgcn_sqrtf(fmaf(dx, dx, dy * dy));
  const float tax = ax - px, tay = ay - py, tbx = bx - px, tby = by - py;
  const float ca = fmaf(tax, ux, tay * uy);
  const float cb = fmaf(tay, ux, -(tax * uy));
  const bool open = act && !closed;
  const bool any_open = __ballot(open) != 0;

  float dv2 = __builtin_huge_valf(), rlo = __builtin_huge_valf(), rhi = -__builtin_huge_valf();
  float de2 = __builtin_huge_valf(), mu = __builtin_huge_valf();
  bool sep = false;
#pragma unroll 2
  for (int l = 0; l < m; ++l) {
    const FpSlot f = fs[l];
    // robot vertex l against edge j; the robot's interval on n'_j
    const float a = fmaf(f.r.x, ux, fmaf(f.r.y, uy, -ca));
    const float b = fmaf(f.r.y, ux, fmaf(-f.r.x, uy, -cb));
    rlo = fminf(rlo, b);
    rhi = fmaxf(rhi, b);
    dv2 = fminf(dv2, frame_d2(a, b, len));
    // the point(s) of slot j against robot edge l, and the overlap on its
    // normal across the group
    const float a2 = fmaf(tax, f.r.z, fmaf(tay, f.r.w, -f.cu));
    const float b2 = fmaf(tax, f.r.w, fmaf(-tay, f.r.z, -f.cn));
    de2 = fminf(de2, frame_d2(a2, b2, f.len));
    float lo = b2, hi = b2;
    if (any_open) {
      const float a3 = fmaf(tbx, f.r.z, fmaf(tby, f.r.w, -f.cu));
      const float b3 = fmaf(tbx, f.r.w, fmaf(-tby, f.r.z, -f.cn));
      if (open) {
        de2 = fminf(de2, frame_d2(a3, b3, f.len));
        lo = fminf(lo, b3);
        hi = fmaxf(hi, b3);
      }
    }
    lo = group_min<G>(lo);
    hi = group_max<G>(hi);
    const float d = fminf(hi - f.oa, f.ob - lo);
    sep = sep || (d < -F.eps_sat);
    mu = fminf(mu, fmaxf(d, 0.0f));
    if (j == 0) dl[l] = d;
  }
  // squared distances are ordered as their bits
  const float near2 = __uint_as_float(group_min_u32<G>(__float_as_uint(fminf(dv2, de2))));
  float dlo = 0.f;   // obstacle axis j
  if (__ballot(act && !sep)) {
    // the obstacle's interval on its own axis j (own_intervals)
    float lo = __builtin_huge_valf(), hi = -__builtin_huge_valf();
#pragma unroll
    for (int k = 0; k < G; ++k) {
      const float wx = group_lane<G>(ax, k), wy = group_lane<G>(ay, k);
      const float q = fmaf(wy - ay, ux, -((wx - ax) * uy));
      lo = fminf(lo, q);
      hi = fmaxf(hi, q);
    }
    if (any_open) {
#pragma unroll
      for (int k = 0; k < G; ++k) {
        const float wx = group_lane<G>(bx, k), wy = group_lane<G>(by, k);
        const float q = fmaf(wy - ay, ux, -((wx - ax) * uy));
        if (open) {
          lo = fminf(lo, q);
          hi = fmaxf(hi, q);
        }
      }
    }
    dlo = fminf(hi - rlo, rhi - lo);
    sep = sep || group_max<G>((dlo < -F.eps_sat) ? 1.f : 0.f) > 0.f;
  }
  float sd = sqrtf(near2);
  if (__ballot(act && !sep)) {
    mu = fminf(mu, group_min<G>(fmaxf(dlo, 0.0f)));
    float depth = mu;
    if (!F.hard) {
      wave_sync();   // dl is written
      // the robot axes' terms G at a time, a lane each; added in slot order
      float acc = 0.0f;
      for (int l0 = 0; l0 < m; l0 += G) {
        const float t = l0 + j < m ? expf(-F.eta * (fmaxf(dl[l0 + j], 0.0f) - mu)) : 0.f;
#pragma unroll
        for (int k = 0; k < G; ++k) {
          const float e = group_lane<G>(t, k);
          if (l0 + k < m) acc += e;
        }
      }
      const float ej = expf(-F.eta * (fmaxf(dlo, 0.0f) - mu));
#pragma unroll
      for (int k = 0; k < G; ++k) {
        const float e = group_lane<G>(ej, k);
        if (k < mi) acc += e;
      }
      depth = mu - logf(acc) / F.eta;
    }
    if (!sep) sd = -depth;
  }
  wave_sync();   // dl is free again
  return sd;
}

}  // namespace psdf
