// Culled evaluation of a batch: the same outputs as evaluating every
// (stage, obstacle) pair, bit for bit, from a bound per pair and the exact
// evaluation of the few obstacles that the bound leaves.
//
// Every obstacle i gets its bounding box, slightly enlarged (cull_box).  For
// a stage at position p with footprint radius rmax about p, and D the
// distance from p to the box,
//     sd_i >= D (1 - rel) - rmax - gamma =: LB_i      whenever LB_i > tau
// for a regular obstacle (a strictly convex closed polygon or one edge, all
// edges long against eps): two convex sets at distance r have an axis with a
// gap of at least kappa r (FpConst), so beyond tau = eps_sat / kappa + ...
// the axis test separates them, and sd is then their distance.  rel and the
// terms of tau cover the rounding of the float evaluation, whose error grows
// with the distance (measured 3e-7 of it), also where kappa is small.
// Any other obstacle (invalid, open chain, not convex, a degenerate edge,
// coordinates beyond 1e15) is irregular: it is always evaluated.
//
// Two launches:
//  * cull_list_kernel, one work-group per segment (kSegObst obstacles) of an
//    instance: boxes, and the list of the segment's obstacles that some stage
//    may need.  With B the bounding box of the instance's stage positions,
//    every stage's phi is at most
//        H = max(min_i (largest distance from B to A_0 of obstacle i) + rmin,
//                tau, log(axes) / eta)
//    (rmin the smallest |v_l|: separated sets are no further apart than a
//    vertex of each, and an obstacle that is not separated has
//    sd <= log(axes) / eta), so an obstacle whose bound from B exceeds H is
//    beyond phi and tau at every stage.
//  * cull_stage_kernel, one wave per stage: the listed obstacle with the
//    smallest D (the seed) is evaluated exactly; its sd, or tau if that
//    is larger, is a bar T >= phi, and every listed obstacle with LB <= T is
//    evaluated exactly.  The minimum key over these is the stage's key: every
//    other obstacle has sd >= LB > T >= phi.  The wave then ends the stage
//    (write_stage).
// What it measured (graph replay per call, one card, full evaluation before):
// 64 instances x 50 stages x 16384 rectangles 557 -> 47 us (list 17 us for
// 67 MB of edges, stage 23 us), 512 uneven instances (23 800 stages, 2.7 M
// edges) 581 -> 208 us (list 18, stage 177 us).
// Lists have a fixed place per segment and are rewritten by every call:
// no counter to reset, nothing kept between calls, no capacity to exceed.
#pragma once

#include <hip/hip_runtime.h>

#include "psdf_batch.hpp"
#include "psdf_quad.hpp"

namespace psdf {

constexpr int kCullThreads = 256;
constexpr int kCullPer = 4;                              // obstacles per thread
constexpr int kSegObst = kCullThreads * kCullPer;        // obstacles per segment
constexpr int kCullPad = 64;                             // list entries read past the last one
constexpr float kCullGamma = 1e-3f;                      // metres
constexpr float kCullMax = 1e15f;                        // coordinates beyond this: irregular

// One segment of an instance's obstacles: [o0, o0 + no), list slots from
// slot0, list length in cnt[its index].
struct CullSeg {
  int inst, o0, no, slot0;
};

// A stage: its row, instance, first list slot and first segment of the
// instance, segments, obstacles, first offset and first edge.
struct CullStage {
  int row, inst, slot0, seg0, nseg, M, obst_off, edge_off;
};

struct CullArgs {
  const FpConst* fps;
  const BatchInst* insts;
  const CullSeg* segs;
  const CullStage* stages;   // this launch's
  const float* poses;
  const float* ax;
  const float* ay;
  const float* bx;
  const float* by;
  const int* off;
  float4* box;    // per list slot: lo.x (NaN: irregular), lo.y, hi.x, hi.y
  int4* meta;     // per list slot: obstacle, first edge (global), edge count, closed | bad << 1
  int* cnt;       // per segment: list length
  float* d;
  int* edge;
  int* obst;
  float* grad;
  uint64_t* keys;
};

// Four consecutive floats at any float address: global loads of several
// dwords need dword alignment only.
struct __attribute__((packed, aligned(4))) Float4u {
  float v[4];
};

// Running facts of an obstacle, edge by edge.
struct CullAcc {
  float lox, loy, hix, hiy;
  float bad;              // NaN once a coordinate is not finite
  float big;              // largest |coordinate| (finite ones)
  bool longe;             // every edge long against eps
  bool left, right;       // every turn strictly left / right
  bool closed;            // B_j == A_{j+1} bitwise
  int flips;              // sign changes of the edges' direction around the boundary
};

__device__ __forceinline__ void cull_point(CullAcc& c, float x, float y) {
  c.lox = fminf(c.lox, x); c.hix = fmaxf(c.hix, x);
  c.loy = fminf(c.loy, y); c.hiy = fmaxf(c.hiy, y);
  c.bad = fmaf(x, 0.f, c.bad);
  c.bad = fmaf(y, 0.f, c.bad);
}
// direction in (-90, 90] degrees
__device__ __forceinline__ bool cull_half(float ex, float ey) {
  return ex > 0.f || (ex == 0.f && ey > 0.f);
}
// the turn from edge (px, py) to edge (ex, ey): strictly left (right) by a
// margin above the rounding of the product
__device__ __forceinline__ void cull_turn(CullAcc& c, float px, float py, float ex, float ey) {
  const float cr = fmaf(px, ey, -(py * ex));
  const float tol = 1e-6f * (fabsf(px) + fabsf(py)) * (fabsf(ex) + fabsf(ey));
  c.left = c.left && cr > tol;
  c.right = c.right && cr < -tol;
  c.flips += cull_half(px, py) != cull_half(ex, ey) ? 1 : 0;
}
__device__ __forceinline__ bool same_bits(float a, float b) {
  return __float_as_uint(a) == __float_as_uint(b);
}

// Box, flags (closed | bad << 1) and regularity of the obstacle with edges
// [e0, e0 + mi), 1 <= mi <= MI and in range; the first edge (mi != 4) or all
// four (mi == 4) are in v (ax, ay, bx, by).
template <int MI>
__device__ __forceinline__ bool cull_obstacle(const float (&v)[4][4], const float* __restrict__ gax,
                                              const float* __restrict__ gay,
                                              const float* __restrict__ gbx,
                                              const float* __restrict__ gby, int e0, int mi,
                                              float minl2, float rel, float4& box,
                                              int& flags) {
  CullAcc c;
  c.lox = c.loy = __builtin_huge_valf();
  c.hix = c.hiy = -__builtin_huge_valf();
  c.bad = 0.f;
  c.longe = c.left = c.right = c.closed = true;
  c.flips = 0;
  if (mi == 4) {
    float ex[4], ey[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      cull_point(c, v[0][j], v[1][j]);
      ex[j] = v[2][j] - v[0][j];
      ey[j] = v[3][j] - v[1][j];
      c.longe = c.longe && fmaf(ex[j], ex[j], ey[j] * ey[j]) >= minl2;
      c.closed = c.closed && same_bits(v[2][j], v[0][(j + 1) & 3]) &&
                 same_bits(v[3][j], v[1][(j + 1) & 3]);
    }
    if (!c.closed) {
#pragma unroll
      for (int j = 0; j < 4; ++j) cull_point(c, v[2][j], v[3][j]);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) cull_turn(c, ex[j], ey[j], ex[(j + 1) & 3], ey[(j + 1) & 3]);
  } else {
    const float ax0 = v[0][0], ay0 = v[1][0];
    float bx = v[2][0], by = v[3][0];
    float ex = bx - ax0, ey = by - ay0;
    const float ex0 = ex, ey0 = ey;
    cull_point(c, ax0, ay0);
    cull_point(c, bx, by);
    c.longe = fmaf(ex, ex, ey * ey) >= minl2;
    for (int j = 1; j < mi; ++j) {
      const float a0 = gax[e0 + j], a1 = gay[e0 + j], b0 = gbx[e0 + j], b1 = gby[e0 + j];
      c.closed = c.closed && same_bits(bx, a0) && same_bits(by, a1);
      cull_point(c, a0, a1);
      cull_point(c, b0, b1);
      const float fx = b0 - a0, fy = b1 - a1;
      c.longe = c.longe && fmaf(fx, fx, fy * fy) >= minl2;
      cull_turn(c, ex, ey, fx, fy);
      ex = fx; ey = fy; bx = b0; by = b1;
    }
    c.closed = c.closed && mi >= 3 && same_bits(bx, ax0) && same_bits(by, ay0);
    cull_turn(c, ex, ey, ex0, ey0);
  }
  const bool bad = c.bad != c.bad;
  flags = (c.closed ? 1 : 0) | (bad ? 2 : 0);
  // a strictly convex polygon turns one way and its direction changes half
  // twice in one round (a star turns one way too, in more rounds)
  const bool convex = mi == 1 || (c.closed && (c.left || c.right) && c.flips <= 2);
  const float big = fmaxf(fmaxf(fabsf(c.lox), fabsf(c.loy)), fmaxf(fabsf(c.hix), fabsf(c.hiy)));
  const bool regular = !bad && convex && c.longe && big < kCullMax;
  // enlarged by its own size (rounding of the evaluation) and by the
  // rounding of the enlargement itself
  const float e = fmaf(rel, (c.hix - c.lox) + (c.hiy - c.loy), 2.5e-7f * big);
  box = regular ? make_float4(c.lox - e, c.loy - e, c.hix + e, c.hiy + e)
                : make_float4(__builtin_nanf(""), 0.f, 0.f, 0.f);
  return regular;
}

// Bound: the read of every edge once.  Each thread holds kCullPer obstacles
// whose loads are all in flight together.
template <int MI>
__global__ __launch_bounds__(kCullThreads) void cull_list_kernel(CullArgs A) {
  __shared__ float red[4][kCullThreads / 64];
  __shared__ float s_h[kCullThreads / 64];
  __shared__ int s_n[kCullThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  typedef const __attribute__((address_space(4))) CullSeg SegC;
  const CullSeg& S = *(const CullSeg*)((SegC*)A.segs + blockIdx.x);
  const BatchInst in = A.insts[S.inst];
  const FpConst& F = fp_const(A.fps, S.inst);
  const int Eend = in.edge_off + in.E;
  const int* off = A.off + in.obst_off + S.o0;

  int e0[kCullPer], mi[kCullPer];
#pragma unroll
  for (int q = 0; q < kCullPer; ++q) {
    const int k = tid + kCullThreads * q;
    e0[q] = mi[q] = 0;
    if (k < S.no) {
      e0[q] = off[k];
      mi[q] = off[k + 1] - e0[q];
      e0[q] += in.edge_off;
    }
  }
  // box of the instance's stage positions
  float plx = __builtin_huge_valf(), ply = plx, phx = -plx, phy = -plx, pbig = 0.f;
  for (int t = tid; t < in.N; t += kCullThreads) {
    const float* p = A.poses + 3 * (in.pose_off + t);
    const float x = p[0], y = p[1];
    if (!(isfinite(x) && isfinite(y))) continue;   // its stage needs no list
    plx = fminf(plx, x); phx = fmaxf(phx, x);
    ply = fminf(ply, y); phy = fmaxf(phy, y);
  }
  // the edges: all four of a four-edge obstacle, else the first
  float v[kCullPer][4][4];
  bool ok[kCullPer];
#pragma unroll
  for (int q = 0; q < kCullPer; ++q) {
    // an edge count or range that the evaluation calls invalid
    ok[q] = mi[q] >= 1 && mi[q] <= MI && e0[q] >= in.edge_off && e0[q] <= Eend - mi[q];
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int j = 0; j < 4; ++j) v[q][k][j] = 0.f;
    if (ok[q]) {
      const float* src[4] = {A.ax + e0[q], A.ay + e0[q], A.bx + e0[q], A.by + e0[q]};
      if (mi[q] == 4) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const Float4u u = *reinterpret_cast<const Float4u*>(src[k]);
#pragma unroll
          for (int j = 0; j < 4; ++j) v[q][k][j] = u.v[j];
        }
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) v[q][k][0] = *src[k];
      }
    }
  }
  {
    const float a = fw_min_f32(plx), b = fw_min_f32(ply), c = fw_min_f32(-phx), d = fw_min_f32(-phy);
    if (lane == 0) { red[0][w] = a; red[1][w] = b; red[2][w] = c; red[3][w] = d; }
  }
  __syncthreads();
  plx = ply = phx = phy = __builtin_huge_valf();
#pragma unroll
  for (int i = 0; i < kCullThreads / 64; ++i) {
    plx = fminf(plx, red[0][i]); ply = fminf(ply, red[1][i]);
    phx = fminf(phx, red[2][i]); phy = fminf(phy, red[3][i]);
  }
  phx = -phx; phy = -phy;
  pbig = fmaxf(fmaxf(fabsf(plx), fabsf(ply)), fmaxf(fabsf(phx), fabsf(phy)));
  const bool none = !(plx <= phx);            // no finite position: no stage needs the list
  const bool all = !(pbig < kCullMax);        // a position beyond the bound's range

  const float minl = 4e6f * F.eps;
  const float minl2 = fmaxf(minl * minl, 1e-24f);
  float4 box[kCullPer];
  int flags[kCullPer];
  float ub = __builtin_huge_valf();           // least largest distance of B to a regular A_0
#pragma unroll
  for (int q = 0; q < kCullPer; ++q) {
    box[q] = make_float4(__builtin_nanf(""), 0.f, 0.f, 0.f);
    flags[q] = 2;
    if (ok[q] && cull_obstacle<MI>(v[q], A.ax, A.ay, A.bx, A.by, e0[q], mi[q], minl2,
                                   F.cull_rel, box[q], flags[q])) {
      const float fx = fmaxf(fabsf(v[q][0][0] - plx), fabsf(v[q][0][0] - phx));
      const float fy = fmaxf(fabsf(v[q][1][0] - ply), fabsf(v[q][1][0] - phy));
      ub = fminf(ub, fmaf(fx, fx, fy * fy));
    }
  }
  ub = fw_min_f32(ub);
  if (lane == 0) s_h[w] = ub;
  __syncthreads();
  ub = s_h[0];
#pragma unroll
  for (int i = 1; i < kCullThreads / 64; ++i) ub = fminf(ub, s_h[i]);
  const float H = fmaxf(fmaf(sqrtf(ub), 1.0f + 1e-5f, F.rmin), F.sd_floor);
  const float bar = (H + F.rmax + kCullGamma) * (1.0f + 2.0f * F.cull_rel);
  const float bar2 = bar * bar;

  // the list, in obstacle order within each wave
  int n = 0;
  bool take[kCullPer];
  int at[kCullPer];
#pragma unroll
  for (int q = 0; q < kCullPer; ++q) {
    const float4 b = box[q];
    const float gx = fmaxf(fmaxf(b.x - phx, plx - b.z), 0.f);
    const float gy = fmaxf(fmaxf(b.y - phy, ply - b.w), 0.f);
    const bool far = b.x == b.x && fmaf(gx, gx, gy * gy) > bar2 && !all;
    take[q] = mi[q] != 0 && !none && !far;
    const uint64_t m = __ballot(take[q]);
    at[q] = n + (int)__popcll(m & ((1ull << lane) - 1ull));
    n += (int)__popcll(m);
  }
  if (lane == 0) s_n[w] = n;
  __syncthreads();
  int base = S.slot0, total = 0;
#pragma unroll
  for (int i = 0; i < kCullThreads / 64; ++i) {
    base += i < w ? s_n[i] : 0;
    total += s_n[i];
  }
#pragma unroll
  for (int q = 0; q < kCullPer; ++q)
    if (take[q]) {
      A.box[base + at[q]] = box[q];
      A.meta[base + at[q]] = make_int4(S.o0 + tid + kCullThreads * q, e0[q], mi[q], flags[q]);
    }
  if (tid == 0) A.cnt[blockIdx.x] = total;
}

constexpr int kCullRounds = 16;   // first list rounds kept in registers
constexpr int kCullCand = 64 * kCullRounds;   // candidates held between evaluations

// Waves per SIMD the compiler must fit: a wave is a chain of dependent loads
// and reductions, so four of them share a SIMD where the registers allow.
template <int MF, int MI>
constexpr int kCullWavesPerEU = (MI == 4 && MF <= 8) ? 4 : 1;

template <int MF, int MI>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(kCullWavesPerEU<MF, MI>)))
void cull_stage_kernel(CullArgs A) {
  __shared__ int cand[kCullCand];
  __shared__ float4 rf[MF];
  __shared__ FpLds fl;
  __shared__ WinnerLds wl;
  const int lane = threadIdx.x;
  typedef const __attribute__((address_space(4))) CullStage StC;
  const CullStage& R = *(const CullStage*)((StC*)A.stages + blockIdx.x);
  const int g = R.row, nseg = R.nseg;
  const float* p = A.poses + 3 * g;
  const float px = p[0], py = p[1], th = p[2];
  const float4* box = A.box + R.slot0;
  const int* cnt = A.cnt + R.seg0;
  // lane s: the length of segment s
  const int cv = lane < nseg ? cnt[lane] : 0;
  auto seg_n = [&](int r) { return (int)lane_u32((uint32_t)cv, r); };
  const FpConst& F = fp_const(A.fps, R.inst);

  // squared distance from the stage position to a box; -1 for an irregular
  // obstacle (last in the seed's order, within every bar)
  const bool within = fmaxf(fabsf(px), fabsf(py)) < kCullMax;
  auto dist2 = [&](const float4& b) {
    const float gx = fmaxf(fmaxf(b.x - px, px - b.z), 0.f);
    const float gy = fmaxf(fmaxf(b.y - py, py - b.w), 0.f);
    return (b.x == b.x && within) ? fmaf(gx, gx, gy * gy) : -1.f;
  };

  // ---- the seed.  Round r < kCullRounds: the first 64 entries of segment r,
  // kept in registers; the rest of the list is read again in the second pass.
  float d2[kCullRounds];
  uint32_t kb = 0xffffffffu;
  int sl = 0;
#pragma unroll
  for (int r0 = 0; r0 < kCullRounds; r0 += 8) {
    float4 b[8];
#pragma unroll
    for (int r = 0; r < 8; ++r)
      b[r] = r0 + r < nseg ? box[(r0 + r) * kSegObst + lane] : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      d2[r0 + r] = __builtin_huge_valf();
      const bool in = lane < seg_n(r0 + r);   // 0 past the last segment
      const float x = dist2(b[r]);
      if (in) {
        d2[r0 + r] = x;
        if (__float_as_uint(x) < kb) { kb = __float_as_uint(x); sl = (r0 + r) * kSegObst + lane; }
      }
    }
  }
  if (lane < MF) {
    float sn0, cs0;
    sincosf(th, &sn0, &cs0);
    rf[lane] = rotated_slot(F, lane, cs0, sn0);
  }
  stage_footprint(fl, F);
  float sn, cs;
  sincosf(th, &sn, &cs);
  // entries past the registers: f(slot, live) for 64 entries at a time
  const bool more = nseg > kCullRounds || __ballot(cv > 64) != 0;
  auto others = [&](auto f) {
    if (!more) return;
    for (int s = 0; s < nseg; ++s) {
      const int n = cnt[s];
      for (int i = s < kCullRounds ? 64 : 0; i < n; i += 64)
        f(s * kSegObst + i + lane, i + lane < n);
    }
  };
  others([&](int slot, bool live) {
    if (live) {
      const uint32_t u = __float_as_uint(dist2(box[slot]));
      if (u < kb) { kb = u; sl = slot; }
    }
  });
  const uint32_t kmin = fw_min_u32(kb);
  wave_sync();   // rf and fl are written

  uint64_t key = kEmptyKey;
  int we0 = 0, wmi = 0;   // the winner's edge range
  const bool pose_ok = isfinite(px) && isfinite(py) && isfinite(cs) && isfinite(sn);
  if (!pose_ok) {
    // every obstacle's sd is NaN: the first one that has an edge entry wins
    const int* off = A.off + R.obst_off;
    for (int o0 = 0; o0 < R.M; o0 += 64) {
      const int o = o0 + lane;
      const uint64_t m = __ballot(o < R.M && off[o + 1] != off[o]);
      if (m) {
        key = (uint64_t)(uint32_t)(o0 + __ffsll((unsigned long long)m) - 1);
        break;
      }
    }
  } else if (kmin != 0xffffffffu) {
    const int first = __ffsll((unsigned long long)__ballot(kb == kmin)) - 1;
    const int seed = (int)lane_u32((uint32_t)sl, first);
    const int4* meta = A.meta + R.slot0;

    // evaluates list slots, a quad of lanes per slot (four-edge class) or a
    // lane per slot, and folds them into (key, we0, wmi)
    auto fold = [&](uint64_t k, int e0, int mi) {
      const uint64_t kw = fw_min_u64(k);
      if (kw < key) {
        key = kw;
        const int f = __ffsll((unsigned long long)__ballot(k == kw)) - 1;
        we0 = (int)lane_u32((uint32_t)e0, f);
        wmi = (int)lane_u32((uint32_t)mi, f);
      }
    };
    auto quads = [&](int slot, bool act) {
      int4 m = make_int4(0, 0, 1, 2);
      if (act) m = meta[slot];
      const bool bad = (m.w & 2) != 0;
      QuadEdge q;
      float ax, ay, bx, by;
      quad_load(q, A.ax, A.ay, A.bx, A.by, m.y, m.z, (m.w & 1) != 0, act && !bad, F.eps, px, py,
                ax, ay, bx, by);
      const float sd = quad_eval<MF>(F, q, rf, [&](float& lo, float& hi) {
        quad_own(q, ax, ay, bx, by, lo, hi);
      });
      const uint32_t k = bad ? 0u : orderable(sd);
      fold(act ? ((uint64_t)k << 32) | (uint32_t)m.x : kEmptyKey, m.y, m.z);
    };
    auto lanes = [&](int slot, bool act) {
      int4 m = make_int4(0, 0, 0, 2);
      if (act) m = meta[slot];
      const bool bad = (m.w & 2) != 0;
      uint32_t k = 0u;
      if (!bad) {
        Obst<MI> ob;
        load_obstacle<MI>(ob, A.ax, A.ay, A.bx, A.by, m.y, m.z, 0x7fffffff, F.eps);
        k = orderable(obstacle_sd<MF, MI, true>(F, ob, rf, px, py));
      }
      fold(act ? ((uint64_t)k << 32) | (uint32_t)m.x : kEmptyKey, m.y, m.z);
    };
    if constexpr (MI == 4) quads(seed, true);
    else lanes(seed, lane == 0);

    // ---- the bar, and every listed obstacle within it
    const float phi = from_orderable((uint32_t)(key >> 32));   // NaN: the bar is tau
    const float bar = (fmaxf(phi, F.cull_tau) + F.rmax + kCullGamma) * (1.0f + 2.0f * F.cull_rel);
    const float bar2 = bar * bar;
    int n = 0;
    auto flush = [&]() {
      wave_sync();
      if (MI == 4 && n <= 32) {
        for (int c0 = 0; c0 < n; c0 += 16) {
          const int c = c0 + (lane >> 2);
          quads(c < n ? cand[c] : 0, c < n);
        }
      } else {
        for (int c0 = 0; c0 < n; c0 += 64) lanes(c0 + lane < n ? cand[c0 + lane] : 0, c0 + lane < n);
      }
      n = 0;
      wave_sync();
    };
    auto collect = [&](int slot, bool t) {
      const uint64_t m = __ballot(t);
      if (t) cand[n + (int)__popcll(m & ((1ull << lane) - 1ull))] = slot;
      n += (int)__popcll(m);
    };
#pragma unroll
    for (int r = 0; r < kCullRounds; ++r) {
      if (r >= nseg) break;
      const int slot = r * kSegObst + lane;
      collect(slot, lane < seg_n(r) && !(d2[r] > bar2) && slot != seed);
    }
    others([&](int slot, bool live) {
      if (n > kCullCand - 64) flush();
      collect(slot, live && slot != seed && !(dist2(box[slot]) > bar2));
    });
    flush();
  }
  const bool valid = key != kEmptyKey && (key >> 32) != 0 && wmi >= 1 && wmi <= kMaxObst;
  write_stage(F, fl, wl, A.ax, A.ay, A.bx, A.by, key, valid, we0, wmi, R.edge_off, cs, sn, px, py,
              g, A.keys, A.d, A.edge, A.obst, A.grad);
}

// Per footprint-size entry points (instantiated in psdf_batch_mf*.hip).
template <int MF>
hipError_t launch_cull_mf(int mi_class, int n_stages, const CullArgs& a, hipStream_t st) {
  if (mi_class == 4) cull_stage_kernel<MF, 4><<<n_stages, 64, 0, st>>>(a);
  else if (mi_class == 8) cull_stage_kernel<MF, 8><<<n_stages, 64, 0, st>>>(a);
  else cull_stage_kernel<MF, 16><<<n_stages, 64, 0, st>>>(a);
  return hipGetLastError();
}

#define PSDF_EXTERN_CULL(MF) \
  extern template hipError_t launch_cull_mf<MF>(int, int, const CullArgs&, hipStream_t);
PSDF_EXTERN_CULL(3)
PSDF_EXTERN_CULL(4)
PSDF_EXTERN_CULL(5)
PSDF_EXTERN_CULL(6)
PSDF_EXTERN_CULL(7)
PSDF_EXTERN_CULL(8)
PSDF_EXTERN_CULL(16)

}  // namespace psdf
