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
// An open chain or a polygon that is not strictly convex has fewer axes than
// its hull: only the robot's may separate it.  Some robot normal n is within
// half an exterior angle, alpha, of the direction u to its box; every point of
// the box lies beyond the nearest one along u and within its diagonal of it, so
// the gap on n at distance r is at least cos(alpha) (r - diagonal tan(alpha)):
// with the box enlarged by diagonal * tan(alpha) the bound above holds again (for
// a sliver of a footprint that is the whole plane).  At one stage more is known:
// a gap on a robot axis above its rounding (cull_separates) makes the evaluation
// call the two separated, and the box as it is bounds the distance.  Such an
// obstacle is stored with its box as it is and a mark; the list enlarges it, and
// tries the stages' axes where that leaves too many (cull_list_kernel), the stage
// kernel tries its axes, the plain kernel does the one or the other.  16 x 50 stages x
// 16384 chains of three edges, enlarged boxes stored -> enlarged where used -> and
// axes tried, us: hexagon 178 -> 27 -> 25 (full evaluation 240), equilateral triangle
// 181 -> 27 -> 27 (153), corner of 20 degrees 202 -> 56 -> 42 (150), of 5 degrees 331 ->
// 265 -> 52 (152); from staged boxes 358 -> 18 -> 17, 334 -> 19 -> 18, 344 -> 49 -> 34
// and 376 -> 256 -> 45.
// Any other obstacle (invalid, a degenerate edge, coordinates beyond 1e15) is
// irregular: it is always evaluated.
//
// Two launches:
//  * cull_list_kernel, one work-group per segment (kSegObst obstacles) of an
//    instance: boxes, and the list of the segment's obstacles that some stage
//    may need.  With B the bounding box of the instance's stage positions,
//    every stage's phi is at most
//        H = max(min_i (largest distance from B to a vertex of obstacle i)
//                + rmin, tau, log(axes) / eta)
//    (rmin the smallest |v_l|: separated sets are no further apart than a
//    vertex of each, and an obstacle that is not separated has
//    sd <= log(axes) / eta), so an obstacle whose bound from B exceeds H is
//    beyond phi and tau at every stage.
//  * cull_stage_kernel, one wave per stage: the listed obstacles nearest by
//    D are evaluated exactly; their least sd, or tau if that is larger, is a
//    bar T >= phi, and every listed obstacle with LB <= T is evaluated
//    exactly.  The minimum key over these is the stage's key: every other
//    obstacle has sd >= LB > T >= phi.  The wave then ends the stage
//    (write_stage).
// What it measured (graph replay per call, one card; full evaluation before):
// 64 instances x 50 stages x 16384 rectangles 539 -> 40 us (list 19 us for
// 67 MB of edges, stage 17.6 us), 512 uneven instances (23 800 stages, 2.7 M
// edges) 583 -> 73 us (list 21, stage 51 us).
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
constexpr float kCullPlane = 1e18f;                      // an enlargement to the whole plane

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

// A stored box is (lo.x, lo.y, hi.x, hi.y); lo.x NaN: irregular; with lo.x and
// hi.x exchanged: a loose obstacle's (CullBox).
struct CullBox {
  float lox, loy, hix, hiy;
  bool loose;
};
__device__ __forceinline__ CullBox cull_box(const float4& b) {
  return CullBox{fminf(b.x, b.z), b.y, fmaxf(b.x, b.z), b.w, b.x > b.z};
}

// What a loose obstacle's box is enlarged by on every side (0 for the others).
__device__ __forceinline__ float cull_enlargement(const FpConst& F, const CullBox& b) {
  const float size = (b.hix - b.lox) + (b.hiy - b.loy);
  return b.loose ? fminf(F.cull_open * size, kCullPlane) : 0.f;
}
// The box with that, unmarked.  (Its rounding is within the enlargement by rel *
// size that the box has: rel is above 1e-5.)
__device__ __forceinline__ float4 cull_enlarged(const FpConst& F, const float4& s) {
  const CullBox b = cull_box(s);
  const float e = cull_enlargement(F, b);
  return b.loose ? make_float4(b.lox - e, b.loy - e, b.hix + e, b.hiy + e) : s;
}

// The least of (W - p) . n over the points W of a box.
__device__ __forceinline__ float cull_axis(const CullBox& b, float px, float py, float nx,
                                           float ny) {
  const float cx = 0.5f * (b.lox + b.hix) - px, cy = 0.5f * (b.loy + b.hiy) - py;
  const float hx = 0.5f * (b.hix - b.lox), hy = 0.5f * (b.hiy - b.loy);
  return fmaf(cx, nx, fmaf(cy, ny, -fmaf(hx, fabsf(nx), hy * fabsf(ny))));
}

// Rounding of a gap on a robot axis between a box and the footprint, and of the
// evaluation's own projections of the obstacle on it: a dozen half ulps of the
// coordinates that enter, at most.
__device__ __forceinline__ float cull_axis_error(const FpConst& F, const CullBox& b, float px,
                                                 float py) {
  const float cx = 0.5f * (b.lox + b.hix) - px, cy = 0.5f * (b.loy + b.hiy) - py;
  const float hx = 0.5f * (b.hix - b.lox), hy = 0.5f * (b.hiy - b.loy);
  return fmaf(2e-6f, (fabsf(cx) + fabsf(cy)) + (hx + hy) + F.rmax, F.eps_sat + 1e-4f);
}

// Whether that gap makes the evaluation call the two separated.
__device__ __forceinline__ bool cull_separates(const FpConst& F, const CullBox& b, float px,
                                               float py, float gap) {
  return gap > cull_axis_error(F, b, px, py);
}

// A listed obstacle, one 64-byte record, so that the scan of the boxes brings
// in what the evaluation reads next: the box, the obstacle's index, first edge
// (global) and edge count, flags, and the points of a closed polygon of at most
// four edges (A_j) or of one edge (A_0, B_0).
constexpr int kListLoose = 1 << 30;
constexpr int kRecClosed = 1, kRecBad = 2, kRecPoints = 4;
struct CullRec {
  float4 box;
  int4 meta;
  float4 pts[2];
};
static_assert(sizeof(CullRec) == 64, "one record, one line");

// Slot l of an instance's footprint, 64 bytes, so that one wave reads a
// footprint with four vector loads:
//   v_l, u_l | e_l, 1 / (|e|^2 + eps), |e_l| | n_l, own interval | cu, cn, oa, ob
struct FpRow {
  float4 q[4];
};
inline FpRow fp_row(const FpConst& F, int l) {
  return FpRow{{make_float4(F.vx[l], F.vy[l], F.ux[l], F.uy[l]),
                make_float4(F.ex[l], F.ey[l], F.einv[l], F.len[l]),
                make_float4(F.nx[l], F.ny[l], F.pa[l], F.pb[l]),
                make_float4(F.cu[l], F.cn[l], F.oa[l], F.ob[l])}};
}

struct CullArgs {
  const FpConst* fps;
  const FpRow* rows;         // kMaxFp per instance
  const BatchInst* insts;
  const CullSeg* segs;
  const CullStage* stages;
  const float* poses;
  const float* ax;
  const float* ay;
  const float* bx;
  const float* by;
  const int* off;
  const float4* sbox;   // staged: every obstacle's box (kEmptyBox in lo.x: no edge) and
  const CullRec* srec;  // record, at slot0 + obstacle (null: from the edges)
  CullRec* rec;   // list slots
  int* cnt;       // per segment: list length, kListLoose where a loose obstacle is in it
  float* d;
  int* edge;
  int* obst;
  float* grad;
  uint64_t* keys;
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

// Box (NaN: irregular; loose: marked) and flags of the obstacle with edges
// [e0, e0 + mi), 1 <= mi <= MI and in range; the first edge (mi != 4) or all four
// (mi == 4) are in v (ax, ay, bx, by), and with kRecPoints in the flags its points
// are afterwards (v[0], v[1]: A_j).
template <int MI>
__device__ __forceinline__ void cull_obstacle(float (&v)[4][4], const float* __restrict__ gax,
                                              const float* __restrict__ gay,
                                              const float* __restrict__ gbx,
                                              const float* __restrict__ gby, int e0, int mi,
                                              float minl2, float rel, float4& box, int& flags) {
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
#pragma unroll
    for (int j = 1; j < (MI == 4 ? 4 : mi); ++j) {
      if (MI == 4 && j >= mi) break;
      const float a0 = gax[e0 + j], a1 = gay[e0 + j], b0 = gbx[e0 + j], b1 = gby[e0 + j];
      c.closed = c.closed && same_bits(bx, a0) && same_bits(by, a1);
      cull_point(c, a0, a1);
      cull_point(c, b0, b1);
      const float fx = b0 - a0, fy = b1 - a1;
      c.longe = c.longe && fmaf(fx, fx, fy * fy) >= minl2;
      cull_turn(c, ex, ey, fx, fy);
      ex = fx; ey = fy; bx = b0; by = b1;
      if (MI == 4) { v[0][j & 3] = a0; v[1][j & 3] = a1; }
    }
    if (mi == 1) { v[0][1] = bx; v[1][1] = by; }
    c.closed = c.closed && mi >= 3 && same_bits(bx, ax0) && same_bits(by, ay0);
    cull_turn(c, ex, ey, ex0, ey0);
  }
  const bool bad = c.bad != c.bad;
  // a strictly convex polygon turns one way and its direction changes half
  // twice in one round (a star turns one way too, in more rounds)
  const bool convex = mi == 1 || (c.closed && (c.left || c.right) && c.flips <= 2);
  const float big = fmaxf(fmaxf(fabsf(c.lox), fabsf(c.loy)), fmaxf(fabsf(c.hix), fabsf(c.hiy)));
  const bool fine = !bad && c.longe && big < kCullMax;
  // enlarged by its own size (rounding of the evaluation) and by the
  // rounding of the enlargement itself
  const float size = (c.hix - c.lox) + (c.hiy - c.loy);
  const float e = fmaf(rel, size, 2.5e-7f * big);
  const float lox = c.lox - e, hix = c.hix + e;
  box = fine && e < kCullMax
            ? make_float4(convex ? lox : hix, c.loy - e, convex ? hix : lox, c.hiy + e)
            : make_float4(__builtin_nanf(""), 0.f, 0.f, 0.f);
  flags = (c.closed ? kRecClosed : 0) | (bad ? kRecBad : 0) |
          (MI == 4 && (c.closed || mi == 1) ? kRecPoints : 0);
}

// The lo.x of a staged box whose obstacle has no edge.
constexpr float kEmptyBox = -__builtin_huge_valf();

__device__ __forceinline__ float cull_minl2(float eps) {
  const float l = kCullEdge * eps;
  return fmaxf(l * l, 1e-24f);
}

// One obstacle's edges on the way to its record: all four of a four-edge
// obstacle, else the first (loads only, so that several are in flight).
template <int MI>
struct CullLoad {
  float v[4][4];
  int e0, mi;
  bool ok;   // an edge count and range that the evaluation calls valid

  __device__ __forceinline__ void load(const CullArgs& A, const BatchInst& in, int Eend) {
    ok = mi >= 1 && mi <= MI && e0 >= in.edge_off && e0 <= Eend - mi;
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int j = 0; j < 4; ++j) v[k][j] = 0.f;
    if (!ok) return;
    const float* src[4] = {A.ax + e0, A.ay + e0, A.bx + e0, A.by + e0};
    if (mi == 4) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const Float4u u = *reinterpret_cast<const Float4u*>(src[k]);
#pragma unroll
        for (int j = 0; j < 4; ++j) v[k][j] = u.v[j];
      }
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k][0] = *src[k];
    }
  }
  __device__ __forceinline__ void finish(const CullArgs& A, const FpConst& F, float4& box,
                                         int& flags) {
    box = make_float4(__builtin_nanf(""), 0.f, 0.f, 0.f);
    flags = kRecBad;
    if (ok)
      cull_obstacle<MI>(v, A.ax, A.ay, A.bx, A.by, e0, mi, cull_minl2(F.eps), F.cull_rel, box,
                        flags);
  }
  __device__ __forceinline__ void record(CullRec* r, const float4& box, int o, int flags) const {
    r->box = box;
    r->meta = make_int4(o, e0, mi, flags);
    r->pts[0] = make_float4(v[0][0], v[1][0], v[0][1], v[1][1]);
    r->pts[1] = make_float4(v[0][2], v[1][2], v[0][3], v[1][3]);
  }
};

// Every obstacle's box and record, once per edge set (psdf_batch_stage).
template <int MI>
__global__ __launch_bounds__(256) void cull_stage_edges_kernel(CullArgs A, float4* sbox,
                                                               CullRec* srec) {
  typedef const __attribute__((address_space(4))) CullSeg SegC;
  const CullSeg& S = *(const CullSeg*)((SegC*)A.segs + blockIdx.y);
  const int k = blockIdx.x * 256 + threadIdx.x;
  if (k >= S.no) return;
  const BatchInst in = A.insts[S.inst];
  const int* off = A.off + in.obst_off + S.o0;
  CullLoad<MI> ld;
  ld.e0 = off[k];
  ld.mi = off[k + 1] - ld.e0;
  ld.e0 += in.edge_off;
  ld.load(A, in, in.edge_off + in.E);
  float4 box;
  int flags;
  ld.finish(A, fp_const(A.fps, S.inst), box, flags);
  if (ld.mi == 0) box.x = kEmptyBox;
  sbox[S.slot0 + k] = box;
  ld.record(srec + S.slot0 + k, box, S.o0 + k, flags);
}

// Bound: the read of every edge once (67 MB in 19 us at 64 x 16384
// rectangles), or of every staged box (17 MB in 10 us, the chain of loads
// and two barriers).  Each thread holds kCullPer obstacles whose loads are all
// in flight together.
constexpr int kAxisHorizon = 64;   // stages whose axes are tried on the list of any instance
constexpr int kAxisStages = kCullThreads / kMaxFp;   // stages whose axes are held at once
template <int MI, bool STAGED>
__global__ __launch_bounds__(kCullThreads) void cull_list_kernel(CullArgs A) {
  __shared__ float red[4][kCullThreads / 64];
  __shared__ float s_h[kCullThreads / 64];
  __shared__ int s_n[kCullThreads / 64];
  __shared__ float4 s_axes[kAxisStages * kMaxFp];   // n_l (world), cn_l
  __shared__ float2 s_pos[kAxisStages];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  typedef const __attribute__((address_space(4))) CullSeg SegC;
  const CullSeg& S = *(const CullSeg*)((SegC*)A.segs + blockIdx.x);
  const BatchInst in = A.insts[S.inst];
  const FpConst& F = fp_const(A.fps, S.inst);
  const int Eend = in.edge_off + in.E;
  const int* off = A.off + in.obst_off + S.o0;

  CullLoad<MI> ld[kCullPer];
  float4 box[kCullPer];
#pragma unroll
  for (int q = 0; q < kCullPer; ++q) {
    const int k = tid + kCullThreads * q;
    ld[q].e0 = ld[q].mi = 0;
    box[q] = make_float4(kEmptyBox, 0.f, 0.f, 0.f);
    if (k < S.no) {
      if (STAGED) {
        box[q] = A.sbox[S.slot0 + k];
      } else {
        ld[q].e0 = off[k];
        ld[q].mi = off[k + 1] - ld[q].e0;
        ld[q].e0 += in.edge_off;
      }
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
  if (!STAGED) {
#pragma unroll
    for (int q = 0; q < kCullPer; ++q) ld[q].load(A, in, Eend);
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

  int flags[kCullPer];
  // least upper bound of phi at every stage: an obstacle has a vertex on each
  // side of its box, so one within the largest distance from B to the
  // nearest-lying side.  The stored side is off by the enlargement and its
  // rounding (e of cull_obstacle and half an ulp, in x and in y: at most 1.5
  // times rel * size + 3.7e-7 * big), which is given back: without the second
  // term footprints ahead of their origin lost their nearest obstacle by up to
  // an ulp of the coordinates (6 cm at 600 km)
  float ub = __builtin_huge_valf();
#pragma unroll
  for (int q = 0; q < kCullPer; ++q) {
    if (!STAGED) {
      ld[q].finish(A, F, box[q], flags[q]);
      if (ld[q].mi == 0) box[q].x = kEmptyBox;
    }
    if (box[q].x == box[q].x && box[q].x != kEmptyBox) {
      const CullBox b = cull_box(box[q]);
      const float x0 = fmaxf(fabsf(b.lox - plx), fabsf(b.lox - phx));
      const float x1 = fmaxf(fabsf(b.hix - plx), fabsf(b.hix - phx));
      const float y0 = fmaxf(fabsf(b.loy - ply), fabsf(b.loy - phy));
      const float y1 = fmaxf(fabsf(b.hiy - ply), fabsf(b.hiy - phy));
      const float xs = fminf(x0, x1), xl = fmaxf(x0, x1), ys = fminf(y0, y1), yl = fmaxf(y0, y1);
      const float far2 = fminf(fmaf(xs, xs, yl * yl), fmaf(xl, xl, ys * ys));
      const float big =
          fmaxf(fmaxf(fabsf(b.lox), fabsf(b.hix)), fmaxf(fabsf(b.loy), fabsf(b.hiy)));
      const float off_side = fmaf(4.0f * F.cull_rel, (b.hix - b.lox) + (b.hiy - b.loy), 6e-7f * big);
      ub = fminf(ub, off_side + sqrtf(far2));
    }
  }
  ub = fw_min_f32(ub);
  if (lane == 0) s_h[w] = ub;
  __syncthreads();
  ub = s_h[0];
#pragma unroll
  for (int i = 1; i < kCullThreads / 64; ++i) ub = fminf(ub, s_h[i]);
  const float H = fmaxf(fmaf(ub, 1.0f + 1e-5f, F.rmin), F.sd_floor);
  const float bar = (H + F.rmax + kCullGamma) * (1.0f + 2.0f * F.cull_rel);
  const float bar2 = bar * bar;

  // the list, in obstacle order within each wave; open: loose obstacles that only
  // the stages' own axes can leave out
  bool take[kCullPer], open[kCullPer], marked = false;
#pragma unroll
  for (int q = 0; q < kCullPer; ++q) {
    const CullBox b = cull_box(box[q]);
    const float gx = fmaxf(fmaxf(b.lox - phx, plx - b.hix), 0.f);
    const float gy = fmaxf(fmaxf(b.loy - phy, ply - b.hiy), 0.f);
    const bool far = box[q].x == box[q].x && fmaf(gx, gx, gy * gy) > bar2 && !all;
    take[q] = box[q].x != kEmptyBox && !none && !far;
    open[q] = far && !none && b.loose;
    marked = marked || b.loose;
  }
  const bool some = __ballot(marked) != 0;   // loose obstacles in this wave
  if (some) {
#pragma unroll
    for (int q = 0; q < kCullPer; ++q) {
      const CullBox b = cull_box(box[q]);
      const float e = cull_enlargement(F, b);
      const float ex = fmaxf(fmaxf(b.lox - phx, plx - b.hix) - e, 0.f);
      const float ey = fmaxf(fmaxf(b.loy - phy, ply - b.hiy) - e, 0.f);
      open[q] = open[q] && !(fmaf(ex, ex, ey * ey) > bar2);
      take[q] = take[q] || open[q];
    }
  }
  // takes the counts (listed, and open among them: at most kSegObst each)
  int at[kCullPer], base, total;
  bool loose;
  auto count = [&]() {
    int n = 0, no = 0, lo = 0;
#pragma unroll
    for (int q = 0; q < kCullPer; ++q) {
      const uint64_t m = __ballot(take[q]);
      at[q] = n + lanes_below(m);
      n += (int)__popcll(m);
      if (some) {
        no += (int)__popcll(__ballot(open[q]));
        lo |= __ballot(take[q] && cull_box(box[q]).loose) ? kListLoose : 0;
      }
    }
    if (lane == 0) s_n[w] = n | no << 16 | lo;
    __syncthreads();
    base = S.slot0;
    total = no = 0;
    loose = false;
#pragma unroll
    for (int i = 0; i < kCullThreads / 64; ++i) {
      const int c = s_n[i] & 0xffff;
      base += i < w ? c : 0;
      total += c;
      no += s_n[i] >> 16 & 0xfff;
      loose = loose || (s_n[i] & kListLoose);
    }
    return no;
  };
  // The axes here cost half a microsecond a stage (three axes, one work-group per
  // CU), one after the other; an open obstacle per segment left on the list costs
  // every stage, which run beside each other, a 64th of a round, one to three times.
  // Worth it where a few hundred are open, and the horizon is short or the lists
  // many.  Chains of three edges, without -> with: 16 x 50 stages x 16384, corner of
  // 5 degrees 164 -> 52 us, of 0.1 degrees 269 -> 115, but 20 degrees, with fewer
  // open, 38 -> 55; 5 degrees, 16 x 100 x 16384 189 -> 80, 16 x 250 x 16384 190 ->
  // 158, but 16 x 200 x 4096 91 -> 157, 1 x 2000 x 16384 217 -> 1260, 1 x 20000 x
  // 2048 235 -> 12300 (full evaluation 376).
  if (count() > 64 * (F.m + 1) && in.N <= max(kAxisHorizon, 16 * ((in.M + kSegObst - 1) / kSegObst))) {
    for (int t0 = 0; t0 < in.N; t0 += kAxisStages) {
      __syncthreads();   // the last stages' axes are read
      {
        const int t = t0 + tid / kMaxFp, l = tid % kMaxFp;
        float4 v = make_float4(0.f, 0.f, -__builtin_huge_valf(), 0.f);   // no such stage: separated
        float2 at_p = make_float2(0.f, 0.f);
        if (t < in.N) {
          const float* p = A.poses + 3 * (in.pose_off + t);
          float sn, cs;
          sincosf(p[2], &sn, &cs);
          if (isfinite(p[0]) && isfinite(p[1]) && isfinite(cs) && isfinite(sn)) {
            const FpRow* r = A.rows + S.inst * kMaxFp + l;
            const float ux = r->q[0].z, uy = r->q[0].w;
            v = make_float4(fmaf(sn, ux, cs * uy), -fmaf(cs, ux, -(sn * uy)), r->q[3].y, 0.f);
            at_p = make_float2(p[0], p[1]);
          }
        }
        s_axes[tid] = v;
        if (l == 0) s_pos[tid / kMaxFp] = at_p;
      }
      __syncthreads();
      // two stages at a time (their table rows exist past the last stage)
      for (int t = 0; t < min(kAxisStages, in.N - t0); t += 2) {
        const float2 p0 = s_pos[t], p1 = s_pos[t + 1];
        float gap0[kCullPer], gap1[kCullPer];
#pragma unroll
        for (int q = 0; q < kCullPer; ++q) gap0[q] = gap1[q] = -__builtin_huge_valf();
        for (int l = 0; l < F.m; ++l) {
          const float4 n0 = s_axes[t * kMaxFp + l], n1 = s_axes[(t + 1) * kMaxFp + l];
#pragma unroll
          for (int q = 0; q < kCullPer; ++q) {
            const CullBox b = cull_box(box[q]);
            gap0[q] = fmaxf(gap0[q], cull_axis(b, p0.x, p0.y, n0.x, n0.y) - n0.z);
            gap1[q] = fmaxf(gap1[q], cull_axis(b, p1.x, p1.y, n1.x, n1.y) - n1.z);
          }
        }
#pragma unroll
        for (int q = 0; q < kCullPer; ++q) {
          const CullBox b = cull_box(box[q]);
          open[q] = open[q] && cull_separates(F, b, p0.x, p0.y, gap0[q]) &&
                    cull_separates(F, b, p1.x, p1.y, gap1[q]);
        }
      }
    }
#pragma unroll
    for (int q = 0; q < kCullPer; ++q) take[q] = take[q] && !open[q];
    __syncthreads();   // s_n and the last stages' axes are read
    count();
  }
#pragma unroll
  for (int q = 0; q < kCullPer; ++q)
    if (take[q]) {
      CullRec* r = A.rec + base + at[q];
      const int k = tid + kCullThreads * q;
      if (STAGED) *r = A.srec[S.slot0 + k];
      else ld[q].record(r, box[q], S.o0 + k, flags[q]);
    }
  if (tid == 0) A.cnt[blockIdx.x] = total | (loose ? kListLoose : 0);
}

constexpr int kCullRounds = 4;    // list entries kept in registers: 64 x this
constexpr int kCullFlat = 4096;   // list entries found through the start bits

// Listed obstacles as the evaluation reads them: the box, the meta word and
// edge j (at most the obstacle's last; act: without it, nothing) of a slot,
// from its record's points or else from the edge arrays.
template <int MI>
struct RecSource {
  const CullArgs& A;
  const CullRec* rec;
  __device__ __forceinline__ float4 box(int sl) const { return rec[sl].box; }
  __device__ __forceinline__ int4 meta(int sl) const { return rec[sl].meta; }
  __device__ __forceinline__ void edge(int sl, const int4& m, int j, bool act, float& ax,
                                       float& ay, float& bx, float& by) const {
    if (!act) return;
    const int e = min(j, m.z - 1);
    if (MI == 4 && (m.w & kRecPoints)) {
      const float2* p = reinterpret_cast<const float2*>(rec[sl].pts);
      const int n = m.z == 1 ? 1 : (e + 1 < m.z ? e + 1 : 0);
      const float2 a = p[e], b = p[n];
      ax = a.x; ay = a.y; bx = b.x; by = b.y;
    } else {
      ax = A.ax[m.y + e]; ay = A.ay[m.y + e]; bx = A.bx[m.y + e]; by = A.by[m.y + e];
    }
  }
};

// The least key so far, and its slot and meta word.
struct CullBest {
  uint64_t key;
  int slot;
  int4 meta;
  // the least sd: NaN once an invalid obstacle is in
  __device__ __forceinline__ float least() const {
    return key == kEmptyKey ? __builtin_huge_valf() : from_orderable((uint32_t)(key >> 32));
  }
};

// Squared distance from (px, py) to a stored box that is not marked; -1 for an
// irregular obstacle, or with ok false (last as unsigned bits, within every bar).
__device__ __forceinline__ float cull_dist2(const float4& s, float px, float py, bool ok) {
  const float gx = fmaxf(fmaxf(s.x - px, px - s.z), 0.f);
  const float gy = fmaxf(fmaxf(s.y - py, py - s.w), 0.f);
  return (s.x == s.x && ok) ? fmaf(gx, gx, gy * gy) : -1.f;
}

// The same at a stage whose rotated footprint fs is visible to the wave, boxes
// marked or not: a loose obstacle's box as it is, where a robot axis is sure to
// separate it, else 0.
__device__ __forceinline__ float cull_stage_dist2(const FpConst& F, const FpSlot* fs,
                                                  const float4& s, float px, float py, bool ok) {
  const CullBox b = cull_box(s);
  float d2 = cull_dist2(make_float4(b.lox, b.loy, b.hix, b.hiy), px, py, true);
  if (__ballot(b.loose)) {
    float gap = -__builtin_huge_valf();
    for (int l = 0; l < F.m; ++l)
      gap = fmaxf(gap, cull_axis(b, px, py, fs[l].r.w, -fs[l].r.z) - fs[l].cn);
    if (b.loose && !cull_separates(F, b, px, py, gap)) d2 = 0.f;
  }
  return (s.x == s.x && ok) ? d2 : -1.f;
}

// The bar of a least sd (a NaN: of tau) as a squared distance to a box.
__device__ __forceinline__ float cull_bar2(const FpConst& F, float sd) {
  const float b = (fmaxf(sd, F.cull_tau) + F.rmax + kCullGamma) * (1.0f + 2.0f * F.cull_rel);
  return b * b;
}

// Past the nearest box, what is evaluated with it, in footprint radii: far
// enough that the bar seldom asks for a second round, near enough that one
// round of groups holds it.
constexpr float kCullReach = 0.5f;

// What to evaluate first, least being the smallest squared distance: what
// every bar includes (T >= tau) or, where nothing is that near, the nearest
// and those not much further (irregular ones in either case); their least sd
// sets the bar, which seldom leaves more.
__device__ __forceinline__ float cull_first(const FpConst& F, float least) {
  const float first = cull_bar2(F, F.cull_tau);
  if (!(least > first)) return first;
  const float b = fmaf(kCullReach, F.rmax, sqrtf(least) * (1.0f + 1e-5f));
  return b * b;
}

constexpr int kCullCand = 192;    // candidates held between evaluations (three per lane)

// Evaluates the n candidates cand[0 .. n) (slots of src), a group of MI lanes
// each, and folds them into best.  More than one round of them is cut down by
// a second bound, the robot's axes against the box: on axis l the overlap is
// at most o_l = cn_l - min over the box of (W - p) . n_l.  Sets that overlap
// are no deeper than their overlap on any axis (and the soft minimum is below
// the minimum); separated ones are at least -o_l apart; ones within eps_sat
// have sd >= 0.  So sd >= -min_l o_l - eps_sat =: lb.  The lowest go first,
// then those whose lb does not exceed the least sd so far (a crowd of 50 to
// 130 overlapping boxes, or the map around a long footprint, leaves one or two
// rounds).  One whole wave; cand may be written just before by the wave.
template <int MI, class Src>
__device__ __forceinline__ void cull_evaluate(const FpConst& F, const FpSlot* fs, float* dls,
                                              const int* cand, uint8_t* pick, int n,
                                              const Src& src, float px, float py,
                                              CullBest& best) {
  const int lane = threadIdx.x & 63;
  wave_sync();
  float lb[kCullCand / 64];
  const bool cut = n > 64 / MI;
  float from = __builtin_nanf(""), to = __builtin_huge_valf();
#pragma unroll
  for (int h = 0; h < kCullCand / 64; ++h) {
    lb[h] = 0.f;
    if (cut && lane + 64 * h < n) {
      const float4 b = src.box(cand[lane + 64 * h]);
      const CullBox t = cull_box(b);
      float gap = -__builtin_huge_valf();
      for (int l = 0; l < F.m; ++l)
        gap = fmaxf(gap, cull_axis(t, px, py, fs[l].r.w, -fs[l].r.z) - fs[l].cn);
      const float low = gap - fmaf(F.cull_rel, F.rmax + 2.0f * fabsf(gap),
                                   cull_axis_error(F, t, px, py));
      lb[h] = b.x == b.x ? low : -__builtin_huge_valf();   // irregular: always
    }
  }
  if (cut) {
    float x = lb[0];
#pragma unroll
    for (int h = 1; h < kCullCand / 64; ++h) x = fminf(x, lb[h]);
    to = fminf(fw_min_f32(x) + 0.1f, best.least());
  }
  for (int step = 0; step < 2; ++step) {
    int np = 0;
#pragma unroll
    for (int h = 0; h < kCullCand / 64; ++h) {
      const bool t = lane + 64 * h < n && !(lb[h] > to) && !(lb[h] <= from);
      const uint64_t m = __ballot(t);
      if (t) pick[np + lanes_below(m)] = (uint8_t)(lane + 64 * h);
      np += (int)__popcll(m);
    }
    wave_sync();
    for (int c0 = 0; c0 < np; c0 += 64 / MI) {
      const int c = c0 + lane / MI;
      const bool act = c < np;
      const int sl = act ? cand[pick[c]] : 0;
      const int4 m = act ? src.meta(sl) : make_int4(0, 0, 1, kRecBad);
      const bool bad = (m.w & kRecBad) != 0;
      float ax = 0.f, ay = 0.f, bx = 0.f, by = 0.f;
      src.edge(sl, m, lane & (MI - 1), !bad, ax, ay, bx, by);
      const float sd = group_sd<MI>(F, fs, dls, ax, ay, bx, by, m.z, (m.w & kRecClosed) != 0, !bad,
                                    px, py);
      // the round's least sd, then its lowest obstacle
      const uint32_t none = 0xffffffffu;
      const uint32_t k = act ? (bad ? 0u : orderable(sd)) : none;
      const uint32_t kmin = fw_min_u32(k);
      const uint32_t omin = fw_min_u32(k == kmin && act ? (uint32_t)m.x : none);
      const uint64_t kw = ((uint64_t)kmin << 32) | omin;
      if (kw < best.key) {
        best.key = kw;
        const int f =
            __ffsll((unsigned long long)__ballot(act && k == kmin && (uint32_t)m.x == omin)) - 1;
        best.slot = (int)lane_u32((uint32_t)sl, f);
        best.meta = make_int4((int)(uint32_t)kw, (int)lane_u32((uint32_t)m.y, f),
                              (int)lane_u32((uint32_t)m.z, f), (int)lane_u32((uint32_t)m.w, f));
      }
    }
    wave_sync();
    if (!cut || best.least() <= to) break;
    from = to;
    to = best.least();
  }
}

// One wave per stage, MI lanes per evaluated obstacle.  Bound by its chain
// (list, footprint, candidates, the adjoint: 7 to 12 us) where the batch has
// few stages, by VALU issue where it has many.  The footprint's slots in a
// loop (group_sd) instead of an instance per footprint size: 72 VGPRs and seven
// waves per SIMD instead of 113 and four, and one launch for all sizes (512
// uneven instances: stage 177 -> 55 us).  A second bound on the candidates,
// and lists longer than the registers walked with four loads in flight, keep
// the crowded stages short (64 x 50 x 16384: 36 -> 19 us).  The segments'
// lists are read as one: lane s holds the
// length of segment s, their prefix sums place each segment's start as a bit
// in LDS, and entry f's segment is the number of bits up to f.
template <int MI>
__global__ __launch_bounds__(64) void cull_stage_kernel(CullArgs A) {
  __shared__ int cand[kCullCand];
  __shared__ uint8_t pick[kCullCand];
  __shared__ int segbase[64];
  __shared__ uint32_t starts[kCullFlat / 32];
  __shared__ FpSlot fs[kMaxFp];
  __shared__ float dls[64 / MI * kMaxFp];
  __shared__ FpLds fl;
  __shared__ WinnerLds wl;
  const int lane = threadIdx.x;
  typedef const __attribute__((address_space(4))) CullStage StC;
  const CullStage& R = *(const CullStage*)((StC*)A.stages + blockIdx.x);
  const int g = R.row, nseg = R.nseg;
  const float* p = A.poses + 3 * g;
  const float px = p[0], py = p[1], th = p[2];
  const CullRec* rec = A.rec + R.slot0;
  const int* cnt = A.cnt + R.seg0;
  const int cl = lane < nseg ? cnt[lane] : 0, cv = cl & ~kListLoose;
  const FpConst& F = fp_const(A.fps, R.inst);
  FpRow fr;
  if (lane < kMaxFp) fr = A.rows[R.inst * kMaxFp + lane];
  starts[lane] = starts[64 + lane] = 0u;

  const bool within = fmaxf(fabsf(px), fabsf(py)) < kCullMax;
  const bool loose = nseg > 64 || __ballot(cl & kListLoose) != 0;
  auto dist2 = [&](const float4& b) {
    return loose ? cull_stage_dist2(F, fs, b, px, py, within) : cull_dist2(b, px, py, within);
  };

  // ---- the list as one
  static_assert(kCullFlat == 64 * 64, "two words of starts per lane");
  int total;
  const int start = fw_scan_i32(cv, &total) - cv;
  wave_sync();
  const uint64_t full = __ballot(cv > 0);
  if (cv > 0) {
    segbase[lanes_below(full)] = lane * kSegObst - start;
    if (start < kCullFlat) atomicOr(&starts[start >> 5], 1u << (start & 31));
  }
  wave_sync();
  const int nflat = min(total, 64 * kCullRounds);
  // the slot of entry 64 r + lane (0 past entry n); ord: segments with entries
  // that start before round r, less one
  auto slot_of = [&](int r, int& ord, int n) {
    const uint64_t m = ((uint64_t)(uint32_t)uniform((int)starts[2 * r + 1]) << 32) |
                       (uint32_t)uniform((int)starts[2 * r]);
    int sl = 0;
    if (r * 64 + lane < n)
      sl = segbase[ord + lanes_below(m) + (int)((m >> lane) & 1ull)] + r * 64 + lane;
    ord += (int)__popcll(m);
    return sl;
  };
  int slot[kCullRounds];
  float d2[kCullRounds];
  uint32_t kb = 0xffffffffu;
  int ord0 = -1;
  float4 b0[kCullRounds];
  slot[0] = slot_of(0, ord0, nflat);
  b0[0] = rec[slot[0]].box;
  const bool longer = nflat > 64;
  if (longer) {
#pragma unroll
    for (int r = 1; r < kCullRounds; ++r) {
      slot[r] = slot_of(r, ord0, nflat);
      b0[r] = rec[slot[r]].box;
    }
  }
  // while these are in flight: the footprint at this stage
  float sn, cs;
  sincosf(th, &sn, &cs);
  if (lane < kMaxFp) {
    const float4 a = fr.q[0], e = fr.q[1], n = fr.q[2], c = fr.q[3];
    fl.vx[lane] = a.x; fl.vy[lane] = a.y;
    fl.ex[lane] = e.x; fl.ey[lane] = e.y; fl.einv[lane] = e.z;
    fl.nx[lane] = n.x; fl.ny[lane] = n.y; fl.pa[lane] = n.z; fl.pb[lane] = n.w;
    fs[lane] = FpSlot{rotated(a.x, a.y, a.z, a.w, cs, sn), c.x, c.y, e.w, c.z, c.w};
  }
  wave_sync();   // fs and fl are written
  d2[0] = dist2(b0[0]);
  if (lane < nflat) kb = __float_as_uint(d2[0]);
  if (longer) {
#pragma unroll
    for (int r = 1; r < kCullRounds; ++r) {
      d2[r] = dist2(b0[r]);
      if (r * 64 + lane < nflat) kb = min(kb, __float_as_uint(d2[r]));
    }
  }
  // The entries past the registers, four rounds of loads in flight:
  // f(slot, D^2, live) per round until it returns false (that round counts).
  // (r, ord) or, for a list longer than kCullFlat or of more than 64 segments,
  // (seg, at) is where the walk stands.
  struct Walk { int r, ord, seg, at; };
  const bool flat = total <= kCullFlat && nseg <= 64;
  auto walk = [&](Walk& k, auto f) {
    bool go = true;
    if (flat) {
      while (go && k.r * 64 < total) {
        int sl[4], ord = k.ord;
        float4 b[4];
        const int r0 = k.r & ~3;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          sl[u] = slot_of(r0 + u, ord, total);
          b[u] = rec[sl[u]].box;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (!go || r0 + u < k.r || (r0 + u) * 64 >= total) continue;
          go = f(sl[u], dist2(b[u]), (r0 + u) * 64 + lane < total);
          k.r = r0 + u + 1;
        }
        if (k.r == r0 + 4) k.ord = ord;
      }
      return k.r * 64 < total;
    }
    while (go && k.seg < nseg) {
      const int c = k.seg < 64 ? (int)lane_u32((uint32_t)cv, k.seg) : cnt[k.seg] & ~kListLoose;
      float4 b[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = k.at + 64 * u + lane;
        b[u] = rec[i < c ? k.seg * kSegObst + i : 0].box;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (!go || k.at >= c) continue;
        const int i = k.at + lane;
        go = f(k.seg * kSegObst + i, dist2(b[u]), i < c);
        k.at += 64;
      }
      if (k.at >= c) {
        ++k.seg;
        k.at = 0;
      }
    }
    return k.seg < nseg;
  };
  const bool in_regs = total <= 64 * kCullRounds && nseg <= 64;
  // past the registers, or (all = true) from the start
  auto walk_from = [&](bool all) {
    return flat && !all ? Walk{kCullRounds, ord0, 0, 0} : Walk{0, -1, 0, 0};
  };
  // (any distance within the bar of tau serves as the least one: cull_first)
  const uint32_t near = __float_as_uint(cull_bar2(F, F.cull_tau));
  if (!in_regs && !__ballot(kb <= near)) {
    Walk k = walk_from(false);
    walk(k, [&](int, float x, bool live) {
      if (live) kb = min(kb, __float_as_uint(x));
      return !__ballot(kb <= near);
    });
  }
  const uint32_t kmin = fw_min_u32(kb);

  CullBest best{kEmptyKey, 0, make_int4(0, 0, 0, 0)};
  const bool pose_ok = isfinite(px) && isfinite(py) && isfinite(cs) && isfinite(sn);
  if (!pose_ok) {
    // every obstacle's sd is NaN: the first one that has an edge entry wins
    const int* off = A.off + R.obst_off;
    for (int o0 = 0; o0 < R.M; o0 += 64) {
      const int o = o0 + lane;
      const uint64_t m = __ballot(o < R.M && off[o + 1] != off[o]);
      if (m) {
        best.key = (uint64_t)(uint32_t)(o0 + __ffsll((unsigned long long)m) - 1);
        break;
      }
    }
  } else if (kmin != 0xffffffffu) {
    const float first = cull_first(F, __uint_as_float(kmin));
    float lo = -2.f, hi = first;   // lo < D^2 <= hi
    for (int pass = 0; pass < 2; ++pass) {
      int n = 0;
      auto take = [&](int sl, float x, bool live) {
        const bool t = live && x > lo && !(x > hi);
        const uint64_t m = __ballot(t);
        const int at = n + lanes_below(m);
        if (t && at < kCullCand) cand[at] = sl;
        n += (int)__popcll(m);
      };
#pragma unroll
      for (int r = 0; r < kCullRounds; ++r) {
        if (r * 64 >= nflat) break;
        take(slot[r], d2[r], r * 64 + lane < nflat);
      }
      // more of the list: what the registers do not hold or, with more
      // candidates in them than the buffer holds (or a list too long for the
      // start bits), all of it again, a buffer at a time
      const bool again = n > kCullCand || !flat;
      bool rest = again || !in_regs;
      if (again) n = 0;
      Walk k = walk_from(again);
      do {
        if (rest && n <= kCullCand - 64)
          rest = walk(k, [&](int sl, float x, bool live) {
            take(sl, x, live);
            return n <= kCullCand - 64;
          });
        cull_evaluate<MI>(F, fs, dls, cand, pick, n, RecSource<MI>{A, rec}, px, py, best);
        n = 0;
      } while (rest);
      const float bar = cull_bar2(F, best.least());
      if (bar <= first) break;
      lo = first;
      hi = bar;
    }
  }
  const int4 wm = best.meta;
  const bool valid =
      best.key != kEmptyKey && (best.key >> 32) != 0 && wm.z >= 1 && wm.z <= kMaxObst;
  write_stage<MI>(F, fl, wl,
                  [&](int j, float& ax, float& ay, float& bx, float& by) {
                    RecSource<MI>{A, rec}.edge(best.slot, wm, j, true, ax, ay, bx, by);
                  },
                  best.key, valid, wm.y, wm.z, R.edge_off, cs, sn, px, py, g, A.keys, A.d, A.edge,
                  A.obst, A.grad);
}

// ------------------------------------------------------------------ plain calls

// Culled form of the plain path's per-stage minimum (psdf_kernels.hpp): the
// same partials for segments of kSegObst obstacles, one work-group per
// (segment, block of SB stages).  The work-group derives the segment's boxes
// once, in LDS; then each wave takes every fourth stage: the distances to
// the boxes, and exact evaluations of the segment's few obstacles within the
// bar that the nearest sets.  The segment's minimum is exact, so the
// epilogue reduces these partials as it does the full kernel's.  Bound by
// latency (12 to 14 us) up to about a million pairs; one pose against 1 M
// rectangles reads 68 MB in 22 us (full form 24 us, its evaluations of every
// obstacle), 50 x 65536 takes 19 us (54 us).
// Loose obstacles (open chains, polygons that are not strictly convex) are
// enlarged for blunt footprints and tried on the stage's axes for sharp ones (a
// corner below 53 degrees: an enlargement by more than twice the size).  200 x 16384
// chains, enlarged -> axes: hexagon 33 us either way, corner of 20 degrees 36 -> 34,
// 5 degrees 62 -> 39 (full 48), 0.1 degrees 80 -> 59 (47: choose_shape keeps it full).
constexpr float kCullSharp = 2.0f;
struct SegSource {
  const float* ax;
  const float* ay;
  const float* bx;
  const float* by;
  const float4* lbox;
  const int* le0;
  const uint16_t* lmeta;   // edge count << 4 | flags
  int o0;
  __device__ __forceinline__ float4 box(int sl) const { return lbox[sl]; }
  __device__ __forceinline__ int4 meta(int sl) const {
    const int m = lmeta[sl];
    return make_int4(o0 + sl, le0[sl], m >> 4, m & 15);
  }
  __device__ __forceinline__ void edge(int, const int4& m, int j, bool act, float& a0, float& a1,
                                       float& b0, float& b1) const {
    if (!act) return;
    const int e = m.y + min(j, m.z - 1);
    a0 = ax[e]; a1 = ay[e]; b0 = bx[e]; b1 = by[e];
  }
};

__device__ __forceinline__ FpSlot cull_slot(const FpConst& F, int l, float c, float s) {
  return FpSlot{rotated_slot(F, l, c, s), F.cu[l], F.cn[l], F.len[l], F.oa[l], F.ob[l]};
}

template <int MI, bool SHARP>
__global__ __launch_bounds__(kCullThreads) __attribute__((amdgpu_waves_per_eu(4)))
void cull_main_kernel(
    FpConst F, const float* __restrict__ poses, int N, int SB, const float* __restrict__ ax,
    const float* __restrict__ ay, const float* __restrict__ bx, const float* __restrict__ by,
    const int* __restrict__ off, int E, int M, ulonglong2* __restrict__ partial) {
  constexpr int kWaves4 = kCullThreads / 64, kBoxRounds = kSegObst / 64;
  __shared__ float4 lbox[kSegObst];
  __shared__ int le0[kSegObst];
  __shared__ uint16_t lmeta[kSegObst];
  __shared__ FpSlot fss[kWaves4][kMaxFp];
  __shared__ float dlss[kWaves4][64 / MI * kMaxFp];
  __shared__ int cands[kWaves4][kCullCand];
  __shared__ uint8_t picks[kWaves4][kCullCand];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int o0 = blockIdx.x * kSegObst, no = min(kSegObst, M - o0);
  const int s0 = blockIdx.y * SB, ns = min(SB, N - s0);
  FpSlot* fs = fss[w];
  float px = 0.f, py = 0.f, sn = 0.f, cs = 0.f;
  // the wave's first pose, in flight with the edges
  float th = 0.f;
  if (w < ns) {
    const float* p = poses + 3 * (s0 + w);
    px = p[0]; py = p[1]; th = p[2];
  }
  {
    CullArgs A{};
    A.ax = ax; A.ay = ay; A.bx = bx; A.by = by;
    BatchInst in{};
    CullLoad<MI> ld[kCullPer];
#pragma unroll
    for (int q = 0; q < kCullPer; ++q) {
      const int k = tid + kCullThreads * q;
      ld[q].e0 = ld[q].mi = 0;
      if (k < no) {
        ld[q].e0 = off[o0 + k];
        ld[q].mi = off[o0 + k + 1] - ld[q].e0;
      }
    }
#pragma unroll
    for (int q = 0; q < kCullPer; ++q) ld[q].load(A, in, E);
    if (w < ns) {
      sincosf(th, &sn, &cs);
      if (lane < F.m) fs[lane] = cull_slot(F, lane, cs, sn);
    }
#pragma unroll
    for (int q = 0; q < kCullPer; ++q) {
      const int k = tid + kCullThreads * q;
      float4 box;
      int flags;
      ld[q].finish(A, F, box, flags);
      if (ld[q].mi == 0) box.x = kEmptyBox;
      lbox[k] = SHARP ? box : cull_enlarged(F, box);
      le0[k] = ld[q].e0;
      lmeta[k] = (uint16_t)((ld[q].mi & 31) << 4 | (flags & 15));
    }
  }
  __syncthreads();
  const SegSource src{ax, ay, bx, by, lbox, le0, lmeta, o0};
  int* cand = cands[w];
  for (int t = w; t < ns; t += kWaves4) {
    const int s = s0 + t;
    if (t != w) {
      const float* p = poses + 3 * s;
      px = p[0]; py = p[1];
      sincosf(p[2], &sn, &cs);
      if (lane < F.m) fs[lane] = cull_slot(F, lane, cs, sn);
      wave_sync();
    }
    const bool within = fmaxf(fabsf(px), fabsf(py)) < kCullMax;
    const bool pose_ok = isfinite(px) && isfinite(py) && isfinite(cs) && isfinite(sn);
    CullBest best{kEmptyKey, 0, make_int4(0, 0, 0, 0)};
    float d2[kBoxRounds];   // NaN: no edge
    uint32_t kb = 0xffffffffu;
#pragma unroll
    for (int r = 0; r < kBoxRounds; ++r) {
      const float4 b = lbox[64 * r + lane];
      const bool empty = b.x == kEmptyBox;
      const float x = SHARP ? cull_stage_dist2(F, fs, b, px, py, within)
                            : cull_dist2(b, px, py, within);
      d2[r] = empty ? __builtin_nanf("") : x;
      kb = min(kb, empty ? 0xffffffffu : __float_as_uint(d2[r]));
    }
    const uint32_t kmin = fw_min_u32(kb);
    if (!pose_ok) {
      // every obstacle's sd is NaN: the segment's first one with an edge wins
      for (int k0 = 0; k0 < no && best.key == kEmptyKey; k0 += 64) {
        const uint64_t m = __ballot(lbox[k0 + lane].x != kEmptyBox);
        if (m) best.key = (uint64_t)(uint32_t)(o0 + k0 + __ffsll((unsigned long long)m) - 1);
      }
    } else if (kmin != 0xffffffffu) {
      const float first = cull_first(F, __uint_as_float(kmin));
      float lo = -2.f, hi = first;   // lo < D^2 <= hi
      for (int pass = 0; pass < 2; ++pass) {
        int r0 = 0;   // rounds before it are done
        do {
          int n = 0;
#pragma unroll
          for (int r = 0; r < kBoxRounds; ++r) {
            const bool t2 = d2[r] > lo && !(d2[r] > hi);
            const uint64_t m = __ballot(t2);
            const int c = (int)__popcll(m);
            if (r < r0 || n + c > kCullCand) continue;
            if (r != r0) continue;
            if (t2) cand[n + lanes_below(m)] = 64 * r + lane;
            n += c;
            ++r0;
          }
          if (n > 0) cull_evaluate<MI>(F, fs, dlss[w], cand, picks[w], n, src, px, py, best);
        } while (r0 < kBoxRounds);
        const float bar = cull_bar2(F, best.least());
        if (bar <= first) break;
        lo = first;
        hi = bar;
      }
    }
    if (lane == 0)
      partial[(size_t)s * gridDim.x + blockIdx.x] =
          make_ulonglong2(best.key, ((uint64_t)(uint32_t)best.meta.y << 32) | (uint32_t)best.meta.z);
  }
}

}  // namespace psdf
