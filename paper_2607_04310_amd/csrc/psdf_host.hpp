// Host-side helpers shared by the C-ABI entry points.
#pragma once

#include <hip/hip_runtime.h>

#include "psdf.h"
#include "psdf_device.hpp"

namespace psdf {

constexpr int kMaxStageBlock = 64;   // stages per work-group in the plain kernel

// Obstacles per work-group of the plain path's culled form.
constexpr int kCullBlk = 1024;

struct LaunchShape {
  int blk;  // obstacles per work-group: 64 or 256 (one per lane), or kCullBlk (culled)
  int sb;   // stages per work-group, 1..kMaxStageBlock
};

const char* last_error();
void clear_error();
int set_error(int code, const char* fmt, ...);
int hip_status(hipError_t err);

// Validate the footprint (m in [3, 16], strictly convex, no zero-length edge),
// orient it counter-clockwise and derive its constants in double precision.
int prepare_footprint(const float* xy, int m, const psdf_params* params, FpConst* out);

// Validate the host-side description of an edge set.
int check_edges(const psdf_edges* in, psdf_edges* out);

// Register class of the per-obstacle edge arrays for a bound mbar.
inline int obst_class(int mbar) { return mbar <= 4 ? 4 : (mbar <= 8 ? 8 : 16); }

// Whether eps leaves the edges of ordinary maps long enough for a bound: a
// centimetre at most (eps <= 2.5e-9).  A map of obstacles without one is evaluated
// whole by a wave per stage: 16 x 50 x 16384 rectangles of 0.1 to 0.8 m, eps 1e-8
// (4 cm) 23 us and full 182, but eps 1e-7 (0.4 m) 1460 and eps 1e-6 2140.
inline bool cull_edges_bounded(const FpConst& F) { return kCullEdge * F.eps <= 0.01f; }

// Footprints with a corner below 11 degrees and below 1.1 (FpConst::cull_open, the
// tangent of half an exterior angle): the bounds of open chains and of polygons that
// are not strictly convex are loose, and where a call is small the full evaluation
// is over before the culled one has left them out.
constexpr float kNeedle = 10.0f, kThinNeedle = 100.0f;

// Whether eps leaves the screens' circles a bound of the evaluation.  Its frame of
// an edge of length L is shrunk by eps / L, which moves a distance r by r eps / L;
// the circles have a millimetre to spare: 0.1 m edges at 100 m.
inline bool circles_bounded(const FpConst& F) { return F.eps <= 1e-6f; }

// Kernel timer: bracket one launch of the dominant kernel with events.
void timer_begin(hipStream_t st);
void timer_end(hipStream_t st);
// Or take an event pair for a launch that records them itself (the
// dispatch's own start and end, hipExtLaunchKernel); false when the timer is
// off or full.
bool timer_kernel_events(hipEvent_t* start, hipEvent_t* stop);

// Default launch shape of the per-stage minimum for N stages and M obstacles
// of at most mbar edges, and a footprint of m vertices.
LaunchShape choose_shape(const FpConst& F, int mbar, int N, int M);

// Launch shape for a problem: an explicit override (psdf_set_launch_shape),
// else choose_shape.
LaunchShape tuned_shape(const FpConst& F, int mbar, int N, int M);

hipError_t launch_plain(const FpConst& F, const float* poses, int N, const psdf_edges& e,
                        uint64_t* partial, const LaunchShape& ls, hipStream_t st);
hipError_t launch_epilogue(const FpConst& F, const float* poses, int N, const psdf_edges& e,
                           const uint64_t* partial, int gx, uint64_t* keys, const float* gout,
                           int mode, float dmin, float* d, int* edge, int* obst, float* grad,
                           float* hj, hipStream_t st);
int partial_columns(int M, const LaunchShape& ls);

}  // namespace psdf
