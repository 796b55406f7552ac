// Explicit instantiation of the persistent batch kernel and the culled stage
// kernel for 5 footprint slots.
#include "psdf_batch.hpp"
#include "psdf_cull.hpp"

namespace psdf {
template hipError_t launch_batch_mf<5>(int, int, int, const BatchArgs&, hipStream_t, hipEvent_t,
                                          hipEvent_t);
template hipError_t launch_cull_mf<5>(int, int, const CullArgs&, hipStream_t);
template hipError_t batch_occupancy_mf<5>(int, int, int*);
}  // namespace psdf
