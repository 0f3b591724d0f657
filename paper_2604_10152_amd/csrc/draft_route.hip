// Speculation-phase expert substitution (SpecMoE Sec. 3.2 "Affinity-based expert selection
// mechanism", Fig. 8): the draft model keeps only N experts of a block resident and uses the
// target's gate unchanged; when the gate picks a non-resident expert, the resident expert that
// is closest to it in an offline table of pairwise L2 distances between the experts' parameters
// takes its place.
//
//   nearest_draft_kernel : remap[e] for one set of draft experts (table: affinity.hip)
//
// The routing kernel applies remap[] to the ids it writes (route_topk.hip).
#include "common.h"

namespace specmoe {
namespace {

// remap[e] = e for a draft expert, else the draft expert with the smallest D[e, .]; equal
// distances go to the lower id.  Ids outside [0, E) in draft_ids are ignored; with no valid id
// at all the map is the identity.
__global__ __launch_bounds__(256) void nearest_draft_kernel(const float* __restrict__ affinity,
                                                            int E,
                                                            const int32_t* __restrict__ draft_ids,
                                                            int n_draft,
                                                            int32_t* __restrict__ remap) {
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= E) return;
    int best = -1;
    float bd = 0.f;
    bool resident = false;
    for (int q = 0; q < n_draft; ++q) {
        const int dd = draft_ids[q];
        if (dd < 0 || dd >= E) continue;
        if (dd == e) resident = true;
        const float dist = affinity[(size_t)e * E + dd];
        if (best < 0 || dist < bd || (dist == bd && dd < best)) { best = dd; bd = dist; }
    }
    remap[e] = (resident || best < 0) ? e : best;
}

}  // namespace

hipError_t launch_nearest_draft(const float* affinity, int E, const int32_t* draft_ids,
                                int n_draft, int32_t* remap, hipStream_t s) {
    hipLaunchKernelGGL(nearest_draft_kernel, dim3((E + 255) / 256), dim3(256), 0, s, affinity, E,
                       draft_ids, n_draft, remap);
    return hipGetLastError();
}

}  // namespace specmoe
