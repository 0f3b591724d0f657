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

#include <type_traits>

namespace specmoe {
namespace {

// remap[e] = e for a draft expert, else the draft expert with the smallest D[e, .]; equal
// distances go to the lower id.  Ids outside [0, E) in draft_ids are ignored; with no valid id
// at all the map is the identity.
// Latency only: an id, then the distance that it points at.  A wave reads 64 ids at once and requests
// up to 16 distances together (64 experts, 16 ids, as a graph node 4.4 -> 3.2 us; 1024, 256 ids 61 ->
// 48); one or two ids take a shorter step, whose instructions they would wait for (1.9; 2.3 with 8).
__global__ __launch_bounds__(256) void nearest_draft_kernel(const float* __restrict__ affinity,
                                                            int E,
                                                            const int32_t* __restrict__ draft_ids,
                                                            int n_draft,
                                                            int32_t* __restrict__ remap) {
    const int e = blockIdx.x * 256 + threadIdx.x, lane = threadIdx.x % kWave;
    const float* row = affinity + (size_t)min(e, E - 1) * E;     // every lane stays for the exchange of ids
    int best = -1;
    float bd = 0.f;
    bool resident = false;
    for (int q0 = 0; q0 < n_draft; q0 += kWave) {
        const int n = min(kWave, n_draft - q0);
        int mine = lane < n ? draft_ids[q0 + lane] : -1;
        if (mine >= E) mine = -1;
        auto step = [&](auto count, int at) __attribute__((always_inline)) {
            constexpr int N = decltype(count)::value;
            int id[N];
            float dist[N];
#pragma unroll
            for (int i = 0; i < N; ++i) {
                id[i] = __builtin_amdgcn_readlane(mine, at + i);
                dist[i] = row[max(id[i], 0)];
            }
#pragma unroll
            for (int i = 0; i < N; ++i) {
                if (id[i] < 0) continue;
                if (id[i] == e) resident = true;
                if (best < 0 || dist[i] < bd || (dist[i] == bd && id[i] < best)) {
                    best = id[i];
                    bd = dist[i];
                }
            }
        };
        if (n <= 2) step(std::integral_constant<int, 2>{}, 0);
        else
            for (int at = 0; at < n; at += 16) step(std::integral_constant<int, 16>{}, at);
    }
    if (e < E) remap[e] = (resident || best < 0) ? e : best;
}

}  // namespace

hipError_t launch_nearest_draft(const float* affinity, int E, const int32_t* draft_ids,
                                int n_draft, int32_t* remap, hipStream_t s) {
    hipLaunchKernelGGL(nearest_draft_kernel, dim3((E + 255) / 256), dim3(256), 0, s, affinity, E,
                       draft_ids, n_draft, remap);
    return hipGetLastError();
}

}  // namespace specmoe
