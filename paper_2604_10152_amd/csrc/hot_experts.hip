// Temporally hot experts of one MoE block (SpecMoE Sec. 3.2 "Expert replacement policy", Fig. 7
// steps 3-4): during verification the activations of every expert are counted, and the N most
// activated experts become the draft experts of the next speculation phase.  The counts are the
// differences of expert_offsets, a by-product of moe_permute.  Ties go to the lower expert id.
// Thread e counts the experts in front of expert e on the key (count descending, id ascending):
// that is its place in the list.  E steps on counts that sit in LDS, against n rounds of a
// wave-wide arg-max before (16 of 64 experts 15.5 -> 3.6 us, 2 of 8 3.5 -> 2.4 us, 64 of 1024
// 235 -> 42 us).
// Integer work only.
#include "common.h"

namespace specmoe {
namespace {

constexpr int kMaxExperts = 1024;                      // SPECMOE_MAX_EXPERTS

__global__ __launch_bounds__(kMaxExperts) void hot_experts_kernel(
    const int32_t* __restrict__ offsets, int E, int n, int32_t* __restrict__ hot_ids,
    int32_t* __restrict__ hot_counts) {
    __shared__ __align__(16) int32_t counts[kMaxExperts];
    const int e = threadIdx.x;                         // blockDim: E rounded up to whole waves
    const int c = e < E ? offsets[e + 1] - offsets[e] : INT32_MIN;
    counts[e] = c;
    __syncthreads();
    int place = 0;
    for (int j0 = 0; j0 < E; j0 += 4) {                // entries beyond E hold INT32_MIN
        const int4 v = *reinterpret_cast<const int4*>(counts + j0);
        place += (v.x > c || (v.x == c && j0 < e)) + (v.y > c || (v.y == c && j0 + 1 < e)) +
                 (v.z > c || (v.z == c && j0 + 2 < e)) + (v.w > c || (v.w == c && j0 + 3 < e));
    }
    if (e < E && place < n) {
        hot_ids[place] = e;
        if (hot_counts) hot_counts[place] = c;
    }
}

}  // namespace

hipError_t launch_hot_experts(const int32_t* offsets, int E, int n, int32_t* hot_ids,
                              int32_t* hot_counts, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(hot_experts_kernel, dim3(1), dim3((E + kWave - 1) / kWave * kWave), 0, s, offsets, E, n, hot_ids,
                       hot_counts);
    return hipGetLastError();
}

}  // namespace specmoe
