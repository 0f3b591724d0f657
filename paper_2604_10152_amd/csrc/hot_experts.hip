// Temporally hot experts of one MoE block (SpecMoE Sec. 3.2 "Expert replacement policy", Fig. 7
// steps 3-4): during verification the activations of every expert are counted, and the N most
// activated experts become the draft experts of the next speculation phase.  The counts are the
// differences of expert_offsets, a by-product of moe_permute.  Ties go to the lower expert id.
// The place of an expert in the list is the number of experts in front of it on the key (count
// descending, id ascending).  A workgroup places 64 experts, one per lane; its waves split the
// experts to compare with and add up in LDS.  With all 1024 experts in one workgroup the E * E
// comparisons keep the four SIMDs of one CU busy for 42 us whatever n is; spread over 16 CUs they
// take 5.9 (64 experts: 2.2).
// Integer work only.
#include "common.h"

namespace specmoe {
namespace {

constexpr int kMaxExperts = 1024;                      // SPECMOE_MAX_EXPERTS
constexpr int kHotWaves = 8;

__global__ __launch_bounds__(kHotWaves * kWave) void hot_experts_kernel(
    const int32_t* __restrict__ offsets, int E, int n, int32_t* __restrict__ hot_ids,
    int32_t* __restrict__ hot_counts) {
    __shared__ __align__(16) int32_t counts[kMaxExperts];
    __shared__ int32_t before[kHotWaves][kWave];
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    const int padded = (E + kWave - 1) / kWave * kWave;
    for (int i = threadIdx.x; i < padded; i += kHotWaves * kWave)
        counts[i] = i < E ? offsets[i + 1] - offsets[i] : INT32_MIN;   // behind every expert
    __syncthreads();
    const int e = blockIdx.x * kWave + lane, c = counts[e];
    const int share = padded / kHotWaves;                               // a multiple of 8
    int place = 0;
    for (int j0 = wave * share; j0 < (wave + 1) * share; j0 += 4) {
        const int4 v = *reinterpret_cast<const int4*>(counts + j0);
        place += (v.x > c || (v.x == c && j0 < e)) + (v.y > c || (v.y == c && j0 + 1 < e)) +
                 (v.z > c || (v.z == c && j0 + 2 < e)) + (v.w > c || (v.w == c && j0 + 3 < e));
    }
    before[wave][lane] = place;
    __syncthreads();
    if (wave != 0 || e >= E) return;
#pragma unroll
    for (int w = 1; w < kHotWaves; ++w) place += before[w][lane];
    if (place < n) {
        hot_ids[place] = e;
        if (hot_counts) hot_counts[place] = c;
    }
}

}  // namespace

hipError_t launch_hot_experts(const int32_t* offsets, int E, int n, int32_t* hot_ids,
                              int32_t* hot_counts, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(hot_experts_kernel, dim3((E + kWave - 1) / kWave), dim3(kHotWaves * kWave), 0,
                       s, offsets, E, n, hot_ids, hot_counts);
    return hipGetLastError();
}

}  // namespace specmoe
