// Index phase of the permutation for up to 64 experts, by one workgroup: a kernel of its own (permute.hip), or the
// last workgroup of the router (route_topk.hip).
#pragma once
#include "common.h"

namespace specmoe {

constexpr int kSmallRows = 16;     // rows of 64 pairs a wave keeps in registers

__device__ __forceinline__ unsigned long long lanes_below(int lane) {
    return lane == 0 ? 0ull : (~0ull >> (kWave - lane));
}

// E <= 64, all WAVES waves of the workgroup; BITS: bits of an expert id; cnt: LDS.  AGENT: idx comes from other
// workgroups of the launch.
template <int WAVES, int BITS, bool AGENT>
__device__ __forceinline__ void permute_index_small(
    const int32_t* idx, int P, int E, int32_t* __restrict__ offsets,
    int32_t* __restrict__ row_src, int32_t* __restrict__ row_of, int (&cnt)[WAVES][kWave]) {
    const int tid = threadIdx.x, lane = tid % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    volatile int* mine = cnt[wave];
    const int per_wave = ((P + WAVES - 1) / WAVES + kWave - 1) / kWave * kWave;
    const int lo = min(P, wave * per_wave), hi = min(P, lo + per_wave);
    const bool once = per_wave <= kSmallRows * kWave;
    int ev[kSmallRows], place[kSmallRows];
    auto id = [&](int p) __attribute__((always_inline)) -> int {
        return AGENT ? __hip_atomic_load(idx + p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : idx[p];
    };
    // kSmallRows rows from `base`: the expert of every pair and its place behind mine[expert]
    auto walk = [&](int base) __attribute__((always_inline)) {
        const int rows = (hi - base + kWave - 1) / kWave;         // wave-uniform
#pragma unroll
        for (int b = 0; b < kSmallRows; ++b) {
            const int p = base + b * kWave + lane;
            ev[b] = p < hi ? id(p) : 0;
        }
#pragma unroll
        for (int b = 0; b < kSmallRows; ++b) {
            if (b >= rows) break;
            const bool valid = base + b * kWave + lane < hi;
            const int e = min(max(ev[b], 0), E - 1);
            unsigned long long same = __ballot(valid);
#pragma unroll
            for (int t = 0; t < BITS; ++t) {
                const unsigned long long m = __ballot((e >> t) & 1);
                same &= ((e >> t) & 1) ? m : ~m;
            }
            const int before = mine[e];
            __builtin_amdgcn_wave_barrier();
            const int rank = __popcll(same & lanes_below(lane));
            ev[b] = e;
            place[b] = before + rank;
            // the last lane of a group moves the count on (LDS accesses of a wave stay in order)
            if (valid && (same >> lane) == 1ull) mine[e] = before + rank + 1;
            __builtin_amdgcn_wave_barrier();
        }
    };
    mine[lane] = 0;                                                // private to the wave
    for (int base = lo; base < hi; base += kSmallRows * kWave) {
        walk(base);
        if (once) break;
#pragma unroll
        for (int b = 0; b < kSmallRows; ++b) {
            const int p = base + b * kWave + lane;
            if (p < hi) row_of[p] = place[b];
        }
    }
    __syncthreads();
    if (wave == 0) {                                               // lane e: expert e
        int c[WAVES], total = 0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) c[w] = cnt[w][lane];
#pragma unroll
        for (int w = 0; w < WAVES; ++w) total += c[w];
        const int incl = wave_scan(total);
        int run = incl - total;
        if (lane < E) offsets[lane] = run;
        if (lane == E - 1) offsets[E] = incl;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            cnt[w][lane] = run;
            run += c[w];
        }
    }
    __syncthreads();
    for (int base = lo; base < hi; base += kSmallRows * kWave) {
        if (!once) {
#pragma unroll
            for (int b = 0; b < kSmallRows; ++b) {
                const int p = base + b * kWave + lane;
                ev[b] = p < hi ? min(max(id(p), 0), E - 1) : 0;
                place[b] = p < hi ? row_of[p] : 0;
            }
        }
#pragma unroll
        for (int b = 0; b < kSmallRows; ++b) {
            const int p = base + b * kWave + lane;
            if (p < hi) {
                const int dest = mine[ev[b]] + place[b];
                row_src[dest] = p;
                row_of[p] = dest;
            }
        }
    }
}

}  // namespace specmoe
