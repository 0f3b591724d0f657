// Gate of one MoE block: router logits in fp64, top-k on logits, softmax gate weights.
// (SpecMoE Sec. 2.1: the gate selects the top-K experts per token.)
//
// Two forms: vector (few tokens, fp32, more than 64 experts) and matrix (route_topk_mfma_kernel).
//
// Vector form: a workgroup owns TOK tokens and consists of 16/W groups of W wavefronts; group g takes
// the expert chunks g, g + 16/W, ... of EC experts each, so the widening of the router weights to fp64
// (every weight is converted once per workgroup) is spread over 1024 lanes.  Inside a group the
// d_model axis is dealt to its 64 W lanes in 16-byte chunks (chunk q -> wave (q/64) % W, lane
// q % 64), every lane keeps fp64 partial sums for TOK tokens x EC experts (TOK*EC <= 16), so one
// router-weight load feeds TOK tokens.
// The TOK*EC partial sums of a wave are reduced over its 64 lanes by a transposing butterfly:
// at the step with lane distance h a lane hands the half of its values that its partner keeps
// to the partner and adds what it receives, so 63 exchange-and-add steps reduce all values at
// once (a plain butterfly needs 6 per value) and lane l ends up with the total of value l.
// Every value is summed over the same pairs of lanes in the same order, and fp addition is
// commutative, so two experts with identical router rows get bit-identical logits and the tie
// goes to the lower id.  The W wave totals are added in fixed order.  Wave t then ranks token
// t, the E logits sitting in LDS.  It is a chain of latencies: the columns are requested one step ahead,
// the bias and (up to 64 experts) the substitution at the start, the lanes exchange in registers: 64 experts x 2048, 64 tokens
// 11.0 -> 8.9 us, 320 tokens 13.4 -> 11.0 (4 of these the fp64 work of one CU, 2.5 the launch).
#include "permute_index.h"

#include <type_traits>

namespace specmoe {
namespace {

constexpr int kRouteThreads = 1024;                   // 16 wavefronts: groups of W, which split the experts
constexpr int kAheadRows = 9;                         // token and router rows a lane can request twice

template <typename T, bool VEC> struct Chunk;
template <> struct Chunk<float, true> {
    static constexpr int N = 4;
    typedef U128 Raw;
    __device__ static Raw load(const float* p) { return *reinterpret_cast<const U128*>(p); }
    __device__ static double get(const Raw& v, int i) { return (double)__uint_as_float(v[i]); }
};
template <> struct Chunk<bf16_t, true> {
    static constexpr int N = 8;
    typedef U128 Raw;
    __device__ static Raw load(const bf16_t* p) { return *reinterpret_cast<const U128*>(p); }
    __device__ static double get(const Raw& v, int i) {
        const uint32_t w = v[i >> 1];
        return (double)__uint_as_float(i & 1 ? w & 0xffff0000u : w << 16);
    }
};
template <typename T> struct Chunk<T, false> {          // any d_model, any alignment
    static constexpr int N = 1;
    typedef float Raw;
    __device__ static Raw load(const T* p) { return load_as_float(p); }
    __device__ static double get(const Raw& v, int) { return (double)v; }
};

// An id goes past the L2, which every die has of its own: the workgroup that permutes may run on another one.
__device__ __forceinline__ void store_id(int32_t* p, int id) {
    __hip_atomic_store(p, id, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// among numbers
__device__ __forceinline__ bool better(double av, int aid, double bv, int bid) {
    return (av > bv) || (av == bv && aid < bid);
}

// Ranks token t by one wave, E <= 64: one expert per lane, on the key (logit descending, id
// ascending; NaN last).  A round per slot (the largest logit that is left, exchanged in registers) costs about 200
// cycles.  Up to 3 k experts every lane counts the experts that beat its own instead - its rank, i.e.
// the slot it would fill -, the other logits arriving through v_readlane broadcasts.  Kernel time, rounds /
// counting: 64 experts x 2048, top-6 8.9 / 11.2 us, top-16 11.0 / 11.6, 16 experts top-4 5.1 / 5.3, 8 top-2 4.3 / 4.3.
// id: what an expert is called in the output (the draft mode's substitution).
template <bool THEN>
__device__ __forceinline__ void rank_token(const double* logit, int lane, int E, int k, int renorm,
                                           int t, int32_t* __restrict__ idx_out,
                                           float* __restrict__ w_out, int id) {
    const bool valid = lane < E;
    const double v = valid ? logit[lane] : 0.0;
    auto lane_value = [&](double val, int src) __attribute__((always_inline)) -> double {
        const long long bits = __double_as_longlong(val);
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)bits, src);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)bits >> 32), src);
        return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
    };
    int rank;
    if (E <= 3 * k) {
        rank = 0;
#pragma unroll 8
        for (int j = 0; j < E; ++j) rank += better(lane_value(v, j), j, v, lane) ? 1 : 0;
        const unsigned long long nan = __ballot(valid && v != v);   // (none of them beats a number)
        if (v != v) rank = E - __popcll(nan) + __popcll(nan & ((1ull << lane) - 1));
    } else {
        rank = k;
        for (int sl = 0; sl < k; ++sl) {
            const bool open = valid && rank == k;
            const double top = wave_max(open ? v : -__builtin_inf());
            unsigned long long at = __ballot(open && v == top);       // the lowest id of equal logits
            if (!at) at = __ballot(open);                             // nothing left but NaN
            if (lane == __ffsll((long long)at) - 1) rank = sl;
        }
    }
    const int first = __builtin_amdgcn_readfirstlane(
        __ffsll((long long)__ballot(valid && rank == 0)) - 1);
    const double vmax = lane_value(v, first);
    // softmax over all E experts, relative to the largest logit
    const double pe = valid ? exp(v - vmax) : 0.0;
    const double p = pe / wave_sum(pe);
    double wsum_sel = 0.0;                            // slot order, identical on every lane
    for (int sl = 0; sl < k; ++sl) {
        const int src = __builtin_amdgcn_readfirstlane(
            __ffsll((long long)__ballot(valid && rank == sl)) - 1);
        wsum_sel += lane_value(p, src);
    }
    if (valid && rank < k) {
        if (THEN) store_id(idx_out + (size_t)t * k + rank, id);
        else idx_out[(size_t)t * k + rank] = id;
        w_out[(size_t)t * k + rank] = (float)(renorm ? p / wsum_sel : p);
    }
}

// What follows the ranking where the caller has a counter for it: the index phase of the permutation, by the workgroup
// that is done last, so that a layer has a launch less (2.4 us of a kernel that does nothing, and the way to it).
// done: workgroups that are, back at 0 behind the last one.  A workgroup counts only when its ids have arrived in memory
// (store_id() and the wait), and the last one reads them there.  Fences of agent scope instead write back and drop the
// whole L2, once per workgroup (320 tokens x 64 experts 11.5 + 4.9 us as two kernels, 20.2 with fences, 16.8 so).
struct Then {
    uint32_t* done;
    int32_t *offsets, *row_src, *row_of;
};
template <int WAVES>
__device__ __forceinline__ void permute_if_last(const Then& then, const int32_t* idx, int P, int E) {
    __shared__ int cnt[WAVES][kWave];
    __shared__ bool last;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) last = atomicInc(then.done, gridDim.x - 1) == gridDim.x - 1;
    __syncthreads();
    if (last) permute_index_small<WAVES, 6, true>(idx, P, E, then.offsets, then.row_src, then.row_of, cnt);
}

// THEN: as Then says.  A form of its own: the registers of the index phase leave room for fewer workgroups (277 tokens of 43
// columns, fp32 layer 34.9 -> 35.9).
template <typename T, bool VEC, int TOK, int EC, int W, bool THEN>
__global__ __launch_bounds__(kRouteThreads) void route_topk_kernel(
    const T* __restrict__ x, const T* __restrict__ wr, const float* __restrict__ bias, int Tn,
    int d, int E, int k, int renorm, int32_t* idx_out, float* __restrict__ w_out,
    const int32_t* __restrict__ remap /* nullable: draft-mode expert substitution, [E] */, Then then) {
    static_assert(TOK * EC <= 16 && (TOK * EC & (TOK * EC - 1)) == 0, "values per wave");
    constexpr int NV = TOK * EC;                      // partial sums per lane and pass
    constexpr int kGroupThreads = W * kWave, kRouteGroups = kRouteThreads / kGroupThreads;
    extern __shared__ double lds_d[];                 // logits[TOK][E], then part[groups][W][NV]
    double* logits = lds_d;
    typedef Chunk<T, VEC> CH;
    constexpr int V = CH::N;
    constexpr int G = EC < 8 ? EC : 8;                // router rows loaded together
    // the next columns are requested before the present ones are used, where the registers allow it
    constexpr bool AHEAD = VEC && EC <= 8 && TOK + EC <= kAheadRows;
    const int lane = threadIdx.x % kWave;
    const int wave_all = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int group = wave_all / W, wave = wave_all % W;
    const int gtid = threadIdx.x % kGroupThreads;     // thread index inside the group
    double* part = lds_d + (size_t)TOK * E + (size_t)group * W * NV;
    const int t0 = blockIdx.x * TOK;
    const int nq = d / V;                             // chunks per row (VEC: d % V == 0)
    // what the ranking needs from memory is requested up front
    const int id = remap && lane < E ? remap[lane] : lane;      // E <= 64

    // every group runs the same number of passes (the barriers inside are workgroup-wide); a
    // group whose chunk lies beyond E skips the arithmetic of that pass
    const int passes = (E + kRouteGroups * EC - 1) / (kRouteGroups * EC);
    for (int pass = 0; pass < passes; ++pass) {
        const int e0 = (pass * kRouteGroups + group) * EC;
        const bool live = e0 < E;
        double acc[NV];                               // index t * EC + c
#pragma unroll
        for (int i = 0; i < NV; ++i) acc[i] = 0.0;
        const int e_mine = e0 + gtid % EC;
        const double shift = bias && gtid < NV && e_mine < E ? (double)bias[e_mine] : 0.0;
        typedef typename CH::Raw Raw;
        auto load_x = [&](Raw (&xr)[TOK], int q) __attribute__((always_inline)) {
#pragma unroll
            for (int t = 0; t < TOK; ++t)
                xr[t] = CH::load(x + (size_t)min(t0 + t, Tn - 1) * d + (size_t)q * V);
        };
        auto load_w = [&](Raw (&w)[G], int c0, int q) __attribute__((always_inline)) {
#pragma unroll
            for (int c = 0; c < G; ++c)
                w[c] = CH::load(wr + (size_t)min(e0 + c0 + c, E - 1) * d + (size_t)q * V);
        };
        auto add = [&](const Raw (&xr)[TOK], const Raw (&w)[G], int c0) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < V; ++i) {
                double xv[TOK];
#pragma unroll
                for (int t = 0; t < TOK; ++t) xv[t] = CH::get(xr[t], i);
#pragma unroll
                for (int c = 0; c < G; ++c) {
                    const double wv = CH::get(w[c], i);
#pragma unroll
                    for (int t = 0; t < TOK; ++t)
                        acc[t * EC + c0 + c] = fma(xv[t], wv, acc[t * EC + c0 + c]);
                }
            }
        };
        if constexpr (AHEAD) {
            Raw xn[TOK], wn[G];
            if (live) {
                load_x(xn, min(gtid, nq - 1));
                load_w(wn, 0, min(gtid, nq - 1));
            }
            for (int q = gtid; live && q < nq; q += kGroupThreads) {
                Raw xr[TOK], w[G];
#pragma unroll
                for (int t = 0; t < TOK; ++t) xr[t] = xn[t];
#pragma unroll
                for (int c = 0; c < G; ++c) w[c] = wn[c];
                const int next = q + kGroupThreads;
                if (next < nq) {
                    load_x(xn, next);
                    load_w(wn, 0, next);
                }
                __builtin_amdgcn_sched_barrier(0);
                add(xr, w, 0);
            }
        } else {
            for (int q = gtid; live && q < nq; q += kGroupThreads) {
                Raw xr[TOK], w[G];
                load_x(xr, q);
#pragma unroll
                for (int c0 = 0; c0 < EC; c0 += G) {
                    load_w(w, c0, q);
                    add(xr, w, c0);
                }
            }
        }
        // lanes -> wave totals (transposing butterfly), waves -> workgroup total (in order)
        TransposeReduce<NV, kWave / 2>::run(acc, lane);
        constexpr int REP = kWave / NV;               // lanes holding the same value
        if (lane % REP == 0) part[wave * NV + lane / REP] = acc[0];
        __syncthreads();
        if (gtid < NV) {
            const int t = gtid / EC, c = gtid % EC;
            if (e0 + c < E) {
                double s = part[gtid];
#pragma unroll
                for (int w = 1; w < W; ++w) s += part[w * NV + gtid];
                logits[(size_t)t * E + e0 + c] = s + shift;
            }
        }
        __syncthreads();
    }

    // wave t of the workgroup ranks token t0 + t (TOK <= 4)
    const int t = t0 + wave_all;
    const double* logit = logits + (size_t)wave_all * E;
    if (E <= kWave) {
        if (wave_all < TOK && t < Tn) rank_token<THEN>(logit, lane, E, k, renorm, t, idx_out, w_out, id);
        if constexpr (THEN) permute_if_last<kRouteThreads / kWave>(then, idx_out, Tn * k, E);
        return;
    }
    if (wave_all >= TOK || t >= Tn) return;
    // More than 64 experts: lane owns experts lane, lane+64, ...; `taken` marks the ones already
    // selected.  Lane s keeps the result of round s (k <= 64), so the final stores are coalesced.
    constexpr int kOwn = 1024 / kWave;                // SPECMOE_MAX_EXPERTS / 64
    double wsum_sel, my_p = 0.0;
    int my_id = 0;
    // NANS: ranks NaN last; without, false if there is one (256 tokens, 1024 columns, 256 experts, top-8: 25.9 us; with
    // the comparison for all tokens, exchanges through LDS as before, 29.2 against 27.3)
    auto rank = [&](auto nans) __attribute__((always_inline)) -> bool {
        constexpr bool NANS = decltype(nans)::value;
        auto wins = [](double av, int aid, double bv, int bid) {
            return better(av, aid, bv, bid) || (NANS && bv != bv && (av == av || aid < bid));
        };
        uint32_t taken = 0;
        double vmax = 0.0, denom = 1.0;
        wsum_sel = 0.0;
        for (int s = 0; s < k; ++s) {
            struct Best { double v; int64_t id; } best = {0.0, -1};      // (no padding: exchanged by words)
#pragma unroll 1
            for (int o = 0; o < kOwn; ++o) {
                int e = lane + o * kWave;
                if (e >= E) break;
                if (taken & (1u << o)) continue;
                double v = logit[e];
                if (best.id < 0 || wins(v, e, best.v, (int)best.id)) best = {v, e};
            }
            best = specmoe::wave_all(best, [&](Best a, Best b) {
                return b.id >= 0 && (a.id < 0 || wins(b.v, (int)b.id, a.v, (int)a.id)) ? b : a;
            });
            const double bv = best.v;
            const int bid = (int)best.id;
            if ((bid % kWave) == lane) taken |= 1u << (bid / kWave);
            if (s == 0) {
                // softmax denominator over all E experts, relative to the largest logit
                vmax = bv;
                double p = 0.0;
                for (int e = lane; e < E; e += kWave) p += exp(logit[e] - vmax);
                denom = wave_sum(p);
                if (!NANS && __any(denom != denom)) return false;
            }
            double p = exp(bv - vmax) / denom;
            wsum_sel += p;                            // slot order, identical on every lane
            if (lane == s) { my_p = p; my_id = bid; }
        }
        return true;
    };
    if (!rank(std::false_type{})) rank(std::true_type{});
    if (lane < k) {
        idx_out[(size_t)t * k + lane] = remap ? remap[my_id] : my_id;
        w_out[(size_t)t * k + lane] = (float)(renorm ? my_p / wsum_sel : my_p);
    }
}

// Many tokens, at most 64 experts, bf16: logits on the fp64 matrix cores.  v_mfma_f64_4x4x4 takes
// 16 cycles for four independent 4 x 4 x 4 blocks - as many multiply-adds per cycle as the vector
// unit - and sums over the contraction by itself, so neither partial sums per lane nor the
// butterfly over 64 lanes are needed, and a workgroup of 8 waves needs few enough registers
// that several share a CU and hide each other's memory and ranking phases.  What bounds it is
// issue on the fp64 pipe, about half of it the widening conversions (as fast as a multiply-add,
// but one per weight and 4 RT tokens).
// A workgroup owns 4 RT tokens (a widened router weight serves RT instructions).  Lane l = i + 4 (b +
// 4 q) of an operand is row i, contraction element q of block b: the blocks hold the same 4 tokens and 4 experts each (16 experts per instruction,
// NG instructions for all), or with KS = 2 or 4 (at most 8 or 4 experts) the same experts at KS
// different column ranges, which are added at the end.  A lane loads 16 bytes, so a unit of 32 KS
// columns is 8 steps; the waves take units in turn.  Every expert's logit goes through the same
// order of additions, so duplicated router rows tie exactly.  Products and sums in fp64 as in the
// vector form.
constexpr int kMfmaWaves = 8;

template <int NG, int KS, int RT>
__global__ __launch_bounds__(kMfmaWaves * kWave) void route_topk_mfma_kernel(
    const bf16_t* __restrict__ x, const bf16_t* __restrict__ wr, const float* __restrict__ bias,
    int Tn, int d, int E, int k, int renorm, int32_t* __restrict__ idx_out,
    float* __restrict__ w_out, const int32_t* __restrict__ remap) {
    typedef Chunk<bf16_t, true> CH;
    constexpr int BE = 4 / KS;                        // blocks with experts of their own
    constexpr int PF = 2;                             // units in flight
    __shared__ double part[kMfmaWaves][RT * NG][kWave];
    __shared__ double logits[4 * RT][kWave];
    const int lane = threadIdx.x % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int t0 = blockIdx.x * (4 * RT);
    const int i = lane & 3, b = (lane >> 2) & 3, q = lane >> 4;
    const int col0 = (b / BE) * 32 + q * 8;           // column of this lane inside a unit
    const bf16_t* xrow[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) xrow[r] = x + (size_t)min(t0 + 4 * r + i, Tn - 1) * d;
    const bf16_t* wrow[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) wrow[g] = wr + (size_t)min(16 * g + 4 * (b % BE) + i, E - 1) * d;
    const int units = (d + 32 * KS - 1) / (32 * KS);
    // what the ranking needs from memory is requested up front
    static_assert(RT * NG <= kMfmaWaves, "a wave adds up one result register");
    const int id = remap && lane < E ? remap[lane] : lane;
    const int e_mine = 16 * (wave % NG) + 4 * (b % BE) + i;
    const double shift = bias && e_mine < E ? (double)bias[e_mine] : 0.0;

    U128 xr[PF][RT], wv[PF][NG];
    bool live[PF];
    auto load = [&](int p, int u) __attribute__((always_inline)) {
        const int col = u * (32 * KS) + col0;
        live[p] = col < d;                            // d % 8 == 0: a whole piece or nothing
        const int at = live[p] ? col : 0;
#pragma unroll
        for (int r = 0; r < RT; ++r) xr[p][r] = CH::load(xrow[r] + at);
#pragma unroll
        for (int g = 0; g < NG; ++g) wv[p][g] = CH::load(wrow[g] + at);
        __builtin_amdgcn_sched_barrier(0);            // the requests stay ahead of their use
    };
    double acc[RT * NG];
#pragma unroll
    for (int g = 0; g < RT * NG; ++g) acc[g] = 0.0;
#pragma unroll
    for (int p = 0; p < PF; ++p) load(p, wave + p * kMfmaWaves);
    for (int u0 = wave; u0 < units; u0 += PF * kMfmaWaves) {
#pragma unroll
        for (int p = 0; p < PF; ++p) {
            const U128 zero = {0, 0, 0, 0};
            U128 xc[RT], wc[NG];
#pragma unroll
            for (int r = 0; r < RT; ++r) xc[r] = live[p] ? xr[p][r] : zero;
#pragma unroll
            for (int g = 0; g < NG; ++g) wc[g] = live[p] ? wv[p][g] : zero;
            load(p, u0 + (p + PF) * kMfmaWaves);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                double xd[RT];
#pragma unroll
                for (int r = 0; r < RT; ++r) xd[r] = CH::get(xc[r], e);
#pragma unroll
                for (int g = 0; g < NG; ++g) {
                    const double wd = CH::get(wc[g], e);
#pragma unroll
                    for (int r = 0; r < RT; ++r)
                        acc[r * NG + g] =
                            __builtin_amdgcn_mfma_f64_4x4x4f64(xd[r], wd, acc[r * NG + g], 0, 0, 0);
                }
            }
        }
    }
    // lane l holds token l / 16, expert column l % 4 of block (l / 4) % 4
#pragma unroll
    for (int g = 0; g < RT * NG; ++g) {
        auto add = [](double u, double v) { return u + v; };
        if (KS >= 2) acc[g] = lane_pair<8>(acc[g], add);
        if (KS >= 4) acc[g] = lane_pair<4>(acc[g], add);
        part[wave][g][lane] = acc[g];
    }
    __syncthreads();
    if (wave < RT * NG && b < BE && e_mine < E) {
        double s = part[0][wave][lane];               // waves in order
#pragma unroll
        for (int w = 1; w < kMfmaWaves; ++w) s += part[w][wave][lane];
        logits[4 * (wave / NG) + q][e_mine] = s + shift;
    }
    __syncthreads();
    static_assert(4 * RT <= kMfmaWaves, "a wave ranks one token");
    if (wave < 4 * RT && t0 + wave < Tn)
        rank_token<false>(logits[wave], lane, E, k, renorm, t0 + wave, idx_out, w_out, id);
}

template <int RT>
void launch_mfma(const bf16_t* x, const bf16_t* wr, const float* bias, int Tn, int d, int E, int k,
                 int renorm, int32_t* idx, float* w, const int32_t* remap, hipStream_t s) {
    const dim3 grid((Tn + 4 * RT - 1) / (4 * RT)), block(kMfmaWaves * kWave);
#define SPECMOE_ROUTE(NG, KS)                                                                    \
    hipLaunchKernelGGL((route_topk_mfma_kernel<NG, KS, RT>), grid, block, 0, s, x, wr, bias, Tn, \
                       d, E, k, renorm, idx, w, remap)
    if (E <= 4) SPECMOE_ROUTE(1, 4);
    else if (E <= 8) SPECMOE_ROUTE(1, 2);
    else if (E <= 16) SPECMOE_ROUTE(1, 1);
    else if (E <= 32) SPECMOE_ROUTE(2, 1);
    else SPECMOE_ROUTE(4, 1);
#undef SPECMOE_ROUTE
}

template <typename T, bool VEC, int TOK, int EC, int W>
void launch_variant(const T* x, const T* wr, const float* bias, int Tn, int d, int E, int k,
                    int renorm, int32_t* idx, float* w, const int32_t* remap, Then then, hipStream_t s) {
    dim3 grid((Tn + TOK - 1) / TOK), block(kRouteThreads);
    size_t lds = ((size_t)TOK * E + (size_t)(kRouteThreads / kWave) * TOK * EC) * sizeof(double);
    // up to 64 tokens and 64 experts come to one token per workgroup and at most 8 columns per pass (launch_typed)
    if constexpr (TOK == 1 && EC <= 8) {
        if (then.done) {
            hipLaunchKernelGGL((route_topk_kernel<T, VEC, TOK, EC, W, true>), grid, block, lds, s, x, wr, bias, Tn,
                               d, E, k, renorm, idx, w, remap, then);
            return;
        }
    }
    hipLaunchKernelGGL((route_topk_kernel<T, VEC, TOK, EC, W, false>), grid, block, lds, s, x, wr, bias, Tn,
                       d, E, k, renorm, idx, w, remap, then);
}

// Experts per group and pass: the group's share of E rounded up to a power of two, at most 16 / TOK.
// Up to 16 experts 4 groups of 4 waves, beyond that 8 groups of 2: twice the columns per lane, but
// half the sums to exchange over the lanes: 64 x 2048, 64 tokens 12.5 -> 11.3 us, 320 tokens 16.0 ->
// 13.6; 64 x 512 12.1 -> 9.2; 256 x 1024 38.1 -> 27.9 (with the exchanges through LDS).
template <typename T, bool VEC, int TOK, int W>
void launch_by_share(const T* x, const T* wr, const float* bias, int Tn, int d, int E, int k,
                     int renorm, int32_t* idx, float* w, const int32_t* remap, Then then, hipStream_t s) {
    constexpr int EC_MAX = 16 / TOK, G = 16 / W;
    const int share = (E + G - 1) / G;
    if (share <= 1)
        launch_variant<T, VEC, TOK, 1, W>(x, wr, bias, Tn, d, E, k, renorm, idx, w, remap, then, s);
    else if (share <= 2 || EC_MAX == 2)
        launch_variant<T, VEC, TOK, (EC_MAX < 2 ? EC_MAX : 2), W>(x, wr, bias, Tn, d, E, k, renorm, idx, w, remap, then, s);
    else if (share <= 4 || EC_MAX == 4)
        launch_variant<T, VEC, TOK, (EC_MAX < 4 ? EC_MAX : 4), W>(x, wr, bias, Tn, d, E, k, renorm, idx, w, remap, then, s);
    else if (share <= 8 || EC_MAX == 8)
        launch_variant<T, VEC, TOK, (EC_MAX < 8 ? EC_MAX : 8), W>(x, wr, bias, Tn, d, E, k, renorm, idx, w, remap, then, s);
    else
        launch_variant<T, VEC, TOK, EC_MAX, W>(x, wr, bias, Tn, d, E, k, renorm, idx, w, remap, then, s);
}
template <typename T, bool VEC, int TOK>
void launch_by_experts(const T* x, const T* wr, const float* bias, int Tn, int d, int E, int k,
                       int renorm, int32_t* idx, float* w, const int32_t* remap, Then then, hipStream_t s) {
    if (E <= 16)
        launch_by_share<T, VEC, TOK, 4>(x, wr, bias, Tn, d, E, k, renorm, idx, w, remap, then, s);
    else
        launch_by_share<T, VEC, TOK, 2>(x, wr, bias, Tn, d, E, k, renorm, idx, w, remap, then, s);
}

template <typename T, int V>
void launch_typed(const void* x, const void* wr, const float* bias, int Tn, int d, int E, int k,
                  int renorm, int32_t* idx, float* w, const int32_t* remap, Then then, hipStream_t s) {
    const bool vec = (d % V == 0) && ((((uintptr_t)x | (uintptr_t)wr) & 15u) == 0);
    const T* xt = (const T*)x;
    const T* wt = (const T*)wr;
    if (!vec) {
        launch_by_experts<T, false, 1>(xt, wt, bias, Tn, d, E, k, renorm, idx, w, remap, then, s);
        return;
    }
    if (then.done) {                              // kRoutePermuteTokens: the minimum below is one token per workgroup
        launch_by_experts<T, true, 1>(xt, wt, bias, Tn, d, E, k, renorm, idx, w, remap, then, s);
        return;
    }
    // Matrix form: from 1025 tokens on with 8 tokens per workgroup (the vector form then needs a
    // second round of workgroups; 2048 tokens, vector -> matrix: 8 x 4096 13.2 -> 10.6 us, 64 x 2048
    // 39.9 -> 22.8, 16 x 5120 23.1 -> 19.2, 4 x 1024 7.9 -> 6.3), and with more than 16 experts also
    // below, 4 tokens per workgroup: from 513 tokens (64 x 2048, 640 tokens 22.8 -> 18.2; up to 32
    // experts only with rows up to 2048: 20 x 5120, 1000 tokens 16.6 against 17.2), or 257 if rows are
    // short (64 x 512, 320 tokens 15.2 -> 10.4).  Its workgroups take longer than the vector form's, so
    // fewer tokens stay there (64 tokens 8.9 against 15).
    if constexpr (sizeof(T) == 2) {
        if (E <= kWave && Tn > 1024) {
            launch_mfma<2>(xt, wt, bias, Tn, d, E, k, renorm, idx, w, remap, s);
            return;
        }
        if (E <= kWave && E > 16 && (E > 32 || d <= 2048) &&
            (Tn > 512 || (Tn > 256 && d <= 1024))) {
            launch_mfma<1>(xt, wt, bias, Tn, d, E, k, renorm, idx, w, remap, s);
            return;
        }
    }
    // Vector form, tokens per workgroup: every group of waves widens its TOK token chunks and its
    // EC router chunks per pass (passes x EC covers the group's share of the experts), so the busiest CU
    // issues work in proportion to
    //   workgroups per CU x passes x (TOK + EC).
    // More tokens per workgroup share the widened router weights but leave CUs idle while the
    // batch is small: take the minimum, which agreed with the measured order over T, d, E, k.
    int best_tok = 1;
    long long best = -1;
    for (int tok = 1; tok <= 4; tok *= 2) {
        const int ec_max = 16 / tok;
        const int groups = E <= 16 ? 4 : 8;
        int ec = 1;
        while (ec < ec_max && ec * groups < E) ec *= 2;
        const long long passes = (E + groups * ec - 1) / (groups * ec);
        const long long wgs = (Tn + tok - 1) / tok;
        const long long per_cu = (wgs + 255) / 256;
        const long long load = per_cu * passes * (tok + ec);
        if (best < 0 || load < best) { best = load; best_tok = tok; }
    }
    if (best_tok == 4) launch_by_experts<T, true, 4>(xt, wt, bias, Tn, d, E, k, renorm, idx, w, remap, then, s);
    else if (best_tok == 2) launch_by_experts<T, true, 2>(xt, wt, bias, Tn, d, E, k, renorm, idx, w, remap, then, s);
    else launch_by_experts<T, true, 1>(xt, wt, bias, Tn, d, E, k, renorm, idx, w, remap, then, s);
}

}  // namespace

hipError_t launch_route_topk(const void* x, const void* wr, const float* bias, int T, int d,
                             int E, int k, int renorm, int dtype, int32_t* idx, float* w,
                             hipStream_t s, const int32_t* remap) {
    if (T == 0) return hipSuccess;
    const Then then{nullptr, nullptr, nullptr, nullptr};
    if (dtype == 0) launch_typed<float, 4>(x, wr, bias, T, d, E, k, renorm, idx, w, remap, then, s);
    else launch_typed<bf16_t, 8>(x, wr, bias, T, d, E, k, renorm, idx, w, remap, then, s);
    return hipGetLastError();
}

hipError_t launch_route_permute(const void* x, const void* wr, const float* bias, int T, int d, int E, int k,
                                int renorm, int dtype, const int32_t* remap, int32_t* idx, float* w,
                                int32_t* offsets, int32_t* row_src, int32_t* row_of, uint32_t* done,
                                hipStream_t s) {
    if (T < 1 || T > kRoutePermuteTokens || E > kWave) return hipErrorInvalidValue;
    const Then then{done, offsets, row_src, row_of};
    if (dtype == 0) launch_typed<float, 4>(x, wr, bias, T, d, E, k, renorm, idx, w, remap, then, s);
    else launch_typed<bf16_t, 8>(x, wr, bias, T, d, E, k, renorm, idx, w, remap, then, s);
    return hipGetLastError();
}

}  // namespace specmoe
