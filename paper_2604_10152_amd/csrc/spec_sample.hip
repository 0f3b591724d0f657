// Verification helpers beyond the greedy rule.
//
// spec_accept_sample_kernel — sampling-based verification (SpecMoE Sec. 6.3: Mixtral-8x7B and
//   Llama-4-Scout are verified with the sampling rule of the speculative-decoding method the
//   paper cites, temperature 1).  Draft token x at position i is kept when
//   u < min(1, pt(x)/pd(x)); at the first rejection the token is redrawn from the normalised
//   positive part of (pt - pd) and the rest is dropped; if every draft is kept one more token
//   is drawn from the target's distribution at position gamma.  The caller supplies the
//   uniforms, so the result is a deterministic function of the inputs.
//   Decisions are taken in fp64 on the fp32 inputs: u*pd and pt-pd are then exact, so the keep
//   test has no rounding at all; the inverse-CDF draw compares fp64 running sums with u*total.
// greedy_tokens_kernel — the greedy head (Sec. 4 "SpecMoE configuration"): id of the largest
//   logit per row, lower id on ties.
// active_expert_bytes_kernel — parameter bytes of the experts that received at least one row
//   (the per-block migration volume the paper's Fig. 3(b) plots; here: the HBM read volume).
#include "common.h"

namespace specmoe {
namespace {

constexpr int kSampleThreads = 1024;  // 16 waves: enough loads in flight for one CU per sequence
constexpr int kSampleWaves = kSampleThreads / kWave;
constexpr int kTileIds = kWave * 4;          // ids one wave covers per step: 4 per lane (16 bytes)
constexpr int kBurst = 8;                    // tiles a wave requests at once
constexpr int kMaxLdsTiles = 2048;           // tile sums kept in LDS (V <= 524288); beyond that
                                             // the tiles are re-summed from memory

// First id of a tile.  The last burst of a wave asks for tiles beyond the row (load_tile answers with
// zeros), whose ids may exceed the int range at the largest vocabularies.
constexpr __host__ __device__ uint32_t tile_id(int tile) { return (uint32_t)tile * kTileIds; }
static_assert(tile_id((INT32_MAX - 1) / kTileIds + (kBurst - 1) * kSampleWaves) >= INT32_MAX,
              "the tiles of the last burst beyond the row must not wrap around to its start");

// inclusive wave scan (fp64)
__device__ __forceinline__ double wave_scan_incl(double v, int lane) {
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const double o = __shfl_up(v, off, kWave);
        if (lane >= off) v += o;
    }
    return v;
}

// One workgroup per sequence.  The draw needs the smallest id whose running weight exceeds
// u * total.  Wave w of the 16 owns the 256-id tiles w, w+16, ...: it requests kBurst of them
// (16-byte loads) before it adds anything up - 128 KB in flight per CU, at V = 32000 the whole
// row - and reduces the kBurst fp64 sums over its lanes with one transposing butterfly.  The tile
// sums meet in LDS; a wave scan over them, 64 tiles at a time, gives the total and then the tile
// where the threshold is crossed, and one wave scans that tile.  Only the order of the fp64
// additions differs from a sequential running sum.  B = 256, gamma = 7, V = 32000: 32 us with one
// tile at a time and a serial walk over the tile sums, 15.4 like this; HBM is the bound (2 V 4 bytes per
// sequence, after two dependent round trips for the first rejection).
__global__ __launch_bounds__(kSampleThreads) void spec_accept_sample_kernel(
    const int32_t* __restrict__ draft, const float* __restrict__ p_draft,
    const float* __restrict__ p_target, const float* __restrict__ u_accept,
    const float* __restrict__ u_sample, int gamma, int V, int32_t* __restrict__ accept_len,
    int32_t* __restrict__ out_tokens) {
    const int b = blockIdx.x, tid = threadIdx.x;
    const int lane = tid % kWave, wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    __shared__ int n_sh;
    __shared__ double tile_sum[kMaxLdsTiles];
    const int32_t* dr = draft + (size_t)b * gamma;
    const float* pd = p_draft + (size_t)b * gamma * V;
    const float* pt = p_target + (size_t)b * (gamma + 1) * V;

    // ---- first rejected position (gamma <= 64: one lane per draft token, first wave)
    if (wave == 0) {
        bool reject = false;
        if (lane < gamma) {
            const int x = dr[lane];
            if (x < 0 || x >= V) {
                reject = true;                      // an id outside the vocabulary is never kept
            } else {
                const double lhs = (double)u_accept[(size_t)b * gamma + lane] *
                                   (double)pd[(size_t)lane * V + x];
                reject = !(lhs < (double)pt[(size_t)lane * V + x]);
            }
        }
        const unsigned long long m = __ballot(reject);
        if (lane == 0) n_sh = m ? __ffsll((long long)m) - 1 : gamma;
    }
    const double u_draw = (double)u_sample[b];
    __syncthreads();
    const int n = __builtin_amdgcn_readfirstlane(n_sh);
    const float* ptn = pt + (size_t)n * V;
    const float* pdn = n < gamma ? pd + (size_t)n * V : nullptr;
    const bool vec = (V % 4 == 0) && ((((uintptr_t)p_draft | (uintptr_t)p_target) & 15u) == 0);
    const int n_tiles = (V - 1) / kTileIds + 1;

    // this lane's 4 probabilities of tile `tile` (0 beyond V) under both models; q = 0 when
    // drawing from pt
    auto load_tile = [&](int tile, bool resid, floatx4& t, floatx4& q) __attribute__((always_inline)) {
        const uint32_t v0 = tile_id(tile) + lane * 4, end = V;
        t = floatx4{0.f, 0.f, 0.f, 0.f};
        q = floatx4{0.f, 0.f, 0.f, 0.f};
        if (vec) {                                  // V % 4 == 0: all four ids or none
            if (v0 < end) {
                t = *reinterpret_cast<const floatx4*>(ptn + v0);
                if (resid) q = *reinterpret_cast<const floatx4*>(pdn + v0);
            }
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (v0 + i < end) {
                    t[i] = ptn[v0 + i];
                    if (resid) q[i] = pdn[v0 + i];
                }
        }
    };
    auto weight = [](float t, float q) -> double {
        const double r = (double)t - (double)q;
        return r > 0.0 ? r : 0.0;
    };
    auto tile_total = [&](int tile, bool resid) -> double {      // whole wave, same in every lane
        floatx4 t, q;
        load_tile(tile, resid, t, q);
        return wave_sum((weight(t[0], q[0]) + weight(t[1], q[1])) +
                        (weight(t[2], q[2]) + weight(t[3], q[3])));
    };
    auto sum_tiles = [&](bool resid) {
        if (n_tiles <= kSampleWaves) {              // at most one tile per wave
            if (wave < n_tiles) {
                const double s = tile_total(wave, resid);
                if (lane == 0) tile_sum[wave] = s;
            }
            __syncthreads();
            return;
        }
        for (int t0 = wave; t0 < n_tiles; t0 += kSampleWaves * kBurst) {
            floatx4 t[kBurst], q[kBurst];
#pragma unroll
            for (int i = 0; i < kBurst; ++i) load_tile(t0 + i * kSampleWaves, resid, t[i], q[i]);
            __builtin_amdgcn_sched_barrier(0);
            double s[kBurst];
#pragma unroll
            for (int i = 0; i < kBurst; ++i)
                s[i] = (weight(t[i][0], q[i][0]) + weight(t[i][1], q[i][1])) +
                       (weight(t[i][2], q[i][2]) + weight(t[i][3], q[i][3]));
            TransposeReduce<kBurst, kWave / 2>::run(s, lane);
            const int tile = t0 + lane / (kWave / kBurst) * kSampleWaves;
            if (lane % (kWave / kBurst) == 0 && tile < n_tiles && tile < kMaxLdsTiles)
                tile_sum[tile] = s[0];
        }
        __syncthreads();
    };
    // inclusive running sums of tiles c0 .. c0 + 63, tile c0 + lane in each lane (s: its own sum)
    auto scan_chunk = [&](int c0, bool resid, double& s) -> double {
        s = 0.0;
        if (c0 < kMaxLdsTiles) {                    // kMaxLdsTiles is a multiple of 64
            if (c0 + lane < n_tiles) s = tile_sum[c0 + lane];
        } else {
            for (int i = 0; i < kWave && c0 + i < n_tiles; ++i) {
                const double v = tile_total(c0 + i, resid);
                if (lane == i) s = v;
            }
        }
        if (n_tiles > kSampleWaves) return wave_scan_incl(s, lane);
        // a small vocabulary: as many steps as it has tiles (one: none; the scan of 64 lanes is a
        // sixth of the kernel, V = 50: 3.6 us against 4.1).  Lanes beyond n_tiles hold no sum.
        double v = s;
        for (int off = 1; off < n_tiles; off <<= 1) {
            const double o = __shfl_up(v, off, kWave);
            if (lane >= off) v += o;
        }
        return v;
    };
    const int last = n_tiles > kSampleWaves ? kWave - 1 : n_tiles - 1;   // lane with a chunk's sum
    auto total_of = [&](bool resid) -> double {     // every wave for itself, same result
        double tot = 0.0, s;
        for (int c0 = 0; c0 < n_tiles; c0 += kWave)
            tot += __shfl(scan_chunk(c0, resid, s), last, kWave);
        return tot;
    };
    bool resid = pdn != nullptr;
    sum_tiles(resid);
    double total = total_of(resid);
    if (resid && !(total > 0.0)) {                   // pt == pd everywhere: draw from pt
        __syncthreads();
        resid = false;
        sum_tiles(false);
        total = total_of(false);
    }
    if (wave != 0) return;
    const double thr = u_draw * total;
    int tok = V - 1;
    double base = 0.0;                               // sum of the chunks in front
    for (int c0 = 0; c0 < n_tiles; c0 += kWave) {
        // Every lane of a scan adds up in an order of its own, so over tiles that hold nothing the
        // running sums still move by a rounding and may pass the threshold there: only a tile
        // (and below, an id) with weight of its own can be the one that crosses it.  With u < 1
        // one always does: the sums agree to 1e-14, u * total lies at least 2^-24 below the total.
        double own;
        const double incl = scan_chunk(c0, resid, own);
        const unsigned long long over = __ballot(own > 0.0 && base + incl > thr);
        if (!over) {
            base += __shfl(incl, last, kWave);
            continue;
        }
        const int at = __ffsll((long long)over) - 1;
        const int tile = c0 + at;
        const double before = at > 0 ? base + __shfl(incl, at - 1, kWave) : base;
        floatx4 t, q;
        load_tile(tile, resid, t, q);
        const double w0 = weight(t[0], q[0]), w1 = weight(t[1], q[1]), w2 = weight(t[2], q[2]),
                     w3 = weight(t[3], q[3]);
        const double c1 = w0, c2 = c1 + w1, c3 = c2 + w2, c4 = c3 + w3;
        const double excl = before + (wave_scan_incl(c4, lane) - c4);
        int first = 4;
        if (w3 > 0.0 && excl + c4 > thr) first = 3;
        if (w2 > 0.0 && excl + c3 > thr) first = 2;
        if (w1 > 0.0 && excl + c2 > thr) first = 1;
        if (w0 > 0.0 && excl + c1 > thr) first = 0;
        const unsigned long long hit = __ballot(first < 4);
        const unsigned long long pos = __ballot(c4 > 0.0);
        if (hit) {
            const int src = __ffsll((long long)hit) - 1;
            tok = tile * kTileIds + src * 4 + __shfl(first, src, kWave);
        } else if (pos) {
            // rounding: the tile's running sums stop a hair below the threshold;
            // take its last id with a positive weight
            const int src = 63 - __clzll((long long)pos);
            const int last = w3 > 0.0 ? 3 : (w2 > 0.0 ? 2 : (w1 > 0.0 ? 1 : 0));
            tok = tile * kTileIds + src * 4 + __shfl(last, src, kWave);
        }
        break;
    }
    int32_t* ot = out_tokens + (size_t)b * (gamma + 1);
    for (int i = lane; i <= gamma; i += kWave) ot[i] = i < n ? dr[i] : (i == n ? tok : -1);
    if (lane == 0) accept_len[b] = n + 1;
}

template <typename T> struct Row;
template <> struct Row<float> {
    static constexpr int N = 4;
    __device__ static float one(const float* p) { return *p; }
    __device__ static float at(const U128& v, int i) { return __uint_as_float(v[i]); }
};
template <> struct Row<bf16_t> {
    static constexpr int N = 8;
    __device__ static float one(const bf16_t* p) {
        return __uint_as_float((uint32_t)*reinterpret_cast<const uint16_t*>(p) << 16);
    }
    __device__ static float at(const U128& v, int i) {
        return __uint_as_float(i & 1 ? v[i >> 1] & 0xffff0000u : v[i >> 1] << 16);
    }
};

constexpr int kRowBurst = 4;          // chunks requested together where few rows leave CUs short of loads

// One workgroup per row.  Thread t visits its ids in ascending order (16-byte chunks t, t+256,
// ... when the row allows it) and keeps the first maximum it sees; the reduction prefers the
// larger value, then the lower id.  Logits must not contain NaN.  STREAM: loads with the non-temporal hint.
template <typename T, bool VEC, int BURST, bool STREAM>
__global__ __launch_bounds__(256) void greedy_tokens_kernel(const T* __restrict__ logits, int V,
                                                            int32_t* __restrict__ tokens) {
    const T* row = logits + (size_t)blockIdx.x * V;
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    float bv = 0.f;
    int bi = -1;
    if (VEC) {
        // BURST chunks are requested before the first is looked at; the ones beyond the row
        // repeat its last chunk, whose ids cannot win again (only a larger value replaces bv)
        constexpr int N = Row<T>::N;
        const int chunks = V / N;
        auto load = [](const U128* p) { return STREAM ? __builtin_nontemporal_load(p) : *p; };
        auto at = [&](int i, int c0) -> int { return i == 0 ? c0 : min(c0 + i * 256, chunks - 1); };
        for (int c0 = tid; c0 < chunks; c0 += 256 * BURST) {
            U128 raw[BURST];
#pragma unroll
            for (int i = 0; i < BURST; ++i)
                raw[i] = load(reinterpret_cast<const U128*>(row + (size_t)at(i, c0) * N));
            if (BURST > 1) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < BURST; ++i) {
                const int c = at(i, c0);
#pragma unroll
                for (int q = 0; q < N; ++q) {
                    const float x = Row<T>::at(raw[i], q);
                    if (bi < 0 || x > bv) { bv = x; bi = c * N + q; }
                }
            }
        }
    } else {
        for (int v = tid; v < V; v += 256) {
            const float x = Row<T>::one(row + v);
            if (bi < 0 || x > bv) { bv = x; bi = v; }
        }
    }
    auto take = [&](float ov, int oi) {
        if (oi >= 0 && (bi < 0 || ov > bv || (ov == bv && oi < bi))) { bv = ov; bi = oi; }
    };
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1)
        take(__shfl_xor(bv, off, kWave), __shfl_xor(bi, off, kWave));
    __shared__ float sv[4];
    __shared__ int si[4];
    if (lane == 0) { sv[wave] = bv; si[wave] = bi; }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < 4; ++w) take(sv[w], si[w]);
        tokens[blockIdx.x] = bi;
    }
}

__global__ __launch_bounds__(kWave) void active_expert_bytes_kernel(
    const int32_t* __restrict__ offsets, int E, long long bytes_per_expert,
    long long* __restrict__ out) {
    int n = 0;
    for (int e = threadIdx.x; e < E; e += kWave) n += (offsets[e + 1] - offsets[e]) > 0;
    n = wave_sum(n);
    if (threadIdx.x == 0) out[0] = (long long)n * bytes_per_expert;
}

}  // namespace

hipError_t launch_spec_accept_sample(const int32_t* draft, const float* p_draft,
                                     const float* p_target, const float* u_accept,
                                     const float* u_sample, int B, int gamma, int V,
                                     int32_t* accept_len, int32_t* out_tokens, hipStream_t s) {
    if (B == 0) return hipSuccess;
    hipLaunchKernelGGL(spec_accept_sample_kernel, dim3(B), dim3(kSampleThreads), 0, s, draft,
                       p_draft, p_target, u_accept, u_sample, gamma, V, accept_len, out_tokens);
    return hipGetLastError();
}

template <typename T>
static void launch_greedy_typed(const void* logits, int R, int V, int32_t* tokens, hipStream_t s) {
    const bool vec = V % Row<T>::N == 0 && ((uintptr_t)logits & 15u) == 0 &&
                     ((size_t)V * sizeof(T)) % 16 == 0;
    // Few rows (up to 640) of at least four chunks per thread: one thread's chunks are requested
    // together, 512 x 32000 bf16 10.5 -> 7.2 us, 640 rows 11.0 -> 8.8.  Up to 1024 rows only where they are
    // long (1024 x 128256 47.4 -> 43.2; 1024 x 32000 12.8 -> 13.0, fp32 21.3 -> 22.1).  More rows keep
    // enough loads in flight by themselves (2048 x 32000 bf16: 22.3 us = 5.9 TB/s, 23.0 with the burst),
    // and shorter rows have nothing to request ahead (2048 x 1000: 4.2 us, 5.3 with it).
    const int per_thread = V / Row<T>::N / 256;
    const bool burst = vec && per_thread >= kRowBurst && (R <= 640 || (R <= 1024 && per_thread >= 48));
    // Non-temporal loads for what the memory-side cache (256 MiB) cannot hold, and from 100 MB on for bf16, which
    // reaches this kernel straight from the head's product; fp32 mostly comes from a cast, which leaves it in that cache.
    // This kernel alone, us, without / with the hint, by what wrote the logits:
    //             MB   product      cast or copy  scaling      nothing since a copy of 1 GB
    //   bf16     102   24.3 / 23.1  21.8 / 26.2   20.1 / 21.6  33.4 / 22.2
    //            131   29.0 / 27.0  25.2 / 28.5   24.0 / 25.4  41.0 / 26.1
    //            205   41.2 / 38.8  43.9 / 39.5   44.1 / 41.2  59.4 / 38.4
    //   fp32     166   35.2 / 28.8  39.3 / 44.4   36.0 / 39.5  50.2 / 31.4
    //            262   58.4 / 42.5  47.6 / 50.0   53.0 / 54.6  75.9 / 43.6
    //            269   70.6 / 49.9  62.4 / 58.8   68.0 / 63.1
    //            352   84.7 / 62.2  102 / 71      98 / 72
    const long long bytes = (long long)R * V * (long long)sizeof(T);
    const bool stream = vec && !burst && (bytes > (256ll << 20) || (sizeof(T) == 2 && bytes >= 100000000ll));
    if (stream)
        hipLaunchKernelGGL((greedy_tokens_kernel<T, true, 1, true>), dim3(R), dim3(256), 0, s,
                           (const T*)logits, V, tokens);
    else if (burst)
        hipLaunchKernelGGL((greedy_tokens_kernel<T, true, kRowBurst, false>), dim3(R), dim3(256), 0, s,
                           (const T*)logits, V, tokens);
    else if (vec)
        hipLaunchKernelGGL((greedy_tokens_kernel<T, true, 1, false>), dim3(R), dim3(256), 0, s,
                           (const T*)logits, V, tokens);
    else
        hipLaunchKernelGGL((greedy_tokens_kernel<T, false, 1, false>), dim3(R), dim3(256), 0, s,
                           (const T*)logits, V, tokens);
}

hipError_t launch_greedy_tokens(const void* logits, int R, int V, int dtype, int32_t* tokens,
                                hipStream_t s) {
    if (R == 0) return hipSuccess;
    if (dtype == 0) launch_greedy_typed<float>(logits, R, V, tokens, s);
    else launch_greedy_typed<bf16_t>(logits, R, V, tokens, s);
    return hipGetLastError();
}

hipError_t launch_active_expert_bytes(const int32_t* offsets, int E, long long bytes_per_expert,
                                      long long* out, hipStream_t s) {
    hipLaunchKernelGGL(active_expert_bytes_kernel, dim3(1), dim3(kWave), 0, s, offsets, E,
                       bytes_per_expert, out);
    return hipGetLastError();
}

}  // namespace specmoe
