// Shared device helpers and launcher declarations of the gfx950 MoE verify-layer library.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace specmoe {

constexpr int kWave = 64;           // CDNA wavefront width
constexpr int kXcds = 8;            // MI355X: 8 accelerator dies, workgroups dealt round-robin
constexpr int kCus = 256;           // compute units of all dies

typedef __bf16 bf16_t;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

typedef uint32_t U128 __attribute__((ext_vector_type(4)));   // one 16-byte register quad

__device__ __forceinline__ float bf16_bits_to_float(uint32_t bits16) {
    return __uint_as_float(bits16 << 16);
}
__device__ __forceinline__ float load_as_float(const float* p) { return *p; }
__device__ __forceinline__ float load_as_float(const bf16_t* p) { return (float)(*p); }
__device__ __forceinline__ void store_from_float(float* p, float v) { *p = v; }
__device__ __forceinline__ void store_from_float(bf16_t* p, float v) { *p = (bf16_t)v; }

// Two floats -> packed bf16 pair (round to nearest even), low half = a.
__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    bf16x2 v = {(bf16_t)a, (bf16_t)b};
    return __builtin_bit_cast(uint32_t, v);
}

// ---- exchanges between the lanes of a wave, in registers: a few cycles each, where __shfl goes through
// the LDS crossbar (over 100 cycles a step, six steps in a row for a sum or a scan).  Every workgroup of
// an expert GEMM starts with a sum and two scans (tile_map.h): gate/up 64 experts x 2048 x 1408, 64 tokens
// 126.4 -> 122.7 us, 1285 tokens uniform 165.8 -> 162.8; packed layer of 320 tokens 212.8 -> 208.6.
// the value of lane ^ BIT (BIT = 1, 2, 4 or 8)
template <int BIT>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v) {
    static_assert(BIT == 1 || BIT == 2 || BIT == 4 || BIT == 8, "inside a row of 16 lanes");
    const int i = (int)v;
    if constexpr (BIT == 1) return (uint32_t)__builtin_amdgcn_update_dpp(i, i, 0xB1, 0xf, 0xf, false);
    if constexpr (BIT == 2) return (uint32_t)__builtin_amdgcn_update_dpp(i, i, 0x4E, 0xf, 0xf, false);
    if constexpr (BIT == 8) return (uint32_t)__builtin_amdgcn_update_dpp(i, i, 0x128, 0xf, 0xf, false);
    const int low = __builtin_amdgcn_update_dpp(i, i, 0x104, 0xf, 0x5, false);     // lanes with bit 2 clear: lane + 4
    return (uint32_t)__builtin_amdgcn_update_dpp(low, i, 0x114, 0xf, 0xa, false);  // the others: lane - 4
}
// BIT = 16 or 32: lanes with the bit clear keep a and receive the partner's a in b, lanes with it set
// receive the partner's b in a and keep b
template <int BIT>
__device__ __forceinline__ void lane_swap(uint32_t& a, uint32_t& b) {
    static_assert(BIT == 16 || BIT == 32, "whole rows of 16 lanes");
    typedef uint32_t Pair __attribute__((ext_vector_type(2)));
    Pair r;
    if constexpr (BIT == 32) r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    else r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}
// f(own, value of lane ^ BIT) for a commutative f
template <int BIT, typename T, typename F>
__device__ __forceinline__ T lane_pair(T v, F f) {
    constexpr int N = sizeof(T) / 4;
    struct Words { uint32_t w[N]; };
    Words a = __builtin_bit_cast(Words, v), b = a;
    if constexpr (BIT >= 16) {
#pragma unroll
        for (int i = 0; i < N; ++i) lane_swap<BIT>(a.w[i], b.w[i]);
    } else {
#pragma unroll
        for (int i = 0; i < N; ++i) b.w[i] = lane_xor<BIT>(a.w[i]);
    }
    return f(__builtin_bit_cast(T, a), __builtin_bit_cast(T, b));
}
// f over all lanes, in every lane; pairs at distance 32 first
template <typename T, typename F>
__device__ __forceinline__ T wave_all(T v, F f) {
    v = lane_pair<32>(v, f);
    v = lane_pair<16>(v, f);
    v = lane_pair<8>(v, f);
    v = lane_pair<4>(v, f);
    v = lane_pair<2>(v, f);
    return lane_pair<1>(v, f);
}
template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
    return wave_all(v, [](T a, T b) { return a + b; });
}
__device__ __forceinline__ double wave_max(double v) {      // of the values that are not NaN
    return wave_all(v, [](double a, double b) { return fmax(a, b); });
}
// inclusive running sum over the lanes
__device__ __forceinline__ int wave_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);     // inside rows of 16
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);     // row 0 into 1, 2 into 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);     // rows 0 and 1 into 2 and 3
    return v;
}

// Transposing butterfly over the 64 lanes of a wave: v[0..CNT) in every lane -> v[0] = total of
// value (lane * CNT0 / 64) where CNT0 is the count at the first step.
template <int CNT, int BIT>
struct TransposeReduce {
    __device__ __forceinline__ static void run(double* v, int lane) {
        auto add = [](double a, double b) { return a + b; };
        if constexpr (CNT > 1) {
            constexpr int H = CNT / 2;
            const bool up = (lane & BIT) != 0;
            struct Words { uint32_t w[2]; };
#pragma unroll
            for (int i = 0; i < H; ++i) {
                if constexpr (BIT >= 16) {
                    Words a = __builtin_bit_cast(Words, v[i]), b = __builtin_bit_cast(Words, v[i + H]);
                    lane_swap<BIT>(a.w[0], b.w[0]);
                    lane_swap<BIT>(a.w[1], b.w[1]);
                    v[i] = __builtin_bit_cast(double, a) + __builtin_bit_cast(double, b);
                } else {
                    Words send = __builtin_bit_cast(Words, up ? v[i] : v[i + H]);
                    const double keep = up ? v[i + H] : v[i];
                    send.w[0] = lane_xor<BIT>(send.w[0]);
                    send.w[1] = lane_xor<BIT>(send.w[1]);
                    v[i] = keep + __builtin_bit_cast(double, send);
                }
            }
            if constexpr (BIT > 1) TransposeReduce<H, BIT / 2>::run(v, lane);
        } else {
            v[0] = lane_pair<BIT>(v[0], add);
            if constexpr (BIT > 1) TransposeReduce<1, BIT / 2>::run(v, lane);
        }
    }
};

__device__ __forceinline__ float silu_f32(float z) { return z / (1.0f + __expf(-z)); }

// Whether the 256-wide tiles (wide outputs each) of a batch leave much of the chip idle: a tile
// takes a whole CU, and with m-tiles of up to 320 rows (estimated from the average rows per
// expert plus 15 % for the spread) there are at most 128 of them, or 64 if an expert needs
// several.  The measurements are at the rules that use it.
struct WideTiles {
    long long m, tiles;         // m-tiles per expert, tiles in all
    WideTiles(int n_rows, int E, int N, int wide)
        : m((115ll * n_rows + 32000ll * E - 1) / (32000ll * E)),
          tiles(E * m * ((N + wide - 1) / wide)) {}
    bool few() const { return tiles <= (m <= 1 ? 128 : 64); }
};
inline bool few_wide_tiles(int n_rows, int E, int N, int wide) {
    return WideTiles(n_rows, E, N, wide).few();
}

// Whether the expert GEMMs store with the non-temporal hint.  What they write is read by the next kernel, from any die,
// and until then every line of it takes the place of operands in the L2.  Measured, packed operands, us, without / with the hint
// (bytes written): gate/up 8 x 4096 x 14336, 175 rows each (40 MB) 377 / 359, 83 rows (19 MB) 339 / 334, 64 x 2048 x 1408, 120
// rows (22 MB) 171 / 165; down, the same, 60 rows (16 MB) 71 / 66.  A small output stays in the L2: gate/up, 6 rows (1 MB) 30.7 / 31.1, 30
// rows (5 MB) 109.5 / 110.4; down, 6 rows (1.6 MB) 42.0 / 42.7, but 30 rows (8 MB) 62.2 / 61.0.  Its price in row-major outputs: an
// instruction stores half a line of each of 16 rows, and the halves leave the L2 by themselves (8 x 14336 x 4096, 512 rows each, y
// of 33.6 MB written as 48; 64 x 1408 x 2048, 190 rows 125 us against 119 without the hint, but gate/up 2048 x 1408, 60 rows 150
// against 158, 120 rows 153 / 164).
inline bool streams_output(int n_rows, int N) { return (long long)n_rows * N * 2 >= (6ll << 20); }

// ---- launchers (host side, defined in the .hip files) -------------------------------
hipError_t launch_route_topk(const void* x, const void* wr, const float* bias, int T, int d,
                             int E, int k, int renorm, int dtype, int32_t* idx, float* w,
                             hipStream_t s, const int32_t* remap = nullptr);
// Router and index phase of the permutation in one launch, done: specmoe.h.  While the router's workgroups are few: they
// count one after the other, and the last one permutes while the others' CUs are idle.  Kernels, us, two / one: 80
// tokens, 2 of 8 5.2 + 5.0 / 7.1; 64 tokens, 6 of 64 8.5 + 4.5 / 11.8; 16 tokens in fp32 4.1 + 2.5 / 6.6; 320 tokens, 6 of 64 11.5 + 4.9 /
// 16.8.  Layers on the same buffers: 16 tokens, 256 x 512 in fp32 22.2 / 20.0, 1 token 24.9 / 24.6, 16 tokens 4096 x 14336 138.7 /
// 137.8; from 80 tokens on level (80 tokens 468.8 / 469.1, 128 tokens 64 x 2048 x 1408 162.8 / 162.9).
constexpr int kRoutePermuteTokens = 64;
hipError_t launch_route_permute(const void* x, const void* wr, const float* bias, int T, int d, int E, int k,
                                int renorm, int dtype, const int32_t* remap, int32_t* idx, float* w,
                                int32_t* offsets, int32_t* row_src, int32_t* row_of, uint32_t* done,
                                hipStream_t s);
// speculation phase (affinity.hip, draft_route.hip)
size_t affinity_workspace_bytes(int E);
hipError_t launch_affinity_table(const void* wg, const void* wu, const void* wd, int E, int d,
                                 int f, int dtype, float* table, void* workspace, hipStream_t s);
hipError_t launch_nearest_draft(const float* affinity, int E, const int32_t* draft_ids,
                                int n_draft, int32_t* remap, hipStream_t s);
// sampling-based acceptance, greedy head, active-expert volume (spec_sample.hip)
hipError_t launch_spec_accept_sample(const int32_t* draft, const float* p_draft,
                                     const float* p_target, const float* u_accept,
                                     const float* u_sample, int B, int gamma, int V,
                                     int32_t* accept_len, int32_t* out_tokens, hipStream_t s);
hipError_t launch_greedy_tokens(const void* logits, int R, int V, int dtype, int32_t* tokens,
                                hipStream_t s);
hipError_t launch_active_expert_bytes(const int32_t* offsets, int E, long long bytes_per_expert,
                                      long long* out, hipStream_t s);
hipError_t launch_permute(const void* x, const int32_t* idx, int T, int d, int E, int k,
                          int dtype, void* x_perm, int32_t* offsets, int32_t* row_src,
                          int32_t* row_of, hipStream_t s);
hipError_t launch_expert_up_f32(const float* x_perm, const int32_t* offsets, const float* wg,
                                const float* wu, int n_rows, int d, int f, int E, float* h,
                                hipStream_t s, const int32_t* row_src = nullptr, int topk = 1);
hipError_t launch_expert_down_f32(const float* h, const int32_t* offsets, const float* wd,
                                  int n_rows, int d, int f, int E, float* y, hipStream_t s);
hipError_t launch_expert_up_bf16(const bf16_t* x_perm, const int32_t* offsets, const bf16_t* wg,
                                 const bf16_t* wu, int n_rows, int d, int f, int E, bf16_t* h,
                                 hipStream_t s, const int32_t* row_src = nullptr, int topk = 1);
hipError_t launch_expert_down_bf16(const bf16_t* h, const int32_t* offsets, const bf16_t* wd,
                                   int n_rows, int d, int f, int E, bf16_t* y, hipStream_t s);
hipError_t launch_expert_up_bf16_large16(const bf16_t* x_perm, const int32_t* offsets,
                                         const bf16_t* wg, const bf16_t* wu, int n_rows, int d,
                                         int f, int E, bf16_t* h, hipStream_t s,
    const int32_t* row_src, int topk);
hipError_t launch_expert_down_bf16_large16(const bf16_t* h, const int32_t* offsets,
                                           const bf16_t* wd, int n_rows, int d, int f, int E,
                                           bf16_t* y, hipStream_t s);
hipError_t launch_expert_up_bf16_packed(const bf16_t* x, const int32_t* offsets,
                                        const bf16_t* wg_packed, const bf16_t* wu_packed,
                                        int n_rows, int d, int f, int E, bf16_t* h_packed,
                                        hipStream_t s, const int32_t* row_src, int topk);
hipError_t launch_expert_down_bf16_packed(const bf16_t* h_packed, const int32_t* offsets,
                                          const bf16_t* wd_packed, int n_rows, int d, int f,
                                          int E, bf16_t* y, hipStream_t s);
hipError_t launch_expert_up_bf16_packed_x(const bf16_t* x_packed, const int32_t* offsets,
                                          const bf16_t* wg_packed, const bf16_t* wu_packed,
                                          int n_rows, int d, int f, int E, bf16_t* h,
                                          bool h_row_major, hipStream_t s);
hipError_t launch_gather_pack_rows(const bf16_t* x, const int32_t* row_src, int topk,
                                   const int32_t* offsets, int n_rows, int E, int K,
                                   bf16_t* dst, hipStream_t s);
hipError_t launch_pack_tiles(const bf16_t* src, long long rows, int K, bf16_t* dst, hipStream_t s);
hipError_t launch_expert_up_bf16_ring_or_mid(const bf16_t* x_perm, const int32_t* offsets,
                                             const bf16_t* wg, const bf16_t* wu, int n_rows, int d,
                                             int f, int E, bf16_t* h, hipStream_t s,
                                             const int32_t* row_src, int topk);
hipError_t launch_expert_down_bf16_small(const bf16_t* h, const int32_t* offsets,
                                         const bf16_t* wd, int n_rows, int d, int f, int E,
                                         bf16_t* y, hipStream_t s);
hipError_t launch_expert_up_bf16_mid(const bf16_t* x_perm, const int32_t* offsets,
                                     const bf16_t* wg, const bf16_t* wu, int n_rows, int d, int f,
                                     int E, bf16_t* h, hipStream_t s, const int32_t* row_src,
                                     int topk);
hipError_t launch_expert_down_bf16_mid(const bf16_t* h, const int32_t* offsets, const bf16_t* wd,
                                       int n_rows, int d, int f, int E, bf16_t* y, hipStream_t s);
hipError_t launch_expert_down_bf16_short(const bf16_t* h, const int32_t* offsets, const bf16_t* wd, int n_rows, int d,
                                         int f, int E, bf16_t* y, hipStream_t s);
hipError_t launch_combine(const void* y_perm, const int32_t* row_of, const float* w,
                          const void* residual, int T, int d, int k, int dtype, void* out,
                          hipStream_t s);
hipError_t launch_rmsnorm(const void* x, const void* gain, int T, int d, float eps, int dtype,
                          void* out, hipStream_t s);
hipError_t launch_hot_experts(const int32_t* offsets, int E, int n, int32_t* hot_ids,
                              int32_t* hot_counts, hipStream_t s);
hipError_t launch_spec_accept(const int32_t* draft, const int32_t* target, int B, int gamma,
                              int32_t* accept_len, int32_t* out_tokens, hipStream_t s);

}  // namespace specmoe
