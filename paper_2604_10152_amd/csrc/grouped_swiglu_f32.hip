// Experts in fp32 mode: grouped SwiGLU FFN in fp32 throughout (v_mfma_f32_16x16x4_f32: fp32
// operands, products and sums; no reduced precision).  (SpecMoE Sec. 2.1: every expert is an
// FFN-sized block; only rows routed to an expert are multiplied with its weights.)
//
// This mode exists for the 1e-5 parity configuration; any d_model / d_ff works.  Its matrices are
// small (an expert of the 16-token configuration is 1.5 MB), so a call is bound by latency: the
// operands go from memory straight into the registers the matrix instruction reads (a lane feeds
// row l % 16 and contraction element l / 16; it loads 16 bytes = its element of four
// instructions, the contraction may be taken in any order), with no LDS or barrier in front, and
// while there are few tiles the four waves of a workgroup each take a quarter of the contraction
// and add up through LDS at the end.  Tiles are RB x 16 rows of one expert by CB x 16 output
// columns; more rows per tile reuse a weight load RB times.  Measured at 16 tokens x 256 x 512, 8
// experts: 31.9 + 31.9 us (64x64x64 tiles through LDS with 4-byte loads, 64 workgroups) ->
// 5.9 + 5.3 us; 512 tokens x 512 x 1024, 4 experts, top-3: 71.8 + 61.4 -> 56.4 + 40.5 us.
#include "common.h"
#include "tile_map.h"

namespace specmoe {
namespace {

constexpr int kWaves = 4, kThreads = kWaves * kWave;
constexpr int kStep = 16;                     // contraction elements per load of a wave

// WK waves share a tile and split its contraction; the other kWaves / WK factor takes the next
// tiles along the output columns.
template <bool SWIGLU, int RB, int CB, int WK, bool VEC>
__global__ __launch_bounds__(kThreads) void grouped_gemm_f32_kernel(
    const float* __restrict__ A, const int32_t* __restrict__ offsets,
    const float* __restrict__ W0, const float* __restrict__ W1, int E, int N, int K,
    float* __restrict__ C, const int32_t* __restrict__ row_src, int topk) {
    constexpr int WN = kWaves / WK, NM = SWIGLU ? 2 : 1;        // matrices per tile (gate, up)
    constexpr int BN = 16 * CB * WN;
    const int NT = (N + BN - 1) / BN;
    TileLoc t;
    if (!locate_tile<16 * RB>(offsets, E, NT, blockIdx.x, t)) return;
    const int lane = threadIdx.x % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int wk = wave % WK, wn = wave / WK;
    const int n0 = t.nt * BN + wn * 16 * CB;
    const int r = lane % 16, kq = (lane / 16) * 4;

    // rows beyond the tile and columns beyond N repeat the last valid one; they are not stored
    const float* a_row[RB];
    const float* w_row[NM][CB];
#pragma unroll
    for (int i = 0; i < RB; ++i) {
        const int row = t.row0 + min(16 * i + r, t.tile_rows - 1);
        a_row[i] = A + (size_t)(row_src ? row_src[row] / topk : row) * K;
    }
#pragma unroll
    for (int c = 0; c < CB; ++c) {
        const size_t at = ((size_t)t.expert * N + min(n0 + 16 * c + r, N - 1)) * K;
        w_row[0][c] = W0 + at;
        if (SWIGLU) w_row[NM - 1][c] = W1 + at;
    }
    // unsigned: the steps in flight run past the largest K
    const uint32_t k_end = K;
    auto load = [&](const float* p, uint32_t k) __attribute__((always_inline)) -> floatx4 {
        floatx4 v = {0.f, 0.f, 0.f, 0.f};
        if (VEC) {                            // K % 4 == 0, rows 16-byte aligned
            if (k < k_end) v = *reinterpret_cast<const floatx4*>(p + k);
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (k + q < k_end) v[q] = p[k + q];
        }
        return v;
    };

    floatx4 acc[NM][RB][CB];
#pragma unroll
    for (int m = 0; m < NM; ++m)
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int c = 0; c < CB; ++c) acc[m][i][c] = floatx4{0.f, 0.f, 0.f, 0.f};

    // PF steps are in flight: the whole quarter of a short contraction, or enough of a long one to
    // cover the way to L2
    constexpr int PF = RB >= 4 ? 2 : 4;
    floatx4 av[PF][RB], wv[PF][NM][CB];
    auto fetch = [&](int p, uint32_t k) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < RB; ++i) av[p][i] = load(a_row[i], k + kq);
#pragma unroll
        for (int m = 0; m < NM; ++m)
#pragma unroll
            for (int c = 0; c < CB; ++c) wv[p][m][c] = load(w_row[m][c], k + kq);
        __builtin_amdgcn_sched_barrier(0);    // keeps the requests PF steps ahead of their use
    };
    constexpr int STRIDE = kStep * WK;
    const uint32_t k_first = wk * kStep;
#pragma unroll
    for (int p = 0; p < PF; ++p) fetch(p, k_first + p * STRIDE);
    for (uint32_t k0 = k_first; k0 < k_end; k0 += PF * STRIDE) {
#pragma unroll
        for (int p = 0; p < PF; ++p) {        // steps beyond K hold zeros
            floatx4 a[RB], w[NM][CB];
#pragma unroll
            for (int i = 0; i < RB; ++i) a[i] = av[p][i];
#pragma unroll
            for (int m = 0; m < NM; ++m)
#pragma unroll
                for (int c = 0; c < CB; ++c) w[m][c] = wv[p][m][c];
            fetch(p, k0 + (p + PF) * STRIDE);
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int i = 0; i < RB; ++i)
#pragma unroll
                    for (int m = 0; m < NM; ++m)
#pragma unroll
                        for (int c = 0; c < CB; ++c)
                            acc[m][i][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                                w[m][c][q], a[i][q], acc[m][i][c], 0, 0, 0);
        }
    }

    if (WK > 1) {                             // quarters of the contraction, added in wave order
        __shared__ floatx4 part[WK > 1 ? WN * (WK - 1) : 1][NM * RB * CB][kWave];
        if (wk > 0) {
#pragma unroll
            for (int m = 0; m < NM; ++m)
#pragma unroll
                for (int i = 0; i < RB; ++i)
#pragma unroll
                    for (int c = 0; c < CB; ++c)
                        part[wn * (WK - 1) + wk - 1][(m * RB + i) * CB + c][lane] = acc[m][i][c];
        }
        __syncthreads();
        if (wk > 0) return;
#pragma unroll
        for (int s = 0; s < WK - 1; ++s)
#pragma unroll
            for (int m = 0; m < NM; ++m)
#pragma unroll
                for (int i = 0; i < RB; ++i)
#pragma unroll
                    for (int c = 0; c < CB; ++c)
                        acc[m][i][c] += part[wn * (WK - 1) + s][(m * RB + i) * CB + c][lane];
    }

    // lane l holds row l % 16 and columns 4 * (l / 16) .. + 3 of a 16 x 16 block
    const bool vec_out = N % 4 == 0 && ((uintptr_t)C & 15u) == 0;
#pragma unroll
    for (int i = 0; i < RB; ++i) {
        const int tr = 16 * i + r;
        if (tr >= t.tile_rows) continue;
        float* crow = C + (size_t)(t.row0 + tr) * N;
#pragma unroll
        for (int c = 0; c < CB; ++c) {
            const int col = n0 + 16 * c + kq;
            floatx4 v = acc[0][i][c];
            if (SWIGLU) {
                // silu in full fp32 precision (expf, true division)
#pragma unroll
                for (int q = 0; q < 4; ++q) v[q] = (v[q] / (1.0f + expf(-v[q]))) * acc[NM - 1][i][c][q];
            }
            if (vec_out) {
                if (col < N) *reinterpret_cast<floatx4*>(crow + col) = v;
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (col + q < N) crow[col + q] = v[q];
            }
        }
    }
}

template <bool SWIGLU, int RB, int CB, int WK>
void launch_f32(const float* A, const int32_t* offsets, const float* W0, const float* W1,
                int n_rows, int E, int N, int K, float* C, hipStream_t s, const int32_t* row_src,
                int topk) {
    const bool vec = K % 4 == 0 && (((uintptr_t)A | (uintptr_t)W0 | (uintptr_t)W1) & 15u) == 0;
    constexpr int BN = 16 * CB * (kWaves / WK);
    const dim3 grid((unsigned)grid_upper_bound(n_rows, E, 16 * RB, (N + BN - 1) / BN));
    if (vec)
        hipLaunchKernelGGL((grouped_gemm_f32_kernel<SWIGLU, RB, CB, WK, true>), grid,
                           dim3(kThreads), 0, s, A, offsets, W0, W1, E, N, K, C, row_src, topk);
    else
        hipLaunchKernelGGL((grouped_gemm_f32_kernel<SWIGLU, RB, CB, WK, false>), grid,
                           dim3(kThreads), 0, s, A, offsets, W0, W1, E, N, K, C, row_src, topk);
}

// Rows per tile by the average rows of an expert (16 up to 16 rows, 32 up to 32, else 64); waves
// split the contraction while the tiles alone would leave SIMDs idle (fewer than 1024 waves).
template <bool SWIGLU>
hipError_t launch_by_rows(const float* A, const int32_t* offsets, const float* W0, const float* W1,
                          int n_rows, int E, int N, int K, float* C, hipStream_t s,
                          const int32_t* row_src, int topk) {
    const int RB = (long long)n_rows <= 16ll * E ? 1 : ((long long)n_rows <= 32ll * E ? 2 : 4);
    const long long tiles = ((long long)n_rows / (16 * RB) + E) * ((N + 31) / 32);
    const bool split = tiles < 1024;
#define SPECMOE_F32(RB, CB, WK)                                                                   \
    launch_f32<SWIGLU, RB, CB, WK>(A, offsets, W0, W1, n_rows, E, N, K, C, s, row_src, topk)
    if (RB == 1) split ? SPECMOE_F32(1, 1, 4) : SPECMOE_F32(1, 2, 1);
    else if (RB == 2) split ? SPECMOE_F32(2, 1, 4) : SPECMOE_F32(2, 2, 1);
    else split ? SPECMOE_F32(4, 1, 4) : SPECMOE_F32(4, 2, 1);
#undef SPECMOE_F32
    return hipGetLastError();
}

}  // namespace

hipError_t launch_expert_up_f32(const float* x_perm, const int32_t* offsets, const float* wg,
                                const float* wu, int n_rows, int d, int f, int E, float* h,
                                hipStream_t s, const int32_t* row_src, int topk) {
    if (n_rows == 0) return hipSuccess;
    return launch_by_rows<true>(x_perm, offsets, wg, wu, n_rows, E, f, d, h, s, row_src, topk);
}

hipError_t launch_expert_down_f32(const float* h, const int32_t* offsets, const float* wd,
                                  int n_rows, int d, int f, int E, float* y, hipStream_t s) {
    if (n_rows == 0) return hipSuccess;
    return launch_by_rows<false>(h, offsets, wd, nullptr, n_rows, E, d, f, y, s, nullptr, 1);
}

}  // namespace specmoe
