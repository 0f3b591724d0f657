// Kernels and launchers of the persistent expert GEMMs (persist_tile.h) on row-major operands.
#include "persist_tile.h"

namespace specmoe {
namespace {

using namespace pipe;

typedef PersistCfg<160, 256, 3, true> Up;
typedef PersistCfg<160, 256, 3, false> Down;

template <typename C, bool GATHER, bool HALVES>
__global__ __launch_bounds__(C::THREADS) void grouped_gemm_bf16_persist_kernel(
    const bf16_t* __restrict__ A, const int32_t* __restrict__ offsets,
    const bf16_t* __restrict__ W0, const bf16_t* __restrict__ W1, int E, int N, int K,
    bf16_t* __restrict__ Cout, const int32_t* __restrict__ row_src, int topk, int group, int stream_out) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds_raw[];
    TileTable<C::BM> table;
    table.load(offsets, E);
    persist_tiles<C, GATHER, HALVES>(lds_raw, table, A, W0, W1, N, K, Cout, row_src, topk, stream_out,
                                            group > 0 && !table.even() ? group : 0);
}

template <typename C, bool GATHER, bool HALVES>
hipError_t launch(const bf16_t* A, const int32_t* offsets, const bf16_t* W0, const bf16_t* W1, int n_rows, int E, int N,
                  int K, bf16_t* Cout, const int32_t* row_src, int topk, int group, hipStream_t s) {
    // one-time, thread-safe (C++11 static initialisation): raise the dynamic LDS limit
    static const hipError_t attr = hipFuncSetAttribute(
        reinterpret_cast<const void*>(&grouped_gemm_bf16_persist_kernel<C, GATHER, HALVES>),
        hipFuncAttributeMaxDynamicSharedMemorySize, (int)C::LDS_BYTES);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL((grouped_gemm_bf16_persist_kernel<C, GATHER, HALVES>), dim3(kCus), dim3(C::THREADS),
                       C::LDS_BYTES, s, A, offsets, W0, W1, E, N, K, Cout, row_src, topk, group,
                       (int)streams_output(n_rows, N));
    return hipGetLastError();
}

// Tiles of an even batch, with 15 % for the spread of its rows; a batch meets no more experts than it has rows.
long long tiles_of(int n_rows, int E, int N, int rows, int outputs) {
    const long long m = (115ll * n_rows + 100ll * rows * E - 1) / (100ll * rows * E);
    return (n_rows < E ? n_rows : E) * m * ((N + outputs - 1) / outputs);
}
// Whether the persistent tiles are the better ones for an even batch: at least three quarters of the CUs get one, and
// they take at most half as many rounds of the chip as the half as wide tiles of the other kernels do (`slack`: more).
bool persist_wins(int n_rows, int E, int N, int outputs, int slack) {
    if (E > kWave) return false;
    const long long tiles = tiles_of(n_rows, E, N, Up::BM, outputs), others = tiles_of(n_rows, E, N, 128, outputs / 2);
    return 4 * tiles >= 3 * kCus && 2 * ((tiles + kCus - 1) / kCus) <= (others + kCus - 1) / kCus + slack;
}

}  // namespace

// Gate/up, us, the other kernels / this one (rows per expert; weights of another layer in between):
//  - contractions of 2048 to 4095, by the rounds that both take.  64 experts x 2048 x 1408: 6 rows 147 / 136, 30 rows 123 / 114, 120
//    rows 163 / 137, skewed (exponent of 1.1) 205 / 190; 16 of them with 28 rows 42 / 41, with 106 rows 56 / 47.  24 x 3840 x
//    1920, 120 rows 190 / 162, but 20 rows (1.4 rounds) 123 / 138; 16 x 2048 x 3072, 120 rows 111 / 101, 30 rows 72 / 76.  Contractions
//    below 2048 gain and lose (64 x 1024 x 1024, 4 rows 29 / 39, 60 rows 67 / 47).
//  - from 4096 on two rounds of one m-tile per expert, with the tile order in groups and the last round in halves:
//    16 x 5120 x 8192, 16 rows 437 / 408, 64 rows 557 / 502, skewed 588 / 504, 128 rows 567 / 520; 8 x 4096 x 14336, 20 rows 309 / 304, 125
//    rows 396 / 349, 83 rows skewed 393 / 335, two of them with 16 rows 79 / 76; but 175 rows (two m-tiles) 447 / 496, and four of 16 x
//    4096 x 2048 40 / 56.  At least one round of the experts that can be met (one row, 16 x 5120 x 8192, layer 76 / 84).
bool launches_expert_up_bf16_persist(int n_rows, int d, int f, int E) {
    if (d < kTailMinK) return d >= 2048 && persist_wins(n_rows, E, f, Up::BN_OUT, 0);
    const long long per_expert = (f + Up::BN_OUT - 1) / Up::BN_OUT;
    return E <= kWave && 115ll * n_rows <= 100ll * Up::BM * E && E * per_expert >= 2 * kCus &&
           n_rows * per_expert >= kCus;
}
hipError_t launch_expert_up_bf16_persist(const bf16_t* x_perm, const int32_t* offsets, const bf16_t* wg,
                                         const bf16_t* wu, int n_rows, int d, int f, int E, bf16_t* h,
                                         hipStream_t s, const int32_t* row_src, int topk) {
    const bool halves = d >= kTailMinK;
    const int group = halves && (f + Up::BN_OUT - 1) / Up::BN_OUT >= 24 ? 8 : 0;     // as tile_group()
    if (row_src)
        return halves ? launch<Up, true, true>(x_perm, offsets, wg, wu, n_rows, E, f, d, h, row_src, topk, group, s)
                      : launch<Up, true, false>(x_perm, offsets, wg, wu, n_rows, E, f, d, h, row_src, topk, group, s);
    return halves ? launch<Up, false, true>(x_perm, offsets, wg, wu, n_rows, E, f, d, h, nullptr, 1, group, s)
                  : launch<Up, false, false>(x_perm, offsets, wg, wu, n_rows, E, f, d, h, nullptr, 1, group, s);
}

// Down, contractions of 1280 to 4095, the same: 64 experts x 1408 x 2048, 6 rows 79 / 61, 30 rows 76 / 62, 120 rows 99 / 74, skewed 102 /
// 108 (three rounds and a few tiles); 37 experts with up to 60 rows 44 / 51, 16 with 106 rows 22 / 33; 24 x 1920 x 3840, 60 rows (1.4
// rounds) 94 / 72, skewed 92 / 80, 20 rows 67 / 70; 16 x 2048 x 4096, 25 rows 69 / 65, 75 rows 85 / 70.  From 4096 on it loses as often (16 x 8192 x
// 5120, 64 rows 250 / 275; 8 x 14336 x 4096, 83 rows 188 / 196).
bool launches_expert_down_bf16_persist(int n_rows, int d, int f, int E) {
    return f >= 1280 && f < 4096 && persist_wins(n_rows, E, d, Down::BN_OUT, (long long)n_rows >= 48ll * E ? 1 : 0);
}
hipError_t launch_expert_down_bf16_persist(const bf16_t* h, const int32_t* offsets, const bf16_t* wd, int n_rows,
                                           int d, int f, int E, bf16_t* y, hipStream_t s) {
    return launch<Down, false, false>(h, offsets, wd, nullptr, n_rows, E, d, f, y, nullptr, 1, 0, s);
}

}  // namespace specmoe
