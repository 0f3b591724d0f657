// Kernels and launchers of the large- and mid-batch expert GEMMs (pipe16_tile.h).
#include "pipe16_tile.h"

namespace specmoe {
namespace {

using namespace pipe;

// 256-wide tiles on tile-packed weights: the last round may be shared out in halves (tile_map.h)
template <typename C, bool PB, bool PO>
constexpr bool kHalves = C::BN == 256 && PB && (PO || !C::SWIGLU);

template <typename C, bool PA, bool PB, bool PO, bool SHARE>
__global__ __launch_bounds__(C::THREADS) void grouped_gemm_bf16_pipe16_kernel(
    const bf16_t* __restrict__ A, const int32_t* __restrict__ offsets,
    const bf16_t* __restrict__ W0, const bf16_t* __restrict__ W1, int E, int N, int K,
    bf16_t* __restrict__ Cout, const int32_t* __restrict__ row_src, int topk, int group,
    int stream_out) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds_raw[];
    TileLoc t;
    const bool halves = kHalves<C, PB, PO> && K >= kTailMinK;
    if (!locate_tile_even<C::BM, 16, SHARE>(offsets, E, (N + C::BN_OUT - 1) / C::BN_OUT, blockIdx.x, t,
                                            group, halves))
        return;
    if constexpr (SHARE && kHalves<C, PB, PO>) {
        if (t.half >= 0) {
            typedef PipeCfg<C::BM, C::BN / 2, C::BK, C::STAGES, C::WM, C::WN, C::SWIGLU> Half;
            t.nt = 2 * t.nt + t.half;
            if (t.nt * Half::BN_OUT < N)
                pipe16_tile<Half, PA, PB, PO>(lds_raw, t, A, W0, W1, N, K, Cout, row_src, topk, stream_out);
            return;
        }
    }
    pipe16_tile<C, PA, PB, PO>(lds_raw, t, A, W0, W1, N, K, Cout, row_src, topk, stream_out);
}

// n-tiles per group of the tile order (tile_map.h) for gate/up batches spread unevenly over the experts.  Measured,
// packed operands, us, expert-major / in groups: 16 x 5120 x 8192, 128 rows per expert on average 578 / 523, 62
// rows 540 / 480; 8 x 4096 x 14336, 375 rows under a Zipf exponent of 1.1 710 / 617, 86 rows, 0.5 434 / 427.  The line at 24 n-tiles
// (means over three seeds, exponents of 1.1 and 0.5; 16 x 2048): 28 n-tiles, 100 rows 110 / 103, 87 / 90, 200 rows 145 / 132, 113 / 109; 24,
// 62 rows 75 / 75, 71 / 71, 200 rows 105 / 103, 103 / 99; 20, 100 rows 75 / 73, 74 / 76, 200 rows 99 / 94, 96 / 91; 12, 200 rows 54 / 56,
// 51 / 52.  With fewer rows it loses as often (64 x 2048 x 1408, 30 rows 108 / 113), and so it does in the down projection (16 x
// 8192 x 5120 297 / 288 to 317).
template <typename C>
int tile_group(int n_rows, int E, int N) {
    return C::SWIGLU && N >= 24 * C::BN_OUT && (long long)n_rows >= 60ll * E ? 8 : 0;
}

template <typename C, bool PA, bool PB, bool PO, bool SHARE>
hipError_t launch_pipe16_form(const bf16_t* A, const int32_t* offsets, const bf16_t* W0,
                              const bf16_t* W1, int n_rows, int E, int N, int K, bf16_t* Cout,
                              hipStream_t s, const int32_t* row_src, int topk, int group) {
    // one-time, thread-safe (C++11 static initialisation): raise the dynamic LDS limit
    static const hipError_t attr = hipFuncSetAttribute(
        reinterpret_cast<const void*>(&grouped_gemm_bf16_pipe16_kernel<C, PA, PB, PO, SHARE>),
        hipFuncAttributeMaxDynamicSharedMemorySize, (int)C::LDS_BYTES);
    if (attr != hipSuccess) return attr;
    const long long NT = (N + C::BN_OUT - 1) / C::BN_OUT;
    const long long grid = grid_upper_bound(n_rows, E, C::BM, NT) +
                           (kHalves<C, PB, PO> && K >= kTailMinK ? kTailBlocks : 0);
    hipLaunchKernelGGL((grouped_gemm_bf16_pipe16_kernel<C, PA, PB, PO, SHARE>), dim3((unsigned)grid),
                       dim3(C::THREADS), C::LDS_BYTES, s, A, offsets, W0, W1, E, N, K, Cout,
                       row_src, topk, group, (int)streams_output(n_rows, N));
    return hipGetLastError();
}

// SHARE: the tile order in groups and the halved last round (tile_map.h).  A form of its own, since working out a
// tile takes 0.3 us longer with them: 64 x 2048 x 1408, 6 rows each, a layer of 83.6 us 84.3.
template <typename C, bool PA = false, bool PB = false, bool PO = false>
hipError_t launch_pipe16(const bf16_t* A, const int32_t* offsets, const bf16_t* W0,
                         const bf16_t* W1, int n_rows, int E, int N, int K, bf16_t* Cout,
                         hipStream_t s, const int32_t* row_src = nullptr, int topk = 1) {
    if constexpr (C::BN == 256) {
        const int group = tile_group<C>(n_rows, E, N);
        if (group > 0 || (kHalves<C, PB, PO> && K >= kTailMinK))
            return launch_pipe16_form<C, PA, PB, PO, true>(A, offsets, W0, W1, n_rows, E, N, K, Cout, s,
                                                           row_src, topk, group);
    }
    return launch_pipe16_form<C, PA, PB, PO, false>(A, offsets, W0, W1, n_rows, E, N, K, Cout, s,
                                                    row_src, topk, 0);
}

// Down projection on packed operands where 256-wide tiles would leave part of the chip idle: the
// form is chosen on the device (launch_expert_down_bf16_packed).
typedef PipeCfg<128, 128, 32, 4, 2, 4, false> DownNarrow;
typedef PipeCfg<320, 128, 32, 4, 2, 4, false> DownNarrowTall;

template <typename Wide>
__global__ __launch_bounds__(Wide::THREADS) void grouped_down_bf16_packed_few_kernel(
    const bf16_t* __restrict__ h, const int32_t* __restrict__ offsets,
    const bf16_t* __restrict__ wd, int E, int N, int K, bf16_t* __restrict__ y, int stream_out) {
    static_assert(Wide::THREADS == DownNarrow::THREADS && Wide::THREADS == DownNarrowTall::THREADS,
                  "one launch serves all");
    static_assert(Wide::LDS_BYTES >= DownNarrow::LDS_BYTES &&
                  Wide::LDS_BYTES >= DownNarrowTall::LDS_BYTES, "one launch serves all");
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds_raw[];
    typedef EvenPolicy<DownNarrow::BM, 16> Low;
    typedef EvenPolicy<DownNarrowTall::BM, 16> High;
    typedef EvenPolicy<Wide::BM, 16> Full;
    const int NT = (N + 127) / 128;
    int low[1], mt[2];
    count_mtiles<Low>(offsets, E, low);
    TileLoc t;
    if (tile_rounds(low[0], NT) == 1) {
        if (locate<Low, From::counted>(offsets, E, NT, blockIdx.x, low[0], t))
            pipe16_tile<DownNarrow, true, true>(lds_raw, t, h, wd, nullptr, N, K, y, nullptr, 1, stream_out);
        return;
    }
    count_mtiles<High, Full>(offsets, E, mt);
    if (tile_rounds(mt[0], NT) == 1) {
        if (locate<High, From::counted>(offsets, E, NT, blockIdx.x, mt[0], t))
            pipe16_tile<DownNarrowTall, true, true>(lds_raw, t, h, wd, nullptr, N, K, y, nullptr, 1, stream_out);
    } else if (locate<Full, From::counted>(offsets, E, (N + Wide::BN_OUT - 1) / Wide::BN_OUT,
                                           blockIdx.x, mt[1], t)) {
        pipe16_tile<Wide, true, true>(lds_raw, t, h, wd, nullptr, N, K, y, nullptr, 1, stream_out);
    }
}

template <typename Wide>
hipError_t launch_down_packed_few(const bf16_t* h, const int32_t* offsets, const bf16_t* wd,
                                  int n_rows, int E, int N, int K, bf16_t* y, hipStream_t s) {
    // one-time, thread-safe (C++11 static initialisation): raise the dynamic LDS limit
    static const hipError_t attr = hipFuncSetAttribute(
        reinterpret_cast<const void*>(&grouped_down_bf16_packed_few_kernel<Wide>),
        hipFuncAttributeMaxDynamicSharedMemorySize, (int)Wide::LDS_BYTES);
    if (attr != hipSuccess) return attr;
    // the narrow forms run only where their tiles make one round
    const long long wide = grid_upper_bound(n_rows, E, Wide::BM, (N + Wide::BN_OUT - 1) / Wide::BN_OUT);
    const long long grid = wide > kCus ? wide : kCus;
    hipLaunchKernelGGL(grouped_down_bf16_packed_few_kernel<Wide>, dim3((unsigned)grid),
                       dim3(Wide::THREADS), Wide::LDS_BYTES, s, h, offsets, wd, E, N, K, y,
                       (int)streams_output(n_rows, N));
    return hipGetLastError();
}

}  // namespace

hipError_t launch_expert_up_bf16_large16(const bf16_t* x_perm, const int32_t* offsets,
                                         const bf16_t* wg, const bf16_t* wu, int n_rows, int d,
                                         int f, int E, bf16_t* h, hipStream_t s,
                                         const int32_t* row_src, int topk) {
    return launch_pipe16<PipeCfg<320, 256, 32, 4, 2, 4, true>>(x_perm, offsets, wg, wu, n_rows, E,
                                                               f, d, h, s, row_src, topk);
}

hipError_t launch_expert_down_bf16_large16(const bf16_t* h, const int32_t* offsets,
                                           const bf16_t* wd, int n_rows, int d, int f, int E,
                                           bf16_t* y, hipStream_t s) {
    return launch_pipe16<PipeCfg<320, 256, 32, 4, 2, 4, false>>(h, offsets, wd, nullptr, n_rows, E,
                                                                d, f, y, s);
}

// Tiles of 128 weight rows instead of 256 where a batch has few tiles: a 256-wide tile takes a
// whole CU (112 or 144 KB of LDS), so up to 128 of them leave half the chip idle.  At most 64 wide
// tiles, or up to 128 in gate/up while an expert's rows (the average plus 15 % for the spread) fit in 128: 128 x
// 128 tiles, 64 KB, two workgroups per CU.  Measured, packed operands, us, 256-wide -> narrow: down 1024 x
// 2048, 16 experts: 64 rows each 32 -> 23, 256 55 -> 32; gate/up 3072 x 1024, 8 experts: 25 rows 38 -> 30, 250
// 63 -> 40 (500: 63 -> 78).  At 256 wide tiles and more the 256-wide ones are ahead or level (gate/up
// 2048 x 1024, 16 experts, 256 rows 39 -> 62).
static bool narrow_tiles(int n_rows, int E, int N, int wide) {
    const WideTiles w(n_rows, E, N, wide);
    return w.few() && (w.tiles <= 64 || 115ll * n_rows <= 12800ll * E);
}

// Otherwise tile height by the average rows per expert, as for the row-major operands: 320-row
// tiles from 192 rows per expert, 192-row tiles below.  h_row_major: h is written [n_rows, f] row-major
// (for a down projection on row-major operands) instead of tile-packed.
hipError_t launch_expert_up_bf16_packed_x(const bf16_t* x_packed, const int32_t* offsets,
                                          const bf16_t* wg_packed, const bf16_t* wu_packed,
                                          int n_rows, int d, int f, int E, bf16_t* h,
                                          bool h_row_major, hipStream_t s) {
    typedef PipeCfg<320, 256, 32, 4, 2, 4, true> Large;
    typedef PipeCfg<192, 256, 32, 4, 2, 4, true> Mid;
    typedef PipeCfg<128, 128, 32, 4, 2, 4, true> Small;
    const bool large = (long long)n_rows >= 192ll * E;
    if (h_row_major)
        return large ? launch_pipe16<Large, true, true, false>(x_packed, offsets, wg_packed,
                                                               wu_packed, n_rows, E, f, d, h, s)
                     : launch_pipe16<Mid, true, true, false>(x_packed, offsets, wg_packed,
                                                             wu_packed, n_rows, E, f, d, h, s);
    if (narrow_tiles(n_rows, E, f, Large::BN_OUT))
        return launch_pipe16<Small, true, true, true>(x_packed, offsets, wg_packed, wu_packed, n_rows,
                                                      E, f, d, h, s);
    return large ? launch_pipe16<Large, true, true, true>(x_packed, offsets, wg_packed, wu_packed,
                                                          n_rows, E, f, d, h, s)
                 : launch_pipe16<Mid, true, true, true>(x_packed, offsets, wg_packed, wu_packed,
                                                        n_rows, E, f, d, h, s);
}

// Tile-packed variant that gathers the token rows itself from the row-major token matrix (per-lane
// row addresses, 64-byte requests on the activation side); weights and h tile-packed.
hipError_t launch_expert_up_bf16_packed(const bf16_t* x, const int32_t* offsets,
                                        const bf16_t* wg_packed, const bf16_t* wu_packed,
                                        int n_rows, int d, int f, int E, bf16_t* h_packed,
                                        hipStream_t s, const int32_t* row_src, int topk) {
    typedef PipeCfg<320, 256, 32, 4, 2, 4, true> Large;
    typedef PipeCfg<192, 256, 32, 4, 2, 4, true> Mid;
    typedef PipeCfg<128, 128, 32, 4, 2, 4, true> Small;
    if (narrow_tiles(n_rows, E, f, Large::BN_OUT))
        return launch_pipe16<Small, false, true, true>(x, offsets, wg_packed, wu_packed, n_rows, E, f, d,
                                                       h_packed, s, row_src, topk);
    if ((long long)n_rows < 192ll * E)
        return launch_pipe16<Mid, false, true, true>(x, offsets, wg_packed, wu_packed, n_rows, E, f, d,
                                                     h_packed, s, row_src, topk);
    return launch_pipe16<Large, false, true, true>(x, offsets, wg_packed, wu_packed, n_rows, E, f, d,
                                                   h_packed, s, row_src, topk);
}

hipError_t launch_expert_down_bf16_packed(const bf16_t* h_packed, const int32_t* offsets,
                                          const bf16_t* wd_packed, int n_rows, int d, int f,
                                          int E, bf16_t* y, hipStream_t s) {
    // Short contractions with up to 12 rows per expert on average: also the 128 x 128 tiles.  Such a
    // batch may activate a few experts only (the draft model: 16 of 64 experts are 128 wide tiles,
    // 24.0 -> 20.2 us at 2048 x 1408; 4 of 16, 1024 x 2048: 23.4 -> 19.5), which the host does not know.
    // With all of them active nothing is lost on even rows (64 of 64: 62.6 -> 62.0), but 8 % on skewed
    // ones (8 rows each under a Zipf exponent of 1.1: 69 -> 75).  Choosing on the device instead gave
    // 64.6, 70.5 and, with 16 of 64 active, 21.0: the even batch pays for it, so the host's rule stayed.
    // Gate/up gains with few active experts (4 of 64: 24.6 -> 20.4) and loses with more (16 of 64: 32.4
    // -> 35.5).
    const bool maybe_few = f < 4096 && (long long)n_rows <= 12ll * E;
    const WideTiles w(n_rows, E, d, 256);
    if (maybe_few || (w.few() && w.tiles <= 64))
        return launch_pipe16<DownNarrow, true, true, false>(h_packed, offsets, wd_packed, nullptr, n_rows,
                                                            E, d, f, y, s);
    // 65 to 128 wide tiles (8 experts x 4096 outputs): the form goes by how many tiles the batch has,
    // which depends on how its rows are spread.  While they make one round of the chip, 128 weight rows
    // per tile keep twice the CUs busy: up to 128 rows, else up to 320; a second round costs more than
    // it gains.  Measured, us, 256-wide / chosen here, 4096 x 14336, 8 experts: 128 x 128 tiles: 70 rows each
    // 228 / 161, two active with 280 rows each 201 / 125; 320 x 128: 170 rows each 272 / 236, 70 rows under a
    // Zipf exponent of 1.1 231 / 224; 256-wide: 130 rows under that exponent 237 (320 x 128 tiles 385).
    typedef PipeCfg<320, 256, 32, 4, 2, 4, false> Large;
    typedef PipeCfg<192, 256, 32, 4, 2, 4, false> Mid;
    const bool large = (long long)n_rows >= 192ll * E;
    if (w.few())
        return large ? launch_down_packed_few<Large>(h_packed, offsets, wd_packed, n_rows, E, d, f, y, s)
                     : launch_down_packed_few<Mid>(h_packed, offsets, wd_packed, n_rows, E, d, f, y, s);
    return large ? launch_pipe16<Large, true, true, false>(h_packed, offsets, wd_packed, nullptr, n_rows,
                                                           E, d, f, y, s)
                 : launch_pipe16<Mid, true, true, false>(h_packed, offsets, wd_packed, nullptr, n_rows, E,
                                                         d, f, y, s);
}

// In between (tens to a few hundred rows per expert, e.g. 16 experts with top-1 routing, 30 to
// 530 rows each), gate/up projection: the same kernel with tiles of at most 192 rows.  Hot experts
// are MFMA-bound, cold ones stream their weights; measured at that shape (gate/up alone): 192- and
// 256-row tiles 668 us, 128-row 796 us, 320-row 732 us, the 32x32x16 kernel with 128 x 128 tiles
// 750 us.  (For the down projection of that shape the 32x32x16 kernel stays ahead: 340 vs 388 us.)
hipError_t launch_expert_up_bf16_mid(const bf16_t* x_perm, const int32_t* offsets,
                                     const bf16_t* wg, const bf16_t* wu, int n_rows, int d, int f,
                                     int E, bf16_t* h, hipStream_t s, const int32_t* row_src,
                                     int topk) {
    return launch_pipe16<PipeCfg<192, 256, 32, 4, 2, 4, true>>(x_perm, offsets, wg, wu, n_rows, E,
                                                               f, d, h, s, row_src, topk);
}

}  // namespace specmoe
