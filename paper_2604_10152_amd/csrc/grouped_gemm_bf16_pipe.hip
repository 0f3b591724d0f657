// Expert GEMMs for few to a few hundred rows per expert on the gfx950 matrix cores
// (v_mfma_f32_32x32x16_bf16): multi-stage LDS ring filled by direct global->LDS loads, MFMA
// fragments double-buffered in registers.
// (SpecMoE Sec. 2.1: only the rows routed to an expert meet its FFN-sized weights; with a
// small verification batch - Sec. 2.2 - an expert sees tens of rows and the kernel is bound
// by streaming its weights from HBM once.)
//
// One workgroup = BM rows of one expert x BN weight rows.  Per step of BK contraction
// elements every wave issues its share of `global_load_lds_dwordx4` instructions: 64 lanes x
// 16 bytes go straight from L2/HBM into 1 KB of LDS, no staging registers, no ds_write.  The
// lane -> global chunk map carries the bank swizzle, so the LDS image is the swizzled tile.
// STAGES buffers form a ring; a stage is requested STAGES-1 steps before it is multiplied and
// must have landed one step before (vmcnt + one barrier per step), which leaves STAGES-2
// steps of MFMA work to cover the HBM latency.  Because readiness is established one step
// ahead, the first fragments of the next stage are read before the barrier and the matrix
// pipe does not drain at step boundaries.
//
// The loads are inline assembly on purpose: the compiler would otherwise put vmcnt(0) in
// front of every LDS read that follows an LDS-DMA load, which collapses the ring to depth 1.
// Hand-placed s_waitcnt vmcnt(n) is safe next to compiler-generated waits: extra outstanding
// loads can only make a compiler-chosen wait stricter, never weaker.
#include "persist_tile.h"
#include "pipe16_tile.h"
#include "pipe_common.h"
#include "stream_tiles.h"

#include <type_traits>

namespace specmoe {
namespace {

using namespace pipe;

// the work of one workgroup: tile t (lds_raw: C::LDS_BYTES)
template <typename C>
__device__ __forceinline__ void pipe_tile(
    unsigned char* lds_raw, const TileLoc& t,
    const bf16_t* __restrict__ A,        // [n_rows, K]
    const bf16_t* __restrict__ W0,       // [E, N, K]   (gate, or down)
    const bf16_t* __restrict__ W1,       // [E, N, K]   (up; SWIGLU only)
    int N, int K, bf16_t* __restrict__ Cout /* [n_rows, N] */,
    const int32_t* __restrict__ row_src /* nullable: A row r is A[row_src[r] / topk] */, int topk,
    bool stream_out /* streams_output() */) {
    static_assert(!C::SWIGLU || ((C::BN / 2 / C::ROWS_PER_DMA) % C::NWAVES == 0 && C::TN % 2 == 0),
                  "gate/up halves must split on a wave-load round and pair up inside a wave");
    const int row0 = t.row0, tile_rows = t.tile_rows;
    const int n0 = t.nt * C::BN_OUT;
    const int nsub = (tile_rows + 31) / 32;

    const int tid = threadIdx.x, lane = tid % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    // Waves w and w+4 share a SIMD.  Giving them different wm means a tile with an odd number
    // of 32-row sub-tiles loads every SIMD equally (5+4 instead of 5+5 and 4+4).
    const int wm = wave / C::WN, wn = wave % C::WN;
    const uint32_t lds_base =
        (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds_raw;

    // ---- global side of the wave-loads -------------------------------------------------
    // with row_src the activation rows are gathered on the fly (A is then the token matrix)
    const unsigned char* a_base = uniform_ptr(
        reinterpret_cast<const unsigned char*>(A + (row_src ? (size_t)0 : (size_t)row0 * K)));
    const size_t wrow = (size_t)t.expert * N + min(n0, N - 1);
    const unsigned char* w0 = uniform_ptr(reinterpret_cast<const unsigned char*>(W0 + wrow * K));
    const unsigned char* w1 =
        C::SWIGLU ? uniform_ptr(reinterpret_cast<const unsigned char*>(W1 + wrow * K)) : nullptr;
    const int n_left = N - n0;
    uint32_t a_off[C::A_PW], b_off[C::B_PW];
    int a_cnt = 0;                               // A wave-loads this wave issues per stage
    {
        const int srow = lane / C::CHUNKS, pc = lane % C::CHUNKS;   // LDS slot of this lane
#pragma unroll
        for (int jj = 0; jj < C::A_PW; ++jj) {
            const int r = (wave + jj * C::NWAVES) * C::ROWS_PER_DMA + srow;
            const int c = pc ^ ((r / C::RPG) % C::CHUNKS);
            const int rr = min(r, tile_rows - 1);
            const unsigned arow = row_src ? (unsigned)(row_src[row0 + rr] / topk) : (unsigned)rr;
            a_off[jj] = (arow * (unsigned)K + (unsigned)(c * 8)) * 2u;
            // this wave's A loads: wave-load j = wave + jj*NWAVES covers tile rows j*16.. ;
            // only loads that hold at least one real row are issued
            if ((wave + jj * C::NWAVES) * C::ROWS_PER_DMA < tile_rows) a_cnt = jj + 1;
        }
#pragma unroll
        for (int jj = 0; jj < C::B_PW; ++jj) {
            const int r = (wave + jj * C::NWAVES) * C::ROWS_PER_DMA + srow;
            const int c = pc ^ ((r / C::RPG) % C::CHUNKS);
            const int rn = (C::SWIGLU && r >= C::BN / 2) ? r - C::BN / 2 : r;
            b_off[jj] = (uint32_t)((min(rn, n_left - 1) * K + c * 8) * 2);
        }
    }
    const int KT = K / C::BK;
    // One wave-load of stage kt into ring slot buf.  Loads 0 .. A_PW-1 are this wave's A rows
    // (issued only if they hold real rows), loads A_PW .. A_PW+B_PW-1 its weight rows.
    // nt_tag: the weight loads carry the non-temporal hint (tiles whose weights no other
    // workgroup reads)
    auto issue_one = [&](auto nt_tag, int which, int kt, int buf) __attribute__((always_inline)) {
        const size_t kb = (size_t)min(kt, KT - 1) * C::ROW_BYTES;   // clamped: tail re-loads
        const uint32_t sbase = lds_base + (uint32_t)buf * C::STAGE_BYTES + wave * 1024u;
#pragma unroll
        for (int jj = 0; jj < C::A_PW; ++jj)
            if (which == jj && jj < a_cnt)
                dma16(a_base + kb, a_off[jj], sbase + jj * C::NWAVES * 1024u);
#pragma unroll
        for (int jj = 0; jj < C::B_PW; ++jj) {
            const bool up = C::SWIGLU && (jj * C::NWAVES * C::ROWS_PER_DMA >= C::BN / 2);
            if (which == C::A_PW + jj) {
                if (decltype(nt_tag)::value)
                    dma16_nt((up ? w1 : w0) + kb, b_off[jj],
                             sbase + C::A_BYTES + jj * C::NWAVES * 1024u);
                else
                    dma16((up ? w1 : w0) + kb, b_off[jj],
                          sbase + C::A_BYTES + jj * C::NWAVES * 1024u);
            }
        }
    };
    auto issue_stage = [&](auto nt_tag, int kt, int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < C::G_MAX; ++q) issue_one(nt_tag, q, kt, buf);
    };

    // ---- LDS side of the fragment reads ---------------------------------------------------
    // A sub-tile i: tile rows 32*(wm + WM*i) + lane%32 ; B sub-tile j: weight rows nb(j) + lane%32.
    // Sub-tile bases are multiples of 32 rows, which leaves the swizzle term unchanged, so one
    // per-lane offset per k-step serves all sub-tiles through immediate offsets.
    int a_rd[C::KK], b_rd[C::KK];
#pragma unroll
    for (int kk = 0; kk < C::KK; ++kk) {
        const int c = kk * 2 + (lane >> 5);
        a_rd[kk] = swz<C>(32 * wm + (lane & 31), c);
        b_rd[kk] = C::A_BYTES + swz<C>((lane & 31), c);
    }
    auto nb = [&](int j) __attribute__((always_inline)) -> int {     // B sub-tile base row
        if (C::SWIGLU) {
            constexpr int H = C::TN / 2;
            return (j < H) ? 32 * (wn * H + j) : C::BN / 2 + 32 * (wn * H + (j - H));
        }
        return 32 * (wn * C::TN + j);
    };

    const int ta = min(C::TM, max(0, (nsub - wm + C::WM - 1) / C::WM));   // active sub-tiles
    // loads this wave has in flight per stage; stages STAGES-3 deep may still be outstanding
    // when the stage needed next must have landed
    const int vm_allow = (C::STAGES - 3) * (a_cnt + C::B_PW);

    auto run = [&](auto ta_tag, auto nt_tag) __attribute__((always_inline)) {
        constexpr int TA = decltype(ta_tag)::value;
        constexpr int TAX = TA > 0 ? TA : 1;
        floatx16 acc[TAX][C::TN];
#pragma unroll
        for (int i = 0; i < TA; ++i)
#pragma unroll
            for (int j = 0; j < C::TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

        bf16x8 af[2][TAX], bfr[2][C::TN];
        auto read_frags = [&](int set, int buf, int kk) __attribute__((always_inline)) {
            if (TA == 0) return;
            const unsigned char* sb = lds_raw + buf * C::STAGE_BYTES;
#pragma unroll
            for (int j = 0; j < C::TN; ++j)
                bfr[set][j] = *reinterpret_cast<const bf16x8*>(sb + b_rd[kk] + nb(j) * C::ROW_BYTES);
#pragma unroll
            for (int i = 0; i < TA; ++i)
                af[set][i] = *reinterpret_cast<const bf16x8*>(sb + a_rd[kk] +
                                                               32 * C::WM * i * C::ROW_BYTES);
        };
        auto mfma_row = [&](int set, int i) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < C::TN; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[set][j], af[set][i],
                                                                    acc[i][j], 0, 0, 0);
        };

        // prologue: request stages 0 .. STAGES-2, wait for 0 and 1
#pragma unroll
        for (int s = 0; s < C::STAGES - 1; ++s) issue_stage(nt_tag, s, s);
        wait_vmcnt_dyn(vm_allow);
        __builtin_amdgcn_s_barrier();
        read_frags(0, 0, 0);

        int buf = 0;                               // ring slot of stage kt
        for (int kt = 0; kt < KT; ++kt) {
            const int buf_next = (buf + 1 == C::STAGES) ? 0 : buf + 1;
            const int buf_free = (buf == 0) ? C::STAGES - 1 : buf - 1;   // held stage kt-1
            // The requests for stage kt+STAGES-1 go out one at a time between the matrix
            // instructions of the first k-step (all eight waves leave the barrier together; a
            // burst of wave-loads would back up the address unit and hold the MFMAs behind it).
            // sched_barrier(0) pins this order: the compiler's scheduler would otherwise sink
            // the fragment reads next to their use and bunch the loads.
#pragma unroll
            for (int kk = 0; kk < C::KK; ++kk) {
                if (kk + 1 < C::KK) read_frags((kk + 1) & 1, buf, kk + 1);
                else read_frags(0, buf_next, 0);         // stage kt+1 landed one step ago
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < TAX; ++i) {
                    if (i < TA) mfma_row(kk & 1, i);
                    __builtin_amdgcn_sched_barrier(0);
                    if (kk == 0) {
                        if (i < C::G_MAX) issue_one(nt_tag, i, kt + C::STAGES - 1, buf_free);
                        if (i == TAX - 1)
#pragma unroll
                            for (int q = TAX; q < C::G_MAX; ++q)
                                issue_one(nt_tag, q, kt + C::STAGES - 1, buf_free);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
            wait_vmcnt_dyn(vm_allow);              // own share of stage kt+2 has landed
            __builtin_amdgcn_s_barrier();
            buf = buf_next;
        }
        wait_vmcnt<0>();                           // no load may outlive the workgroup's LDS

        // epilogue.  The matrix instruction is issued as (weights x activations^T), so a lane
        // holds ONE tile row (lane%32) and, for each g = r/4, four consecutive output columns
        // 8g + 4*(lane/32) + r%4, i.e. 8 bytes of bf16.
        //  - SwiGLU tile (BN/2 = 64 output columns): the 8-byte pieces go to an LDS image of the tile
        //    and the workgroup then writes whole 128-byte rows.
        //  - plain tile: lanes l and l ^ 32 exchange halves of two g, so a lane stores 8 columns (without the
        //    hint: the row-major down projection is level or 2 % behind with it).
        const int row = lane & 31, chalf = (lane >> 5) * 4;
        if (C::SWIGLU) __builtin_amdgcn_s_barrier();   // every wave's loads have landed: LDS is free
#pragma unroll
        for (int i = 0; i < TA; ++i) {
            const int sub = 32 * (wm + C::WM * i), trow = sub + row;
            if (!C::SWIGLU && trow >= tile_rows) continue;
            constexpr int JN = C::SWIGLU ? C::TN / 2 : C::TN;
#pragma unroll
            for (int j = 0; j < JN; ++j) {
                const int c0 = 32 * (wn * JN + j);                // first column inside the tile
                auto value = [&](int g) __attribute__((always_inline)) -> uint2 {
                    float v[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        if (C::SWIGLU) {
                            const float gt = acc[i][j][4 * g + q], up = acc[i][j + JN][4 * g + q];
                            v[q] = gt * __builtin_amdgcn_rcpf(1.0f + __expf(-gt)) * up;
                        } else {
                            v[q] = acc[i][j][4 * g + q];
                        }
                    }
                    return make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
                };
                if (C::SWIGLU) {
#pragma unroll
                    for (int g = 0; g < 4; ++g)
                        *reinterpret_cast<uint2*>(lds_raw + trow * kStageRowBytes + (c0 + chalf + 8 * g) * 2) = value(g);
                } else if (n0 + c0 < N) {                         // N is a multiple of 64
#pragma unroll
                    for (int g = 0; g < 4; g += 2) {
                        uint2 a = value(g), b = value(g + 1);
                        lane_swap<32>(a.x, b.x);
                        lane_swap<32>(a.y, b.y);
                        store16(false, Cout + (size_t)(row0 + sub) * N + n0 + c0,
                                (uint32_t)(row * N + 8 * g + 2 * chalf) * 2u, U128{a.x, a.y, b.x, b.y});
                    }
                }
            }
        }
        // the barrier behind does not wait for the writes to the LDS
        if (C::SWIGLU) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    };

    static_assert(C::TM <= 5, "extend the dispatch below");
    // An expert with a single m-tile: every weight tile of it is read by exactly one workgroup,
    // once - a pure stream out of HBM, which the non-temporal hint speeds up (dma16_nt;
    // which tiles of gate/up have it: pipe16_tile.h).  With several m-tiles the workgroups that share a weight tile meet
    // in the L2, and the hint would cost those hits.
    // (whole 128-byte lines per row and stage only: half-line loads rely on the L2 keeping the
    // other half for the next stage)
    const bool w_once = C::ROW_BYTES >= 128 && t.mt == 1 && (!C::SWIGLU || tile_rows <= 64 || t.single);
    auto run_sel = [&](auto ta_tag) __attribute__((always_inline)) {
        if (w_once) run(ta_tag, std::true_type{});
        else run(ta_tag, std::false_type{});
    };
    switch (ta) {
        case 0: run_sel(std::integral_constant<int, 0>{}); break;
        case 1: run_sel(std::integral_constant<int, 1>{}); break;
        case 2: if constexpr (C::TM >= 2) run_sel(std::integral_constant<int, 2>{}); break;
        case 3: if constexpr (C::TM >= 3) run_sel(std::integral_constant<int, 3>{}); break;
        case 4: if constexpr (C::TM >= 4) run_sel(std::integral_constant<int, 4>{}); break;
        default: if constexpr (C::TM >= 5) run_sel(std::integral_constant<int, 5>{}); break;
    }

    if (C::SWIGLU) {
        // cooperative write-out of the staged tile: 16 bytes per lane, whole rows
        static_assert(!C::SWIGLU || (size_t)C::BM * kStageRowBytes <= C::LDS_BYTES, "stage tile");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");                      // no read moves up across it
        constexpr int CPR = C::BN_OUT / 8;                  // 16-byte chunks per tile row
        constexpr int RPP = C::THREADS / CPR;               // rows per pass
        const int cr = tid / CPR, cc = tid % CPR;
        const int col = n0 + cc * 8;
        for (int r = cr; r < tile_rows; r += RPP) {
            const U128 v = *reinterpret_cast<const U128*>(lds_raw + r * kStageRowBytes + cc * 16);
            if (col < N)                                    // N is a multiple of 64
                store16(stream_out, Cout + (size_t)row0 * N, (uint32_t)(r * N + col) * 2u, v);
        }
    }
}

// Down projection with few rows per expert: by the number of tiles this batch has (known on the
// device only) the ring above or the independent streams of stream_tiles.h.
typedef PipeCfg<64, 128, 64, 6, 1, 4, false> DownSmall;
constexpr size_t kDownSmallLds =
    DownSmall::LDS_BYTES > stream::kStreamLds ? DownSmall::LDS_BYTES : stream::kStreamLds;

__global__ __launch_bounds__(DownSmall::THREADS) void grouped_down_bf16_small_kernel(
    const bf16_t* __restrict__ h, const int32_t* __restrict__ offsets,
    const bf16_t* __restrict__ wd, int E, int N, int K, bf16_t* __restrict__ y) {
    static_assert(DownSmall::THREADS == stream::kStreamThreads, "one launch serves both");
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds_raw[];
    typedef EvenPolicy<DownSmall::BM, 32> Ring;
    int mt[2];
    count_mtiles<stream::Split, Ring>(offsets, E, mt);
    const int streams = __builtin_amdgcn_readfirstlane(mt[0]);
    const int NT = (N + DownSmall::BN_OUT - 1) / DownSmall::BN_OUT;
    TileLoc t;
    if (stream::stream_few(streams, N))
        stream::stream_tiles(lds_raw, h, offsets, wd, E, N, K, y, streams);
    else if (locate<Ring, From::counted>(offsets, E, NT, blockIdx.x, mt[1], t))
        pipe_tile<DownSmall>(lds_raw, t, h, wd, nullptr, N, K, y, nullptr, 1, false);
}

// Down projection from tens of rows per expert on: 128-row tiles, or 192-row ones if the chip then
// needs fewer rounds (launch_expert_down_bf16_mid).
typedef PipeCfg<128, 128, 64, 4, 2, 4, false> DownMid;
typedef PipeCfg<192, 128, 64, 4, 2, 4, false> DownTall;

__global__ __launch_bounds__(DownTall::THREADS) void grouped_down_bf16_mid_kernel(
    const bf16_t* __restrict__ h, const int32_t* __restrict__ offsets,
    const bf16_t* __restrict__ wd, int E, int N, int K, bf16_t* __restrict__ y, int group) {
    static_assert(DownTall::THREADS == DownMid::THREADS && DownTall::BN_OUT == DownMid::BN_OUT,
                  "one launch serves both");
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds_raw[];
    typedef EvenPolicy<DownMid::BM, 32> Mid;
    typedef EvenPolicy<DownTall::BM, 32> Tall;
    const int NT = (N + DownMid::BN_OUT - 1) / DownMid::BN_OUT;
    int mt[2];
    count_mtiles<Mid, Tall>(offsets, E, mt);
    TileLoc t;
    if (tile_rounds(mt[1], NT) < tile_rounds(mt[0], NT)) {
        if (locate<Tall, From::counted>(offsets, E, NT, blockIdx.x, mt[1], t, group))
            pipe_tile<DownTall>(lds_raw, t, h, wd, nullptr, N, K, y, nullptr, 1, false);
    } else if (locate<Mid, From::counted>(offsets, E, NT, blockIdx.x, mt[0], t, group)) {
        pipe_tile<DownMid>(lds_raw, t, h, wd, nullptr, N, K, y, nullptr, 1, false);
    }
}

// Down projection of contractions of a few dozen stages: persistent tiles, wide ones or low and narrow ones, or the two
// forms above, one tile after the other (launch_expert_down_bf16_short).  kCus workgroups; E <= 64.
typedef PersistCfg<160, 256, 3, false> DownWide;
typedef PersistCfg<64, 128, 6, false> DownLow;
constexpr size_t kDownShortLds = DownTall::LDS_BYTES > DownWide::LDS_BYTES ? DownTall::LDS_BYTES : DownWide::LDS_BYTES;

__global__ __launch_bounds__(DownTall::THREADS) void grouped_down_bf16_short_kernel(
    const bf16_t* __restrict__ h, const int32_t* __restrict__ offsets,
    const bf16_t* __restrict__ wd, int E, int N, int K, bf16_t* __restrict__ y, int group, int stream_out) {
    static_assert(DownTall::THREADS == DownWide::THREADS && DownTall::THREADS == DownLow::THREADS &&
                      kDownShortLds >= DownLow::LDS_BYTES && kDownShortLds >= DownMid::LDS_BYTES,
                  "one launch serves all");
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds_raw[];
    typedef EvenPolicy<DownMid::BM, 32> Mid;
    typedef EvenPolicy<DownTall::BM, 32> Tall;
    typedef EvenPolicy<DownLow::BM, 16> Low;
    typedef EvenPolicy<DownWide::BM, 16> Wide;
    const int NT = (N + DownMid::BN_OUT - 1) / DownMid::BN_OUT, NW = (N + DownWide::BN_OUT - 1) / DownWide::BN_OUT;
    const ExpertRows experts(offsets, E);
    const int mid = experts.mtiles<Mid>(), tall = experts.mtiles<Tall>(), low = experts.mtiles<Low>();
    const bool taller = tile_rounds(tall, NT) < tile_rounds(mid, NT);
    const int mt = taller ? tall : mid;
    // what a form takes, in parts of a tile's time: seven tenths by its rounds and three by its tiles
    auto cost = [](int tile, int mt, int nt) -> long long {
        return tile * (7ll * kCus * tile_rounds(mt, nt) + 3ll * mt * nt);
    };
    const long long wide_cost = cost(40, experts.mtiles<Wide>(), NW), mid_cost = cost(27, mt, NT);
    const long long low_cost = tile_rounds(low, NT) > 1 && 4 * low <= 5 * mt ? cost(20, low, NT) : mid_cost;
    if (wide_cost <= min(mid_cost, low_cost)) {
        persist_tiles<DownWide, false, false>(lds_raw, experts, h, wd, nullptr, N, K, y, nullptr, 1, stream_out, 0);
    } else if (low_cost < mid_cost) {
        persist_tiles<DownLow, false, false>(lds_raw, experts, h, wd, nullptr, N, K, y, nullptr, 1, stream_out, 0);
    } else {
        TileLoc t;
        for (unsigned at = blockIdx.x;; at += kCus) {
            if (!(taller ? locate<Tall, From::counted>(offsets, E, NT, at, mt, t, group)
                         : locate<Mid, From::counted>(offsets, E, NT, at, mt, t, group)))
                break;
            if (taller) pipe_tile<DownTall>(lds_raw, t, h, wd, nullptr, N, K, y, nullptr, 1, false);
            else pipe_tile<DownMid>(lds_raw, t, h, wd, nullptr, N, K, y, nullptr, 1, false);
            __syncthreads();                       // the next tile's loads overwrite the LDS
        }
    }
}

// Gate/up on row-major operands: the ring above with 128-row tiles, the 192-row tiles of pipe16_tile.h, or persistent
// tiles (launch_expert_up_bf16_ring_or_mid).  PERSIST: kCus workgroups, E <= 64; otherwise a workgroup for each tile.
typedef PipeCfg<128, 128, 64, 4, 4, 2, true> UpRing;
typedef PipeCfg<192, 256, 32, 4, 2, 4, true> UpMid;
typedef PersistCfg<160, 256, 3, true> UpWide;
typedef PersistCfg<64, 128, 6, true> UpLow;
enum class Persist { no, whole, halves };
template <Persist PERSIST>
constexpr size_t kUpLds = PERSIST == Persist::no || UpRing::LDS_BYTES > UpWide::LDS_BYTES ? UpRing::LDS_BYTES
                                                                                         : UpWide::LDS_BYTES;

template <Persist PERSIST, bool GATHER>
__global__ __launch_bounds__(UpRing::THREADS) void grouped_up_bf16_kernel(
    const bf16_t* __restrict__ A, const int32_t* __restrict__ offsets,
    const bf16_t* __restrict__ wg, const bf16_t* __restrict__ wu, int E, int N, int K,
    bf16_t* __restrict__ h, const int32_t* __restrict__ row_src, int topk, int mid_if_less,
    int mid_if_equal, int group, int wide_group, int stream_out) {
    static_assert(UpRing::THREADS == UpMid::THREADS && UpRing::LDS_BYTES >= UpMid::LDS_BYTES &&
                      UpRing::THREADS == UpWide::THREADS && UpWide::BN_OUT == UpMid::BN_OUT &&
                      UpRing::THREADS == UpLow::THREADS && UpLow::BN_OUT == UpRing::BN_OUT &&
                      UpWide::LDS_BYTES >= UpLow::LDS_BYTES,
                  "one launch serves all");
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds_raw[];
    typedef EvenPolicy<UpRing::BM, 32> Ring;
    typedef EvenPolicy<UpMid::BM, 16> Mid;
    const int NR = (N + UpRing::BN_OUT - 1) / UpRing::BN_OUT;
    const int NM = (N + UpMid::BN_OUT - 1) / UpMid::BN_OUT;
    // every count costs a workgroup two divisions per expert and lane: a form is counted where it may win
    int mt[2] = {0, 0};
    const ExpertRows experts(offsets, PERSIST != Persist::no ? E : 0);
    if constexpr (PERSIST != Persist::no) {
        mt[0] = experts.mtiles<Ring>();
        if (mid_if_less) mt[1] = experts.mtiles<Mid>();
    } else if (mid_if_less) {
        count_mtiles<Ring, Mid>(offsets, E, mt);
    } else {
        int ring[1];
        count_mtiles<Ring>(offsets, E, ring);
        mt[0] = ring[0];
    }
    bool mid = false;
    if (mid_if_less) {
        const int ring_rounds = tile_rounds(mt[0], NR), mid_rounds = 2 * tile_rounds(mt[1], NM);
        mid = mid_rounds < ring_rounds || (mid_rounds == ring_rounds && mid_if_equal);
    }
    // contractions below 4096: a second round of ring tiles that is at most half full
    const long long tiles = (long long)__builtin_amdgcn_readfirstlane(mt[0]) * NR;
    if (!mid && K < 4096 && tiles > kCus && 2 * tiles <= 3 * kCus) {
        if constexpr (PERSIST != Persist::no) {
            mt[1] = experts.mtiles<Mid>();
        } else {
            int one[1];
            count_mtiles<Mid>(offsets, E, one);
            mt[1] = one[0];
        }
        const long long mid_tiles = (long long)__builtin_amdgcn_readfirstlane(mt[1]) * NM;
        mid = mid_tiles <= kCus && 2 * mid_tiles >= kCus;
    }
    if constexpr (PERSIST != Persist::no) {
        if (tiles > kCus) {
            typedef EvenPolicy<UpWide::BM, 16> Wide;
            typedef EvenPolicy<UpLow::BM, 16> Low;
            // a round's time: wide 20, mid 26, low 9, ring 12 in short contractions and 10 in long ones
            constexpr int kRing = PERSIST == Persist::whole ? 12 : 10;
            const int wide = experts.mtiles<Wide>(), low = PERSIST == Persist::whole && !mid ? experts.mtiles<Low>() : 0;
            const int other = mid ? 26 * tile_rounds(mt[1], NM) : kRing * tile_rounds(mt[0], NR);
            const int low_cost = low > 0 && 4 * low <= 5 * mt[0] ? 9 * tile_rounds(low, NR) : other;
            const bool fills = PERSIST == Persist::whole || (long long)wide * NM >= kCus;
            if (fills && 20 * tile_rounds(wide, NM) <= min(low_cost, other)) {
                persist_tiles<UpWide, GATHER, PERSIST == Persist::halves>(lds_raw, experts, A, wg, wu, N, K, h, row_src,
                                                                          topk, stream_out, wide_group);
                return;
            }
            if (PERSIST == Persist::whole && low_cost < other) {
                persist_tiles<UpLow, GATHER, false>(lds_raw, experts, A, wg, wu, N, K, h, row_src, topk, stream_out, 0);
                return;
            }
        }
    }
    TileLoc t;
    for (unsigned at = blockIdx.x;; at += kCus) {
        if (!(mid ? locate<Mid, From::counted>(offsets, E, NM, at, mt[1], t, group)
                  : locate<Ring, From::counted>(offsets, E, NR, at, mt[0], t, group)))
            break;
        if (mid) pipe16_tile<UpMid>(lds_raw, t, A, wg, wu, N, K, h, row_src, topk, stream_out);
        else pipe_tile<UpRing>(lds_raw, t, A, wg, wu, N, K, h, row_src, topk, stream_out);
        if (PERSIST == Persist::no) break;         // a workgroup for each tile
        __syncthreads();                           // the next tile's loads overwrite the LDS
    }
}

template <Persist PERSIST, bool GATHER>
hipError_t launch_up(unsigned grid, const bf16_t* A, const int32_t* offsets, const bf16_t* wg, const bf16_t* wu, int E,
                     int N, int K, bf16_t* h, const int32_t* row_src, int topk, int mid_if_less, int mid_if_equal,
                     int group, int wide_group, int stream_out, hipStream_t s) {
    // one-time, thread-safe (C++11 static initialisation): raise the dynamic LDS limit
    static const hipError_t attr = hipFuncSetAttribute(
        reinterpret_cast<const void*>(&grouped_up_bf16_kernel<PERSIST, GATHER>),
        hipFuncAttributeMaxDynamicSharedMemorySize, (int)kUpLds<PERSIST>);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL((grouped_up_bf16_kernel<PERSIST, GATHER>), dim3(PERSIST == Persist::no ? grid : kCus),
                       dim3(UpRing::THREADS), kUpLds<PERSIST>, s, A, offsets, wg, wu, E, N, K, h, row_src, topk,
                       mid_if_less, mid_if_equal, group, wide_group, stream_out);
    return hipGetLastError();
}

}  // namespace

// Gate/up on row-major operands, up to 192 rows per expert.
//  - ring: 128 x 128 tiles (64 gate and 64 up rows), 128-byte rows per step (BK = 64; 64-byte rows lose
//    ~10 % of HBM throughput), 4-stage ring of 128 KB, 8 wavefronts, one workgroup per CU.
//  - mid: 192-row tiles of 128 gate and 128 up rows, twice the weights per workgroup, so about twice the
//    time, in half lines.
//  - persistent tiles of 160 rows and 128 outputs (persist_tile.h), for up to 64 experts and contractions below 4096, or
//    longer ones with two rounds of them when every expert has one (those with the tile order in groups and the last round in
//    halves).  Where their rounds, 20 each, cost no more than those of the ring (12, or 10 in long contractions) or of mid (26), and
//    in long contractions they fill the chip once (8 x 4096 x 14336, one token, 224 tiles 90 / 94; 7 tokens at 12 a ring round 275 / 285).  us, the ring or
//    mid / persistent (rounds: persistent, ring, mid): 64 x 2048 x 1408, 6 rows 140 / 126 (2.8, 5.5, 2.8), the same on 37 experts 90 / 84
//    (1.6, 3.2, 1.6), 30 rows on 16 experts 64 / 46 (0.9, 2.1, 0.9), 120 rows 182 / 153 (2.8, 6.8, 2.8), under an exponent of 1.1 202 / 188
//    (4.2, 9.4, 3.9), but 90 rows on 24 experts 102 / 116 (2.1, 5.1, 1.9); 24 x 3840 x 1920, 107 rows on 16 of them 116 / 159 (1.4, 3.8, 0.9);
//    16 x 2048 x 3072, 150 rows 115 / 95 (1.9, 6.0, 1.5); 16 x 5120 x 8192, 6 rows 455 / 439 (4, 8, 4), 75 rows on four experts 260 / 285 (2.3, 6, 2); 8 x
//    4096 x 14336, 83 rows under an exponent of 1.1 392 / 334 (3.9, 8.8, 3.9), on two experts 184 / 217 (2.6, 5.3, 1.8).
//  - low: persistent tiles of 64 rows and 64 outputs (9 a round), for contractions below 4096 with more than one round of
//    ring tiles, where they are at most 5/4 as many: 64 x 2048 x 1408, 12 rows on 24 experts 62 / 58 (2.1 and 2.4 rounds),
//    16 x 2048 x 3072, 12 rows under an exponent of 1.1 69 / 63 (2.6, 2.8).
// Where persistent tiles may be chosen, the launch has one workgroup per CU, which takes the other kinds' tiles one after the
// other: surplus workgroups would each cost the CU 1 to 2 us behind the last tile.
// The ring is ahead of mid unless its smaller tiles take more rounds of the chip than twice the mid tiles.
// How many a batch takes depends on how its rows are spread: the draft model routes everything to a
// few experts.  Measured, us, ring / mid (rounds): 4096 x 14336, 8 experts, 70 rows each 335 (7) / 381 (4),
// the same rows on two experts 219 (6) / 174 (2); 5120 x 8192, 16 experts, 70 rows under a Zipf exponent of 0.5
// 590 (9) / 555 (4); 2048 x 1408, 64 experts, 70 rows, exponent 1.1 169 (8) / 196 (4).
// At equal rounds mid is ahead only for long contractions from about 88 rows on (5120 x 8192, 16
// experts: 92 rows 550 / 530, 110 rows 575 / 546; 52 rows 490 / 502), and where a short one leaves the
// ring's second round at most half full (2048 x 1408, 16 of 64 experts active, 40 rows each: 43 / 33).
// The tile order goes by groups of n-tiles (tile_map.h) from 48 ring tiles per expert: with 1536 in all (six rounds of the
// chip) from 48 rows on, with fewer from 96.  Expert-major / in groups of 8 (4 below 96), us, means over three
// seeds, under an exponent of 1.1, of 0.5 and even: 16 x 5120 x 8192, 50 rows 530 / 515, 516 / 484, 482 / 479, 100 rows 664 / 614, 636 / 604, 544 /
// 539; 8 x 4096 x 14336, 64 rows 364 / 344, 361 / 324, 343 / 317; 16 x 4096 x 4096, 100 rows 278 / 253, 226 / 225, 212 / 207.  With fewer
// tiles and rows an even batch reads the token rows on more dies for nothing (16 x 2048 x 3072, 50 rows 82 / 79, 70 / 72, 73 / 80, 100
// rows 104 / 100, 100 / 97, 89 / 90; 12 x 2048 x 6144, 50 rows 106 / 110, 107 / 110, 113 / 120, 180 rows 189 / 182, 171 / 159, 165 / 161).
// With fewer tiles per expert it loses as often: 64 x 2048 x 1408, 94 rows 193 / 198.
// Below 60 rows per expert a mid tile of a hot expert outlasts the round it saves (4096 x 8192, 8 experts,
// 52 rows, exponent 1.1: 201 / 254).
hipError_t launch_expert_up_bf16_ring_or_mid(const bf16_t* x_perm, const int32_t* offsets,
                                             const bf16_t* wg, const bf16_t* wu, int n_rows, int d,
                                             int f, int E, bf16_t* h, hipStream_t s,
                                             const int32_t* row_src, int topk) {
    const int mid_if_less = (long long)n_rows >= 60ll * E;
    const int mid_if_equal = d >= 4096 && (long long)n_rows >= 88ll * E;
    const long long NR = (f + UpRing::BN_OUT - 1) / UpRing::BN_OUT, NW = (f + UpWide::BN_OUT - 1) / UpWide::BN_OUT;
    const int min_rows = E * NR >= 1536 ? 48 : 96;
    const int group = (long long)n_rows < (long long)min_rows * E ? 0 : NR >= 96 ? 8 : NR >= 48 ? 4 : 0;
    const unsigned grid = (unsigned)grid_upper_bound(n_rows, E, UpRing::BM, NR);
    auto up = [&](auto persist, auto gather) {
        constexpr Persist P = decltype(persist)::value;
        return launch_up<P, decltype(gather)::value>(grid, x_perm, offsets, wg, wu, E, f, d, h, row_src, topk,
                                                     mid_if_less, mid_if_equal, group,
                                                     P == Persist::halves && NW >= 24 ? 8 : 0,   // as tile_group()
                                                     (int)streams_output(n_rows, f), s);
    };
    const std::integral_constant<Persist, Persist::whole> whole;
    const std::integral_constant<Persist, Persist::halves> halves;
    // wide tiles need two rounds of ring tiles or more to be chosen; an expert that is met has a row
    const long long most = (n_rows < E ? n_rows : E) + n_rows / UpRing::BM;
    if (most * NR <= kCus) return up(std::integral_constant<Persist, Persist::no>{}, std::false_type{});
    if (E <= kWave && d < kTailMinK) return row_src ? up(whole, std::true_type{}) : up(whole, std::false_type{});
    if (E <= kWave && E * NW >= 2 * kCus) return row_src ? up(halves, std::true_type{}) : up(halves, std::false_type{});
    return up(std::integral_constant<Persist, Persist::no>{}, std::false_type{});
}

// Down projection with few rows per expert and a long contraction: the weights stream from HBM
// once and nothing else matters.  64-row tiles, 6-stage ring (~120 KB in flight per CU), or the
// private streams where few experts are active.
hipError_t launch_expert_down_bf16_small(const bf16_t* h, const int32_t* offsets,
                                         const bf16_t* wd, int n_rows, int d, int f, int E,
                                         bf16_t* y, hipStream_t s) {
    // one-time, thread-safe (C++11 static initialisation): raise the dynamic LDS limit
    static const hipError_t attr = hipFuncSetAttribute(
        reinterpret_cast<const void*>(&grouped_down_bf16_small_kernel),
        hipFuncAttributeMaxDynamicSharedMemorySize, (int)kDownSmallLds);
    if (attr != hipSuccess) return attr;
    const long long NT = (d + DownSmall::BN_OUT - 1) / DownSmall::BN_OUT;
    const long long tiles = grid_upper_bound(n_rows, E, DownSmall::BM, NT);
    const long long grid = tiles > kCus ? tiles : kCus;
    hipLaunchKernelGGL(grouped_down_bf16_small_kernel, dim3((unsigned)grid),
                       dim3(DownSmall::THREADS), kDownSmallLds, s, h, offsets, wd, E, d, f, y);
    return hipGetLastError();
}

// In between (tens to a few hundred rows per expert), down projection: still bound by streaming the
// weights, but 64-row tiles would re-read them several times through L2.  128-byte rows per step, 4-stage
// ring, tiles of up to 128 or 192 rows, one workgroup per CU.  A workgroup's time hardly depends on its
// rows, so the form with fewer rounds of the chip is ahead, and how many a batch takes depends on how
// its rows are spread, which only the device knows.  Measured, us, 128 / 192 rows (rounds): 12 experts x
// 2048 x 3072, 130 rows each 59 (2) / 44 (1); 4096 x 14336, 8 experts, 120 rows 301 (2) / 198 (1), two
// active with 440 rows each 112 (1) / 128 (1), under a Zipf exponent of 1.1 253 (2) / 296 (2).
// Tile order by groups of four n-tiles (tile_map.h) where the weight tiles take more than one round of the chip.  us,
// contraction x outputs, expert-major / in groups (means over three seeds), under an exponent of 1.1, of 0.5 and even: 64 experts x 1408 x
// 2048, 180 rows 138 / 131, 125 / 124, 120 / 117; 16 x 8192 x 5120, 100 rows 272 / 277, 270 / 267, 272 / 266, 180 rows 392 / 356, 373 / 356,
// 328 / 328; 20 x 3072 x 4096, 180 rows 151 / 145, 154 / 140, 150 / 142.  With 256 weight tiles or fewer an even batch reads
// the rows of h on more dies for nothing (16 x 4096 x 2048, 62 rows 76 / 70, 66 / 71, 61 / 73; 8 x 14336 x 4096, 100 rows 257 / 233, 195 / 199,
// 177 / 179).
constexpr int kDownGroup = 4;

hipError_t launch_expert_down_bf16_mid(const bf16_t* h, const int32_t* offsets, const bf16_t* wd,
                                       int n_rows, int d, int f, int E, bf16_t* y,
                                       hipStream_t s) {
    // one-time, thread-safe (C++11 static initialisation): raise the dynamic LDS limit
    static const hipError_t attr = hipFuncSetAttribute(
        reinterpret_cast<const void*>(&grouped_down_bf16_mid_kernel),
        hipFuncAttributeMaxDynamicSharedMemorySize, (int)DownTall::LDS_BYTES);
    if (attr != hipSuccess) return attr;
    const long long NT = (d + DownMid::BN_OUT - 1) / DownMid::BN_OUT;
    const long long grid = grid_upper_bound(n_rows, E, DownMid::BM, NT);
    hipLaunchKernelGGL(grouped_down_bf16_mid_kernel, dim3((unsigned)grid), dim3(DownTall::THREADS),
                       DownTall::LDS_BYTES, s, h, offsets, wd, E, d, f, y, E * NT > kCus ? kDownGroup : 0);
    return hipGetLastError();
}

// Contractions of 1280 to 4095, up to 64 experts: the time is mostly that of the rounds of the chip, and how many the batch
// takes is known on the device only.  Wide persistent tiles, low ones (their six stages keep more in flight, and the next
// tile's first stages are under way in the unfinished round) where these are at most 5/4 as many as the 128- or 192-row
// ones, or the mid kernel's, by the least cost: 40, 20 and 27 for a tile's time, seven tenths of it by the rounds and three by
// the tiles, as the CUs that have a tile less leave the others their share of the memory.
// Measured, us, weights out of HBM, register-staged (grouped_swiglu_bf16.hip; *: the mid kernel, which the size took
// before) / wide / mid or tall / low (rounds; the one chosen first):
//   64 x 1408 x 2048      6 rows, 64 experts active   77 / 60 (2.0) / 67 (4.0) / 59 (4.0)    wide
//                         6 rows, 37 active           45 / 51 (1.2) / 48 (2.3) / 45 (2.3)    low
//                         12 rows, 38 active          44 / 54 (1.2) / 48 (2.4) / 43 (2.6)    low
//                         30 rows, 55 active          75 / 62 (1.8) / 67 (3.6) / 68 (4.5)    wide
//                         30 rows, 32 active          58 / 56 (1.1) / 48 (2.2) / 54 (3.1)    tall
//                         45 rows, 12 active          52 / 33 (0.7) / 36 (1.2) / 57 (3.2)    wide
//                         120 rows, even              100* / 74 (2.0) / 100 (4.0) / 124      wide
//                         120 rows, exponent of 1.1   108* / 107 (3.1) / 105 (5.7) / 144     wide
//   16 x 2048 x 4096      42 rows, exponent of 1.1    75 / 91 (1.1) / 68 (2.1) / 65 (2.6)    low
//                         80 rows                     83 / 61 (1.0) / 64 (2.0) / 75 (4.0)    wide
//                         150 rows                    77* / 91 (1.2) / 75 (2.0) / 112        tall
//   16 x 3072 x 2048      6 rows                      53 / 43 (0.5) / 36 (1.0) / 35 (1.0)    mid
//                         150 rows                    50* / 66 (0.6) / 51 (1.0) / 87         tall
// (mid and tall as launches of their own; one tile after the other they are up to 7 % slower.)  The choice against the kernel that
// the size took before, 352 batches of 6 shapes, 1 to 1800 tokens, even, skewed and on 2 to 48 experts: 0.83 times the time
// on average; twelve of them more than 3 % behind, up to 9 % (64 x 1408 x 2048, 6 rows on 37 experts 44 / 45, 8 tokens 39 / 43).
hipError_t launch_expert_down_bf16_short(const bf16_t* h, const int32_t* offsets, const bf16_t* wd, int n_rows, int d,
                                         int f, int E, bf16_t* y, hipStream_t s) {
    // one-time, thread-safe (C++11 static initialisation): raise the dynamic LDS limit
    static const hipError_t attr = hipFuncSetAttribute(
        reinterpret_cast<const void*>(&grouped_down_bf16_short_kernel),
        hipFuncAttributeMaxDynamicSharedMemorySize, (int)kDownShortLds);
    if (attr != hipSuccess) return attr;
    const long long NT = (d + DownMid::BN_OUT - 1) / DownMid::BN_OUT;
    hipLaunchKernelGGL(grouped_down_bf16_short_kernel, dim3(kCus), dim3(DownTall::THREADS), kDownShortLds, s, h, offsets,
                       wd, E, d, f, y, E * NT > kCus ? kDownGroup : 0, (int)streams_output(n_rows, d));
    return hipGetLastError();
}

}  // namespace specmoe
