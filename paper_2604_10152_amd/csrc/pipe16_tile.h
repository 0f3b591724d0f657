// Large- and mid-batch expert GEMMs (tiles of up to 320 or 192 rows), v_mfma_f32_16x16x32_bf16
// flavour of the pipelined kernel.
// (SpecMoE Sec. 2.1 / 2.2: the rows routed to an expert meet its FFN-sized weights; at
// verification time each expert sees hundreds of rows, so the contraction is MFMA-bound.)
//
// Same data movement as grouped_gemm_bf16_pipe.hip (global->LDS ring of BK = 32 stages),
// different matrix instruction: one 16x16x32 MFMA consumes a whole 64-byte tile row per lane,
// so a stage is ONE k-step.
// Why this shape: under the chip's power limit the 16x16x32 instruction sustains more bf16
// flops than 32x32x16 on the same operands (2.1 vs 1.8 PFLOP/s measured in a register-only
// loop with changing operands), and its 16-row granule wastes fewer matrix instructions on
// the ragged last rows of an expert.
//
// Loop schedule: ping-pong.  The two waves of a SIMD alternate between multiplying a k-step
// out of registers and loading / reading the next one.
//
// Operands may be tile-packed (pipe_common.h: 1 KB blocks of 16 rows x 32 columns that hold the
// LDS image of the piece).  A wave-load then reads 1 KB of consecutive memory, i.e. whole
// 128-byte lines, instead of sixteen 64-byte half lines of sixteen rows; the L2 serves requests,
// not bytes, and the kernel is bound by that request rate (row-major operands: 852 / 427 us
// for the gate/up / down projection of the 2048-token Mixtral-shaped layer, both operands packed:
// 788 / 380 us in the same harness).  PA: activations packed (the down projection's h, written
// packed by the gate/up kernel: PO); PB: weights packed (moe_pack_weights).
#pragma once
#include "pipe_common.h"

#include <type_traits>
#include <utility>

namespace specmoe {
namespace pipe {

template <typename F, int... Is>
__device__ __forceinline__ void dispatch_count(int n, F& f, std::integer_sequence<int, Is...>) {
    ((n == Is ? (f(std::integral_constant<int, Is>{}), 0) : 0), ...);
}

// What a lane holds of a 16 x 16 sub-tile: one row and 4 consecutive columns, as bf16.  acc: the
// wave's sub-tiles of these rows; SwiGLU: the second half of them are the `up` columns.
template <bool SWIGLU, int TN>
__device__ __forceinline__ uint2 sub_tile(const floatx4 (&acc)[TN], int j) {
    float v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        v[q] = acc[j][q];
        if constexpr (SWIGLU) v[q] = v[q] * __builtin_amdgcn_rcpf(1.0f + __expf(-v[q])) * acc[j + TN / 2][q];
    }
    return make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
}

// A wave's sub-tiles straight to global memory (acc[i]: tile rows 16 * (wm + WM * i) ..; PO: tile-packed).  Lanes l and
// l ^ 16 exchange halves of two sub-tiles (neighbours in columns, or in rows where a wave has one column of them),
// so a lane stores 16 bytes: a packed block of 1 KB, or 64 bytes of 16 rows, by one instruction.
template <int TA, int WM, bool SWIGLU, bool PO, int TAX, int TN>
__device__ __forceinline__ void write_sub_tiles(const floatx4 (&acc)[TAX][TN], const TileLoc& t, int n0, int N,
                                                bf16_t* __restrict__ Cout, int wm, int wn, bool stream_out) {
    constexpr int JN = SWIGLU ? TN / 2 : TN;
    const int lane = threadIdx.x % kWave, mrow = lane & 15, cq = (lane >> 4) * 4;
    const int odd = (lane >> 4) & 1, c8 = (lane >> 5) * 8;
    // Row mrow of sub-tile i, `at` columns behind column `col` of the tile: the address is a uniform base and a
    // lane's offset that is the same for all sub-tiles.  Columns go on for N, a multiple of 64.
    auto lane_offset = [&](int at) __attribute__((always_inline)) -> uint32_t {
        return PO ? (uint32_t)((4 * mrow + ((at >> 3) ^ ((mrow >> 1) & 3))) * 16 + (at & 4) * 2)
                  : (uint32_t)(mrow * N + at) * 2u;
    };
    auto store = [&](auto v, int i, int col, uint32_t offset, int trow) __attribute__((always_inline)) {
        if (n0 + col >= N) return;
        const int sub = wm + WM * i;
        unsigned char* base = reinterpret_cast<unsigned char*>(
            Cout + (PO ? (size_t)(t.blk0 + sub) * 16 * N + (size_t)((n0 + col) / 32) * 512
                       : (size_t)(t.row0 + 16 * sub) * N + n0 + col));
        if (PO) {
            // rows beyond the tile's last one (padding of the expert's last block) are zeros
            if (trow >= t.tile_rows) v = decltype(v){};
        } else if (trow >= t.tile_rows) {
            return;
        }
        if constexpr (sizeof(v) == 16) store16(stream_out, base, offset, v);
        else *reinterpret_cast<decltype(v)*>(base + offset) = v;
    };
    auto exchange = [&](uint2 a, uint2 b) __attribute__((always_inline)) -> U128 {
        lane_swap<16>(a.x, b.x);
        lane_swap<16>(a.y, b.y);
        return U128{a.x, a.y, b.x, b.y};           // 8 columns of a (even lanes) or of b (odd ones)
    };
    if constexpr (JN % 2 == 0) {
        const uint32_t offset = lane_offset(16 * odd + c8);
#pragma unroll
        for (int i = 0; i < TA; ++i)
#pragma unroll
            for (int j = 0; j < JN; j += 2)
                store(exchange(sub_tile<SWIGLU>(acc[i], j), sub_tile<SWIGLU>(acc[i], j + 1)), i,
                      16 * (wn * JN + j), offset, 16 * (wm + WM * i) + mrow);
    } else {
        static_assert(JN == 1, "sub-tiles pair up in columns or in rows");
        // odd lanes: the next sub-tile's rows.  A packed block has 32 columns, the wave 16 of them.
        const int col = PO ? 32 * (wn / 2) : 16 * wn, in_block = PO ? 16 * (wn & 1) : 0;
        const uint32_t offset = lane_offset(in_block + c8) + (uint32_t)odd * (32u * WM) * (uint32_t)N;
#pragma unroll
        for (int i = 0; i + 1 < TA; i += 2)
            store(exchange(sub_tile<SWIGLU>(acc[i], 0), sub_tile<SWIGLU>(acc[i + 1], 0)), i, col, offset,
                  16 * (wm + WM * (i + odd)) + mrow);
        if constexpr (TA % 2 == 1) {
            typedef uint32_t U64 __attribute__((ext_vector_type(2)));
            const uint2 v = sub_tile<SWIGLU>(acc[TA - 1], 0);
            store(U64{v.x, v.y}, TA - 1, col, lane_offset(in_block + cq), 16 * (wm + WM * (TA - 1)) + mrow);
        }
    }
}

// the work of one workgroup: tile t (lds_raw: C::LDS_BYTES)
template <typename C, bool PA = false, bool PB = false, bool PO = false>
__device__ __forceinline__ void pipe16_tile(
    unsigned char* lds_raw, const TileLoc& t,
    const bf16_t* __restrict__ A,        // [n_rows, K]
    const bf16_t* __restrict__ W0,       // [E, N, K]   (gate, or down)
    const bf16_t* __restrict__ W1,       // [E, N, K]   (up; SWIGLU only)
    int N, int K, bf16_t* __restrict__ Cout /* [n_rows, N] */,
    const int32_t* __restrict__ row_src /* nullable: A row r is A[row_src[r] / topk] */, int topk,
    bool stream_out /* streams_output() */) {
    static_assert(C::BK == 32, "a stage is exactly one 16x16x32 k-step");
    constexpr int TM16 = C::BM / (16 * C::WM);       // 16-row A sub-tiles per wave
    constexpr int TN16 = C::BN / (16 * C::WN);       // 16-col B sub-tiles per wave
    constexpr int A_SUB_BYTES = 16 * C::WM * C::ROW_BYTES;   // LDS distance of consecutive i
    static_assert(!C::SWIGLU || TN16 % 2 == 0, "gate and up sub-tiles pair up inside a wave");
    static_assert((16 * C::WM) % (C::RPG * C::CHUNKS) == 0, "sub-tile step must keep the swizzle");

    const int row0 = t.row0, tile_rows = t.tile_rows;
    const int n0 = t.nt * C::BN_OUT;
    const int nsub = (tile_rows + 15) / 16;

    const int tid = threadIdx.x, lane = tid % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    // waves w and w+4 share a SIMD: different wm keeps an odd sub-tile count balanced
    const int wm = wave / C::WN, wn = wave % C::WN;
    const uint32_t lds_base =
        (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds_raw;

    // ---- global side of the wave-loads (identical to the 32x32 kernel) --------------------
    // with row_src the activation rows are gathered on the fly (A is then the token matrix)
    // tile-packed operands: row block rb (16 rows) of a matrix with K columns starts at element
    // rb * 16 * K, its k-step kt at + kt * 512 (one 1 KB block)
    const unsigned char* a_base = uniform_ptr(reinterpret_cast<const unsigned char*>(
        A + (PA ? (size_t)t.blk0 * 16 * K : (row_src ? (size_t)0 : (size_t)row0 * K))));
    const size_t wrow = (size_t)t.expert * N + min(n0, N - 1);      // packed: a multiple of 16
    const unsigned char* w0 = uniform_ptr(reinterpret_cast<const unsigned char*>(W0 + wrow * K));
    const unsigned char* w1 =
        C::SWIGLU ? uniform_ptr(reinterpret_cast<const unsigned char*>(W1 + wrow * K)) : nullptr;
    const int n_left = N - n0;
    constexpr uint32_t A_KSTEP = PA ? 1024u : (uint32_t)C::ROW_BYTES;   // bytes per k-step
    constexpr uint32_t B_KSTEP = PB ? 1024u : (uint32_t)C::ROW_BYTES;
    uint32_t a_off[C::A_PW], b_off[C::B_PW];
    int a_cnt = 0;                               // A wave-loads this wave issues per stage
    {
        const int srow = lane / C::CHUNKS, pc = lane % C::CHUNKS;   // LDS slot of this lane
#pragma unroll
        for (int jj = 0; jj < C::A_PW; ++jj) {
            const int r = (wave + jj * C::NWAVES) * C::ROWS_PER_DMA + srow;
            const int c = pc ^ ((r / C::RPG) % C::CHUNKS);
            const int rr = min(r, tile_rows - 1);
            if (PA) {
                // wave-load j = row block j of the tile: 1 KB, lane l its l-th 16-byte piece
                const int jb = min(wave + jj * C::NWAVES, (tile_rows + 15) / 16 - 1);
                a_off[jj] = (unsigned)jb * 16u * (unsigned)K * 2u + (unsigned)lane * 16u;
            } else {
                const unsigned arow =
                    row_src ? (unsigned)(row_src[row0 + rr] / topk) : (unsigned)rr;
                a_off[jj] = (arow * (unsigned)K + (unsigned)(c * 8)) * 2u;
            }
            if ((wave + jj * C::NWAVES) * C::ROWS_PER_DMA < tile_rows) a_cnt = jj + 1;
        }
#pragma unroll
        for (int jj = 0; jj < C::B_PW; ++jj) {
            const int r = (wave + jj * C::NWAVES) * C::ROWS_PER_DMA + srow;
            const int c = pc ^ ((r / C::RPG) % C::CHUNKS);
            const int rn = (C::SWIGLU && r >= C::BN / 2) ? r - C::BN / 2 : r;
            if (PB) {
                const int jb = min(rn / 16, n_left / 16 - 1);        // row block of the weight tile
                b_off[jj] = (uint32_t)jb * 16u * (uint32_t)K * 2u + (uint32_t)lane * 16u;
            } else {
                b_off[jj] = (uint32_t)((min(rn, n_left - 1) * K + c * 8) * 2);
            }
        }
    }
    const int KT = K / C::BK;                    // even: the ABI requires K % 64 == 0
    // nt_tag: the weight loads carry the non-temporal hint (tiles whose weights no other
    // workgroup reads)
    auto issue_one = [&](auto nt_tag, int which, int kt, int buf) __attribute__((always_inline)) {
        // the k offset rides in the per-lane offset (one vector add per load); the base
        // pointers stay loop-invariant scalars.  Clamped: the last steps re-load stage KT-1.
        const uint32_t kq = (uint32_t)min(kt, KT - 1);
        const uint32_t ka = kq * A_KSTEP, kb = kq * B_KSTEP;
        const uint32_t sbase = lds_base + (uint32_t)buf * C::STAGE_BYTES + wave * 1024u;
#pragma unroll
        for (int jj = 0; jj < C::A_PW; ++jj)
            if (which == jj && jj < a_cnt)
                dma16(a_base, a_off[jj] + ka, sbase + jj * C::NWAVES * 1024u);
#pragma unroll
        for (int jj = 0; jj < C::B_PW; ++jj) {
            // the gate / up halves split on a round of wave-loads, or inside a round between waves
            const bool up =
                C::SWIGLU &&
                ((C::BN / 2 / C::ROWS_PER_DMA) % C::NWAVES == 0
                     ? jj * C::NWAVES * C::ROWS_PER_DMA >= C::BN / 2
                     : (wave + jj * C::NWAVES) * C::ROWS_PER_DMA >= C::BN / 2);
            if (which == C::A_PW + jj) {
                if (decltype(nt_tag)::value)
                    dma16_nt(up ? w1 : w0, b_off[jj] + kb,
                             sbase + C::A_BYTES + jj * C::NWAVES * 1024u);
                else
                    dma16(up ? w1 : w0, b_off[jj] + kb,
                          sbase + C::A_BYTES + jj * C::NWAVES * 1024u);
            }
        }
    };

    // ---- LDS side: lane l reads row (l%16) of a sub-tile, 16-byte chunk l/16 -----------------
    const int a_rd = swz<C>(16 * wm + (lane & 15), lane >> 4);
    const int b_rd = C::A_BYTES + swz<C>(lane & 15, lane >> 4);
    auto nb = [&](int j) __attribute__((always_inline)) -> int {     // B sub-tile base row
        if (C::SWIGLU) {
            constexpr int H = TN16 / 2;
            return (j < H) ? 16 * (wn * H + j) : C::BN / 2 + 16 * (wn * H + (j - H));
        }
        return 16 * (wn * TN16 + j);
    };

    const int ta = min(TM16, max(0, (nsub - wm + C::WM - 1) / C::WM));   // active A sub-tiles

    // epilogue: row-major SwiGLU tiles are staged in LDS and written as whole rows by the workgroup; tile-packed ones
    // and plain tiles go straight to global memory.  acc[i] is the wave's i-th A sub-tile (tile rows
    // 16 * (wm + WM * i) ..).
    auto epilogue = [&](auto& acc, auto ta_tag) __attribute__((always_inline)) {
        constexpr int TA = decltype(ta_tag)::value;
        wait_vmcnt<0>();                           // no load may outlive the workgroup's LDS
        if constexpr (C::SWIGLU && !PO) {
            constexpr int JN = TN16 / 2;
            __builtin_amdgcn_s_barrier();          // every wave's loads have landed
#pragma unroll
            for (int i = 0; i < TA; ++i)
#pragma unroll
                for (int j = 0; j < JN; ++j)
                    *reinterpret_cast<uint2*>(lds_raw + (16 * (wm + C::WM * i) + (lane & 15)) * kStageRowBytes +
                                              (16 * (wn * JN + j) + (lane >> 4) * 4) * 2) =
                        sub_tile<C::SWIGLU>(acc[i], j);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // the barrier behind does not wait for the writes
        } else {
            write_sub_tiles<TA, C::WM, C::SWIGLU, PO>(acc, t, n0, N, Cout, wm, wn, stream_out);
        }
    };

    // ---- ping-pong schedule ----------------------------------------------------------------
    // The two waves that share a SIMD belong to different groups (wm = 0 / 1) and alternate:
    // while one multiplies a whole k-step out of registers (nothing but matrix instructions),
    // the other issues its wave-loads and reads its next fragments; a barrier, and they swap.
    // The matrix pipe of every SIMD always has exactly one wave feeding it, and fragment reads
    // and load issue never sit between two matrix instructions.  Group 1 runs one phase behind
    // group 0 (one extra barrier up front, group 0 pays it back at the end).
    //   phase 2kt  : group 0 reads stage kt            | group 1 multiplies stage kt-1
    //   phase 2kt+1: group 0 multiplies stage kt       | group 1 reads stage kt
    // Stage kt+3 is requested in the read phase of stage kt (its slot held stage kt-1, which
    // group 1 finished reading one phase earlier); before the barrier that ends phase 2kt+1
    // every wave waits for its share of stage kt+1, so a stage has 4 to 5 phases to land.
    auto run_pp = [&](auto ta_tag, auto nt_tag) __attribute__((always_inline)) {
        static_assert(C::WM == 2 && C::STAGES == 4, "two wave groups, ring of four");
        constexpr int TA = decltype(ta_tag)::value;
        constexpr int TAX = TA > 0 ? TA : 1;
        floatx4 acc[TAX][TN16];
#pragma unroll
        for (int i = 0; i < TA; ++i)
#pragma unroll
            for (int j = 0; j < TN16; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.f;
        bf16x8 af[TAX], bfr[TN16];
        const int allow2 = 2 * (a_cnt + C::B_PW);          // two younger stages may be in flight

        // prologue: stages 0..2 requested, stage 0 landed and visible
#pragma unroll
        for (int s = 0; s < C::STAGES - 1; ++s)
#pragma unroll
            for (int q = 0; q < C::G_MAX; ++q) issue_one(nt_tag, q, s, s);
        wait_vmcnt_dyn(allow2);
        __builtin_amdgcn_s_barrier();
        if (wm == 1) __builtin_amdgcn_s_barrier();         // group 1 sits out phase 0

        int buf = 0;
        for (int kt = 0; kt < KT; ++kt) {
            // ---- read phase
#pragma unroll
            for (int q = 0; q < C::G_MAX; ++q)
                issue_one(nt_tag, q, kt + C::STAGES - 1, (buf + 3) & 3);
            if (TA > 0) {
                const unsigned char* sa = lds_raw + buf * C::STAGE_BYTES + a_rd;
                const unsigned char* sb = lds_raw + buf * C::STAGE_BYTES + b_rd;
#pragma unroll
                for (int j = 0; j < TN16; ++j)
                    bfr[j] = *reinterpret_cast<const bf16x8*>(sb + nb(j) * C::ROW_BYTES);
#pragma unroll
                for (int i = 0; i < TA; ++i)
                    af[i] = *reinterpret_cast<const bf16x8*>(sa + i * A_SUB_BYTES);
            }
            if (wm == 1) wait_vmcnt_dyn(allow2);           // phase 2kt+1 ends: stage kt+1 landed
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);             // nothing moves across the barriers
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
            // ---- multiply phase
#pragma unroll
            for (int i = 0; i < TA; ++i)
#pragma unroll
                for (int j = 0; j < TN16; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[j], af[i], acc[i][j],
                                                                        0, 0, 0);
            if (wm == 0) wait_vmcnt_dyn(allow2);           // phase 2kt+1 ends: stage kt+1 landed
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
            buf = (buf + 1) & 3;
        }
        if (wm == 0) __builtin_amdgcn_s_barrier();         // group 0 waits out group 1's last phase
        epilogue(acc, ta_tag);
    };

    // An expert with a single m-tile: every weight tile of it is read by exactly one workgroup,
    // once - a pure stream out of HBM, which the non-temporal hint speeds up (dma16_nt).
    // With several m-tiles the workgroups that share a weight tile meet
    // in the L2, and the hint would cost those hits.  In gate/up a batch in which some expert has several m-tiles keeps it to
    // tiles of up to 64 rows: us, up to 64 rows / all, 8 x 4096 x 14336, 83 rows each 334 / 314, 125 rows 359 / 336, 16 x 5120 x 8192, 75
    // rows 461 / 421, but 64 x 2048 x 1408, 30 rows under a Zipf exponent of 1.1 115 / 120.
    // Only with tile-packed weights: a wave-load then covers whole 128-byte lines.  Row-major, a
    // BK = 32 stage takes half of every line and the next stage the other half; without
    // allocation in the L2 every line would come out of HBM twice (measured: 363 -> 469 us).
    const bool w_once = PB && t.mt == 1 && (!C::SWIGLU || tile_rows <= 64 || t.single);
    auto run_sel = [&](auto ta_tag) __attribute__((always_inline)) {
        if (w_once) run_pp(ta_tag, std::true_type{});
        else run_pp(ta_tag, std::false_type{});
    };
    dispatch_count(ta, run_sel, std::make_integer_sequence<int, TM16 + 1>{});

    if (C::SWIGLU && !PO) {
        // cooperative write-out of the staged tile: 16 bytes per lane, whole rows
        static_assert(!C::SWIGLU || PO || (size_t)C::BM * kStageRowBytes <= C::LDS_BYTES, "stage tile");
        static_assert(!C::SWIGLU || PO || C::BN_OUT == 128, "stage row pitch assumes 128 columns");
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

}  // namespace pipe
}  // namespace specmoe
