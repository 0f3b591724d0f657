// Down projection of few active experts with few rows each: tiles of at most 32 rows whose four
// waves stream their weights independently of each other (v_mfma_f32_32x32x16_bf16).
// (SpecMoE Sec. 3.2: the draft model keeps as few as two experts of a block, each with the rows
// of a handful of tokens.)
//
// The bound is streaming the weights of the ACTIVE experts out of HBM, and how many those are is
// known on the device only.  The ring of grouped_gemm_bf16_pipe.hip shares a stage of 128 weight
// rows between its waves: two active experts of 4096 x 14336 are then 64 workgroups on 256 CUs
// (90 us, 2.6 TB/s).  Here every wave owns 32 weight rows and a private LDS ring of BK = 64 stages
// (one 128-byte line per row), so no barrier sits in the loop, and the four waves of a workgroup
// split the contraction of one slab of 32 weight rows.  Two slabs with two waves each where that gives
// every CU a workgroup, i.e. at the line below: 8192 outputs, 2 active experts 32 us against 41 with
// one slab (4096 outputs, 4 of them 94 / 90; 4 m-tiles of 2 experts 78 / 84).  The partial sums of
// the waves meet in LDS in wave order (deterministic).
// Measured, down projection of 4096 x 14336, 16 rows per active expert, ring / this: 1 expert 83 /
// 37 us, 2 90 / 47, 3 99 / 79, 4 111 / 91, 6 133 / 146; 5120 x 8192: 1 expert 46 / 26, 2 54 / 48, 4 67 / 89.
// Hence the line at 128 tiles of 32 x 128 (half the CUs): stream_few().
#pragma once
#include "pipe_common.h"

namespace specmoe {
namespace stream {

using namespace pipe;

constexpr int kStreamWaves = 4, kStreamThreads = kStreamWaves * kWave;
constexpr int kBM = 32, kBK = 64, kRowBytes = kBK * 2;
constexpr int kWBytes = 32 * kRowBytes;                     // weight part of a stage (4 KB)
constexpr int kRingBytes = 40 * 1024;                       // LDS of one wave
constexpr size_t kStreamLds = (size_t)kStreamWaves * kRingBytes;
typedef EvenPolicy<kBM, 16> Split;

// chunk c of row r of a 128-byte-row image sits at chunk c ^ ((r / 2) % 8): conflict-free for
// the 32-row fragment reads (pipe_common.h)
__device__ __forceinline__ int stream_swz(int r, int c) {
    return r * kRowBytes + ((c ^ ((r >> 1) & 7)) << 4);
}

// whether a batch of total_mt m-tiles is for the code below: at most half the CUs would get one of
// the ring's 128-row weight tiles
__device__ __forceinline__ bool stream_few(int total_mt, int N) {
    return (long long)total_mt * ((N + 127) / 128) <= kCus / 2;
}

// y = h . w_down^T for the tiles of workgroup blockIdx.x (of gridDim.x, a multiple of kXcds).
// lds: kStreamLds bytes.  K % 64 == 0, N % 64 == 0.
__device__ __forceinline__ void stream_tiles(
    unsigned char* lds, const bf16_t* __restrict__ A, const int32_t* __restrict__ offsets,
    const bf16_t* __restrict__ W, int E, int N, int K, bf16_t* __restrict__ Cout, int total_mt) {
    constexpr int OUT = 32;                                 // weight rows = output columns of a wave
    const int lane = threadIdx.x % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int slabs = N / OUT;                              // of an expert: an even number
    const int KW = (long long)total_mt * (slabs / 2) >= kCus ? 2 : 4;
    const int NW = kStreamWaves / KW, NT = slabs / NW;
    const int wk = wave % KW, wn = wave / KW;
    const long long G = (long long)total_mt * NT;
    const long long per_xcd = (G + kXcds - 1) / kXcds;
    const int KT = K / kBK, steps = (KT - wk + KW - 1) / KW;
    unsigned char* ring = lds + wave * kRingBytes;
    const uint32_t ring_addr =
        (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)ring;

    for (long long slot = blockIdx.x / kXcds; slot < per_xcd;
         slot += gridDim.x / kXcds) {
        const long long L = (long long)(blockIdx.x % kXcds) * per_xcd + slot;
        TileLoc t;
        if (L >= G || !locate<Split, From::place>(offsets, E, NT, L, 0, t)) break;
        const int n0 = (t.nt * NW + wn) * OUT;

        // ---- wave-loads: 8 rows of 128 bytes each; lane -> row lane / 8, LDS chunk lane % 8
        const int srow = lane >> 3, pc = lane & 7;
        const unsigned char* a_base = uniform_ptr(
            reinterpret_cast<const unsigned char*>(A + (size_t)t.row0 * K));
        const size_t wrow = (size_t)t.expert * N + n0;
        const unsigned char* w_base =
            uniform_ptr(reinterpret_cast<const unsigned char*>(W + wrow * K));
        const int a_cnt = (t.tile_rows + 7) / 8;            // wave-loads that hold real rows, 1..4
        uint32_t a_off[4], w_off[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int r = 8 * j + srow, c = pc ^ ((r >> 1) & 7);
            a_off[j] = ((unsigned)min(r, t.tile_rows - 1) * (unsigned)K + (unsigned)(c * 8)) * 2u;
            w_off[j] = ((unsigned)r * (unsigned)K + (unsigned)(c * 8)) * 2u;
        }
        const bool once = t.mt == 1;                        // no other workgroup reads these weights
        const int a_bytes = a_cnt * 1024, stage = kWBytes + a_bytes;
        const int S = min(kRingBytes / stage, steps + 1);   // 8, 6, 5 or 5 stages
        const int per_stage = a_cnt + 4;
        auto issue = [&](int i, int buf) __attribute__((always_inline)) {
            const size_t kb = (size_t)(wk + KW * min(i, steps - 1)) * kRowBytes;   // tail re-loads
            const uint32_t dst = ring_addr + (uint32_t)buf * stage;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (j < a_cnt) dma16(a_base + kb, a_off[j], dst + j * 1024);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (once) dma16_nt(w_base + kb, w_off[j], dst + a_bytes + j * 1024);
                else dma16(w_base + kb, w_off[j], dst + a_bytes + j * 1024);
            }
        };

        // fragment reads: lane l reads row l % 32, chunk 2 * kk + l / 32.  With fewer than 32
        // rows the activation reads run on into the weight part: those rows are not stored.
        int a_rd[4], w_rd[4];
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            a_rd[kk] = stream_swz(lane & 31, kk * 2 + (lane >> 5));
            w_rd[kk] = a_bytes + a_rd[kk];
        }
        floatx16 acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.f;
        for (int i = 0; i < S - 1; ++i) issue(i, i);
        const int allow = (S - 2) * per_stage;
        int buf = 0, free = S - 1;
        for (int i = 0; i < steps; ++i) {
            wait_vmcnt_dyn(allow);                          // stage i has landed (own loads only)
            issue(i + S - 1, free);                         // its slot was read out in step i - 1
            const unsigned char* st = ring + buf * stage;
            bf16x8 af[4], wf[4];
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                wf[kk] = *reinterpret_cast<const bf16x8*>(st + w_rd[kk]);
                af[kk] = *reinterpret_cast<const bf16x8*>(st + a_rd[kk]);
            }
#pragma unroll
            for (int kk = 0; kk < 4; ++kk)
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[kk], af[kk], acc, 0, 0, 0);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // this slot may be overwritten now
            __builtin_amdgcn_sched_barrier(0);
            free = buf;
            buf = buf + 1 == S ? 0 : buf + 1;
        }
        wait_vmcnt<0>();                                    // the tail's re-loads
        {                                                   // partial sums of the KW waves, in order
            floatx4* part = reinterpret_cast<floatx4*>(ring);
            if (wk > 0) {
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    part[g * kWave + lane] =
                        floatx4{acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]};
            }
            __syncthreads();
            if (wk == 0) {
                for (int s = 1; s < KW; ++s) {
                    const floatx4* p = reinterpret_cast<const floatx4*>(ring + s * kRingBytes);
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const floatx4 v = p[g * kWave + lane];
#pragma unroll
                        for (int q = 0; q < 4; ++q) acc[4 * g + q] += v[q];
                    }
                }
            }
            __syncthreads();                                // the rings belong to the next tile
        }
        // a lane holds row l % 32 and weight rows 8 g + 4 (l / 32) + q of the slab
        const int row = lane & 31, ch = (lane >> 5) * 4;
        if (wk == 0 && row < t.tile_rows) {
            bf16_t* crow = Cout + (size_t)(t.row0 + row) * N;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                *reinterpret_cast<uint2*>(crow + n0 + 8 * g + ch) =
                    make_uint2(pack_bf16x2(acc[4 * g], acc[4 * g + 1]),
                               pack_bf16x2(acc[4 * g + 2], acc[4 * g + 3]));
            }
        }
    }
}

}  // namespace stream
}  // namespace specmoe
