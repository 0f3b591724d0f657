// Persistent form of the expert GEMMs, v_mfma_f32_16x16x32_bf16: one workgroup per CU takes its tiles one after the
// other, and the first stages of the next tile are requested under the last k-steps of the present one.
// (SpecMoE Sec. 2.1 / 2.2: experts of a few hundred to a few thousand columns with tens to hundreds of rows
// each at verification time; a tile of such a contraction lives for 20 to 60 microseconds.)
//
// What a tile costs besides its k loop in the other kernels - finding it 1.1 us, the first stage's way out of HBM
// 1.3, the epilogue 1.2, and the time until the next workgroup starts - passes while requests are in flight here.
//
// Row-major operands.  A stage is 64 columns, whole 128-byte lines; S stages in the LDS, of which S - 2 or S - 1 are
// in flight.  Two k-steps per stage, in the ping-pong
// schedule of pipe16_tile.h (s = k-step, q = s / 2 its stage):
//   phase 2s  : group 0 reads step s        | group 1 multiplies step s-1
//   phase 2s+1: group 0 multiplies step s   | group 1 reads step s
// Stage q+S-1 is requested in the read phases of stage q (its slot held stage q-1, which group 1 finished reading one
// phase before), and every wave waits for its share of stage q+1 before the barrier that ends stage q.
#pragma once
#include "pipe16_tile.h"

namespace specmoe {
namespace pipe {

template <int BM_, int BN_, int STAGES_, bool SWIGLU_>
struct PersistCfg {
    static constexpr int BM = BM_, BN = BN_, STAGES = STAGES_, WM = 2, WN = 4;
    static constexpr bool SWIGLU = SWIGLU_;
    static constexpr int BK = 64, KSUB = BK / 32, ROW_BYTES = BK * 2;
    static constexpr int NWAVES = WM * WN, THREADS = NWAVES * kWave;
    static constexpr int TM = BM / (16 * WM), TN = BN / (16 * WN);   // 16 x 16 sub-tiles per wave
    static constexpr int BN_OUT = SWIGLU ? BN / 2 : BN;
    // wave-loads of 1 KB per stage and wave: 8 rows of whole lines
    static constexpr int A_PW = (BM / 8 + NWAVES - 1) / NWAVES;
    static constexpr int B_PW = BN / 8 / NWAVES;
    static constexpr int A_BYTES = BM * ROW_BYTES, STAGE_BYTES = (BM + BN) * ROW_BYTES;
    static constexpr size_t LDS_BYTES = (size_t)STAGES * STAGE_BYTES + (BM + kWave - 1) / kWave * 256;   // row numbers of the next tile
    static_assert(BM % (16 * WM) == 0 && BN % (32 * WN) == 0, "tile");
    static_assert(!SWIGLU || BN / 2 / 8 % NWAVES == 0, "a round of wave-loads is all gate or all up");
    static_assert(STAGES >= 3 && (STAGES - 2) * (A_PW + B_PW) <= 63, "ring depth (vmcnt is 6 bits)");
    static_assert(LDS_BYTES <= 160 * 1024, "LDS");
};

// Up to 64 experts in registers, one per lane: where an expert's rows start and how many it has.
struct ExpertRows {
    int lo, rows;
    __device__ __forceinline__ ExpertRows(const int32_t* __restrict__ offsets, int E) {
        const int e = threadIdx.x % kWave;
        lo = e < E ? offsets[e] : 0;
        rows = e < E ? offsets[e + 1] - lo : 0;
    }
    // m-tiles of all
    template <typename Split>
    __device__ __forceinline__ int mtiles() const {
        return __builtin_amdgcn_readfirstlane(wave_sum(Split::of(rows).mt));
    }
};
// Their tiles.
template <int BM>
struct TileTable {
    int lo, rows, mt, rpt, incl;             // of the lane's expert; incl: m-tiles up to it
    int total;                               // m-tiles of all
    __device__ __forceinline__ TileTable(ExpertRows r) : lo(r.lo), rows(r.rows) {
        const EvenSplit s = even_split<BM, 16>(rows);
        mt = s.mt;
        rpt = s.rpt;
        incl = wave_scan(mt);
        total = __builtin_amdgcn_readlane(incl, kWave - 1);
    }
    // whether every expert that has rows has equally many m-tiles
    __device__ __forceinline__ bool even() const {
        const unsigned long long has = __ballot(mt > 0);
        const int some = __builtin_amdgcn_readlane(mt, has ? __ffsll((long long)has) - 1 : 0);
        return __ballot(mt > 0 && mt != some) == 0;
    }
    // tile L < total * NT of the order (group of n-tiles,) expert, n-tile, m-tile
    __device__ __forceinline__ TileLoc at(unsigned L, int NT, int group) const {
        int nt0 = 0, ntn = NT;
        if (group > 0) {
            const unsigned per_group = (unsigned)total * (unsigned)group, q = L / per_group;
            L -= q * per_group;
            nt0 = (int)q * group;
            ntn = min(group, NT - nt0);
        }
        const unsigned long long hit = __ballot(mt > 0 && L < (unsigned)incl * (unsigned)ntn);
        const int e = __ffsll((long long)hit) - 1;
        auto of = [&](int v) { return __builtin_amdgcn_readlane(v, e); };
        TileLoc t;
        t.expert = e;
        t.mt = of(mt);
        const unsigned rem = L - (unsigned)(of(incl) - t.mt) * (unsigned)ntn;
        const int j = (int)(rem / (unsigned)t.mt), first = ((int)rem - j * t.mt) * of(rpt);
        t.nt = nt0 + j;
        t.row0 = of(lo) + first;
        t.tile_rows = min(of(rpt), of(rows) - first);
        t.blk0 = 0;                          // (of tile-packed rows)
        t.half = -1;
        t.single = __ballot(mt > 1) == 0;
        return t;
    }
};

// 64 lanes x 4 bytes: global -> LDS [lds_addr, + 256); the base as in dma16
__device__ __forceinline__ void dma4(const void* gbase, uint32_t voff, uint32_t lds_addr) {
    uint64_t base;
    asm volatile("s_mov_b32 m0, %3\n\ts_mov_b64 %0, %2\n\tglobal_load_lds_dword %1, %0"
                 : "=&s"(base) : "v"(voff), "s"(gbase), "s"(lds_addr) : "memory", "m0");
}
// waits until at most STEP * n loads are in flight, BASE <= n <= BASE + MORE
template <int STEP, int BASE, int MORE>
__device__ __forceinline__ void wait_stages(int n) {
    if constexpr (MORE == 0) {
        wait_vmcnt<STEP * BASE>();
    } else {
        if (n >= BASE + MORE) wait_vmcnt<STEP * (BASE + MORE)>();
        else wait_stages<STEP, BASE, MORE - 1>(n);
    }
}

// The tiles of workgroup blockIdx.x < kCus.  lds_raw: C::LDS_BYTES.  K >= 64 * S, K % 64 == 0.
// GATHER: row r of the activations is A[row_src[r] / topk].  group: of n-tiles (tile_map.h), unless the batch is even.
template <typename C, bool GATHER, bool HALVES>
__device__ __forceinline__ void persist_tiles(
    unsigned char* lds_raw, const ExpertRows& experts, const bf16_t* __restrict__ A,
    const bf16_t* __restrict__ W0, const bf16_t* __restrict__ W1, int N, int K,
    bf16_t* __restrict__ Cout, const int32_t* __restrict__ row_src, int topk, bool stream_out, int group) {
    constexpr int S = C::STAGES, KSUB = C::KSUB;
    constexpr int B_MIN = HALVES ? C::B_PW / 2 : C::B_PW, MORE = C::A_PW + C::B_PW - B_MIN;     // wave-loads of a stage
    const int lane = threadIdx.x % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int wm = wave / C::WN, wn = wave % C::WN;
    const int KT = K / C::BK, NT = (N + C::BN_OUT - 1) / C::BN_OUT;
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds_raw;
    const int* lds_rows = reinterpret_cast<const int*>(lds_raw + S * C::STAGE_BYTES);
    const TileTable<C::BM> table(experts);
    if (group > 0 && table.even()) group = 0;

    const unsigned G = (unsigned)table.total * (unsigned)NT, per_xcd = (G + kXcds - 1) / kXcds;
    const unsigned first = blockIdx.x % kXcds * per_xcd, n = first < G ? min(per_xcd, G - first) : 0u;
    // HALVES: a die's last round is shared out in half tiles where whole ones would keep at most half of its CUs busy
    const unsigned slots = kCusPerXcd, rem = n % slots;
    const unsigned whole = HALVES && 2 * rem <= slots ? n - rem : n, end = n + (n - whole);
    unsigned slot = blockIdx.x / kXcds;
    if (slot >= end) return;
    auto tile_at = [&](unsigned slot) __attribute__((always_inline)) -> TileLoc {
        if (!HALVES || slot < whole) return table.at(first + slot, NT, group);
        TileLoc t = table.at(first + whole + (slot - whole) / 2, NT, group);
        t.half = (int)(slot - whole) & 1;
        return t;
    };
    auto column = [](const TileLoc& t) { return t.nt * C::BN_OUT + (HALVES && t.half > 0 ? C::BN_OUT / 2 : 0); };
    TileLoc t = tile_at(slot);

    // ---- requests.  Lane l of a wave-load brings chunk (l % 8) ^ swizzle of row l / 8; the swizzle
    // 2 * ((row / 2) % 4) keeps 16-row reads of 128-byte rows free of bank conflicts.
    const unsigned char *a_base, *w0, *w1 = nullptr;
    uint32_t a_off[C::A_PW], b_off[C::B_PW];
    int a_cnt, b_cnt;                            // wave-loads of a stage
    bool once;                                   // no other workgroup reads the tile's weights
    auto request_from = [&](const TileLoc& t, auto from_lds) __attribute__((always_inline)) {
        a_base = uniform_ptr(reinterpret_cast<const unsigned char*>(
            A + (GATHER ? (size_t)0 : (size_t)t.row0 * K)));
        const int n0 = HALVES ? min(column(t), N - 16) : column(t), n_left = N - n0;   // a second half may lie beyond N
        const int bn = HALVES && t.half >= 0 ? C::BN / 2 : C::BN;    // weight rows of the tile
        b_cnt = HALVES && t.half >= 0 ? C::B_PW / 2 : C::B_PW;
        const size_t wrow = (size_t)t.expert * N + n0;
        w0 = uniform_ptr(reinterpret_cast<const unsigned char*>(W0 + wrow * K));
        if (C::SWIGLU) w1 = uniform_ptr(reinterpret_cast<const unsigned char*>(W1 + wrow * K));
        a_cnt = 0;
        once = t.mt == 1 && (!C::SWIGLU || t.tile_rows <= 64 || t.single);
        const uint32_t chunk = (uint32_t)(((lane & 7) ^ ((lane >> 3) & 6)) * 16);
#pragma unroll
        for (int jj = 0; jj < C::A_PW; ++jj) {
            const int j = wave + jj * C::NWAVES, rr = min(j * 8 + (lane >> 3), t.tile_rows - 1);
            unsigned row = (unsigned)rr;
            if (GATHER)
                row = (unsigned)((decltype(from_lds)::value ? lds_rows[rr] : row_src[t.row0 + rr]) / topk);
            a_off[jj] = row * (unsigned)K * 2u + chunk;
            if (j * 8 < t.tile_rows) a_cnt = jj + 1;
        }
#pragma unroll
        for (int jj = 0; jj < C::B_PW; ++jj) {
            const int r = (wave + jj * C::NWAVES) * 8 + (lane >> 3);
            const int rn = C::SWIGLU && r >= bn / 2 ? r - bn / 2 : r;
            b_off[jj] = (uint32_t)min(rn, n_left - 1) * (uint32_t)K * 2u + chunk;
        }
    };
    // Part `part` of KSUB of this wave's share of stage kq, into ring slot buf.
    auto request = [&](int part, int kq, int buf) __attribute__((always_inline)) {
        const uint32_t kb = (uint32_t)kq * (uint32_t)C::ROW_BYTES;
        const uint32_t to = lds_base + (uint32_t)buf * C::STAGE_BYTES + wave * 1024u;
#pragma unroll
        for (int jj = 0; jj < C::A_PW; ++jj)
            if (jj % KSUB == part && jj < a_cnt) dma16(a_base, a_off[jj] + kb, to + jj * C::NWAVES * 1024u);
#pragma unroll
        for (int jj = 0; jj < C::B_PW; ++jj)
            if (jj % KSUB == part && jj < b_cnt) {
                const bool up = C::SWIGLU && jj >= b_cnt / 2;
                const uint32_t at = to + C::A_BYTES + jj * C::NWAVES * 1024u;
                if (once) dma16_nt(up ? w1 : w0, b_off[jj] + kb, at);
                else dma16(up ? w1 : w0, b_off[jj] + kb, at);
            }
    };
    // ---- fragment reads: lane l reads row l % 16 of a sub-tile, 16-byte chunk l / 16 of the k-step (the second k-step
    // of a stage: + 4, which the swizzle makes address ^ 64)
    const int b_rd = (lane & 15) * C::ROW_BYTES + (((lane >> 4) ^ (lane & 6)) << 4);
    const int a_rd = b_rd + 16 * wm * C::ROW_BYTES;

    request_from(t, std::false_type{});
#pragma unroll
    for (int s = 0; s < S - 1; ++s)
#pragma unroll
        for (int h = 0; h < KSUB; ++h) request(h, s, s);
    wait_stages<S - 2, B_MIN, MORE>(b_cnt + a_cnt);
    __builtin_amdgcn_s_barrier();
    if (wm == 1) __builtin_amdgcn_s_barrier();   // group 1 runs one phase behind

    int buf = 0, allow = b_cnt + a_cnt;        // loads of a stage that may be in flight at its end
    for (;;) {
        slot += slots;
        const bool more = slot < end;
        TileLoc next = t;
        if (more) {
            next = tile_at(slot);
            // its row numbers by way of the LDS: a load to a register would wait for all requests before it.  Older than
            // stage S - 1, so they are there, and every wave's, long before request_from() reads them.
            if (GATHER && wave < (C::BM + kWave - 1) / kWave)
                dma4(row_src, (uint32_t)(next.row0 + min(wave * kWave + lane, next.tile_rows - 1)) * 4u,
                     lds_base + S * C::STAGE_BYTES + wave * 256u);
        }
        const int nsub = (t.tile_rows + 15) / 16;
        const int ta = min(C::TM, max(0, (nsub - wm + C::WM - 1) / C::WM));
        auto tile = [&](auto ta_tag, auto tn_tag) __attribute__((always_inline)) {
            constexpr int TA = decltype(ta_tag)::value, TAX = TA > 0 ? TA : 1, TN = decltype(tn_tag)::value;
            auto nb = [&](int j) __attribute__((always_inline)) -> int {     // B sub-tile base row
                constexpr int JN = C::SWIGLU ? TN / 2 : TN;
                return j < JN ? 16 * (wn * JN + j) : 16 * C::WN * JN + 16 * (wn * JN + (j - JN));
            };
            floatx4 acc[TAX][TN];
#pragma unroll
            for (int i = 0; i < TA; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
            bf16x8 af[TAX], bfr[TN];
            int kq = S - 1, step = 1, stages = KT - (S - 1);
            // first the stages whose successors belong to this tile, then those whose successors are the next tile's
#pragma unroll 1
            for (int part = 0; part < 2; ++part) {
#pragma unroll 1
                for (int i = 0; i < stages; ++i) {
#pragma unroll
                    for (int h = 0; h < KSUB; ++h) {
                        request(h, kq, buf == 0 ? S - 1 : buf - 1);
                        if (TA > 0) {
                            const unsigned char* st = lds_raw + buf * C::STAGE_BYTES;
                            const unsigned char* sa = st + (a_rd ^ (h * 64));
                            const unsigned char* sb = st + C::A_BYTES + (b_rd ^ (h * 64));
#pragma unroll
                            for (int j = 0; j < TN; ++j)
                                bfr[j] = *reinterpret_cast<const bf16x8*>(sb + nb(j) * C::ROW_BYTES);
#pragma unroll
                            for (int m = 0; m < TA; ++m)
                                af[m] = *reinterpret_cast<const bf16x8*>(sa + m * 16 * C::WM * C::ROW_BYTES);
                        }
                        if (h == KSUB - 1 && wm == 1) wait_stages<S - 2, B_MIN, MORE>(allow);
                        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                        __builtin_amdgcn_sched_barrier(0);
                        __builtin_amdgcn_s_barrier();
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int m = 0; m < TA; ++m)
#pragma unroll
                            for (int j = 0; j < TN; ++j)
                                acc[m][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[j], af[m], acc[m][j], 0, 0, 0);
                        if (h == KSUB - 1 && wm == 0) wait_stages<S - 2, B_MIN, MORE>(allow);
                        __builtin_amdgcn_sched_barrier(0);
                        __builtin_amdgcn_s_barrier();
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    kq += step;
                    buf = buf + 1 == S ? 0 : buf + 1;
                }
                if (part == 0) {
                    stages = S - 1;
                    if (more) {
                        const int before = b_cnt + a_cnt;
                        request_from(next, std::true_type{});
                        allow = min(before, b_cnt + a_cnt);
                        kq = 0;
                    } else {                     // the last stage again, so that the counts stay what they are
                        kq = KT - 1;
                        step = 0;
                    }
                }
            }
            allow = b_cnt + a_cnt;
            // (stores count as loads in flight: the waits that follow are stricter, never weaker)
            write_sub_tiles<TA, C::WM, C::SWIGLU, false>(acc, t, column(t), N, Cout, wm, wn, stream_out);
        };
        auto run = [&](auto ta_tag) __attribute__((always_inline)) {
            if constexpr (HALVES) {
                if (t.half >= 0) return tile(ta_tag, std::integral_constant<int, C::TN / 2>{});
            }
            tile(ta_tag, std::integral_constant<int, C::TN>{});
        };
        dispatch_count(ta, run, std::make_integer_sequence<int, C::TM + 1>{});
        if (!more) break;
        t = next;
    }
    if (wm == 0) __builtin_amdgcn_s_barrier();
    wait_vmcnt<0>();                             // no load may outlive the workgroup's LDS
}

}  // namespace pipe
}  // namespace specmoe
