// Device-side map from a workgroup id to its (expert, n-tile, m-tile) for the grouped expert
// GEMMs.  m-tiles never straddle experts; the map is computed from expert_offsets on the
// device so that no host read-back sits between the permutation and the GEMM.
//
// XCD awareness: the hardware deals workgroup ids round-robin to the 8 accelerator dies
// (id % 8), each with its own L2.  Logical tiles are ordered expert-major, then n-tile, then
// m-tile, and die x takes the x-th contiguous eighth of that order: the m-tiles that share a
// weight tile, and the n-tiles that share an activation tile, run on one die at about the
// same time and meet in its L2.
#pragma once
#include "common.h"

namespace specmoe {

struct TileLoc {
    int expert;      // expert id
    int row0;        // first row of the tile in the permuted row space
    int tile_rows;   // valid rows in the tile (1 .. BM)
    int nt;          // n-tile index
    int blk0;        // 16-row blocks in front of the tile when every expert's rows are padded to
                     // a whole number of blocks (row numbering of the tile-packed matrices)
    int half;        // -1, or the half of the tile's outputs that the workgroup takes
    int mt;          // m-tiles of the tile's expert (1: its weight tiles are read by one workgroup)
    int single;      // no expert of the 64 at a time up to the tile's has several (a whole word: padding bytes that a copy
                     // takes along go through scratch memory, and with them every load in flight)
};

// Even split: an expert with M rows gets ceil(M / BM_MAX) m-tiles of equal height (rounded up
// to the row granule of the matrix instruction in use, 32 or 16), so no tile is a thin
// remainder that would stream a whole weight tile for a handful of rows.
struct EvenSplit {
    int mt;    // m-tiles of the expert
    int rpt;   // rows per tile (multiple of GRAN, <= BM_MAX); the last tile may hold fewer
};
template <int BM_MAX, int GRAN>
__device__ __forceinline__ EvenSplit even_split(int M) {
    EvenSplit s{0, 0};
    if (M <= 0) return s;
    const unsigned m = M, mt0 = (m + BM_MAX - 1) / BM_MAX;
    s.rpt = (int)(((m + mt0 - 1) / mt0 + GRAN - 1) / GRAN * GRAN);
    s.mt = (int)((m + s.rpt - 1) / (unsigned)s.rpt);
    return s;
}

// GRAN = row granule of the matrix instruction in use (32 or 16).
// Wave-parallel: lane e works out expert e's split (64 experts per sweep), the running tile
// count comes from a wave scan, and the owning expert is the first lane whose range reaches the
// tile index.  Every wave of the workgroup calls this with all 64 lanes active and gets the same
// answer; a scalar walk over the experts costs several microseconds of integer divisions per
// workgroup, this one memory round trip and ~100 vector instructions, exchanges between lanes included.
template <int BM_MAX, int GRAN>
struct EvenPolicy {
    __device__ __forceinline__ static EvenSplit of(int M) { return even_split<BM_MAX, GRAN>(M); }
};
// fixed tile height BM: ceil(M / BM) tiles, the last one ragged
template <int BM>
struct FixedPolicy {
    __device__ __forceinline__ static EvenSplit of(int M) {
        EvenSplit s{0, BM};
        if (M > 0) s.mt = (M + BM - 1) / BM;
        return s;
    }
};

// m-tiles of all experts together, one total per split, from one sweep over the offsets (the same in
// every lane; not made scalar here: that would put the next step of every workgroup behind this
// one's round trip to memory, measured at 1 us per launch)
template <typename... Split>
__device__ __forceinline__ void count_mtiles(const int32_t* __restrict__ offsets, int E,
                                             int (&total)[sizeof...(Split)]) {
    const int lane = threadIdx.x % kWave;
    for (int& n : total) n = 0;
    for (int e0 = 0; e0 < E; e0 += kWave) {
        const int e = e0 + lane;
        const int M = e < E ? offsets[e + 1] - offsets[e] : 0;
        int i = 0;
        ((total[i++] += wave_sum(Split::of(M).mt)), ...);
    }
}

// Rounds of the chip that a batch's workgroups take, one per CU at a time.
__device__ __forceinline__ int tile_rounds(int total_mt, int NT) {
    return __builtin_amdgcn_readfirstlane((int)(((long long)total_mt * NT + kCus - 1) / kCus));
}

enum class From { workgroup, counted, place };

// A die's last round is shared out in half tiles (`halves`) where whole ones would keep at most half of its CUs
// busy: a batch of 3.5 rounds takes 3.5 rounds' time and not 4.  More halves than that would start a
// second round of them.  Measured, packed operands, us, whole / half: gate/up 8 x 4096 x 14336 (896 tiles): 83 rows
// each 372 / 364, 150 rows 397 / 383, 250 rows 457 / 442; down 16 x 8192 x 5120 (320 tiles), 88 rows 276 / 260; 200 rows
// 329 / 299 under a Zipf exponent of 0.5.  A hot expert's tile in halves at the end may cost more than it saves: the same, 30
// rows under an exponent of 1.1 233 / 253 (a size that the layer runs row-major); gate/up 16 x 4096 x 4096, 200 rows 260 / 268.
// Halving every unfinished round: the same where it is under half full, 64 x 2048 x 1408 109 -> 123.  For
// contractions from kTailMinK on: below (64 x 2048 x 1408, 94 rows 145.7 / 146.5) the surplus workgroups cost as much.
constexpr int kCusPerXcd = kCus / kXcds;
constexpr int kTailBlocks = kXcds * (kCusPerXcd / 2);       // more workgroups than tiles, at most
constexpr int kTailMinK = 4096;

// Groups of n-tiles (`group` > 0): the logical order is n-tile group, expert, n-tile, m-tile.  A die then
// meets every expert; expert-major, the dies that get cold experts read several times the weights that
// those of a hot expert do, and the launch waits for them.  From::workgroup drops it where every active
// expert has equally many m-tiles: the dies are even already (and 83 rows each, 8 x 4096 x 14336, 361 -> 363).
// The launchers state the sizes and figures.
//
// The tile of workgroup `at` (From::counted: of total_mt m-tiles), or at place `at` of the logical
// order (expert, n-tile, m-tile).  One function: with the second half in one of its own the compiler
// lays the packed GEMM kernels out differently, 1 to 4 % slower on batches of few tiles.
template <typename Split, From FROM, bool SHARE = false>
__device__ __forceinline__ bool locate(const int32_t* __restrict__ offsets, int E, int NT,
                                       long long at, int total_mt, TileLoc& t, int group = 0,
                                       bool halves = false) {
    constexpr bool GROUPS = SHARE || FROM == From::counted;
    const int lane = threadIdx.x % kWave;
    unsigned L = (unsigned)at;                    // a grid has less than 2^32 threads
    int nt0 = 0, ntn = NT, half = -1;             // n-tiles of the tile's group: the first, how many
    if constexpr (FROM != From::place) {
        if constexpr (FROM == From::workgroup) {
            total_mt = 0;
            int first_mt = 0;                     // m-tiles of the first expert that has any
            bool even = true;
            for (int e0 = 0; e0 < E; e0 += kWave) {
                const int e = e0 + lane;
                const int M = e < E ? offsets[e + 1] - offsets[e] : 0;
                const int mt = Split::of(M).mt;
                total_mt += wave_sum(mt);
                if (SHARE && group > 0) {
                    const unsigned long long has = __ballot(mt > 0);
                    if (first_mt == 0 && has)
                        first_mt = __builtin_amdgcn_readlane(mt, __ffsll((long long)has) - 1);
                    even = even && __ballot(mt > 0 && mt != first_mt) == 0;
                }
            }
            if (even) group = 0;
        }
        const unsigned block_id = (unsigned)at;
        const unsigned G = (unsigned)total_mt * (unsigned)NT;
        const unsigned per_xcd = (G + kXcds - 1) / kXcds;
        const unsigned first = block_id % kXcds * per_xcd;
        unsigned slot = block_id / kXcds;
        const unsigned n = first < G ? min(per_xcd, G - first) : 0u;      // the die's tiles
        if (SHARE && halves) {
            const unsigned rem = n % kCusPerXcd, whole = n - rem;
            if (slot >= whole && rem <= kCusPerXcd / 2) {
                half = (int)((slot - whole) & 1u);
                slot = whole + (slot - whole) / 2;
            }
        }
        L = first + slot;
        if (slot >= n) return false;
        if (GROUPS && group > 0) {
            const unsigned per_group = (unsigned)total_mt * (unsigned)group, q = L / per_group;
            L -= q * per_group;
            nt0 = (int)q * group;
            ntn = min(group, NT - nt0);
        }
    }
    int base_mt = 0;                              // m-tiles of the experts before this sweep
    int base_blk = 0;                             // 16-row blocks of the experts before this sweep
    int expert = -1, row0 = 0, rows = 0, nt = 0, blk0 = 0, mts = 0;
    t.single = 1;
    for (int e0 = 0; e0 < E && expert < 0; e0 += kWave) {
        const int e = e0 + lane;
        const int lo = e < E ? offsets[e] : 0, hi = e < E ? offsets[e + 1] : 0;
        const EvenSplit sp = Split::of(hi - lo);
        const int nblk = (hi - lo + 15) / 16;
        const int incl = wave_scan(sp.mt), incl_blk = wave_scan(nblk);   // inclusive
        const unsigned end = (unsigned)(base_mt + incl) * (unsigned)ntn; // tiles up to and incl. e
        const unsigned long long hit = __ballot(sp.mt > 0 && L < end);
        t.single &= __ballot(sp.mt > 1) == 0;
        if (hit) {
            const int src = __ffsll((long long)hit) - 1;              // first such expert
            auto of = [&](int v) { return __builtin_amdgcn_readlane(v, src); };
            const int mt = of(sp.mt), rpt = of(sp.rpt), excl = of(incl) - mt;
            const unsigned rem = L - (unsigned)(base_mt + excl) * (unsigned)ntn;
            const unsigned j = rem / (unsigned)mt;
            nt = nt0 + (int)j;
            const int mi = (int)(rem - j * (unsigned)mt);
            expert = e0 + src;
            mts = mt;
            row0 = of(lo) + mi * rpt;
            rows = min(rpt, of(hi) - row0);
            blk0 = base_blk + of(incl_blk) - of(nblk) + mi * rpt / 16;   // tile heights are multiples of 16
        }
        base_mt += __builtin_amdgcn_readlane(incl, kWave - 1);
        base_blk += __builtin_amdgcn_readlane(incl_blk, kWave - 1);
    }
    // the values are the same in every lane; say so to the compiler (scalar registers)
    t.expert = __builtin_amdgcn_readfirstlane(expert);
    t.row0 = __builtin_amdgcn_readfirstlane(row0);
    t.tile_rows = __builtin_amdgcn_readfirstlane(rows);
    t.nt = __builtin_amdgcn_readfirstlane(nt);
    t.blk0 = __builtin_amdgcn_readfirstlane(blk0);
    t.half = __builtin_amdgcn_readfirstlane(half);
    t.mt = __builtin_amdgcn_readfirstlane(mts);
    return t.expert >= 0;
}

template <int BM_MAX, int GRAN = 32, bool SHARE = false>
__device__ __forceinline__ bool locate_tile_even(const int32_t* __restrict__ offsets, int E,
                                                 int NT, unsigned block_id, TileLoc& t,
                                                 int group = 0, bool halves = false) {
    return locate<EvenPolicy<BM_MAX, GRAN>, From::workgroup, SHARE>(offsets, E, NT, block_id, 0, t,
                                                                    group, halves);
}
template <int BM>
__device__ __forceinline__ bool locate_tile(const int32_t* __restrict__ offsets, int E, int NT,
                                            unsigned block_id, TileLoc& t) {
    return locate<FixedPolicy<BM>, From::workgroup>(offsets, E, NT, block_id, 0, t);
}

// Upper bound of the grid (host side): sum_e ceil(M_e/BM) <= floor(n_rows/BM) + E.
inline long long grid_upper_bound(int n_rows, int E, int BM, long long NT) {
    long long g = ((long long)(n_rows / BM) + E) * NT;
    return (g + kXcds - 1) / kXcds * kXcds;
}

}  // namespace specmoe
