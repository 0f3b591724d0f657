// Offline table of pairwise L2 distances between the experts of one block (SpecMoE Sec. 3.2
// "Affinity-based expert selection mechanism", Fig. 8).  An expert's parameters are its three
// matrices together, so D[i,j]^2 = sum over gate, up and down of (W_i - W_j)^2.
//
// More than 8 experts.  Summing the squared differences pair by pair costs a subtraction and a
// fused multiply-add per element and PAIR (2016 pairs for 64 experts: bound by the vector units,
// 3.36 ms at 64 experts x 3 x 2048 x 1408).  Here the table comes out of one Gram matrix: with
// V_i = W_i - W_0 (distances do not change when one expert is subtracted from all),
//   D[i,j]^2 = G[i,i] + G[j,j] - 2 G[i,j],   G = V V^T.
// bf16, up to 64 experts: exact integer products of the digits of V (affinity_gram_exact_kernel).
// Otherwise (fp32, more experts, few weights) products and sums in fp64: v_mfma_f64_16x16x4 takes 64
// cycles for 16 x 16 pairs x 4 columns; a wave holds up to 64 experts at a time (10 tiles of the upper
// triangle: 640 cycles per 4 columns of 64 experts, 0.57 ms at the shape above) and reads and converts
// every weight once.  Measured, bf16, us, pair by pair / fp64 / integer products: 12 experts x 2048 x 2048
// 249 / 169 / 109, 16 x 4096 x 4096 966 / 614 / 418, 24 x 2048 x 1408 500 / 253 / 142, 40 x 2048 x 1408
// - / 452 / 237, 64 x 2048 x 1408 3360 / 703 / 307; 130 x 1024 x 704 7390 / 1430.
// Cancellation: subtracting W_0 removes what all experts have in common (experts grown from one
// dense model).  A pair that still lies closer together than 2^-10 of its norms - a copy, or any pair
// where expert 0 lies far from all others - takes its distance from its differences: the finish
// kernel lists the 8 x 8 blocks of the table that hold such a pair, and a second pass sums the
// differences of all pairs of a listed block, so no distance is less exact than a direct sum.  A
// block costs as much however many of its pairs are close: with every pair close, 64 experts x 2048 x 1408
// take 1.94 ms in all, 16 x 4096 x 4096 0.99 - where direct sums alone would take 0.97, so up to 16 experts such
// a table is the one case where they would be faster.
//
// Up to 8 experts (28 pairs): the direct sums are the faster form (the matrix kernel spends the
// same 64 cycles on 16 rows however few experts there are: 1.03 ms at 8 x 4096 x 14336 with two
// column slices in the 16 rows): affinity_pairs_kernel, bound by HBM since the next pieces are
// requested ahead (4 x 4096 x 14336 247 us = 5.7 TB/s, 675 without; 8 x 4096 x 14336 525 us = 5.4
// TB/s, 883 without).
//
// All sums run in a fixed order (deterministic, no floating-point atomics).
//
//   affinity_pairs_kernel     partial sums of squared differences, one set per workgroup
//   affinity_pairs_finish_kernel
//   affinity_gram_kernel, affinity_gram_exact_kernel   partial Gram matrices, one per workgroup
//   affinity_finish_kernel    adds the partials, writes the table, lists the blocks with close pairs
//   affinity_close_kernel     differences of the listed blocks (exits at once when there are none)
//   affinity_close_finish_kernel
#include "common.h"

#include <type_traits>

namespace specmoe {
namespace {

typedef double doublex4 __attribute__((ext_vector_type(4)));

constexpr int kRows = 16;           // experts of one matrix-instruction operand
constexpr int kSuper = 4;           // row blocks a wave keeps: 64 experts
constexpr int kMaxGroups = 256;     // workgroups (partials): one per CU
constexpr int kCloseThreads = 256, kCloseGroups = 1024;
constexpr int kCloseSide = 8;       // a block of the second pass: 8 x 8 pairs
constexpr int kCloseSlabs = 512;    // partials per block
constexpr int kPairThreads = 256, kPairGroups = 1024;   // up to 8 experts
constexpr double kClose = 1.0 / (1 << 20);   // D^2 below this share of the norms: sum differences
constexpr double kDrift = 1.0 / (1 << 27);   // D may be off by this share of it before its differences are summed

__host__ __device__ inline int row_blocks(int E) { return (E + kRows - 1) / kRows; }
// tile (I, J), I <= J, in row-major order over the upper triangle of nb x nb blocks
__host__ __device__ inline int tile_index(int I, int J, int nb) {
    return I * nb - I * (I - 1) / 2 + (J - I);
}
constexpr int kTile = kRows * kRows;
// What the finish kernel hands to the second pass.  It follows the partial sums in the workspace.
__host__ __device__ inline int side_blocks(int E) { return (E + kCloseSide - 1) / kCloseSide; }
__host__ __device__ inline int side_pairs(int E) { return side_blocks(E) * (side_blocks(E) + 1) / 2; }
struct CloseList {
    int* n;             // listed blocks
    int* blocks;        // [n] I * side_blocks + J, I <= J, in any order
    int* flags;         // [side_blocks^2] listed already
    __host__ __device__ CloseList(double* partial, int E)
        : n(reinterpret_cast<int*>(partial + (size_t)side_pairs(E) * kCloseSlabs * 64)),
          blocks(n + 2), flags(blocks + side_pairs(E)) {}
    // behind the list: [groups][2][16 row_blocks(E)] (affinity_gram_exact_kernel)
    double* spread(int E) const {
        return reinterpret_cast<double*>(((uintptr_t)(flags + side_blocks(E) * side_blocks(E)) + 7) & ~(uintptr_t)7);
    }
};

template <typename T> struct Piece;                 // one 16-byte piece of a weight row
template <> struct Piece<float> {
    static constexpr int N = 4;
    __device__ static float get(const U128& v, int i) { return __uint_as_float(v[i]); }
};
template <> struct Piece<bf16_t> {
    static constexpr int N = 8;
    __device__ static float get(const U128& v, int i) {
        const uint32_t w = v[i >> 1];
        return __uint_as_float(i & 1 ? w & 0xffff0000u : w << 16);
    }
};

typedef uint32_t U64 __attribute__((ext_vector_type(2)));
template <typename T> struct Half;                  // one 8-byte piece
template <> struct Half<float> {
    __device__ static float get(const U64& v, int i) { return __uint_as_float(v[i]); }
};
template <> struct Half<bf16_t> {
    __device__ static float get(const U64& v, int i) {
        const uint32_t w = v[i >> 1];
        return __uint_as_float(i & 1 ? w & 0xffff0000u : w << 16);
    }
};

// Up to NE = 4 or 8 experts: every thread keeps the sums of all NE (NE - 1) / 2 pairs in fp64
// (N squares in fp32, then one fp64 add per 16-byte piece).  The next pieces of all experts are
// requested before the current ones are used: about 450 vector instructions per 128 bytes (28
// pairs) then run under the loads instead of after them.
template <typename T, int NE>
__global__ __launch_bounds__(kPairThreads) void affinity_pairs_kernel(
    const T* __restrict__ wg, const T* __restrict__ wu, const T* __restrict__ wd, int E, size_t n1,
    double* __restrict__ partial /* [groups][64] */) {
    constexpr int N = Piece<T>::N, NP = NE * (NE - 1) / 2;
    const size_t pieces = n1 / N, stride = (size_t)gridDim.x * kPairThreads;
    const size_t first = (size_t)blockIdx.x * kPairThreads + threadIdx.x;
    double acc[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) acc[p] = 0.0;
    auto matrix = [&](const T* W) __attribute__((always_inline)) {
        const U128* rows[NE];
#pragma unroll
        for (int e = 0; e < NE; ++e)
            rows[e] = reinterpret_cast<const U128*>(W + (size_t)min(e, E - 1) * n1);
        U128 next[NE];
#pragma unroll
        for (int e = 0; e < NE; ++e) next[e] = rows[e][first < pieces ? first : 0];
        __builtin_amdgcn_sched_barrier(0);
        for (size_t q = first; q < pieces; q += stride) {
            U128 cur[NE];
#pragma unroll
            for (int e = 0; e < NE; ++e) cur[e] = next[e];
            const size_t qn = q + stride < pieces ? q + stride : q;
#pragma unroll
            for (int e = 0; e < NE; ++e) next[e] = rows[e][qn];
            __builtin_amdgcn_sched_barrier(0);          // the requests go out before the arithmetic
            float s[NP];
#pragma unroll
            for (int p = 0; p < NP; ++p) s[p] = 0.f;
#pragma unroll
            for (int k = 0; k < N; ++k) {
                float v[NE];
#pragma unroll
                for (int e = 0; e < NE; ++e) v[e] = Piece<T>::get(cur[e], k);
                int p = 0;
#pragma unroll
                for (int i = 0; i < NE; ++i)
#pragma unroll
                    for (int j = i + 1; j < NE; ++j, ++p) {
                        const float df = v[i] - v[j];
                        s[p] = fmaf(df, df, s[p]);
                    }
            }
#pragma unroll
            for (int p = 0; p < NP; ++p) acc[p] += (double)s[p];
        }
    };
    matrix(wg);
    matrix(wu);
    matrix(wd);
    // workgroup sum of every pair: xor butterfly per wave, then the 4 waves through LDS
    __shared__ double red[kPairThreads / kWave][NP];
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const double v = wave_sum(acc[p]);
        if (lane == 0) red[wave][p] = v;
    }
    __syncthreads();
    if (threadIdx.x < NP) {
        double v = 0.0;
        for (int w = 0; w < kPairThreads / kWave; ++w) v += red[w][threadIdx.x];
        partial[(size_t)blockIdx.x * 64 + threadIdx.x] = v;
    }
}

// One wavefront per table entry: lane l adds partials l, l+64, ... in order, then a butterfly.
__global__ __launch_bounds__(kWave) void affinity_pairs_finish_kernel(
    const double* __restrict__ partial, int E, int groups, float* __restrict__ table) {
    const int i = blockIdx.x / E, j = blockIdx.x % E;
    if (i == j) {
        if (threadIdx.x == 0) table[blockIdx.x] = 0.f;
        return;
    }
    const int lo = min(i, j), hi = max(i, j), ne = E <= 4 ? 4 : 8;
    const int slot = lo * ne - lo * (lo + 1) / 2 + (hi - lo - 1);   // pairs lo < hi in order
    double s = 0.0;
    for (int g = threadIdx.x; g < groups; g += kWave) s += partial[(size_t)g * 64 + slot];
    s = wave_sum(s);
    if (threadIdx.x == 0) table[blockIdx.x] = (float)sqrt(s);
}

// A wave multiplies NBI row blocks (16 experts each) with themselves (OFF = false: upper
// triangle) or with NBI other row blocks (OFF = true).  Operand layout of the instruction: lane
// l feeds row l % 16 and column l / 16; a lane loads 16 bytes, so a unit of 4 x N columns takes
// N instructions per tile, element i of every lane's piece being one of them (the columns of a
// Gram matrix may be taken in any order).
// PF units are in flight in registers: 1 KB per load, 16 waves x 4 KB per CU with one row block,
// less where 10 tiles share the loads.
template <typename T, int NBI, bool OFF, int WAVES, int PF>
__global__ __launch_bounds__(WAVES * kWave) void affinity_gram_kernel(
    const T* __restrict__ wg, const T* __restrict__ wu, const T* __restrict__ wd, int E,
    size_t n1 /* elements of one matrix of one expert, a multiple of N */,
    double* __restrict__ partial /* [tiles][groups][kTile] */, CloseList close) {
    constexpr int N = Piece<T>::N;
    constexpr int NR = OFF ? 2 * NBI : NBI;                     // row blocks loaded
    constexpr int TILES = OFF ? NBI * NBI : NBI * (NBI + 1) / 2;
    __shared__ double sum[TILES * kTile];
    const int lane = threadIdx.x % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int nb = row_blocks(E);
    int SI = blockIdx.y, SJ = SI;                               // super-blocks of this workgroup
    if (OFF) {                                                  // blockIdx.y-th pair SI < SJ
        const int ns = (nb + kSuper - 1) / kSuper;
        int rem = blockIdx.y;
        SI = 0;
        while (rem >= ns - 1 - SI) { rem -= ns - 1 - SI; ++SI; }
        SJ = SI + 1 + rem;
    }
    if (blockIdx.x == 0 && blockIdx.y == 0 && !OFF) {          // nothing listed yet
        const int ns = side_blocks(E);
        if (threadIdx.x == 0) *close.n = 0;
        for (int i = threadIdx.x; i < ns * ns; i += WAVES * kWave) close.flags[i] = 0;
    }

    size_t row_off[NR];
#pragma unroll
    for (int b = 0; b < NR; ++b) {
        const int blk = b < NBI ? SI * kSuper + b : SJ * kSuper + (b - NBI);
        row_off[b] = (size_t)min(blk * kRows + lane % kRows, E - 1) * n1;
    }
    const int units = (int)((n1 + 4 * N - 1) / (4 * N));        // per matrix
    const int total = 3 * units;
    const int stride = gridDim.x * WAVES;

    // the matrix is chosen by address arithmetic: a choice between pointers becomes generic loads,
    // which cannot be waited for one by one
    const uint64_t base = (uint64_t)wg, to_up = (uint64_t)wu - base, to_down = (uint64_t)wd - (uint64_t)wu;
    typedef const U128 __attribute__((address_space(1)))* Global;
    U128 raw[PF][NR + 1];                                       // [NR]: the same piece of expert 0
    bool live[PF];
    auto load = [&](int p, int u) __attribute__((always_inline)) {
        const int uc = min(u, total - 1);
        const int m = uc / units;
        const uint64_t W = base + (m >= 1 ? to_up : 0) + (m == 2 ? to_down : 0);
        const size_t col = (size_t)(uc - m * units) * (4 * N) + (size_t)(lane / kRows) * N;
        live[p] = u < total && col < n1;
        const uint64_t at = W + (live[p] ? col : 0) * sizeof(T);
#pragma unroll
        for (int b = 0; b < NR; ++b) raw[p][b] = *(Global)(at + row_off[b] * sizeof(T));
        raw[p][NR] = *(Global)at;
        __builtin_amdgcn_sched_barrier(0);      // the loads stay here, PF units ahead of their use
    };

    doublex4 acc[TILES];
#pragma unroll
    for (int t = 0; t < TILES; ++t) acc[t] = doublex4{0.0, 0.0, 0.0, 0.0};
    const int first = blockIdx.x * WAVES + wave;
#pragma unroll
    for (int p = 0; p < PF; ++p) load(p, first + p * stride);
    for (int u0 = first; u0 < total; u0 += PF * stride) {
#pragma unroll
        for (int p = 0; p < PF; ++p) {
            U128 cur[NR + 1];                                   // zeros beyond the last column
#pragma unroll
            for (int b = 0; b <= NR; ++b)
                cur[b] = live[p] ? raw[p][b] : U128{0, 0, 0, 0};
            load(p, u0 + (p + PF) * stride);
#pragma unroll
            for (int i = 0; i < N; ++i) {
                // a reference element that is not finite is left out, for all experts alike
                const float f0 = Piece<T>::get(cur[NR], i);
                const double ref = (double)(__builtin_isfinite(f0) ? f0 : 0.f);
                double v[NR];
#pragma unroll
                for (int b = 0; b < NR; ++b) v[b] = (double)Piece<T>::get(cur[b], i) - ref;
                int t = 0;
#pragma unroll
                for (int a = 0; a < NBI; ++a)
#pragma unroll
                    for (int b = OFF ? 0 : a; b < NBI; ++b) {
                        acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[a], v[OFF ? NBI + b : b],
                                                                      acc[t], 0, 0, 0);
                        ++t;
                    }
            }
        }
    }

    // waves of the workgroup, in order; element q of a lane is row 4 * q + lane / 16, column
    // lane % 16 of its tile
    for (int w = 0; w < WAVES; ++w) {
        if (wave == w) {
#pragma unroll
            for (int t = 0; t < TILES; ++t)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    double* s = sum + t * kTile + (4 * q + lane / kRows) * kRows + lane % kRows;
                    *s = w == 0 ? acc[t][q] : *s + acc[t][q];
                }
        }
        __syncthreads();
    }
    int t = 0;
#pragma unroll
    for (int a = 0; a < NBI; ++a)
#pragma unroll
        for (int b = OFF ? 0 : a; b < NBI; ++b, ++t) {
            const int I = SI * kSuper + a, J = SJ * kSuper + b;
            if (I < nb && J < nb && threadIdx.x < kTile)
                partial[((size_t)tile_index(I, J, nb) * gridDim.x + blockIdx.x) * kTile +
                        threadIdx.x] = sum[t * kTile + threadIdx.x];
        }
}

// bf16, 9 to 64 experts: the same partial Gram matrices from exact integer products.  A difference
// v = w - w_0 of two bf16 numbers has few significant bits, so it is written as q * 2^ex, with one ex per
// expert for as long as it fits, q a whole number below 2^22 in three signed 8-bit digits, and
// v_mfma_i32_16x16x64_i8 multiplies the digits: 64 columns of 16 x 16 pairs in 9 instructions of 16 cycles
// where the fp64 instruction takes 16 of 64.  int32 sums are exact; they move to fp64 sums in LDS when
// an ex changes and after kExactUnits units.  So the table holds the exact distances of the rounded
// vectors q * 2^ex.  A v with bits below 2^ex (which is at most 2^-17 of the largest of a row's 64
// columns) is off by a residual r of at most half of it.  The kernel adds up r^2 (of a quarter of the
// columns: 13 % less time than of all), alone (spread[0]) and
// with the squares of the values next to it (spread[1]), and the finish kernel sends the pairs whose
// distance this may move by 2^-27 to the second pass; fp32 rounds it at 2^-25.  Normal weights stay at 2^-31 from
// 200 thousand on (hardly any of them rounds), with the heaviest tails a few millions do.
// Units of 64 columns with a number that is not finite, or beyond 2^+-100, go through the fp64 instruction.
// Bound by HBM and, close behind, by the vector instructions that make the digits (6 to 7 per weight).
// So every weight is converted once: a team of two waves shares a unit, each wave converts half of the
// row blocks, the digits meet in LDS, and each wave multiplies half of the tiles.  The two waves of a
// SIMD belong to one team; between two barriers one multiplies unit i and then converts unit i + 1, the
// other does it in the opposite order, so matrix and vector units run side by side.  64 experts x 2048 x
// 1408: 0.29 ms (1.1 GB: 3.8 TB/s), 0.69 with the fp64 instruction; converting alone 0.24, multiplying alone 0.12.
constexpr int kExactUnits = 512;             // 3 products per sum, 64 x 2^14 each: below 2^31
constexpr float kMagic = 12582912.f + 32896.f;   // 1.5 * 2^23 + 0x8080: the low bits are q + 0x8080
constexpr int kTopBit = 19;                  // a new ex puts the largest v of a unit at 2^19 .. 2^20
constexpr float kFits = 4.1e6f;              // below 2^22 - 0x8080
constexpr int kNoEx = -1000;                 // no v but zero so far
constexpr int kUnit = 64;                    // columns of a unit: 16 per lane

typedef int intx4 __attribute__((ext_vector_type(4)));

// whether an expert's ex suits a unit whose largest |v| is top (NaN: no)
__device__ __forceinline__ bool row_fits(float top, float scale) {
    return top == 0.f || (top * scale < kFits && top * scale >= (float)(1 << (kTopBit - 2)));
}

template <int NBI> struct Exact {
    static constexpr int WAVES = NBI <= 2 ? 16 : 8;             // as many as the registers allow
    static constexpr int TILES = NBI * (NBI + 1) / 2, DIGITS = 3;
    static constexpr int TEAM = NBI > 1 ? 2 : 1, TEAMS = WAVES / TEAM;
    static constexpr int CB = (NBI + TEAM - 1) / TEAM;          // row blocks a wave converts
    static constexpr int HT = (TILES + TEAM - 1) / TEAM;        // tiles a wave multiplies
    // teams that add at a time, each to sums of its own (as many as the LDS holds)
    static constexpr int BANKS = NBI == 4 ? 2 : TEAMS;
    static constexpr int SPREAD = 2 * NBI * kRows;
    static constexpr size_t SUMS = (size_t)BANKS * TILES * kTile * sizeof(double);
    static constexpr size_t DIGIT_BYTES = (size_t)2 * TEAMS * NBI * DIGITS * kWave * 16;
    static constexpr int EX = TEAMS * NBI * kRows;
    static constexpr size_t LDS = SUMS + DIGIT_BYTES + EX * (2 * sizeof(int) + sizeof(float)) +
                                  BANKS * SPREAD * sizeof(double) + 2 * WAVES * sizeof(int);
    static_assert(LDS <= 160 * 1024, "LDS");
};
// tiles of the upper triangle of n x n row blocks, in rows (known at compile time once t is)
__device__ constexpr int kTriRow[5][10] = {{}, {0}, {0, 0, 1}, {0, 0, 0, 1, 1, 2}, {0, 0, 0, 0, 1, 1, 1, 2, 2, 3}};
__device__ constexpr int kTriCol[5][10] = {{}, {0}, {0, 1, 1}, {0, 1, 2, 1, 2, 2}, {0, 1, 2, 3, 1, 2, 3, 2, 3, 3}};

template <int NBI>
__global__ __launch_bounds__(Exact<NBI>::WAVES * kWave) void affinity_gram_exact_kernel(
    const bf16_t* __restrict__ wg, const bf16_t* __restrict__ wu, const bf16_t* __restrict__ wd, int E,
    size_t n1 /* elements of one matrix of one expert, a multiple of 8 */,
    double* __restrict__ partial /* [tiles][groups][kTile] */, CloseList close,
    double* __restrict__ spread_out /* [groups][2][NBI * kRows] */) {
    typedef Exact<NBI> X;
    constexpr int DIGITS = X::DIGITS, CB = X::CB, HT = X::HT, TEAMS = X::TEAMS;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    double* sums = reinterpret_cast<double*>(lds_raw);          // [BANKS][TILES][4][kWave]
    intx4* digits = reinterpret_cast<intx4*>(lds_raw + X::SUMS);   // [2][TEAMS][NBI][DIGITS][kWave]
    double* spread = reinterpret_cast<double*>(lds_raw + X::SUMS + X::DIGIT_BYTES);   // [BANKS][2][NBI * kRows]
    float* rest = reinterpret_cast<float*>(spread + X::BANKS * X::SPREAD);   // [TEAMS][NBI][kRows]: sum of (r / 2^ex)^2
    int* ex_now = reinterpret_cast<int*>(rest + X::EX);         // the same: ex of acc
    int* ex_new = ex_now + X::EX;                               // ex of the newest digits
    int* flags = ex_new + X::EX;                                // [2][waves]: 1 ex changed, 2 fp64 unit
    const int lane = threadIdx.x % kWave, g = lane / kRows;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int half = wave / TEAMS, team = wave % TEAMS;         // waves w and w + 4 share a SIMD
    const int nb = row_blocks(E);
    if (blockIdx.x == 0) {                                      // nothing listed yet
        const int ns = side_blocks(E);
        if (threadIdx.x == 0) *close.n = 0;
        for (int i = threadIdx.x; i < ns * ns; i += X::WAVES * kWave) close.flags[i] = 0;
    }
    for (int i = threadIdx.x; i < X::BANKS * X::TILES * kTile; i += X::WAVES * kWave) sums[i] = 0.0;
    for (int i = threadIdx.x; i < 2 * X::EX; i += X::WAVES * kWave) ex_now[i] = kNoEx;
    for (int i = threadIdx.x; i < X::BANKS * X::SPREAD; i += X::WAVES * kWave) spread[i] = 0.0;

    const int units = (int)((n1 + kUnit - 1) / kUnit), total = 3 * units;
    const int stride = gridDim.x * TEAMS, iters = (total + stride - 1) / stride;
    const int first = blockIdx.x * TEAMS + team;
    const uint64_t base = (uint64_t)wg, to_up = (uint64_t)wu - base, to_down = (uint64_t)wd - (uint64_t)wu;
    typedef const U128 __attribute__((address_space(1)))* Global;
    // unit u: its matrix and first column (the last unit of a matrix may be ragged)
    auto unit_base = [&](int u, size_t& col0) __attribute__((always_inline)) -> uint64_t {
        const int uc = min(u, total - 1), m = uc / units;
        col0 = (size_t)(uc - m * units) * kUnit;
        return base + (m >= 1 ? to_up : 0) + (m == 2 ? to_down : 0);
    };
    auto row_bytes = [&](int b) __attribute__((always_inline)) -> size_t {
        return (size_t)min(b * kRows + lane % kRows, E - 1) * n1 * 2;
    };

    // ---- loads: this wave's row blocks and expert 0; a lane's columns are two pieces of 8.  In place of a
    // ragged unit the last whole one is read (its digits are not used).
    uint64_t row_at[CB + 1];
#pragma unroll
    for (int c = 0; c <= CB; ++c) row_at[c] = (c < CB ? row_bytes(half * CB + c) : 0) + 16 * g;
    U128 raw[CB + 1][2];
    auto load = [&](int u) __attribute__((always_inline)) {
        size_t col0;
        const uint64_t W = unit_base(u, col0);
        const uint64_t at = W + (col0 + kUnit > n1 ? n1 - kUnit : col0) * 2;
#pragma unroll
        for (int c = 0; c <= CB; ++c)
#pragma unroll
            for (int h = 0; h < 2; ++h) raw[c][h] = *(Global)(at + row_at[c] + 64 * h);
        __builtin_amdgcn_sched_barrier(0);      // the loads stay here, ahead of their use
    };

    // ---- digits of unit i (in raw) into slot i % 2, then the next loads
    float scale[CB];                            // 2^-ex of row lane % 16; 0 before the first unit
    float left[CB], left_new[CB];               // sampled sums of (r / 2^ex)^2: units in acc, newest unit
#pragma unroll
    for (int c = 0; c < CB; ++c) scale[c] = left[c] = left_new[c] = 0.f;
    auto convert = [&](int i) __attribute__((always_inline)) {
        const int u = first + i * stride;
        auto element = [&](int c, int j) __attribute__((always_inline)) -> float {
            return Piece<bf16_t>::get(raw[c][j / 8], j % 8);
        };
        intx4* slot = digits + (size_t)((i & 1) * TEAMS + team) * NBI * DIGITS * kWave;
        float top[CB];                          // the largest |v| of this lane, NaN if one is
        int flag = 0;
#pragma unroll
        for (int c = 0; c < CB; ++c) left[c] += left_new[c];
        for (bool once = true;; once = false) {
            bool fits = true;
            float ref[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) ref[j] = element(CB, j);
#pragma unroll
            for (int c = 0; c < CB; ++c) {
                const int b = half * CB + c;
                top[c] = left_new[c] = 0.f;
                if (b >= NBI) continue;
                intx4 d[DIGITS];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    uint32_t q[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const float v = element(c, 4 * j + k) - ref[4 * j + k];
                        top[c] = __builtin_elementwise_maximum(top[c], __builtin_fabsf(v));
                        const float whole = fmaf(v, scale[c], kMagic);
                        if (k == j) {                           // a sample of 4 of 16
                            const float r = fmaf(v, scale[c], kMagic - whole);
                            left_new[c] = fmaf(r, r, left_new[c]);
                        }
                        q[k] = __float_as_uint(whole);
                    }
                    const uint32_t p01 = __builtin_amdgcn_perm(q[1], q[0], 0x05010400u);
                    const uint32_t p23 = __builtin_amdgcn_perm(q[3], q[2], 0x05010400u);
                    const uint32_t hi = __builtin_amdgcn_perm(q[1], q[0], 0x0c0c0602u) |
                                        __builtin_amdgcn_perm(q[3], q[2], 0x06020c0cu);
                    d[0][j] = (int)(__builtin_amdgcn_perm(p23, p01, 0x05040100u) ^ 0x80808080u);
                    d[1][j] = (int)(__builtin_amdgcn_perm(p23, p01, 0x07060302u) ^ 0x80808080u);
                    // the top byte is 64 + digit, in 0 .. 127: minus 64, byte by byte without a borrow
                    d[2][j] = (int)(((hi ^ 0x80808080u) - 0x40404040u) ^ 0x80808080u);
                }
#pragma unroll
                for (int x = 0; x < DIGITS; ++x) slot[(b * DIGITS + x) * kWave + lane] = d[x];
                const float in_units = top[c] * scale[c];
                fits = fits && in_units < kFits &&
                       (top[c] == 0.f || in_units >= (float)(1 << (kTopBit - 4)));
                __builtin_amdgcn_sched_barrier(0);              // registers: one block at a time
            }
            if (__all(fits) || !once) break;
            // the largest |v| of each row: its four lanes
            bool keep = true, plain = true;
#pragma unroll
            for (int c = 0; c < CB; ++c) {
                top[c] = __builtin_elementwise_maximum(top[c], __shfl_xor(top[c], 16, kWave));
                top[c] = __builtin_elementwise_maximum(top[c], __shfl_xor(top[c], 32, kWave));
                keep = keep && row_fits(top[c], scale[c]);
                plain = plain && (top[c] == 0.f || (top[c] > 0x1p-100f && top[c] < 0x1p+100f));
            }
            if (!__all(plain)) {
                flag = 2;
                break;
            }
            if (__all(keep)) break;
            flag = 1;
#pragma unroll
            for (int c = 0; c < CB; ++c)
                if (!row_fits(top[c], scale[c])) {
                    const int ex = (int)(__float_as_uint(top[c]) >> 23) - 127 - kTopBit;
                    scale[c] = __uint_as_float((uint32_t)(127 - ex) << 23);
                    ex_new[(team * NBI + half * CB + c) * kRows + lane % kRows] = ex;
                }
        }
        if ((size_t)(u % units + 1) * kUnit > n1) flag = 2;     // ragged
        if (flag == 2 || u >= total)
#pragma unroll
            for (int c = 0; c < CB; ++c) left_new[c] = 0.f;
        if (lane == 0) flags[(i & 1) * X::WAVES + wave] = u < total ? flag : 0;
        load(u + stride);
    };

    // ---- the main loop, for each half of a team
    auto run = [&](auto half_tag) __attribute__((always_inline)) {
    constexpr int H = decltype(half_tag)::value;
    // products of a slot; this wave's tiles
    intx4 acc[HT][2 * DIGITS - 1];              // [x + y]: digit x of the row times digit y of the column
    auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < HT; ++t)
#pragma unroll
            for (int s = 0; s < 2 * DIGITS - 1; ++s) acc[t][s] = intx4{0, 0, 0, 0};
    };
    auto multiply = [&](int i) __attribute__((always_inline)) {
        const intx4* slot = digits + (size_t)((i & 1) * TEAMS + team) * NBI * DIGITS * kWave + lane;
        intx4 da[DIGITS], db[DIGITS];
#pragma unroll
        for (int t = 0; t < HT; ++t) {
            const int tile = H * HT + t;
            if (tile >= X::TILES) continue;
            const int a = kTriRow[NBI][tile], b = kTriCol[NBI][tile];
#pragma unroll
            for (int x = 0; x < DIGITS; ++x) {
                if (t == 0 || a != kTriRow[NBI][tile - 1]) da[x] = slot[(a * DIGITS + x) * kWave];
                db[x] = a == b ? da[x] : slot[(b * DIGITS + x) * kWave];
            }
#pragma unroll
            for (int z = 0; z < DIGITS; ++z)
#pragma unroll
                for (int x = 0; x < DIGITS; ++x) {              // neighbours add to different sums
                    const int y = (x + z) % DIGITS;
                    acc[t][x + y] =
                        __builtin_amdgcn_mfma_i32_16x16x64_i8(da[x], db[y], acc[t][x + y], 0, 0, 0);
                }
        }
    };
    // all waves: acc into the sums (in one order of additions); wide: unit i of this team in fp64
    auto settle = [&](int i, int held, bool wide) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < CB; ++c) {
            left[c] += __shfl_xor(left[c], 16, kWave);
            left[c] += __shfl_xor(left[c], 32, kWave);
            if (half * CB + c < NBI) rest[(team * NBI + half * CB + c) * kRows + lane % kRows] = left[c];
            left[c] = 0.f;
        }
        __syncthreads();
        double* mine = sums + (size_t)(team % X::BANKS) * X::TILES * kTile;
        double* spread_mine = spread + (team % X::BANKS) * X::SPREAD;
        for (int turn = 0; turn < TEAMS / X::BANKS; ++turn) {
            if (turn == team / X::BANKS) {
#pragma unroll
                for (int t = 0; t < HT; ++t) {
                    const int tile = H * HT + t;
                    if (tile >= X::TILES || held == 0) continue;
                    const int a = kTriRow[NBI][tile], b = kTriCol[NBI][tile];
                    const int* ea = ex_now + (team * NBI + a) * kRows + 4 * g;
                    const int eb = ex_now[(team * NBI + b) * kRows + lane % kRows];
                    // a lane holds rows 4 * (lane / 16) + r, r = 0 .. 3, column lane % 16
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        double v = (double)acc[t][4][r];
#pragma unroll
                        for (int s = 3; s >= 0; --s) v = fma(v, 256.0, (double)acc[t][s][r]);
                        v = ldexp(v, ea[r] + eb);
                        mine[(tile * 4 + r) * kWave + lane] += v;
                        if (a == b && 4 * g + r == lane % kRows) {      // v: squares of a row
                            const double r2 = ldexp(4.0 * rest[(team * NBI + a) * kRows + 4 * g + r], 2 * eb);
                            spread_mine[a * kRows + 4 * g + r] += r2;
                            spread_mine[(NBI + a) * kRows + 4 * g + r] += r2 * v / (kUnit * held);
                        }
                    }
                }
                if (wide) {
                    size_t col0;
                    const uint64_t W = unit_base(first + i * stride, col0);
                    for (int t = 0; t < HT && H * HT + t < X::TILES; ++t) {
                        const int tile = H * HT + t;
                        const size_t oa = row_bytes(kTriRow[NBI][tile]), ob = row_bytes(kTriCol[NBI][tile]);
                        doublex4 d = doublex4{0.0, 0.0, 0.0, 0.0};
                        for (int h = 0; h < 2; ++h) {
                            const size_t col = col0 + 32 * h + 8 * g;
                            U128 ra = {0, 0, 0, 0}, rb = ra, r0 = ra;
                            if (col < n1) {
                                ra = *(Global)(W + col * 2 + oa);
                                rb = *(Global)(W + col * 2 + ob);
                                r0 = *(Global)(W + col * 2);
                            }
#pragma unroll
                            for (int j = 0; j < 8; ++j) {
                                // a reference that is not finite is left out, for all experts alike
                                const float f0 = Piece<bf16_t>::get(r0, j);
                                const double rd = (double)(__builtin_isfinite(f0) ? f0 : 0.f);
                                d = __builtin_amdgcn_mfma_f64_16x16x4f64(
                                    (double)Piece<bf16_t>::get(ra, j) - rd,
                                    (double)Piece<bf16_t>::get(rb, j) - rd, d, 0, 0, 0);
                            }
                        }
                        // element q of a lane is row 4 * q + lane / 16, column lane % 16 of its tile
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            mine[(tile * 4 + g) * kWave + 16 * q + lane % kRows] += d[q];
                    }
                }
            }
            __syncthreads();
        }
        for (int j = threadIdx.x; j < X::EX; j += X::WAVES * kWave) ex_now[j] = ex_new[j];
        __syncthreads();
        clear();
    };

    clear();
    int held = 0;                               // units in acc
    for (int i = 0;; ++i) {
        __syncthreads();                        // digits and flags of unit i are there
        const int flag = i < iters ? flags[(i & 1) * X::WAVES + lane % X::WAVES] : 1;
        bool plain = first + i * stride < total;                // the same in both waves of a team
        if (held == kExactUnits || __any(flag != 0)) {
            const bool wide = __any(flag == 2 && lane % TEAMS == team);
            settle(i, held, wide);
            plain = plain && !wide;
            held = 0;
        }
        if (i == iters) break;
        ++held;
        if (H == 0 && plain) multiply(i);
        convert(i + 1);
        if (H == 1 && plain) multiply(i);
    }
    };
    load(first);
    __syncthreads();                            // ex_new is cleared
    convert(0);
    if (half == 0) run(std::integral_constant<int, 0>{});
    else run(std::integral_constant<int, X::TEAM - 1>{});
    for (int j = threadIdx.x; j < X::TILES * kTile; j += X::WAVES * kWave) {
        const int tile = j / kTile, row = j % kTile / kRows, c = j % kRows;
        const int a = kTriRow[NBI][tile], b = kTriCol[NBI][tile];
        if (b >= nb) continue;
        double v = 0.0;
        for (int k = 0; k < X::BANKS; ++k)
            v += sums[((size_t)(k * X::TILES + tile) * 4 + row % 4) * kWave + 16 * (row / 4) + c];
        partial[((size_t)tile_index(a, b, nb) * gridDim.x + blockIdx.x) * kTile + j % kTile] = v;
    }
    if (threadIdx.x < X::SPREAD) {
        double v = 0.0;
        for (int k = 0; k < X::BANKS; ++k) v += spread[k * X::SPREAD + threadIdx.x];
        spread_out[(size_t)blockIdx.x * X::SPREAD + threadIdx.x] = v;
    }
}

// One workgroup per row segment: entries (i, 16 J .. 16 J + 15) of the table.  Thread (s, c) adds
// the partials s, s + 16, ... of G[i,j], G[j,j] and G[i,i]; the 16 slices are added in order.
// spread (EXACT, [groups][2][16 nb]): what affinity_gram_exact_kernel rounded away of each expert.
template <bool EXACT>
__global__ __launch_bounds__(256) void affinity_finish_kernel(
    const double* __restrict__ partial, int E, int groups, float* __restrict__ table,
    CloseList close, const double* __restrict__ spread, double columns) {
    constexpr int SUMS = EXACT ? 7 : 3;
    __shared__ double red[SUMS][16][kRows];
    const int nb = row_blocks(E);
    const int i = blockIdx.x, J = blockIdx.y, I = i / kRows;
    if (J < I) return;
    const int c = threadIdx.x % kRows, s = threadIdx.x / kRows, j = J * kRows + c;
    double sum[SUMS];                                           // G[i,j], G[i,i], G[j,j], spread of i and j
#pragma unroll
    for (int m = 0; m < SUMS; ++m) sum[m] = 0.0;
    if (j < E && j >= i) {
        const int ri = i % kRows;
        const double* pij = partial + (size_t)tile_index(I, J, nb) * groups * kTile + ri * kRows + c;
        const double* pii = partial + (size_t)tile_index(I, I, nb) * groups * kTile + ri * kRows + ri;
        const double* pjj = partial + (size_t)tile_index(J, J, nb) * groups * kTile + c * kRows + c;
        for (int g = s; g < groups; g += 16) {
            sum[0] += pij[(size_t)g * kTile];
            sum[1] += pii[(size_t)g * kTile];
            sum[2] += pjj[(size_t)g * kTile];
            if constexpr (EXACT) {
                const double* at = spread + (size_t)g * 2 * nb * kRows;
                sum[3] += at[i];
                sum[4] += at[j];
                sum[5] += at[nb * kRows + i];
                sum[6] += at[nb * kRows + j];
            }
        }
    }
#pragma unroll
    for (int m = 0; m < SUMS; ++m) red[m][s][c] = sum[m];
    __syncthreads();
    if (s != 0 || j >= E || j < i) return;
#pragma unroll
    for (int m = 0; m < SUMS; ++m) {
        sum[m] = 0.0;
        for (int k = 0; k < 16; ++k) sum[m] += red[m][k][c];
    }
    const double gij = sum[0], gii = sum[1], gjj = sum[2];
    if (i == j) {
        table[(size_t)i * E + i] = 0.f;
        return;
    }
    const double norms = gii + gjj;
    double sq = norms - 2.0 * gij;
    // an infinite weight in one of the two experts: the distance is infinite
    if (__builtin_isinf(norms) && (__builtin_isfinite(gii) || __builtin_isfinite(gjj))) sq = norms;
    const float dist = (float)sqrt(sq);
    table[(size_t)i * E + j] = dist;
    table[(size_t)j * E + i] = dist;
    bool drifts = false;
    if constexpr (EXACT) {
        // D^2 = sum of (v_i - v_j)^2 moves by the sum of r^2, and by 2 (v_i - v_j) (r_i - r_j) at random: with
        // independent signs a variance of 4 (v_i^2 + v_j^2) (r_i^2 + r_j^2), taken twice; of D a quarter of it / D^2
        const double r2 = sum[3] + sum[4];
        const double var = 2.0 * (sum[5] + sum[6] + (sum[3] * gjj + sum[4] * gii) / columns);
        drifts = var > kDrift * kDrift * sq * sq || r2 > kDrift * sq;
    }
    // (order of the list does not matter; two experts with infinite weights go there as well)
    if (sq < kClose * norms || drifts || (__builtin_isinf(gii) && __builtin_isinf(gjj))) {
        const int at = i / kCloseSide * side_blocks(E) + j / kCloseSide;
        if (atomicExch(close.flags + at, 1) == 0) close.blocks[atomicAdd(close.n, 1)] = at;
    }
}

// The listed blocks: squared differences of all 64 pairs in fp64, bound by the vector units (a
// subtraction and a multiply-add per pair and element).  The concatenated columns of the three
// matrices are dealt in `slabs` contiguous slabs; a workgroup takes a slab of a block at a time.
// The blocks of a slab run next to each other on one die and share its weights in the L2.  8-byte
// pieces: 16 of them, the next 16 and 64 fp64 sums fit in 256 registers.
template <typename T>
__global__ __launch_bounds__(kCloseThreads, 2) void affinity_close_kernel(
    const T* __restrict__ wg, const T* __restrict__ wu, const T* __restrict__ wd, int E, size_t n1,
    int slabs, CloseList close, double* __restrict__ partial /* [n][slabs][64] */) {
    constexpr int N = 8 / sizeof(T), S = kCloseSide;            // elements of a piece
    typedef const U64 __attribute__((address_space(1)))* Global;
    __shared__ double red[kCloseThreads / kWave][S * S];
    const int n = __builtin_amdgcn_readfirstlane(*close.n);
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    const size_t row_bytes = n1 * sizeof(T);
    const int per_matrix = (int)((row_bytes + 8 * kCloseThreads - 1) / (8 * kCloseThreads));
    const uint64_t base = (uint64_t)wg, to_up = (uint64_t)wu - base, to_down = (uint64_t)wd - (uint64_t)wu;
    const int die = blockIdx.x % kXcds, mine = (slabs - die + kXcds - 1) / kXcds;   // slabs of this die
    for (long long item = blockIdx.x / kXcds; item < (long long)mine * n; item += gridDim.x / kXcds) {
        const int slab = die + kXcds * (int)(item / n), at = (int)(item % n);
        const int code = __builtin_amdgcn_readfirstlane(close.blocks[at]);
        const int I = code / side_blocks(E), J = code % side_blocks(E);
        const int u0 = (int)(3ll * per_matrix * slab / slabs), u1 = (int)(3ll * per_matrix * (slab + 1) / slabs);
        double acc[S * S];                                      // diagonal blocks: the pairs a < b
#pragma unroll
        for (int p = 0; p < S * S; ++p) acc[p] = 0.0;
        auto sum = [&](auto diagonal) __attribute__((always_inline)) {
            constexpr bool DIAG = decltype(diagonal)::value;
            constexpr int ROWS = DIAG ? S : 2 * S;              // rows of I, then rows of J
            U64 next[ROWS];
            auto load = [&](int u) __attribute__((always_inline)) {
                const int uc = min(u, u1 - 1), m = uc / per_matrix;
                const size_t col = ((size_t)(uc - m * per_matrix) * kCloseThreads + threadIdx.x) * 8;
                const uint64_t p =
                    base + (m >= 1 ? to_up : 0) + (m == 2 ? to_down : 0) + (col < row_bytes ? col : 0);
#pragma unroll
                for (int r = 0; r < ROWS; ++r)
                    next[r] = *(Global)(p + (size_t)min((r < S ? I : J) * S + r % S, E - 1) * row_bytes);
                if (col >= row_bytes) {
#pragma unroll
                    for (int r = 0; r < ROWS; ++r) next[r] = U64{0, 0};
                }
                __builtin_amdgcn_sched_barrier(0);              // the requests stay ahead of their use
            };
            load(u0);
            for (int u = u0; u < u1; ++u) {
                U64 cur[ROWS];
#pragma unroll
                for (int r = 0; r < ROWS; ++r) cur[r] = next[r];
                load(u + 1);
#pragma unroll
                for (int k = 0; k < N; ++k) {
                    double v[ROWS];
#pragma unroll
                    for (int r = 0; r < ROWS; ++r) v[r] = (double)Half<T>::get(cur[r], k);
#pragma unroll
                    for (int a = 0; a < S; ++a)
#pragma unroll
                        for (int b = DIAG ? a + 1 : 0; b < S; ++b) {
                            const double df = v[a] - v[DIAG ? b : S + b];
                            acc[a * S + b] = fma(df, df, acc[a * S + b]);
                        }
                }
            }
        };
        if (I == J) sum(std::true_type{});
        else sum(std::false_type{});
        TransposeReduce<S * S, kWave / 2>::run(acc, lane);      // lane p: pair p of the wave
        red[wave][lane] = acc[0];
        __syncthreads();
        if (wave == 0) {
            double v = red[0][lane];
            for (int w = 1; w < kCloseThreads / kWave; ++w) v += red[w][lane];
            partial[((size_t)at * slabs + slab) * (S * S) + lane] = v;
        }
        __syncthreads();
    }
}

// One workgroup per listed block: thread (g, p) adds the slabs g, g + 4, ... of pair p.
__global__ __launch_bounds__(256) void affinity_close_finish_kernel(
    CloseList close, const double* __restrict__ partial, int slabs, int E, float* __restrict__ table) {
    constexpr int S = kCloseSide;
    __shared__ double red[4][S * S];
    const int n = *close.n, p = threadIdx.x % (S * S), g = threadIdx.x / (S * S);
    for (int at = blockIdx.x; at < n; at += gridDim.x) {
        double s = 0.0;
#pragma unroll 8
        for (int slab = g; slab < slabs; slab += 4) s += partial[((size_t)at * slabs + slab) * (S * S) + p];
        red[g][p] = s;
        __syncthreads();
        const int code = close.blocks[at];
        const int i = code / side_blocks(E) * S + p / S, j = code % side_blocks(E) * S + p % S;
        if (g == 0 && i < j && j < E) {
            const float dist = (float)sqrt(((red[0][p] + red[1][p]) + red[2][p]) + red[3][p]);
            table[(size_t)i * E + j] = dist;
            table[(size_t)j * E + i] = dist;
        }
        __syncthreads();
    }
}

template <int NBI>
hipError_t launch_gram_exact(const bf16_t* wg, const bf16_t* wu, const bf16_t* wd, int E, size_t n1,
                             double* partial, const CloseList& close, double* spread, hipStream_t s, int& groups) {
    typedef Exact<NBI> X;
    // one-time, thread-safe (C++11 static initialisation): raise the dynamic LDS limit
    static const hipError_t attr =
        hipFuncSetAttribute(reinterpret_cast<const void*>(&affinity_gram_exact_kernel<NBI>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)X::LDS);
    if (attr != hipSuccess) return attr;
    const size_t units = 3 * ((n1 + kUnit - 1) / kUnit), teams = X::TEAMS;
    groups = (int)(units < kMaxGroups * teams ? (units + teams - 1) / teams : kMaxGroups);
    hipLaunchKernelGGL((affinity_gram_exact_kernel<NBI>), dim3(groups), dim3(X::WAVES * kWave), X::LDS,
                       s, wg, wu, wd, E, n1, partial, close, spread);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_affinity_typed(const T* wg, const T* wu, const T* wd, int E, size_t n1,
                                 float* table, double* partial, hipStream_t s) {
    if (E <= 8) {
        const size_t want = (n1 / Piece<T>::N + kPairThreads - 1) / kPairThreads;
        const int pair_groups = (int)(want < (size_t)kPairGroups ? want : kPairGroups);
        if (E <= 4)
            hipLaunchKernelGGL((affinity_pairs_kernel<T, 4>), dim3(pair_groups), dim3(kPairThreads),
                               0, s, wg, wu, wd, E, n1, partial);
        else
            hipLaunchKernelGGL((affinity_pairs_kernel<T, 8>), dim3(pair_groups), dim3(kPairThreads),
                               0, s, wg, wu, wd, E, n1, partial);
        hipLaunchKernelGGL(affinity_pairs_finish_kernel, dim3(E * E), dim3(kWave), 0, s, partial, E,
                           pair_groups, table);
        return hipGetLastError();
    }
    const int nb = row_blocks(E), ns = (nb + kSuper - 1) / kSuper;
    const CloseList close(partial, E);
    const size_t pieces = 3 * ((n1 * sizeof(T) + 8 * kCloseThreads - 1) / (8 * kCloseThreads));
    const int slabs = (int)(pieces < (size_t)kCloseSlabs ? pieces : kCloseSlabs);
    int groups;                                  // workgroups of the Gram kernel, each with partial sums
    bool exact = false;
    if constexpr (std::is_same<T, bf16_t>::value) {
        // integer products from 2.5 million weights per matrix on (9 experts x 512 x 704: 34.1 -> 31.0 us, 40 x
        // 256 x 256: 31.4 -> 29.0); below, the passes that move int32 sums to fp64 cost more than the
        // products gain (32 x 256 x 256: 23.9 -> 27.7, 64 x 264 x 65: 30.0 -> 36.6)
        exact = nb <= kSuper && (size_t)E * n1 >= 2500000;
        if (exact) {
            double* out = close.spread(E);
            hipError_t err;
            if (nb == 1) err = launch_gram_exact<1>(wg, wu, wd, E, n1, partial, close, out, s, groups);
            else if (nb == 2) err = launch_gram_exact<2>(wg, wu, wd, E, n1, partial, close, out, s, groups);
            else if (nb == 3) err = launch_gram_exact<3>(wg, wu, wd, E, n1, partial, close, out, s, groups);
            else err = launch_gram_exact<4>(wg, wu, wd, E, n1, partial, close, out, s, groups);
            if (err != hipSuccess) return err;
            hipLaunchKernelGGL(affinity_finish_kernel<true>, dim3(E, nb), dim3(256), 0, s, partial, E, groups,
                               table, close, out, 3.0 * (double)n1);
        }
    }
    if (!exact) {
        const size_t units = 3 * ((n1 + 4 * Piece<T>::N - 1) / (4 * Piece<T>::N));
        groups = (int)(units < (size_t)kMaxGroups * 8 ? (units + 7) / 8 : kMaxGroups);
#define SPECMOE_GRAM(NBI, OFF, WAVES, PF, GY)                                                     \
    hipLaunchKernelGGL((affinity_gram_kernel<T, NBI, OFF, WAVES, PF>), dim3(groups, GY),          \
                       dim3(WAVES * kWave), 0, s, wg, wu, wd, E, n1, partial, close)
        if (nb == 1) SPECMOE_GRAM(1, false, 16, 4, 1);
        else if (nb == 2) SPECMOE_GRAM(2, false, 8, 4, 1);
        else if (nb == 3) SPECMOE_GRAM(3, false, 8, 2, 1);
        else SPECMOE_GRAM(4, false, 8, 2, ns);
        if (ns > 1) SPECMOE_GRAM(4, true, 8, 1, ns * (ns - 1) / 2);
#undef SPECMOE_GRAM
        hipLaunchKernelGGL(affinity_finish_kernel<false>, dim3(E, nb), dim3(256), 0, s, partial, E, groups,
                           table, close, nullptr, 0.0);
    }
    hipLaunchKernelGGL((affinity_close_kernel<T>), dim3(kCloseGroups), dim3(kCloseThreads), 0, s, wg,
                       wu, wd, E, n1, slabs, close, partial);
    hipLaunchKernelGGL(affinity_close_finish_kernel, dim3(256), dim3(256), 0, s, close, partial, slabs,
                       E, table);
    return hipGetLastError();
}

}  // namespace

// Room for 1024 partials of 64 doubles per pair of 8-expert blocks: what the direct sums of up to
// 8 experts take.  Beyond that half of it holds the partial sums - of the Gram matrix (at most
// kMaxGroups x 256 doubles per pair of 16-expert blocks: with n = row_blocks(E), n (n + 1) / 2 x 128
// partials of 512 doubles, and 8-expert blocks come in at least n (2 n - 1) >= n (n + 1) pairs from
// n = 2 on, in 3 for n = 1, of 64 partials of 512 doubles), then of the listed blocks - and CloseList
// follows them, with at most 256 x 128 doubles behind it.
size_t affinity_workspace_bytes(int E) {
    const size_t nb8 = (size_t)(E + 7) / 8;
    return nb8 * (nb8 + 1) / 2 * 1024 * 64 * sizeof(double);
}

hipError_t launch_affinity_table(const void* wg, const void* wu, const void* wd, int E, int d,
                                 int f, int dtype, float* table, void* workspace, hipStream_t s) {
    const size_t n1 = (size_t)d * f;
    double* partial = static_cast<double*>(workspace);
    if (dtype == 0)
        return launch_affinity_typed((const float*)wg, (const float*)wu, (const float*)wd, E, n1,
                                     table, partial, s);
    return launch_affinity_typed((const bf16_t*)wg, (const bf16_t*)wu, (const bf16_t*)wd, E, n1,
                                 table, partial, s);
}

}  // namespace specmoe
