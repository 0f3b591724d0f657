// Offline table of pairwise L2 distances between the experts of one block (SpecMoE Sec. 3.2
// "Affinity-based expert selection mechanism", Fig. 8).  An expert's parameters are its three
// matrices together, so D[i,j]^2 = sum over gate, up and down of (W_i - W_j)^2.
//
// More than 8 experts.  Summing the squared differences pair by pair costs a subtraction and a
// fused multiply-add per element and PAIR (2016 pairs for 64 experts: bound by the vector units,
// 3.36 ms at 64 experts x 3 x 2048 x 1408).  Here the table comes out of one Gram matrix,
//   D[i,j]^2 = G[i,i] + G[j,j] - 2 G[i,j].
// bf16, up to 64 experts, from 2.5 million weights per matrix on: G = W W^T from integer products of the digits of W
// (affinity_gram_exact_kernel): a distance may differ by 2^-27 of it from the direct sum, in general not at all.
// Otherwise G = V V^T with V_i = W_i - W_0 (distances do not change when one expert is subtracted from all),
// products and sums in fp64: v_mfma_f64_16x16x4 takes 64 cycles for 16 x 16 pairs x 4 columns; a wave holds
// up to 64 experts at a time (10 tiles of the upper triangle: 640 cycles per 4 columns of 64 experts,
// 0.57 ms at the shape above) and reads and converts every weight once.  Measured, bf16, normal weights, us, fp64 /
// integer products: 12 experts x 2048 x 2048 159 / 120 (pair by pair 249), 16 x 4096 x 4096 587 / 389, 24 x 2048 x 1408
// 253 / 169 (500), 40 x 2048 x 1408 450 / 263, 64 x 2048 x 1408 702 / 365 (3360); 130 x 1024 x 704 in fp64 1430.
// Cancellation: a pair that lies closer together than 2^-10 of its norms (of W or V: subtracting W_0 removes what
// all experts have in common) - a copy, or in fp64 any pair where expert 0 lies far from all others - takes its
// distance from its differences: the finish kernel lists the 8 x 8 blocks of the table that hold such a pair, and a
// second pass sums the differences of all pairs of a listed block.  The pairs that the integer products may have moved by
// more than 2^-27 go there too.  A block costs as much however many of its pairs are listed: all of them, 64 experts x 2048 x
// 1408, take 1.9 ms more, 16 x 4096 x 4096 0.9 - where direct sums alone would take 0.97, so up to 16 experts such
// a table is the one case where they would be faster.
// What the integer products take by the kind of weights (64 x 2048 x 1408, a call waited for, us; fp64 760 for any
// weights): normal, or Student's t of 3 degrees 440; experts of magnitudes from 1e-3 to 1e3 455; 1 % of the weights 3000 times
// larger 515; half of them 1e-34 times smaller 495; magnitudes that spread over more than about 2^22, so that the whole table is
// listed (log-normal with a standard deviation of 2 times normal, or steps up to 2^24) 2250 to 2360.
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
    // behind the list: [groups][16 row_blocks(E)] (affinity_gram_exact_kernel)
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

// bf16, 9 to 64 experts: the Gram matrix of W itself from exact integer products.  bf16 numbers have few significant
// bits, so a weight is written as q * 2^ex, with one ex per row block (16 experts) for as long as it fits, q a whole
// number below 2^30 in four signed 8-bit digits, and v_mfma_i32_16x16x64_i8 multiplies the digits: 64 columns of
// 16 x 16 pairs in 16 instructions of 16 cycles where the fp64 instruction takes 16 of 64.  int32 sums are exact;
// they move to fp64 sums in LDS when an ex changes and after kExactColumns columns.  So the table holds the exact
// distances of the vectors q * 2^ex.  These are the weights themselves where none but zero is below 2^(ex + 7), whose
// last bit is 2^ex; ex puts the largest of the 16 x 64 weights at 2^(ex + 27) .. 2^(ex + 30) in general.  Where a weight is smaller,
// the squares of all residuals r = w - q * 2^ex of the unit (below 2^ex each) are added up.  By the triangle
// inequality a distance moves by at most |r_i| + |r_j|, in whatever columns and with whatever signs they are, and
// the finish kernel sends the pairs that this may move by more than 2^-27 to the second pass; fp32 rounds at 2^-24.
// Units of 64 columns with a number that is not finite, and the ragged last ones, go through the fp64 instruction.
// A team of waves shares a unit: each converts one row block, the digits meet in LDS, each multiplies a share
// of the tiles.  Between two barriers half of the waves of a SIMD multiply unit i and then convert unit i + 1, the others
// do it in the opposite order, so matrix and vector units run side by side.  At 64 x 2048 x 1408 either is busy for
// less than half of the time (10 vector instructions per weight and lane); the rest is the chain of a step: barrier,
// digits out of LDS, products, conversion.  So 64 experts take 128 columns per step (a call waited for: 64 columns 518 us, 128
// 440); 12 waves with 64 columns take 449.
constexpr int kExactColumns = 28672;         // 4 products per sum, at most 2^14 each: below 2^31
constexpr int kTopBit = 27;                  // a new ex puts the largest weight of a unit at 2^27 .. 2^28
constexpr int kLowBit = 17;                  // below, a unit whose weights lose bits may take a new ex
constexpr int kLowUnits = 32;                // ... if it has been the same for so many units
constexpr int kMinEx = -120;                 // 2^-ex is a float

typedef int intx4 __attribute__((ext_vector_type(4)));
typedef unsigned short ushortx2 __attribute__((ext_vector_type(2)));

// twice the bits without the sign (which order bf16 numbers by size) from which ex holds a weight with its
// last one, and from which it would overflow
__device__ __forceinline__ int holds_from(int ex) { return (ex + 7 + 127) << 8; }
__device__ __forceinline__ int overflows_at(int ex) { return min((ex + 30 + 127) << 8, 0xff00); }

template <int NBI> struct Exact {
    static constexpr int SUB = NBI == 4 ? 2 : 1, UNIT = 64 * SUB;       // columns of a unit: 16 * SUB per lane
    static constexpr int WAVES = NBI == 4 ? 8 : NBI > 1 ? 12 : 16;     // as many as the registers allow
    static constexpr int AHEAD = 2;                             // units in flight per team
    static constexpr int TILES = NBI * (NBI + 1) / 2, DIGITS = 4;
    static constexpr int TEAM = NBI, TEAMS = WAVES / TEAM;
    static constexpr int HT = (TILES + TEAM - 1) / TEAM;        // tiles a wave multiplies, at most
    __host__ __device__ static constexpr int first_tile(int part) {
        return part * (TILES / TEAM) + (part < TILES % TEAM ? part : TILES % TEAM);
    }
    // teams that add at a time, each to sums of its own (as the LDS holds)
    static constexpr int BANKS = NBI == 4 ? 1 : NBI == 1 ? 8 : TEAMS;
    static constexpr int SPREAD = NBI * kRows;
    static constexpr size_t SUMS = (size_t)BANKS * TILES * kTile * sizeof(double);
    static constexpr size_t DIGIT_BYTES = (size_t)2 * WAVES * SUB * DIGITS * kWave * 16;
    static constexpr int REST = WAVES * kRows;
    static constexpr size_t LDS = SUMS + DIGIT_BYTES + BANKS * SPREAD * sizeof(double) +
                                  REST * sizeof(float) + 4 * WAVES * sizeof(int);
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
    double* __restrict__ spread_out /* [groups][NBI * kRows] */) {
    typedef Exact<NBI> X;
    constexpr int DIGITS = X::DIGITS, TEAMS = X::TEAMS, SUB = X::SUB, UNIT = X::UNIT;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    double* sums = reinterpret_cast<double*>(lds_raw);          // [BANKS][TILES][4][kWave]
    intx4* digits = reinterpret_cast<intx4*>(lds_raw + X::SUMS);   // [2][TEAMS][NBI][SUB][DIGITS][kWave]
    double* spread = reinterpret_cast<double*>(lds_raw + X::SUMS + X::DIGIT_BYTES);   // [BANKS][NBI * kRows]
    float* rest = reinterpret_cast<float*>(spread + X::BANKS * X::SPREAD);   // [waves][kRows]: sum of (r / 2^ex)^2
    int* ex_now = reinterpret_cast<int*>(rest + X::REST);       // [waves]: ex of acc
    int* ex_new = ex_now + X::WAVES;                            // ex of the newest digits
    int* flags = ex_new + X::WAVES;                             // [2][waves]: 1 ex changed, 2 fp64 unit
    const int lane = threadIdx.x % kWave, g = lane / kRows;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int part = wave / TEAMS, team = wave % TEAMS;         // part: the row block that the wave converts
    const int nb = row_blocks(E);
    if (blockIdx.x == 0) {                                      // nothing listed yet
        const int ns = side_blocks(E);
        if (threadIdx.x == 0) *close.n = 0;
        for (int i = threadIdx.x; i < ns * ns; i += X::WAVES * kWave) close.flags[i] = 0;
    }
    for (int i = threadIdx.x; i < X::BANKS * X::TILES * kTile; i += X::WAVES * kWave) sums[i] = 0.0;
    for (int i = threadIdx.x; i < X::BANKS * X::SPREAD; i += X::WAVES * kWave) spread[i] = 0.0;
    if (threadIdx.x < 2 * X::WAVES) ex_now[threadIdx.x] = kMinEx;

    const int units = (int)((n1 + UNIT - 1) / UNIT), total = 3 * units;
    const int stride = gridDim.x * TEAMS, iters = (total + stride - 1) / stride;
    const int first = blockIdx.x * TEAMS + team;
    const uint64_t base = (uint64_t)wg, to_up = (uint64_t)wu - base, to_down = (uint64_t)wd - (uint64_t)wu;
    typedef const U128 __attribute__((address_space(1)))* Global;
    // unit u: its matrix and first column (the last unit of a matrix may be ragged)
    auto unit_base = [&](int u, size_t& col0) __attribute__((always_inline)) -> uint64_t {
        const int uc = min(u, total - 1), m = uc / units;
        col0 = (size_t)(uc - m * units) * UNIT;
        return base + (m >= 1 ? to_up : 0) + (m == 2 ? to_down : 0);
    };
    auto row_bytes = [&](int b) __attribute__((always_inline)) -> size_t {
        return (size_t)min(b * kRows + lane % kRows, E - 1) * n1 * 2;
    };

    // ---- loads, AHEAD units ahead: this wave's row block; a lane's columns are pieces of 8.  In place of a
    // ragged unit the last whole one is read (its digits are not used).
    const uint64_t row_at = row_bytes(part) + 16 * g;
    U128 raw[X::AHEAD][2 * SUB];
    auto load = [&](U128 (&to)[2 * SUB], int u) __attribute__((always_inline)) {
        size_t col0;
        const uint64_t W = unit_base(u, col0);
        const uint64_t at = W + (col0 + UNIT > n1 ? n1 - UNIT : col0) * 2;
#pragma unroll
        for (int h = 0; h < 2 * SUB; ++h) to[h] = *(Global)(at + row_at + 64 * h);
        __builtin_amdgcn_sched_barrier(0);      // the loads stay here, ahead of their use
    };

    // ---- digits of unit i (in `from`) into slot i % 2, then the loads of unit i + AHEAD
    int ex = kMinEx, ex_since = -kLowUnits;     // ex and the first unit that had it
    float left = 0.f, left_new = 0.f;           // sum of (r / 2^ex)^2 of row lane % 16: units in acc, newest unit
    auto convert = [&](U128 (&from)[2 * SUB], int i) __attribute__((always_inline)) {
        const int u = first + i * stride;
        left += left_new;
        left_new = 0.f;
        ushortx2 most2 = {0, 0}, least2 = {0xffff, 0xffff};     // of this lane's columns; least: minus 1 (zero: 0xffff)
#pragma unroll
        for (int j = 0; j < 8 * SUB; ++j) {
            const uint32_t pair = from[j / 4][j % 4];
            const ushortx2 a = __builtin_bit_cast(ushortx2, pair) << 1;
            most2 = __builtin_elementwise_max(most2, a);
            least2 = __builtin_elementwise_min(least2, (ushortx2)(a - (ushortx2){1, 1}));
        }
        int most = max((int)most2[0], (int)most2[1]), least = min((int)least2[0], (int)least2[1]) + 1;
        int flag = 0;
        bool loses = false;
        if (!__all(most < overflows_at(ex) && least >= holds_from(ex))) {
            most = __builtin_amdgcn_readfirstlane(wave_all(most, [](int a, int b) { return max(a, b); }));
            least = __builtin_amdgcn_readfirstlane(wave_all(least, [](int a, int b) { return min(a, b); }));
            if (most >= 0xff00) {
                flag = 2;
            } else if (most >= overflows_at(ex) || (most < (ex + kLowBit + 127) << 8 && ex > kMinEx &&
                                                    i - ex_since >= kLowUnits)) {
                flag = 1;
                ex = max((most >> 8) - 127 - kTopBit, kMinEx);
                ex_since = i;
                if (lane == 0) ex_new[wave] = ex;
            }
            loses = least < holds_from(ex);
        }
        const float scale = __uint_as_float((uint32_t)(127 - ex) << 23);    // 2^-ex
        intx4* slot = digits + ((size_t)((i & 1) * TEAMS + team) * NBI + part) * SUB * DIGITS * kWave + lane;
#pragma unroll
        for (int c = 0; c < SUB; ++c) {
            intx4 d[DIGITS];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                uint32_t q[4];                      // + 0x808080: the three low digits + 128, the top one as it is
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    q[k] = (uint32_t)(int)(Piece<bf16_t>::get(from[2 * c + j / 2], (4 * j + k) % 8) * scale) + 0x808080u;
                const uint32_t p01 = __builtin_amdgcn_perm(q[1], q[0], 0x05010400u);
                const uint32_t p23 = __builtin_amdgcn_perm(q[3], q[2], 0x05010400u);
                const uint32_t h01 = __builtin_amdgcn_perm(q[1], q[0], 0x07030602u);
                const uint32_t h23 = __builtin_amdgcn_perm(q[3], q[2], 0x07030602u);
                d[0][j] = (int)(__builtin_amdgcn_perm(p23, p01, 0x05040100u) ^ 0x80808080u);
                d[1][j] = (int)(__builtin_amdgcn_perm(p23, p01, 0x07060302u) ^ 0x80808080u);
                d[2][j] = (int)(__builtin_amdgcn_perm(h23, h01, 0x05040100u) ^ 0x80808080u);
                d[3][j] = (int)__builtin_amdgcn_perm(h23, h01, 0x07060302u);
            }
#pragma unroll
            for (int x = 0; x < DIGITS; ++x) slot[(c * DIGITS + x) * kWave] = d[x];
        }
        if ((size_t)(u % units + 1) * UNIT > n1) flag = 2;     // ragged
        if (flag != 2 && u < total && loses) {
#pragma unroll
            for (int j = 0; j < 16 * SUB; ++j) {
                const float a = Piece<bf16_t>::get(from[j / 8], j % 8) * scale, r = a - truncf(a);
                left_new += r != 0.f ? fmaxf(r * r, 0x1p-100f) : 0.f;       // (no underflow)
            }
        }
        if (lane == 0) flags[(i & 1) * X::WAVES + wave] = u < total ? flag : 0;
        load(from, u + X::AHEAD * stride);
    };

    // ---- the main loop, for each part of a team (PART); FIRST: multiplies before it converts
    auto run = [&](auto part_tag, auto first_tag) __attribute__((always_inline)) {
    constexpr int T0 = X::first_tile(decltype(part_tag)::value), T1 = X::first_tile(decltype(part_tag)::value + 1);
    constexpr bool FIRST = decltype(first_tag)::value;
    // products of a slot; this wave's tiles
    intx4 acc[X::HT][2 * DIGITS - 1];           // [x + y]: digit x of the row times digit y of the column
    auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < X::HT; ++t)
#pragma unroll
            for (int s = 0; s < 2 * DIGITS - 1; ++s) acc[t][s] = intx4{0, 0, 0, 0};
    };
    auto multiply = [&](int i) __attribute__((always_inline)) {
        const intx4* slot = digits + (size_t)((i & 1) * TEAMS + team) * NBI * SUB * DIGITS * kWave + lane;
#pragma unroll
        for (int c = 0; c < SUB; ++c) {
            intx4 da[DIGITS], db[DIGITS];
#pragma unroll
            for (int t = T0; t < T1; ++t) {
                const int a = kTriRow[NBI][t], b = kTriCol[NBI][t];
#pragma unroll
                for (int x = 0; x < DIGITS; ++x) {
                    if (t == T0 || a != kTriRow[NBI][t - 1]) da[x] = slot[((a * SUB + c) * DIGITS + x) * kWave];
                    db[x] = a == b ? da[x] : slot[((b * SUB + c) * DIGITS + x) * kWave];
                }
#pragma unroll
                for (int z = 0; z < DIGITS; ++z)
#pragma unroll
                    for (int x = 0; x < DIGITS; ++x) {              // neighbours add to different sums
                        const int y = (x + z) % DIGITS;
                        acc[t - T0][x + y] =
                            __builtin_amdgcn_mfma_i32_16x16x64_i8(da[x], db[y], acc[t - T0][x + y], 0, 0, 0);
                    }
            }
        }
    };
    // all waves: acc into the sums (in one order of additions); wide: unit i of this team in fp64
    auto settle = [&](int i, int held, bool wide) __attribute__((always_inline)) {
        left += __shfl_xor(left, 16, kWave);
        left += __shfl_xor(left, 32, kWave);
        rest[wave * kRows + lane % kRows] = left;
        left = 0.f;
        __syncthreads();
        double* mine = sums + (size_t)(team % X::BANKS) * X::TILES * kTile;
        double* spread_mine = spread + (team % X::BANKS) * X::SPREAD;
        for (int turn = 0; turn < TEAMS / X::BANKS; ++turn) {
            if (turn == team / X::BANKS) {
#pragma unroll
                for (int t = T0; t < T1; ++t) {
                    if (held == 0) continue;
                    const int a = kTriRow[NBI][t], b = kTriCol[NBI][t];
                    const int wa = a * TEAMS + team, wb = b * TEAMS + team;     // the waves that converted them
                    const int both = ex_now[wa] + ex_now[wb];
                    // a lane holds rows 4 * (lane / 16) + r, r = 0 .. 3, column lane % 16
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        double v = (double)acc[t - T0][2 * DIGITS - 2][r];
#pragma unroll
                        for (int s = 2 * DIGITS - 3; s >= 0; --s) v = fma(v, 256.0, (double)acc[t - T0][s][r]);
                        mine[(t * 4 + r) * kWave + lane] += ldexp(v, both);
                        if (a == b && 4 * g + r == lane % kRows)
                            spread_mine[a * kRows + lane % kRows] +=
                                ldexp((double)rest[wa * kRows + lane % kRows], both);
                    }
                }
                if (wide) {
                    size_t col0;
                    const uint64_t W = unit_base(first + i * stride, col0);
                    for (int t = T0; t < T1; ++t) {
                        const size_t oa = row_bytes(kTriRow[NBI][t]), ob = row_bytes(kTriCol[NBI][t]);
                        doublex4 d = doublex4{0.0, 0.0, 0.0, 0.0};
                        for (int h = 0; h < 2 * SUB; ++h) {
                            const size_t col = col0 + 32 * h + 8 * g;
                            U128 ra = {0, 0, 0, 0}, rb = ra;
                            if (col < n1) {
                                ra = *(Global)(W + col * 2 + oa);
                                rb = *(Global)(W + col * 2 + ob);
                            }
#pragma unroll
                            for (int j = 0; j < 8; ++j)
                                d = __builtin_amdgcn_mfma_f64_16x16x4f64((double)Piece<bf16_t>::get(ra, j),
                                                                         (double)Piece<bf16_t>::get(rb, j), d, 0, 0, 0);
                        }
                        // element q of a lane is row 4 * q + lane / 16, column lane % 16 of its tile
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            mine[(t * 4 + g) * kWave + 16 * q + lane % kRows] += d[q];
                    }
                }
            }
            __syncthreads();
        }
        if (threadIdx.x < X::WAVES) ex_now[threadIdx.x] = ex_new[threadIdx.x];
        __syncthreads();
        clear();
    };

    clear();
    int held = 0;                               // units in acc
    // unit i; `next` has the weights of unit i + 1; true after the last one
    auto step = [&](int i, U128 (&next)[2 * SUB]) __attribute__((always_inline)) -> bool {
        __syncthreads();                        // digits and flags of unit i are there
        const int flag = i < iters ? flags[(i & 1) * X::WAVES + lane % X::WAVES] : 1;
        bool plain = first + i * stride < total;                // the same in all waves of a team
        if (held == kExactColumns / UNIT || __any(flag != 0)) {
            const bool wide = __any(flag == 2 && lane % X::WAVES % TEAMS == team);
            settle(i, held, wide);
            plain = plain && !wide;
            held = 0;
        }
        if (i == iters) return true;
        ++held;
        if (FIRST && plain) multiply(i);
        convert(next, i + 1);
        if (!FIRST && plain) multiply(i);
        return false;
    };
    bool done = false;
    for (int i = 0; !done; i += X::AHEAD) {
#pragma unroll
        for (int p = 0; p < X::AHEAD; ++p)
            if (!done) done = step(i + p, raw[(p + 1) % X::AHEAD]);
    }
    };
#pragma unroll
    for (int p = 0; p < X::AHEAD; ++p) load(raw[p], first + p * stride);
    __syncthreads();                            // ex_new is cleared
    convert(raw[0], 0);
    // The waves of a team meet in barriers of several copies of this code: a barrier counts the waves that have
    // arrived, wherever they are.
    auto of = [&](auto part_tag) __attribute__((always_inline)) {
        if constexpr (X::TEAM == 1) {
            if (2 * wave < X::WAVES) run(part_tag, std::true_type{});
            else run(part_tag, std::false_type{});
        } else {
            run(part_tag, std::integral_constant<bool, 2 * decltype(part_tag)::value < X::TEAM>{});
        }
    };
    if (part == 0) of(std::integral_constant<int, 0>{});
    if constexpr (NBI > 1) if (part == 1) of(std::integral_constant<int, 1>{});
    if constexpr (NBI > 2) if (part == 2) of(std::integral_constant<int, 2>{});
    if constexpr (NBI > 3) if (part == 3) of(std::integral_constant<int, 3>{});
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
// spread (EXACT, [groups][16 nb]): squares of what affinity_gram_exact_kernel rounded away of each expert.
template <bool EXACT>
__global__ __launch_bounds__(256) void affinity_finish_kernel(
    const double* __restrict__ partial, int E, int groups, float* __restrict__ table,
    CloseList close, const double* __restrict__ spread) {
    constexpr int SUMS = EXACT ? 5 : 3;
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
                const double* at = spread + (size_t)g * nb * kRows;
                sum[3] += at[i];
                sum[4] += at[j];
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
        // the squares were summed in fp32: 1 % covers that
        const double moves = sqrt(sum[3]) + sqrt(sum[4]);
        drifts = 1.01 * moves * moves > kDrift * kDrift * sq;
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
    const size_t units = 3 * ((n1 + X::UNIT - 1) / X::UNIT), teams = X::TEAMS;
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
        // integer products from 2.5 million weights per matrix on (fp64 / integer, us: 9 experts x 512 x 704 33.2 /
        // 29.9, 40 x 256 x 256 31.1 / 27.2); below, the passes that move int32 sums to fp64 cost what the products
        // gain (9 x 256 x 512 21.4 / 24.2, 16 x 256 x 512 21.6 / 24.6, 32 x 256 x 256 23.8 / 23.8)
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
                               table, close, out);
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
                           table, close, nullptr);
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
// follows them, with at most 256 x 64 doubles behind it.
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
