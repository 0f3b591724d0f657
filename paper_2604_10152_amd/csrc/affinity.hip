// Offline table of pairwise L2 distances between the experts of one block (SpecMoE Sec. 3.2
// "Affinity-based expert selection mechanism", Fig. 8).  An expert's parameters are its three
// matrices together, so D[i,j]^2 = sum over gate, up and down of (W_i - W_j)^2.
//
// More than 8 experts.  Summing the squared differences pair by pair costs a subtraction and a
// fused multiply-add per element and PAIR (2016 pairs for 64 experts: bound by the vector units,
// 3.36 ms at 64 experts x 3 x 2048 x 1408).  Here the table comes out of one Gram matrix on the
// fp64 matrix cores: with V_i = W_i - W_0 (distances do not change when one expert is subtracted
// from all),
//   D[i,j]^2 = G[i,i] + G[j,j] - 2 G[i,j],   G = V V^T,
// products and sums in fp64.  v_mfma_f64_16x16x4 takes 64 cycles for 16 x 16 pairs x 4 columns; a
// wave holds up to 64 experts at a time (10 tiles of the upper triangle: 640 cycles per 4 columns
// of 64 experts, 0.57 ms at the shape above) and reads and converts every weight once.  Measured,
// bf16, pair by pair / Gram matrix: 12 experts x 2048 x 2048 249 / 160 us, 16 x 5120 x 8192 2.29 / 1.45
// ms, 24 x 2048 x 1408 500 / 253 us, 64 x 2048 x 1408 3.36 / 0.70 ms, 130 x 1024 x 704 7.39 / 1.43.
// Cancellation: subtracting W_0 removes what all experts have in common (experts grown from one
// dense model).  A pair that still lies closer together than 2^-10 of its norms - a copy, or any pair
// where expert 0 lies far from all others - takes its distance from its differences: the finish
// kernel lists the 8 x 8 blocks of the table that hold such a pair, and a second pass sums the
// differences of all pairs of a listed block, so no distance is less exact than a direct sum.  A
// block costs as much however many of its pairs are close.  Measured, us: no pair close / two copies /
// expert 0 far from all others (every other pair close) / direct sums of the whole table: 64 experts x
// 2048 x 1408 708 / 738 / 2340 / 3360, 16 x 4096 x 4096 608 / 735 / 1210 / 966, 12 x 2048 x 2048 168 / 204 /
// 329 / 260 - so up to 16 experts a table full of close pairs is the one case where direct sums alone
// would be faster.
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
//   affinity_gram_kernel      partial Gram matrices, one per workgroup
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

// One workgroup per row segment: entries (i, 16 J .. 16 J + 15) of the table.  Thread (s, c) adds
// the partials s, s + 16, ... of G[i,j], G[j,j] and G[i,i]; the 16 slices are added in order.
__global__ __launch_bounds__(256) void affinity_finish_kernel(
    const double* __restrict__ partial, int E, int groups, float* __restrict__ table,
    CloseList close) {
    __shared__ double red[3][16][kRows];
    const int nb = row_blocks(E);
    const int i = blockIdx.x, J = blockIdx.y, I = i / kRows;
    if (J < I) return;
    const int c = threadIdx.x % kRows, s = threadIdx.x / kRows, j = J * kRows + c;
    double gij = 0.0, gii = 0.0, gjj = 0.0;
    if (j < E && j >= i) {
        const int ri = i % kRows;
        const double* pij = partial + (size_t)tile_index(I, J, nb) * groups * kTile + ri * kRows + c;
        const double* pii = partial + (size_t)tile_index(I, I, nb) * groups * kTile + ri * kRows + ri;
        const double* pjj = partial + (size_t)tile_index(J, J, nb) * groups * kTile + c * kRows + c;
        for (int g = s; g < groups; g += 16) {
            gij += pij[(size_t)g * kTile];
            gii += pii[(size_t)g * kTile];
            gjj += pjj[(size_t)g * kTile];
        }
    }
    red[0][s][c] = gij; red[1][s][c] = gii; red[2][s][c] = gjj;
    __syncthreads();
    if (s != 0 || j >= E || j < i) return;
    gij = gii = gjj = 0.0;
    for (int k = 0; k < 16; ++k) { gij += red[0][k][c]; gii += red[1][k][c]; gjj += red[2][k][c]; }
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
    // (order of the list does not matter; two experts with infinite weights go there as well)
    if (sq < kClose * norms || (__builtin_isinf(gii) && __builtin_isinf(gjj))) {
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
    const size_t units = 3 * ((n1 + 4 * Piece<T>::N - 1) / (4 * Piece<T>::N));
    const int groups = (int)(units < (size_t)kMaxGroups * 8 ? (units + 7) / 8 : kMaxGroups);
    const CloseList close(partial, E);
    const size_t pieces = 3 * ((n1 * sizeof(T) + 8 * kCloseThreads - 1) / (8 * kCloseThreads));
    const int slabs = (int)(pieces < (size_t)kCloseSlabs ? pieces : kCloseSlabs);
#define SPECMOE_GRAM(NBI, OFF, WAVES, PF, GY)                                                     \
    hipLaunchKernelGGL((affinity_gram_kernel<T, NBI, OFF, WAVES, PF>), dim3(groups, GY),          \
                       dim3(WAVES * kWave), 0, s, wg, wu, wd, E, n1, partial, close)
    if (nb == 1) SPECMOE_GRAM(1, false, 16, 4, 1);
    else if (nb == 2) SPECMOE_GRAM(2, false, 8, 4, 1);
    else if (nb == 3) SPECMOE_GRAM(3, false, 8, 2, 1);
    else SPECMOE_GRAM(4, false, 8, 2, ns);
    if (ns > 1) SPECMOE_GRAM(4, true, 8, 1, ns * (ns - 1) / 2);
#undef SPECMOE_GRAM
    hipLaunchKernelGGL(affinity_finish_kernel, dim3(E, nb), dim3(256), 0, s, partial, E, groups,
                       table, close);
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
// follows them.
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
