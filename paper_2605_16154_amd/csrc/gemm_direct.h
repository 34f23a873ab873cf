// Products of fp32 matrices that lie as the caller gave them, row-major and unpadded, on the fp32 matrix instructions
// (v_mfma_f32_32x32x2_f32), with the activation fused into their epilogues (internal header): the direct route of the fp32 path.
// Against operands in blocks (gemm_floats.h, gemm_thirds.h) nothing is re-laid-out before the first product, which is what counts for few
// rows under a wide head and for heads of a tile or two.
#pragma once

#include "gemm_floats.h"

namespace pcm {

constexpr int kDirectThreads = 256;
constexpr int kDirectStep = 16;        // reduction steps are 16 wide
constexpr int kDirectRowTile = 128;    // live rows are rounded up to this: the tallest row tile

struct F32Problem {
    const float *A, *B;
    const float *A2, *B2;   // operands of a second product of the same sizes and layouts (see Second)
    int64_t lda, ldb;
    int M, N, K;
    int k_per_split;        // slice blockIdx.z covers [z, z + 1) * k_per_split of the reduction
    int tiles_n;            // column tiles of one right operand
    // rows of the batch: kLiveM: row tiles beyond the live rows (rounded up to kDirectRowTile) are skipped; kLiveK: the
    // reduction ends with the live rows
    const int32_t* n_kept;
    int max_chunks, rows_per_chunk, live;
};
enum LiveRows : int { kLiveUnused = 0, kLiveM = 1, kLiveK = 2 };

// A second product in the launch: kNone; kPair: column tiles tiles_n .. 2 tiles_n - 1 are those of A B2; kInterleaved: the
// columns are 32 of B, the same 32 of B2, and so on, so that a wavefront holds both of a pair; kSum: slice 0 is A B,
// slice 1 A2 B2, to be added as the slices of a split reduction are.
enum Second : int { kNone = 0, kPair = 1, kInterleaved = 2, kSum = 3 };

// Where a lane's accumulators belong: register e of tile (i, j) is row row(i, e), column col(j) of the product.
// (kInterleaved: col(j) is the column of B for even j and of B2 for odd j.)
template <int kI, int kJ, int kSecond>
struct F32Coord {
    int m0, n0, wm, wn, lane, split, right;
    __device__ int row(int i, int e) const { return m0 + (wm * kI + i) * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3); }
    __device__ int col(int j) const {
        if (kSecond == kInterleaved) return n0 / 2 + wn * (kJ / 2) * 32 + (j / 2) * 32 + (lane & 31);
        return n0 + (wn * kJ + j) * 32 + (lane & 31);
    }
};

__device__ inline int64_t live_rows_of(const F32Problem& p) { return live_rows(p.n_kept, p.max_chunks, p.rows_per_chunk); }

// One tile of 64 kI x 64 kJ per workgroup of four wavefronts (2 x 2), each 32 kI x 32 kJ.  Steps are 16 wide; operand
// tiles are double-buffered in LDS as [k][row] (a lane feeds one row and every second k, so a fragment is one 4-byte read
// of consecutive rows) and the next step's values are on the way to registers meanwhile.  Bound by the matrix pipe: an
// MFMA occupies it for 64 cycles and needs one 4-byte read per operand (counters of the large products: matrix pipes busy
// 75 % of the cycles, LDS 17 - 38 %; 51 - 66 % and 26 - 34 % in those too short to fill the chip throughout).  128 x 128 tiles for the reuse in L2, smaller
// ones where those share out badly (see plan_tiles).  Steps of 32 and values fetched two steps ahead were no faster.
// kVec: 16-byte loads (sizes and strides multiples of four floats, aligned pointers); otherwise single floats.
//
// Measured (gate and up projection with the activation, 8192 x 2816 x 1024 each, 94 GFLOP): 0.87 - 0.92 ms = 105 TFLOP/s
// of a nominal 157, where the vector-ALU kernel of 64 x 64 tiles it replaces and its separate activation took 2.5 ms.
// Whole step at 10752 rows, 1024 -> 2816 -> 1024 -> 256 (24 % of the rows not kept): 11.0 -> 3.7 ms; at 5376 rows,
// 256 -> 1024 -> 256 -> 256: 1.17 -> 0.39 ms.  The MFMA adds its products one k after the other, as the vector kernel
// did, and no sum is longer than there: the outputs of both steps are the same to the last bit.
template <int kI, int kJ, int kLayA, int kLayB, int kSecond, bool kVec, class Epilogue>
__global__ __launch_bounds__(kDirectThreads) void gemm_direct(F32Problem p, Epilogue epi) {
    constexpr int TM = 64 * kI, TN = 64 * kJ;
    constexpr int SA = TM + 4, SB = TN + 4;                     // floats between k-rows
    __shared__ __attribute__((aligned(16))) float As[2][kDirectStep * SA], Bs[2][kDirectStep * SB];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int right = kSecond == kPair ? (int)blockIdx.x / p.tiles_n : 0;
    const int m0 = blockIdx.y * TM, n0 = ((int)blockIdx.x - right * p.tiles_n) * TN;
    const F32Coord<kI, kJ, kSecond> tc{m0, n0, wave >> 1, wave & 1, lane, (int)blockIdx.z, right};
    int K = p.K;
    if (p.live == kLiveM && m0 >= (live_rows_of(p) + kDirectRowTile - 1) / kDirectRowTile * kDirectRowTile) return;   // the same rows whatever the tile
    if (p.live == kLiveK) K = (int)min((int64_t)K, live_rows_of(p));
    const bool second_sum = kSecond == kSum && blockIdx.z == 1;
    const int k_first = kSecond == kSum ? 0 : (int)blockIdx.z * p.k_per_split, k_last = min(K, k_first + p.k_per_split);
    const int steps = k_last > k_first ? (k_last - k_first + kDirectStep - 1) / kDirectStep : 0;

    // A tile of kT rows x 16 k as 4-float pieces: [rows][K] four k of a row, [K][rows] four rows of a k.  Rows beyond the
    // matrix are read as its last ones (whatever they give is not stored); only a step that ends beyond the reduction
    // needs a check per piece.
    constexpr int kPiecesA = TM * kDirectStep / 4 / kDirectThreads, kPiecesB = TN * kDirectStep / 4 / kDirectThreads;
    f32x4 ra[kPiecesA], rb[kPiecesB];
    const float *pa[kPiecesA], *pb[kPiecesB];                    // this thread's pieces of the next step to fetch
    int ea[4], eb[4];                                            // element offsets within a piece (not kVec)
    auto row_in = [](int row, int rows) { return kVec ? min(row, (rows + 3) / 4 * 4 - 4) : min(row, rows - 1); };
    auto point_at = [&](const float* A, const float* B, const float* B_odd, int k0) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < kPiecesA; ++q) {
            const int piece = tid + q * kDirectThreads;
            const int row = kLayA == kRowsByK ? min(m0 + piece / 4, p.M - 1) : row_in(m0 + piece % (TM / 4) * 4, p.M);
            const int k = k0 + (kLayA == kRowsByK ? piece % 4 * 4 : piece / (TM / 4));
            pa[q] = A + (kLayA == kRowsByK ? (int64_t)row * p.lda + k : (int64_t)k * p.lda + row);
#pragma unroll
            for (int e = 0; e < 4; ++e) ea[e] = kLayA == kRowsByK ? e : min(row + e, p.M - 1) - row;
        }
#pragma unroll
        for (int q = 0; q < kPiecesB; ++q) {
            const int piece = tid + q * kDirectThreads;
            const int c = kLayB == kRowsByK ? piece / 4 : piece % (TN / 4) * 4;      // column within the tile
            const int k = k0 + (kLayB == kRowsByK ? piece % 4 * 4 : piece / (TN / 4));
            const int n = kSecond == kInterleaved ? n0 / 2 + c / 64 * 32 + c % 32 : n0 + c;
            const float* const from = kSecond == kInterleaved && (c & 32) ? B_odd : B;
            const int row = kLayB == kRowsByK ? min(n, p.N - 1) : row_in(n, p.N);
            pb[q] = from + (kLayB == kRowsByK ? (int64_t)row * p.ldb + k : (int64_t)k * p.ldb + row);
#pragma unroll
            for (int e = 0; e < 4; ++e) eb[e] = kLayB == kRowsByK ? e : min(row + e, p.N - 1) - row;
        }
    };
    const int64_t inc_a = kLayA == kRowsByK ? kDirectStep : kDirectStep * p.lda, inc_b = kLayB == kRowsByK ? kDirectStep : kDirectStep * p.ldb;
    auto load4 = [](const float* at, const int (&e)[4]) __attribute__((always_inline)) -> f32x4 {
        if (kVec) return *reinterpret_cast<const f32x4*>(at);
        return f32x4{at[e[0]], at[e[1]], at[e[2]], at[e[3]]};
    };
    auto load4_checked = [](const float* at, const int (&e)[4], bool k_is_within, int left) __attribute__((always_inline)) -> f32x4 {
        f32x4 v = {0.f, 0.f, 0.f, 0.f};                          // left: k from the piece's first one to the end
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if ((k_is_within ? t : 0) < left) v[t] = at[e[t]];
        return v;
    };
    auto fetch = [&](int s) __attribute__((always_inline)) {
        const int left = k_last - k_first - s * kDirectStep;
        if (left >= kDirectStep) {                                     // uniform
#pragma unroll
            for (int q = 0; q < kPiecesA; ++q) ra[q] = load4(pa[q], ea);
#pragma unroll
            for (int q = 0; q < kPiecesB; ++q) rb[q] = load4(pb[q], eb);
        } else {
#pragma unroll
            for (int q = 0; q < kPiecesA; ++q) {
                const int piece = tid + q * kDirectThreads;
                ra[q] = load4_checked(pa[q], ea, kLayA == kRowsByK, left - (kLayA == kRowsByK ? piece % 4 * 4 : piece / (TM / 4)));
            }
#pragma unroll
            for (int q = 0; q < kPiecesB; ++q) {
                const int piece = tid + q * kDirectThreads;
                rb[q] = load4_checked(pb[q], eb, kLayB == kRowsByK, left - (kLayB == kRowsByK ? piece % 4 * 4 : piece / (TN / 4)));
            }
        }
#pragma unroll
        for (int q = 0; q < kPiecesA; ++q) pa[q] += inc_a;
#pragma unroll
        for (int q = 0; q < kPiecesB; ++q) pb[q] += inc_b;
    };
    auto stash = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < kPiecesA; ++q) {
            const int piece = tid + q * kDirectThreads;
            if (kLayA == kRowsByK) {
#pragma unroll
                for (int e = 0; e < 4; ++e) As[buf][(piece % 4 * 4 + e) * SA + piece / 4] = ra[q][e];
            } else {
                *reinterpret_cast<f32x4*>(&As[buf][piece / (TM / 4) * SA + piece % (TM / 4) * 4]) = ra[q];
            }
        }
#pragma unroll
        for (int q = 0; q < kPiecesB; ++q) {
            const int piece = tid + q * kDirectThreads;
            if (kLayB == kRowsByK) {
#pragma unroll
                for (int e = 0; e < 4; ++e) Bs[buf][(piece % 4 * 4 + e) * SB + piece / 4] = rb[q][e];
            } else {
                *reinterpret_cast<f32x4*>(&Bs[buf][piece / (TN / 4) * SB + piece % (TN / 4) * 4]) = rb[q];
            }
        }
    };

    f32x16 acc[kI][kJ];
#pragma unroll
    for (int i = 0; i < kI; ++i)
#pragma unroll
        for (int j = 0; j < kJ; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    if (steps > 0) {                                             // uniform over the workgroup
        // Fragments are read one group of MFMAs (two k) ahead, the values fetched at the start of a step go to the other
        // LDS buffer behind the sixth group, and the barrier that hands it over stands before the last, behind which the
        // first fragments of the next step are read: the matrix pipe has work through each of these waits.
        point_at(second_sum ? p.A2 : p.A, right || second_sum ? p.B2 : p.B, p.B2, k_first);
        fetch(0);
        stash(0);
        __syncthreads();
        const int a_at = (lane >> 5) * SA + tc.wm * kI * 32 + (lane & 31), b_at = (lane >> 5) * SB + tc.wn * kJ * 32 + (lane & 31);
        float fa[2][kI], fb[2][kJ];
        auto read = [&](int set, int buf, int kk) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < kI; ++i) fa[set][i] = As[buf][kk * SA + a_at + i * 32];
#pragma unroll
            for (int j = 0; j < kJ; ++j) fb[set][j] = Bs[buf][kk * SB + b_at + j * 32];
        };
        read(0, 0, 0);
        constexpr int kGroups = kDirectStep / 2;
        for (int s = 0; s < steps; ++s) {
            const int buf = s & 1;
            const bool more = s + 1 < steps;
            if (more) fetch(s + 1);
#pragma unroll
            for (int g = 0; g < kGroups; ++g) {
                if (g + 1 < kGroups) read((g + 1) & 1, buf, 2 * (g + 1));
                else if (more) read(0, buf ^ 1, 0);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < kI; ++i)
#pragma unroll
                    for (int j = 0; j < kJ; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[g & 1][i], fb[g & 1][j], acc[i][j], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (g == kGroups - 3 && more) stash(buf ^ 1);    // read last in the step before this one
                if (g == kGroups - 2 && more) __syncthreads();
            }
        }
    }
    epi(tc, acc, p);
}

// C (row-major, ldc) = acc; slice z of a split reduction goes to C + z * split_stride, the second product of a pair to
// C2 (one product: C2 = C).  Skipped tiles are not written.
struct F32Store {
    float *C, *C2;
    int64_t ldc, split_stride;
    template <class Coord, int kI, int kJ>
    __device__ void operator()(const Coord& tc, const f32x16 (&acc)[kI][kJ], const F32Problem& p) const {
        float* const out = (tc.right ? C2 : C) + tc.split * split_stride;
#pragma unroll
        for (int i = 0; i < kI; ++i)
#pragma unroll
            for (int j = 0; j < kJ; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int m = tc.row(i, e), n = tc.col(j);
                    if (m < p.M && n < p.N) out[(int64_t)m * ldc + n] = acc[i][j][e];
                }
    }
};

// Gate and up projection interleaved: acc[i][even] = u, acc[i][odd] = v of the same columns; a = silu(u) v.
struct F32SwigluForward {
    float *u, *v, *a;
    template <class Coord, int kI, int kJ>
    __device__ void operator()(const Coord& tc, const f32x16 (&acc)[kI][kJ], const F32Problem& p) const {
#pragma unroll
        for (int i = 0; i < kI; ++i)
#pragma unroll
            for (int j = 0; j < kJ; j += 2)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int m = tc.row(i, e), n = tc.col(j);
                    if (m >= p.M || n >= p.N) continue;
                    const int64_t at = (int64_t)m * p.N + n;
                    const float x = acc[i][j][e], y = acc[i][j + 1][e];
                    u[at] = x;
                    v[at] = y;
                    a[at] = x / (1.f + expf(-x)) * y;
                }
    }
};

// acc = da.  In place: u <- du = da * v * silu'(u), v <- dv = da * silu(u).
struct F32SwigluBackward {
    float *u, *v;
    template <class Coord, int kI, int kJ>
    __device__ void operator()(const Coord& tc, const f32x16 (&acc)[kI][kJ], const F32Problem& p) const {
#pragma unroll
        for (int i = 0; i < kI; ++i)
#pragma unroll
            for (int j = 0; j < kJ; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int m = tc.row(i, e), n = tc.col(j);
                    if (m >= p.M || n >= p.N) continue;
                    const int64_t at = (int64_t)m * p.N + n;
                    const float x = u[at], vv = v[at], g = acc[i][j][e];
                    const float s = 1.f / (1.f + expf(-x));
                    u[at] = g * vv * (s * (1.f + x * (1.f - s)));
                    v[at] = g * (x * s);
                }
    }
};

}  // namespace pcm
