// fp32 path of the masked GRPO actor step (Eq. 11): fp32 matrix-core products (v_mfma_f32_32x32x2_f32: fp32 operands,
// products and sums) with the activation fused into their epilogues.
//
// This path exists for small heads and for checking the method at fp32 accuracy.  One GEMM kernel template serves all
// products of the forward and backward pass; reductions over the row dimension (the weight gradients) are split across
// workgroups into partial products that a second kernel adds in slice order, so the results are the same from run to
// run (no atomics).  Row tiles beyond the kept count are skipped.
#include <algorithm>

#include "actor.h"

namespace pcm {
namespace {

typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int kThreads = 256;
constexpr int kStep = 16;           // reduction steps are 16 wide
constexpr int kRowTile = 128;       // live rows are rounded up to this: the tallest row tile

// How an operand of C[m, n] = sum_k A(m, k) B(n, k) is stored (ld = distance between rows of the storage).
enum Layout : int { kRowsByK = 0, kKByRows = 1 };

struct F32Problem {
    const float *A, *B;
    const float *A2, *B2;   // operands of a second product of the same sizes and layouts (see Second)
    int64_t lda, ldb;
    int M, N, K;
    int k_per_split;        // slice blockIdx.z covers [z, z + 1) * k_per_split of the reduction
    int tiles_n;            // column tiles of one right operand
    // rows of the batch: kLiveM: row tiles beyond the live rows (rounded up to kRowTile) are skipped; kLiveK: the
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
__global__ __launch_bounds__(kThreads) void gemm_f32(F32Problem p, Epilogue epi) {
    constexpr int TM = 64 * kI, TN = 64 * kJ;
    constexpr int SA = TM + 4, SB = TN + 4;                     // floats between k-rows
    __shared__ __attribute__((aligned(16))) float As[2][kStep * SA], Bs[2][kStep * SB];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int right = kSecond == kPair ? (int)blockIdx.x / p.tiles_n : 0;
    const int m0 = blockIdx.y * TM, n0 = ((int)blockIdx.x - right * p.tiles_n) * TN;
    const F32Coord<kI, kJ, kSecond> tc{m0, n0, wave >> 1, wave & 1, lane, (int)blockIdx.z, right};
    int K = p.K;
    if (p.live == kLiveM && m0 >= (live_rows_of(p) + kRowTile - 1) / kRowTile * kRowTile) return;   // the same rows whatever the tile
    if (p.live == kLiveK) K = (int)min((int64_t)K, live_rows_of(p));
    const bool second_sum = kSecond == kSum && blockIdx.z == 1;
    const int k_first = kSecond == kSum ? 0 : (int)blockIdx.z * p.k_per_split, k_last = min(K, k_first + p.k_per_split);
    const int steps = k_last > k_first ? (k_last - k_first + kStep - 1) / kStep : 0;

    // A tile of kT rows x 16 k as 4-float pieces: [rows][K] four k of a row, [K][rows] four rows of a k.  Rows beyond the
    // matrix are read as its last ones (whatever they give is not stored); only a step that ends beyond the reduction
    // needs a check per piece.
    constexpr int kPiecesA = TM * kStep / 4 / kThreads, kPiecesB = TN * kStep / 4 / kThreads;
    f32x4 ra[kPiecesA], rb[kPiecesB];
    const float *pa[kPiecesA], *pb[kPiecesB];                    // this thread's pieces of the next step to fetch
    int ea[4], eb[4];                                            // element offsets within a piece (not kVec)
    auto row_in = [](int row, int rows) { return kVec ? min(row, (rows + 3) / 4 * 4 - 4) : min(row, rows - 1); };
    auto point_at = [&](const float* A, const float* B, const float* B_odd, int k0) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < kPiecesA; ++q) {
            const int piece = tid + q * kThreads;
            const int row = kLayA == kRowsByK ? min(m0 + piece / 4, p.M - 1) : row_in(m0 + piece % (TM / 4) * 4, p.M);
            const int k = k0 + (kLayA == kRowsByK ? piece % 4 * 4 : piece / (TM / 4));
            pa[q] = A + (kLayA == kRowsByK ? (int64_t)row * p.lda + k : (int64_t)k * p.lda + row);
#pragma unroll
            for (int e = 0; e < 4; ++e) ea[e] = kLayA == kRowsByK ? e : min(row + e, p.M - 1) - row;
        }
#pragma unroll
        for (int q = 0; q < kPiecesB; ++q) {
            const int piece = tid + q * kThreads;
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
    const int64_t inc_a = kLayA == kRowsByK ? kStep : kStep * p.lda, inc_b = kLayB == kRowsByK ? kStep : kStep * p.ldb;
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
        const int left = k_last - k_first - s * kStep;
        if (left >= kStep) {                                     // uniform
#pragma unroll
            for (int q = 0; q < kPiecesA; ++q) ra[q] = load4(pa[q], ea);
#pragma unroll
            for (int q = 0; q < kPiecesB; ++q) rb[q] = load4(pb[q], eb);
        } else {
#pragma unroll
            for (int q = 0; q < kPiecesA; ++q) {
                const int piece = tid + q * kThreads;
                ra[q] = load4_checked(pa[q], ea, kLayA == kRowsByK, left - (kLayA == kRowsByK ? piece % 4 * 4 : piece / (TM / 4)));
            }
#pragma unroll
            for (int q = 0; q < kPiecesB; ++q) {
                const int piece = tid + q * kThreads;
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
            const int piece = tid + q * kThreads;
            if (kLayA == kRowsByK) {
#pragma unroll
                for (int e = 0; e < 4; ++e) As[buf][(piece % 4 * 4 + e) * SA + piece / 4] = ra[q][e];
            } else {
                *reinterpret_cast<f32x4*>(&As[buf][piece / (TM / 4) * SA + piece % (TM / 4) * 4]) = ra[q];
            }
        }
#pragma unroll
        for (int q = 0; q < kPiecesB; ++q) {
            const int piece = tid + q * kThreads;
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
        constexpr int kGroups = kStep / 2;
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

__device__ inline float wave_max(float x) {
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) x = fmaxf(x, __shfl_xor(x, d, kWave));
    return x;
}
__device__ inline float wave_sum(float x) {
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) x += __shfl_xor(x, d, kWave);
    return x;
}

// One wavefront per row: log-softmax at the target bin, entropy, ratio, clipped surrogate, and (in
// place) z <- dz = coef * (onehot - softmax) + entropy part.  With a per-chunk ratio the factor is
// not known yet: z <- onehot - softmax and the entropy part goes to `extra`; the rows are scaled
// once the chunk ratios are known.
__global__ __launch_bounds__(kThreads) void loss_rows(float* __restrict__ z, float* __restrict__ extra, int V,
                                                      const uint8_t* __restrict__ token,
                                                      const float* __restrict__ logp_old,
                                                      const float* __restrict__ adv_row,
                                                      const int32_t* __restrict__ n_kept, int max_chunks, int A,
                                                      int64_t rows_total, LossOptions opt, int write_dz,
                                                      float* logp_out, RowOut out) {
    const int lane = threadIdx.x % kWave;
    const int64_t r = (int64_t)blockIdx.x * (kThreads / kWave) + threadIdx.x / kWave;
    const int64_t rows = live_rows(n_kept, max_chunks, A);
    if (r >= rows_total || r >= (rows + kRowTile - 1) / kRowTile * kRowTile) return;   // later rows: skipped tiles, read by nothing
    const bool live = r < rows;
    const float scale = objective_scale(opt, rows);
    float* zr = z + r * V;
    float mx = -INFINITY;
    for (int j = lane; j < V; j += kWave) mx = fmaxf(mx, zr[j]);
    mx = wave_max(mx);
    float se = 0.f, sz = 0.f;
    for (int j = lane; j < V; j += kWave) {
        const float e = expf(zr[j] - mx);
        se += e;
        sz += e * zr[j];
    }
    se = wave_sum(se);
    sz = wave_sum(sz);
    const int b = token[r];
    const float lse = mx + logf(se);
    const float lp = zr[b] - lse;
    const float H = lse - sz / se;                      // -sum p log p
    const float w = (opt.chunk_weight && live) ? opt.chunk_weight[r / A] : 1.f;
    const LossRow lr = loss_row(lp, logp_old[r], adv_row[r], w, opt, scale);
    if (lane == 0) {
        out.dlogp[r] = lr.dlogp;
        out.entropy[r] = live ? H : 0.f;
        if (!opt.chunk_ratio) {
            out.term[r] = live ? lr.term : 0.f;
            out.ratio[r] = lr.ratio;
            out.clipped[r] = lr.clipped;
        }
        if (logp_out && live) logp_out[r] = lp;
    }
    if (write_dz) {
        const float coef = opt.chunk_ratio ? (live ? 1.f : 0.f) : (live ? lr.coef : 0.f);
        const float ec = live ? opt.entropy_coef * scale : 0.f;
        for (int j = lane; j < V; j += kWave) {
            const float zj = zr[j];
            const float p = expf(zj - lse);
            const float pg = coef * ((j == b ? 1.f : 0.f) - p);
            const float ent = ec * p * (zj - lse + H);
            if (opt.chunk_ratio) {
                zr[j] = pg;
                extra[r * V + j] = ent;
            } else {
                zr[j] = pg + ent;
            }
        }
    }
}

// Tile and reduction split of an M x N product (n_right of them in one launch) over K: the tile whose workgroups,
// shared out over the 256 CUs, have the least to do.  The matrix pipes are shared by the workgroups of a CU, so a CU's
// time is the number of its tiles times their size, plus about half a tile that the dispatcher, which puts several
// workgroups on one CU while others have none left, costs; the smaller tile counts 1.08 times its size because each of
// its values is loaded for half as many products.  Measured on both sides of the line, 128-wide against 64-wide tiles:
// 8192 x 1024 x 2816 (512 tiles of 128) 559 / 503 us, twice that 1112 / 981 us; 8192 x 5632 x 1024 (2816 tiles) 871 / 917 us;
// a pair of 1024 x 2816 over 8192 rows 902 / 957 us.  Splits (if allowed) aim at two workgroups per CU, and at least at
// 1024 tiles of 64 x 64 (shorter sums are also more accurate), but not at slices of fewer than about four steps: as many
// slices as that allows, rounded up, so that a sum over few rows is in slices of at most 64.
struct TilePlan {
    int kI, kJ, splits, k_per_split;
};
TilePlan plan_tiles(int M, int N, int K, int n_right, bool may_split, bool interleaved) {
    TilePlan best{};
    double best_cost = 0.0;
    for (int big = 1; big >= 0; --big) {
        const int kI = big ? 2 : 1, kJ = big || interleaved ? 2 : 1;
        const int64_t tiles = (int64_t)ceil_div(M, 64 * kI) * ceil_div(interleaved ? 2 * N : N, 64 * kJ) * n_right;
        int64_t splits = 1;
        if (may_split) {
            splits = std::max(ceil_div64(512, tiles), ceil_div64(1024, (int64_t)ceil_div(M, 64) * ceil_div(N, 64)));
            splits = std::max<int64_t>(1, std::min<int64_t>(splits, ceil_div(K, 4 * kStep)));
        }
        const int k_per = ceil_div(ceil_div(K, (int)splits), kStep) * kStep;
        splits = ceil_div(K, k_per);
        const double cost = ((double)ceil_div64(tiles * splits, 256) + 0.5) * kI * kJ * k_per * (big ? 1.0 : 1.08);
        if (big || cost < best_cost) {
            best = TilePlan{kI, kJ, (int)splits, k_per};
            best_cost = cost;
        }
    }
    return best;
}
size_t split_floats(int M, int N, int K, int n_right) {
    const TilePlan t = plan_tiles(M, N, K, n_right, true, false);
    return t.splits > 1 ? (size_t)t.splits * M * N * n_right : 0;
}

struct F32Workspace {
    float *X, *u, *v, *a, *y, *z, *z_extra, *dy;
    float *Wdo, *G;   // composed evaluation: Wd Wo and a^T dz, both [ff, V]
    float *parts, *parts_d;   // partial products of the split reductions; those of dWd
    RowMeta meta;
    RowOut out;
    size_t bytes;
};

F32Workspace carve(void* ws, const ActorShape& sh, bool grads) {
    Carver c(ws);
    F32Workspace w{};
    const size_t M = (size_t)sh.rows_max();
    w.X = c.take<float>(M * sh.d);
    w.u = c.take<float>(M * sh.ff);
    w.v = c.take<float>(M * sh.ff);
    w.a = c.take<float>(M * sh.ff);
    w.y = c.take<float>(M * sh.d);
    w.z = c.take<float>(M * sh.V);
    w.meta.token = c.take<uint8_t>(M);
    w.meta.logp_old = c.take<float>(M);
    w.meta.adv = c.take<float>(M);
    w.out.term = c.take<float>(M);
    w.out.ratio = c.take<float>(M);
    w.out.dlogp = c.take<float>(M);
    w.out.clipped = c.take<uint8_t>(M);
    w.out.entropy = c.take<float>(M);
    w.out.coef = c.take<float>(M);
    w.Wdo = c.take<float>((size_t)sh.ff * sh.V);
    w.G = c.take<float>((size_t)sh.ff * sh.V);
    if (grads) {
        w.z_extra = c.take<float>(M * sh.V);
        w.dy = c.take<float>(M * sh.d);
        const int rows = (int)M;
        // partial products: of dWo = y^T dz and dWd = a^T dy side by side (composed: of G = a^T dz, then of dWo = Wd^T G); once
        // those are added up, of dWg and dWu
        const size_t o = align_up(split_floats(sh.d, sh.V, rows, 1), 64), o_composed = split_floats(sh.d, sh.V, sh.ff, 1);
        const size_t d = split_floats(sh.ff, sh.d, rows, 1);
        w.parts = c.take<float>(std::max({o + d, o_composed, split_floats(sh.ff, sh.V, rows, 1), split_floats(sh.d, sh.ff, rows, 2)}));
        w.parts_d = w.parts + o;
    }
    w.bytes = c.used();
    return w;
}

bool vec_ok(std::initializer_list<const void*> pointers, std::initializer_list<int64_t> sizes) {
    for (const void* q : pointers)
        if (reinterpret_cast<uintptr_t>(q) & 15u) return false;
    for (int64_t n : sizes)
        if (n % 4 != 0) return false;
    return true;
}

template <int kLayA, int kLayB, int kSecond, class Epilogue>
void launch(F32Problem p, const TilePlan& t, const Epilogue& epi, hipStream_t s) {
    const bool vec = vec_ok({p.A, p.B, p.A2, p.B2}, {p.lda, p.ldb, p.M, p.N, p.K});
    const int columns = kSecond == kInterleaved ? 2 * p.N : p.N;
    p.k_per_split = t.k_per_split;
    p.tiles_n = ceil_div(columns, 64 * t.kJ);
    const dim3 grid((unsigned)p.tiles_n * (kSecond == kPair ? 2u : 1u), (unsigned)ceil_div(p.M, 64 * t.kI),
                    kSecond == kSum ? 2u : (unsigned)t.splits);
    constexpr int kSmallJ = kSecond == kInterleaved ? 2 : 1;
    if (t.kI == 2 && vec) gemm_f32<2, 2, kLayA, kLayB, kSecond, true><<<grid, kThreads, 0, s>>>(p, epi);
    else if (t.kI == 2) gemm_f32<2, 2, kLayA, kLayB, kSecond, false><<<grid, kThreads, 0, s>>>(p, epi);
    else if (vec) gemm_f32<1, kSmallJ, kLayA, kLayB, kSecond, true><<<grid, kThreads, 0, s>>>(p, epi);
    else gemm_f32<1, kSmallJ, kLayA, kLayB, kSecond, false><<<grid, kThreads, 0, s>>>(p, epi);
}

// The rows a launch runs over: those of the batch (their live count in device memory), or none.
struct BatchRows {
    const int32_t* n_kept;
    int max_chunks, rows_per_chunk;
};
F32Problem problem(const float* A, int64_t lda, const float* B, int64_t ldb, int M, int N, int K, const BatchRows& rows, int live) {
    return F32Problem{A, B, A, B, lda, ldb, M, N, K, 0, 0, rows.n_kept, rows.max_chunks, rows.rows_per_chunk,
                      rows.n_kept ? live : (int)kLiveUnused};
}

// C[M, N] = A B with A [M, K], and B [K, N] (or [N, K] if b_t), all row-major.
void gemm(hipStream_t s, const float* A, const float* B, bool b_t, float* C, int M, int N, int K, const BatchRows& rows) {
    const F32Problem p = problem(A, K, B, b_t ? K : N, M, N, K, rows, kLiveM);
    const TilePlan t = plan_tiles(M, N, K, 1, false, false);
    const F32Store epi{C, C, N, 0};
    if (b_t) launch<kRowsByK, kRowsByK, kNone>(p, t, epi, s);
    else launch<kRowsByK, kKByRows, kNone>(p, t, epi, s);
}

// C[M, N] = A^T B with A [K, M], B [K, N] row-major: the weight-gradient shape (reduction over rows).  With B2 also
// C2 = A^T B2 in the same launch.  A reduction in slices leaves them in `parts`, and their sum in `sums` for a later launch.
void gemm_reduce_rows(hipStream_t s, const float* A, const float* B, float* C, const float* B2, float* C2, int M, int N, int K,
                      float* parts, PartsSums& sums, const BatchRows& rows) {
    const int n_right = B2 ? 2 : 1;
    F32Problem p = problem(A, M, B, N, M, N, K, rows, kLiveK);
    if (B2) p.B2 = B2;
    const TilePlan t = plan_tiles(M, N, K, n_right, true, false);
    const size_t n = (size_t)M * N;
    float* const parts2 = parts + (size_t)t.splits * n;
    const F32Store epi = t.splits > 1 ? F32Store{parts, parts2, N, (int64_t)n} : F32Store{C, C2, N, 0};
    if (B2) launch<kKByRows, kKByRows, kPair>(p, t, epi, s);
    else launch<kKByRows, kKByRows, kNone>(p, t, epi, s);
    if (t.splits > 1) {
        sums.add(parts, t.splits, n, n, C);
        if (B2) sums.add(parts2, t.splits, n, n, C2);
    }
}

}  // namespace

size_t actor_f32_workspace_bytes(const ActorShape& sh, bool want_grads) {
    return carve(nullptr, sh, want_grads).bytes;
}

int actor_f32_run(const ActorShape& sh, const ActorIO& io, void* ws, hipStream_t s) {
    const bool bwd = io.want_grads() || io.dX != nullptr;
    F32Workspace w = carve(ws, sh, bwd);
    const int M = (int)sh.rows_max();
    const int d = sh.d, ff = sh.ff, V = sh.V;
    const float* Wg = static_cast<const float*>(io.Wg);
    const float* Wu = static_cast<const float*>(io.Wu);
    const float* Wd = static_cast<const float*>(io.Wd);
    const float* Wo = static_cast<const float*>(io.Wo);
    const BatchRows rows{io.n_kept, sh.max_chunks, sh.A}, none{nullptr, 0, 0};

    int rc = launch_gather(sh, io, 4, w.X, 0, M, w.meta, TransposeList{}, nullptr, 0, s);
    if (rc != PCM_OK) return rc;
    {
        StageTimer t(ST_F32_FORWARD, s);
        F32Problem p = problem(w.X, d, Wg, ff, M, ff, d, rows, kLiveM);                        // u, v, a
        p.B2 = Wu;
        launch<kRowsByK, kKByRows, kInterleaved>(p, plan_tiles(M, ff, d, 1, false, true), F32SwigluForward{w.u, w.v, w.a}, s);
        if (io.composed) {
            gemm(s, Wd, Wo, false, w.Wdo, ff, V, d, none);                                   // W_do = Wd Wo
            gemm(s, w.a, w.Wdo, false, w.z, M, V, ff, rows);                                 // z = a W_do
        } else {
            gemm(s, w.a, Wd, false, w.y, M, d, ff, rows);
            gemm(s, w.y, Wo, false, w.z, M, V, d, rows);
        }
    }
    {
        StageTimer t(ST_F32_LOSS, s);
        loss_rows<<<(unsigned)ceil_div64(M, kThreads / kWave), kThreads, 0, s>>>(
            w.z, w.z_extra, V, w.meta.token, w.meta.logp_old, w.meta.adv, io.n_kept, sh.max_chunks, sh.A, M, io.opt,
            bwd ? 1 : 0, io.logp_out, w.out);
    }
    if (io.opt.chunk_ratio) {
        rc = launch_chunk_ratio(sh, io, w.meta, w.out, 0, M, s);
        if (rc != PCM_OK) return rc;
        if (bwd) {
            rc = launch_scale_rows_f32(sh, io, w.z, io.opt.entropy_coef != 0.f ? w.z_extra : nullptr, w.out.coef, M, s);
            if (rc != PCM_OK) return rc;
        }
    }
    if (!bwd) return launch_finish(sh, io, w.out, PartsSums{}, FinalPanel{}, true, SumsqLists{}, s);
    PartsSums sums{};
    float* const dz = w.z;
    if (io.want_grads() && io.composed) {
        PartsSums g{};
        {
            StageTimer t(ST_F32_BACKWARD, s);
            gemm_reduce_rows(s, w.a, dz, w.G, nullptr, nullptr, ff, V, M, w.parts, g, rows);               // G = a^T dz
        }
        rc = launch_finish(sh, io, w.out, g, FinalPanel{}, false, SumsqLists{}, s);
        if (rc != PCM_OK) return rc;
    }
    {
        StageTimer t(ST_F32_BACKWARD, s);
        if (io.want_grads()) {
            if (io.composed) {
                gemm(s, w.G, Wo, true, io.dWd, ff, d, V, none);                                        // dWd = G Wo^T
                gemm_reduce_rows(s, Wd, w.G, io.dWo, nullptr, nullptr, d, V, ff, w.parts, sums, none);   // dWo = Wd^T G
            } else {
                gemm_reduce_rows(s, w.y, dz, io.dWo, nullptr, nullptr, d, V, M, w.parts, sums, rows);    // dWo = y^T dz
            }
        }
        if (!io.composed) {
            gemm(s, dz, Wo, true, w.dy, M, d, V, rows);                                                // dy = dz Wo^T
            if (io.want_grads()) gemm_reduce_rows(s, w.a, w.dy, io.dWd, nullptr, nullptr, ff, d, M, w.parts_d, sums, rows);   // dWd = a^T dy
        }
        // da = dy Wd^T (composed: dz W_do^T); u <- du, v <- dv
        const int k = io.composed ? V : d;
        const F32Problem p = io.composed ? problem(dz, V, w.Wdo, V, M, ff, k, rows, kLiveM) : problem(w.dy, d, Wd, d, M, ff, k, rows, kLiveM);
        launch<kRowsByK, kRowsByK, kNone>(p, plan_tiles(M, ff, k, 1, false, false), F32SwigluBackward{w.u, w.v}, s);
    }
    if (io.want_grads() && sums.n > 0 && split_floats(d, ff, M, 2) > 0) {                              // the parts' memory is needed again
        rc = launch_finish(sh, io, w.out, sums, FinalPanel{}, false, SumsqLists{}, s);
        if (rc != PCM_OK) return rc;
        sums = PartsSums{};
    }
    {
        StageTimer t(ST_F32_BACKWARD, s);
        if (io.want_grads())
            gemm_reduce_rows(s, w.X, w.u, io.dWg, w.v, io.dWu, d, ff, M, w.parts, sums, rows);         // dWg = X^T du, dWu = X^T dv
        if (io.dX) {                                                                                   // dX = du Wg^T + dv Wu^T
            // as two products, in place of y and dy (no longer needed), and their sum: twice the workgroups, sums half as long
            F32Problem p = problem(w.u, ff, Wg, ff, M, d, ff, rows, kLiveM);
            p.A2 = w.v; p.B2 = Wu;
            launch<kRowsByK, kRowsByK, kSum>(p, plan_tiles(M, d, ff, 2, false, false), F32Store{w.y, w.y, d, w.dy - w.y}, s);
            sums.add(w.y, 2, (size_t)M * d, (size_t)(w.dy - w.y), static_cast<float*>(io.dX), false, nullptr, d);
        }
    }
    return launch_finish(sh, io, w.out, sums, FinalPanel{}, true, SumsqLists{}, s);
}

}  // namespace pcm
