// fp32 path of the masked GRPO actor step (Eq. 11): fp32 operands, sums and results.
//
// Forward: products on the fp32 matrix instructions (gemm_floats.h), every sum one chain in the order of k, so that loss and
// log-probabilities have the bits of the definition's order of additions whatever the tile.
//
// Backward: products on the bf16 matrix cores.  Every operand is held as three bf16 matrices whose sum it is exactly (thirds.h),
// and a product of two is six products of such parts (gemm_thirds.h; the three left out are below 2^-23 of the whole).  The
// matrix cores add up 32 products at a time in fp32, so a sum has a thirty-second of the roundings that one by fp32
// multiply-adds has, and they do 16 times the multiply-adds of the fp32 ones: six products take 3/8 of the time at the same share
// of their rates.
// Measured against fp32 matrix instructions throughout, steps: 10,752 rows of 1024 -> 2816 -> 1024 -> 256, a quarter of them not kept,
// 3.74 -> 2.54 ms; 5376 of 256 -> 1024 -> 256 -> 256 362 -> 273 us; 360 of 473 -> 333 -> 473 -> 512 185 -> 124, 1440 of 619 -> 1302 -> 619 ->
// 256 413 -> 201, 8960 of 103 -> 149 -> 103 -> 256, composed, where most of the padded tiles is padding, 171 -> 149; faster at 16 of 16
// sizes, 1.15 to 2.06 times.  Loss, log-probabilities and statistics have the same bits; errors of the gradients against 64 bits,
// root mean square over six inputs each: dX 4.85e-6 -> 4.74e-6 and 2.78e-6 -> 2.71e-6 at the first two, no larger at any of ten sizes.
// (The forward products as thirds too: 2.08 ms and 232 us, and a third of the error; but the loss may be a sum of terms of both
// signs that nearly cancel, and any other rounding of the logits moves it by more than a part in 10^4 then.)
//
// Who reads a matrix only as an operand gets its operand form alone: X, a and y as floats in blocks and as thirds, dz, dy, du and
// dv as thirds.  Wg and Wu are one matrix with columns in blocks of 32 of each in turn, so that a wavefront holds a gate column
// and its up column, and so are u and v, and du and dv.  Operands are padded with zeros to whole blocks in the workspace, so any
// size runs; results are written as far as they reach.
//
// Backward products of one dependency level share a launch and long reductions are split into parts that a later launch adds up
// in order (no atomics), as in the bf16 path.  Row tiles beyond the kept count are skipped.
#include <algorithm>

#include "gemm_floats.h"
#include "gemm_thirds.h"

namespace pcm {
namespace {

constexpr int kThreads = 256;
constexpr int kW = kSmallTile;
using ThirdsCoord = TileCoord<kW>;
using ThirdsSums = Accumulators<kW>;

__device__ __forceinline__ void split4(f32x4 v, bf16x4 (&out)[3]) {
    const float x[4] = {v[0], v[1], v[2], v[3]};
    uint32_t part[3][2];
    split_in_three(x, part);
#pragma unroll
    for (int t = 0; t < 3; ++t) out[t] = __builtin_bit_cast(bf16x4, (uint64_t)part[t][0] | (uint64_t)part[t][1] << 32);
}
// Four consecutive columns n .. n + 3 of a row with N of them, as far as they are there.
__device__ __forceinline__ void store4(float* row, int n, int N, f32x4 v) {
    if (n + 3 < N) {
        *reinterpret_cast<f32x4_any*>(row + n) = v;
    } else {
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if (n + t < N) row[n + t] = v[t];
    }
}

// The parts of kRows rows of kRowBytes each from a staging area, rows `stride` bytes apart and the parts of a row kRowBytes, to C
// from (row, column) on, multiples of kRows and 32; rows at and beyond n_rows are not written.
template <int kRows, int kRowBytes>
__device__ __forceinline__ void copy_thirds_out(const char* st, int stride, const Thirds& C, int64_t row, int64_t column, int n_rows, int lane) {
    constexpr int kLanesPerRow = kRowBytes / 16, kRowsPerPass = 64 / kLanesPerRow;
    static_assert(kRowsPerPass % 2 == 0 && kThirdsUnit % kRows == 0, "both rows of a line in a pass, all rows in a block");
    const int r = lane / kLanesPerRow, c = lane % kLanesPerRow;
    bf16* const out = C.p + Thirds::at(row + r, column + c * 8, C.ld);
    const char* const src = st + r * stride + c * 16;
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int pass = 0; pass < kRows / kRowsPerPass; ++pass)
            if (pass * kRowsPerPass < n_rows)            // wave-uniform: n_rows is a multiple of a pass's rows
                *reinterpret_cast<u32x4*>(out + t * kThirdsPart + pass * kRowsPerPass * 32) =
                    *reinterpret_cast<const u32x4*>(src + t * kRowBytes + pass * kRowsPerPass * stride);
}

// ---- epilogues: results go through the wavefront's staging area, as those of the bf16 path do -------------------------

// C = acc as thirds.  Columns up to C.ld (a multiple of a wavefront's), rows below `rows`.
struct EpiThirds {
    Thirds C;
    int rows;
    __device__ __forceinline__ void operator()(const ThirdsCoord& tc, const ThirdsSums& acc, char* lds) const {
        constexpr int RW = kWaveRows<kW>, kRow = RW * 2, kStride = 3 * kRow + 16;
        const int col_base = tc.col0();
        if (col_base >= C.ld) return;
        char* const st = wave_stage(tc, lds);
#pragma unroll
        for (int i = 0; i < RW / 32; ++i) {                // 32 rows per pass
#pragma unroll
            for (int ii = 0; ii < 2; ++ii)
#pragma unroll
                for (int j = 0; j < kW; ++j) {
                    bf16x4 part[3];
                    split4(acc[2 * i + ii][j], part);
                    char* const at = st + (ii * 16 + (tc.lane & 15)) * kStride + (j * 16 + 4 * (tc.lane >> 4)) * 2;
#pragma unroll
                    for (int t = 0; t < 3; ++t) *reinterpret_cast<bf16x4*>(at + t * kRow) = part[t];
                    __builtin_amdgcn_sched_barrier(0);
                }
            __builtin_amdgcn_wave_barrier();
            const int row_base = tc.row0() + i * 32;
            copy_thirds_out<32, kRow>(st, kStride, C, row_base, col_base, rows - row_base, tc.lane);
            __builtin_amdgcn_wave_barrier();
        }
    }
};

// C = acc in fp32, M x N with rows ldc apart, of any alignment; part s of a split reduction goes to C + s * split_stride.
struct EpiFloats {
    float* C;
    int64_t ldc, split_stride;
    int M, N;
    __device__ __forceinline__ void operator()(const ThirdsCoord& tc, const ThirdsSums& acc, char* lds) const {
        constexpr int RW = kWaveRows<kW>, kStride = RW * 4 + 16, kLanesPerRow = RW / 4, kRowsPerPass = 64 / kLanesPerRow;
        char* const st = wave_stage(tc, lds);
        float* const out = C + tc.split * split_stride;
        const int n = tc.col0() + tc.lane % kLanesPerRow * 4;
#pragma unroll
        for (int i = 0; i < RW / 32; ++i) {                // 32 rows per pass
#pragma unroll
            for (int ii = 0; ii < 2; ++ii)
#pragma unroll
                for (int j = 0; j < kW; ++j)
                    *reinterpret_cast<f32x4*>(st + (ii * 16 + (tc.lane & 15)) * kStride + (j * 16 + 4 * (tc.lane >> 4)) * 4) = acc[2 * i + ii][j];
            __builtin_amdgcn_wave_barrier();
            const int row0 = tc.row0() + i * 32 + tc.lane / kLanesPerRow;
#pragma unroll 8
            for (int q = 0; q < 32 / kRowsPerPass; ++q) {
                const int row = row0 + q * kRowsPerPass;
                const f32x4 v = *reinterpret_cast<const f32x4*>(st + (q * kRowsPerPass + tc.lane / kLanesPerRow) * kStride + tc.lane % kLanesPerRow * 16);
                if (row < M) store4(out + (int64_t)row * ldc, n, N, v);
            }
            __builtin_amdgcn_wave_barrier();
        }
    }
};

// The same where the product's columns are 32 of one matrix and the same 32 of another in turn (each M x N, rows N apart).
struct EpiFloatsPair {
    float* C[2];
    int64_t split_stride;
    int M, N;
    __device__ __forceinline__ void operator()(const ThirdsCoord& tc, const ThirdsSums& acc, char* lds) const {
        constexpr int RW = kWaveRows<kW>, kStride = RW * 4 + 16, kLanesPerRow = RW / 4, kRowsPerPass = 64 / kLanesPerRow;
        char* const st = wave_stage(tc, lds);
        const int packed = tc.col0() + tc.lane % kLanesPerRow * 4, n = packed / 64 * 32 + packed % 32;
        float* const out = (packed & 32 ? C[1] : C[0]) + tc.split * split_stride;
#pragma unroll
        for (int i = 0; i < RW / 32; ++i) {                // 32 rows per pass
#pragma unroll
            for (int ii = 0; ii < 2; ++ii)
#pragma unroll
                for (int j = 0; j < kW; ++j)
                    *reinterpret_cast<f32x4*>(st + (ii * 16 + (tc.lane & 15)) * kStride + (j * 16 + 4 * (tc.lane >> 4)) * 4) = acc[2 * i + ii][j];
            __builtin_amdgcn_wave_barrier();
            const int row0 = tc.row0() + i * 32 + tc.lane / kLanesPerRow;
#pragma unroll 8
            for (int q = 0; q < 32 / kRowsPerPass; ++q) {
                const int row = row0 + q * kRowsPerPass;
                const f32x4 v = *reinterpret_cast<const f32x4*>(st + (q * kRowsPerPass + tc.lane / kLanesPerRow) * kStride + tc.lane % kLanesPerRow * 16);
                if (row < M) store4(out + (int64_t)row * N, n, N, v);
            }
            __builtin_amdgcn_wave_barrier();
        }
    }
};

// acc = da.  du = da v silu'(u) and dv = da silu(u) as thirds, in blocks of 32 columns of each in turn, as u and v are.
struct EpiGateUpBackward {
    const float* uv;         // [rows, duv.ld]
    Thirds duv;
    __device__ __forceinline__ void operator()(const ThirdsCoord& tc, const ThirdsSums& acc, char* lds) const {
        constexpr int RW = kWaveRows<kW>, kRow = 2 * RW * 2, kStride = 3 * kRow + 16;
        const int col_base = 2 * tc.col0();                // packed column of this wavefront's block of 2 RW
        if (col_base >= duv.ld) return;
        char* const st = wave_stage(tc, lds);
        constexpr int kTogether = 4;                       // tiles whose u and v are on their way together
#pragma unroll
        for (int i = 0; i < kW; ++i) {                     // 16 rows per pass
            const int64_t row_base = tc.row0() + i * 16;
            const float* const from = uv + (row_base + (tc.lane & 15)) * duv.ld + col_base + 4 * (tc.lane >> 4);
            char* const to = st + (tc.lane & 15) * kStride + 4 * (tc.lane >> 4) * 2;
#pragma unroll
            for (int j0 = 0; j0 < kW; j0 += kTogether) {
                f32x4 u[kTogether], v[kTogether];
#pragma unroll
                for (int q = 0; q < kTogether; ++q) {
                    const int at = (j0 + q) / 2 * 64 + (j0 + q) % 2 * 16;
                    u[q] = *reinterpret_cast<const f32x4*>(from + at);
                    v[q] = *reinterpret_cast<const f32x4*>(from + at + 32);
                }
#pragma unroll
                for (int q = 0; q < kTogether; ++q) {
                    const int at = (j0 + q) / 2 * 64 + (j0 + q) % 2 * 16;
                    f32x4 du, dv;
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const float x = u[q][t], g = acc[i][j0 + q][t], s = 1.f / (1.f + expf(-x));
                        du[t] = g * v[q][t] * (s * (1.f + x * (1.f - s)));
                        dv[t] = g * (x * s);
                    }
                    bf16x4 pu[3], pv[3];
                    split4(du, pu);
                    split4(dv, pv);
#pragma unroll
                    for (int t = 0; t < 3; ++t) {
                        *reinterpret_cast<bf16x4*>(to + t * kRow + at * 2) = pu[t];
                        *reinterpret_cast<bf16x4*>(to + t * kRow + (at + 32) * 2) = pv[t];
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            __builtin_amdgcn_wave_barrier();
            copy_thirds_out<16, kRow>(st, kStride, duv, row_base, col_base, 16, tc.lane);
            __builtin_amdgcn_wave_barrier();
        }
    }
};

// ---- forward ------------------------------------------------------------------------------------

// 32 rows x 32 columns of a wavefront of gemm_floats, v[g] columns 8 g + 4 (lane >> 5) .. + 3 of row (lane & 31), to C and, if it is
// there, to C3, from (row, column) on.
__device__ __forceinline__ void put_square(char* st, int lane, const f32x4 (&v)[4], const FloatBlocks& C, const Thirds& C3, int64_t row,
                                           int64_t column) {
    constexpr int kStride = 128 + 16, kStride3 = 3 * 64 + 16;
    const int r = lane & 31, half = lane >> 5;
#pragma unroll
    for (int g = 0; g < 4; ++g) {                          // the even columns of eight, then the odd ones
        *reinterpret_cast<float2*>(st + r * kStride + g * 32 + half * 8) = make_float2(v[g][0], v[g][2]);
        *reinterpret_cast<float2*>(st + r * kStride + g * 32 + 16 + half * 8) = make_float2(v[g][1], v[g][3]);
    }
    __builtin_amdgcn_wave_barrier();
    copy_rows_out<32, 128>(st, kStride, reinterpret_cast<char*>(C.p + FloatBlocks::at(row, column, C.ld)), 128, 32, lane);
    __builtin_amdgcn_wave_barrier();
    if (C3.p == nullptr) return;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        bf16x4 part[3];
        split4(v[g], part);
#pragma unroll
        for (int t = 0; t < 3; ++t) *reinterpret_cast<bf16x4*>(st + r * kStride3 + t * 64 + (8 * g + 4 * half) * 2) = part[t];
    }
    __builtin_amdgcn_wave_barrier();
    copy_thirds_out<32, 64>(st, kStride3, C3, row, column, 32, lane);
    __builtin_amdgcn_wave_barrier();
}
template <int kJ>
__device__ __forceinline__ void put_rows(char* st, int lane, const f32x16 (&acc)[kJ], float* C, int64_t ldc) {   // 32 rows, row-major
    constexpr int kStride = 32 * kJ * 4 + 16;
#pragma unroll
    for (int j = 0; j < kJ; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            *reinterpret_cast<f32x4*>(st + (lane & 31) * kStride + (j * 32 + 8 * g + 4 * (lane >> 5)) * 4) =
                f32x4{acc[j][4 * g], acc[j][4 * g + 1], acc[j][4 * g + 2], acc[j][4 * g + 3]};
    __builtin_amdgcn_wave_barrier();
    copy_rows_out<32, 32 * kJ * 4>(st, kStride, reinterpret_cast<char*>(C), ldc * 4, 32, lane);
    __builtin_amdgcn_wave_barrier();
}

// Gate and up projection, columns in blocks of 32 of each in turn: a = silu(u) v, and for a backward pass u and v as they are in
// the product.
struct EpiGateUp {
    float* uv;               // [rows, 2 a.ld] or null
    FloatBlocks a;
    Thirds a3;
    template <int kI, int kJ>
    __device__ __forceinline__ void operator()(const FloatsCoord<kI, kJ>& tc, const f32x16 (&acc)[kI][kJ], char* st) const {
        static_assert(kJ == 2, "a gate block and its up block");
#pragma unroll
        for (int i = 0; i < kI; ++i) {
            const int64_t row = tc.row0 + 32 * i;
            if (uv != nullptr) put_rows(st, tc.lane, acc[i], uv + row * 2 * a.ld + tc.col0, 2 * a.ld);
            f32x4 r[4];
#pragma unroll
            for (int g = 0; g < 4; ++g)
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const float x = acc[i][0][4 * g + t], y = acc[i][1][4 * g + t];
                    r[g][t] = x / (1.f + expf(-x)) * y;
                }
            put_square(st, tc.lane, r, a, a3, row, tc.col0 / 2);
        }
    }
};
// A product that is an operand of others.
struct EpiOperand {
    FloatBlocks C;
    Thirds C3;
    template <int kI, int kJ>
    __device__ __forceinline__ void operator()(const FloatsCoord<kI, kJ>& tc, const f32x16 (&acc)[kI][kJ], char* st) const {
#pragma unroll
        for (int i = 0; i < kI; ++i)
#pragma unroll
            for (int j = 0; j < kJ; ++j) {
                f32x4 v[4];
#pragma unroll
                for (int e = 0; e < 16; ++e) v[e / 4][e % 4] = acc[i][j][e];
                put_square(st, tc.lane, v, C, C3, tc.row0 + 32 * i, tc.col0 + 32 * j);
            }
    }
};
// C row-major.
struct EpiRows {
    float* C;
    int64_t ldc;
    template <int kI, int kJ>
    __device__ __forceinline__ void operator()(const FloatsCoord<kI, kJ>& tc, const f32x16 (&acc)[kI][kJ], char* st) const {
#pragma unroll
        for (int i = 0; i < kI; ++i) put_rows(st, tc.lane, acc[i], C + (int64_t)(tc.row0 + 32 * i) * ldc + tc.col0, ldc);
    }
};

// The tile whose workgroups, shared out over the 256 CUs, have the least to do: the matrix pipes are shared by the workgroups of
// a CU, so a CU's time is the number of its tiles times their size; the smaller tile counts 1.08 times its size.  By themselves
// 128 x 128, 64 x 128 and 64 x 64 take at 8192 x 5632 x 1024 802 / 731 / 717 us, at 8192 x 1024 x 2816 332 / 336 / 341, at 8192 x 1024 x
// 11264 1299 / 1325 / 1426; within a step, where the backward products have brought the clock down, the larger ones are ahead:
// gate and up of 10,752 rows at 1024 -> 2816 871 / 916, steps of 5376 at 890 -> 849 478 / 503.  kPairs: a wavefront takes 64 columns.
template <bool kPairs, class Epilogue>
void launch_floats(const FloatsProblem& p, const Epilogue& epi, hipStream_t s) {
    const int64_t large = (int64_t)(p.M / 128) * (p.N / 128);
    constexpr int kSmallJ = kPairs ? 2 : 1, kPerLarge = 4 / kSmallJ;
    const double cost_large = 4.0 * (double)ceil_div64(large, 256), cost_small = 1.08 * kSmallJ * (double)ceil_div64(kPerLarge * large, 256);
    if (cost_large <= cost_small) gemm_floats<2, 2><<<(unsigned)large, 256, 0, s>>>(p, epi);
    else gemm_floats<1, kSmallJ><<<(unsigned)(kPerLarge * large), 256, 0, s>>>(p, epi);
}

// ---- backward products -----------------------------------------------------------------------------------

// A product of thirds among others of its launch.
template <int kLayA, int kLayB, class Epilogue>
struct ThirdsProduct {
    GemmProblem p;
    Epilogue epi;
    int first;                   // its first workgroup, a multiple of eight (see tile_of_workgroup)
    int workgroups(int tile) {   // operands are padded, so a tile may reach beyond the matrix
        p.M = ceil_div(p.M, tile) * tile;
        p.N = ceil_div(p.N, tile) * tile;
        return p.M / tile * (p.N / tile) * p.splits;
    }
    __device__ __forceinline__ void run(int block, ThirdsRing& smem) const { thirds_tile<kLayA, kLayB>(p, epi, block - first, smem); }
};
template <int kLayA, int kLayB, class Epilogue>
ThirdsProduct<kLayA, kLayB, Epilogue> job(const GemmProblem& p, const Epilogue& epi) { return {p, epi, 0}; }

template <class... Jobs>
__global__ __launch_bounds__(kGemmThreads, 1) void gemm_f32(Jobs... jobs) {
    __shared__ ThirdsRing smem;
    run_job((int)blockIdx.x, smem, jobs...);
}
template <class... Jobs>
void launch_products(hipStream_t s, Jobs... jobs) {
    int grid = 0;
    ((grid = place_job(jobs, kThirdsUnit, grid)), ...);
    gemm_f32<<<(unsigned)grid, kGemmThreads, 0, s>>>(jobs...);
}

// C = the sum over the parts of a split reduction, as thirds; parts are n floats (rows of C.ld) apart.
__global__ __launch_bounds__(kThreads) void sum_parts_thirds(const float* parts, int n_parts, size_t n, Thirds C) {
    constexpr int kTogether = 4;      // loads under way together
    const size_t stride = (size_t)gridDim.x * kThreads * 4;
    for (size_t i = ((size_t)blockIdx.x * kThreads + threadIdx.x) * 4; i < n; i += stride) {
        f32x4 acc = *reinterpret_cast<const f32x4*>(parts + i);
        for (int s0 = 1; s0 < n_parts; s0 += kTogether) {
            f32x4 v[kTogether];
#pragma unroll
            for (int u = 0; u < kTogether; ++u) v[u] = *reinterpret_cast<const f32x4*>(parts + (size_t)min(s0 + u, n_parts - 1) * n + i);
#pragma unroll
            for (int u = 0; u < kTogether; ++u)
                if (s0 + u < n_parts) acc += v[u];
        }
        bf16x4 part[3];
        split4(acc, part);
#pragma unroll
        for (int t = 0; t < 3; ++t) *reinterpret_cast<bf16x4*>(C.p + Thirds::at(i / C.ld, i % C.ld, C.ld) + t * kThirdsPart) = part[t];
    }
}

// ---- loss ---------------------------------------------------------------------------------------

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

// One wavefront per row, a column per lane and 64: log-softmax at the target bin, entropy, ratio, clipped surrogate, and dz =
// coef * (onehot - softmax) + entropy part as thirds.  With a per-chunk ratio the factor is not known yet: z <- onehot - softmax
// and the entropy part goes to `extra`; scale_rows makes dz of them once the chunk ratios are known.
constexpr int kMaxV = 1024;
struct LossArgs {
    float* z;                // [rows, ld]
    int V, ld;
    float* extra;            // [rows, V]
    Thirds dz;               // p null: no backward pass
    RowMeta meta;
    const int32_t* n_kept;
    int max_chunks, A;
    LossOptions opt;
    float* logp_out;
    RowOut out;
};
__global__ __launch_bounds__(kThreads) void loss_rows(LossArgs p) {
    constexpr int kQ = kMaxV / kWave;
    const int lane = threadIdx.x % kWave;
    const int64_t r = (int64_t)blockIdx.x * (kThreads / kWave) + threadIdx.x / kWave;
    const int64_t rows = live_rows(p.n_kept, p.max_chunks, p.A);
    if (r >= (rows + kTileM - 1) / kTileM * kTileM) return;     // later rows: skipped tiles, read by nothing
    const bool live = r < rows;
    const float scale = objective_scale(p.opt, rows);
    float* const zr = p.z + r * p.ld;
    const int b = p.meta.token[r];
    const float zb = zr[b];
    float z[kQ];
    float mx = -INFINITY;
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
        const int j = q * kWave + lane;
        z[q] = j < p.V ? zr[j] : -INFINITY;
        mx = fmaxf(mx, z[q]);
    }
    mx = wave_max(mx);
    float se = 0.f, sz = 0.f;
#pragma unroll
    for (int q = 0; q < kQ; ++q)
        if (q * kWave + lane < p.V) {
            const float e = expf(z[q] - mx);
            se += e;
            sz += e * z[q];
        }
    se = wave_sum(se);
    sz = wave_sum(sz);
    const float lse = mx + logf(se);
    const float lp = zb - lse;
    const float H = lse - sz / se;                      // -sum p log p
    const float w = (p.opt.chunk_weight && live) ? p.opt.chunk_weight[r / p.A] : 1.f;
    const LossRow lr = loss_row(lp, p.meta.logp_old[r], p.meta.adv[r], w, p.opt, scale);
    if (lane == 0) {
        p.out.dlogp[r] = lr.dlogp;
        p.out.entropy[r] = live ? H : 0.f;
        if (!p.opt.chunk_ratio) {
            p.out.term[r] = live ? lr.term : 0.f;
            p.out.ratio[r] = lr.ratio;
            p.out.clipped[r] = lr.clipped;
        }
        if (p.logp_out && live) p.logp_out[r] = lp;
    }
    if (p.dz.p == nullptr) return;
    const float coef = p.opt.chunk_ratio ? (live ? 1.f : 0.f) : (live ? lr.coef : 0.f);
    const float ec = live ? p.opt.entropy_coef * scale : 0.f;
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
        const int j = q * kWave + lane;
        if (j >= p.ld) continue;
        float pg = 0.f, ent = 0.f;
        if (j < p.V) {
            const float pr = expf(z[q] - lse);
            pg = coef * ((j == b ? 1.f : 0.f) - pr);
            ent = ec * pr * (z[q] - lse + H);
        }
        if (p.opt.chunk_ratio) {
            zr[j] = pg;
            if (live && j < p.V) p.extra[r * p.V + j] = ent;
        } else {
            const float x[2] = {pg + ent, 0.f};
            uint32_t part[3][1];
            split_in_three(x, part);
#pragma unroll
            for (int t = 0; t < 3; ++t) reinterpret_cast<uint16_t*>(p.dz.p)[Thirds::at(r, j, p.dz.ld) + t * kThirdsPart] = (uint16_t)part[t][0];
        }
    }
}

// Per-chunk ratio: dz[r, :] = coef[r] z[r, :] (+ extra[r, :] if given) for the live rows, zeros to the end of their last tile.
__global__ __launch_bounds__(kThreads) void scale_rows(const float* z, const float* extra, int V, const float* coef, const int32_t* n_kept,
                                                       int max_chunks, int A, Thirds dz) {
    const int64_t rows = live_rows(n_kept, max_chunks, A), n = (rows + kTileM - 1) / kTileM * kTileM * dz.ld;
    const int64_t stride = (int64_t)gridDim.x * kThreads * 4;
    for (int64_t i = ((int64_t)blockIdx.x * kThreads + threadIdx.x) * 4; i < n; i += stride) {
        f32x4 x = {};
        const int64_t r = i / dz.ld;
        if (r < rows) {
            x = *reinterpret_cast<const f32x4*>(z + i);
            const float c = coef[r];
#pragma unroll
            for (int t = 0; t < 4; ++t) x[t] = c * x[t];
            if (extra) {
                const int n = (int)(i - r * dz.ld);
#pragma unroll
                for (int t = 0; t < 4; ++t) x[t] += n + t < V ? extra[r * V + n + t] : 0.f;
            }
        }
        bf16x4 part[3];
        split4(x, part);
#pragma unroll
        for (int t = 0; t < 3; ++t) *reinterpret_cast<bf16x4*>(dz.p + Thirds::at(r, i - r * dz.ld, dz.ld) + t * kThirdsPart) = part[t];
    }
}

// ---- the step -------------------------------------------------------------------------------------

int64_t padded(int64_t n) { return ceil_div64(n, kThirdsUnit) * kThirdsUnit; }
int steps64(int64_t n) { return (int)ceil_div64(n, kTileK) * kTileK; }
int64_t tiles256(int64_t n) { return ceil_div64(n, kTileM) * kTileM; }

// Reduction splits of products that share a launch: those with the least estimated time (as plan_group of the bf16 path).  A
// workgroup takes about 6 us to start and to write its tile and 1 us per step of 32 k; the launch takes what its longest
// workgroup does, or the work shared out over 256 CUs and about half a workgroup more at the end; parts are written, read back
// and added up at about 4 TB/s.  Each number of parts forced on its product at ten sizes: within 2 % of the best at seven of them,
// 3 to 7 % at three.
struct ProductShape {
    int64_t M, N;
    int steps;
    int most_parts;        // 1: not to be split
};
template <int kN>
void plan_products(const ProductShape (&jobs)[kN], float us_sum, int (&splits)[kN]) {
    constexpr float kUsPerStep = 1.f, kUsFixed = 6.f;
    float best_us = 0.f;
    for (int most : {8, 12, 16, 24, 32, 48, 64, 96, 128, 192, 256, 1 << 20}) {    // longest reduction of a workgroup
        int parts[kN], longest = 0;
        int64_t workgroups = 0;
        float work = 0.f, sum = 0.f;
        for (int q = 0; q < kN; ++q) {
            const ProductShape& j = jobs[q];
            const int s = parts[q] = std::max(1, std::min(j.most_parts, ceil_div(j.steps, most))), len = ceil_div(j.steps, s);
            const int64_t n = ceil_div64(j.M, kThirdsUnit) * ceil_div64(j.N, kThirdsUnit) * s;
            longest = std::max(longest, len);
            workgroups += n;
            work += (float)n * (kUsFixed + kUsPerStep * (float)len);
            if (s > 1) sum += (float)(2 * s + 1) * (float)j.M * (float)j.N * (4 / 4e6f);
        }
        float us = kUsFixed + kUsPerStep * (float)longest;
        if (workgroups > 256) us = std::max(us, work / 256 + 0.5f * us);
        if (sum > 0.f) us += us_sum + sum;
        if (best_us == 0.f || us < best_us) {
            best_us = us;
            for (int q = 0; q < kN; ++q) splits[q] = parts[q];
        }
    }
}
struct F32Plan {
    int G, dWo, dWd, dWgu, dX;      // parts of each
};
constexpr int kMaxParts = 64;
F32Plan plan_step(const ActorShape& sh, int64_t Mp, bool composed) {
    const int64_t d = sh.d, ff = sh.ff, V = sh.V, gu = 2 * padded(ff);
    const auto shape = [](int64_t M, int64_t N, int64_t K, int most) { return ProductShape{M, N, steps64(K) / kThirdsK, most}; };
    F32Plan p{1, 1, 1, 1, 1};
    const auto two = [&](const ProductShape& a, const ProductShape& b, int& of_a, int& of_b) {
        int s[2];
        plan_products<2>({a, b}, 2.f, s);
        of_a = s[0];
        of_b = s[1];
    };
    int unsplit;
    if (composed) {
        int G[1];
        plan_products<1>({shape(ff, V, Mp, kMaxParts)}, 5.f, G);
        p.G = G[0];
        two(shape(ff, d, V, 1), shape(d, V, ff, kMaxParts), unsplit, p.dWo);
    } else {
        two(shape(Mp, d, V, 1), shape(d, V, Mp, kMaxParts), unsplit, p.dWo);
        two(shape(Mp, ff, d, 1), shape(ff, d, Mp, kMaxParts), unsplit, p.dWd);
    }
    // dX in two parts at most: one goes to dX itself, which the other is added to
    two(shape(Mp, d, gu, 2), shape(d, gu, Mp, kMaxParts), p.dX, p.dWgu);
    if (d <= 64 && ff <= 64) p.dWgu = ceil_div((int)sh.rows_max(), 64);       // a small weight gradient in slices of 64 rows
    return p;
}

struct F32Workspace {
    FloatBlocks X, a, y, WguT, WdT, WoT;          // forward; weights with their columns as rows (composed: Wd as it is for WdT)
    FloatBlocks WdoT;                             // composed evaluation: (Wd Wo)^T [V, ff]
    Thirds Wgu, Wd, Wo, X3, a3, y3, dz, dy, duv;  // backward
    Thirds WdoT3, G;                              // composed: the same, and a^T dz [ff, V]
    float *uv, *z, *z_extra;
    float* dX_part;          // the second of two parts of dX
    float* parts_G;          // composed
    float *parts_o, *parts_d, *parts_g, *parts_u;   // of the weight gradients, where they are computed in parts
    F32Plan plan;
    RowMeta meta;
    RowOut out;
    int64_t Mp;
    size_t bytes;
};

// One layout for calls with and without gradients: those without hold the buffers of the backward products too, and those with
// have three more at the end.
F32Workspace carve(void* ws, const ActorShape& sh, bool bwd, bool composed) {
    Carver c(ws);
    F32Workspace w{};
    const int64_t Mp = w.Mp = tiles256(sh.rows_max());
    const auto thirds = [&](int64_t rows, int64_t columns) { return Thirds{c.take<bf16>((size_t)(3 * padded(rows) * padded(columns))), padded(columns)}; };
    const auto floats = [&](int64_t rows, int64_t columns) { return FloatBlocks{c.take<float>((size_t)(padded(rows) * padded(columns))), padded(columns)}; };
    w.plan = plan_step(sh, Mp, composed);
    const F32Plan& plan = w.plan;
    const int64_t ffp = padded(sh.ff), Vp = padded(sh.V);
    w.X = floats(Mp, sh.d);
    w.a = floats(Mp, sh.ff);
    w.WguT = floats(2 * ffp, sh.d);
    w.WdT = composed ? floats(sh.ff, sh.d) : floats(sh.d, sh.ff);
    w.WoT = floats(sh.V, sh.d);
    if (composed) w.WdoT = floats(sh.V, sh.ff);
    else w.y = floats(Mp, sh.d);
    w.z = c.take<float>((size_t)Mp * Vp);
    w.meta.token = c.take<uint8_t>(Mp);
    w.meta.logp_old = c.take<float>(Mp);
    w.meta.adv = c.take<float>(Mp);
    w.out.term = c.take<float>(Mp);
    w.out.ratio = c.take<float>(Mp);
    w.out.dlogp = c.take<float>(Mp);
    w.out.clipped = c.take<uint8_t>(Mp);
    w.out.entropy = c.take<float>(Mp);
    w.out.coef = c.take<float>(Mp);
    const size_t M = (size_t)sh.rows_max(), d = sh.d, ff = sh.ff, V = sh.V;
    F32Workspace b{};                     // of the backward pass
    b.uv = c.take<float>((size_t)Mp * 2 * ffp);
    b.Wgu = thirds(d, 2 * ffp);
    b.Wd = thirds(ff, d);
    b.Wo = thirds(d, V);
    b.X3 = thirds(Mp, d);
    b.a3 = thirds(Mp, ff);
    b.dz = thirds(Mp, V);
    b.duv = thirds(Mp, 2 * ffp);
    if (composed) {
        b.WdoT3 = thirds(V, ff);
        b.G = thirds(ff, V);
        b.parts_G = c.take<float>((size_t)plan.G * ffp * Vp);
    } else {
        b.y3 = thirds(Mp, d);
        b.dy = thirds(Mp, d);
    }
    const int o = plan.dWo, dd = plan.dWd, gu = plan.dWgu;
    if (o > 1) b.parts_o = c.take<float>(o * d * V);
    if (dd > 1) b.parts_d = c.take<float>(dd * ff * d);
    if (bwd) {
        w.uv = b.uv; w.Wgu = b.Wgu; w.Wd = b.Wd; w.Wo = b.Wo; w.X3 = b.X3; w.a3 = b.a3; w.y3 = b.y3; w.dz = b.dz; w.dy = b.dy; w.duv = b.duv;
        w.WdoT3 = b.WdoT3; w.G = b.G; w.parts_G = b.parts_G; w.parts_o = b.parts_o; w.parts_d = b.parts_d;
        w.z_extra = c.take<float>(M * V);
        w.dX_part = c.take<float>(M * d);
        if (gu > 1) w.parts_g = c.take<float>(2 * gu * d * ff);
        w.parts_u = w.parts_g + gu * d * ff;
    }
    w.bytes = c.used();
    return w;
}

}  // namespace

size_t actor_f32_workspace_bytes(const ActorShape& sh, bool bwd, bool composed) {
    return carve(nullptr, sh, bwd, composed).bytes;
}

int actor_f32_run(const ActorShape& sh, const ActorIO& io, void* ws, hipStream_t s) {
    const bool grads = io.want_grads(), bwd = grads || io.dX != nullptr;
    const F32Workspace w = carve(ws, sh, bwd, io.composed);
    const F32Plan& plan = w.plan;
    const int Mp = (int)w.Mp, M = (int)sh.rows_max(), d = sh.d, ff = sh.ff, V = sh.V;
    const int ffp = (int)padded(ff), Vp = (int)padded(V), dp = (int)padded(d);

    // C[M, N] = sum_k A(m, k) B(n, k) with the batch's rows as M or K (role) or not at all
    const auto product = [&](const Thirds& A, const Thirds& B, int m, int n, int k, int role, int splits = 1) {
        GemmProblem p{};
        p.A = p.A2 = A.p; p.lda = A.ld;
        p.B = p.B2 = B.p; p.ldb = B.ld;
        p.M = m; p.N = n; p.K1 = steps64(k); p.splits = splits;
        if (role != kRowsUnused) { p.kept = io.n_kept; p.kept_max = sh.max_chunks; p.rows_per_kept = sh.A; }
        p.rows_role = role;
        return p;
    };
    PartsSums sums{};
    // C [m, n] in fp32, or its parts for the launch behind the last product
    const auto floats = [&](int splits, float* parts, float* C, int m, int n) {
        const int64_t size = (int64_t)m * n;
        if (splits == 1) return EpiFloats{C, n, 0, m, n};
        sums.add(parts, splits, (size_t)size, (size_t)size, C);
        return EpiFloats{parts, n, size, m, n};
    };

    const Thirds none3{};
    const FloatBlocks none{};
    const float *const Wg = static_cast<const float*>(io.Wg), *const Wu = static_cast<const float*>(io.Wu);
    const float *const Wd = static_cast<const float*>(io.Wd), *const Wo = static_cast<const float*>(io.Wo);
    WeightJobs weights{};
    weights.add(WeightJob{Wg, w.WguT, none3, d, ff, true, kPackGate});
    weights.add(WeightJob{Wu, w.WguT, none3, d, ff, true, kPackUp});
    weights.add(WeightJob{Wd, w.WdT, none3, ff, d, !io.composed, kPackNone});
    weights.add(WeightJob{Wo, w.WoT, none3, d, V, true, kPackNone});
    if (io.dX) weights.add(WeightJob{Wg, none, w.Wgu, d, ff, false, kPackGate});
    if (io.dX) weights.add(WeightJob{Wu, none, w.Wgu, d, ff, false, kPackUp});
    if (bwd && (grads || !io.composed)) weights.add(WeightJob{Wd, none, w.Wd, ff, d, false, kPackNone});
    if (bwd && (grads || !io.composed)) weights.add(WeightJob{Wo, none, w.Wo, d, V, false, kPackNone});
    int rc = launch_prepare_f32(sh, io, w.X, grads ? w.X3 : none3, Mp, w.meta, weights, static_cast<float*>(io.dX), s);
    if (rc != PCM_OK) return rc;
    {
        StageTimer t(ST_F32_FORWARD, s);
        // C[m, n] = sum_k A(m, k) B(n, k)
        const auto forward = [&](const FloatBlocks& A, const FloatBlocks& B, int m, int n, int k, bool batch) {
            return FloatsProblem{A.p, B.p, A.ld, B.ld, m, n, (int)ceil_div64(k, 32) * 32, batch ? io.n_kept : nullptr, sh.max_chunks, sh.A};
        };
        launch_floats<true>(forward(w.X, w.WguT, Mp, 2 * ffp, d, true), EpiGateUp{w.uv, w.a, grads ? w.a3 : none3}, s);
        if (io.composed) {                                                                             // (Wd Wo)^T, then z = a Wd Wo
            launch_floats<false>(forward(w.WoT, w.WdT, Vp, ffp, d, false), EpiOperand{w.WdoT, w.WdoT3}, s);
            launch_floats<false>(forward(w.a, w.WdoT, Mp, Vp, ff, true), EpiRows{w.z, Vp}, s);
        } else {                                                                                       // y = a Wd, z = y Wo
            launch_floats<false>(forward(w.a, w.WdT, Mp, dp, ff, true), EpiOperand{w.y, grads ? w.y3 : none3}, s);
            launch_floats<false>(forward(w.y, w.WoT, Mp, Vp, d, true), EpiRows{w.z, Vp}, s);
        }
    }
    {
        StageTimer t(ST_F32_LOSS, s);
        loss_rows<<<(unsigned)(Mp / (kThreads / kWave)), kThreads, 0, s>>>(
            LossArgs{w.z, V, Vp, w.z_extra, w.dz, w.meta, io.n_kept, sh.max_chunks, sh.A, io.opt, io.logp_out, w.out});
    }
    if (io.opt.chunk_ratio) {
        rc = launch_chunk_ratio(sh, io, w.meta, w.out, 0, M, s);
        if (rc != PCM_OK) return rc;
        if (bwd) {
            StageTimer t(ST_REDUCE, s);
            const int64_t blocks = ceil_div64((int64_t)Mp * Vp / 4, kThreads);
            scale_rows<<<(unsigned)std::min<int64_t>(blocks, 4096), kThreads, 0, s>>>(
                w.z, io.opt.entropy_coef != 0.f ? w.z_extra : nullptr, V, w.out.coef, io.n_kept, sh.max_chunks, sh.A, w.dz);
        }
    }
    if (!bwd) return launch_finish(sh, io, w.out, PartsSums{}, FinalPanel{}, true, SumsqLists{}, s);
    {
        StageTimer t(ST_F32_BACKWARD, s);
        const EpiGateUpBackward swiglu{w.uv, w.duv};
        if (io.composed) {
            launch_products(s, job<kRowsByK, kKByRows>(product(w.dz, w.WdoT3, Mp, ffp, V, kRowsAreM), swiglu));   // da = dz (Wd Wo)^T
            if (grads) {
                const size_t n = (size_t)ffp * Vp;                                                     // G = a^T dz
                launch_products(s, job<kKByRows, kKByRows>(product(w.a3, w.dz, ffp, Vp, Mp, kRowsAreK, plan.G), EpiFloats{w.parts_G, Vp, (int64_t)n, ffp, Vp}));
                sum_parts_thirds<<<(unsigned)std::min<size_t>((n / 4 + kThreads - 1) / kThreads, 2048), kThreads, 0, s>>>(w.parts_G, plan.G, n, w.G);
                const auto dWd = job<kRowsByK, kRowsByK>(product(w.G, w.Wo, ff, d, V, kRowsUnused), EpiFloats{io.dWd, d, 0, ff, d});   // G Wo^T
                const int o = plan.dWo;
                const auto dWo = job<kKByRows, kKByRows>(product(w.Wd, w.G, d, V, ff, kRowsUnused, o), floats(o, w.parts_o, io.dWo, d, V));   // Wd^T G
                launch_products(s, dWo, dWd);
            }
        } else {
            const auto dy = job<kRowsByK, kRowsByK>(product(w.dz, w.Wo, Mp, dp, V, kRowsAreM), EpiThirds{w.dy, Mp});     // dy = dz Wo^T
            const auto da = job<kRowsByK, kRowsByK>(product(w.dy, w.Wd, Mp, ffp, d, kRowsAreM), swiglu);                 // da = dy Wd^T
            if (grads) {
                const int o = plan.dWo, dd = plan.dWd;
                launch_products(s, job<kKByRows, kKByRows>(product(w.y3, w.dz, d, V, Mp, kRowsAreK, o), floats(o, w.parts_o, io.dWo, d, V)), dy);
                launch_products(s, da, job<kKByRows, kKByRows>(product(w.a3, w.dy, ff, d, Mp, kRowsAreK, dd), floats(dd, w.parts_d, io.dWd, ff, d)));
            } else {
                launch_products(s, dy);
                launch_products(s, da);
            }
        }
        float* const out_X = static_cast<float*>(io.dX);
        const int x = plan.dX;                                                         // dX = du Wg^T + dv Wu^T
        const auto dX = job<kRowsByK, kRowsByK>(product(w.duv, w.Wgu, Mp, d, 2 * ffp, kRowsAreM, x), EpiFloats{out_X, d, w.dX_part - out_X, M, d});
        if (out_X && x > 1) sums.add(w.dX_part, 1, (size_t)M * d, (size_t)M * d, out_X, true, nullptr, d);
        if (grads) {
            const int gu = plan.dWgu;                                                    // dWg = X^T du, dWu = X^T dv
            EpiFloatsPair epi{{io.dWg, io.dWu}, 0, d, ff};
            if (gu > 1) {
                const size_t n = (size_t)d * ff;
                sums.add(w.parts_g, gu, n, n, io.dWg);
                sums.add(w.parts_u, gu, n, n, io.dWu);
                epi = EpiFloatsPair{{w.parts_g, w.parts_u}, (int64_t)n, d, ff};
            }
            const auto dWgu = job<kKByRows, kKByRows>(product(w.X3, w.duv, d, 2 * ffp, Mp, kRowsAreK, gu), epi);
            if (io.dX) launch_products(s, dX, dWgu);
            else launch_products(s, dWgu);
        } else {
            launch_products(s, dX);
        }
    }
    return launch_finish(sh, io, w.out, sums, FinalPanel{}, true, SumsqLists{}, s);
}

}  // namespace pcm
