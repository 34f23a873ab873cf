// What the products of the fp32 path do with their sums (internal header).
#pragma once

#include "gemm_floats.h"
#include "gemm_thirds.h"

namespace pcm {

using ThirdsCoord = TileCoord<kSmallTile>;
using ThirdsSums = Accumulators<kSmallTile>;

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
    static constexpr int kChainSteps = 0;
    Thirds C;
    int rows;
    __device__ __forceinline__ void operator()(const ThirdsCoord& tc, const ThirdsSums& acc, char* lds) const {
        constexpr int RW = kWaveRows<kSmallTile>, kRow = RW * 2, kStride = 3 * kRow + 16;
        const int col_base = tc.col0();
        if (col_base >= C.ld) return;
        char* const st = wave_stage(tc, lds);
#pragma unroll
        for (int i = 0; i < RW / 32; ++i) {                // 32 rows per pass
#pragma unroll
            for (int ii = 0; ii < 2; ++ii)
#pragma unroll
                for (int j = 0; j < kSmallTile; ++j) {
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
    static constexpr int kChainSteps = 0;
    float* C;
    int64_t ldc, split_stride;
    int M, N;
    __device__ __forceinline__ void operator()(const ThirdsCoord& tc, const ThirdsSums& acc, char* lds) const {
        constexpr int RW = kWaveRows<kSmallTile>, kStride = RW * 4 + 16, kLanesPerRow = RW / 4, kRowsPerPass = 64 / kLanesPerRow;
        char* const st = wave_stage(tc, lds);
        float* const out = C + tc.split * split_stride;
        const int n = tc.col0() + tc.lane % kLanesPerRow * 4;
#pragma unroll
        for (int i = 0; i < RW / 32; ++i) {                // 32 rows per pass
#pragma unroll
            for (int ii = 0; ii < 2; ++ii)
#pragma unroll
                for (int j = 0; j < kSmallTile; ++j)
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

// The same with short chains of additions, for a product over the rows that further sums are taken of (composed head).  Sums of one sign, dWo of
// 5376 rows of 473 -> 333 -> 512, error against 64 bits: 1.88e-7 with one chain, 1.72e-7 with these (1.74e-7 on the direct route).
struct EpiFloatsInChains : EpiFloats {
    static constexpr int kChainSteps = 8;
};

// C = acc where the product's columns are 32 of one matrix and the same 32 of another in turn (each M x N, rows N apart).
struct EpiFloatsPair {
    // Sums of one sign, error of dWg against 64 bits, direct route / one chain per part / these: 5376 rows of 256 -> 1024 1.24e-7 / 1.56e-7 /
    // 1.02e-7, 2688 of 300 -> 700 1.19 / 1.35 / 1.08.  No slower (step of the first 263 us with and without).
    static constexpr int kChainSteps = 16;
    float* C[2];
    int64_t split_stride;
    int M, N;
    __device__ __forceinline__ void operator()(const ThirdsCoord& tc, const ThirdsSums& acc, char* lds) const {
        constexpr int RW = kWaveRows<kSmallTile>, kStride = RW * 4 + 16, kLanesPerRow = RW / 4, kRowsPerPass = 64 / kLanesPerRow;
        char* const st = wave_stage(tc, lds);
        const int packed = tc.col0() + tc.lane % kLanesPerRow * 4, n = packed / 64 * 32 + packed % 32;
        float* const out = (packed & 32 ? C[1] : C[0]) + tc.split * split_stride;
#pragma unroll
        for (int i = 0; i < RW / 32; ++i) {                // 32 rows per pass
#pragma unroll
            for (int ii = 0; ii < 2; ++ii)
#pragma unroll
                for (int j = 0; j < kSmallTile; ++j)
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
    static constexpr int kChainSteps = 0;
    const float* uv;         // [rows, duv.ld]
    Thirds duv;
    __device__ __forceinline__ void operator()(const ThirdsCoord& tc, const ThirdsSums& acc, char* lds) const {
        constexpr int RW = kWaveRows<kSmallTile>, kRow = 2 * RW * 2, kStride = 3 * kRow + 16;
        const int col_base = 2 * tc.col0();                // packed column of this wavefront's block of 2 RW
        if (col_base >= duv.ld) return;
        char* const st = wave_stage(tc, lds);
        constexpr int kTogether = 4;                       // tiles whose u and v are on their way together
#pragma unroll
        for (int i = 0; i < kSmallTile; ++i) {                     // 16 rows per pass
            const int64_t row_base = tc.row0() + i * 16;
            const float* const from = uv + (row_base + (tc.lane & 15)) * duv.ld + col_base + 4 * (tc.lane >> 4);
            char* const to = st + (tc.lane & 15) * kStride + 4 * (tc.lane >> 4) * 2;
#pragma unroll
            for (int j0 = 0; j0 < kSmallTile; j0 += kTogether) {
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

}  // namespace pcm
