// fp32 path of the masked GRPO actor step (Eq. 11): fp32 operands, sums and results, on the bf16 matrix cores.
//
// Every operand of a product is held as three bf16 matrices whose sum it is exactly (thirds.h); a product of two is six
// products of such parts, as six segments of one reduction of the bf16 GEMM's main loop, the small ones first (the three left
// out are below 2^-23 of the whole).  The matrix cores add up 32 products at a time in fp32, so a sum has a thirty-second of
// the roundings that one by fp32 multiply-adds has.  Errors against 64 bits, root mean square over six inputs each, fp32 matrix
// instructions / thirds: at 1024 -> 2816 -> 1024 -> 256 log-probabilities 4.8e-7 / 1.7e-7, gradients 4.9e-6 / 1.8e-6; at 256 -> 1024
// 2.7e-7 / 1.0e-7 and 2.8e-6 / 1.1e-6; at eight further sizes of 169 .. 619 -> 133 .. 2026 every one 0.29 to 0.48 of what it was.
// (With the six products of every 32 k added up one behind the other the sums had a bias of 1e-7 to 4e-7: the matrix cores cut
// off what they add; in segments, small ones first, a sixth of the additions do so at full size.)
// The bf16 matrix cores do 16 times the multiply-adds of the fp32 ones, so six products take 3/8 of the time at the same
// share of their rates.  Steps: 10,752 rows of 1024 -> 2816 -> 1024 -> 256, a quarter of them not kept, 4.00 -> 2.45 ms; 5376 of
// 256 -> 1024 -> 256 -> 256 363 -> 316 us; 360 of 473 -> 333 -> 473 -> 512 185 -> 143, 1440 of 619 -> 1302 -> 619 -> 256 413 -> 243,
// 8960 of 103 -> 149 -> 103 -> 256, composed, where most of the padded tiles is padding, 171 -> 164; faster at 16 of 16 sizes.
//
// Who reads a matrix only as an operand gets the thirds alone: X, a, y, dz, dy, du and dv, and the weights, are never stored
// in fp32.  Wg and Wu are one matrix with columns in blocks of 32 of each in turn, so that a wavefront holds a gate column and
// its up column, and so are u and v, and du and dv.  Operands are padded with zeros to whole tiles in the workspace, so any
// size runs; results are written as far as they reach.
//
// Products of one dependency level share a launch and long reductions are split into parts that a later launch adds up in
// order (no atomics), as in the bf16 path.  Row tiles beyond the kept count are skipped.
#include <algorithm>

#include "gemm_bf16.h"
#include "thirds.h"

namespace pcm {
namespace {

constexpr int kThreads = 256;

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

// ---- epilogues: results go through the wavefront's staging area, as those of the bf16 path do -------------------------

// C = acc as thirds.  Columns up to C.ld (a multiple of a wavefront's), rows below `rows`.
struct EpiThirds {
    Thirds C;
    int rows;
    template <int kW>
    __device__ __forceinline__ void operator()(const TileCoord<kW>& tc, const Accumulators<kW>& acc, char* lds) const {
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
#pragma unroll
            for (int t = 0; t < 3; ++t)
                copy_rows_out<32, kRow>(st + t * kRow, kStride, reinterpret_cast<char*>(C.p + t * C.third + (int64_t)row_base * C.ld + col_base),
                                        C.ld * 2, rows - row_base, tc.lane);
            __builtin_amdgcn_wave_barrier();
        }
    }
};

// C = acc in fp32, M x N with rows ldc apart, of any alignment; part s of a split reduction goes to C + s * split_stride.
struct EpiFloats {
    float* C;
    int64_t ldc, split_stride;
    int M, N;
    template <int kW>
    __device__ __forceinline__ void operator()(const TileCoord<kW>& tc, const Accumulators<kW>& acc, char* lds) const {
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
    template <int kW>
    __device__ __forceinline__ void operator()(const TileCoord<kW>& tc, const Accumulators<kW>& acc, char* lds) const {
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

// Gate and up projection, columns in blocks of 32 of each in turn: a = silu(u) v as thirds, and for a backward pass u and v in
// fp32 as they are in the product.
struct EpiGateUp {
    float* uv;               // [rows, 2 a.ld] or null
    Thirds a;
    template <int kW>
    __device__ __forceinline__ void operator()(const TileCoord<kW>& tc, const Accumulators<kW>& acc, char* lds) const {
        constexpr int RW = kWaveRows<kW>, CW = RW / 2, kRow = CW * 2;
        constexpr int kStrideUv = RW * 4 + 16, kStride = 3 * kRow + 16;
        const int col_base = tc.col0();
        if (col_base >= 2 * a.ld) return;
        char* const st = wave_stage(tc, lds);
#pragma unroll
        for (int i = 0; i < RW / 32; ++i) {                // 32 rows per pass
            const int64_t row_base = tc.row0() + i * 32;
            if (uv != nullptr) {
#pragma unroll
                for (int ii = 0; ii < 2; ++ii)
#pragma unroll
                    for (int j = 0; j < kW; ++j)
                        *reinterpret_cast<f32x4*>(st + (ii * 16 + (tc.lane & 15)) * kStrideUv + (j * 16 + 4 * (tc.lane >> 4)) * 4) = acc[2 * i + ii][j];
                __builtin_amdgcn_wave_barrier();
                copy_rows_out<32, RW * 4>(st, kStrideUv, reinterpret_cast<char*>(uv + row_base * 2 * a.ld + col_base), a.ld * 8, 32, tc.lane);
                __builtin_amdgcn_wave_barrier();
            }
#pragma unroll
            for (int ii = 0; ii < 2; ++ii)
#pragma unroll
                for (int q = 0; q < kW / 2; ++q) {
                    const int j = q / 2 * 4 + q % 2;       // u; v: j + 2
                    const f32x4 x = acc[2 * i + ii][j], y = acc[2 * i + ii][j + 2];
                    f32x4 r;
#pragma unroll
                    for (int t = 0; t < 4; ++t) r[t] = x[t] / (1.f + expf(-x[t])) * y[t];
                    bf16x4 part[3];
                    split4(r, part);
                    char* const at = st + (ii * 16 + (tc.lane & 15)) * kStride + (q * 16 + 4 * (tc.lane >> 4)) * 2;
#pragma unroll
                    for (int t = 0; t < 3; ++t) *reinterpret_cast<bf16x4*>(at + t * kRow) = part[t];
                    __builtin_amdgcn_sched_barrier(0);
                }
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int t = 0; t < 3; ++t)
                copy_rows_out<32, kRow>(st + t * kRow, kStride, reinterpret_cast<char*>(a.p + t * a.third + row_base * a.ld + col_base / 2),
                                        a.ld * 2, 32, tc.lane);
            __builtin_amdgcn_wave_barrier();
        }
    }
};

// acc = da.  du = da v silu'(u) and dv = da silu(u) as thirds, in blocks of 32 columns of each in turn, as u and v are.
struct EpiGateUpBackward {
    const float* uv;         // [rows, duv.ld]
    Thirds duv;
    template <int kW>
    __device__ __forceinline__ void operator()(const TileCoord<kW>& tc, const Accumulators<kW>& acc, char* lds) const {
        constexpr int RW = kWaveRows<kW>, kRow = 2 * RW * 2, kStride = 3 * kRow + 16;
        const int col_base = 2 * tc.col0();                // packed column of this wavefront's block of 2 RW
        if (col_base >= duv.ld) return;
        char* const st = wave_stage(tc, lds);
        constexpr int kTogether = kW == kLargeTile ? 4 : 4;      // tiles whose u and v are on their way together
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
#pragma unroll
            for (int t = 0; t < 3; ++t)
                copy_rows_out<16, kRow>(st + t * kRow, kStride, reinterpret_cast<char*>(duv.p + t * duv.third + row_base * duv.ld + col_base),
                                        duv.ld * 2, 16, tc.lane);
            __builtin_amdgcn_wave_barrier();
        }
    }
};

// ---- products -----------------------------------------------------------------------------------

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
    template <int kW, int kSlots>
    __device__ __forceinline__ void run(int block, OperandRing<kW, kSlots>& smem) const {
        gemm_tile<kLayA, kLayB, true, true>(p, epi, block - first, smem);
    }
};
template <int kLayA, int kLayB, class Epilogue>
ThirdsProduct<kLayA, kLayB, Epilogue> job(const GemmProblem& p, const Epilogue& epi) { return {p, epi, 0}; }

template <int kW, int kSlots, class... Jobs>
__global__ __launch_bounds__(kGemmThreads, kW == kLargeTile || kSlots > kRingSlots ? 1 : 2) void gemm_f32(Jobs... jobs) {
    __shared__ OperandRing<kW, kSlots> smem;
    const int block = blockIdx.x;
    run_job(block, smem, jobs...);
}
inline int steps_of(const GemmProblem& p) { return ceil_div(kSegmentsOfThree * (p.K1 / kTileK), p.splits); }
template <class... Jobs>
void launch_products(int kW, hipStream_t s, Jobs... jobs) {
    int grid = 0;
    ((grid = place_job(jobs, 32 * kW, grid)), ...);
    if (kW == kLargeTile) gemm_f32<kLargeTile, kRingSlots><<<(unsigned)grid, kGemmThreads, 0, s>>>(jobs...);
    else if (grid <= 256 && std::max({steps_of(jobs.p)...}) >= kDeepSteps) gemm_f32<kSmallTile, kDeepRingSlots><<<(unsigned)grid, kGemmThreads, 0, s>>>(jobs...);
    else gemm_f32<kSmallTile, kRingSlots><<<(unsigned)grid, kGemmThreads, 0, s>>>(jobs...);
}

// C = the sum over the parts of a split reduction, as thirds; parts are n floats (rows of C.ld) apart and in the row tiles of the
// live rows (live.kept set) or all of them.
__global__ __launch_bounds__(kThreads) void sum_parts_thirds(const float* parts, int n_parts, size_t n, Thirds C, const int32_t* n_kept,
                                                            int max_chunks, int A) {
    constexpr int kTogether = 4;      // loads under way together
    size_t limit = n;
    if (n_kept != nullptr) limit = min(n, (size_t)((live_rows(n_kept, max_chunks, A) + kTileM - 1) / kTileM * kTileM) * (size_t)C.ld);
    const size_t stride = (size_t)gridDim.x * kThreads * 4;
    for (size_t i = ((size_t)blockIdx.x * kThreads + threadIdx.x) * 4; i < limit; i += stride) {
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
        for (int t = 0; t < 3; ++t) *reinterpret_cast<bf16x4*>(C.p + t * C.third + i) = part[t];
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

// One wavefront per row, four columns per lane and 256: the logits as the sum of their parts, log-softmax at the target bin,
// entropy, ratio, clipped surrogate, and dz = coef * (onehot - softmax) + entropy part as thirds.  With a per-chunk ratio the
// factor is not known yet: the first part of z <- onehot - softmax and the entropy part goes to `extra`; scale_rows makes dz of
// them once the chunk ratios are known.
constexpr int kMaxV = 1024;
struct LossArgs {
    float* z;                // [n_parts][rows, ld]
    int n_parts, V, ld;
    size_t part_stride;
    float* extra;            // [rows, V], unpadded
    Thirds dz;               // p null: no backward pass
    RowMeta meta;
    const int32_t* n_kept;
    int max_chunks, A;
    LossOptions opt;
    float* logp_out;
    RowOut out;
};
__global__ __launch_bounds__(kThreads) void loss_rows(LossArgs p) {
    constexpr int kQ = kMaxV / 256;
    const int lane = threadIdx.x % kWave;
    const int64_t r = (int64_t)blockIdx.x * (kThreads / kWave) + threadIdx.x / kWave;
    const int64_t rows = live_rows(p.n_kept, p.max_chunks, p.A);
    if (r >= (rows + kTileM - 1) / kTileM * kTileM) return;     // later rows: skipped tiles, read by nothing
    const bool live = r < rows;
    const float scale = objective_scale(p.opt, rows);
    float* const zr = p.z + r * p.ld;
    const int b = p.meta.token[r];
    f32x4 z[kQ];
    float mx = -INFINITY, zt = 0.f;
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
        const int c = q * 256 + 4 * lane;
        if (c >= p.ld) continue;
        z[q] = *reinterpret_cast<const f32x4*>(zr + c);
        for (int s = 1; s < p.n_parts; ++s) z[q] += *reinterpret_cast<const f32x4*>(zr + s * p.part_stride + c);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            if (c + t < p.V) mx = fmaxf(mx, z[q][t]);
            if (c + t == b) zt = z[q][t];
        }
    }
    mx = wave_max(mx);
    float se = 0.f, sz = 0.f;
#pragma unroll
    for (int q = 0; q < kQ; ++q)
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if (q * 256 + 4 * lane + t < p.V) {
                const float e = expf(z[q][t] - mx);
                se += e;
                sz += e * z[q][t];
            }
    se = wave_sum(se);
    sz = wave_sum(sz);
    zt = wave_sum(zt);
    const float lse = mx + logf(se);
    const float lp = zt - lse;
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
        const int c = q * 256 + 4 * lane;
        if (c >= p.ld) continue;
        f32x4 g = {}, ent = {};
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if (c + t < p.V) {
                const float pr = expf(z[q][t] - lse);
                g[t] = coef * ((c + t == b ? 1.f : 0.f) - pr);
                ent[t] = ec * pr * (z[q][t] - lse + H);
            }
        if (p.opt.chunk_ratio) {
            *reinterpret_cast<f32x4*>(zr + c) = g;
            if (live) store4(p.extra + r * p.V, c, p.V, ent);
        } else {
            bf16x4 part[3];
            split4(g + ent, part);
#pragma unroll
            for (int t = 0; t < 3; ++t) *reinterpret_cast<bf16x4*>(p.dz.p + t * p.dz.third + r * p.ld + c) = part[t];
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
        for (int t = 0; t < 3; ++t) *reinterpret_cast<bf16x4*>(dz.p + t * dz.third + i) = part[t];
    }
}

// ---- the step -------------------------------------------------------------------------------------

int64_t padded(int64_t n) { return ceil_div64(n, kThirdsUnit) * kThirdsUnit; }
int steps64(int64_t n) { return (int)ceil_div64(n, kTileK) * kTileK; }
int64_t tiles256(int64_t n) { return ceil_div64(n, kTileM) * kTileM; }

// Reduction splits of the products: of those with a fp32 result, into parts.
struct F32Plan {
    GroupPlan gate, down, logits, wdo, G;      // composed: Wdo and G; else down
    GroupPlan level[3];                        // as written {dy, dWo}, {da, dWd}, {dX, dWgu}; composed {da, G}, {dWo, dWd}, {dX, dWgu}
};
// One product's plan: tile and, if it may be split, parts.  (The plans are those of the bf16 path, with six times the steps.  Each
// tile and number of parts forced on its launch at six sizes: within 3 % of the best at five of them, 6 % at 5376 rows of 256.)
GroupPlan plan_one(int64_t M, int64_t N, int64_t K, bool split, int shortest, float us_sum) {
    return plan_group<1>({{tiles256(M), tiles256(N), kSegmentsOfThree * steps64(K) / kTileK, 1, split, shortest}}, us_sum);
}
F32Plan plan_step(const ActorShape& sh, int64_t Mp, bool composed) {
    const int64_t d = sh.d, ff = sh.ff, V = sh.V;
    const auto shape = [](int64_t M, int64_t N, int64_t K, bool split) {
        return GroupShape{tiles256(M), tiles256(N), kSegmentsOfThree * steps64(K) / kTileK, 1, split};
    };
    F32Plan p{};
    p.gate = plan_one(Mp, 2 * padded(ff), d, false, 1, 0.f);
    if (composed) p.wdo = plan_one(ff, V, d, false, 1, 0.f);
    else p.down = plan_one(Mp, d, ff, true, 16, 5.f);
    p.logits = plan_one(Mp, V, composed ? ff : d, true, 8, 0.f);
    if (composed) {
        p.level[0] = plan_group<1>({shape(Mp, ff, V, false)}, 2.f);
        p.G = plan_one(ff, V, Mp, true, 8, 5.f);
        p.level[1] = plan_group<2>({shape(ff, d, V, false), shape(d, V, ff, true)}, 2.f);
    } else {
        p.level[0] = plan_group<2>({shape(Mp, d, V, false), shape(d, V, Mp, true)}, 2.f);
        p.level[1] = plan_group<2>({shape(Mp, ff, d, false), shape(ff, d, Mp, true)}, 2.f);
    }
    GroupShape dX = shape(Mp, d, 2 * padded(ff), true);      // in two parts at most: one goes to dX itself, which the other is added to
    dX.shortest = ceil_div(dX.steps, 2);
    p.level[2] = plan_group<2>({dX, shape(d, 2 * padded(ff), Mp, true)}, 2.f);
    // a small weight gradient in slices of 64 rows
    if (d <= kTileK && ff <= kTileK) p.level[2].splits[1] = ceil_div((int)sh.rows_max(), kTileK);
    return p;
}

struct F32Workspace {
    Thirds Wgu, Wd, Wo, X, a, y, dz, dy, duv;
    Thirds Wdo, G;           // composed evaluation: Wd Wo and a^T dz, both [ff, V]
    float *uv, *z, *z_extra;
    float* dX_part;          // the second of two parts of dX
    float* parts_y;          // parts of y (composed: of G)
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
    const auto thirds = [&](int64_t rows, int64_t columns) {
        Thirds t{};
        t.ld = padded(columns);
        t.third = tiles256(rows) * t.ld;
        t.p = c.take<bf16>((size_t)(3 * t.third + kTileN));      // a tile may read beyond the last row's columns
        return t;
    };
    w.plan = plan_step(sh, Mp, composed);
    const F32Plan& plan = w.plan;
    const int64_t ffp = padded(sh.ff), Vp = padded(sh.V), dp = padded(sh.d);
    w.Wgu = thirds(sh.d, 2 * ffp);
    w.Wd = thirds(sh.ff, sh.d);
    w.Wo = thirds(sh.d, sh.V);
    w.X = thirds(Mp, sh.d);
    w.a = thirds(Mp, sh.ff);
    if (composed) w.Wdo = thirds(sh.ff, sh.V);
    else w.y = thirds(Mp, sh.d);
    if (!composed && plan.down.splits[0] > 1) w.parts_y = c.take<float>((size_t)plan.down.splits[0] * Mp * dp);
    w.z = c.take<float>((size_t)plan.logits.splits[0] * Mp * Vp);
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
    w.uv = c.take<float>((size_t)Mp * 2 * ffp);
    const Thirds dz = thirds(Mp, V);
    Thirds dy{};
    if (!composed) dy = thirds(Mp, d);
    w.duv = thirds(Mp, 2 * ffp);
    if (composed) w.G = thirds(ff, V);
    if (composed) w.parts_y = c.take<float>((size_t)plan.G.splits[0] * ffp * Vp);
    const int o = composed ? plan.level[1].splits[1] : plan.level[0].splits[1], dd = composed ? 1 : plan.level[1].splits[1];
    const int gu = plan.level[2].splits[1];
    if (o > 1) w.parts_o = c.take<float>(o * d * V);
    if (dd > 1) w.parts_d = c.take<float>(dd * ff * d);
    if (bwd) {
        w.dz = dz;
        w.dy = dy;
        w.z_extra = c.take<float>(M * V);
        w.dX_part = c.take<float>(M * d);
        if (gu > 1) w.parts_g = c.take<float>(2 * gu * d * ff);
        w.parts_u = w.parts_g + gu * d * ff;
    } else {
        w.uv = nullptr;
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
        p.A = A.p; p.A2 = A.p + A.third; p.lda = A.ld;
        p.B = B.p; p.B2 = B.p + B.third; p.ldb = B.ld;
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
    const auto sum_thirds = [&](const float* parts, int n_parts, int64_t rows, const Thirds& C, bool batch) {
        const size_t n = (size_t)rows * C.ld;
        sum_parts_thirds<<<(unsigned)std::min<size_t>((n / 4 + kThreads - 1) / kThreads, 2048), kThreads, 0, s>>>(
            parts, n_parts, n, C, batch ? io.n_kept : nullptr, sh.max_chunks, sh.A);
    };

    ThirdsList weights{};
    const int d_rows = (int)padded(d), ff_rows = (int)padded(ff);
    weights.add(ThirdsJob{static_cast<const float*>(io.Wg), w.Wgu, d, ff, d_rows, kPackGate});
    weights.add(ThirdsJob{static_cast<const float*>(io.Wu), w.Wgu, d, ff, d_rows, kPackUp});
    weights.add(ThirdsJob{static_cast<const float*>(io.Wd), w.Wd, ff, d, ff_rows, kPackNone});
    weights.add(ThirdsJob{static_cast<const float*>(io.Wo), w.Wo, d, V, d_rows, kPackNone});
    int rc = launch_prepare_f32(sh, io, w.X, Mp, w.meta, weights, static_cast<float*>(io.dX), s);
    if (rc != PCM_OK) return rc;
    {
        StageTimer t(ST_F32_FORWARD, s);
        launch_products(plan.gate.kW, s, job<kRowsByK, kKByRows>(product(w.X, w.Wgu, Mp, 2 * ffp, d, kRowsAreM), EpiGateUp{w.uv, w.a}));
        if (io.composed) {                                                                             // W_do = Wd Wo
            launch_products(plan.wdo.kW, s, job<kRowsByK, kKByRows>(product(w.Wd, w.Wo, ffp, Vp, d, kRowsUnused), EpiThirds{w.Wdo, ffp}));
        } else if (plan.down.splits[0] == 1) {
            launch_products(plan.down.kW, s, job<kRowsByK, kKByRows>(product(w.a, w.Wd, Mp, dp, ff, kRowsAreM), EpiThirds{w.y, Mp}));
        } else {
            const int n_parts = plan.down.splits[0];
            launch_products(plan.down.kW, s, job<kRowsByK, kKByRows>(product(w.a, w.Wd, Mp, dp, ff, kRowsAreM, n_parts),
                                                                     EpiFloats{w.parts_y, dp, (int64_t)Mp * dp, Mp, dp}));
            sum_thirds(w.parts_y, n_parts, Mp, w.y, true);
        }
        const int n_parts = plan.logits.splits[0];                                                     // z = y Wo, or a W_do
        launch_products(plan.logits.kW, s,
                        job<kRowsByK, kKByRows>(io.composed ? product(w.a, w.Wdo, Mp, Vp, ff, kRowsAreM, n_parts)
                                                            : product(w.y, w.Wo, Mp, Vp, d, kRowsAreM, n_parts),
                                                EpiFloats{w.z, Vp, (int64_t)Mp * Vp, Mp, Vp}));
    }
    {
        StageTimer t(ST_F32_LOSS, s);
        loss_rows<<<(unsigned)(Mp / (kThreads / kWave)), kThreads, 0, s>>>(
            LossArgs{w.z, plan.logits.splits[0], V, Vp, (size_t)Mp * Vp, w.z_extra, w.dz, w.meta, io.n_kept, sh.max_chunks, sh.A, io.opt,
                     io.logp_out, w.out});
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
            const auto da = job<kRowsByK, kRowsByK>(product(w.dz, w.Wdo, Mp, ffp, V, kRowsAreM), swiglu);      // da = dz W_do^T
            launch_products(plan.level[0].kW, s, da);
            if (grads) {
                const int n_parts = plan.G.splits[0];                                                  // G = a^T dz
                launch_products(plan.G.kW, s, job<kKByRows, kKByRows>(product(w.a, w.dz, ffp, Vp, Mp, kRowsAreK, n_parts),
                                                                      EpiFloats{w.parts_y, Vp, (int64_t)ffp * Vp, ffp, Vp}));
                sum_thirds(w.parts_y, n_parts, ffp, w.G, false);
                const auto dWd = job<kRowsByK, kRowsByK>(product(w.G, w.Wo, ff, d, V, kRowsUnused), EpiFloats{io.dWd, d, 0, ff, d});   // G Wo^T
                const int o = plan.level[1].splits[1];
                const auto dWo = job<kKByRows, kKByRows>(product(w.Wd, w.G, d, V, ff, kRowsUnused, o), floats(o, w.parts_o, io.dWo, d, V));   // Wd^T G
                launch_products(plan.level[1].kW, s, dWo, dWd);
            }
        } else {
            const auto dy = job<kRowsByK, kRowsByK>(product(w.dz, w.Wo, Mp, dp, V, kRowsAreM), EpiThirds{w.dy, Mp});     // dy = dz Wo^T
            const auto da = job<kRowsByK, kRowsByK>(product(w.dy, w.Wd, Mp, ffp, d, kRowsAreM), swiglu);                 // da = dy Wd^T
            if (grads) {
                const int o = plan.level[0].splits[1], dd = plan.level[1].splits[1];
                launch_products(plan.level[0].kW, s, job<kKByRows, kKByRows>(product(w.y, w.dz, d, V, Mp, kRowsAreK, o), floats(o, w.parts_o, io.dWo, d, V)), dy);
                launch_products(plan.level[1].kW, s, da, job<kKByRows, kKByRows>(product(w.a, w.dy, ff, d, Mp, kRowsAreK, dd), floats(dd, w.parts_d, io.dWd, ff, d)));
            } else {
                launch_products(plan.level[0].kW, s, dy);
                launch_products(plan.level[1].kW, s, da);
            }
        }
        float* const out_X = static_cast<float*>(io.dX);
        const int x = plan.level[2].splits[0];                                                         // dX = du Wg^T + dv Wu^T
        const auto dX = job<kRowsByK, kRowsByK>(product(w.duv, w.Wgu, Mp, d, 2 * ffp, kRowsAreM, x), EpiFloats{out_X, d, w.dX_part - out_X, M, d});
        if (out_X && x > 1) sums.add(w.dX_part, 1, (size_t)M * d, (size_t)M * d, out_X, true, nullptr, d);
        if (grads) {
            const int gu = plan.level[2].splits[1];                                                    // dWg = X^T du, dWu = X^T dv
            EpiFloatsPair epi{{io.dWg, io.dWu}, 0, d, ff};
            if (gu > 1) {
                const size_t n = (size_t)d * ff;
                sums.add(w.parts_g, gu, n, n, io.dWg);
                sums.add(w.parts_u, gu, n, n, io.dWu);
                epi = EpiFloatsPair{{w.parts_g, w.parts_u}, (int64_t)n, d, ff};
            }
            const auto dWgu = job<kKByRows, kKByRows>(product(w.X, w.duv, d, 2 * ffp, Mp, kRowsAreK, gu), epi);
            if (io.dX) launch_products(plan.level[2].kW, s, dX, dWgu);
            else launch_products(plan.level[2].kW, s, dWgu);
        } else {
            launch_products(plan.level[2].kW, s, dX);
        }
    }
    return launch_finish(sh, io, w.out, sums, FinalPanel{}, true, SumsqLists{}, s);
}

}  // namespace pcm
