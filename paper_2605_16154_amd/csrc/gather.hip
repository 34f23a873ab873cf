// Physical shrinking of the batch (Sec. 4.5): copy the kept chunks' hidden rows into a dense
// matrix and expand the per-trajectory advantage to rows; plus the fixed-order reduction of the
// per-row loss terms of Eq. 11.
//
// The gather is a pure streaming copy (row r of the compacted batch is token r % A of chunk
// kept_idx[r / A]); each workgroup moves a block of rows with 16-byte accesses, several loads in
// flight per lane.  Rows from n_kept * A to the end of their tile of 256 are zero-filled with advantage 0, so they add
// nothing downstream.
#include <algorithm>

#include "actor.h"
#include "thirds.h"

namespace pcm {
namespace {

constexpr int kThreads = 256;
constexpr int kRowsPerBlock = 8;

template <typename Vec>
__device__ inline Vec zero_vec();
template <>
__device__ inline uint4 zero_vec<uint4>() { return make_uint4(0, 0, 0, 0); }
template <>
__device__ inline uint32_t zero_vec<uint32_t>() { return 0u; }
template <>
__device__ inline uint16_t zero_vec<uint16_t>() { return 0; }

// The metadata of rows [r0, r0 + kRowsPerBlock) of the panel, and where they come from (row of hidden, or -1 for a row of zeros).
template <typename Vec>
__device__ inline void gather_metadata(const GatherArgs<Vec>& p, int64_t r0, int64_t rows_valid, int64_t (&src_row)[kRowsPerBlock]) {
    const int tid = threadIdx.x, A = p.A;
    if (tid < kRowsPerBlock) {
        const int64_t r = r0 + tid;
        int64_t src = -1;
        if (r < rows_valid) {
            const int ci = (int)((r + p.row_offset) / A), tok = (int)((r + p.row_offset) % A);
            int id = p.kept_idx[ci];
            float a = 0.f;
            if (id >= 0 && (int64_t)id < (int64_t)p.T * p.N) a = p.adv[id / p.N];
            else id = 0;
            src = (int64_t)id * A + tok;
            const int b = p.tokens[src];                 // all loads before the first store, which might alias them
            const float logp_old = p.logp_old[src];
            p.meta.token[r] = (uint8_t)(b < p.V ? b : p.V - 1);
            p.meta.logp_old[r] = logp_old;
            p.meta.adv[r] = a;
        } else if (r < p.rows_pad) {
            p.meta.token[r] = 0;
            p.meta.logp_old[r] = 0.f;
            p.meta.adv[r] = 0.f;
        }
        src_row[tid] = src;
    }
    __syncthreads();
}
// Rows [block * kRowsPerBlock, + kRowsPerBlock) of the panel.
template <typename Vec>
__device__ inline void gather_rows(const GatherArgs<Vec>& p, int block) {
    __shared__ int64_t src_row[kRowsPerBlock];
    const int vec_per_row = p.vec_per_row, tid = threadIdx.x;
    const int64_t rows_valid = live_rows(p.n_kept, p.max_chunks, p.A) - p.row_offset;
    const int64_t r0 = (int64_t)block * kRowsPerBlock;
    if (r0 >= (rows_valid + 255) / 256 * 256) return;   // beyond the last live row tile: read by nothing (a quarter of the
    gather_metadata(p, r0, rows_valid, src_row);        // copy of a list three quarters full)
    const int total = kRowsPerBlock * vec_per_row;
    constexpr int kUnroll = 8;
    for (int base = tid; base < total; base += kThreads * kUnroll) {
        Vec v[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int e = base + u * kThreads;
            v[u] = zero_vec<Vec>();
            if (e < total) {
                const int64_t src = src_row[e / vec_per_row];
                if (src >= 0) v[u] = p.hidden[src * vec_per_row + e % vec_per_row];
            }
        }
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int e = base + u * kThreads;
            if (e < total) {
                const int64_t r = r0 + e / vec_per_row;
                if (r < p.rows_pad) p.X[r * vec_per_row + e % vec_per_row] = v[u];
            }
        }
    }
}

// Transposed copies of weights: dst[map(c), r] = src[r, c] for [R, C] bf16 matrices (R, C multiples of 64), a workgroup per
// 64 x 64 tile.  kStream: non-temporal stores, which leave the memory-side cache to the sources.
__device__ inline int packed_row(int c, int mode) {
    if (mode == kPackNone) return c;
    return (c / 64) * 128 + (c % 64) + (mode == kPackUp ? 64 : 0);
}
template <bool kStream>
__device__ inline void transpose_tile(const TransposeList& list, int block) {
    __shared__ uint16_t tile[64][66];
    int which = 0;
#pragma unroll
    for (int q = 1; q < TransposeList::kMax; ++q) which += q < list.n && block >= list.first[q] ? 1 : 0;
    const TransposeJob job = list.job[which];
    block -= list.first[which];
    const int tiles_c = job.C / 64;
    const int r0 = block / tiles_c * 64, c0 = block % tiles_c * 64;
    const uint16_t* const src = reinterpret_cast<const uint16_t*>(job.src);
    uint16_t* const dst = reinterpret_cast<uint16_t*>(job.dst);
    const int t = threadIdx.x, tr = t >> 4, tv = t & 15;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int row = tr + 16 * q;
        const uint2 v = *reinterpret_cast<const uint2*>(src + (int64_t)(r0 + row) * job.C + c0 + tv * 4);
        tile[row][tv * 4 + 0] = (uint16_t)(v.x & 0xFFFF);
        tile[row][tv * 4 + 1] = (uint16_t)(v.x >> 16);
        tile[row][tv * 4 + 2] = (uint16_t)(v.y & 0xFFFF);
        tile[row][tv * 4 + 3] = (uint16_t)(v.y >> 16);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int c = tr + 16 * q;
        uint2 v;
        v.x = (uint32_t)tile[tv * 4 + 0][c] | ((uint32_t)tile[tv * 4 + 1][c] << 16);
        v.y = (uint32_t)tile[tv * 4 + 2][c] | ((uint32_t)tile[tv * 4 + 3][c] << 16);
        uint16_t* const to = dst + (int64_t)packed_row(c0 + c, job.mode) * job.R + r0 + tv * 4;
        if (kStream) __builtin_nontemporal_store((uint64_t)v.x | (uint64_t)v.y << 32, reinterpret_cast<uint64_t*>(to));
        else *reinterpret_cast<uint2*>(to) = v;
    }
}
template <bool kStream>
__global__ __launch_bounds__(kThreads) void transpose_weights(TransposeList list) { transpose_tile<kStream>(list, blockIdx.x); }

// What a step does before its first product, in one launch: the weight layouts (if the caller keeps none), the gather of the
// panel's rows, and zeros in a list of fp64 slots.  The three touch different memory, and of a small head each takes a few
// microseconds, which is what a launch costs.  At 2072 rows of 512 -> 768 -> 512 -> 256: five launches of
// 15.4 us -> one of 5.3.  The re-layout by itself 13.2 -> 6.4 us at 512 -> 3328, 98 -> 87 at 4096 -> 11008.
struct ZeroSlots {
    double* p;
    int n;
};
template <typename Vec, bool kLayouts>
__global__ __launch_bounds__(kThreads) void prepare_step(GatherArgs<Vec> gather, int gather_blocks, TransposeList list, ZeroSlots zero) {
    int block = blockIdx.x;
    if (block < gather_blocks) return gather_rows(gather, block);
    block -= gather_blocks;
    if (kLayouts) {
        if (block < list.blocks) return transpose_tile<false>(list, block);
        block -= list.blocks;
    }
    const int i = block * kThreads + (int)threadIdx.x;
    if (i < zero.n) zero.p[i] = 0.0;
}

// Columns c .. c + 7 of a row of C floats, zeros from its end on.
__device__ __forceinline__ void load_eight(const float* row, int c, int C, float (&x)[8]) {
    if (c + 8 <= C) {
        const f32x4_any lo = *reinterpret_cast<const f32x4_any*>(row + c), hi = *reinterpret_cast<const f32x4_any*>(row + c + 4);
#pragma unroll
        for (int t = 0; t < 4; ++t) { x[t] = lo[t]; x[4 + t] = hi[t]; }
    } else {
#pragma unroll
        for (int t = 0; t < 8; ++t) x[t] = c + t < C ? row[c + t] : 0.f;
    }
}
__device__ __forceinline__ void store_thirds(const float (&x)[8], bf16* at) {
    uint32_t part[3][4];
    split_in_three(x, part);
#pragma unroll
    for (int t = 0; t < 3; ++t) *reinterpret_cast<uint4*>(at + t * kThirdsPart) = make_uint4(part[t][0], part[t][1], part[t][2], part[t][3]);
}
__device__ __forceinline__ void store_floats(const float (&x)[8], float* at) {
    *reinterpret_cast<float4*>(at) = make_float4(x[0], x[2], x[4], x[6]);
    *reinterpret_cast<float4*>(at + 4) = make_float4(x[1], x[3], x[5], x[7]);
}
// The fp32 path's counterpart of prepare_step (see launch_prepare_f32).  Bound by memory: four bytes read and four or six written
// per value; every thread has four groups of eight values under way.
__device__ inline void gather_rows_f32(const PrepareF32& p, int block) {
    __shared__ int64_t src_row[kRowsPerBlock];
    const GatherArgs<float>& g = p.gather;
    const int d = g.vec_per_row, tid = threadIdx.x, groups = (int)(p.X.ld / 8);
    const int64_t rows_valid = live_rows(g.n_kept, g.max_chunks, g.A), r0 = (int64_t)block * kRowsPerBlock;
    if (r0 >= (rows_valid + 255) / 256 * 256) {
        if (p.dX != nullptr) {
            const int64_t end = min(r0 + kRowsPerBlock, (int64_t)g.max_chunks * g.A) * d;
            for (int64_t i = r0 * d + tid; i < end; i += kThreads) p.dX[i] = 0.f;
        }
        return;
    }
    gather_metadata(g, r0, rows_valid, src_row);
    const int total = kRowsPerBlock * groups;
    constexpr int kUnroll = 4;
    for (int base = tid; base < total; base += kThreads * kUnroll) {
        float x[kUnroll][8];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int e = base + u * kThreads, row = e / groups;
            const int64_t src = e < total ? src_row[row] : -1;
#pragma unroll
            for (int t = 0; t < 8; ++t) x[u][t] = 0.f;
            if (src >= 0) load_eight(g.hidden + src * d, (e - row * groups) * 8, d, x[u]);
        }
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int e = base + u * kThreads, row = e / groups, c = (e - row * groups) * 8;
            if (e >= total) continue;
            store_floats(x[u], p.X.p + FloatBlocks::at(r0 + row, c, p.X.ld));
            if (p.X3.p != nullptr) store_thirds(x[u], p.X3.p + Thirds::at(r0 + row, c, p.X3.ld));
        }
    }
}
__device__ inline void lay_out_weights(const WeightJobs& list, int block) {
    int which = 0;
#pragma unroll
    for (int q = 1; q < WeightJobs::kMax; ++q) which += q < list.n && block >= list.first[q] ? 1 : 0;
    const WeightJob job = list.job[which];
    const int rows = (job.R + kThirdsUnit - 1) / kThirdsUnit * kThirdsUnit, columns = (job.C + kThirdsUnit - 1) / kThirdsUnit * kThirdsUnit;
    const int64_t total = (int64_t)rows * columns / 8, e0 = (int64_t)(block - list.first[which]) * WeightJobs::kUnits + threadIdx.x;
    constexpr int kUnroll = WeightJobs::kUnits / kThreads;
    auto packed = [&](int c) { return job.mode == kPackNone ? c : c / 32 * 64 + c % 32 + (job.mode == kPackUp ? 32 : 0); };
    // The unit e: eight columns of a row; transposed, eight rows of a column, a wavefront taking 16 columns of 32 rows.
    auto place = [&](int64_t e, int& row, int& c) {
        if (!job.transposed) {
            const int groups = columns / 8;
            row = (int)(e / groups);
            c = (int)(e - (int64_t)row * groups) * 8;
        } else {
            const int64_t wave = e / kWave;
            const int lane = (int)(e % kWave), across = columns / 16;
            row = (int)(wave / across) * 32 + lane / 16 * 8;
            c = (int)(wave % across) * 16 + lane % 16;
        }
    };
    float x[kUnroll][8];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
        const int64_t e = e0 + u * kThreads;
        int row = 0, c = 0;
        if (e < total) place(e, row, c);
        if (!job.transposed) {
            load_eight(job.src + (int64_t)min(row, job.R - 1) * job.C, c, e < total && row < job.R ? job.C : 0, x[u]);
        } else {
#pragma unroll
            for (int t = 0; t < 8; ++t) x[u][t] = e < total && c < job.C && row + t < job.R ? job.src[(int64_t)(row + t) * job.C + c] : 0.f;
        }
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
        const int64_t e = e0 + u * kThreads;
        if (e >= total) continue;
        int row, c;
        place(e, row, c);
        if (job.transposed) store_floats(x[u], job.to.p + FloatBlocks::at(packed(c), row, job.to.ld));
        else if (job.to.p != nullptr) store_floats(x[u], job.to.p + FloatBlocks::at(row, packed(c), job.to.ld));
        else store_thirds(x[u], job.to3.p + Thirds::at(row, packed(c), job.to3.ld));
    }
}
__global__ __launch_bounds__(kThreads) void prepare_step_f32(PrepareF32 p) {
    const int block = blockIdx.x;
    if (block < p.gather_blocks) gather_rows_f32(p, block);
    else lay_out_weights(p.weights, block - p.gather_blocks);
}

constexpr int kFinishThreads = 1024;
// Sum over the workgroup by a fixed tree (thread 0 has the result).
template <int kN>
__device__ inline void tree_sum(double (&acc)[kN], double (&red)[kN][kFinishThreads]) {
    for (int q = 0; q < kN; ++q) red[q][threadIdx.x] = acc[q];
    __syncthreads();
    for (int half = kFinishThreads / 2; half > 0; half >>= 1) {
        if ((int)threadIdx.x < half)
            for (int q = 0; q < kN; ++q) red[q][threadIdx.x] += red[q][threadIdx.x + half];
        __syncthreads();
    }
    for (int q = 0; q < kN; ++q) acc[q] = red[q][0];
}
__device__ inline void sum_lists(const SumsqLists& lists, double* out, double (&red)[1][kFinishThreads]) {
    double sq[1] = {0.0};
    for (int q = 0; q < 4; ++q)
        for (int i = threadIdx.x; i < lists.count[q]; i += kFinishThreads) sq[0] += lists.parts[q][i];
    tree_sum(sq, red);
    if (threadIdx.x == 0) *out = sq[0];
}
__global__ __launch_bounds__(kFinishThreads) void sum_of_squares(SumsqLists lists, double* out) {
    __shared__ double red[1][kFinishThreads];
    sum_lists(lists, out, red);
}

struct LossReduceArgs {
    RowOut row;
    const int32_t* n_kept;
    int max_chunks, A;
    LossOptions opt;
    float *loss_out, *stats_out;
    int n_stats;
};
// One workgroup; lane-strided fp64 partials combined by a fixed tree, so the result does not
// depend on anything but the row values.
__device__ inline void reduce_loss(const LossReduceArgs& p) {
    __shared__ double red[5][kFinishThreads];
    const int64_t rows = live_rows(p.n_kept, p.max_chunks, p.A);
    double acc[5] = {0, 0, 0, 0, 0};
    for (int64_t r = threadIdx.x; r < rows; r += kFinishThreads) {
        acc[0] += (double)p.row.term[r];
        acc[1] += (double)p.row.ratio[r];
        acc[2] += (double)p.row.dlogp[r];
        acc[3] += (double)p.row.clipped[r];
        acc[4] += (double)p.row.entropy[r];
    }
    tree_sum(acc, red);
    if (threadIdx.x != 0) return;
    const double scale = (double)objective_scale(p.opt, rows);
    *p.loss_out = (float)(-scale * acc[0] - (double)p.opt.entropy_coef * scale * acc[4]);
    if (p.stats_out) {
        const double n = rows > 0 ? (double)rows : 1.0;
        p.stats_out[0] = (float)(acc[3] / n);
        p.stats_out[1] = (float)(acc[1] / n);
        p.stats_out[2] = (float)(acc[2] / n);
        p.stats_out[3] = (float)rows;
        if (p.n_stats > 4) p.stats_out[4] = (float)(acc[4] / n);
    }
}

__global__ __launch_bounds__(kFinishThreads) void finish_loss(LossReduceArgs loss) { reduce_loss(loss); }

// A workgroup's share of a sum of parts; returns the thread's sum of the squares of what it wrote.  Bound by memory: the
// parts are read eight at a time, so that their loads are under way together (the five sums and the loss of a step of 5376 fp32 rows of
// 256 -> 1024 -> 256: six launches of 46 us -> two of 20).
template <class Vec>
__device__ inline double sum_parts(const PartsSum& job, int block, size_t n, size_t limit) {
    constexpr int kPer = sizeof(Vec) / sizeof(float), kTogether = 8;
    if ((int)threadIdx.x >= job.threads) return 0.0;
    const size_t stride = (size_t)job.blocks * job.threads * kPer;
    double sq = 0.0;
    for (size_t i = ((size_t)block * job.threads + threadIdx.x) * kPer; i < n; i += stride) {
        auto part = [&](int s) { return *reinterpret_cast<const Vec*>(job.parts + (size_t)s * job.stride + i); };
        Vec acc = {};
        if (i < limit) acc = job.add ? *reinterpret_cast<const Vec*>(job.out + i) + part(0) : part(0);
        for (int s0 = 1; i < limit && s0 < job.n_parts; s0 += kTogether) {
            Vec v[kTogether];
#pragma unroll
            for (int u = 0; u < kTogether; ++u) v[u] = part(min(s0 + u, job.n_parts - 1));
#pragma unroll
            for (int u = 0; u < kTogether; ++u)
                if (s0 + u < job.n_parts) acc = acc + v[u];
        }
        *reinterpret_cast<Vec*>(job.out + i) = acc;
        if (job.sumsq != nullptr)
            for (int e = 0; e < kPer; ++e) sq += (double)reinterpret_cast<const float*>(&acc)[e] * (double)reinterpret_cast<const float*>(&acc)[e];
    }
    return sq;
}
typedef __attribute__((ext_vector_type(4))) float f32x4;
__global__ __launch_bounds__(kFinishThreads) void finish_step(PartsSums sums, FinalPanel panel, LossReduceArgs loss, int with_loss) {
    int block = blockIdx.x;
    if (with_loss && block == 0) return reduce_loss(loss);       // first: it takes longest where the sums are small
    block -= with_loss;
    int which = 0;
#pragma unroll
    for (int q = 1; q < PartsSums::kMax; ++q) which += q < sums.n && block >= sums.job[q].first ? 1 : 0;
    const PartsSum job = sums.job[which];
    block -= job.first;
    size_t n = job.n, limit = job.n;              // with live_row a multiple of four, or n
    if (job.live_row > 0) {
        const int64_t tile = job.live_tile, live = live_rows(loss.n_kept, loss.max_chunks, loss.A);
        limit = min(n, (size_t)((live + tile - 1) / tile * tile) * job.live_row);
        if (job.add) n = limit;
    }
    double sq = job.vec ? sum_parts<f32x4>(job, block, n, limit) : sum_parts<float>(job, block, n, limit);
    if (job.sumsq == nullptr || !panel()) return;
    __shared__ double wave_part[kFinishThreads / kWave];
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) sq += __shfl_xor(sq, o, kWave);
    if (threadIdx.x % kWave == 0) wave_part[threadIdx.x / kWave] = sq;
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int q = 1; q < kFinishThreads / kWave; ++q) sq += wave_part[q];
    job.sumsq[block] = sq;
}

// One wavefront per chunk slot.  rho_c = exp(sum over the chunk's tokens of (logp - logp_old)), the sum in fp64 (its terms
// cancel).  With one lane per slot the rows of a chunk were read one after the other: 192 chunks 31 -> 6 us.
constexpr int kRatioThreads = 256, kRatioSlots = kRatioThreads / kWave;   // chunk slots per workgroup
__global__ __launch_bounds__(kRatioThreads) void chunk_ratio_rows(const float* __restrict__ dlogp,
                                                                  const float* __restrict__ adv_row,
                                                                  const int32_t* __restrict__ n_kept, int max_chunks, int A,
                                                                  int64_t row_offset, int64_t rows_pad, LossOptions opt,
                                                                  float* __restrict__ term, float* __restrict__ ratio,
                                                                  uint8_t* __restrict__ clipped, float* __restrict__ coef) {
    // chunk slots of a panel that starts at batch row row_offset (a multiple of A); the arrays are the panel's
    const int lane = threadIdx.x % kWave;
    const int64_t c = (int64_t)blockIdx.x * kRatioSlots + threadIdx.x / kWave;
    const int64_t r0 = c * A;
    if (r0 >= rows_pad) return;                         // uniform over the wavefront, as is all that follows
    const int64_t rows_batch = live_rows(n_kept, max_chunks, A);
    const int64_t rows = rows_batch - row_offset;
    const int64_t r1 = r0 + A < rows_pad ? r0 + A : rows_pad;
    if (r0 >= rows) return;                             // beyond the kept chunks: nothing reads these rows
    double sum = 0.0;
    for (int64_t r = r0 + lane; r < r1; r += kWave) sum -= (double)dlogp[r];
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) sum += __shfl_xor(sum, o, kWave);
    const float w = opt.chunk_weight ? opt.chunk_weight[c + row_offset / A] : 1.f;
    const LossRow lr = loss_from_ratio(expf((float)sum), adv_row[r0], w, opt, objective_scale(opt, rows_batch));
    for (int64_t r = r0 + lane; r < r1; r += kWave) {
        term[r] = r == r0 ? lr.term : 0.f;
        ratio[r] = lr.ratio;
        clipped[r] = lr.clipped;
        coef[r] = lr.coef;
    }
}

// Rows [0, live rows) only: rows beyond them hold zeros (or, in row tiles that the logit product
// skipped, nothing) and are not read by anything downstream.
__global__ __launch_bounds__(256) void scale_rows_f32(float* __restrict__ dz, const float* __restrict__ extra,
                                                      const float* __restrict__ coef, const int32_t* __restrict__ n_kept,
                                                      int max_chunks, int A, int64_t rows_max, int V) {
    const int64_t live = live_rows(n_kept, max_chunks, A), rows = live < rows_max ? live : rows_max;
    const int64_t n = rows * V;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        float x = coef[i / V] * dz[i];
        if (extra) x += extra[i];
        dz[i] = x;
    }
}

// Rows whose gradient factor is zero (ratio cut by the clip, zero advantage, zero weight) have an all-zero row of dz and
// add nothing to any gradient.  This launch lists the panel's other rows in order, decides whether the backward products run
// over that list or over all live rows, copies the listed rows of up to four matrices into dense ones, and clears the rows of
// dX that the products will not write.
//
// The kernels that know a row's factor leave the number of rows with a gradient in every block of kListBlock rows; a
// workgroup here owns one such block, or a quarter of one where the blocks are few, and adds up the counts before it (and all
// of them, for the decision) by itself, so there is no launch that only makes the list.  The copies are bound by memory: a
// workgroup moves its listed rows as one contiguous stretch of the dense matrix, 16 bytes per thread and eight in flight.
// (A wavefront per row instead: all of them start in the same column of rows a power of two apart, 430 -> 650 us.)  The list, four copies
// and the zeros, six launches against this one: 2072 rows of 512 and 768 16.9 -> 3.5 us, 43,008 rows of 4096 and 11008
// (24 thousand listed) 429 -> 422 us.
constexpr int kListThreads = 256, kListWaves = kListThreads / kWave;
// Workgroups per block where there are no more than two blocks to a CU: the copies of a block are then spread over four.  Whole
// steps, one / four to a block: 672 rows of 512 -> 768 76.0 / 74.8 us, of 1024 -> 2816 133.9 / 130.5; 2072 of 512 -> 768 81.3 / 80.1,
// 7616 143.8 / 143.1; beyond the line (about 8000 rows) 8960 161 / 163, 14,336 238 / 239.
constexpr int kListParts = 4;
struct ListArgs {
    const uint8_t* clipped;
    const float* adv;
    const float* chunk_weight;      // by chunk of the batch, or null
    const int32_t* counts;          // [rows_pad / kListBlock]
    const int32_t* n_kept;
    int max_chunks, A;
    int64_t row_offset;
    int rows_pad, rows_in_dX, dX_vecs;
    uint4* dX;                      // or null
    LiveSources whole, listed;
    int row_vecs[LiveSources::kCount];   // 16-byte units per row; 0: not copied
    int32_t* idx;
    LivePlan* plan;
    int parts;                      // workgroups per block: 1 or kListParts
};
// Rows from[0 .. n) of src -> dst[0 .. n) (dense), rows of `vecs` units, by the whole workgroup.
__device__ __forceinline__ void copy_rows(const uint4* __restrict__ src, uint4* __restrict__ dst, int vecs, const int32_t* from, int n) {
    constexpr int kUnroll = 8;
    const int total = n * vecs;
    for (int base = threadIdx.x; base < total; base += kListThreads * kUnroll) {
        uint4 v[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int el = base + u * kListThreads;
            v[u] = make_uint4(0, 0, 0, 0);
            if (el < total) {
                const int row = (uint32_t)el / (uint32_t)vecs;
                v[u] = src[(int64_t)from[row] * vecs + (el - row * vecs)];
            }
        }
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int el = base + u * kListThreads;
            if (el < total) dst[el] = v[u];
        }
    }
}
__global__ __launch_bounds__(kListThreads) void list_live_rows(ListArgs p) {
    __shared__ int part[2][kListWaves];
    __shared__ int32_t from[kListBlock];
    const int t = threadIdx.x, lane = t % kWave, wave = t / kWave;
    const int block = blockIdx.x / p.parts, of_block = blockIdx.x % p.parts;
    const int64_t rows64 = live_rows(p.n_kept, p.max_chunks, p.A) - p.row_offset;
    const int rows = (int)(rows64 < 0 ? 0 : (rows64 > p.rows_pad ? p.rows_pad : rows64));
    const int blocks = (rows + kListBlock - 1) / kListBlock, tile_end = (rows + 255) / 256 * 256;
    const int panel_blocks = p.rows_pad / kListBlock;
    if (block > 0 && block < panel_blocks && block * kListBlock >= tile_end) return;   // uniform; the first one writes the plan
    int all = 0, before = 0;
#pragma unroll 4
    for (int i = t; i < blocks; i += kListThreads) {
        const int c = p.counts[i];
        all += c;
        before += i < block ? c : 0;
    }
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) {
        all += __shfl_xor(all, o, kWave);
        before += __shfl_xor(before, o, kWave);
    }
    if (lane == 0) {
        part[0][wave] = all;
        part[1][wave] = before;
    }
    __syncthreads();
    all = before = 0;
#pragma unroll
    for (int q = 0; q < kListWaves; ++q) {
        all += part[0][q];
        before += part[1][q];
    }
    // the list pays once the rows it drops outweigh the copies it needs: at least one row in sixteen
    const bool use_list = (int64_t)(rows - all) * 16 >= rows && rows > 0;
    const int n = use_list ? all : rows;
    if (blockIdx.x == 0 && t == 0) {
        p.plan->n_rows = n;
        p.plan->listed = use_list ? 1 : 0;
        for (int q = 0; q < LiveSources::kCount; ++q) p.plan->src[q] = use_list ? p.listed.p[q] : p.whole.p[q];
    }
    if (block >= panel_blocks) {                        // zero rows from the end of the list to the end of its last row tile
        const int m0 = n + (block - panel_blocks) * kListBlock + of_block * (kListBlock / p.parts);
        const int pad = min((n + 255) / 256 * 256 - m0, kListBlock / p.parts);
        if (t < pad) p.idx[m0 + t] = -1;
        if (!use_list) return;
#pragma unroll
        for (int q = 0; q < LiveSources::kCount; ++q) {
            uint4* const dst = static_cast<uint4*>(const_cast<void*>(p.listed.p[q])) + (int64_t)m0 * p.row_vecs[q];
            for (int at = t; at < pad * p.row_vecs[q]; at += kListThreads) dst[at] = make_uint4(0, 0, 0, 0);
        }
        return;
    }
    const int r0 = block * kListBlock, q = r0 + lane % kListBlock;     // the block's flags, by every wavefront alike
    const bool in = q < rows;
    const int at = in ? q : r0 < rows ? rows - 1 : 0;                  // all loads unconditional
    const uint8_t cut = p.clipped[at];
    const float a = p.adv[at];
    const float w = p.chunk_weight != nullptr && rows > 0 ? p.chunk_weight[(at + p.row_offset) / p.A] : 1.f;
    const uint32_t mask = (uint32_t)__ballot(in && cut == 0 && a != 0.f && w != 0.f) & ((1u << kListBlock) - 1u);
    const int listed = __popc(mask), k0 = listed * of_block / p.parts, k1 = listed * (of_block + 1) / p.parts;
    if (t < kListBlock) {
        const int k = __popc(mask & ((1u << t) - 1u));
        if (((mask >> t) & 1u) != 0) from[k] = r0 + t;
        if (use_list && ((mask >> t) & 1u) != 0 && of_block == 0) p.idx[before + k] = r0 + t;
        if (!use_list && r0 + t < rows && of_block == 0) p.idx[r0 + t] = r0 + t;
    }
    __syncthreads();
    if (use_list)
#pragma unroll
        for (int k = 0; k < LiveSources::kCount; ++k)
            copy_rows(static_cast<const uint4*>(p.whole.p[k]),
                      static_cast<uint4*>(const_cast<void*>(p.listed.p[k])) + (int64_t)(before + k0) * p.row_vecs[k], p.row_vecs[k], from + k0,
                      k1 - k0);
    if (p.dX == nullptr) return;
    for (int r = r0 + of_block; r < min(r0 + kListBlock, min(tile_end, p.rows_in_dX)); r += p.parts)
        if (((mask >> (r - r0)) & 1u) == 0)
            for (int v = t; v < p.dX_vecs; v += kListThreads) p.dX[(int64_t)r * p.dX_vecs + v] = make_uint4(0, 0, 0, 0);
}

}  // namespace

int launch_live_rows(const ActorShape& sh, const ActorIO& io, const uint8_t* clipped, const float* adv, const int32_t* counts,
                     int64_t row_offset, int64_t rows_pad, const LiveSources& whole, const LiveSources& listed,
                     const int64_t (&row_bytes)[LiveSources::kCount], void* dX, int64_t rows_in_dX, int32_t* idx, LivePlan* plan,
                     hipStream_t s) {
    StageTimer t(ST_LIVE_ROWS, s);
    ListArgs p{clipped, adv, io.opt.chunk_weight, counts, io.n_kept, sh.max_chunks, sh.A, row_offset, (int)rows_pad, (int)rows_in_dX,
               (int)((int64_t)sh.d * 2 / 16), static_cast<uint4*>(dX), whole, listed, {}, idx, plan, 1};
    for (int q = 0; q < LiveSources::kCount; ++q) p.row_vecs[q] = (int)(row_bytes[q] / 16);
    const int64_t blocks = (rows_pad + 256) / kListBlock;          // those of the panel, and a row tile behind the list
    if (blocks <= 512) p.parts = kListParts;                        // see kListParts
    list_live_rows<<<(unsigned)(blocks * p.parts), kListThreads, 0, s>>>(p);
    return launch_status();
}

int launch_prepare_f32(const ActorShape& sh, const ActorIO& io, const FloatBlocks& X, const Thirds& X3, int64_t rows_pad, RowMeta meta,
                       const WeightJobs& weights, float* dX, hipStream_t s) {
    StageTimer t(ST_GATHER, s);
    const GatherArgs<float> gather{static_cast<const float*>(io.hidden), io.tokens, io.logp_old, io.adv, io.kept_idx, io.n_kept,
                                   sh.max_chunks, sh.T, sh.N, sh.A, sh.V, sh.d, 0, rows_pad, nullptr, meta};
    const int blocks = (int)ceil_div64(rows_pad, kRowsPerBlock);
    prepare_step_f32<<<(unsigned)(blocks + weights.blocks), kThreads, 0, s>>>(PrepareF32{gather, X, X3, weights, dX, blocks});
    return launch_status();
}

namespace {
int gather(const ActorShape& sh, const ActorIO& io, int elem_bytes, void* X, int64_t row_offset, int64_t rows_pad,
                  RowMeta meta, const TransposeList& layouts, double* zero, int n_zero, hipStream_t s) {
    StageTimer t(ST_GATHER, s);
    const int64_t row_bytes = (int64_t)sh.d * elem_bytes;
    const unsigned blocks = (unsigned)ceil_div64(rows_pad, kRowsPerBlock);
    const unsigned grid = (unsigned)layouts.blocks + blocks + (unsigned)ceil_div(n_zero, kThreads);
    const bool aligned16 = row_bytes % 16 == 0 && (reinterpret_cast<uintptr_t>(io.hidden) & 15u) == 0 &&
                           (reinterpret_cast<uintptr_t>(X) & 15u) == 0;
    auto launch = [&](auto vec, int64_t vec_per_row) {
        using Vec = decltype(vec);
        const GatherArgs<Vec> args{static_cast<const Vec*>(io.hidden), io.tokens, io.logp_old, io.adv, io.kept_idx, io.n_kept,
                                   sh.max_chunks, sh.T, sh.N, sh.A, sh.V, (int)vec_per_row, row_offset, rows_pad,
                                   static_cast<Vec*>(X), meta};
        if (layouts.n > 0) prepare_step<Vec, true><<<grid, kThreads, 0, s>>>(args, (int)blocks, layouts, ZeroSlots{zero, n_zero});
        else prepare_step<Vec, false><<<grid, kThreads, 0, s>>>(args, (int)blocks, layouts, ZeroSlots{zero, n_zero});
    };
    if (aligned16) launch(uint4{}, row_bytes / 16);
    else if (elem_bytes == 4) launch(uint32_t{}, sh.d);
    else launch(uint16_t{}, sh.d);
    return launch_status();
}
}  // namespace
int launch_gather(const ActorShape& sh, const ActorIO& io, void* X, int64_t row_offset, int64_t rows_pad, RowMeta meta,
                  const TransposeList& layouts, double* zero, int n_zero, hipStream_t s) {
    return gather(sh, io, 2, X, row_offset, rows_pad, meta, layouts, zero, n_zero, s);
}
int launch_gather_f32(const ActorShape& sh, const ActorIO& io, float* X, int64_t rows_pad, RowMeta meta, hipStream_t s) {
    return gather(sh, io, 4, X, 0, rows_pad, meta, TransposeList{}, nullptr, 0, s);
}

void launch_transposes(const TransposeList& list, bool stream, hipStream_t s) {
    StageTimer t(ST_WEIGHT_LAYOUT, s);
    if (stream) transpose_weights<true><<<(unsigned)list.blocks, kThreads, 0, s>>>(list);
    else transpose_weights<false><<<(unsigned)list.blocks, kThreads, 0, s>>>(list);
}

// A CU reads about 70 GB/s, so a small sum of many parts wants many workgroups rather than full ones: the widest shape that
// has 256 of them (56 parts of 65,536 floats in 16 / 256 workgroups 13 / 8 us; of few parts the thinner ones only take longer
// to start).
struct SumShape {
    int blocks, threads, vec;
};
static SumShape sum_shape(size_t n_floats, bool may_vec, int n_parts) {
    const SumShape shapes[4] = {{0, kFinishThreads, 1}, {0, kThreads, 1}, {0, kFinishThreads, 0}, {0, kThreads, 0}};
    SumShape best{};
    for (const SumShape& q : shapes) {
        if (q.vec && !may_vec) continue;
        best = q;
        const int64_t want = ceil_div64((int64_t)n_floats, (int64_t)q.threads * (q.vec ? 4 : 1));
        best.blocks = (int)std::min<int64_t>(want, PartsSums::kBlocksMax);
        if (want >= 256 || n_parts < 16) break;
    }
    return best;
}
void PartsSums::add(const float* parts, int n_parts, size_t n_floats, size_t stride, float* out, bool add_to, double* sumsq, int live_row,
                    int live_tile) {
    PartsSum& p = job[n++];
    p = PartsSum{parts, n_parts, add_to ? 1 : 0, n_floats, stride, out, sumsq, live_row, live_tile, blocks, 0, 0, 0};
    const bool may_vec = n_floats % 4 == 0 && stride % 4 == 0 && ((reinterpret_cast<uintptr_t>(out) | reinterpret_cast<uintptr_t>(parts)) & 15u) == 0;
    const SumShape shape = sum_shape(n_floats, may_vec, n_parts);
    p.blocks = shape.blocks;
    p.threads = shape.threads;
    p.vec = shape.vec;
    blocks += p.blocks;
}
int PartsSums::blocks_for(size_t n_floats, int n_parts) {
    return std::max(sum_shape(n_floats, true, n_parts).blocks, sum_shape(n_floats, false, n_parts).blocks);
}

int launch_finish(const ActorShape& sh, const ActorIO& io, RowOut out, const PartsSums& sums, const FinalPanel& panel, bool with_loss,
                  const SumsqLists& lists, hipStream_t s) {
    StageTimer t(ST_REDUCE, s);
    const LossReduceArgs loss{out, io.n_kept, sh.max_chunks, sh.A, io.opt, io.loss_out, io.stats_out, io.n_stats};
    if (sums.blocks > 0)
        finish_step<<<(unsigned)(sums.blocks + (with_loss ? 1 : 0)), kFinishThreads, 0, s>>>(sums, panel, loss, with_loss ? 1 : 0);
    else if (with_loss)
        finish_loss<<<1, kFinishThreads, 0, s>>>(loss);
    if (lists.parts[0] != nullptr) sum_of_squares<<<1, kFinishThreads, 0, s>>>(lists, io.opt.grad_sumsq_out);
    return launch_status();
}

int launch_chunk_ratio(const ActorShape& sh, const ActorIO& io, RowMeta meta, RowOut out, int64_t row_offset,
                       int64_t rows_pad, hipStream_t s) {
    StageTimer t(ST_REDUCE, s);
    const int64_t slots = ceil_div64(rows_pad, sh.A);
    chunk_ratio_rows<<<(unsigned)ceil_div64(slots, kRatioSlots), kRatioThreads, 0, s>>>(out.dlogp, meta.adv, io.n_kept, sh.max_chunks,
                                                                      sh.A, row_offset, rows_pad, io.opt, out.term,
                                                                      out.ratio, out.clipped, out.coef);
    return launch_status();
}

int launch_scale_rows_f32(const ActorShape& sh, const ActorIO& io, float* dz, const float* extra, const float* coef,
                          int64_t rows, hipStream_t s) {
    StageTimer t(ST_REDUCE, s);
    const int64_t blocks = ceil_div64(rows * sh.V, 256);
    scale_rows_f32<<<(unsigned)(blocks < 4096 ? blocks : 4096), 256, 0, s>>>(dz, extra, coef, io.n_kept, sh.max_chunks, sh.A, rows, sh.V);
    return launch_status();
}

}  // namespace pcm
