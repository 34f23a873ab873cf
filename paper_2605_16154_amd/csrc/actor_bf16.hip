// bf16 path of the masked GRPO actor step (Eq. 11): matrix-core GEMMs with fused epilogues.
//
// Forward:  X -> [gate|up] GEMM with silu(u)*v fused -> down GEMM -> logit GEMM (fp32, split reduction) ->
//           log-softmax / ratio / clipped surrogate / dz in one pass over the rows.
// Backward: dy = dz Wo^T; da = dy Wd^T with the gated-activation derivative fused (du, dv
//           overwrite the two factors the forward epilogue stored); weight gradients reduce over
//           the row dimension (small outputs as partial products over slices of the rows, summed at the
//           end of the panel: no atomics); dX = du Wg^T + dv Wu^T as one GEMM over two
//           reduction segments.  Products that do not depend on one another share a launch (see plan_backward).
// Composed evaluation (an option): the down and the logit projection as the one matrix
//           W_do = Wd Wo [ff, V] formed at the start of the call: z = a W_do; G = a^T dz,
//           dWd = G Wo^T, dWo = Wd^T G, da = dz W_do^T.  y and dy are never formed; the three
//           products through d shrink to products through V.
//
// The forward and input-gradient products take both operands reduction-contiguous; for the forward
// pass the [in, out] weights are first copied transposed (gate and up interleaved in blocks of 64
// columns so that the activation can be fused).  The weight-gradient products reduce over the row
// dimension and read the activations as they are, through the GEMM's LDS transpose reads.
//
// Buffers are padded to a multiple of 256 rows.  The rows from the last live one to the end of its
// row tile are zero with zero advantage, so they contribute nothing to any output; rows behind that
// tile are neither written nor read, by any launch.
//
// Backward over the rows that carry a gradient: a row whose ratio the clip cuts (or whose advantage or weight is
// zero) has an all-zero row of dz, hence of dy, du, dv and dX, and adds nothing to a weight gradient.  After the loss
// a kernel lists the other rows; when at least one row in sixteen drops out, dz, y, a and X are copied row by row
// into dense matrices of the listed rows and every backward product runs over those (the da epilogue reads its
// factors through the list, dX is written through it, its other rows zero-filled).  The decision, the row count and
// the operand addresses stay in device memory: no host synchronisation.  Without an entropy bonus only (with one,
// every row has a gradient), and not in the composed evaluation.
//
// A long batch is worked through in row panels (kPanelRows rows, a multiple of both the tile height
// and the chunk length): gather, forward, loss and backward run panel by panel over the same
// activation buffers, the weight gradients of every panel after the first are added to what the
// earlier ones left, and the per-row loss terms are reduced once at the end.  The workspace is then
// bounded by the panel (about 5 GB at d = 4096, ff = 11008) instead of growing with the batch, and
// a panel's activations are still in the memory-side cache when its backward pass reads them.
#include "gemm_bf16.h"

namespace pcm {
namespace {

constexpr size_t kMaxSplitTiles = 256;   // tiles x parts of a split reduction: one workgroup per CU
constexpr size_t kSumBlocksMax = PartsSums::kBlocksMax;

// Rows of a product over a panel of the batch that its row tiles cover, from the device-side count (kept as in GemmProblem).
struct LiveTiles {
    const int32_t* kept;
    int kept_max, rows_per_kept, row_offset, row_length;
    __device__ size_t rows() const {
        const int64_t rows = live_rows(kept, kept_max, rows_per_kept) - row_offset;
        return rows <= 0 ? 0 : (size_t)((rows + kTileM - 1) / kTileM * kTileM);
    }
};

// out[i] = the sum over the parts of a split reduction (n is a multiple of 4; parts are n floats apart), rounded once to bf16: a
// product that the next GEMM takes as an operand.  Of a product over the rows of the batch (live.kept is set) only the row tiles
// that it computed: of a list far shorter than its buffer the rest are parts that nobody wrote.  Log-probabilities, all rows of
// the buffer / live tiles: 112 rows in a buffer of 2296, 1024 -> 11008, six parts 87.0 / 80.1 us; 448 in one of 5376, 1024 -> 8192,
// three parts 101.8 / 93.1; 56 in one of 672, 4096 -> 11008, five parts 175.1 / 166.3.
__global__ void sum_parts_bf16(const float* parts, int n_parts, size_t n, bf16* out, LiveTiles live) {
    constexpr int kTogether = 4;      // loads under way together
    const size_t stride = (size_t)gridDim.x * blockDim.x * 4, limit = live.kept != nullptr ? min(n, live.rows() * live.row_length) : n;
    for (size_t i = ((size_t)blockIdx.x * blockDim.x + threadIdx.x) * 4; i < limit; i += stride) {
        f32x4 acc = *reinterpret_cast<const f32x4*>(parts + i);
        for (int s0 = 1; s0 < n_parts; s0 += kTogether) {
            f32x4 v[kTogether];
#pragma unroll
            for (int u = 0; u < kTogether; ++u) v[u] = *reinterpret_cast<const f32x4*>(parts + (size_t)min(s0 + u, n_parts - 1) * n + i);
#pragma unroll
            for (int u = 0; u < kTogether; ++u)
                if (s0 + u < n_parts) acc += v[u];
        }
        *reinterpret_cast<bf16x4*>(out + i) = to_bf16x4(acc[0], acc[1], acc[2], acc[3]);
    }
}

void launch_sum_bf16(const float* parts, int n_parts, size_t n, bf16* out, const LiveTiles& live, hipStream_t s) {
    const size_t blocks = (n / 4 + 255) / 256;
    sum_parts_bf16<<<(unsigned)(blocks < kSumBlocksMax ? blocks : kSumBlocksMax), 256, 0, s>>>(parts, n_parts, n, out, live);
}

// The loss over the rows of a panel: log-softmax at the target bin, row entropy, ratio, clipped surrogate and
// dz = coef * (onehot - softmax) + entropy_coef * scale * softmax * (log softmax + H) as bf16.  The logits arrive in fp32
// as the partial products of a split reduction, parts[s][row][256], summed here.  With a per-chunk ratio the factor is
// not known yet: dz <- onehot - softmax, the entropy part goes to dz_extra, and the rows are scaled once the chunk
// ratios are known.
//
// A launch of its own and not an epilogue of the logit product: a product with a single column of tiles has few
// workgroups (9 for 2072 rows), so its reduction has to be split, and as straight-line code over the accumulators the
// loss was 64 KB of instructions that each of those workgroups fetched for one use.  16 lanes hold a row, 4 x 4
// columns each (1 KB of a row per four loads), so that the reductions are four shuffles; bound by reading the logits,
// which are still in the memory-side cache.  Logit product and loss together, before and after: 2072 rows at d = 512
// 31.5 -> 20.9 us, 672 rows at d = 4096 83 -> 25 us, 5376 rows 109 -> 34 us.
constexpr int kLossThreads = 256, kLossRows = kLossThreads / 16;   // rows per workgroup
struct LossRowsArgs {
    const float* parts;
    int n_parts;
    size_t part_stride;      // floats between two parts
    const uint8_t* token;
    const float* logp_old;
    const float* adv_row;
    const int32_t* n_kept;
    int max_chunks, A;
    int row_offset;          // batch row of the panel's row 0 (the per-row arrays are the panel's parts)
    int rows_pad;            // rows of the panel
    LossOptions opt;
    bf16* dz;                // [rows_pad, 256] or nullptr
    bf16* dz_extra;          // [rows_pad, 256]: entropy part, per-chunk ratio only
    float* logp_out;         // may be nullptr
    RowOut out;
    int32_t* live_count;     // [rows_pad / kLossRows] rows with a gradient, or nullptr
};
static_assert(kLossRows == kListBlock, "a workgroup counts one block of the list");
// The number of rows with a gradient among the workgroup's 16 (all of whose threads call this; `has`: of a thread's row).
__device__ inline void count_live_rows(bool has, int32_t* to) {
    __shared__ int32_t wave_count[kLossThreads / kWave];
    const uint64_t votes = __ballot(has);
    if (threadIdx.x % kWave == 0) wave_count[threadIdx.x / kWave] = __popcll(votes) / 16;
    __syncthreads();
    if (threadIdx.x == 0) *to = wave_count[0] + wave_count[1] + wave_count[2] + wave_count[3];
}
__device__ inline float sum16(float x) {
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    return x;
}
__global__ __launch_bounds__(kLossThreads) void loss_rows_bf16(LossRowsArgs p) {
    const int64_t rows_batch = live_rows(p.n_kept, p.max_chunks, p.A);
    const int64_t rows_live = rows_batch - p.row_offset;        // live rows of this panel (may be <= 0)
    const int m = blockIdx.x * kLossRows + (int)(threadIdx.x >> 4), lane = threadIdx.x & 15;
    // rows up to the end of the last live row tile are written (as rows without a gradient); nothing reads later ones
    const int64_t limit = rows_live <= 0 ? 0 : (rows_live + kTileM - 1) / kTileM * kTileM;
    if (m >= limit || m >= p.rows_pad) return;                  // uniform over the workgroup: both are multiples of 16
    const float scale = objective_scale(p.opt, rows_batch);
    const float* src = p.parts + (size_t)m * 256 + lane * 4;
    f32x4 z[4];                                                 // z[q][t]: column 64 q + 4 lane + t
#pragma unroll
    for (int q = 0; q < 4; ++q) z[q] = *reinterpret_cast<const f32x4*>(src + q * 64);
    for (int s = 1; s < p.n_parts; ++s) {
        src += p.part_stride;
#pragma unroll
        for (int q = 0; q < 4; ++q) z[q] += *reinterpret_cast<const f32x4*>(src + q * 64);
    }
    const int tok = p.token[m];
    float mx = -INFINITY;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int t = 0; t < 4; ++t) mx = fmaxf(mx, z[q][t]);
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
    float se = 0.f, sz = 0.f, zt = 0.f;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const float e = __expf(z[q][t] - mx);
            se += e;
            sz += e * z[q][t];
            zt += (q * 64 + lane * 4 + t == tok) ? z[q][t] : 0.f;
        }
    se = sum16(se);
    sz = sum16(sz);
    zt = sum16(zt);
    const float lse = mx + __logf(se), lp = zt - lse, ent = lse - sz / se;      // H = -sum p log p
    const bool live = m < rows_live;
    const float w = (p.opt.chunk_weight && live) ? p.opt.chunk_weight[(m + p.row_offset) / p.A] : 1.f;
    const LossRow lr = loss_row(lp, p.logp_old[m], p.adv_row[m], w, p.opt, scale);
    if (lane == 0) {
        p.out.dlogp[m] = lr.dlogp;
        p.out.entropy[m] = live ? ent : 0.f;
        if (!p.opt.chunk_ratio) {
            p.out.term[m] = live ? lr.term : 0.f;
            p.out.ratio[m] = lr.ratio;
            p.out.clipped[m] = lr.clipped;
        }
        if (p.logp_out && live) p.logp_out[m] = lp;
    }
    if (p.live_count != nullptr)
        count_live_rows(live && lr.clipped == 0 && p.adv_row[m] != 0.f && w != 0.f, p.live_count + blockIdx.x);
    if (p.dz == nullptr) return;
    const float coef = live ? (p.opt.chunk_ratio ? 1.f : lr.coef) : 0.f;
    const float ec = live ? p.opt.entropy_coef * scale : 0.f;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float g[4], h[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const float lpj = z[q][t] - lse, pr = __expf(lpj);
            g[t] = coef * ((q * 64 + lane * 4 + t == tok ? 1.f : 0.f) - pr);
            h[t] = ec * pr * (lpj + ent);
        }
        const int64_t at = (int64_t)m * 256 + q * 64 + lane * 4;
        if (p.opt.chunk_ratio) {
            *reinterpret_cast<bf16x4*>(p.dz + at) = to_bf16x4(g[0], g[1], g[2], g[3]);
            *reinterpret_cast<bf16x4*>(p.dz_extra + at) = to_bf16x4(h[0], h[1], h[2], h[3]);
        } else {
            *reinterpret_cast<bf16x4*>(p.dz + at) = to_bf16x4(g[0] + h[0], g[1] + h[1], g[2] + h[2], g[3] + h[3]);
        }
    }
}

// Per-chunk ratio: dz[r, :] = coef[r] dz[r, :] (+ extra[r, :]) over the live rows of a panel, 16 lanes per row as above, and
// the counts of rows with a gradient, which are known only now.
struct ScaleRowsArgs {
    bf16* dz;
    const bf16* extra;               // or nullptr
    const float *coef, *adv_row;
    const uint8_t* clipped;
    const float* chunk_weight;       // by chunk of the batch, or nullptr
    const int32_t* n_kept;
    int max_chunks, A, row_offset, rows_pad;
    int32_t* live_count;             // or nullptr
};
__global__ __launch_bounds__(kLossThreads) void scale_rows_bf16(ScaleRowsArgs p) {
    const int64_t rows = min(live_rows(p.n_kept, p.max_chunks, p.A) - p.row_offset, (int64_t)p.rows_pad);
    if ((int64_t)blockIdx.x * kLossRows >= rows) return;        // uniform
    const int m = blockIdx.x * kLossRows + (int)(threadIdx.x >> 4), lane = threadIdx.x & 15;
    const bool live = m < rows;
    if (p.live_count != nullptr) {
        const int at = live ? m : blockIdx.x * kLossRows;
        const float w = p.chunk_weight != nullptr ? p.chunk_weight[(at + p.row_offset) / p.A] : 1.f;
        count_live_rows(live && p.clipped[at] == 0 && p.adv_row[at] != 0.f && w != 0.f, p.live_count + blockIdx.x);
    }
    if (!live) return;
    const float coef = p.coef[m];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int64_t at = (int64_t)m * 256 + q * 128 + lane * 8;
        const bf16x8 v = *reinterpret_cast<const bf16x8*>(p.dz + at);
        bf16x8 e = {};
        if (p.extra != nullptr) e = *reinterpret_cast<const bf16x8*>(p.extra + at);
        bf16x8 r;
#pragma unroll
        for (int t = 0; t < 8; ++t) r[t] = (__bf16)__builtin_fmaf(coef, (float)v[t], (float)e[t]);
        *reinterpret_cast<bf16x8*>(p.dz + at) = r;
    }
}

// The forward products' operand layouts of the four weight matrices, in one buffer.
struct PackedHead {
    bf16 *WguT, *WdT, *WoT;
    size_t bytes;
};
PackedHead carve_packed(void* base, int d, int ff, int V) {
    Carver c(base);
    PackedHead p;
    p.WguT = c.take<bf16>((size_t)2 * ff * d);
    p.WdT = c.take<bf16>((size_t)d * ff);
    p.WoT = c.take<bf16>((size_t)V * d);
    p.bytes = c.used();
    return p;
}

constexpr int64_t kPanelRows = 57344;   // target height of a row panel (224 row tiles)

// Height of the row panels a batch of `sh.rows_max()` rows is worked through in: the whole (padded) batch if it
// is at most a panel and a quarter, or if the head is evaluated in composed form; otherwise the largest common
// multiple of the tile height and the chunk length that does not exceed the target (the caller's, else kPanelRows).
int64_t panel_rows(const ActorShape& sh, bool composed, int target) {
    const int64_t Mp = ceil_div64(sh.rows_max(), kTileM) * kTileM;
    if (composed) return Mp;
    const int64_t want = target > 0 ? target : kPanelRows;
    int64_t x = kTileM, y = sh.A;
    while (y != 0) { const int64_t t = x % y; x = y; y = t; }             // gcd
    const int64_t unit = (int64_t)kTileM / x * sh.A;                        // lcm(256, A)
    const int64_t rp = unit * (want / unit > 0 ? want / unit : 1);
    return Mp <= rp + rp / 4 ? Mp : rp;
}

// Reduction split for an output of `tiles` tiles and `steps` 64-wide reduction steps.  An output
// that already covers the 256 CUs is not split; a small output is split so that tiles * splits
// fills the chip (and never exceeds kMaxSplitTiles, which sizes the buffer of partial products),
// keeping at least 8 steps per workgroup.
int pick_splits(int tiles, int steps) {
    if (tiles >= 256) return 1;
    int s = (int)kMaxSplitTiles / tiles;
    const int max_s = steps / 8 > 0 ? steps / 8 : 1;
    if (s > max_s) s = max_s;
    return s < 1 ? 1 : s;
}

// Tile and reduction splits of products that share a launch: those with the least estimated time.  A workgroup takes a few
// microseconds to start and to write its tile, and per 64-wide step 0.94 us with the large tile (the matrix pipe) or 0.46 with
// the small one (LDS, which two workgroups of a CU share; see tile_for).  The launch takes what its longest workgroup does, or
// the work shared out over 256 CUs and about half a workgroup more at the end; parts are written, read back and added up at
// about 4 TB/s.  Measured against every one of these choices forced on all three launches of a step (tile, and the longest
// reduction from 6 steps to all of them): the estimate is within 1 % of the best, or better, at 14 of 16 sizes from 448 rows
// of 3072 -> 768 to 5376 of 3328 -> 7168, and 2 to 3 % off at 9856 rows of 1792 -> 1792 and 2688 of 3072 -> 2560.
struct GroupShape {
    int64_t M, N;
    int steps, count;      // `count` products of these sizes
    bool split;            // whether the reduction may be split (fp32 parts, summed by a later launch)
    int shortest = 1;      // and into no fewer steps than these
};
struct GroupPlan {
    static constexpr int kMax = 4;
    int kW, splits[kMax];
};
template <int kN>
GroupPlan plan_group(const GroupShape (&jobs)[kN], float us_sum) {
    // (little arithmetic: every call of a step comes through here, and a small one is bound by the host)
    int large[kN], most_splits[kN], longest_split = 0;
    float part_us[kN];                                   // writing or reading one part
    for (int q = 0; q < kN; ++q) {
        const GroupShape& j = jobs[q];
        large[q] = (int)(j.M / kTileM) * (int)(j.N / kTileN);
        most_splits[q] = j.split ? std::max(1, std::min({(int)kMaxSplitTiles / large[q], j.steps / j.shortest, 64})) : 1;
        part_us[q] = (float)large[q] * (float)j.count * (kTileM * kTileN * 4 / 4e6f);
        if (most_splits[q] > 1) longest_split = std::max(longest_split, j.steps);
    }
    GroupPlan best{};
    float best_us = 0.f;
    for (int kW : {kLargeTile, kSmallTile}) {
        const float us_per_step = kW == kLargeTile ? 0.94f : 0.46f, us_fixed = kW == kLargeTile ? 5.f : 3.f;
        const int tiles_per_large = kW == kLargeTile ? 1 : 4;
        for (int most : {4, 6, 8, 12, 16, 24, 32, 48, 64, 96, 1 << 20}) {     // longest reduction of a workgroup
            if (most < longest_split || most == 1 << 20 || longest_split == 0) {
                GroupPlan plan{kW, {}};
                int steps = 0;                           // of the longest workgroup
                int64_t workgroups = 0;
                float work = 0.f, sum = 0.f;
                for (int q = 0; q < kN; ++q) {
                    const GroupShape& j = jobs[q];
                    const int s = std::min(most_splits[q], ceil_div(j.steps, most)), len = s > 1 ? ceil_div(j.steps, s) : j.steps;
                    plan.splits[q] = s;
                    steps = std::max(steps, len);
                    const int64_t n = (int64_t)large[q] * (tiles_per_large * s * j.count);
                    workgroups += n;
                    work += (float)n * (us_fixed + us_per_step * (float)len);
                    if (s > 1) sum += (float)(2 * s + 1) * part_us[q];
                }
                float us = us_fixed + us_per_step * (float)steps;
                if (workgroups > 256) us = std::max(us, work / 256 + 0.5f * work / (float)workgroups);
                if (sum > 0.f) us += us_sum + sum;
                if (best.kW == 0 || us < best_us) {
                    best = plan;
                    best_us = us;
                }
            }
            if (longest_split == 0) break;
        }
    }
    return best;
}

// Whole steps with a launch per product / with launches shared by the products of a dependency level (and the sums at the
// end): 2072 rows of 512 -> 768 121 / 79 us, 448 of 3072 -> 768 137 / 107, 512 of 3072 -> 1536 182 / 145, 5376 of 3328 -> 7168
// 1578 / 1454; at 4096 -> 11008 4704 rows, three quarters live, 2679 / 2530, 10,752 with a chunk ratio 6758 / 6500.
//
// Rows of a panel up to which the listed rows of a, du and dv have buffers of their own, so that dWd, which reads the first,
// and da, which writes the others, may run side by side.  What that saves shrinks as the launches grow, while the two further
// buffers of ff columns grow with them.  Whole steps, half to two thirds of the rows listed, apart / side by side: 2296 rows of
// 512 -> 768 88.8 / 81.0 us, of 1024 -> 2816 219.6 / 186.7, of 4096 -> 11008 1401 / 1332; 4480 105 / 98.9, 344 / 318, 2227 / 2225;
// 8064 152 / 144, 449 / 454, 3702 / 3717; 8960 162 / 158, 493 / 501, 4176 / 4154; 16,128 253 / 234, 739 / 744, 7115 / 7162; 32,256
// 397 / 394, 1372 / 1365, 14,210 / 14,080.
constexpr int64_t kApartRows = 8192;

// Large tiles of dX up to which it shares a launch with dWg and dWu.  What sharing saves is the part-filled last round of each;
// with many rounds that is little, and where the products meet the workgroups of an XCD no longer walk through the same
// panels in step.  Whole steps, every row, apart / shared, us:
//   4096 -> 11008:  672 tiles 6340 / 6240, 1344 12,625 / 12,380, 2016 18,370 / 18,800, 2688 24,715 / 24,960; unmasked, panels of
//                   3584, 129.4 / 130.9 ms (dWg and dWu in front where their reductions are the longer: 133.5 ms)
//   4096 -> 2048:   672 1423 / 1369, 1344 2792 / 2750, 1792 3549 / 3488
//   2048 -> 5632:   672 3635 / 3540, 1344 7206 / 7174, 1568 8389 / 8438, 1792 9407 / 9585
//   8192 -> 8192:   672 4781 / 4748, 1344 9288 / 9425, 1696 11,461 / 11,544, 2016 13,494 / 13,584, 2688 17,988 / 18,144
// The composed evaluation, one panel whatever the batch, all its levels: 4096 -> 11008 2688 17,520 / 17,760, 5376 34,550 / 35,510;
// 2048 -> 5632 2688 10,415 / 10,710, 5376 20,485 / 21,260.
constexpr int64_t kGroupTiles = 6 * 256;

// How the backward products of a panel are launched.
struct BackwardPlan {
    // as written: {dy, dWo}, then {da, dWd}, then {dX, dWg and dWu}; composed: {da, G}, then {dX, dWg and dWu, dWo, dWd}, where not
    // grouped dWg, dWu, {dWo, dWd}, dX
    GroupPlan level[3];
    bool group[3];
    int split_o, split_d, split_gu, split_G;
};
BackwardPlan plan_backward(const ActorShape& sh, int64_t Rp, bool composed, bool listed) {
    const int64_t d = sh.d, ff = sh.ff, V = sh.V;
    const int rows = (int)(Rp / kTileK), by_d = sh.d / kTileK, by_ff = sh.ff / kTileK, by_V = sh.V / kTileK;
    BackwardPlan b{};
    if (composed) {
        b.group[0] = b.group[2] = Rp / kTileM * (d / kTileN) <= kGroupTiles;
        b.level[0] = plan_group<2>({{Rp, ff, by_V, 1, false}, {ff, V, rows, 1, true}}, 2.f);
        if (b.group[2]) {
            b.level[2] = plan_group<4>({{d, V, by_ff, 1, true}, {ff, d, by_V, 1, false}, {Rp, d, 2 * by_ff, 1, false}, {d, ff, rows, 2, true}}, 2.f);
            b.split_gu = b.level[2].splits[3];
        } else {
            b.level[2] = plan_group<2>({{d, V, by_ff, 1, true}, {ff, d, by_V, 1, false}}, 2.f);
        }
        b.split_G = b.group[0] ? b.level[0].splits[1] : pick_splits((int)(ff / kTileM), rows);
        b.split_o = b.level[2].splits[0];
        b.split_d = 1;
    } else {
        b.level[0] = plan_group<2>({{Rp, d, by_V, 1, false}, {d, V, rows, 1, true}}, 2.f);
        b.level[1] = plan_group<2>({{Rp, ff, by_d, 1, false}, {ff, d, rows, 1, true}}, 2.f);
        b.level[2] = plan_group<2>({{Rp, d, 2 * by_ff, 1, false}, {d, ff, rows, 2, true}}, 2.f);
        b.group[0] = true;
        b.group[1] = !listed || Rp <= kApartRows;
        b.group[2] = Rp / kTileM * (d / kTileN) <= kGroupTiles;
        b.split_o = b.level[0].splits[1];
        b.split_d = b.level[1].splits[1];
        b.split_gu = b.level[2].splits[1];
        if (!b.group[1]) b.split_d = pick_splits((int)(ff / kTileM * (d / kTileN)), rows);
    }
    if (!b.group[2]) b.split_gu = pick_splits((int)(d / kTileM * (ff / kTileN)), rows);
    return b;
}
// fp32 buffer that products use one after the other: the logits, and parts of split reductions that the next launch adds up
// into a bf16 matrix.
struct SharedParts {
    float* at;
    size_t floats;
    bool hold(size_t n) const { return n <= floats; }
};
struct Bf16Workspace {
    bf16 *WguT, *WdT, *WoT;
    bf16 *X, *fu, *fv, *a, *y, *dz, *dz_extra;   // one panel each; fu, fv: SwiGLU derivative factors, then du, dv
    bf16 *a_lo, *y_lo;                           // per-chunk ratio: rounding remainders of a and y
    bf16* dy;
    bf16 *yc, *Xc, *dzc, *ac;   // backward over listed rows: those of y, X, dz and a
    bf16 *du, *dv;              // and du, dv, which in tall panels take the places of ac and a (see kApartRows)
    int32_t* live_count;   // [Rp / 16] rows with a gradient by block of 16
    int32_t* live_idx;     // [Rp] the listed rows
    LivePlan* plan;        // null: backward over all rows
    double* sumsq[4];      // sums of squares of the final dWg, dWu, dWd, dWo by workgroup (null: not asked for)
    int sumsq_count[4];
    bf16 *Wdo, *G;  // composed evaluation: Wd Wo and a^T dz, both [ff, V]
    SharedParts parts;   // the logits; parts of the down projection, of W_do and of G
    float *parts_o, *parts_d, *parts_g, *parts_u;   // those of dWo, dWd, dWg, dWu, which are added up at the end of a panel
    BackwardPlan plan_b;
    RowMeta meta;   // whole batch
    RowOut out;     // whole batch
    int64_t Mp;     // padded rows of the batch
    int64_t Rp;     // rows of a panel
    size_t bytes;
};

// Whether the backward products of a call run over the listed rows (see the head of this file).
bool lists_live_rows(const LossOptions& opt, bool bwd, bool composed) {
    return bwd && !composed && !opt.dense_backward && opt.entropy_coef == 0.f;
}

Bf16Workspace carve(void* ws, const ActorShape& sh, bool bwd, bool grads, const LossOptions& opt, bool composed) {
    Carver c(ws);
    Bf16Workspace w{};
    const bool split = opt.chunk_ratio != 0;
    const int panel_target = opt.panel_rows;
    const size_t Mp = (size_t)ceil_div64(sh.rows_max(), kTileM) * kTileM;
    const size_t Rp = (size_t)panel_rows(sh, composed, panel_target);
    const size_t d = sh.d, ff = sh.ff, V = sh.V;
    w.Mp = (int64_t)Mp;
    w.Rp = (int64_t)Rp;
    w.WguT = c.take<bf16>(2 * ff * d);
    w.WdT = c.take<bf16>(d * ff);
    w.WoT = c.take<bf16>(V * d);
    w.X = c.take<bf16>(Rp * d);
    w.a = c.take<bf16>(Rp * ff);
    if (bwd) w.fu = c.take<bf16>(Rp * ff);
    if (bwd) w.fv = c.take<bf16>(Rp * ff);
    w.y = c.take<bf16>(Rp * d);
    if (split) w.a_lo = c.take<bf16>(Rp * ff);
    if (split) w.y_lo = c.take<bf16>(Rp * d);
    w.dz = c.take<bf16>(Rp * V);
    w.meta.token = c.take<uint8_t>(Mp);
    w.meta.logp_old = c.take<float>(Mp);
    w.meta.adv = c.take<float>(Mp);
    w.out.term = c.take<float>(Mp);
    w.out.ratio = c.take<float>(Mp);
    w.out.dlogp = c.take<float>(Mp);
    w.out.clipped = c.take<uint8_t>(Mp);
    w.out.entropy = c.take<float>(Mp);
    w.out.coef = c.take<float>(Mp);
    if (bwd) w.dz_extra = c.take<bf16>(Rp * V);
    if (bwd) w.dy = c.take<bf16>(Rp * d);
    if (lists_live_rows(opt, bwd, composed)) {
        w.ac = c.take<bf16>(Rp * ff);
        w.du = (int64_t)Rp <= kApartRows ? c.take<bf16>(Rp * ff) : w.ac;
        w.dv = (int64_t)Rp <= kApartRows ? c.take<bf16>(Rp * ff) : w.a;
        w.yc = c.take<bf16>(Rp * d);
        w.Xc = c.take<bf16>(Rp * d);
        w.dzc = c.take<bf16>(Rp * V);
        w.live_count = c.take<int32_t>(Rp / kListBlock);
        w.live_idx = c.take<int32_t>(Rp);
        w.plan = c.take<LivePlan>(1);
    }
    if (bwd) w.plan_b = plan_backward(sh, (int64_t)Rp, composed, lists_live_rows(opt, bwd, composed));
    const BackwardPlan& plan = w.plan_b;
    if (grads) {
        if (plan.split_o > 1) w.parts_o = c.take<float>((size_t)plan.split_o * d * V);
        if (plan.split_d > 1) w.parts_d = c.take<float>((size_t)plan.split_d * ff * d);
        if (plan.split_gu > 1) w.parts_g = c.take<float>((size_t)plan.split_gu * d * ff);
        if (plan.split_gu > 1) w.parts_u = c.take<float>((size_t)plan.split_gu * d * ff);
    }
    if (grads && opt.grad_sumsq_out != nullptr) {
        const size_t size[4][2] = {{d, ff}, {d, ff}, {ff, d}, {d, V}};
        const int level[4] = {2, 2, 1, 0}, splits[4] = {plan.split_gu, plan.split_gu, plan.split_d, plan.split_o};
        for (int q = 0; q < 4; ++q) {       // unsplit: one per wavefront of the product; else one per workgroup of the sum
            const int kW = plan.group[level[q]] ? plan.level[level[q]].kW : tile_for((int64_t)size[q][0], (int64_t)size[q][1], 1);
            const size_t tile = 32 * (size_t)kW, waves = 4 * (size[q][0] / tile) * (size[q][1] / tile);
            w.sumsq_count[q] = splits[q] == 1 ? (int)waves : PartsSums::blocks_for(size[q][0] * size[q][1], splits[q]);
            w.sumsq[q] = c.take<double>((size_t)w.sumsq_count[q]);
        }
    }
    w.Wdo = c.take<bf16>(ff * V);
    if (grads) w.G = c.take<bf16>(ff * V);
    // parts of split reductions; of the logits (one column of tiles) there is at least one part whatever the panel's height
    const size_t row_tiles = Rp / kTileM;
    w.parts.floats = (row_tiles > kMaxSplitTiles ? row_tiles : kMaxSplitTiles) * (size_t)kTileM * kTileN;
    w.parts.at = c.take<float>(w.parts.floats);
    w.bytes = c.used();
    return w;
}

// Which GEMM dimension runs over the kept rows, so that work beyond the device-side count is skipped; the rows
// are those of a panel that starts at batch row `row_offset`.
struct KeptRows {
    const int32_t* kept;
    int kept_max, rows_per_kept;
    int row_offset;
};

// Where a weight-gradient launch leaves the sums of the squares of its final values: the unsplit GEMM four per
// output tile, the kernel that sums a split reduction one per workgroup (parts == nullptr: nowhere).
struct SumsqTarget {
    double* parts;
    FinalPanel final_panel;
};

// A product with a long reduction whose fp32 result goes to C, or is added to it (accumulate), as one launch or as parts that
// launch_finish adds up (no atomics): p.splits, the epilogue and, for parts, the entry in `sums`.  The weight gradients are the
// case A^T B over the kept rows with both operands stored [rows][features].
EpiStoreF32 reduction_epilogue(GemmProblem& p, int splits, float* C, float* parts, bool accumulate, const SumsqTarget& sq, PartsSums& sums) {
    p.splits = splits;
    p.skip_if_empty = splits == 1 && accumulate ? 1 : 0;
    const size_t n = (size_t)p.M * p.N;
    if (splits == 1) return EpiStoreF32{C, p.N, 0, accumulate ? 1 : 0, sq.parts, sq.final_panel};
    sums.add(parts, splits, n, n, C, accumulate, sq.parts);
    return EpiStoreF32{parts, p.N, (int64_t)n, 0, nullptr, FinalPanel{}};
}
// C = a product with a long reduction and a small output, as parts and rounded once to bf16.
template <int kLayA, int kLayB>
[[nodiscard]] int launch_reduction_bf16(GemmProblem p, bf16* C, const SharedParts& parts, int stage, hipStream_t s) {
    StageTimer t(stage, s);
    p.splits = pick_splits((p.M / kTileM) * (p.N / kTileN), p.K1 / kTileK);
    const size_t n = (size_t)p.M * p.N;
    if (p.splits == 1) {
        launch_gemm<kLayA, kLayB>(p, EpiStoreBf16{C, p.N, p.M}, s);
        return PCM_OK;
    }
    if (!parts.hold(p.splits * n)) return PCM_EWORKSPACE;
    launch_gemm<kLayA, kLayB>(p, EpiStoreF32{parts.at, p.N, (int64_t)n, 0, nullptr, FinalPanel{}}, s);
    launch_sum_bf16(parts.at, p.splits, n, C, LiveTiles{}, s);
    return PCM_OK;
}

GemmProblem problem(const bf16* A, int64_t lda, const bf16* B, int64_t ldb, int M, int N, int K,
                    const KeptRows& kr, int rows_role) {
    GemmProblem p{};
    p.A = A; p.lda = lda; p.B = B; p.ldb = ldb;
    p.A2 = A; p.B2 = B;
    p.M = M; p.N = N; p.K1 = K; p.K2 = 0; p.splits = 1;
    p.kept = kr.kept; p.kept_max = kr.kept_max; p.rows_per_kept = kr.rows_per_kept; p.rows_role = rows_role;
    p.row_offset = kr.row_offset; p.skip_if_empty = 0; p.cut = kCutNone;
    return p;
}

// C [M, N] bf16 = a product over the rows of the batch.  With few tiles and a long reduction it is computed as parts of a
// split reduction (fp32) and summed, if the estimate of plan_group says so; at least 16 steps a part.
// Measured, whole passes without gradients, before (small tiles only, at most four parts) / now: 672 rows of 4096 -> 11008, five
// parts on large tiles, 262 / 237 us (its down projection 96 -> 62, the sum 6 -> 10); 512 of 512 -> 9984 58.7 / 52.2; 896 of
// 2304 -> 2560 86 / 79.
// The plan is made for a full buffer, so that a row's bits do not depend on how many others are in the list.  Lists up to a quarter
// of the buffer would like more parts: plan / that rule before, full and with a quarter of the list: 2296 rows of 1024 -> 11008
// 194.7 and 108.4 / 199.9 and 120.2 us, 1344 of 2048 -> 5632 124 and 94 / 135 and 88, 5376 of 512 -> 5632 137 and 86 / 145 and 74
// (112 rows of those 68 / 54).
[[nodiscard]] int launch_rows_bf16(GemmProblem p, bf16* C, const SharedParts& parts, hipStream_t s) {
    const GroupPlan plan = plan_group<1>({{p.M, p.N, (p.K1 + p.K2) / kTileK, 1, true, 16}}, 5.f);
    if (plan.splits[0] == 1) {
        launch_row_gemm(p, EpiStoreBf16{C, p.N, p.M}, s);
        return PCM_OK;
    }
    p.splits = plan.splits[0];
    const size_t n = (size_t)p.M * p.N;
    if (!parts.hold(p.splits * n)) return PCM_EWORKSPACE;
    const EpiStoreF32 epi{parts.at, p.N, (int64_t)n, 0, nullptr, FinalPanel{}};
    if (plan.kW == kSmallTile) launch_gemm_tile<kRowsByK, kRowsByK, kSmallTile>(p, epi, s);
    else launch_gemm_tile<kRowsByK, kRowsByK, kLargeTile>(p, epi, s);
    launch_sum_bf16(parts.at, p.splits, n, C, LiveTiles{p.kept, p.kept_max, p.rows_per_kept, p.row_offset, p.N}, s);
    return PCM_OK;
}

}  // namespace

// Packed weights of more than this are stored non-temporally.  The cache holds 256 MB: of a small head the next step finds
// the result there, of a large one it does not, and the stores displace the bf16 weights that the optimizer has just
// written and the re-layout reads.  Optimizer, re-layout and the step after them, ordinary / non-temporal stores:
// log-probabilities of 672 rows 67 MB 324 / 330 us, 102 MB 457 / 464, 146 MB 632 / 621, 194 MB 837 / 818, 260 MB 1138 / 1112,
// 338 MB 1464 / 1438; a training step of 1344 rows 67 MB 706 / 721, 146 MB 1263 / 1268, 194 MB 1599 / 1584, 260 MB 2195 / 2166.
constexpr size_t kStreamPackBytes = (size_t)160 << 20;

size_t packed_head_bytes(int d, int ff, int V) { return carve_packed(nullptr, d, ff, V).bytes; }

int pack_head_weights(const void* Wg, const void* Wu, const void* Wd, const void* Wo, int d, int ff, int V, void* packed,
                      hipStream_t s) {
    const PackedHead p = carve_packed(packed, d, ff, V);
    const bool stream = p.bytes > kStreamPackBytes;
    TransposeList list{};
    list.add(static_cast<const bf16*>(Wg), d, ff, p.WguT, kPackGate);
    list.add(static_cast<const bf16*>(Wu), d, ff, p.WguT, kPackUp);
    list.add(static_cast<const bf16*>(Wd), ff, d, p.WdT, kPackNone);
    list.add(static_cast<const bf16*>(Wo), d, V, p.WoT, kPackNone);
    launch_transposes(list, stream, s);
    return launch_status();
}

size_t actor_bf16_workspace_bytes(const ActorShape& sh, bool want_grads, const LossOptions& opt, bool composed) {
    return carve(nullptr, sh, want_grads, want_grads, opt, composed).bytes;
}

int actor_bf16_run(const ActorShape& sh, const ActorIO& io, void* ws, hipStream_t s) {
    const bool grads = io.want_grads();
    const bool bwd = grads || io.dX != nullptr;
    // With one ratio per chunk the log-probabilities of a chunk's A rows add up in the exponent, and so do their
    // errors: the forward pass then carries a and y as pairs of bf16 values (value and rounding remainder) through
    // the down and the logit product, which brings the error of a log-probability from about 2e-3 down to 1e-5.
    const bool split = io.opt.chunk_ratio != 0;
    Bf16Workspace w = carve(ws, sh, bwd, grads, io.opt, io.composed);
    const int d = sh.d, ff = sh.ff, V = sh.V;
    const bf16* Wg = static_cast<const bf16*>(io.Wg);
    const bf16* Wu = static_cast<const bf16*>(io.Wu);
    const bf16* Wd = static_cast<const bf16*>(io.Wd);
    const bf16* Wo = static_cast<const bf16*>(io.Wo);

    const KeptRows all_rows{nullptr, 0, 0, 0};
    int rc = PCM_OK;
    TransposeList layouts{};
    if (io.opt.packed_weights != nullptr) {               // layouts kept by the caller: nothing to re-lay-out
        const PackedHead ph = carve_packed(const_cast<void*>(io.opt.packed_weights), d, ff, V);
        w.WguT = ph.WguT; w.WdT = ph.WdT; w.WoT = ph.WoT;
    } else {
        layouts.add(Wg, d, ff, w.WguT, kPackGate);         // [d, ff] -> packed rows of [2 ff, d]
        layouts.add(Wu, d, ff, w.WguT, kPackUp);
        if (io.composed) {
            // W_do = Wd Wo [ff, V], from the weights as given (Wd [rows][K], Wo [K][rows])
            rc = launch_reduction_bf16<kRowsByK, kKByRows>(problem(Wd, d, Wo, V, ff, V, d, all_rows, kRowsUnused), w.Wdo, w.parts,
                                                           ST_WEIGHT_LAYOUT, s);
            if (rc != PCM_OK) return rc;
        } else {
            layouts.add(Wd, ff, d, w.WdT, kPackNone);      // [ff, d] -> [d, ff]
            layouts.add(Wo, d, V, w.WoT, kPackNone);       // [d, V]  -> [V, d]
        }
    }

    // slots for sums of squares that no launch of this call writes must read as zero: cleared with the first gather
    const bool want_sumsq = grads && io.opt.grad_sumsq_out != nullptr && ws != nullptr && w.sumsq[0] != nullptr;
    const int n_zero = want_sumsq ? (int)(w.sumsq[3] - w.sumsq[0]) + w.sumsq_count[3] : 0;   // the four lists follow one another

    PartsSums last_sums{};
    FinalPanel last_panel{};
    for (int64_t row0 = 0; row0 < w.Mp; row0 += w.Rp) {
        // this panel: batch rows [row0, row0 + Mp); all row-indexed arrays below are its parts
        const int Mp = (int)(w.Mp - row0 < w.Rp ? w.Mp - row0 : w.Rp);
        const bool first = row0 == 0;
        const KeptRows kr{io.n_kept, sh.max_chunks, sh.A, (int)row0};
        SumsqTarget sq[4] = {};    // dWg, dWu, dWd, dWo
        if (want_sumsq) {
            const FinalPanel fp{io.n_kept, sh.max_chunks, sh.A, row0, row0 + w.Rp >= w.Mp ? INT64_MAX : row0 + w.Rp};
            for (int q = 0; q < 4; ++q) sq[q] = SumsqTarget{w.sumsq[q], fp};
        }
        const RowMeta meta{w.meta.token + row0, w.meta.logp_old + row0, w.meta.adv + row0};
        const RowOut out{w.out.term + row0, w.out.ratio + row0, w.out.dlogp + row0, w.out.clipped + row0,
                         w.out.entropy + row0, w.out.coef + row0};
        rc = launch_gather(sh, io, w.X, row0, Mp, meta, first ? layouts : TransposeList{}, w.sumsq[0], first ? n_zero : 0, s);
        if (rc != PCM_OK) return rc;
        {
            StageTimer t(ST_GEMM_GATE_UP, s);
            const GemmProblem p = problem(w.X, d, w.WguT, d, Mp, 2 * ff, d, kr, kRowsAreM);
            if (split && bwd) launch_row_gemm(p, EpiSwigluForward<true, true>{w.fu, w.fv, w.a, w.a_lo, ff}, s);
            else if (split) launch_row_gemm(p, EpiSwigluForward<false, true>{nullptr, nullptr, w.a, w.a_lo, ff}, s);
            else if (bwd) launch_row_gemm(p, EpiSwigluForward<true>{w.fu, w.fv, w.a, nullptr, ff}, s);
            else launch_row_gemm(p, EpiSwigluForward<false>{nullptr, nullptr, w.a, nullptr, ff}, s);
        }
        if (!io.composed) {
            StageTimer t(ST_GEMM_DOWN, s);
            GemmProblem p = problem(w.a, ff, w.WdT, ff, Mp, d, ff, kr, kRowsAreM);
            if (split) {                                       // y = [a | a_lo] [Wd; Wd], kept as y + y_lo
                p.A2 = w.a_lo; p.B2 = w.WdT; p.K2 = ff;
                launch_row_gemm(p, EpiStoreBf16Split{w.y, w.y_lo, d, Mp}, s);
            } else {
                rc = launch_rows_bf16(p, w.y, w.parts, s);
                if (rc != PCM_OK) return rc;
            }
        }
        {
            StageTimer t(ST_GEMM_LOGITS_LOSS, s);
            const size_t n_z = (size_t)Mp * V;                         // z in fp32, as parts of a split reduction
            int n_parts;
            if (io.composed) {   // z = a W_do, W_do read as [K][rows]
                GemmProblem p = problem(w.a, ff, w.Wdo, V, Mp, V, ff, kr, kRowsAreM);
                n_parts = p.splits = pick_splits(Mp / kTileM, ff / kTileK);
                if (!w.parts.hold(n_parts * n_z)) return PCM_EWORKSPACE;
                launch_gemm<kRowsByK, kKByRows>(p, EpiStoreF32{w.parts.at, V, (int64_t)n_z, 0, nullptr, FinalPanel{}}, s);
            } else {
                GemmProblem p = problem(w.y, d, w.WoT, d, Mp, V, d, kr, kRowsAreM);
                if (split) { p.A2 = w.y_lo; p.B2 = w.WoT; p.K2 = d; }   // z = [y | y_lo] [Wo; Wo]
                n_parts = p.splits = pick_splits(Mp / kTileM, (p.K1 + p.K2) / kTileK);
                if (!w.parts.hold(n_parts * n_z)) return PCM_EWORKSPACE;
                launch_gemm(p, EpiStoreF32{w.parts.at, V, (int64_t)n_z, 0, nullptr, FinalPanel{}}, s);
            }
            loss_rows_bf16<<<(unsigned)(Mp / kLossRows), kLossThreads, 0, s>>>(LossRowsArgs{
                w.parts.at, n_parts, n_z, meta.token, meta.logp_old, meta.adv, io.n_kept, sh.max_chunks, sh.A, (int)row0, Mp,
                io.opt, bwd ? w.dz : nullptr, w.dz_extra, io.logp_out ? io.logp_out + row0 : nullptr, out,
                io.opt.chunk_ratio ? nullptr : w.live_count});
        }
        if (io.opt.chunk_ratio) {
            rc = launch_chunk_ratio(sh, io, meta, out, row0, Mp, s);
            if (rc != PCM_OK) return rc;
            if (bwd) {
                StageTimer t(ST_REDUCE, s);
                scale_rows_bf16<<<(unsigned)(Mp / kLossRows), kLossThreads, 0, s>>>(
                    ScaleRowsArgs{w.dz, io.opt.entropy_coef != 0.f ? w.dz_extra : nullptr, out.coef, meta.adv, out.clipped,
                                  io.opt.chunk_weight, io.n_kept, sh.max_chunks, sh.A, (int)row0, Mp, w.live_count});
            }
        }
        if (!bwd) continue;

        // Which rows the backward products run over, and where their row-indexed operands are: all live rows; or those with a
        // gradient, where row count and operands come from the plan that a launch leaves in device memory.
        const bool listed = w.plan != nullptr;
        const BackwardPlan& plan = w.plan_b;
        const int64_t rows_left = sh.rows_max() - row0;
        bf16* const dX = io.dX ? static_cast<bf16*>(io.dX) + row0 * d : nullptr;
        bf16* const du = listed ? w.du : w.fu;
        bf16* const dv = listed ? w.dv : w.fv;
        const KeptRows br = listed ? KeptRows{&w.plan->n_rows, Mp, 1, 0} : kr;
        const bf16* const* const src = listed ? reinterpret_cast<const bf16* const*>(w.plan->src) : nullptr;
        auto source = [&](int which) { return listed ? src + which : nullptr; };
        if (listed) {
            const LiveSources whole{{w.dz, w.y, w.a, w.X}}, rows{{w.dzc, w.yc, w.ac, w.Xc}};
            const int64_t both = grads ? 2 : 0;         // without weight gradients only dz is read by row of the list
            rc = launch_live_rows(sh, io, out.clipped, meta.adv, w.live_count, row0, Mp, whole, rows, {2 * V, both * d, both * ff, both * d},
                                  dX, rows_left < Mp ? rows_left : Mp, w.live_idx, w.plan, s);
            if (rc != PCM_OK) return rc;
        }
        PartsSums sums{};
        // dWg (+)= X^T du, dWu (+)= X^T dv
        GemmPairJob<kKByRows, kKByRows, EpiStoreF32> dWgu{problem(w.X, d, du, ff, d, ff, Mp, br, kRowsAreK), {du, dv}, {}, 0, 0};
        dWgu.p.A_sel = source(LiveSources::kX);
        // dX = du Wg^T + dv Wu^T
        GemmProblem pX = problem(du, ff, Wg, ff, Mp, d, ff, br, kRowsAreM);
        pX.A2 = dv; pX.B2 = Wu; pX.K2 = ff;
        const EpiScatterBf16 scatter_X{dX, d, w.live_idx};
        const EpiStoreBf16 store_X{dX, d, (int)(rows_left < Mp ? rows_left : Mp)};
        const EpiSwigluBackward<true> swiglu_listed{w.fu, w.fv, ff, w.live_idx, du, dv};
        const EpiSwigluBackward<false> swiglu{w.fu, w.fv, ff, nullptr, nullptr, nullptr};   // fu <- du, fv <- dv
        auto weights_apart = [&] {
            StageTimer t(ST_GEMM_DWG_DWU, s);
            launch_gemm<kKByRows, kKByRows>(dWgu.p, dWgu.epi[0], s);
            dWgu.p.B = dWgu.p.B2 = dv;
            launch_gemm<kKByRows, kKByRows>(dWgu.p, dWgu.epi[1], s);
        };
        auto rows_apart = [&] {
            StageTimer t(ST_GEMM_DX, s);
            if (listed) launch_row_gemm(pX, scatter_X, s);
            else launch_row_gemm(pX, store_X, s);
        };
        if (io.composed) {      // one panel: nothing to add to
            // da = dz W_do^T, and G = a^T dz [ff, V] over the kept rows, rounded to bf16 as the operand of two products below
            const GemmProblem pa = problem(w.dz, V, w.Wdo, V, Mp, ff, V, kr, kRowsAreM);
            const GemmJob<kRowsByK, kRowsByK, EpiSwigluBackward<false>> da{pa, swiglu, 0};
            if (grads) {
                GemmProblem p = problem(w.a, ff, w.dz, V, ff, V, Mp, kr, kRowsAreK);
                const size_t n = (size_t)ff * V;
                if (!plan.group[0]) {
                    rc = launch_reduction_bf16<kKByRows, kKByRows>(p, w.G, w.parts, ST_GEMM_DWD, s);
                    if (rc != PCM_OK) return rc;
                    StageTimer t(ST_GEMM_DA, s);
                    launch_row_gemm(pa, swiglu, s);
                } else if (plan.split_G == 1) {   // wide enough by itself (and wider than the parts that there is room for)
                    StageTimer t(ST_GEMM_DA, s);
                    launch_gemm_group(plan.level[0].kW, s, da, GemmJob<kKByRows, kKByRows, EpiStoreBf16>{p, EpiStoreBf16{w.G, V, ff}, 0});
                } else {
                    StageTimer t(ST_GEMM_DA, s);
                    p.splits = plan.split_G;
                    if (!w.parts.hold(p.splits * n)) return PCM_EWORKSPACE;
                    launch_gemm_group(plan.level[0].kW, s, da,
                                      GemmJob<kKByRows, kKByRows, EpiStoreF32>{p, EpiStoreF32{w.parts.at, V, (int64_t)n, 0, nullptr, FinalPanel{}}, 0});
                    launch_sum_bf16(w.parts.at, p.splits, n, w.G, LiveTiles{}, s);
                }
                for (int q = 0; q < 2; ++q)
                    dWgu.epi[q] = reduction_epilogue(dWgu.p, plan.split_gu, q ? io.dWu : io.dWg, q ? w.parts_u : w.parts_g, false, SumsqTarget{}, sums);
                GemmProblem po = problem(Wd, d, w.G, V, d, V, ff, all_rows, kRowsUnused);                        // dWo = Wd^T G
                const EpiStoreF32 eo = reduction_epilogue(po, plan.split_o, io.dWo, w.parts_o, false, SumsqTarget{}, sums);
                const GemmJob<kKByRows, kKByRows, EpiStoreF32> dWo{po, eo, 0};
                const GemmJob<kRowsByK, kRowsByK, EpiStoreF32> dWd{problem(w.G, V, Wo, V, ff, d, V, all_rows, kRowsUnused),   // dWd = G Wo^T
                                                                   EpiStoreF32{io.dWd, d, 0, 0, nullptr, FinalPanel{}}, 0};
                if (!plan.group[2]) {
                    weights_apart();
                    {
                        StageTimer t(ST_GEMM_DWD, s);
                        launch_gemm_group(plan.level[2].kW, s, dWo, dWd);
                    }
                    if (dX) rows_apart();
                } else {
                    StageTimer t(ST_GEMM_DX, s);
                    if (dX) launch_gemm_group(plan.level[2].kW, s, GemmJob<kRowsByK, kRowsByK, EpiStoreBf16>{pX, store_X, 0}, dWgu, dWo, dWd);
                    else launch_gemm_group(plan.level[2].kW, s, dWgu, dWo, dWd);
                }
            } else {
                {
                    StageTimer t(ST_GEMM_DA, s);
                    launch_row_gemm(pa, swiglu, s);
                }
                rows_apart();
            }
        } else {
            GemmProblem py = problem(w.dz, V, Wo, V, Mp, d, V, br, kRowsAreM);                                   // dy = dz Wo^T
            py.A_sel = source(LiveSources::kDz);
            GemmProblem po = problem(w.y, d, w.dz, V, d, V, Mp, br, kRowsAreK);                                  // dWo (+)= y^T dz
            po.A_sel = source(LiveSources::kY);
            po.B_sel = source(LiveSources::kDz);
            const GemmProblem pa = problem(w.dy, d, Wd, d, Mp, ff, d, br, kRowsAreM);                            // du, dv from da = dy Wd^T
            GemmProblem pd = problem(w.a, ff, w.dy, d, ff, d, Mp, br, kRowsAreK);                                // dWd (+)= a^T dy
            pd.A_sel = source(LiveSources::kA);
            const EpiStoreBf16 store_y{w.dy, d, Mp};
            if (!grads) {
                {
                    StageTimer t(ST_GEMM_DY, s);
                    launch_row_gemm(py, store_y, s);
                }
                {
                    StageTimer t(ST_GEMM_DA, s);
                    if (listed) launch_row_gemm(pa, swiglu_listed, s);
                    else launch_row_gemm(pa, swiglu, s);
                }
                rows_apart();
                continue;
            }
            const EpiStoreF32 eo = reduction_epilogue(po, plan.split_o, io.dWo, w.parts_o, !first, sq[3], sums);
            const EpiStoreF32 ed = reduction_epilogue(pd, plan.split_d, io.dWd, w.parts_d, !first, sq[2], sums);
            const GemmJob<kKByRows, kKByRows, EpiStoreF32> dWo{po, eo, 0}, dWd{pd, ed, 0};
            for (int q = 0; q < 2; ++q)
                dWgu.epi[q] = reduction_epilogue(dWgu.p, plan.split_gu, q ? io.dWu : io.dWg, q ? w.parts_u : w.parts_g, !first, sq[q], sums);
            {
                StageTimer t(ST_GEMM_DY, s);
                launch_gemm_group(plan.level[0].kW, s, dWo, GemmJob<kRowsByK, kRowsByK, EpiStoreBf16>{py, store_y, 0});
            }
            if (plan.group[1]) {
                StageTimer t(ST_GEMM_DA, s);
                if (listed) launch_gemm_group(plan.level[1].kW, s, GemmJob<kRowsByK, kRowsByK, EpiSwigluBackward<true>>{pa, swiglu_listed, 0}, dWd);
                else launch_gemm_group(plan.level[1].kW, s, GemmJob<kRowsByK, kRowsByK, EpiSwigluBackward<false>>{pa, swiglu, 0}, dWd);
            } else {
                {
                    StageTimer t(ST_GEMM_DWD, s);
                    launch_gemm<kKByRows, kKByRows>(dWd.p, dWd.epi, s);
                }
                StageTimer t(ST_GEMM_DA, s);
                if (listed) launch_row_gemm(pa, swiglu_listed, s);
                else launch_row_gemm(pa, swiglu, s);
            }
            if (plan.group[2]) {
                StageTimer t(ST_GEMM_DX, s);
                if (!dX) launch_gemm_group(plan.level[2].kW, s, dWgu);
                else if (listed) launch_gemm_group(plan.level[2].kW, s, GemmJob<kRowsByK, kRowsByK, EpiScatterBf16>{pX, scatter_X, 0}, dWgu);
                else launch_gemm_group(plan.level[2].kW, s, GemmJob<kRowsByK, kRowsByK, EpiStoreBf16>{pX, store_X, 0}, dWgu);
            } else {
                weights_apart();
                if (dX) rows_apart();
            }
        }
        if (grads && row0 + w.Rp < w.Mp) {      // the last panel's sums go with the loss
            rc = launch_finish(sh, io, w.out, sums, sq[0].final_panel, false, SumsqLists{}, s);
            if (rc != PCM_OK) return rc;
        } else {
            last_sums = sums;
            last_panel = sq[0].final_panel;
        }
    }
    SumsqLists lists{};
    if (want_sumsq)
        for (int q = 0; q < 4; ++q) { lists.parts[q] = w.sumsq[q]; lists.count[q] = w.sumsq_count[q]; }
    return launch_finish(sh, io, w.out, last_sums, last_panel, true, lists, s);
}

}  // namespace pcm
