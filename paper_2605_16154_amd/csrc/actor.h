// Internal declarations for the masked GRPO actor step (Eq. 11): pieces shared by the fp32 and
// bf16 paths.  Not part of the C boundary.
#pragma once

#include <hip/hip_bf16.h>

#include "common.h"

namespace pcm {

using bf16 = __hip_bfloat16;

// Host scalars of one actor-step call.
struct ActorShape {
    int max_chunks;   // capacity of kept_idx (kept chunks at most)
    int T, N, A;      // trajectories, chunk slots per trajectory, tokens per chunk
    int d, ff, V;     // head sizes
    int64_t rows_max() const { return (int64_t)max_chunks * A; }
};

// How the objective is assembled from the rows (Eq. 11 plus the training details of App. D).
struct LossOptions {
    float eps_low, eps_high;     // clip thresholds
    float loss_scale;            // multiplies the summed objective
    float entropy_coef;          // subtracts entropy_coef * scale * sum of row entropies
    int token_mean;              // scale = loss_scale / (kept rows) instead of loss_scale
    int chunk_ratio;             // one ratio (and one clipped term) per chunk instead of per token
    const float* chunk_weight;   // device [max_chunks] or null: multiplies the terms of a chunk
    int panel_rows;              // bf16 path: target height of the row panels (0 = the library's choice)
    const void* packed_weights;  // bf16 path: operand layouts written by pcm_pack_head_weights, or null
    int dense_backward;          // bf16 path: backward products over all kept rows, also those without a gradient
    double* grad_sumsq_out;      // bf16 path: device [1] or null: sum of the squares of all four weight gradients
};

struct ActorIO {
    const void* hidden;
    const uint8_t* tokens;
    const float* logp_old;
    const float* adv;
    const int32_t* kept_idx;
    const int32_t* n_kept;
    const void *Wg, *Wu, *Wd, *Wo;
    LossOptions opt;
    float* loss_out;
    float* logp_out;
    float *dWg, *dWu, *dWd, *dWo;
    void* dX;
    float* stats_out;
    int n_stats;      // 4, or 5 when the mean row entropy is reported too
    bool composed;    // down and logit projection applied as one matrix Wd Wo (PCM_HEAD_COMPOSED)
    bool want_grads() const { return dWg != nullptr; }
};

// Per-row quantities produced by the gather and consumed by the loss stage.
struct RowMeta {
    uint8_t* token;    // [rows_pad] target bin (clamped to V-1)
    float* logp_old;   // [rows_pad]
    float* adv;        // [rows_pad] advantage of the row's trajectory; 0 from the last live row to the end of its tile of 256
};

// Per-row results of the loss stage, reduced in a fixed order afterwards.  Like the arrays above they are written up to the end
// of the last live row's tile; what lies behind it is neither written nor read.
struct RowOut {
    float* term;       // [rows_pad] min(rho A, clip(rho) A); 0 behind the last live row
    float* ratio;      // [rows_pad]
    float* dlogp;      // [rows_pad] logp_old - logp
    uint8_t* clipped;  // [rows_pad] 1 if the row's gradient is cut by the clip
    float* entropy;    // [rows_pad] entropy of the row's distribution over the V bins
    float* coef;       // [rows_pad] per-chunk ratio only: factor of (onehot - softmax) in dz
};

// gather.hip ---------------------------------------------------------------------------------
// Weights to be copied transposed: dst[map(c), r] = src[r, c], [R, C] bf16 row-major, R and C multiples of 64.
enum PackMode : int { kPackNone = 0, kPackGate = 1, kPackUp = 2 };   // map: identity, or gate and up in blocks of 64 in turn
struct TransposeJob {
    const bf16* src;
    bf16* dst;
    int R, C, mode;
};
struct TransposeList {
    static constexpr int kMax = 4;
    TransposeJob job[kMax];
    int first[kMax];      // workgroup of each one's first tile
    int n, blocks;
    void add(const bf16* src, int R, int C, bf16* dst, int mode) {
        job[n] = TransposeJob{src, dst, R, C, mode};
        first[n++] = blocks;
        blocks += R / 64 * (C / 64);
    }
};
// A launch of nothing but transposes; stream: non-temporal stores.
void launch_transposes(const TransposeList& list, bool stream, hipStream_t s);

// What the copy of the kept chunks' rows reads and writes, in units of Vec.
template <typename Vec>
struct GatherArgs {
    const Vec* hidden;
    const uint8_t* tokens;
    const float *logp_old, *adv;
    const int32_t *kept_idx, *n_kept;
    int max_chunks, T, N, A, V, vec_per_row;
    int64_t row_offset, rows_pad;   // rows are those of a panel that starts at batch row row_offset;
    Vec* X;                         // X and the metadata arrays are the panel's
    RowMeta meta;
};
// Copies the kept chunks' hidden rows into X [rows_pad, d] (rows from n_kept*A to the end of
// their tile of 256 are zero-filled, later ones left as they are: nothing reads them) and fills the row metadata (bf16).
// With row_offset > 0 the rows are those of a panel of the batch that starts at that row: X and the metadata
// arrays are the panel's own, `rows_pad` its height.  The same holds for the two per-chunk-ratio launches below
// (row_offset a multiple of A, so no chunk straddles two panels).
// In the same launch: the transposes of `layouts`, and zeros in zero[0 .. n_zero).
[[nodiscard]] int launch_gather(const ActorShape& sh, const ActorIO& io, void* X, int64_t row_offset, int64_t rows_pad,
                  RowMeta meta, const TransposeList& layouts, double* zero, int n_zero, hipStream_t s);

// The same of fp32 rows, as they are, of the whole batch.
[[nodiscard]] int launch_gather_f32(const ActorShape& sh, const ActorIO& io, float* X, int64_t rows_pad, RowMeta meta, hipStream_t s);

// Partial sums of squares of the four weight gradients, left by the launches that wrote their final values.
struct SumsqLists {
    const double* parts[4];
    int count[4];
};
// Sums of partial products that split reductions left: out = (add: out +) parts[0] + parts[1] + .. in that order (fp32, n
// floats, parts `stride` floats apart).  With live_row > 0 it is one over the rows of the batch, live_row floats each, the parts of which end
// with the last live one's tile of live_tile rows; behind it `out` is left as it is if added to, and zero otherwise.  With sumsq, on the final panel every workgroup also leaves the sum of the squares of what it wrote in
// sumsq[its number within the job].
struct PartsSum {
    const float* parts;
    int n_parts, add;
    size_t n, stride;
    float* out;
    double* sumsq;
    int live_row, live_tile;
    int first, blocks, threads, vec;   // workgroups, their threads that take part; vec: 16-byte accesses
};
struct PartsSums {
    static constexpr int kMax = 5, kBlocksMax = 2048;
    PartsSum job[kMax];
    int n, blocks;
    static int blocks_for(size_t n_floats, int n_parts);      // workgroups of a sum at most
    void add(const float* parts, int n_parts, size_t n_floats, size_t stride, float* out, bool add_to = false, double* sumsq = nullptr,
             int live_row = 0, int live_tile = 256);
};
// What a step does behind its last product, in one launch: sums of parts, and if asked for (with_loss) the per-row loss terms
// and statistics of the whole batch, in a fixed order (one workgroup, fp64 accumulators).  With lists the partial sums of
// squares of the weight gradients are added up behind it, into io.opt.grad_sumsq_out.
struct FinalPanel;
[[nodiscard]] int launch_finish(const ActorShape& sh, const ActorIO& io, RowOut out, const PartsSums& sums, const FinalPanel& panel, bool with_loss,
                  const SumsqLists& lists, hipStream_t s);

// Per-chunk ratio: from the per-row dlogp, one ratio, one clipped term and one dz factor per kept chunk
// (written to every row of the chunk; the term only to its first row).
[[nodiscard]] int launch_chunk_ratio(const ActorShape& sh, const ActorIO& io, RowMeta meta, RowOut out, int64_t row_offset,
                       int64_t rows_pad, hipStream_t s);

// fp32 path, direct route: dz[r, :] = coef[r] * dz[r, :] (+ extra[r, :] if extra is given) for the live rows r (V columns each).
[[nodiscard]] int launch_scale_rows_f32(const ActorShape& sh, const ActorIO& io, float* dz, const float* extra, const float* coef,
                          int64_t rows, hipStream_t s);

// Backward pass over the rows that carry a gradient only (bf16 path).  A kernel lists the panel's rows whose factor
// in dz is non-zero and writes, to device memory, what the backward products then read: their row count and which
// buffers hold their row-indexed operands (the panel's own, or copies of the listed rows).
struct LiveSources {
    static constexpr int kCount = 4;
    enum : int { kDz = 0, kY = 1, kA = 2, kX = 3 };
    const void* p[kCount];
};
struct LivePlan {
    const void* src[LiveSources::kCount];
    int32_t n_rows;    // rows of the backward products
    int32_t listed;    // 1: the products run over the listed rows (operands copied), 0: over all live rows
};
// A row carries a gradient when the clip does not cut it (RowOut::clipped) and its advantage and chunk weight are
// non-zero; clipped and adv are the panel's parts of those arrays, counts the rows with a gradient in each of the panel's
// blocks of kListBlock rows (up to the last live one).  Writes the plan, the list idx and, when the plan says listed, the
// listed rows of the four sources (rows of row_bytes, a multiple of 16; 0: not wanted) with zero rows up to the end of the
// last row tile.  Rows of dX (or null; rows_in_dX rows exist) that the listed products do not write are cleared.
constexpr int kListBlock = 16;
[[nodiscard]] int launch_live_rows(const ActorShape& sh, const ActorIO& io, const uint8_t* clipped, const float* adv, const int32_t* counts,
                     int64_t row_offset, int64_t rows_pad, const LiveSources& whole, const LiveSources& listed,
                     const int64_t (&row_bytes)[LiveSources::kCount], void* dX, int64_t rows_in_dX, int32_t* idx, LivePlan* plan,
                     hipStream_t s);

// Number of live rows from the device-side kept count.
__device__ inline int64_t live_rows(const int32_t* n_kept, int max_chunks, int A) {
    int nk = *n_kept;
    nk = nk < 0 ? 0 : (nk > max_chunks ? max_chunks : nk);
    return (int64_t)nk * A;
}
// Factor in front of the summed objective.
__device__ inline float objective_scale(const LossOptions& o, int64_t rows_live) {
    if (!o.token_mean) return o.loss_scale;
    return rows_live > 0 ? o.loss_scale / (float)rows_live : 0.f;
}

// Whether a row panel [row_begin, row_end) of a batch holds the batch's last live rows (panel 0 if there are none):
// the weight gradients that panel leaves are the final ones.
struct FinalPanel {
    const int32_t* n_kept;
    int max_chunks, A;
    int64_t row_begin, row_end;
    __device__ bool operator()() const {
        const int64_t rows = live_rows(n_kept, max_chunks, A);
        return rows <= row_end && (rows > row_begin || row_begin == 0);
    }
};

// Clipped-surrogate math of one ratio (device), shared by both paths and both ratio levels.
// term = weight * min(rho A, clip(rho) A); coef is the factor c in dz = c * (onehot - softmax):
// c = -scale * weight * rho * A where the gradient flows, else 0.
struct LossRow {
    float term, ratio, dlogp, coef;
    uint8_t clipped;
};
__device__ inline LossRow loss_from_ratio(float ratio, float adv, float weight, const LossOptions& o, float scale) {
    LossRow r;
    r.dlogp = 0.f;
    r.ratio = ratio;
    const float lo = 1.f - o.eps_low, hi = 1.f + o.eps_high;
    const float clipped_ratio = fminf(fmaxf(ratio, lo), hi);
    r.term = weight * fminf(ratio * adv, clipped_ratio * adv);
    const bool flows = (adv >= 0.f && ratio <= hi) || (adv < 0.f && ratio >= lo);
    r.clipped = flows ? 0 : 1;
    r.coef = flows ? -scale * weight * ratio * adv : 0.f;
    return r;
}
__device__ inline LossRow loss_row(float logp, float logp_old, float adv, float weight, const LossOptions& o,
                                   float scale) {
    LossRow r = loss_from_ratio(expf(logp - logp_old), adv, weight, o, scale);
    r.dlogp = logp_old - logp;
    return r;
}

// actor_f32.hip / actor_bf16.hip ---------------------------------------------------------------
// fp32: bytes with which a call is fastest, and those that are enough for any call of the shape.
size_t actor_f32_workspace_bytes(const ActorShape& sh, bool bwd, const LossOptions& opt, bool composed);
size_t actor_f32_least_bytes(const ActorShape& sh, bool bwd);
int actor_f32_run(const ActorShape& sh, const ActorIO& io, void* ws, size_t ws_bytes, hipStream_t s);
size_t actor_bf16_workspace_bytes(const ActorShape& sh, bool want_grads, const LossOptions& opt, bool composed);
int actor_bf16_run(const ActorShape& sh, const ActorIO& io, void* ws, hipStream_t s);
size_t packed_head_bytes(int d, int ff, int V);
int pack_head_weights(const void* Wg, const void* Wu, const void* Wd, const void* Wo, int d, int ff, int V, void* packed,
                      hipStream_t s);

}  // namespace pcm
