// The fp32 path of the actor step: what its two routes share (internal header).
#pragma once

#include "thirds.h"

namespace pcm {

// One wavefront per row, a column per lane and 64: log-softmax at the target bin, entropy, ratio, clipped surrogate, and dz =
// coef * (onehot - softmax) + entropy part, as thirds or in place of z.  With a per-chunk ratio the factor is not known yet:
// z <- onehot - softmax and the entropy part goes to `extra`; a launch behind it makes dz of them once the chunk ratios are known.
constexpr int kMaxV = 1024;
struct LossArgs {
    float* z;                // [rows, ld]
    int V, ld;
    float* extra;            // [rows, V]
    Thirds dz;               // p null: in place of z (in_place), or no backward pass
    bool in_place;
    RowMeta meta;
    const int32_t* n_kept;
    int max_chunks, A;
    int rows, row_tile;      // rows of z; those behind the live rows' last tile of row_tile are skipped, nothing reads them
    LossOptions opt;
    float* logp_out;
    RowOut out;
};
void launch_loss_rows(const LossArgs& p, hipStream_t s);

// The direct route (actor_f32_direct.hip).  A launch has a row of workgroups per 64 rows, and at most 65,535 of them.
constexpr int64_t kDirectRowsMax = 65535 * 64;
size_t direct_workspace_bytes(const ActorShape& sh, bool bwd);
int direct_run(const ActorShape& sh, const ActorIO& io, void* ws, hipStream_t s);

}  // namespace pcm
