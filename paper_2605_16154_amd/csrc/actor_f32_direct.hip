// The direct route of the fp32 actor step: operands as the caller gave them (gemm_direct.h), sums and results in fp32.
//
// One GEMM kernel template serves all products of the forward and backward pass; reductions over the row dimension (the weight
// gradients) are split across workgroups into partial products that a second kernel adds in slice order, so the results are the same
// from run to run (no atomics).  Row tiles beyond the kept count are skipped.
#include <algorithm>
#include <initializer_list>

#include "actor_f32.h"
#include "gemm_direct.h"

namespace pcm {
namespace {

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
            splits = std::max<int64_t>(1, std::min<int64_t>(splits, ceil_div(K, 4 * kDirectStep)));
        }
        const int k_per = ceil_div(ceil_div(K, (int)splits), kDirectStep) * kDirectStep;
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
    if (t.kI == 2 && vec) gemm_direct<2, 2, kLayA, kLayB, kSecond, true><<<grid, kDirectThreads, 0, s>>>(p, epi);
    else if (t.kI == 2) gemm_direct<2, 2, kLayA, kLayB, kSecond, false><<<grid, kDirectThreads, 0, s>>>(p, epi);
    else if (vec) gemm_direct<1, kSmallJ, kLayA, kLayB, kSecond, true><<<grid, kDirectThreads, 0, s>>>(p, epi);
    else gemm_direct<1, kSmallJ, kLayA, kLayB, kSecond, false><<<grid, kDirectThreads, 0, s>>>(p, epi);
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

size_t direct_workspace_bytes(const ActorShape& sh, bool bwd) {
    return carve(nullptr, sh, bwd).bytes;
}

int direct_run(const ActorShape& sh, const ActorIO& io, void* ws, hipStream_t s) {
    const bool bwd = io.want_grads() || io.dX != nullptr;
    F32Workspace w = carve(ws, sh, bwd);
    const int M = (int)sh.rows_max();
    const int d = sh.d, ff = sh.ff, V = sh.V;
    const float* Wg = static_cast<const float*>(io.Wg);
    const float* Wu = static_cast<const float*>(io.Wu);
    const float* Wd = static_cast<const float*>(io.Wd);
    const float* Wo = static_cast<const float*>(io.Wo);
    const BatchRows rows{io.n_kept, sh.max_chunks, sh.A}, none{nullptr, 0, 0};

    int rc = launch_gather_f32(sh, io, w.X, M, w.meta, s);
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
        LossArgs loss{};
        loss.z = w.z;
        loss.V = loss.ld = V;
        loss.extra = w.z_extra;
        loss.in_place = bwd;
        loss.meta = w.meta;
        loss.n_kept = io.n_kept;
        loss.max_chunks = sh.max_chunks;
        loss.A = sh.A;
        loss.rows = M;
        loss.row_tile = kDirectRowTile;
        loss.opt = io.opt;
        loss.logp_out = io.logp_out;
        loss.out = w.out;
        launch_loss_rows(loss, s);
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
            sums.add(w.y, 2, (size_t)M * d, (size_t)(w.dy - w.y), static_cast<float*>(io.dX), false, nullptr, d, kDirectRowTile);
        }
    }
    return launch_finish(sh, io, w.out, sums, FinalPanel{}, true, SumsqLists{}, s);
}

}  // namespace pcm
