// fp32 path of the masked GRPO actor step (Eq. 11): fp32 operands, sums and results.
//
// Forward: products on the fp32 matrix instructions (gemm_floats.h), every sum one chain in the order of k, so that loss and
// log-probabilities have the bits of the definition's order of additions whatever the tile.
//
// Backward: products on the bf16 matrix cores.  Every operand is held as three bf16 matrices whose sum it is exactly (thirds.h),
// and a product of two is six products of such parts (gemm_thirds.h; the three left out come to less than 2^-24 of the whole, the
// rounding of one fp32 operation).  The matrix cores round a sum a few times per 32 products, where multiply-adds in fp32 do so 32
// times, and sums over many rows are in chains that are added up.  They do 16 times the multiply-adds of the fp32 ones: six
// products take 3/8 of the time at the same share of their rates.
// Measured against fp32 matrix instructions throughout, steps: 10,752 rows of 1024 -> 2816 -> 1024 -> 256, a quarter of them not kept,
// 3.74 -> 2.54 ms; 5376 of 256 -> 1024 -> 256 -> 256 362 -> 259 to 287 us, by the box; 360 of 473 -> 333 -> 473 -> 512 185 -> 124, 1440
// of 619 -> 1302 -> 619 -> 256 413 -> 201, 8960 of 103 -> 149 -> 103 -> 256, composed, where most of the padded tiles is padding,
// 171 -> 149; faster at 16 of 16 sizes, 1.15 to 2.06 times.  Loss, log-probabilities and statistics have the same bits; errors of the
// gradients against 64 bits, root mean square over six inputs each: dX 4.85e-6 -> 4.74e-6 and 2.78e-6 -> 2.71e-6 at the first two, no
// larger at any of ten sizes; with sums of one sign dWg 1.24e-7 -> 1.02e-7 at the second, no larger for any gradient of 14 sizes.
// (The forward products as thirds too: 2.08 ms and 232 us, and a third of the error; but the loss may be a sum of terms of both
// signs that nearly cancel, and any other rounding of the logits moves it by more than a part in 10^4 then.)
//
// Who reads a matrix only as an operand gets its operand form alone: X, a and y as floats in blocks and as thirds, dz, dy, du and
// dv as thirds.  Wg and Wu are one matrix with columns in blocks of 32 of each in turn, so that a wavefront holds a gate column
// and its up column, and so are u and v, and du and dv.  Operands are padded with zeros to whole blocks in the workspace, so any
// size runs; results are written as far as they reach.
//
// Heads and batches for which that does not pay, and calls whose workspace is too short for it, take their matrices as they are
// (actor_f32_direct.hip; uses_blocks).
//
// Backward products of one dependency level share a launch and long reductions are split into parts that a later launch adds up
// in order (no atomics), as in the bf16 path.  Row tiles beyond the kept count are skipped.
#include <algorithm>

#include "actor_f32.h"
#include "epilogues_f32.h"

namespace pcm {
namespace {

constexpr int kThreads = 256;
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

// (see LossArgs; kQ * 64 columns at most: with the checks of 1024, 43,008 rows of 256 take 4 us longer, 2688 of 512 0.9)
template <int kQ, bool kInPlace>
__global__ __launch_bounds__(kThreads) void loss_rows(LossArgs p) {
    const int lane = threadIdx.x % kWave;
    const int64_t r = (int64_t)blockIdx.x * (kThreads / kWave) + threadIdx.x / kWave;
    const int64_t rows = live_rows(p.n_kept, p.max_chunks, p.A);
    if (r >= p.rows || r >= (rows + p.row_tile - 1) / p.row_tile * p.row_tile) return;     // later rows: skipped tiles, read by nothing
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
    if (!kInPlace && p.dz.p == nullptr) return;
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
        } else if (kInPlace) {
            zr[j] = pg + ent;
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

// (Where all of a step stays in the caches, what the next one reads first is better not the place that was written last: 2688 rows of
// 93 -> 250 with du and dv of 9 MB 98.4 us in the place of X, a and y, 96.4 apart; 5376 of 256 -> 1024, 66 MB, 272.8 and 274.3.)
constexpr size_t kOverlayBytes = (size_t)32 << 20;

F32Workspace carve(void* ws, const ActorShape& sh, bool bwd, const LossOptions& opt, bool composed) {
    Carver c(ws);
    F32Workspace w{};
    const int64_t Mp = w.Mp = tiles256(sh.rows_max());
    const auto thirds = [&](int64_t rows, int64_t columns) { return Thirds{c.take<bf16>((size_t)(3 * padded(rows) * padded(columns))), padded(columns)}; };
    const auto floats = [&](int64_t rows, int64_t columns) { return FloatBlocks{c.take<float>((size_t)(padded(rows) * padded(columns))), padded(columns)}; };
    const F32Plan& plan = w.plan = plan_step(sh, Mp, composed);
    const int64_t ffp = padded(sh.ff), Vp = padded(sh.V);
    const size_t M = (size_t)sh.rows_max(), d = sh.d, ff = sh.ff, V = sh.V;
    // du and dv come when X, a and y as floats are no longer needed, and lie in their place if they are large
    w.X = floats(Mp, sh.d);
    w.a = floats(Mp, sh.ff);
    if (!composed) w.y = floats(Mp, sh.d);
    if (bwd) {
        const size_t bytes = (size_t)Mp * 2 * ffp * 3 * sizeof(bf16);
        if (bytes > kOverlayBytes) {
            w.duv = Thirds{reinterpret_cast<bf16*>(w.X.p), 2 * ffp};
            if (bytes > c.used()) c.take<uint8_t>(bytes - c.used());
        } else {
            w.duv = thirds(Mp, 2 * ffp);
        }
    }
    w.WguT = floats(2 * ffp, sh.d);
    w.WdT = composed ? floats(sh.ff, sh.d) : floats(sh.d, sh.ff);
    w.WoT = floats(sh.V, sh.d);
    if (composed) w.WdoT = floats(sh.V, sh.ff);
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
    if (!bwd) {
        w.bytes = c.used();
        return w;
    }
    w.uv = c.take<float>((size_t)Mp * 2 * ffp);
    w.Wgu = thirds(sh.d, 2 * ffp);
    w.Wd = thirds(sh.ff, sh.d);
    w.Wo = thirds(sh.d, sh.V);
    w.X3 = thirds(Mp, sh.d);
    w.a3 = thirds(Mp, sh.ff);
    w.dz = thirds(Mp, sh.V);
    if (composed) {
        w.WdoT3 = thirds(sh.V, sh.ff);
        w.G = thirds(sh.ff, sh.V);
        w.parts_G = c.take<float>((size_t)plan.G * ffp * Vp);
    } else {
        w.y3 = thirds(Mp, sh.d);
        w.dy = thirds(Mp, sh.d);
    }
    const size_t o = plan.dWo, dd = plan.dWd, gu = plan.dWgu;
    if (o > 1) w.parts_o = c.take<float>(o * d * V);
    if (dd > 1) w.parts_d = c.take<float>(dd * ff * d);
    if (gu > 1) w.parts_g = c.take<float>(2 * gu * d * ff);
    w.parts_u = w.parts_g + gu * d * ff;
    if (plan.dX > 1) w.dX_part = c.take<float>(M * d);
    if (opt.chunk_ratio) w.z_extra = c.take<float>(M * V);
    w.bytes = c.used();
    return w;
}

// Whether operands go into blocks first, or a step takes them as they are (the direct route).  Blocks cost a pass over the weights
// before the first product, padding to 128 and, for the composed head with gradients, a launch more; what they give grows with rows x
// head.  Measured, direct / blocks, us a call (f: forward, s: step, c: composed; V = 256), by the lines below:
//   few rows, wide head
//     4096 -> 11008  56 rows s 1695 / 1725, c f 830 / 937, c s 1840 / 1951 (f 877 / 820); 168 rows s 2216 / 1793, c f 1072 / 940
//     3072 -> 8192   56 rows s 1241 / 1068, c f 580 / 539, c s 1290 / 1234
//   many rows, head narrower than a block: the products wait for memory, and what is padded to 128 is twice as long
//     64 -> 300      43,008 rows f 157 / 171, s 393 / 531, c s 477 / 560; 10,752 rows f 64.6 / 65.1, s 170 / 160, c s 192 / 179
//     64 -> 1024     43,008 rows f 321 / 312, s 846 / 1017; c f 432 / 374, c s 1173 / 1151; 10,752 rows f 107 / 105, s 282 / 307
//     1024 -> 64     43,008 rows f 493 / 549, s 1380 / 1393, c s 724 / 808; 10,752 rows f 170 / 178, s 436 / 404, c s 276 / 276
//     128 -> 128     43,008 rows f 147.6 / 146.8, s 355 / 365, c s 316 / 342; 86,016 rows f 264 / 259, s 662 / 638, c s 571 / 578
//   small heads
//     64 -> 64       56 rows f 26.3 / 28.2, s 62.5 / 71.6; 10,752 rows f 49.4 / 54.6, s 116.5 / 116.8, c s 117 / 134
//     64 -> 128      2688 rows f 33.2 / 32.5, s 84.7 / 89.4, c s 98.9 / 107.9; 5376 rows f 39.7 / 38.0, s 101.4 / 96.6, c s 110 / 118;
//                    21,504 rows f 70 / 77, s 184 / 162, c s 189 / 178
//     128 -> 128     1344 rows f 35.5 / 34.2, s 86.9 / 86.5, c s 93.6 / 101.7; 2688 rows c s 105.7 / 110.9; 5376 rows c s 118 / 120
//     100 -> 300     1344 rows f 41.8 / 38.3, s 106 / 97, c s 115 / 116; 2688 rows c s 125.0 / 124.7
//     256 -> 256     56 rows c s 95 / 99, 168 rows 104.8 / 103.8
// Elsewhere blocks are ahead, up to 1.8 times.
bool uses_blocks(const ActorShape& sh, bool bwd, bool composed) {
    const int64_t rows = sh.rows_max(), head = (int64_t)sh.d * sh.ff, M = 1 << 20;
    if (rows > kDirectRowsMax) return true;
    if (rows <= 64 && head > 32 * M && (bwd || composed)) return false;
    if (std::min(sh.d, sh.ff) <= 64 && rows > 32768 && (!composed || sh.ff <= 512)) return false;
    if (head <= 4 * 1024) return false;
    if (head <= 8 * 1024) return bwd && rows * head > (composed ? 44 : 22) * M;
    return !(composed && bwd && head <= 36 * 1024 && rows * head <= 44 * M);
}

}  // namespace

void launch_loss_rows(const LossArgs& p, hipStream_t s) {
    const unsigned grid = (unsigned)ceil_div(p.rows, kThreads / kWave);
    const auto launch = [&](auto columns) {
        if (p.in_place) loss_rows<decltype(columns)::value, true><<<grid, kThreads, 0, s>>>(p);
        else loss_rows<decltype(columns)::value, false><<<grid, kThreads, 0, s>>>(p);
    };
    if (p.ld <= 4 * kWave) launch(Index<4>{});
    else if (p.ld <= 8 * kWave) launch(Index<8>{});
    else launch(Index<kMaxV / kWave>{});
}

size_t actor_f32_least_bytes(const ActorShape& sh, bool bwd) { return direct_workspace_bytes(sh, bwd); }
size_t actor_f32_workspace_bytes(const ActorShape& sh, bool bwd, const LossOptions& opt, bool composed) {
    const size_t least = direct_workspace_bytes(sh, bwd);      // enough for any other options of the shape, too
    return uses_blocks(sh, bwd, composed) ? std::max(least, carve(nullptr, sh, bwd, opt, composed).bytes) : least;
}

int actor_f32_run(const ActorShape& sh, const ActorIO& io, void* ws, size_t ws_bytes, hipStream_t s) {
    const bool grads = io.want_grads(), bwd = grads || io.dX != nullptr;
    if (!uses_blocks(sh, bwd, io.composed)) return direct_run(sh, io, ws, s);
    const F32Workspace w = carve(ws, sh, bwd, io.opt, io.composed);
    if (w.bytes > ws_bytes) return sh.rows_max() > kDirectRowsMax ? (int)PCM_EWORKSPACE : direct_run(sh, io, ws, s);
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
        launch_loss_rows(LossArgs{w.z, V, Vp, w.z_extra, w.dz, false, w.meta, io.n_kept, sh.max_chunks, sh.A, Mp, kTileM, io.opt, io.logp_out, w.out}, s);
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
                launch_products(s, job<kKByRows, kKByRows>(product(w.a3, w.dz, ffp, Vp, Mp, kRowsAreK, plan.G), EpiFloatsInChains{{w.parts_G, Vp, (int64_t)n, ffp, Vp}}));
                sum_parts_thirds<<<(unsigned)std::min<size_t>((n / 4 + kThreads - 1) / kThreads, 2048), kThreads, 0, s>>>(w.parts_G, plan.G, n, w.G);
                const auto dWd = job<kRowsByK, kRowsByK>(product(w.G, w.Wo, ff, d, V, kRowsUnused), EpiFloatsInChains{{io.dWd, d, 0, ff, d}});   // G Wo^T
                const int o = plan.dWo;
                const auto dWo = job<kKByRows, kKByRows>(product(w.Wd, w.G, d, V, ff, kRowsUnused, o),                                     // Wd^T G
                                                         EpiFloatsInChains{floats(o, w.parts_o, io.dWo, d, V)});
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
        const auto dX = job<kRowsByK, kRowsByK>(product(w.duv, w.Wgu, Mp, d, 2 * ffp, kRowsAreM, x), EpiFloats{out_X, d, x > 1 ? w.dX_part - out_X : 0, M, d});
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
