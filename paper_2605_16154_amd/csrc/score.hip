// pcm_score_phases: group-relative advantages (Eq. 1) and the batch phase score C_c (Eq. 5).
//
// Three routes on the caller's stream, with the same results bit for bit (the rules and what they measured stand at is_small,
// table_slices and fuses_tail):
//   small         one launch of one workgroup: all sums in LDS, pair scores and mean behind them
//   tables        two launches: a table of sums per trajectory or slice of one; tables to pair scores, last workgroup to mean
//   accumulators  two launches, four where the work behind the accumulation is long:
//     prepare     zero the integer accumulators and the arrival counters; one thread per trajectory writes
//                 advantage/active
//     accumulate  streaming pass over the action tensor: every workgroup owns a slice of one
//                 trajectory's chunks, keeps per-phase integer sums in LDS and adds the
//                 phases it met to the group's accumulators with 64-bit global atomics.  The last workgroup of a group
//                 to arrive forms the group's pair scores (difference of pooled means, squared terms in parallel, added
//                 in index order by one lane per phase, square root); the last group to arrive forms the mean of the pair
//                 scores over contributing groups, one lane per phase.  Nobody waits for anybody: a workgroup that is not
//                 the last one leaves.
//     pairs, mean the same two steps as launches of their own: a wavefront per (group, phase), then one workgroup
//
// The action pass of large batches is bandwidth-bound (224 B per chunk plus one phase byte); everything after it
// touches a few KB.  Integer accumulation makes the sums independent of slice and arrival order,
// which is what lets the sampler downstream be reproduced bit for bit.
//
// This file must be compiled without floating-point contraction: the fp64 tail is specified as
// separate multiplies and adds.
#include <algorithm>
#include <mutex>

#include "common.h"

#pragma clang fp contract(off)

namespace pcm {
namespace {

constexpr int kThreads = 256;
// LDS for sums, squared terms and pair scores: the 64 KB that a workgroup may take by default, less the word of arrive_last
// and the counts of the mean
constexpr size_t kLdsMax = 64 * 1024 - (PCM_MAX_PHASES + 4) * sizeof(int);
constexpr float kActionScale = 16777216.0f;                 // 2^24
constexpr double kActionUnscale = 1.0 / 16777216.0;         // 2^-24

using ull = unsigned long long;

struct ScoreWorkspace {
    ull* sums;            // [n_groups][2][K][A] integer sums of rint(a * 2^24); outcome 1 = success
    int* counts;          // [n_groups][2][K] chunks pooled
    double* pair;         // [n_groups][K] per-(group, phase) score, negative if the pair is skipped; until the group's
                          // scores are written, the first word of its row counts the group's workgroups that are done
    int* groups_done;     // groups whose pair scores are written
    size_t zero_words;    // 32-bit words to clear at the start (everything up to groups_done is contiguous)
    size_t bytes;
};

ScoreWorkspace carve(void* ws, int n_groups, int A, int K) {
    Carver c(ws);
    ScoreWorkspace w;
    const size_t n_sum = (size_t)n_groups * 2 * K * A;
    const size_t n_cnt = (size_t)n_groups * 2 * K;
    w.sums = c.take<ull>(n_sum);
    w.counts = c.take<int>(n_cnt);
    w.pair = c.take<double>((size_t)n_groups * K);
    const size_t after_pairs = c.used();
    w.groups_done = reinterpret_cast<int*>(c.take<uint8_t>((size_t)n_groups * K));   // one int is used of it
    w.zero_words = (after_pairs + sizeof(int)) / 4;
    w.bytes = c.used();
    return w;
}

__global__ __launch_bounds__(kThreads) void score_prepare(uint32_t* zero, size_t zero_words,
                                                          const uint8_t* __restrict__ reward, int T,
                                                          int G, double adv_eps, float* adv_out,
                                                          uint8_t* active_out) {
    const size_t gid = (size_t)blockIdx.x * kThreads + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * kThreads;
    for (size_t w = gid; w < zero_words; w += stride) zero[w] = 0u;
    for (size_t i = gid; i < (size_t)T; i += stride) {
        const int g = (int)(i / G);
        int s = 0;
        for (int r0 = 0; r0 < G; r0 += 8)             // eight loads under way together
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const uint8_t x = reward[(size_t)g * G + min(r0 + u, G - 1)];
                s += r0 + u < G && x != 0;
            }
        float a = 0.f;
        uint8_t act = 0;
        if (s != 0 && s != G) {
            const double mu = (double)s / (double)G;
            const double sigma = sqrt(mu * (1.0 - mu));
            const double r = reward[i] != 0 ? 1.0 : 0.0;
            a = (float)((r - mu) / (sigma + adv_eps));
            act = 1;
        }
        if (adv_out) adv_out[i] = a;
        if (active_out) active_out[i] = act;
    }
}

// rint(a 2^24) as a double, and sums of up to kExactRun of them, are exact while |a| <= 2^20: they stay below 2^53.  Four
// instructions a value where the conversion to a 64-bit integer and its addition take fourteen: the small
// route at 16 trajectories of 32 chunks of 56 values 10.8 -> 7.6 us, the tables of 512 trajectories of up to
// 256 chunks 9.3 -> 8.7, of 256 of up to 128 6.4 -> 6.1 us.
__device__ inline double to_fixed(float a) { return (double)rintf(a * kActionScale); }
constexpr int kExactRun = 256;
// Values beyond that, infinities and NaN among them, are converted one by one and added as integers, so that they leave the
// other chunks of a run as they are and the sums do not depend on the route.
constexpr float kExactMax = 1048576.0f;                     // 2^20
__device__ inline ull to_integer(float a) { return (ull)__float2ll_rn(a * kActionScale); }

template <int VEC>
struct ActionVec;
template <>
struct ActionVec<4> {
    float v[4];
    __device__ void load(const float* p) {
        const float4 t = *reinterpret_cast<const float4*>(p);
        v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
    }
    __device__ bool exact() const {
        return fabsf(v[0]) <= kExactMax && fabsf(v[1]) <= kExactMax && fabsf(v[2]) <= kExactMax && fabsf(v[3]) <= kExactMax;
    }
};
template <>
struct ActionVec<1> {
    float v[1];
    __device__ void load(const float* p) { v[0] = *p; }
    __device__ bool exact() const { return fabsf(v[0]) <= kExactMax; }
};

// Values that workgroups hand to one another within the launch are written and read with device-scope atomic operations
// only (adds to the accumulators, stores of the pair scores, the loads below): these go past the XCDs' own L2 caches, so
// there is nothing to write back or to invalidate, and a fence, which would write back the whole L2 of the XCD (2048
// workgroups doing so: 147 instead of 17 us), is not needed.  What is needed is that a workgroup's operations are
// complete before it is counted: every thread waits for its own, then the barrier, then one thread adds.
template <typename T>
__device__ inline T load_shared(const T* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename T>
__device__ inline void store_shared(T* p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename T>
__device__ inline void add_shared(T* p, T v) { (void)__hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Whether this workgroup is the last of `expected` to arrive at *counter (every workgroup arrives once).
__device__ inline bool arrive_last(int* counter, int expected) {
    __shared__ int is_last;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");              // this thread's adds and stores are complete
    __syncthreads();
    if (threadIdx.x == 0)
        is_last = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == expected - 1 ? 1 : 0;
    __syncthreads();
    const bool last = is_last != 0;
    __syncthreads();                                              // is_last may be written again
    return last;
}

// Sums and counts by phase of a workgroup's slice of a trajectory, in LDS.
template <int VEC, int kT>
__device__ inline void accumulate_slice(const float* __restrict__ actions, const uint8_t* __restrict__ phase,
                                        int i, int k0, int k1, int N, int A, int K, int c0, int kb, ull* lds_sum, int* lds_cnt) {
    const int tid = threadIdx.x;
    for (int e = tid; e < kb * A; e += kT) lds_sum[e] = 0;
    for (int c = tid; c < kb; c += kT) lds_cnt[c] = 0;
    __syncthreads();

    const int AV = A / VEC;            // vectors per chunk
    const int CPI = kT / AV;           // chunks per pass of the workgroup
    const int jv = tid % AV, cs = tid / AV;
    if (cs < CPI) {
        double acc[VEC];
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[v] = 0.0;
        int cur = -1, run = 0;
        auto flush = [&]() {
            if (cur >= 0 && cur < kb && run > 0) {
#pragma unroll
                for (int v = 0; v < VEC; ++v)
                    atomicAdd(&lds_sum[(size_t)cur * A + jv * VEC + v], (ull)__double2ll_rn(acc[v]));
                if (jv == 0) atomicAdd(&lds_cnt[cur], run);
            }
        };
        const float* row = actions + (size_t)i * N * A + (size_t)jv * VEC;
        const uint8_t* ph = phase + (size_t)i * N;
        constexpr int kAhead = 4;      // chunks under way together: what a slice costs is mostly the latency of its loads
        for (int kb0 = k0 + cs; kb0 < k1; kb0 += kAhead * CPI) {
            int ph_id[kAhead];
            ActionVec<VEC> x[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const int k = kb0 + u * CPI;
                if (k < k1) {
                    ph_id[u] = ph[k];
                    x[u].load(row + (size_t)k * A);
                }
            }
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                if (kb0 + u * CPI >= k1) break;
                const int c = min(ph_id[u], K - 1) - c0;  // ids beyond the last phase count as the last; outside [0, kb): another block's
                if (c != cur || run == kExactRun) {
                    flush();
                    cur = c;
                    run = 0;
#pragma unroll
                    for (int v = 0; v < VEC; ++v) acc[v] = 0.0;
                }
                ++run;
                if (__ballot(!x[u].exact()) == 0) {      // (one flag for all four costs 2 us of 25)
#pragma unroll
                    for (int v = 0; v < VEC; ++v) acc[v] += to_fixed(x[u].v[v]);
                } else if (c >= 0 && c < kb) {
#pragma unroll
                    for (int v = 0; v < VEC; ++v) atomicAdd(&lds_sum[(size_t)c * A + jv * VEC + v], to_integer(x[u].v[v]));
                }
            }
        }
        flush();
    }
    __syncthreads();
}

__device__ inline double squared_difference(ull s_pos, int n_pos, ull s_neg, int n_neg) {
    const double mp = (double)(long long)s_pos / (double)n_pos;
    const double mn = (double)(long long)s_neg / (double)n_neg;
    const double diff = mp - mn;
    return diff * diff;
}

// Pair scores of group g for all phases by one workgroup; LDS holds the squared terms of all of them (see fuses_tail).
__device__ inline void score_pairs_of_group(int g, int A, int K, const ull* sums, const int* counts, double* lds, double* pair) {
    const size_t pos = ((size_t)g * 2 + 1) * K, neg = ((size_t)g * 2 + 0) * K;
    __syncthreads();
    const int my_c = (int)threadIdx.x < K ? threadIdx.x : 0;      // the phase this thread adds up (K <= 64)
    const int my_pos = load_shared(&counts[pos + my_c]), my_neg = load_shared(&counts[neg + my_c]);
    for (int e0 = threadIdx.x; e0 < K * A; e0 += 4 * kThreads) {
        int n_pos[4], n_neg[4];                                   // all loads of four terms under way together
        ull s_pos[4], s_neg[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = min(e0 + u * kThreads, K * A - 1), c = e / A;
            n_pos[u] = load_shared(&counts[pos + c]);
            n_neg[u] = load_shared(&counts[neg + c]);
            s_pos[u] = load_shared(&sums[pos * A + e]);
            s_neg[u] = load_shared(&sums[neg * A + e]);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = e0 + u * kThreads;
            if (e < K * A && n_pos[u] > 0 && n_neg[u] > 0) lds[e] = squared_difference(s_pos[u], n_pos[u], s_neg[u], n_neg[u]);
        }
    }
    __syncthreads();
    if ((int)threadIdx.x < K) {
        const int c = threadIdx.x;
        double score = -1.0;                                      // skipped: no chunks of one of the outcomes
        if (my_pos > 0 && my_neg > 0) {
            double acc = 0.0;
#pragma unroll 8
            for (int j = 0; j < A; ++j) acc = acc + lds[c * A + j];
            score = sqrt(acc) * kActionUnscale;
        }
        store_shared(&pair[(size_t)g * K + c], score);
    }
}

// The same as a launch of its own: one wavefront per (group, phase), striding by the grid.  All threads reach the barrier.
__global__ __launch_bounds__(kThreads) void score_pairs(const ull* __restrict__ sums, const int* __restrict__ counts, int n_groups,
                                                        int A, int K, double* pair) {
    __shared__ double sq[kThreads / kWave][256];
    const int wv = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    const int64_t n = (int64_t)n_groups * K, step = (int64_t)gridDim.x * (kThreads / kWave);
    for (int64_t w0 = (int64_t)blockIdx.x * (kThreads / kWave); w0 < n; w0 += step) {
        const int64_t w = w0 + wv, at = w < n ? w : n - 1;
        const int64_t g = at / K, c = at % K;
        const size_t pos = ((size_t)g * 2 + 1) * K + c, neg = ((size_t)g * 2 + 0) * K + c;
        const int n_pos = counts[pos], n_neg = counts[neg];
        const bool ok = n_pos > 0 && n_neg > 0;
        if (ok)
            for (int j = lane; j < A; j += kWave) sq[wv][j] = squared_difference(sums[pos * A + j], n_pos, sums[neg * A + j], n_neg);
        __syncthreads();
        if (w < n && lane == 0) {
            double score = -1.0;
            if (ok) {
                double acc = 0.0;
#pragma unroll 8
                for (int j = 0; j < A; ++j) acc = acc + sq[wv][j];
                score = sqrt(acc) * kActionUnscale;
            }
            pair[w] = score;
        }
    }
}

constexpr int64_t kPairBlocksMax = 1 << 16;   // workgroups of score_pairs at most

// Batch score of phase c = mean over the groups that contributed, added for g ascending (the order is
// part of the definition: the result must not depend on the launch).  One workgroup: the per-group values
// are brought into LDS a block of groups at a time with coalesced loads, then lane c of the first wavefront adds its
// column in order while lane c of the second counts the groups in it.
template <int kBlock, class Load>
__device__ inline void mean_of_groups(const double* pair, int n_groups, int K, double* lds, int lds_entries, double* C_out,
                                      uint8_t* valid_out, Load load) {
    __shared__ int contributing[PCM_MAX_PHASES];
    const int c = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    const int block_groups = lds_entries / K;
    double tot = 0.0;
    int n = 0;
    for (int g0 = 0; g0 < n_groups; g0 += block_groups) {
        const int groups = min(block_groups, n_groups - g0);
        __syncthreads();
        // eight loads per thread in flight before the first is stored
        for (int i0 = threadIdx.x; i0 < groups * K; i0 += 8 * kBlock) {
            double v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int i = i0 + u * kBlock;
                v[u] = i < groups * K ? load(&pair[(size_t)g0 * K + i]) : 0.0;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (i0 + u * kBlock < groups * K) lds[i0 + u * kBlock] = v[u];
        }
        __syncthreads();
        if (c < K && wave == 0) {
            // the additions stay in group order; a skipped pair adds +0.0, which leaves the non-negative sum as it is
#pragma unroll 8
            for (int g = 0; g < groups; ++g) tot = tot + fmax(lds[g * K + c], 0.0);
        } else if (c < K && wave == 1) {
#pragma unroll 8
            for (int g = 0; g < groups; ++g) n += lds[g * K + c] >= 0.0 ? 1 : 0;
        }
    }
    if (c < K && wave == 1) contributing[c] = n;
    __syncthreads();
    if (c < K && wave == 0) {
        n = contributing[c];
        C_out[c] = n > 0 ? tot / (double)n : 0.0;
        valid_out[c] = n > 0 ? 1 : 0;
    }
}

// The mean as a launch of its own.  Bound by the loads of a block and by the additions behind them; with 1024 threads
// instead of 256 a block is one round of loads (4096 groups of 64 phases: 284 -> 233 us for all four launches).
constexpr int kMeanThreads = 1024, kMeanEntries = 4096;
__global__ __launch_bounds__(kMeanThreads) void score_mean(const double* __restrict__ pair, int n_groups, int K, double* C_out,
                                                       uint8_t* valid_out) {
    __shared__ double val[kMeanEntries];
    mean_of_groups<kMeanThreads>(pair, n_groups, K, val, kMeanEntries, C_out, valid_out, [](const double* p) { return *p; });
}

// grid = T * slices * phase_blocks workgroups; a workgroup pools the phases [c0, c0 + Kb) of its
// chunks (phase_blocks is 1 unless K*A sums do not fit in LDS; then the chunks are read once per
// block of phases).  LDS: Kb*A 64-bit sums followed by Kb chunk counts, indexed by phase - c0; with kTail afterwards the
// squared terms of a group's pairs, then the pair scores.
template <int VEC, bool kTail>
__global__ __launch_bounds__(kThreads) void score_accumulate(
    const float* __restrict__ actions, const uint8_t* __restrict__ phase,
    const uint8_t* __restrict__ reward, const int32_t* __restrict__ n_chunks, int n_groups, int G, int N, int A,
    int K, int Kb, int slices, int lds_entries, ScoreWorkspace w, double* C_out, uint8_t* valid_out) {
    extern __shared__ ull lds_sum[];
    const int phase_blocks = (K + Kb - 1) / Kb;
    const int c0 = (blockIdx.x % phase_blocks) * Kb;
    const int kb = min(Kb, K - c0);                     // phases of this workgroup
    const int slice = (blockIdx.x / phase_blocks) % slices;
    const int i = blockIdx.x / phase_blocks / slices;
    const int g = i / G;
    int s = 0;                                          // successes of the group, 64 rollouts at a time
    for (int r0 = 0; r0 < G; r0 += kWave) {
        const int r = r0 + (int)(threadIdx.x % kWave);
        const uint8_t x = reward[(size_t)g * G + min(r, G - 1)];
        s += __popcll(__ballot(r < G && x != 0));
    }
    if (s != 0 && s != G) {      // with uniform rewards the group has no score; its counts stay zero
        int Ni = n_chunks ? n_chunks[i] : N;
        Ni = Ni < 0 ? 0 : (Ni > N ? N : Ni);
        const int per = (N + slices - 1) / slices;
        const int k0 = slice * per, k1 = min(Ni, k0 + per);
        if (k0 < k1) {
            int* const lds_cnt = reinterpret_cast<int*>(lds_sum + (size_t)Kb * A);
            accumulate_slice<VEC, kThreads>(actions, phase, i, k0, k1, N, A, K, c0, kb, lds_sum, lds_cnt);
            const size_t base = ((size_t)g * 2 + (reward[i] != 0)) * K + c0;
            for (int e = threadIdx.x; e < kb * A; e += kThreads)
                if (lds_cnt[e / A] > 0) add_shared(&w.sums[base * A + e], lds_sum[e]);
            for (int c = threadIdx.x; c < kb; c += kThreads)
                if (lds_cnt[c] > 0) add_shared(&w.counts[base + c], lds_cnt[c]);
        }
    }
    if (kTail) {
        double* const lds = reinterpret_cast<double*>(lds_sum);
        if (!arrive_last(reinterpret_cast<int*>(w.pair + (size_t)g * K), G * slices * phase_blocks)) return;
        score_pairs_of_group(g, A, K, w.sums, w.counts, lds, w.pair);
        if (!arrive_last(w.groups_done, n_groups)) return;
        mean_of_groups<kThreads>(w.pair, n_groups, K, lds, lds_entries, C_out, valid_out, [](const double* p) { return load_shared(p); });
    }
}

// ---- small and ordinary batches: a table per trajectory ------------------------------------------
//
// Two launches and no accumulators to clear.  The first gives every trajectory, or slice of one, a workgroup and a table of its
// own: sums and counts by phase from LDS, written as they are.  The second adds up the tables of a group, a thread per sum, or
// several where a group has more than eight tables (1 x 8 x 1024 chunks: 15.0 -> 11.1 us a call), forms the pair scores, and its
// last workgroup the mean.  Bound by latency: two loads deep in the first, three in the second.
// Kernel times, 256 trajectories of up to 128 chunks of 56 values, 5 phases: 2.1 + 11.6 us with accumulators (the additions to
// them and the hand-over to the last workgroup are the longer part), 6.1 + 7.5 with tables; 512 of up to 256 with 12 phases
// 2.2 + 10.5 + 3.8 + 2.9 against 8.7 + 7.6.
constexpr int kTableThreads = 1024;
// Workgroups of 256 threads where these load a slice in one go (four vectors each), and where there are no more sums than that: the
// wavefronts of a workgroup wait for each other several times.  Calls one after another, 1024 / 256 threads (groups x trajectories
// x chunks, values, phases): 40 x 8 x 100, 14, 5 12.9 / 10.6 us; 54 x 5 x 47, 12, 12 11.2 / 9.9; 32 x 8 x 128 in two slices, 56, 5
// 12.7 / 11.7; 32 x 8 x 64, 56, 5 10.8 / 10.9.
constexpr int kNarrowThreads = 256, kNarrowLoads = 4 * kNarrowThreads;
constexpr int kTableMeanEntries = 2048;                  // pair scores in LDS at a time
constexpr int kTableTrajectoriesMax = 768, kTableGroupsMax = 128;
constexpr size_t kTableBytesMax = PCM_SCORE_STATIC_MAX_BYTES;

struct TableWorkspace {
    ull* sums;            // [T * slices][K][A]; of phases without a chunk unwritten
    int* counts;          // [T * slices][K]
    double* pair;         // [n_groups][K]
    int* done;            // workgroups of the second launch that are done
    size_t bytes;
};
TableWorkspace carve_tables(void* ws, int n_groups, int G, int A, int K, int slices) {
    Carver c(ws);
    TableWorkspace w;
    const size_t tables = (size_t)n_groups * G * slices;
    w.sums = c.take<ull>(tables * K * A);
    w.counts = c.take<int>(tables * K);
    w.pair = c.take<double>((size_t)n_groups * K);
    w.done = c.take<int>(1);
    w.bytes = c.used();
    return w;
}
constexpr int kTablesTogether = 8;                       // tables that a thread of the second launch loads at once
// Threads of the second launch that share a sum, each a part of the group's tables, and phases per workgroup (A <= 256)
struct PairBlock {
    int parts, phases;
};
PairBlock pair_block(int A, int tables) {
    const int parts = std::min(ceil_div(tables, kTablesTogether), kTableThreads / A);
    return {parts, kTableThreads / (A * parts)};
}

// Slices per trajectory, or 0 where the batch takes the accumulators: the tables have to fit in 4 MiB, so that a shape fits the
// library's own array if it did with those, and in the workspace that the caller brings (one that holds the accumulators is enough
// for any call).  A slice is at least one chunk per thread, and no more are made than 64 tables per group or about two workgroups per
// compute unit.  Calls one after another, tables / accumulators, 56 values and 5 phases if not said (groups x trajectories x chunks):
// 2 x 8 x 64 9.2 / 9.9 us; 32 x 8 x 128 11.7 / 13.2; 64 x 8 x 256, 12 phases 16.5 / 18.7; 8 x 4 x 4096 14.2 / 21.6; 4 x 10 x 1024 12.1 /
// 16.4; 4 x 64 x 64 12.0 / 15.7; 4 x 32 x 256 of 256 values, 8 phases 19.9 / 30.2; 20 x 25 x 100 15.8 / 16.4.
// Trajectories that are loaded in one go (four chunks a thread) gain nothing from slices while they are few: 2 x 8 x 256 11.2 / 10.4, 8 x 8 x
// 100 of 35 values, 12 phases 10.8 / 10.2, 14 x 5 x 256 11.7 / 11.7, 16 x 8 x 256 12.2 / 12.8.  Nor from more than fit side by side: 56 x 8 x 256
// in two 18.7, in one 15.1, accumulators 17.1; 40 x 8 x 256 16.1 / 14.5 / 15.7; but four rather than three: 20 x 8 x 256 12.7, 13.8, 13.6.
// Longer ones do while they are few: 8 x 8 x 1024 13.6 / 17.6, 14 x 5 x 1024 15.5 / 16.5, 16 x 8 x 4096 25.7 / 26.7, but 20 x 8 x 1024 18.2 /
// 16.7, 33 x 8 x 1024 21.8 / 20.7, 56 x 8 x 1024 26.5 / 24.4; and a slice of more than 20 chunks a thread takes longer than the finer ones of
// the accumulators (24 x 8 x 4096 in two, 28 a thread, 34.6 / 32.0).
// Beyond 768 trajectories nothing is gained (64 chunks 13.9 / 15.8 at 96 x 8, but 256 19.4 / 19.5 there and 23.7 / 21.3 at 128 x 8), and
// beyond 128 groups the mean is too long for the last workgroup (128 x 4 x 64 14.1 / 15.6, 160 x 4 x 256 20.7 / 20.6, 170 x 3 x 100 18.9 /
// 17.4).
int table_slices(int n_groups, int G, int N, int A, int K, size_t bytes_max) {
    if ((size_t)K * A * sizeof(ull) + (size_t)K * sizeof(int) > kLdsMax || G > kWave) return 0;
    if (n_groups > kTableGroupsMax || (int64_t)n_groups * G > kTableTrajectoriesMax) return 0;
    const int T = n_groups * G, per_pass = kTableThreads / (A % 4 == 0 ? A / 4 : A);
    const bool one_go = N <= 4 * per_pass;
    int slices = one_go ? std::max(1, 512 / T) : ceil_div(512, T);
    if (one_go && slices == 3) slices = 4;
    slices = std::min({slices, ceil_div(N, per_pass), kWave / G});
    if (one_go ? slices > 1 && T <= 96 : T > 128) return 0;
    for (; slices > 0; --slices)
        if (carve_tables(nullptr, n_groups, G, A, K, slices).bytes <= std::min(bytes_max, kTableBytesMax)) break;
    return slices > 0 && ceil_div(N, slices) <= 20 * per_pass ? slices : 0;
}

// Successes of the group (a bit per trajectory, G <= 64), the same in every wavefront.
__device__ inline uint64_t successes_of(const uint8_t* reward, int g, int G) {
    const int r = threadIdx.x % kWave;
    const uint8_t x = reward[(size_t)g * G + min(r, G - 1)];
    return __ballot(r < G && x != 0);
}

template <int VEC, int kT>
__global__ __launch_bounds__(kT) void score_tables(const float* __restrict__ actions, const uint8_t* __restrict__ phase,
                                                   const uint8_t* __restrict__ reward, const int32_t* __restrict__ n_chunks, int G, int N,
                                                   int A, int K, int slices, double adv_eps, float* adv_out, uint8_t* active_out,
                                                   TableWorkspace w) {
    extern __shared__ ull lds_sum[];
    int* const lds_cnt = reinterpret_cast<int*>(lds_sum + (size_t)K * A);
    const int i = blockIdx.x / slices, slice = blockIdx.x % slices, g = i / G, tid = threadIdx.x;
    int Ni = n_chunks ? n_chunks[i] : N;
    const uint64_t won = successes_of(reward, g, G);
    const int s = __popcll(won);
    const bool mixed = s != 0 && s != G;
    Ni = Ni < 0 ? 0 : (Ni > N ? N : Ni);
    if (mixed) {                                  // with uniform rewards the group has no score; nobody reads its tables
        const int per = (N + slices - 1) / slices, k0 = slice * per, k1 = min(Ni, k0 + per);
        accumulate_slice<VEC, kT>(actions, phase, i, k0, k1, N, A, K, 0, K, lds_sum, lds_cnt);
        ull* const sums = w.sums + (size_t)blockIdx.x * K * A;
        for (int e = tid; e < K * A; e += kT)
            if (lds_cnt[e / A] > 0) sums[e] = lds_sum[e];
        if (tid < K) w.counts[(size_t)blockIdx.x * K + tid] = lds_cnt[tid];
    }
    if (tid != kT - 1) return;         // a thread that has had little to do
    if (blockIdx.x == 0) *w.done = 0;
    if (slice != 0) return;
    float a = 0.f;
    if (mixed) {
        const double mu = (double)s / (double)G;
        const double sigma = sqrt(mu * (1.0 - mu));
        const double r = (won >> (i - g * G)) & 1u ? 1.0 : 0.0;
        a = (float)((r - mu) / (sigma + adv_eps));
    }
    if (adv_out) adv_out[i] = a;
    if (active_out) active_out[i] = mixed ? 1 : 0;
}

template <bool kParts, int kT>
__global__ __launch_bounds__(kT) void score_of_tables(const uint8_t* __restrict__ reward, int n_groups, int G, int A, int K, int slices,
                                                                 int parts, int phases, TableWorkspace w, double* C_out, uint8_t* valid_out) {
    __shared__ double lds[kTableMeanEntries];
    __shared__ int part_n[2][kParts ? kTableThreads : 1];
    static_assert(!kParts || kT == kTableThreads);
    static_assert(kTableMeanEntries >= 2 * kTableThreads, "the parts of the sums fit");
    __shared__ int n_of[2][PCM_MAX_PHASES];
    const int blocks = (K + phases - 1) / phases, g = blockIdx.x / blocks, c0 = blockIdx.x % blocks * phases, kb = min(phases, K - c0);
    const int tid = threadIdx.x;
    const uint64_t won = successes_of(reward, g, G);
    const int s = __popcll(won);
    const bool mixed = s != 0 && s != G;
    const int sums = kb * A, tables = G * slices;
    int n_pos = 0, n_neg = 0;
    ull s_pos = 0, s_neg = 0;
    const int step = kParts ? parts * kTablesTogether : kTablesTogether;
    if (mixed && tid < (kParts ? sums * parts : sums)) {
        const int part = kParts ? tid / sums : 0, e = tid - part * sums, c = e / A;
        const size_t first = (size_t)g * tables;
        const int* const counts = w.counts + first * K + c0 + c;
        const ull* const table_sums = w.sums + first * K * A + (size_t)c0 * A + e;
        for (int t0 = part * kTablesTogether; t0 < tables; t0 += step) {
            int n[kTablesTogether];
            ull v[kTablesTogether];
#pragma unroll
            for (int u = 0; u < kTablesTogether; ++u) {
                const int t = min(t0 + u, tables - 1);
                n[u] = counts[(size_t)t * K];
                v[u] = table_sums[(size_t)t * K * A];
            }
#pragma unroll
            for (int u = 0; u < kTablesTogether; ++u) {
                if (t0 + u >= tables || n[u] == 0) continue;       // (a sum without a chunk was not written)
                if ((won >> ((t0 + u) / slices)) & 1u) { n_pos += n[u]; s_pos += v[u]; }
                else { n_neg += n[u]; s_neg += v[u]; }
            }
        }
        if (!kParts && e == c * A) {
            n_of[0][c] = n_neg;
            n_of[1][c] = n_pos;
        }
    }
    if (kParts && mixed) {                        // uniform
        ull* const part_sum = reinterpret_cast<ull*>(lds);         // [2][kTableThreads]
        part_sum[tid] = s_neg;
        part_sum[kTableThreads + tid] = s_pos;
        part_n[0][tid] = n_neg;
        part_n[1][tid] = n_pos;
        __syncthreads();
        if (tid < sums)
            for (int q = 1; q < parts; ++q) {
                s_neg += part_sum[q * sums + tid];
                s_pos += part_sum[kTableThreads + q * sums + tid];
                n_neg += part_n[0][q * sums + tid];
                n_pos += part_n[1][q * sums + tid];
            }
        if (tid < sums && tid % A == 0) {
            n_of[0][tid / A] = n_neg;
            n_of[1][tid / A] = n_pos;
        }
        __syncthreads();
    }
    if (mixed && tid < sums && n_pos > 0 && n_neg > 0) lds[tid] = squared_difference(s_pos, n_pos, s_neg, n_neg);
    __syncthreads();
    if (tid < kb) {
        double score = -1.0;                      // skipped: uniform rewards, or no chunks of one of the outcomes
        if (mixed && n_of[0][tid] > 0 && n_of[1][tid] > 0) {
            double acc = 0.0;
#pragma unroll 8
            for (int j = 0; j < A; ++j) acc = acc + lds[tid * A + j];
            score = sqrt(acc) * kActionUnscale;
        }
        store_shared(&w.pair[(size_t)g * K + c0 + tid], score);
    }
    if (!arrive_last(w.done, (int)gridDim.x)) return;
    mean_of_groups<kT>(w.pair, n_groups, K, lds, kTableMeanEntries, C_out, valid_out, [](const double* p) { return load_shared(p); });
}

// ---- the smallest batches: one workgroup, one launch ---------------------------------------------
//
// Bound by latency alone, so nothing is handed from one workgroup to another: all sums in LDS, every thread a run of
// consecutive chunks (one or two flushes), pair scores and mean behind it.
// 16 trajectories of 32 chunks of 56 values, 4 phases: one launch of 7.6 us against 2.0 + 7.6 with
// accumulators.  The line: calls one after another, this route / tables, 16 trajectories of 4 chunks 4.8 / 8.9 us,
// of 18 6.4 / 9.0, of 36 (eight chunks a thread, sixteen spill: 15.7) 8.0 / 9.1; 72 chunks each in one group of 12 phases 8.4 / 9.8;
// 4 groups of 8 trajectories of 18 chunks 8.8 / 9.0, 18 groups of 8 of 4 chunks 9.4 / 9.4 (4032 pair terms: no gain beyond 4096).
constexpr int kSmallThreads = 1024;
constexpr int kSmallPerThread = 8;            // chunks per thread at most
struct SmallShape {
    int n_groups, G, N, A, K;
    __host__ __device__ int sums() const { return n_groups * 2 * K * A; }
    // LDS: the sums; chunks pooled [n_groups][2][K]; squared terms [n_groups][K][A]; pair scores [n_groups][K]
    __host__ __device__ size_t lds_bytes() const {
        return (size_t)sums() * 8 + (size_t)n_groups * K * A * 8 + (size_t)n_groups * K * 8 + (size_t)n_groups * 2 * K * 4;
    }
};
bool is_vec4(const float* actions, int A) { return A % 4 == 0 && (reinterpret_cast<uintptr_t>(actions) & 15u) == 0; }
bool is_small(const SmallShape& p, bool vec4) {
    const int chunks_at_once = kSmallThreads / (vec4 ? p.A / 4 : p.A);
    return (int64_t)p.n_groups * p.G * p.N <= (int64_t)chunks_at_once * kSmallPerThread && (int64_t)p.n_groups * p.G <= kSmallThreads &&
           p.G <= kWave && (int64_t)p.n_groups * p.K * p.A <= 4096 && p.lds_bytes() <= kLdsMax - 2 * kSmallThreads * sizeof(int);
}
template <int VEC>
__global__ __launch_bounds__(kSmallThreads) void score_small(const float* __restrict__ actions, const uint8_t* __restrict__ phase,
                                                             const uint8_t* __restrict__ reward, const int32_t* __restrict__ n_chunks, SmallShape p,
                                                             double adv_eps, double* C_out, uint8_t* valid_out, float* adv_out,
                                                             uint8_t* active_out) {
    extern __shared__ ull lds_sum[];
    const int G = p.G, N = p.N, A = p.A, K = p.K, T = p.n_groups * G, tid = threadIdx.x;
    double* const sq = reinterpret_cast<double*>(lds_sum + p.sums());
    double* const pair = sq + (size_t)p.n_groups * K * A;
    int* const counts = reinterpret_cast<int*>(pair + (size_t)p.n_groups * K);
    __shared__ int table_of[kSmallThreads];       // of each trajectory: its (group, outcome), or -1 in a group of uniform rewards
    __shared__ int valid_of[kSmallThreads];       // and how many of its chunks are there
    const int AV = A / VEC, CPI = kSmallThreads / AV;             // vectors per chunk; threads per vector
    const int jv = tid % AV, cs = tid / AV;
    const int per = (T * N + CPI - 1) / CPI, q0 = cs * per, q1 = cs < CPI ? min(q0 + per, T * N) : q0;
    int ph[kSmallPerThread];
    ActionVec<VEC> x[kSmallPerThread];
#pragma unroll
    for (int u = 0; u < kSmallPerThread; ++u)                     // all loads of a thread under way together
        if (q0 + u < q1) {
            ph[u] = phase[q0 + u];
            x[u].load(actions + (size_t)(q0 + u) * A + (size_t)jv * VEC);
        }
    for (int e = tid; e < p.sums(); e += kSmallThreads) lds_sum[e] = 0;
    for (int e = tid; e < p.n_groups * 2 * K; e += kSmallThreads) counts[e] = 0;
    if (tid < T) {
        const int g = tid / G;
        int s = 0;
        for (int r0 = 0; r0 < G; r0 += 8)             // eight loads under way together
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const uint8_t x = reward[(size_t)g * G + min(r0 + u, G - 1)];
                s += r0 + u < G && x != 0;
            }
        const bool won = reward[tid] != 0, mixed = s != 0 && s != G;
        int Ni = n_chunks ? n_chunks[tid] : N;
        valid_of[tid] = Ni < 0 ? 0 : (Ni > N ? N : Ni);
        table_of[tid] = mixed ? g * 2 + (won ? 1 : 0) : -1;
    }
    __syncthreads();
    double acc[VEC];
    int i = q0 / N, k = q0 - i * N;                               // trajectory and slot
    int cur = -1, run = 0;                                        // the sums under way: (table, phase)
    auto flush = [&]() {
        if (run == 0) return;
#pragma unroll
        for (int v = 0; v < VEC; ++v) atomicAdd(&lds_sum[(size_t)cur * A + jv * VEC + v], (ull)__double2ll_rn(acc[v]));
        if (jv == 0) atomicAdd(&counts[cur], run);
    };
#pragma unroll
    for (int u = 0; u < kSmallPerThread; ++u) {
        if (q0 + u >= q1) break;
        const int table = table_of[i], slot = k++;
        const bool in = table >= 0 && slot < valid_of[i];
        if (k == N) {
            k = 0;
            ++i;
        }
        if (!in) continue;
        const int to = table * K + min(ph[u], K - 1);             // ids beyond the last phase count as the last
        if (to != cur) {
            flush();
            cur = to;
            run = 0;
#pragma unroll
            for (int v = 0; v < VEC; ++v) acc[v] = 0.0;
        }
        ++run;
        if (__ballot(!x[u].exact()) == 0) {
#pragma unroll
            for (int v = 0; v < VEC; ++v) acc[v] += to_fixed(x[u].v[v]);
        } else {
#pragma unroll
            for (int v = 0; v < VEC; ++v) atomicAdd(&lds_sum[(size_t)to * A + jv * VEC + v], to_integer(x[u].v[v]));
        }
    }
    flush();
    __syncthreads();
    for (int e = tid; e < p.n_groups * K * A; e += kSmallThreads) {
        const int g = e / (K * A), r = e - g * K * A, c = r / A;
        const int n_neg = counts[(g * 2) * K + c], n_pos = counts[(g * 2 + 1) * K + c];
        if (n_pos > 0 && n_neg > 0)
            sq[e] = squared_difference(lds_sum[(size_t)(g * 2 + 1) * K * A + r], n_pos, lds_sum[(size_t)(g * 2) * K * A + r], n_neg);
    }
    __syncthreads();
    if (tid >= kSmallThreads - T) {                               // advantages, by the last threads: the first ones add up the pairs
        const int t = tid - (kSmallThreads - T), table = table_of[t];
        float a = 0.f;
        if (table >= 0) {
            int s = 0;
            for (int r = t / G * G; r < t / G * G + G; ++r) s += table_of[r] & 1;
            const double mu = (double)s / (double)G;
            const double sigma = sqrt(mu * (1.0 - mu));
            a = (float)(((double)(table & 1) - mu) / (sigma + adv_eps));
        }
        if (adv_out) adv_out[t] = a;
        if (active_out) active_out[t] = table >= 0 ? 1 : 0;
    }
    for (int e = tid; e < p.n_groups * K; e += kSmallThreads) {
        const int g = e / K, c = e - g * K;
        double score = -1.0;                                      // skipped: no chunks of one of the outcomes
        if (counts[(g * 2) * K + c] > 0 && counts[(g * 2 + 1) * K + c] > 0) {
            double sum = 0.0;
#pragma unroll 8
            for (int j = 0; j < A; ++j) sum = sum + sq[(size_t)e * A + j];
            score = sqrt(sum) * kActionUnscale;
        }
        pair[e] = score;
    }
    __syncthreads();
    if (tid < K) {                                                // the mean over contributing groups, added for g ascending
        double tot = 0.0;
        int n = 0;
#pragma unroll 8
        for (int g = 0; g < p.n_groups; ++g) {
            const double v = pair[g * K + tid];
            tot = tot + fmax(v, 0.0);                             // a skipped pair adds +0.0, which leaves the non-negative sum as it is
            n += v >= 0.0 ? 1 : 0;
        }
        C_out[tid] = n > 0 ? tot / (double)n : 0.0;
        valid_out[tid] = n > 0 ? 1 : 0;
    }
}

// Whether pair scores and mean are formed behind the accumulation (two launches in all) or by launches of their own (four).
// Two launches save about 5 us, which count while the calls are bound by issuing them.  Behind the accumulation a group's
// pair scores are the work of one workgroup and the mean waits for loads past the L2 caches, and every workgroup pays for
// arriving.  Measured per call, two / four launches, the other bound held:
//   by the pair terms of a group, one group:  12 phases of 56 values 11.9 / 17.4 us; 24 of 128 (3072 terms) 15.0 / 17.3,
//   33 of 128 (4224) 17.4 / 17.4, 24 of 256 (6144) 21.4 / 18.7, 64 of 256 40.6 / 19.9
//   by those of all groups:  32 groups of 5 x 56 (8960) 14.0 / 14.8 us, 8 of 24 x 128 (24576) 15.8 / 16.9, 8 of 33 x 128
//   (33792) 18.4 / 17.5, 64 of 12 x 56 (43008, 256 chunks each) 19.4 / 18.6, 256 of 12 x 56 29.6 / 26.5, 1024 of 12 x 56
//   88.5 / 75.5
bool fuses_tail(int n_groups, int A, int K) {
    static_assert(4096 * sizeof(ull) + PCM_MAX_PHASES * sizeof(int) <= kLdsMax, "a group's sums and squared terms fit in LDS");
    return K * A <= 4096 && (int64_t)n_groups * K * A <= 32768;
}

bool shape_ok(int n_groups, int G, int N, int A, int K) {
    return n_groups >= 1 && G >= 1 && N >= 1 && A >= 1 && A <= 256 && K >= 1 && K <= PCM_MAX_PHASES &&
           (int64_t)n_groups * G * N < (int64_t)1 << 31;
}

}  // namespace
}  // namespace pcm

using namespace pcm;

extern "C" size_t pcm_score_phases_workspace_bytes(int n_groups, int G, int N, int A, int K) {
    if (!shape_ok(n_groups, G, N, A, K)) return 0;
    const int slices = table_slices(n_groups, G, N, A, K, kTableBytesMax);
    return std::max(carve(nullptr, n_groups, A, K).bytes, slices > 0 ? carve_tables(nullptr, n_groups, G, A, K, slices).bytes : 0);
}

// ---- scratch memory owned by the library, for the entry point that takes no workspace -------------
// Every GPU holds its own copy of this array at its own address.  In host code the array's name is
// only a handle for hipGetSymbolAddress: the address that kernels and fills receive is the one that
// call returns on the device that is current, looked up once per device and kept.
constexpr size_t kStaticScratchBytes = PCM_SCORE_STATIC_MAX_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {

int run_small(const float* actions, const uint8_t* phase, const uint8_t* reward, const int32_t* n_chunks, const SmallShape& p, double adv_eps,
              double* C_out, uint8_t* valid_out, float* adv_out, uint8_t* active_out, hipStream_t s) {
    StageTimer t(ST_SCORE_ACCUMULATE, s);
    if (is_vec4(actions, p.A))
        score_small<4><<<1, kSmallThreads, p.lds_bytes(), s>>>(actions, phase, reward, n_chunks, p, adv_eps, C_out, valid_out, adv_out, active_out);
    else
        score_small<1><<<1, kSmallThreads, p.lds_bytes(), s>>>(actions, phase, reward, n_chunks, p, adv_eps, C_out, valid_out, adv_out, active_out);
    return launch_status();
}
int run_tables(const float* actions, const uint8_t* phase, const uint8_t* reward, const int32_t* n_chunks, int n_groups, int G, int N, int A,
               int K, double adv_eps, double* C_out, uint8_t* valid_out, float* adv_out, uint8_t* active_out, int slices,
               const TableWorkspace& w, hipStream_t s) {
    {
        StageTimer t(ST_SCORE_ACCUMULATE, s);
        const bool vec4 = is_vec4(actions, A);
        const unsigned grid = (unsigned)(n_groups * G) * (unsigned)slices;
        const size_t lds_bytes = (size_t)K * A * sizeof(ull) + (size_t)K * sizeof(int);
        const bool narrow = (int64_t)ceil_div(N, slices) * (vec4 ? A / 4 : A) <= kNarrowLoads;
#define PCM_TABLES(VEC, THREADS)                                                                                               \
    score_tables<VEC, THREADS><<<grid, THREADS, lds_bytes, s>>>(actions, phase, reward, n_chunks, G, N, A, K, slices, adv_eps, \
                                                                adv_out, active_out, w)
        if (vec4 && narrow) PCM_TABLES(4, kNarrowThreads);
        else if (vec4) PCM_TABLES(4, kTableThreads);
        else if (narrow) PCM_TABLES(1, kNarrowThreads);
        else PCM_TABLES(1, kTableThreads);
#undef PCM_TABLES
    }
    StageTimer t(ST_SCORE_FINALISE, s);
    const PairBlock block = pair_block(A, G * slices);
    const unsigned grid = (unsigned)n_groups * (unsigned)ceil_div(K, block.phases);
#define PCM_OF_TABLES(PARTS, THREADS)                                                                                       \
    score_of_tables<PARTS, THREADS><<<grid, THREADS, 0, s>>>(reward, n_groups, G, A, K, slices, block.parts, block.phases, w, C_out, valid_out)
    if (block.parts > 1) PCM_OF_TABLES(true, kTableThreads);
    else if (K * A <= kNarrowThreads) PCM_OF_TABLES(false, kNarrowThreads);
    else PCM_OF_TABLES(false, kTableThreads);
#undef PCM_OF_TABLES
    return launch_status();
}

int run_score(const float* actions, const uint8_t* phase, const uint8_t* reward, const int32_t* n_chunks,
              int n_groups, int G, int N, int A, int K, double adv_eps, double* C_out, uint8_t* valid_out,
              float* adv_out, uint8_t* active_out, const ScoreWorkspace& w, hipStream_t s) {
    // phases per workgroup: all K if their sums fit in LDS (A <= 256: at least 31 do)
    int Kb = (int)(kLdsMax / ((size_t)A * sizeof(ull) + sizeof(int)));
    if (Kb > K) Kb = K;
    const int phase_blocks = ceil_div(K, Kb);
    size_t lds_bytes = (size_t)Kb * A * sizeof(ull) + (size_t)Kb * sizeof(int);
    const bool tail = fuses_tail(n_groups, A, K);
    if (tail) {
        // all pair scores, but no more than lets eight workgroups share a CU (a group's scores fit, whatever K): the mean
        // waits for loads once per block of groups that fits here
        lds_bytes = std::max(lds_bytes, std::min((size_t)n_groups * K * sizeof(double), (size_t)16 * 1024));
    }
    const int lds_entries = (int)(lds_bytes / sizeof(double));
    const int T = n_groups * G;
    {
        StageTimer t(ST_SCORE_PREPARE, s);
        const size_t work = w.zero_words > (size_t)T ? w.zero_words : (size_t)T;
        const int blocks = (int)((work + kThreads - 1) / kThreads);
        score_prepare<<<blocks < 1024 ? blocks : 1024, kThreads, 0, s>>>(
            reinterpret_cast<uint32_t*>(w.sums), w.zero_words, reward, T, G, adv_eps, adv_out,
            active_out);
    }
    {
        StageTimer t(ST_SCORE_ACCUMULATE, s);
        const bool vec4 = is_vec4(actions, A);
        const int chunks_per_pass = kThreads / (vec4 ? A / 4 : A);
        // enough workgroups to cover the chip several times over, but at least two passes each
        int slices = ceil_div(2048, T);
        const int max_slices = ceil_div(N, 2 * chunks_per_pass);
        if (slices > max_slices) slices = max_slices;
        if (slices < 1) slices = 1;
        const unsigned grid = (unsigned)T * (unsigned)slices * (unsigned)phase_blocks;
#define PCM_ACCUMULATE(VEC, TAIL)                                                                                         \
    score_accumulate<VEC, TAIL><<<grid, kThreads, lds_bytes, s>>>(actions, phase, reward, n_chunks, n_groups, G, N, A, K, Kb, \
                                                                  slices, lds_entries, w, C_out, valid_out)
        if (vec4 && tail) PCM_ACCUMULATE(4, true);
        else if (vec4) PCM_ACCUMULATE(4, false);
        else if (tail) PCM_ACCUMULATE(1, true);
        else PCM_ACCUMULATE(1, false);
#undef PCM_ACCUMULATE
    }
    if (!tail) {
        StageTimer t(ST_SCORE_FINALISE, s);
        const int64_t pair_blocks = ceil_div64((int64_t)n_groups * K, kThreads / kWave);
        score_pairs<<<(unsigned)std::min<int64_t>(pair_blocks, kPairBlocksMax), kThreads, 0, s>>>(w.sums, w.counts, n_groups, A, K,
                                                                                                w.pair);
        score_mean<<<1, kMeanThreads, 0, s>>>(w.pair, n_groups, K, C_out, valid_out);
    }
    return launch_status();
}

// The launches of either entry point; the workspace holds the accumulators at least.
int run_in(void* workspace, size_t workspace_bytes, const float* actions, const uint8_t* phase, const uint8_t* reward, const int32_t* n_chunks, int n_groups, int G,
           int N, int A, int K, double adv_eps, double* C_out, uint8_t* valid_out, float* adv_out, uint8_t* active_out, hipStream_t s) {
    const SmallShape small{n_groups, G, N, A, K};
    if (is_small(small, is_vec4(actions, A)))
        return run_small(actions, phase, reward, n_chunks, small, adv_eps, C_out, valid_out, adv_out, active_out, s);
    if (const int slices = table_slices(n_groups, G, N, A, K, workspace_bytes); slices > 0)
        return run_tables(actions, phase, reward, n_chunks, n_groups, G, N, A, K, adv_eps, C_out, valid_out, adv_out, active_out, slices,
                          carve_tables(workspace, n_groups, G, A, K, slices), s);
    return run_score(actions, phase, reward, n_chunks, n_groups, G, N, A, K, adv_eps, C_out, valid_out, adv_out, active_out,
                     carve(workspace, n_groups, A, K), s);
}

bool args_ok(const float* actions, const uint8_t* phase, const uint8_t* reward, int n_groups, int G, int N, int A,
             int K, double adv_eps, const double* C_out, const uint8_t* valid_out) {
    return actions && phase && reward && C_out && valid_out && shape_ok(n_groups, G, N, A, K) && adv_eps >= 0.0;
}

constexpr int kMaxDevices = 64;
std::mutex scratch_mu;
void* scratch_of_device[kMaxDevices] = {};

int static_scratch(void** out) {
    int device = -1;
    if (hipGetDevice(&device) != hipSuccess) return PCM_EHIP;
    if (device < 0 || device >= kMaxDevices) return PCM_EUNSUPPORTED;
    std::lock_guard<std::mutex> lock(scratch_mu);
    if (scratch_of_device[device] == nullptr) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) {
            (void)hipGetLastError();
            return PCM_EHIP;
        }
        scratch_of_device[device] = p;
    }
    *out = scratch_of_device[device];
    return PCM_OK;
}

}  // namespace

extern "C" int pcm_score_phases(const float* actions, const uint8_t* phase, const uint8_t* reward,
                                const int32_t* n_chunks, int n_groups, int G, int N, int A, int K,
                                double adv_eps, double* C_out, uint8_t* valid_out, float* adv_out,
                                uint8_t* active_out, void* workspace, size_t workspace_bytes,
                                void* stream) {
    if (!args_ok(actions, phase, reward, n_groups, G, N, A, K, adv_eps, C_out, valid_out)) return PCM_EINVAL;
    if (!workspace_ok(workspace, workspace_bytes, carve(nullptr, n_groups, A, K).bytes)) return PCM_EWORKSPACE;
    return run_in(workspace, workspace_bytes, actions, phase, reward, n_chunks, n_groups, G, N, A, K, adv_eps, C_out, valid_out, adv_out, active_out,
                  static_cast<hipStream_t>(stream));
}

extern "C" int pcm_score_phases_static(const float* actions, const uint8_t* phase, const uint8_t* reward,
                                       const int32_t* n_chunks, int n_groups, int G, int N, int A, int K,
                                       double adv_eps, double* C_out, uint8_t* valid_out, float* adv_out,
                                       uint8_t* active_out, void* stream) {
    if (!args_ok(actions, phase, reward, n_groups, G, N, A, K, adv_eps, C_out, valid_out)) return PCM_EINVAL;
    if (carve(nullptr, n_groups, A, K).bytes > kStaticScratchBytes) return PCM_EWORKSPACE;
    void* base = nullptr;
    const int rc = static_scratch(&base);
    if (rc != PCM_OK) return rc;
    return run_in(base, kStaticScratchBytes, actions, phase, reward, n_chunks, n_groups, G, N, A, K, adv_eps, C_out, valid_out, adv_out, active_out,
                  static_cast<hipStream_t>(stream));
}
