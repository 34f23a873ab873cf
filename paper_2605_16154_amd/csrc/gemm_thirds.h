// Products of fp32 matrices held as three bf16 matrices each (thirds.h), on tiles of 128 x 128 (internal header).
//
// A workgroup of four wavefronts (2 x 2, each 64 x 64) brings in the three parts of both operands for 32 k (48 KB) and forms
// six products of them: every part is loaded once and used two or three times, where six reductions of the bf16 main loop would
// load it as often (all products of a step that way, as segments of one reduction on tiles of 256 and 128: 10,752 rows of 1024 -> 2816
// 2.45 ms against 2.20, 5376 of 256 -> 1024 303 us against 230).  One workgroup per CU; the fragments of a whole step are in
// registers, so a step's memory is free again when it begins, and three steps are on their way or being read.
//
// Bound by the matrix pipe: a step's 96 MFMAs take 0.73 us at 2.1 GHz, and one workgroup alone takes 0.76 a step with all loads
// and reads; over the whole chip the power cap sets the clock: 8192 x 1024 x 2816 [rows][K] both 214 us (1.32 PFLOP/s of bf16
// products), [K][rows] both 204, 8192 x 1024 x 5632 355 and 368.  Without the loads 10 to 15 % less, without the reads 3 to 7.
#pragma once

#include "gemm_bf16.h"
#include "thirds.h"

namespace pcm {

constexpr int kThirdsK = 32;                                          // k per step
constexpr uint32_t kPartBytes = kTile<kSmallTile> * kThirdsK * 2;     // a part of an operand tile
constexpr uint32_t kThirdsSlot = 6 * kPartBytes;                      // A and B tile of a step
constexpr int kThirdsSlots = 3, kThirdsLoads = 12;                    // steps in LDS; wave-wide loads per wavefront and step
using ThirdsRing = OperandRing<kSmallTile, kDeepRingSlots>;
static_assert(kThirdsSlots * kThirdsSlot == sizeof(ThirdsRing), "three steps");

// The compiler does not know how long an MFMA in inline assembly takes to write its results: whatever reads these accumulators
// afterwards goes through the assembly here and comes behind the wait.
__device__ __forceinline__ void wait_mfma_results(Accumulators<kSmallTile>& acc) {
    static_assert(kSmallTile == 4);
    asm volatile("s_nop 15\n\ts_nop 15" : "+a"(acc[0][0]), "+a"(acc[0][1]), "+a"(acc[0][2]), "+a"(acc[0][3]), "+a"(acc[1][0]), "+a"(acc[1][1]),
                 "+a"(acc[1][2]), "+a"(acc[1][3]));
    asm volatile("" : "+a"(acc[2][0]), "+a"(acc[2][1]), "+a"(acc[2][2]), "+a"(acc[2][3]), "+a"(acc[3][0]), "+a"(acc[3][1]), "+a"(acc[3][2]),
                 "+a"(acc[3][3]));
}

template <int kLayA, int kLayB, class Epilogue>
__device__ __forceinline__ void thirds_tile(const GemmProblem& p, const Epilogue& epi, int block, ThirdsRing& smem) {
    constexpr int kW = kSmallTile, T = kTile<kW>;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int tiles_m = p.M / T, tiles_n = p.N / T, n_tiles = tiles_m * tiles_n;
    const int split = block / n_tiles;
    if (split >= p.splits) return;                               // workgroups come in multiples of eight
    int k1 = p.K1, live_m = tiles_m;
    if (p.kept != nullptr) {
        const int rows = p.live_rows();
        if (p.rows_role == kRowsAreM) live_m = min(tiles_m, (rows + kTileM - 1) / kTileM * (kTileM / T));
        if (p.rows_role == kRowsAreK) k1 = min(k1, (rows + kTileK - 1) / kTileK * kTileK);
    }
    int tm, tn;
    if (!tile_of_workgroup<kLargeTile>(block % n_tiles, n_tiles, live_m, tiles_n, tm, tn)) return;   // (one workgroup per CU, as of large tiles)
    const int m0 = tm * T, n0 = tn * T;
    const int steps_all = k1 / kThirdsK, per_split = (steps_all + p.splits - 1) / p.splits;
    const int step_begin = split * per_split, step_end = min(steps_all, step_begin + per_split);

    // Global -> LDS as in gemm_tile.  A part of an operand tile is 8 KB:
    //   [rows][K]: rows of 64 B; a load fills 16 rows, wave w rows 32 w .. 32 w + 31; the 16-byte piece q of row r sits in place
    //     q ^ ((r >> 2) & 3), so that the 16 rows of a fragment read spread over all banks.
    //   [K][rows]: k-rows of 256 B; a load fills 4 k-rows, wave w k-rows 8 w .. 8 w + 7; 32-byte units in place swizzle_unit.
    const uint32_t lds_base = (uint32_t)(uintptr_t)PCM_AS_LDS(smem.data);
    uint32_t off[2][2], step_bytes[2];
    int64_t row_bytes[2];                                        // of the blocks of 128 rows
    const char* from[2][3];                                      // [operand][part]: of the newest step requested so far
#pragma unroll
    for (int operand = 0; operand < 2; ++operand) {
        const uint32_t ld = (uint32_t)(operand == 0 ? p.lda : p.ldb);
        const int row0 = operand == 0 ? m0 : n0, layout = operand == 0 ? kLayA : kLayB;
        row_bytes[operand] = (int64_t)(ld / 32) * kThirdsBlock * 2;
        int64_t at;
        if (layout == kRowsByK) {
            at = Thirds::at(row0 + wave * 32, (int64_t)step_begin * kThirdsK, ld);
            off[operand][0] = (uint32_t)(lane >> 2) * 64u + (uint32_t)((lane & 3) ^ ((lane >> 4) & 3)) * 16u;
            off[operand][1] = off[operand][0] + 1024u;
            step_bytes[operand] = kThirdsBlock * 2;
        } else {
            at = Thirds::at((int64_t)step_begin * kThirdsK + wave * 8, row0, ld);
            const int unit = swizzle_unit((lane & 15) >> 1, wave * 8 + (lane >> 4));
            off[operand][0] = (uint32_t)(unit >> 1) * (kThirdsBlock * 2u) + (uint32_t)(lane >> 4) * 64u + (uint32_t)(unit & 1) * 32u + (uint32_t)(lane & 1) * 16u;
            off[operand][1] = off[operand][0] + 256u;
            step_bytes[operand] = 2048;                          // to the next 32 rows of the blocks; after four the next blocks
        }
#pragma unroll
        for (int t = 0; t < 3; ++t) from[operand][t] = tile_address<true>((operand == 0 ? p.A : p.B) + at + t * kThirdsPart);
    }
    // from the tile of step s to that of the next one
    auto to_next = [&](int operand, int s) -> int64_t {
        if ((operand == 0 ? kLayA : kLayB) == kRowsByK) return step_bytes[operand];
        return (s & 3) == 3 ? row_bytes[operand] - 3 * (int64_t)step_bytes[operand] : (int64_t)step_bytes[operand];
    };
    const uint32_t my_lds = lds_base + (uint32_t)wave * 2048u;
    // LDS address of this lane's share of fragment 0, part 0, of a step in slot 0 (see gemm_tile)
    auto fragment_base = [&](int layout, int sub_row0) -> uint32_t {
        if (layout == kRowsByK) {
            const int row = sub_row0 + (lane & 15);
            return lds_base + (uint32_t)(row * 64 + (((lane >> 4) ^ ((row >> 2) & 3)) << 4));
        }
        const int k = (lane >> 4) * 8 + ((lane & 15) >> 2);
        return lds_base + (uint32_t)(k * 256 + (swizzle_unit(sub_row0 >> 4, k) << 5) + ((lane & 3) << 3));
    };
    const uint32_t base_a = fragment_base(kLayA, wm * 64), base_b = fragment_base(kLayB, wn * 64) + 3 * kPartBytes;

    // Sums of the products of first parts, and of the five small ones: the matrix cores cut off what they add, and of what is
    // 2^-8 of the whole that does not count.  With kChainSteps the first are one chain of additions over that many steps (an even
    // number), and the chains are added up: over the rows of a batch a single chain rounds more often than the parts of a sum on the
    // fp32 matrix instructions do.  (A flush per chain in a loop around the steps: as a branch among them it costs 2.6 % of a step.)
    Accumulators<kW> high, low, whole;                          // whole: of the chains before this one, if there are any
    bool chained = false;
#pragma unroll
    for (int i = 0; i < kW; ++i)
#pragma unroll
        for (int j = 0; j < kW; ++j) high[i][j] = low[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    if (step_begin < step_end) {
        const int last = step_end - 1;
        bf16x8 fa[2][3][kW], fb[2][3][kW];                       // fragments of this step and the next
        auto read = [](int layout, uint32_t at, int i, int part) -> bf16x8 {     // `at`: of fragment i if [K][rows], else of fragment 0
            if (layout == kRowsByK) return *(const __attribute__((address_space(3))) bf16x8*)(uintptr_t)(at + (uint32_t)i * 1024u + (uint32_t)part * kPartBytes);
            return join_halves(read_transposed(at + (uint32_t)part * kPartBytes), read_transposed(at + (uint32_t)part * kPartBytes + 1024u));
        };
        // Prologue: the first three steps are requested (steps past the end re-request the last one, which nobody reads).
#pragma unroll
        for (int s = 0; s < kThirdsSlots; ++s) {
#pragma unroll
            for (int n = 0; n < kThirdsLoads; ++n)
                direct_load_16B(from[n / 6][n % 6 / 2], off[n / 6][n % 2],
                                my_lds + (uint32_t)s * kThirdsSlot + (uint32_t)(n / 2) * kPartBytes + (uint32_t)(n % 2) * 1024u);
            const bool more = step_begin + s + 1 <= last;
#pragma unroll
            for (int n = 0; n < 6; ++n) from[n / 3][n % 3] += more ? to_next(n / 3, step_begin + s) : 0;
        }
        wait_direct_loads<2 * kThirdsLoads>();
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kW; ++i)
#pragma unroll
            for (int t = 0; t < 3; ++t) {
                fa[0][t][i] = read(kLayA, kLayA == kRowsByK ? base_a : base_a ^ (uint32_t)(32 * i), i, t);
                fb[0][t][i] = read(kLayB, kLayB == kRowsByK ? base_b : base_b ^ (uint32_t)(32 * i), i, t);
            }
        // One step of 32 k per call, its fragments in set `set`; those of the next step are read meanwhile, and the step three
        // further is requested into the slot whose fragments every wavefront holds in registers.  96 MFMAs in a fixed order,
        // one small thing in each gap (see gemm_tile): a load every eighth, then the fragment reads, the scalar bookkeeping last.
        uint32_t cur = 0, next = kThirdsSlot, far = 2 * kThirdsSlot;
        auto step = [&](auto which, int s) __attribute__((always_inline)) {
            constexpr int set = decltype(which)::value;
            wait_direct_loads<kThirdsLoads>();
            __syncthreads();
            const uint32_t refill = my_lds + cur, rd_a = fragment_address_sum(base_a, next), rd_b = fragment_address_sum(base_b, next);
            const bool more = s + kThirdsSlots + 1 <= last;
            const int64_t stride[2] = {more ? to_next(0, s + kThirdsSlots) : 0, more ? to_next(1, s + kThirdsSlots) : 0};
            uint32_t tr_at = 0;
            s16x4 tr_low = {0, 0, 0, 0};
            static_for<96>([&](auto number) __attribute__((always_inline)) {
                constexpr int n = decltype(number)::value;
                constexpr int kLeft[6] = {2, 0, 1, 1, 0, 0}, kRight[6] = {0, 2, 1, 0, 1, 0};
                constexpr int term = n / 16, i = n % 16 / 4, j = (i & 1) ? 3 - n % 4 : n % 4;
                f32x4& acc = term == 5 ? high[i][j] : low[i][j];
                if constexpr (n % 8 == 0) {
                    constexpr int load = n / 8;
                    mfma_16x16x32_and_load<(load / 2) * kPartBytes + (load % 2) * 1024u>(
                        acc, fb[set][kRight[term]][j], fa[set][kLeft[term]][i], from[load / 6][load % 6 / 2], off[load / 6][load % 2], refill);
                } else {
                    mfma_16x16x32(acc, fb[set][kRight[term]][j], fa[set][kLeft[term]][i]);
                }
                __builtin_amdgcn_sched_barrier(0);
                // fragment reads: seven gaps for each i of an operand, an address and three reads in halves ([K][rows]) or three reads
                constexpr int piece = n % 7, f = n / 7;          // f 0 .. 3: A, 4 .. 7: B
                if constexpr (f < 8) {
                    constexpr int layout = f < 4 ? kLayA : kLayB, at = f % 4;
                    auto& to = f < 4 ? fa[set ^ 1] : fb[set ^ 1];
                    const uint32_t rd = f < 4 ? rd_a : rd_b;
                    if constexpr (layout == kRowsByK) {
                        if constexpr (piece % 2 == 1) to[piece / 2][at] = read(layout, rd, at, piece / 2);
                    } else {
                        if constexpr (piece == 0) tr_at = fragment_address(rd, 32 * at);
                        else if constexpr (piece % 2 == 1) tr_low = read_transposed(tr_at + (piece / 2) * kPartBytes);
                        else to[piece / 2 - 1][at] = join_halves(tr_low, read_transposed(tr_at + (piece / 2 - 1) * kPartBytes + 1024u));
                    }
                }
                if constexpr (n >= 90) {
                    constexpr int q = n - 90;
                    from[q / 3][q % 3] += stride[q / 3];
                }
                __builtin_amdgcn_sched_barrier(0);
            });
            const uint32_t was = cur;
            cur = next;
            next = far;
            far = was;
        };
        for (int s = step_begin;;) {
            const int chain_end = Epilogue::kChainSteps > 0 ? min(step_end, s + Epilogue::kChainSteps) : step_end;
            for (; s < chain_end; s += 2) {
                step(Index<0>{}, s);
                if (s + 1 >= step_end) continue;
                step(Index<1>{}, s + 1);
            }
            if (Epilogue::kChainSteps == 0 || s >= step_end) break;
            wait_mfma_results(high);
#pragma unroll
            for (int i = 0; i < kW; ++i)
#pragma unroll
                for (int j = 0; j < kW; ++j) {
                    whole[i][j] = chained ? whole[i][j] + high[i][j] : high[i][j];
                    high[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
                    asm volatile("s_nop 1" : "+a"(high[i][j]));             // an MFMA may follow
                }
            chained = true;
        }
        wait_direct_loads<0>();
        wait_mfma_results(high);
        wait_mfma_results(low);
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < kW; ++i)
#pragma unroll
        for (int j = 0; j < kW; ++j) {
            if (chained) high[i][j] += whole[i][j];
            high[i][j] += low[i][j];
        }
    const TileCoord<kW> tc{m0, n0, wm, wn, lane, split};
    epi(tc, high, reinterpret_cast<char*>(smem.data));
}

}  // namespace pcm
