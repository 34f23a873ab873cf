// bf16 matrix-core GEMM for gfx950 with fused epilogues (internal header).
//
// C[m, n] = sum_k A(m, k) * B(n, k).  Each operand may be stored either with the reduction index
// contiguous ([rows][K], the layout the MFMA operand registers want: a lane feeds 8 consecutive k
// of one row, read with ds_read_b128) or with the reduction index as the slow dimension
// ([K][rows], e.g. activations in the weight-gradient products); the latter is brought into
// operand layout by gfx950's LDS transpose reads (ds_read_b64_tr_b16), so no operand is ever
// copied transposed in memory.
//
// Tiling: 256 x 256 x 64 per workgroup of 4 wavefronts (2 x 2), each wavefront owning 128 x 128 =
// 8 x 8 tiles of v_mfma_f32_16x16x32_bf16 with fp32 accumulators (256 accumulation registers per
// lane, one wavefront per SIMD).  Operand tiles (32 KB each) live in a ring of five LDS slots
// filled by direct global-to-LDS loads (no staging registers): two slots are being multiplied,
// up to three are in flight, so the load path never drains at the per-step barrier.  Rows are
// 128 B and the eight 16-byte pieces of a row are XOR-swizzled with the row index so that the
// 16-byte fragment reads spread over all banks.
//
// What bounds it, and why this MFMA shape: at full load the board sits at its power cap and the clock gives way, so
// energy per multiply-add is what counts.  From registers alone, on random operands, 32x32x16 MFMAs sustain 1.79 PFLOP/s
// at 1.81 GHz and 16x16x32 ones 2.03 PFLOP/s at 2.07 GHz: per multiply-add they move half the accumulators.  They also
// take twice the instructions, so the loop is scheduled by hand (see there).  Measured on one box against the
// 32x32x16 loop it replaces: gate/up without the factors for a backward pass (43008 x 22016 x 4096) 5.40 -> 5.05 ms
// (1.44 -> 1.54 PFLOP/s; the instance of a training step, which also writes those, 5.82 -> 5.42 on other boxes), down
// (43008 x 4096 x 11008) 2.59 -> 2.45 ms (1.50 -> 1.59), dWg (4096 x 11008 over 26112 rows) 1.73 -> 1.59 ms
// (1.36 -> 1.48); with 16 workgroups on the chip, where the clock stays up and the step is issue-bound, 0.92 -> 0.94 us
// per step.
//
// The MFMA is issued with the B fragment as the first operand, so the accumulator tile is the
// transpose of the usual one: a lane holds, for one output row m, runs of 4 consecutive n.
// Epilogues therefore see 4-wide row-contiguous vectors (8-byte writes into the staging area,
// from which whole rows leave as 16-byte-per-lane stores).
#pragma once

#include <algorithm>

#include "actor.h"

namespace pcm {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;   // 16 bytes that only pass through registers
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;

// How an operand of C[m, n] = sum_k A(m, k) B(n, k) is stored.
enum OperandLayout : int {
    kRowsByK = 0,   // [rows][K]: element (row, k) at ptr[row * ld + k]
    kKByRows = 1    // [K][rows]: element (row, k) at ptr[k * ld + row]
};

constexpr int kTileM = 256, kTileN = 256, kTileK = 64;   // rows are padded to, and skipped in, units of kTileM whatever the tile
constexpr int kGemmThreads = 256;
constexpr int kNumXcd = 8;
// Two tile sizes, 32 kW x 32 kW with kW x kW MFMA tiles per wavefront: 256 (kW = 8: one workgroup per CU, its operand
// ring is the whole LDS) and 128 (kW = 4: two workgroups per CU) where the larger tile leaves CUs idle, see tile_for.
constexpr int kLargeTile = 8, kSmallTile = 4;
template <int kW> constexpr int kTile = 32 * kW;                     // rows and columns of a workgroup's tile
template <int kW> constexpr int kWaveRows = 16 * kW;                 // rows and columns of a wavefront's part of it
// Operand tiles resident or in flight in LDS: five (160 KB, the whole LDS, or 80 KB).  Launches of small tiles with at most one
// workgroup per CU have the LDS of a second one to spare and, if a workgroup has kDeepSteps steps or more, keep nine, four steps
// ahead instead of two: their steps wait for loads that no neighbour covers.  Whole steps with five / nine: 2072 rows of
// 512 -> 768 80.0 / 78.7 us, composed 1152 of 3584 -> 1024 125.5 / 121.2, 1344 of 1024 -> 1024 without gradients 42.3 / 40.2; where
// more than 256 workgroups run the neighbour is worth more and they keep five.
constexpr int kRingSlots = 5, kDeepRingSlots = 9;
template <int kW, int kSlots = kRingSlots> constexpr int kRingBytes = kSlots * kTile<kW> * kTileK * 2;
// Epilogues pass their results through LDS so that global stores are whole 128-byte lines: each
// wavefront owns a private staging area (no workgroup barrier needed; LDS operations of one
// wavefront execute in order).
template <int kW> constexpr int kWaveStageBytes = kRingBytes<kW> / 4;

struct GemmProblem {
    const bf16* A;    // M x K1 operand, leading dimension lda (layout given by the kernel's template arguments)
    const bf16* B;    // N x K1 operand, leading dimension ldb
    const bf16* A2;   // optional second reduction segment (same M, N, layouts and leading dimensions), K2 columns;
    const bf16* B2;   // when K2 == 0 both must still point at valid operands (A, B)
    int64_t lda, ldb;
    int M, N, K1, K2;  // M, N multiples of 256; K1, K2 multiples of 64
    int splits;        // reduction split (grid multiplies by it); epilogue must combine partials
    // Device-side row count: when `kept` is set, only the first min(*kept, kept_max) * rows_per_kept
    // rows of the row dimension carry data.  rows_role says which GEMM dimension that is:
    // kRowsAreM: row tiles entirely beyond the count exit at once; kRowsAreK: the reduction stops at
    // the count rounded up to a whole step (rows up to there are valid, zero-padded).
    // With row_offset the operand rows are a panel of a longer batch: the panel's live rows are the batch's live
    // rows beyond row_offset.  skip_if_empty: a workgroup whose reduction range is empty leaves without running the
    // epilogue (for epilogues that add to what is already there).
    const int32_t* kept;
    int kept_max, rows_per_kept, rows_role;
    int row_offset, skip_if_empty;
    __device__ int live_rows() const {       // kept is set
        int nk = *kept;
        nk = nk < 0 ? 0 : (nk > kept_max ? kept_max : nk);
        return max(0, nk * rows_per_kept - row_offset);
    }
    // Operands chosen on the device: when set, the first-segment operand is read from *A_sel (*B_sel) instead of A
    // (B); an earlier kernel of the same stream decides which buffer that is.  Single reduction segment only.
    const bf16* const* A_sel;
    const bf16* const* B_sel;
    // A product whose last columns go to a second launch, on small tiles (launch_row_gemm): which of the two this is.  Both
    // are given the whole product; how many columns that is (cut_columns) follows from the live rows.
    int cut;
};
enum Cut : int { kCutNone = 0, kCutHead = 1, kCutTail = 2 };
enum RowsRole : int { kRowsUnused = 0, kRowsAreM = 1, kRowsAreK = 2 };

// Accumulators of a wavefront: kW x kW tiles of 16 x 16.  Tile (i, j), register t of a lane is
//   row  m = row0() + i * 16 + (lane & 15)
//   col  n = col0() + j * 16 + 4 * (lane >> 4) + t
template <int kW>
using Accumulators = f32x4[kW][kW];
template <int kW>
struct TileCoord {
    int m0, n0, wm, wn, lane;
    int split;   // which part of a split reduction this workgroup computed
    __device__ int row0() const { return m0 + wm * kWaveRows<kW>; }
    __device__ int col0() const { return n0 + wn * kWaveRows<kW>; }
};

// f(0), f(1), .. f(kN - 1) with the number as a constant.
template <int kI>
struct Index { static constexpr int value = kI; };
template <int kN, int kI = 0, class F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (kI < kN) {
        f(Index<kI>{});
        static_for<kN, kI + 1>(f);
    }
}

__device__ inline bf16x4 to_bf16x4(float a, float b, float c, float d) {
    bf16x4 r;
    r[0] = (__bf16)a; r[1] = (__bf16)b; r[2] = (__bf16)c; r[3] = (__bf16)d;
    return r;
}

// LDS has 64 four-byte banks (256 B per cycle), so a 16-byte-per-lane read is served 16 lanes at a
// time and a 128-byte tile row covers half the banks.  [rows][K] tiles: 16 consecutive rows must
// fall on 16 different 16-byte columns of the 256-byte window, hence the XOR with row bits 1..3
// (bit 0 already selects the half window).
__device__ inline int swizzle_piece(int row, int piece) { return piece ^ ((row >> 1) & 7); }
// [K][rows] tiles (512-byte k-rows, read by transpose reads of four k-rows x 32 bytes per 16 lanes,
// 32 lanes per cycle): a k-row spans all banks twice, so the 32-byte unit alone decides the banks.  The
// four k-rows of a 16-lane group are spread by XOR with k & 3; the two groups served together read the
// same unit eight k-rows apart, hence bit 3 of k on unit bit 2.  Self-inverse for fixed k.
__device__ inline int swizzle_unit(int unit, int k) { return unit ^ (k & 3) ^ ((k >> 1) & 4); }

// Workgroup id -> (tile_m, tile_n), or false if the workgroup has no tile.  Consecutive hardware
// workgroup ids go to different XCDs (id mod 8), each with its own L2.  The live tiles are numbered
// in column-major bands of 4 row-tiles, so that 32 consecutive numbers are a block of 4 x 8 tiles
// (12 operand panels between them); such blocks are dealt to the XCDs in turn.  The 32 workgroups
// that run together on one XCD then share their panels in that XCD's L2, and the eight XCDs work
// side by side on the same band at the same time, so that a panel one of them has brought in from
// HBM is found in the memory-side cache by the others.  (Giving each XCD a contiguous range of tiles
// instead costs 3 % on the gate/up shape: the XCDs then stream eight different bands through the
// memory-side cache at once.)  Of the n_wg workgroups launched only tiles_m * tiles_n have a tile
// (the row dimension may be cut short by a device-side count); only those are numbered, so a short
// batch still spreads over all XCDs.
template <int kW>
__device__ inline bool tile_of_workgroup(int wg, int n_wg, int tiles_m, int tiles_n, int& tm, int& tn) {
    (void)n_wg;
    constexpr int kBlock = kW == kLargeTile ? 32 : 64;   // tiles per XCD block = workgroups resident on one XCD
    const int n_live = tiles_m * tiles_n;
    const int xcd = wg % kNumXcd, idx = wg / kNumXcd;
    const int full = n_live / (kBlock * kNumXcd);   // rounds in which every XCD gets a whole block
    int logical;
    if (idx < full * kBlock) logical = ((idx / kBlock) * kNumXcd + xcd) * kBlock + idx % kBlock;
    else {                                          // the rest: neighbouring tiles to the same XCD, as evenly as they go
        const int rest = n_live - full * kBlock * kNumXcd, at = idx - full * kBlock;
        if (at >= rest / kNumXcd + (xcd < rest % kNumXcd ? 1 : 0)) return false;
        logical = full * kBlock * kNumXcd + xcd * (rest / kNumXcd) + min(xcd, rest % kNumXcd) + at;
    }
    constexpr int kBand = kW == kLargeTile ? 4 : 8;
    const int band_size = kBand * tiles_n;
    const int band = logical / band_size;
    const int first = band * kBand;
    const int rows = min(tiles_m - first, kBand);
    const int in_band = logical % band_size;
    tm = first + in_band % rows;
    tn = in_band / rows;
    return true;
}

// How many 256-wide columns of a product of `live_tiles` x `tn` large tiles a launch of small tiles takes over: those that
// leave whole rounds of large tiles on the 256 CUs, if one round of small tiles (256 run side by side at the rate this is
// about) holds them.
__host__ __device__ inline int cut_columns(int live_tiles, int tn) {
    if (live_tiles <= 0) return 0;
    const int rest = live_tiles * tn % 256, columns = (rest + live_tiles - 1) / live_tiles;
    return columns < tn && 4 * live_tiles * columns <= 256 ? columns : 0;
}

#define PCM_AS_LDS(p) ((__attribute__((address_space(3))) void*)(p))
#define PCM_AS_GLOBAL(p) ((const __attribute__((address_space(1))) void*)(p))

// One wave-wide 16-byte-per-lane load from global memory straight into LDS: lane l's 16 bytes land
// at lds_addr + 16 l.  Written as inline assembly so that the compiler does not serialise the
// fragment reads of one stage behind loads into the other; completion is awaited explicitly
// (wait_direct_loads) before the barrier that publishes the stage.
__device__ inline void direct_load_16B(const char* base, uint32_t lane_offset, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :
                 : "s"(lds_addr), "v"(lane_offset), "s"(base)
                 : "memory");
}
// acc += B fragment x A fragment.  Inline assembly so that the accumulators stay in the accumulation registers: through
// the builtin the register allocator moves them back and forth.  Operands of the next MFMAs come from LDS reads (the
// compiler waits for those before it passes the registers on), never from a vector instruction right before.
__device__ __forceinline__ void mfma_16x16x32(f32x4& acc, bf16x8 b, bf16x8 a) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(b), "v"(a));
}
// The same around direct_load_16B to lds_addr + kLdsOffset: a load into LDS may not follow the write of m0 directly,
// and the MFMA is the instruction in between.
template <uint32_t kLdsOffset>
__device__ __forceinline__ void mfma_16x16x32_and_load(f32x4& acc, bf16x8 b, bf16x8 a, const char* base, uint32_t lane_offset,
                                                       uint32_t lds_addr) {
    asm volatile("s_add_u32 m0, %1, %2\n\t"
                 "v_mfma_f32_16x16x32_bf16 %0, %3, %4, %0\n\t"
                 "global_load_lds_dwordx4 %5, %6"
                 : "+a"(acc)
                 : "s"(lds_addr), "n"(kLdsOffset), "v"(b), "v"(a), "v"(lane_offset), "s"(base)
                 : "memory", "scc");
}
// Direct loads retire in issue order, so waiting until at most `newest` remain outstanding
// guarantees that all older ones have landed.
template <int kNewest>
__device__ inline void wait_direct_loads() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kNewest) : "memory");
}

// 4 bf16 of one operand row at 4 consecutive k, from a [K][rows] tile: a transpose read.  Within a group of 16 lanes the
// instruction hands lane j the j-th 16-bit element of each of the four 32-byte runs addressed by lanes
// 4 q .. 4 q + 3 (q = 0..3); the callers point run q at k-row q, so lane j receives k = 0..3 of row j.
__device__ inline s16x4 read_transposed(uint32_t lds_addr) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(uintptr_t)lds_addr);
}
__device__ inline bf16x8 join_halves(s16x4 lo, s16x4 hi) {
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// A wave-uniform address: where several products share a kernel (kShared) the compiler may lose sight of that, and assembly
// takes it in scalar registers.
template <bool kShared>
__device__ __forceinline__ const char* tile_address(const void* p) {
    if (!kShared) return static_cast<const char*>(p);
    const uint64_t at = (uint64_t)(uintptr_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)at), hi = __builtin_amdgcn_readfirstlane((uint32_t)(at >> 32));
    return reinterpret_cast<const char*>((uintptr_t)((uint64_t)hi << 32 | lo));
}

// Addresses of LDS reads, written as assembly so that they stay where the main loop puts them, a gap before the read.
__device__ __forceinline__ uint32_t fragment_address(uint32_t base, int xor_with) {
    uint32_t at;
    asm volatile("v_xor_b32 %0, %1, %2" : "=v"(at) : "i"(xor_with), "v"(base));
    return at;
}
__device__ __forceinline__ uint32_t fragment_address_sum(uint32_t lane_base, uint32_t slot) {
    uint32_t at;
    asm volatile("v_add_u32 %0, %1, %2" : "=v"(at) : "s"(slot), "v"(lane_base));
    return at;
}

// An epilogue may ask to run although the workgroup's reduction range is empty and skip_if_empty is set (it then
// sees a zero accumulator): it says so through a member runs_when_empty().
template <class E>
__device__ inline auto runs_when_empty(const E& e, int) -> decltype(e.runs_when_empty()) { return e.runs_when_empty(); }
template <class E>
__device__ inline bool runs_when_empty(const E&, long) { return false; }

// An epilogue that combines columns 64 apart (of every 128) says so through a member kPairedColumns.
template <class E>
constexpr auto paired_columns(int) -> decltype(E::kPairedColumns) { return E::kPairedColumns; }
template <class E>
constexpr bool paired_columns(long) { return false; }

template <int kW, int kSlots>
struct OperandRing {
    __attribute__((aligned(1024))) __bf16 data[kRingBytes<kW, kSlots> / 2];   // [slot][row][64]
};

// The work of workgroup `block` of a product; smem: the kernel's LDS.  kShared: one of several products of a launch.
template <int kLayA, int kLayB, bool kShared, class Epilogue, int kW, int kSlots>
__device__ __forceinline__ void gemm_tile(const GemmProblem& p, const Epilogue& epi, int block, OperandRing<kW, kSlots>& smem) {
    constexpr int TM = kTile<kW>, TN = kTile<kW>;
    constexpr uint32_t kTileBytes = TM * kTileK * 2;             // one operand tile
    constexpr int kLoadsPerTile = kW;                            // wave-wide loads per wavefront per tile
    constexpr int kSmemBytes = kRingBytes<kW, kSlots>;
    constexpr int kAhead = kSlots / 2;                           // steps requested ahead of the one being multiplied

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform, kept in a scalar register
    const int wm = wave >> 1, wn = wave & 1;
    const int tiles_m = p.M / TM;
    int tiles_n = p.N / TN, n_first = 0;
    const int n_tiles = tiles_m * tiles_n;
    const int split = block / n_tiles;
    if (kShared && split >= p.splits) return;                    // their workgroups come in multiples of eight
    int k1 = p.K1, live_m = tiles_m;
    if (p.kept != nullptr) {
        const int rows = p.live_rows();
        if (p.rows_role == kRowsAreM) live_m = min(tiles_m, (rows + kTileM - 1) / kTileM * (kTileM / TM));
        if (p.rows_role == kRowsAreK) k1 = min(k1, (rows + kTileK - 1) / kTileK * kTileK);
    }
    if (p.cut != kCutNone) {
        const int columns = cut_columns(live_m / (kTileM / TM), p.N / kTileN);
        n_first = p.cut == kCutTail ? p.N - columns * kTileN : 0;
        tiles_n = (p.cut == kCutTail ? columns : p.N / kTileN - columns) * (kTileN / TN);
    }
    int tm, tn;
    if (!tile_of_workgroup<kW>(block % n_tiles, n_tiles, live_m, tiles_n, tm, tn)) return;   // before any barrier
    const int m0 = tm * TM, n0 = n_first + tn * TN;
    // reduction range of this workgroup, in 64-wide steps over the concatenation of both segments
    const int steps1 = k1 / kTileK, steps_all = steps1 + p.K2 / kTileK;
    const int per_split = (steps_all + p.splits - 1) / p.splits;
    const int step_begin = split * per_split;
    const int step_end = min(steps_all, step_begin + per_split);

    // Global -> LDS: one wave-wide load fills 1 KB of LDS, lane l landing in 16-byte slot l; the
    // swizzle is therefore applied on the global side (the lane that lands in a slot fetches the
    // piece that belongs there).  Addresses are a wave-uniform base (tile origin + k offset) plus
    // a 32-bit per-lane byte offset.
    //   [rows][K] operand: the tile is [32 kW rows][128 B]; wave w fills rows [8 kW w, 8 kW (w + 1)), 8 rows
    //     per load; piece p of row r sits in slot swizzle_piece(r, p).
    //   [K][rows] operand: the tile is [64 k][64 kW B]; wave w fills k-rows [16 w, 16 w + 16), 16 / kW per
    //     load; the 32-byte unit u of k-row k sits in unit swizzle_unit(u, k).
    const uint32_t lds_base = (uint32_t)(uintptr_t)PCM_AS_LDS(smem.data);
    struct LoadCtx {
        const char* base;        // wave-uniform
        uint32_t off[4];         // per-lane byte offset of a load before the per-load stride, by load_variant()
        uint32_t stride;         // bytes between consecutive loads
        uint32_t dst;            // LDS byte address of this wave's part of the slot
    };
    // operand 0 = A rows m0.., operand 1 = B rows n0..  Per-lane offsets do not depend on the step; the
    // tile origin is a wave-uniform pointer that walks along k.
    uint32_t lane_off[2][4], load_stride[2];
    const char* seg_origin[2][2];          // [operand][segment]: this tile's bytes at k = 0 of the segment
    uint32_t k_step_bytes[2];              // distance between consecutive steps
#pragma unroll
    for (int operand = 0; operand < 2; ++operand) {
        const uint32_t ld = (uint32_t)(operand == 0 ? p.lda : p.ldb);
        const int row0 = operand == 0 ? m0 : n0;
        const int layout = operand == 0 ? kLayA : kLayB;
        const bf16* const* sel = operand == 0 ? p.A_sel : p.B_sel;
        const bf16* s1 = sel != nullptr ? *sel : (operand == 0 ? p.A : p.B);
        const bf16* s2 = sel != nullptr ? s1 : (operand == 0 ? p.A2 : p.B2);
        if (layout == kRowsByK) {
            const uint32_t row = (uint32_t)wave * (8u * kW) + (uint32_t)(lane >> 3);   // + 8 r for load r
#pragma unroll
            for (uint32_t var = 0; var < 4; ++var) {                                 // the swizzle uses row bit 3
                const uint32_t piece = (uint32_t)swizzle_piece((lane >> 3) + 8 * (var & 1), lane & 7);
                lane_off[operand][var] = (row * ld + piece * 8u) * 2u;
            }
            load_stride[operand] = 16u * ld;
            seg_origin[operand][0] = tile_address<kShared>(s1 + (int64_t)row0 * ld);
            seg_origin[operand][1] = tile_address<kShared>(s2 + (int64_t)row0 * ld);
            k_step_bytes[operand] = kTileK * 2;
        } else {
            constexpr int kLanes = 4 * kW;                                            // lanes per k-row
            const uint32_t krow = (uint32_t)wave * 16u + (uint32_t)(lane / kLanes);   // + (16 / kW) r for load r
#pragma unroll
            for (uint32_t var = 0; var < 4; ++var) {                                  // bits 0, 1 and 3 of the k-row
                const int k = lane / kLanes + (kW == kLargeTile ? 2 * (int)(var & 1) + 8 * (int)(var >> 1) : 8 * (int)(var & 1));
                const uint32_t piece = 2u * (uint32_t)swizzle_unit((lane % kLanes) >> 1, k) + (uint32_t)(lane & 1);
                lane_off[operand][var] = (krow * ld + piece * 8u) * 2u;
            }
            load_stride[operand] = (32u / kW) * ld;
            seg_origin[operand][0] = tile_address<kShared>(s1 + row0);
            seg_origin[operand][1] = tile_address<kShared>(s2 + row0);
            k_step_bytes[operand] = (uint32_t)kTileK * ld * 2u;
        }
    }
    auto tile_origin = [&](int operand, int step) {
        const bool seg1 = step < steps1;
        return seg_origin[operand][seg1 ? 0 : 1] + (int64_t)(seg1 ? step : step - steps1) * (int64_t)k_step_bytes[operand];
    };
    // `slot` is the byte offset of a ring slot
    auto load_ctx_at = [&](int operand, uint32_t slot, const char* origin) {
        LoadCtx c;
        c.base = origin;
#pragma unroll
        for (int var = 0; var < 4; ++var) c.off[var] = lane_off[operand][var];
        c.stride = load_stride[operand];
        c.dst = lds_base + slot + (uint32_t)wave * (kTileBytes / 4u);
        return c;
    };
    auto load_ctx = [&](int operand, uint32_t slot, int step) { return load_ctx_at(operand, slot, tile_origin(operand, step)); };
    // which of the per-lane offsets load r takes
    auto load_variant = [](int layout, int r) { return layout == kRowsByK ? r & 1 : (kW == kLargeTile ? (r & 1) | ((r >> 1) & 2) : r >> 1); };
    auto issue_tile = [&](int operand, uint32_t slot, int step) {
        const LoadCtx c = load_ctx(operand, slot, step);
#pragma unroll
        for (uint32_t r = 0; r < (uint32_t)kLoadsPerTile; ++r)
            direct_load_16B(c.base, c.off[load_variant(operand == 0 ? kLayA : kLayB, r)] + r * c.stride, c.dst + r * 1024u);
    };

    Accumulators<kW> acc;
#pragma unroll
    for (int i = 0; i < kW; ++i)
#pragma unroll
        for (int j = 0; j < kW; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Fragment registers are double-buffered: while the kW * kW MFMAs of one 32-wide k-slice run, the
    // 2 kW fragment reads of the next slice are in flight.  Fragment i = rows 16 i .. 16 i + 15 of
    // the wavefront's A or B sub-tile; lane l holds row l & 15, k = 8 (l >> 4) .. + 7 of the slice.
    bf16x8 fa[2][kW], fb[2][kW];
    // LDS address of this lane's fragment 0 of slice ks in a tile in ring slot 0.
    //   [rows][K]: one 16-byte read; fragment i is 16 rows (2 KB) further.
    //   [K][rows]: two transpose reads, the lane's run starting in k-row 8 (l >> 4) + ((l & 15) >> 2), the second four
    //     k-rows further; fragment i is unit i of the wavefront's eight and the swizzle an XOR with a number below
    //     eight, so it is at address ^ 32 i.
    auto fragment_base = [&](int layout, int sub_row0, int ks) -> uint32_t {
        if (layout == kRowsByK) {
            const int row = sub_row0 + (lane & 15);
            return lds_base + (uint32_t)(row * (kTileK * 2) + swizzle_piece(row, ks * 4 + (lane >> 4)) * 16);
        }
        const int k = (lane >> 4) * 8 + ((lane & 15) >> 2);
        return lds_base + (uint32_t)((ks * 32 + k) * (64 * kW) + (swizzle_unit(sub_row0 >> 4, k) << 5) + ((lane & 3) << 3));
    };
    // B fragment j is rows 16 j .. of the wavefront's part; with paired columns (64 columns of one kind followed by the 64
    // matching ones of another per 128, a wavefront needing both) and the small tile, half of its fragments come from each.
    constexpr bool kPaired = paired_columns<Epilogue>(0) && kW == kSmallTile;
    auto b_row = [](int j) { return kPaired ? j / (kW / 2) * 64 + j % (kW / 2) * 16 : j * 16; };
    const int b_row0 = kPaired ? wn * (kWaveRows<kW> / 2) : wn * kWaveRows<kW>;
    static_assert(!kPaired || kLayB == kRowsByK, "paired columns: rows by k only");
    const uint32_t base_a[2] = {fragment_base(kLayA, wm * kWaveRows<kW>, 0), fragment_base(kLayA, wm * kWaveRows<kW>, 1)};
    const uint32_t base_b[2] = {fragment_base(kLayB, b_row0, 0), fragment_base(kLayB, b_row0, 1)};
    constexpr uint32_t kHalfFragment = 4 * 64 * kW;
    // `at`: the address of the fragment for [K][rows] tiles; for [rows][K] tiles that of fragment 0, `row` rows before it.
    auto read_fragment = [](int layout, uint32_t at, int row) -> bf16x8 {
        if (layout == kRowsByK) return *(const __attribute__((address_space(3))) bf16x8*)(uintptr_t)(at + (uint32_t)row * 128u);
        return join_halves(read_transposed(at), read_transposed(at + kHalfFragment));
    };
    // ring slots are named by their byte offset in LDS
    auto next_slot = [](uint32_t s) { return s + kTileBytes >= (uint32_t)kSmemBytes ? s + kTileBytes - kSmemBytes : s + kTileBytes; };

    if (step_begin < step_end) {
        // Operand tiles are numbered 2 s + o (o = 0 for A, 1 for B of step s) and tile t lives in ring
        // slot t mod kSlots.  Prologue: as many tiles as there are slots (five: steps 0, 1 and the A tile of step 2) are
        // requested; steps past the end re-request the last step's tiles, which nobody reads.
        const int last = step_end - 1;
#pragma unroll
        for (int t = 0; t < kSlots; ++t) issue_tile(t & 1, (uint32_t)t * kTileBytes, min(step_begin + t / 2, last));
        wait_direct_loads<(kSlots - 2) * kLoadsPerTile>();
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kW; ++i) {
            fa[0][i] = read_fragment(kLayA, kLayA == kRowsByK ? base_a[0] : base_a[0] ^ (uint32_t)(32 * i), i * 16);
            const uint32_t at_b0 = base_b[0] + kTileBytes;
            fb[0][i] = read_fragment(kLayB, kLayB == kRowsByK ? at_b0 : at_b0 ^ (uint32_t)(32 * i), b_row(i));
        }
        // One 64-wide step per trip.  `sa`, `sb` are the slots of this step's tiles, `na`, `nb` the next step's, the two
        // after them in the ring.  Fragment set 0 holds slice 0 of this step on entry and slice 0 of the next step on
        // exit.  The single barrier sits before the second slice: by then every wavefront has issued all its reads of
        // `sa`, `sb`, so both slots can be refilled, `sa` with the B tile of step + kAhead (during the second slice) and `sb`
        // with the A tile of step + kAhead + 1 (during the next step's first).  At the barrier the next step's tiles must have
        // landed and only newer ones (of five slots, the newest A tile) may still be in flight.  The body is branch-free: near the
        // end it re-requests tiles that nobody reads.
        //
        // A wavefront issues in order and an MFMA keeps the matrix pipe busy for 16 cycles.  Measured with one wavefront
        // per SIMD: between two MFMAs one scalar instruction, two vector instructions or an LDS read cost nothing, three
        // dependent scalar ones 4 cycles, an LDS read right behind the vector instruction that makes its address 8.  The
        // order is therefore fixed by hand: per MFMA row of a slice (8 MFMAs) one refill load (16 per step: issued
        // together they would hold the texture path for about 1000 cycles) and, in the first six rows, up to three
        // fragment reads of the next slice, with their addresses made at least one MFMA earlier.  The last two rows have
        // no reads, so that the reads of a slot have long landed when the barrier that frees the slot waits for them;
        // they carry the scalar bookkeeping of the tile pointers, a few instructions per gap.
        //
        // (The small tile has two workgroups per CU to fill each other's gaps; its rows are 4 MFMAs, the first three carry
        // a fragment read per gap.)
        //
        // Fragments of the next slice are read in the order its MFMAs need them: A0, B0, B1, .., A1, A2, ..
        auto is_a = [](int n) { return n == 0 || n > kW; };
        auto fragment_of = [&](int n) { return n == 0 ? 0 : (n <= kW ? n - 1 : n - kW); };
        // The kW * kW MFMAs of a slice walk the tiles in serpentine order, so that consecutive
        // instructions always share one operand fragment.
        // refilled: the operand whose tile is refilled meanwhile, c: from and to where; rd_a, rd_b: bases of the fragments of
        // the next slice.
        auto slice = [&](int set, auto refilled, const LoadCtx& c, uint32_t rd_a, uint32_t rd_b, auto hook) {
            uint32_t tr_at = rd_a;       // [K][rows]: address of the fragment being read
            s16x4 tr_lo = {0, 0, 0, 0};  // [K][rows]: its first half
            auto transposed = [&](int n) { return is_a(n) ? kLayA == kKByRows : kLayB == kKByRows; };
            auto read_rows = [&](int n) {                      // [rows][K]: read n
                const int f = fragment_of(n);
                if (is_a(n)) fa[set ^ 1][f] = read_fragment(kLayA, rd_a, f * 16);
                else fb[set ^ 1][f] = read_fragment(kLayB, rd_b, b_row(f));
            };
            auto read_low = [&] { tr_lo = read_transposed(tr_at); };
            auto read_high = [&](int n) {
                (is_a(n) ? fa : fb)[set ^ 1][fragment_of(n)] = join_halves(tr_lo, read_transposed(tr_at + kHalfFragment));
            };
            auto next_address = [&](int n) {                   // [K][rows]: of read n
                if (n < 2 * kW && transposed(n)) tr_at = fragment_address(is_a(n) ? rd_a : rd_b, 32 * fragment_of(n));
            };
            static_for<kW>([&](auto row) __attribute__((always_inline)) {
                constexpr int g = decltype(row)::value;
                constexpr int j0 = (g & 1) ? kW - 1 : 0;
                constexpr int layout = decltype(refilled)::value == 0 ? kLayA : kLayB;
                mfma_16x16x32_and_load<g * 1024u>(acc[g][j0], fb[set][j0], fa[set][g], c.base,
                                                  c.off[load_variant(layout, g)] + g * c.stride, c.dst);
#pragma unroll
                for (int jj = 1; jj < kW; ++jj) {
                    const int j = (g & 1) ? kW - 1 - jj : jj;
                    mfma_16x16x32(acc[g][j], fb[set][j], fa[set][g]);
                    __builtin_amdgcn_sched_barrier(0);
                    if (kW == kLargeTile) {
                        // read n of the next slice: [rows][K] in gap jj, [K][rows] in halves in gaps jj and jj + 1 with the
                        // address of the next one made behind the second (behind the last one of a row in gap 7)
                        const int n = 3 * g + (jj - 1) / 2;
                        if (g < 6 && jj < 7 && n < 2 * kW) {
                            if (!transposed(n)) { if (jj & 1) read_rows(n); }
                            else if (jj & 1) read_low();
                            else read_high(n);
                        }
                        if (g < 6 && (jj == 2 || jj == 4 || jj == 7)) next_address(3 * g + jj / 2);
                        if (g >= 6 && !(jj & 1)) hook(3 * (g - 6) + jj / 2 - 1);
                    } else {
                        const int n = 3 * g + jj - 1;
                        if (g < 3 && n < 2 * kW) {
                            if (!transposed(n)) read_rows(n);
                            else { read_low(); read_high(n); }
                            next_address(n + 1);
                        }
                        if (g == 3) { hook(2 * jj - 2); hook(2 * jj - 1); }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            });
        };
        // Tile streams: origin of the newest tile requested so far of each operand.  On entry of a step the newest A
        // tile is that of step + kAhead (its loads are those of the first slice: on the first trip a harmless second request),
        // the newest B tile one step before that; the first slice then moves each on by one step.  Past `last` an origin
        // stands still, or lands once on the start of the second segment, which is valid memory whether or not that
        // segment is used.
        const char* origin_a = tile_origin(0, min(step_begin + kAhead, last));
        const char* origin_b = tile_origin(1, min(step_begin + kAhead - 1, last));
        uint32_t sa = 0, sb = next_slot(sa), refill_a = (kSlots - 1) * kTileBytes, na = next_slot(sb), nb = next_slot(na);
        uint32_t rd_a = base_a[1] + sa, rd_b = base_b[1] + sb, stride_now = 0;
        // In six pieces of two or three scalar instructions; the A origin only after the last load from it.
        auto between_a = [&](int step, int piece) {
            const int operand = piece < 3 ? 1 : 0;
            const int at = step + kAhead + (operand == 0 ? 1 : 0);
            const char*& origin = operand == 0 ? origin_a : origin_b;
            if (piece % 3 == 0) {
                stride_now = at <= last ? k_step_bytes[operand] : 0u;
                if (piece == 0) rd_a = fragment_address_sum(base_a[0], na);
                else rd_b = fragment_address_sum(base_b[0], nb);
            } else if (piece % 3 == 1) {
                origin += stride_now;
            } else {
                origin = at == steps1 ? seg_origin[operand][1] : origin;
            }
        };
        auto between_b = [&](int piece) {
            if (piece == 0) rd_a = fragment_address_sum(base_a[1], na);
            else if (piece == 1) rd_b = fragment_address_sum(base_b[1], nb);
            else if (piece == 2) refill_a = sb;
            else if (piece == 3) sa = na;
            else if (piece == 4) na = next_slot(sb = nb);
            else nb = next_slot(na);
        };
        for (int step = step_begin; step < step_end; ++step) {
            slice(0, Index<0>{}, load_ctx_at(0, refill_a, origin_a), rd_a, rd_b, [&](int piece) { between_a(step, piece); });
            wait_direct_loads<(kSlots - 4) * kLoadsPerTile>();
            __syncthreads();
            slice(1, Index<1>{}, load_ctx_at(1, sa, origin_b), rd_a, rd_b, between_b);   // tile 2 s + kSlots -> slot of tile 2 s
        }
        wait_direct_loads<0>();
        // the last MFMAs' results: the compiler does not know how long inline assembly takes to write them
        asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
        __syncthreads();
    }

    if (p.skip_if_empty && step_begin >= step_end && !runs_when_empty(epi, 0)) return;   // nothing to add (uniform over the workgroup)
    const TileCoord<kW> tc{m0, n0, wm, wn, lane, split};
    epi(tc, acc, reinterpret_cast<char*>(smem.data));
}

template <class Epilogue, int kLayA, int kLayB, int kW, int kSlots = kRingSlots>
__global__ __launch_bounds__(kGemmThreads, kW == kLargeTile || kSlots > kRingSlots ? 1 : 2) void gemm_bf16(GemmProblem p, Epilogue epi) {
    __shared__ OperandRing<kW, kSlots> smem;
    gemm_tile<kLayA, kLayB, false>(p, epi, blockIdx.x, smem);
}

// Products that depend on the same launches and not on one another, as one launch: the workgroups of one fill the CUs that
// another leaves idle (its last, part-filled round, or all through where it has few tiles), its reductions need fewer parts to
// fill the chip, and of a small head a launch takes as long to begin and end as its products do.  Figures at BackwardPlan.
template <int kLayA, int kLayB, class Epilogue>
struct GemmJob {
    GemmProblem p;
    Epilogue epi;
    int first;                   // its first workgroup, a multiple of eight (see tile_of_workgroup)
    int workgroups(int tile) const { return p.M / tile * (p.N / tile) * p.splits; }
    template <int kW, int kSlots>
    __device__ __forceinline__ void run(int block, OperandRing<kW, kSlots>& smem) const {
        gemm_tile<kLayA, kLayB, true>(p, epi, block - first, smem);
    }
};
// Two products of the same A and sizes with a right operand and a result each.
template <int kLayA, int kLayB, class Epilogue>
struct GemmPairJob {
    GemmProblem p;
    const bf16* B[2];
    Epilogue epi[2];
    int first, each;             // workgroups of one product, a multiple of eight
    int workgroups(int tile) {
        each = ceil_div(p.M / tile * (p.N / tile) * p.splits, kNumXcd) * kNumXcd;
        return 2 * each;
    }
    template <int kW, int kSlots>
    __device__ __forceinline__ void run(int block, OperandRing<kW, kSlots>& smem) const {
        const bool second = block - first >= each;
        GemmProblem q = p;
        q.B = q.B2 = second ? B[1] : B[0];       // (an index instead of the choice would put the pair into scratch memory)
        gemm_tile<kLayA, kLayB, true>(q, epi[0].or_second(second, epi[1]), block - first - (second ? each : 0), smem);
    }
};
// The last job whose first workgroup is not beyond `block` runs it.
template <class Ring, class Job>
__device__ __forceinline__ void run_job(int block, Ring& smem, const Job& job) { job.run(block, smem); }
template <class Ring, class Job, class Next, class... More>
__device__ __forceinline__ void run_job(int block, Ring& smem, const Job& job, const Next& next, const More&... more) {
    if (block < next.first) job.run(block, smem);
    else run_job(block, smem, next, more...);
}
template <int kW, int kSlots, class... Jobs>
__global__ __launch_bounds__(kGemmThreads, kW == kLargeTile || kSlots > kRingSlots ? 1 : 2) void gemm_group(Jobs... jobs) {
    __shared__ OperandRing<kW, kSlots> smem;
    const int block = blockIdx.x;
    run_job(block, smem, jobs...);
}

// ---- epilogues -------------------------------------------------------------------------------

// 1 / (1 + e^-x) with the hardware exponential and reciprocal (about 1 ulp each; the results are
// rounded to bf16 afterwards).
__device__ inline float fast_sigmoid(float x) { return __builtin_amdgcn_rcpf(1.f + __expf(-x)); }

template <int kW>
__device__ inline char* wave_stage(const TileCoord<kW>& tc, char* lds) {
    return lds + (tc.wm * 2 + tc.wn) * kWaveStageBytes<kW>;
}

// Writes bf16 of four consecutive columns per lane for the 16-column tiles 0 .. kN - 1 of one tile row into a
// staging area whose rows are `stride` bytes apart.  The 32 lanes served together write
// 16 rows x 16 bytes, so a stride of 16 bytes times an odd number spreads them over all banks.
template <int kN, class F>
__device__ inline void stage_tile_row(char* stage, int stride, int lane, int local_row, F value) {
#pragma unroll
    for (int jj = 0; jj < kN; ++jj) {
        const f32x4 v = value(jj);
        *reinterpret_cast<bf16x4*>(stage + local_row * stride + (jj * 16 + 4 * (lane >> 4)) * 2) = to_bf16x4(v[0], v[1], v[2], v[3]);
    }
}

// Staging area -> global memory, 16 bytes per lane: kRowBytes / 16 lanes cover one row, so a pass moves
// 1024 / kRowBytes rows and a 16-lane group writes whole 128-byte lines.  `dst` is this lane's address
// in row 0; rows at and beyond n_rows (wave-uniform) are not written.
template <int kRows, int kRowBytes>
__device__ inline void copy_rows_out(const char* st, int stride, char* dst, int64_t ld_bytes, int n_rows, int lane) {
    constexpr int kLanesPerRow = kRowBytes / 16, kRowsPerPass = 64 / kLanesPerRow;
    const char* src = st + (lane / kLanesPerRow) * stride + (lane % kLanesPerRow) * 16;
    char* out = dst + (lane / kLanesPerRow) * ld_bytes + (lane % kLanesPerRow) * 16;
    const int64_t out_step = kRowsPerPass * ld_bytes;
    if (n_rows >= kRows) {
#pragma unroll 8
        for (int pass = 0; pass < kRows / kRowsPerPass; ++pass) {
            *reinterpret_cast<u32x4*>(out) = *reinterpret_cast<const u32x4*>(src);
            src += kRowsPerPass * stride;
            out += out_step;
        }
    } else {
        int r = lane / kLanesPerRow;
        for (int pass = 0; pass < kRows / kRowsPerPass && pass * kRowsPerPass < n_rows; ++pass) {
            if (r < n_rows) *reinterpret_cast<u32x4*>(out) = *reinterpret_cast<const u32x4*>(src);
            src += kRowsPerPass * stride;
            out += out_step;
            r += kRowsPerPass;
        }
    }
}
// The same for fp32 rows that are added to what global memory holds (16 bytes = 4 floats per lane).
template <int kRows, int kRowBytes>
__device__ inline void add_rows_out(char* st, int stride, char* dst, int64_t ld_bytes, int lane) {
    constexpr int kLanesPerRow = kRowBytes / 16, kRowsPerPass = 64 / kLanesPerRow;
    char* src = st + (lane / kLanesPerRow) * stride + (lane % kLanesPerRow) * 16;
    char* out = dst + (lane / kLanesPerRow) * ld_bytes + (lane % kLanesPerRow) * 16;
    const int64_t out_step = kRowsPerPass * ld_bytes;
#pragma unroll 8
    for (int pass = 0; pass < kRows / kRowsPerPass; ++pass) {
        const f32x4 add = *reinterpret_cast<const f32x4*>(src);
        f32x4 cur = *reinterpret_cast<const f32x4*>(out);
        cur += add;
        *reinterpret_cast<f32x4*>(out) = cur;
        *reinterpret_cast<f32x4*>(src) = cur;      // the staging area now holds what was written (see staged_sum_of_squares)
        src += kRowsPerPass * stride;
        out += out_step;
    }
}
// Sum of the squares of the kRows fp32 rows in the staging area, this lane's share (the 16 bytes per pass that
// copy_rows_out / add_rows_out move), in fp64: squares of large fp32 values leave the fp32 range.
template <int kRows, int kRowBytes>
__device__ inline double staged_sum_of_squares(const char* st, int stride, int lane) {
    constexpr int kLanesPerRow = kRowBytes / 16, kRowsPerPass = 64 / kLanesPerRow;
    const char* src = st + (lane / kLanesPerRow) * stride + (lane % kLanesPerRow) * 16;
    double sq = 0.0;
#pragma unroll 1
    for (int pass = 0; pass < kRows / kRowsPerPass; ++pass) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(src);
        sq += (double)v[0] * (double)v[0] + (double)v[1] * (double)v[1] + (double)v[2] * (double)v[2] + (double)v[3] * (double)v[3];
        src += kRowsPerPass * stride;
    }
    return sq;
}
// Global memory -> staging area, the mirror image of copy_rows_out (all kRows rows), in two halves so
// that the loads can be in flight while other work runs: fetch_rows issues them into registers,
// stash_rows writes the registers to the staging area.
template <int kRows, int kRowBytes>
struct RowFetch {
    static constexpr int kLanesPerRow = kRowBytes / 16, kRowsPerPass = 64 / kLanesPerRow, kPasses = kRows / kRowsPerPass;
    u32x4 r[kPasses];
    __device__ __forceinline__ void fetch_rows(const char* src_row0, int64_t ld_bytes, int lane) {
        // a wave-uniform row address plus a 32-bit lane offset: one address register for all passes
        const uint32_t at = (uint32_t)(lane / kLanesPerRow) * (uint32_t)ld_bytes + (uint32_t)(lane % kLanesPerRow) * 16u;
#pragma unroll
        for (int pass = 0; pass < kPasses; ++pass)
            r[pass] = *reinterpret_cast<const u32x4*>(src_row0 + pass * kRowsPerPass * ld_bytes + at);
    }
    // The same with the rows given by number: rows[pass] is the row of a matrix (whose row 0, at this wavefront's
    // columns, is src_col0) that this lane fetches in that pass; a negative number stands for a row of zeros.
    __device__ __forceinline__ void fetch_rows_at(const char* src_col0, int64_t ld_bytes, const int (&rows)[kPasses], int lane) {
        const char* in = src_col0 + (lane % kLanesPerRow) * 16;
#pragma unroll
        for (int pass = 0; pass < kPasses; ++pass)
            r[pass] = rows[pass] >= 0 ? *reinterpret_cast<const u32x4*>(in + (int64_t)rows[pass] * ld_bytes)
                                      : u32x4{0, 0, 0, 0};
    }
    __device__ __forceinline__ void stash_rows(char* st, int stride, int lane) const {
        char* dst = st + (lane / kLanesPerRow) * stride + (lane % kLanesPerRow) * 16;
#pragma unroll
        for (int pass = 0; pass < kPasses; ++pass) *reinterpret_cast<u32x4*>(dst + pass * kRowsPerPass * stride) = r[pass];
    }
};
// copy_rows_out with the destination rows given by number (row i of the staging area goes to row rows[i] of the
// matrix whose row 0, at this wavefront's columns, is dst_col0; negative: not written).
template <int kRows, int kRowBytes>
__device__ inline void copy_rows_out_at(const char* st, int stride, char* dst_col0, int64_t ld_bytes, const int32_t* rows,
                                        int lane) {
    constexpr int kLanesPerRow = kRowBytes / 16, kRowsPerPass = 64 / kLanesPerRow;
    const char* src = st + (lane / kLanesPerRow) * stride + (lane % kLanesPerRow) * 16;
    char* out = dst_col0 + (lane % kLanesPerRow) * 16;
#pragma unroll 8
    for (int pass = 0; pass < kRows / kRowsPerPass; ++pass) {
        const int row = rows[lane / kLanesPerRow + pass * kRowsPerPass];
        if (row >= 0) *reinterpret_cast<u32x4*>(out + (int64_t)row * ld_bytes) = *reinterpret_cast<const u32x4*>(src);
        src += kRowsPerPass * stride;
    }
}

// C (bf16, row-major) = acc; rows at and beyond row_limit are not written.
struct EpiStoreBf16 {
    bf16* C;
    int64_t ldc;
    int row_limit;
    template <int kW>
    __device__ __forceinline__ void operator()(const TileCoord<kW>& tc, const Accumulators<kW>& acc, char* lds) const {
        constexpr int RW = kWaveRows<kW>;                  // rows and columns of the wavefront's block
        constexpr int kStride = RW * 2 + 16;
        char* st = wave_stage(tc, lds);
#pragma unroll
        for (int i = 0; i < kW; ++i) {
            stage_tile_row<kW>(st, kStride, tc.lane, i * 16 + (tc.lane & 15), [&](int j) { return acc[i][j]; });
            __builtin_amdgcn_sched_barrier(0);   // one tile row's conversions at a time: all at once spill
        }
        __builtin_amdgcn_wave_barrier();
        const int row_base = tc.row0(), col_base = tc.col0();
        copy_rows_out<RW, RW * 2>(st, kStride, reinterpret_cast<char*>(C + (int64_t)row_base * ldc + col_base), ldc * 2,
                                row_limit - row_base, tc.lane);
    }
};

// Rows of acc written to the rows of C (bf16, row-major) that row_idx names: row m of the product goes to row
// row_idx[m]; negative entries are not written.
struct EpiScatterBf16 {
    bf16* C;
    int64_t ldc;
    const int32_t* row_idx;
    template <int kW>
    __device__ __forceinline__ void operator()(const TileCoord<kW>& tc, const Accumulators<kW>& acc, char* lds) const {
        constexpr int RW = kWaveRows<kW>;                  // rows and columns of the wavefront's block
        constexpr int kStride = RW * 2 + 16;
        char* st = wave_stage(tc, lds);
#pragma unroll
        for (int i = 0; i < kW; ++i) {
            stage_tile_row<kW>(st, kStride, tc.lane, i * 16 + (tc.lane & 15), [&](int j) { return acc[i][j]; });
            __builtin_amdgcn_sched_barrier(0);   // one tile row's conversions at a time: all at once spill
        }
        __builtin_amdgcn_wave_barrier();
        const int row_base = tc.row0(), col_base = tc.col0();
        copy_rows_out_at<RW, RW * 2>(st, kStride, reinterpret_cast<char*>(C + col_base), ldc * 2, row_idx + row_base, tc.lane);
    }
};

// C (row-major) = acc as the sum of two bf16 matrices: hi = bf16(acc), lo = bf16(acc - hi), which together
// carry 16 bits of significand.  A following product that reads [hi | lo] as two reduction segments against the
// same second operand sees the value to about 2^-17 instead of 2^-9.  Rows at and beyond row_limit are not written.
struct EpiStoreBf16Split {
    bf16 *hi, *lo;
    int64_t ldc;
    int row_limit;
    template <int kW>
    __device__ __forceinline__ void operator()(const TileCoord<kW>& tc, const Accumulators<kW>& acc, char* lds) const {
        constexpr int RW = kWaveRows<kW>;                  // rows and columns of the wavefront's block
        constexpr int kStride = RW * 4 + 16;               // [hi | lo] bf16 + 16 bytes
        char* st = wave_stage(tc, lds);
        const int col_base = tc.col0();
#pragma unroll
        for (int half = 0; half < RW / 64; ++half) {       // 64 rows per pass
#pragma unroll
            for (int ii = 0; ii < 4; ++ii) {
                const int i = half * 4 + ii;
                char* row = st + (ii * 16 + (tc.lane & 15)) * kStride;
#pragma unroll
                for (int j = 0; j < kW; ++j) {
                    float r[4];
                    bf16x4 h;
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const float x = acc[i][j][t];
                        h[t] = (__bf16)x;
                        r[t] = x - (float)h[t];
                    }
                    char* at = row + (j * 16 + 4 * (tc.lane >> 4)) * 2;
                    *reinterpret_cast<bf16x4*>(at) = h;
                    *reinterpret_cast<bf16x4*>(at + RW * 2) = to_bf16x4(r[0], r[1], r[2], r[3]);
                }
            }
            __builtin_amdgcn_wave_barrier();
            const int row_base = tc.row0() + half * 64;
            const int64_t at = (int64_t)row_base * ldc + col_base;
            copy_rows_out<64, RW * 2>(st, kStride, reinterpret_cast<char*>(hi + at), ldc * 2, row_limit - row_base, tc.lane);
            copy_rows_out<64, RW * 2>(st + RW * 2, kStride, reinterpret_cast<char*>(lo + at), ldc * 2, row_limit - row_base, tc.lane);
            __builtin_amdgcn_wave_barrier();
        }
    }
};

// C (fp32, row-major) = acc.  With a split reduction, part s goes to C + s * split_stride (its own
// M x N matrix; the caller sums the parts), so no atomics are needed and the sum is reproducible.
// accumulate: C += acc instead (a batch processed in row panels adds every panel's weight gradient).
// sumsq_parts (unsplit outputs with ldc = N only): on the final panel every wavefront also writes the sum of the
// squares of the values it leaves in C to sumsq_parts[4 * tile + wavefront] (for the gradient norm of the optimizer
// step, which then needs no pass of its own over the gradients).
struct EpiStoreF32 {
    float* C;
    int64_t ldc;
    int64_t split_stride;
    int accumulate;
    double* sumsq_parts;
    FinalPanel final_panel;
    __device__ bool runs_when_empty() const { return sumsq_parts != nullptr && final_panel(); }
    // This one or `other`, which differs in where it stores.
    __device__ EpiStoreF32 or_second(bool second, const EpiStoreF32& other) const {
        return EpiStoreF32{second ? other.C : C, ldc, split_stride, accumulate, second ? other.sumsq_parts : sumsq_parts, final_panel};
    }
    template <int kW>
    __device__ __forceinline__ void operator()(const TileCoord<kW>& tc, const Accumulators<kW>& acc, char* lds) const {
        constexpr int RW = kWaveRows<kW>;                  // rows and columns of the wavefront's block
        float* const C = this->C + tc.split * split_stride;
        constexpr int kStride = RW * 4 + 16;               // conflict-free 16-byte accesses
        char* st = wave_stage(tc, lds);
        const int col_base = tc.col0();
        const bool want_sq = sumsq_parts != nullptr && final_panel();
        double sq = 0.0;
#pragma unroll
        for (int i = 0; i < RW / 32; ++i) {                // 32 rows per pass
#pragma unroll
            for (int ii = 0; ii < 2; ++ii)
#pragma unroll
                for (int j = 0; j < kW; ++j)
                    *reinterpret_cast<f32x4*>(st + (ii * 16 + (tc.lane & 15)) * kStride + (j * 16 + 4 * (tc.lane >> 4)) * 4) =
                        acc[2 * i + ii][j];
            __builtin_amdgcn_wave_barrier();
            const int row_base = tc.row0() + i * 32;
            char* const dst = reinterpret_cast<char*>(C + (int64_t)row_base * ldc + col_base);
            if (accumulate) add_rows_out<32, RW * 4>(st, kStride, dst, ldc * 4, tc.lane);
            else copy_rows_out<32, RW * 4>(st, kStride, dst, ldc * 4, 32, tc.lane);
            if (want_sq) sq += staged_sum_of_squares<32, RW * 4>(st, kStride, tc.lane);
            __builtin_amdgcn_wave_barrier();
        }
        if (want_sq) {
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) sq += __shfl_xor(sq, o, 64);
            const int tile = (tc.m0 / kTile<kW>) * (int)(ldc / kTile<kW>) + tc.n0 / kTile<kW>;
            if (tc.lane == 0) sumsq_parts[tile * 4 + tc.wm * 2 + tc.wn] = sq;
        }
    }
};

// Gate/up projection with the activation fused: the B operand holds, per 128 packed rows, 64 gate
// columns followed by the 64 up columns of the same index range, and the first half of a wavefront's tiles j
// are u (gate), the second half the matching v (up) (see paired_columns).  Writes a = silu(u) * v (bf16, [M, ff]) and, for
// a backward pass to come, the two factors it will need, computed here where the sigmoid is at
// hand: fu = v * silu'(u) (so du = da * fu) and fv = silu(u) (so dv = da * fv).
// With kKeepLow the rounding remainder of a is written as well (a_lo = bf16(a - bf16(a))), for products
// that need the activation to more than bf16 precision (they read [a | a_lo] as two reduction segments).
template <bool kKeepFactors, bool kKeepLow = false>
struct EpiSwigluForward {
    static constexpr bool kPairedColumns = true;
    bf16 *fu, *fv, *a, *a_lo;
    int64_t ld;
    template <int kW>
    __device__ __forceinline__ void operator()(const TileCoord<kW>& tc, const Accumulators<kW>& acc, char* lds) const {
        constexpr int RW = kWaveRows<kW>;                  // rows and columns of the wavefront's block
        constexpr int CW = RW / 2;                         // columns of the activation in this wavefront's block
        // staged row: [a | fu | fv | a_lo] bf16 (the parts that are kept) + 16 bytes
        constexpr int kPart = CW * 2, kLowAt = kKeepFactors ? 3 * kPart : kPart;
        constexpr int kStride = 16 + kPart * (1 + (kKeepFactors ? 2 : 0) + (kKeepLow ? 1 : 0));
        char* st = wave_stage(tc, lds);
        const int col_base = tc.n0 / 2 + tc.wn * CW;
#pragma unroll
        for (int half = 0; half < RW / 64; ++half) {       // 64 rows per pass
#pragma unroll
            for (int ii = 0; ii < 4; ++ii) {
                const int i = half * 4 + ii;
                char* row = st + (ii * 16 + (tc.lane & 15)) * kStride;
#pragma unroll
                for (int j = 0; j < kW / 2; ++j) {
                    float av[4], fuv[4], fvv[4];
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const float x = acc[i][j][t], y = acc[i][j + kW / 2][t];
                        const float sg = kKeepLow ? 1.f / (1.f + expf(-x)) : fast_sigmoid(x);   // full accuracy where it is kept
                        fvv[t] = x * sg;
                        av[t] = fvv[t] * y;
                        const float ys = y * sg;
                        fuv[t] = __builtin_fmaf(ys, x - fvv[t], ys);     // y sg (1 + x (1 - sg))
                    }
                    char* at = row + (j * 16 + 4 * (tc.lane >> 4)) * 2;
                    const bf16x4 a4 = to_bf16x4(av[0], av[1], av[2], av[3]);
                    *reinterpret_cast<bf16x4*>(at) = a4;
                    if (kKeepFactors) {
                        *reinterpret_cast<bf16x4*>(at + kPart) = to_bf16x4(fuv[0], fuv[1], fuv[2], fuv[3]);
                        *reinterpret_cast<bf16x4*>(at + 2 * kPart) = to_bf16x4(fvv[0], fvv[1], fvv[2], fvv[3]);
                    }
                    if (kKeepLow)
                        *reinterpret_cast<bf16x4*>(at + kLowAt) = to_bf16x4(av[0] - (float)a4[0], av[1] - (float)a4[1],
                                                                         av[2] - (float)a4[2], av[3] - (float)a4[3]);
                }
            }
            __builtin_amdgcn_wave_barrier();
            const int row_base = tc.row0() + half * 64;
            const int64_t at = (int64_t)row_base * ld + col_base;     // 64 rows x CW columns of each output
            copy_rows_out<64, kPart>(st, kStride, reinterpret_cast<char*>(a + at), ld * 2, 64, tc.lane);
            if (kKeepFactors) {
                copy_rows_out<64, kPart>(st + kPart, kStride, reinterpret_cast<char*>(fu + at), ld * 2, 64, tc.lane);
                copy_rows_out<64, kPart>(st + 2 * kPart, kStride, reinterpret_cast<char*>(fv + at), ld * 2, 64, tc.lane);
            }
            if (kKeepLow) copy_rows_out<64, kPart>(st + kLowAt, kStride, reinterpret_cast<char*>(a_lo + at), ld * 2, 64, tc.lane);
            __builtin_amdgcn_wave_barrier();
        }
    }
};

// acc = da.  du = da * fu, dv = da * fv (bf16, [M, ff]; the factors are those written by the forward epilogue).
// kIndexed = false: in place, fu <- du, fv <- dv.  kIndexed = true: the rows of the product are a selection of the
// rows the forward pass ran over: product row m takes its factors from row row_idx[m] of fu, fv (negative: a row of
// zeros) and writes row m of du, dv (other buffers).  Works through the wavefront's block in passes of
// 32 rows; the rows of the next pass are fetched into registers while the current pass is computed.
template <bool kIndexed>
struct EpiSwigluBackward {
    bf16 *fu, *fv;
    int64_t ld;
    const int32_t* row_idx;
    bf16 *du, *dv;
    template <int kW>
    __device__ __forceinline__ void operator()(const TileCoord<kW>& tc, const Accumulators<kW>& acc, char* lds) const {
        constexpr int RW = kWaveRows<kW>;                  // rows and columns of the wavefront's block
        constexpr int kStride = RW * 4 + 16;               // [du | dv] bf16 + 16 bytes
        char* st = wave_stage(tc, lds);
        const int row_base = tc.row0(), col_base = tc.col0();
        const int64_t ld_bytes = ld * 2;
        const int64_t at = (kIndexed ? 0 : (int64_t)row_base * ld) + col_base;
        const char* const u0 = reinterpret_cast<const char*>(fu + at);
        const char* const v0 = reinterpret_cast<const char*>(fv + at);
        char* const du0 = reinterpret_cast<char*>((kIndexed ? du : fu) + (int64_t)row_base * ld + col_base);
        char* const dv0 = reinterpret_cast<char*>((kIndexed ? dv : fv) + (int64_t)row_base * ld + col_base);
        // the row numbers of this wavefront's block, one or two per lane; a pass hands them to the lanes that fetch the rows
        int idx_lo = 0, idx_hi = 0;
        if (kIndexed) {
            idx_lo = row_idx[row_base + tc.lane];
            if (RW > 64) idx_hi = row_idx[row_base + 64 + tc.lane];
        }
        using Fetch = RowFetch<32, RW * 2>;
        Fetch ru, rv;
        auto fetch = [&](int pass) __attribute__((always_inline)) {
            if (kIndexed) {
                int rows[Fetch::kPasses];
#pragma unroll
                for (int q = 0; q < Fetch::kPasses; ++q)
                    rows[q] = __shfl(pass < 2 ? idx_lo : idx_hi,
                                     (pass & 1) * 32 + tc.lane / Fetch::kLanesPerRow + q * Fetch::kRowsPerPass, 64);
                ru.fetch_rows_at(u0, ld_bytes, rows, tc.lane);
                rv.fetch_rows_at(v0, ld_bytes, rows, tc.lane);
            } else {
                ru.fetch_rows(u0 + pass * 32 * ld_bytes, ld_bytes, tc.lane);
                rv.fetch_rows(v0 + pass * 32 * ld_bytes, ld_bytes, tc.lane);
            }
        };
        fetch(0);
#pragma unroll
        for (int i = 0; i < RW / 32; ++i) {                // 32 rows per pass
            ru.stash_rows(st, kStride, tc.lane);
            rv.stash_rows(st + RW * 2, kStride, tc.lane);
            if (i < RW / 32 - 1) fetch(i + 1);
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int ii = 0; ii < 2; ++ii)
#pragma unroll
                for (int j = 0; j < kW; ++j) {
                    const int col = j * 16 + 4 * (tc.lane >> 4);
                    char* pu = st + (ii * 16 + (tc.lane & 15)) * kStride + col * 2;
                    char* pv = pu + RW * 2;
                    const bf16x4 u4 = *reinterpret_cast<const bf16x4*>(pu);
                    const bf16x4 v4 = *reinterpret_cast<const bf16x4*>(pv);
                    const f32x4 g = acc[2 * i + ii][j];
                    float gu[4], gv[4];
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        gu[t] = g[t] * (float)u4[t];
                        gv[t] = g[t] * (float)v4[t];
                    }
                    *reinterpret_cast<bf16x4*>(pu) = to_bf16x4(gu[0], gu[1], gu[2], gu[3]);
                    *reinterpret_cast<bf16x4*>(pv) = to_bf16x4(gv[0], gv[1], gv[2], gv[3]);
                    if (j & 1) __builtin_amdgcn_sched_barrier(0);   // two tiles at a time: beside the fetched rows more spill
                }
            __builtin_amdgcn_wave_barrier();
            copy_rows_out<32, RW * 2>(st, kStride, du0 + i * 32 * ld_bytes, ld_bytes, 32, tc.lane);
            copy_rows_out<32, RW * 2>(st + RW * 2, kStride, dv0 + i * 32 * ld_bytes, ld_bytes, 32, tc.lane);
            __builtin_amdgcn_wave_barrier();
        }
    }
};

// The tile for a product of M x N: a CU's time is the number of its tiles times what one takes.  A 64-wide step takes
// 0.94 us with the large tile (the matrix pipe) and 0.46 us with the small one, not a quarter: it brings in 32 KB for a
// quarter of the products, and the path from L2 into LDS carries about 70 GB/s per CU.  So the small tile pays where the
// large ones are few: measured, large against small, 2072 rows at 512 -> 768 (54 tiles) 19.9 / 10.2 us, 672 x 4096 x 11008
// (48 tiles) 181 / 116 us, 5376 x 4096 x 11008 (336 tiles) 261 / 416 us.
inline int tile_for(int64_t M, int64_t N, int splits) {
    const int64_t large = (M / kTileM) * (N / kTileN) * splits;
    const double cost_large = 0.94 * (double)((large + 255) / 256), cost_small = 0.46 * (double)((4 * large + 255) / 256);
    return cost_small < cost_large ? kSmallTile : kLargeTile;
}

// Steps of a part from which the deep ring pays: shorter ones are all requested at the start, and the first tile waits behind
// nine.  Whole passes, always / from 9 steps / never: 32 rows of 512 -> 512 30.4 / 29.4 / 29.4 us, 2072 of 512 -> 768 78.6 / 78.3 /
// 79.8, 1344 of 1024 -> 1024 39.4 / 39.6 / 42.0, 512 of 3072 -> 1536 145.7 / 145.4 / 150.7.
constexpr int kDeepSteps = 9;
inline int steps_per_part(const GemmProblem& p) { return ceil_div((p.K1 + p.K2) / kTileK, p.splits); }

template <int kLayA = kRowsByK, int kLayB = kRowsByK, int kW = kLargeTile, class Epilogue>
inline void launch_gemm_tile(const GemmProblem& p, const Epilogue& epi, hipStream_t s) {
    const unsigned grid = (unsigned)(p.M / kTile<kW>) * (unsigned)(p.N / kTile<kW>) * (unsigned)p.splits;
    if (kW == kSmallTile && grid <= 256 && steps_per_part(p) >= kDeepSteps) gemm_bf16<Epilogue, kLayA, kLayB, kSmallTile, kDeepRingSlots><<<grid, kGemmThreads, 0, s>>>(p, epi);
    else gemm_bf16<Epilogue, kLayA, kLayB, kW><<<grid, kGemmThreads, 0, s>>>(p, epi);
}
// The jobs of a group in one launch on tiles of kW, their workgroups in the order given.
template <class Job>
inline int place_job(Job& job, int tile, int first) {
    job.first = first;
    return first + ceil_div(job.workgroups(tile), kNumXcd) * kNumXcd;
}
template <class... Jobs>
inline void launch_gemm_group(int kW, hipStream_t s, Jobs... jobs) {
    int grid = 0;
    ((grid = place_job(jobs, 32 * kW, grid)), ...);
    if (kW == kLargeTile) gemm_group<kLargeTile, kRingSlots><<<(unsigned)grid, kGemmThreads, 0, s>>>(jobs...);
    else if (grid <= 256 && std::max({steps_per_part(jobs.p)...}) >= kDeepSteps) gemm_group<kSmallTile, kDeepRingSlots><<<(unsigned)grid, kGemmThreads, 0, s>>>(jobs...);
    else gemm_group<kSmallTile, kRingSlots><<<(unsigned)grid, kGemmThreads, 0, s>>>(jobs...);
}
template <int kLayA = kRowsByK, int kLayB = kRowsByK, class Epilogue>
inline void launch_gemm(const GemmProblem& p, const Epilogue& epi, hipStream_t s) {
    if (tile_for(p.M, p.N, p.splits) == kSmallTile) launch_gemm_tile<kLayA, kLayB, kSmallTile>(p, epi, s);
    else launch_gemm_tile<kLayA, kLayB, kLargeTile>(p, epi, s);
}

// A product over the rows of a batch (columns: weights), both operands [rows][K].  When whole rounds of large tiles leave a
// few over, the last columns go to a launch of their own on small tiles, if one round of those holds them: it takes about
// 0.65 us per step where one more round of large tiles takes 0.94.  Below 32 steps the launch costs more than that.
// Measured: 768 x 22016 x 4096 (258 large tiles) 157 -> 137 us, 5376 x 22016 x 4096 (1806) 615 -> 600 us; with two rounds of
// small tiles, 5376 x 4096 x 22016 (336), 508 -> 706 us.  Which columns, if any, the kernels work out from the live rows
// (a list shorter than its buffer has other tiles left over); the second launch is made where a full list takes it, and
// its workgroups leave at once where the live one does not.  One group's step in a buffer of 21 row tiles, columns chosen by
// the buffer / none / by the live rows: 13 live row tiles 2254 / 2218 / 2221 us, 16 2552 / 2516 / 2522, 17 3162 / 3114 / 3117,
// 21 3539 / 3555 / 3550.  The second launch has at most one workgroup per CU and keeps the deep ring: 768 x 22016 x 4096, its twelve
// tiles 45 -> 36 us.
template <class Epilogue>
inline void launch_row_gemm(const GemmProblem& p, const Epilogue& epi, hipStream_t s) {
    const int tm = p.M / kTileM, tn = p.N / kTileN, steps = (p.K1 + p.K2) / kTileK;
    if (tile_for(p.M, p.N, 1) != kLargeTile || steps < 32 || tm > 64 || cut_columns(tm, tn) == 0) {
        launch_gemm(p, epi, s);
        return;
    }
    int most = 0;                                           // small tiles, over the lists that the buffer can hold
    for (int live = 1; live <= tm; ++live) most = std::max(most, 4 * live * cut_columns(live, tn));
    GemmProblem head = p, tail = p;
    head.cut = kCutHead;
    tail.cut = kCutTail;
    launch_gemm_tile<kRowsByK, kRowsByK, kLargeTile>(head, epi, s);
    gemm_bf16<Epilogue, kRowsByK, kRowsByK, kSmallTile, kDeepRingSlots><<<(unsigned)most, kGemmThreads, 0, s>>>(tail, epi);
}

}  // namespace pcm
