// Products of fp32 matrices on the fp32 matrix instructions (v_mfma_f32_32x32x2_f32), for the forward pass of the fp32 path
// (internal header).  The MFMA adds its products one k after the other, and every sum here is one chain over all k, so the
// result does not depend on the tile.
//
// Operands in blocks (FloatBlocks) go from global memory to LDS directly; a fragment read of 16 bytes serves four MFMAs, so between
// the MFMAs of an octet of k there is next to nothing.  Bound by the matrix pipe: 8192 x 1024 x 2816 by itself 332 us, 142 TFLOP/s
// of a nominal 157 (registers alone: 147 - 155; without the loads 145, without the fragment reads 148); within a step, where the
// bf16 products have brought the clock down, gate and up of 10,752 rows at 1024 -> 2816 with the activation 871 us, 108 TFLOP/s.
// Two workgroups per CU of the largest tile, three of the smaller ones: one with more of its steps in LDS is 3 % slower.
#pragma once

#include "gemm_bf16.h"
#include "thirds.h"

namespace pcm {

typedef __attribute__((ext_vector_type(16))) float f32x16;

template <int kI, int kJ> constexpr int kFloatsSlots = kI + kJ == 2 ? 3 : 2;     // steps of 32 k in LDS
template <int kI, int kJ> constexpr int kFloatsPerCu = kI + kJ == 4 ? 2 : 3;

// Sums of a wavefront: kI x kJ tiles of 32 x 32; element 4 g + t of tile (i, j) is row row0 + 32 i + (lane & 31), column
// col0 + 32 j + 8 g + 4 (lane >> 5) + t.
template <int kI, int kJ>
struct FloatsCoord {
    int row0, col0, lane;
};
template <int kI, int kJ>
struct FloatsRing {
    __attribute__((aligned(1024))) float data[kFloatsSlots<kI, kJ> * 64 * (kI + kJ) * 32];
    static constexpr uint32_t kSlotBytes = 64 * (kI + kJ) * 128, kStageBytes = kFloatsSlots<kI, kJ> * kSlotBytes / 4;
};

// C[m, n] = sum_k A(m, k) B(n, k), both operands in blocks; M, N multiples of the tile of 64 kI x 64 kJ; rows of the batch beyond
// the live ones are skipped.  Four wavefronts, 2 x 2, each 32 kI x 32 kJ.
struct FloatsProblem {
    const float *A, *B;
    int64_t lda, ldb;
    int M, N, K;                         // K a multiple of 32
    const int32_t* n_kept;               // null: no rows of the batch
    int max_chunks, A_rows;
};
template <int kI, int kJ, class Epilogue>
__global__ __launch_bounds__(256, (kFloatsPerCu<kI, kJ>)) void gemm_floats(FloatsProblem p, Epilogue epi) {
    constexpr int TM = 64 * kI, TN = 64 * kJ, kLoadsA = 2 * kI, kLoads = 2 * (kI + kJ), kSlots = kFloatsSlots<kI, kJ>;
    using Ring = FloatsRing<kI, kJ>;
    __shared__ Ring smem;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave >> 1, wn = wave & 1;
    const int tiles_m = p.M / TM, tiles_n = p.N / TN;
    int live_m = tiles_m;
    if (p.n_kept != nullptr)
        live_m = (int)min((int64_t)tiles_m, (live_rows(p.n_kept, p.max_chunks, p.A_rows) + kTileM - 1) / kTileM * (kTileM / TM));
    int tm, tn;
    if (!tile_of_workgroup<kSmallTile>((int)blockIdx.x, tiles_m * tiles_n, live_m, tiles_n, tm, tn)) return;
    const int m0 = tm * TM, n0 = tn * TN, steps = p.K / 32;

    // Global -> LDS: a load fills eight rows of 128 bytes; piece q (16 bytes) of row r sits in place swizzle_piece(r, q).
    const uint32_t lds_base = (uint32_t)(uintptr_t)PCM_AS_LDS(smem.data);
    uint32_t off[2];
#pragma unroll
    for (int odd = 0; odd < 2; ++odd) off[odd] = (uint32_t)(lane >> 3) * 128u + (uint32_t)swizzle_piece((lane >> 3) + 8 * odd, lane & 7) * 16u;
    const char* from[2];
    from[0] = reinterpret_cast<const char*>(p.A + FloatBlocks::at(m0 + wave * (TM / 4), 0, p.lda));
    from[1] = reinterpret_cast<const char*>(p.B + FloatBlocks::at(n0 + wave * (TN / 4), 0, p.ldb));
    auto load = [&](uint32_t slot, int n) __attribute__((always_inline)) {
        const int operand = n < kLoadsA ? 0 : 1, r = operand == 0 ? n : n - kLoadsA;
        const uint32_t to = lds_base + slot + (operand == 0 ? (uint32_t)wave * (TM / 4) * 128u : (uint32_t)TM * 128u + (uint32_t)wave * (TN / 4) * 128u);
        direct_load_16B(from[operand], off[r & 1] + (uint32_t)r * 1024u, to + (uint32_t)r * 1024u);
    };
    // A fragment read brings this lane's row and four k of its half's parity: those of four MFMAs.
    auto fragment_at = [&](int row, int octet) { return (uint32_t)(row * 128 + swizzle_piece(row, 2 * octet + (lane >> 5)) * 16); };
    uint32_t base_a[4], base_b[4];
#pragma unroll
    for (int o = 0; o < 4; ++o) {
        base_a[o] = lds_base + fragment_at(wm * 32 * kI + (lane & 31), o);
        base_b[o] = lds_base + (uint32_t)TM * 128u + fragment_at(wn * 32 * kJ + (lane & 31), o);
    }
    auto read = [](uint32_t at) { return *(const __attribute__((address_space(3))) f32x4*)(uintptr_t)at; };

    f32x16 acc[kI][kJ];
#pragma unroll
    for (int i = 0; i < kI; ++i)
#pragma unroll
        for (int j = 0; j < kJ; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    const int last = steps - 1;
#pragma unroll
    for (int s = 0; s < kSlots; ++s) {                     // steps past the end re-request the last one, which nobody reads
#pragma unroll
        for (int n = 0; n < kLoads; ++n) load((uint32_t)s * Ring::kSlotBytes, n);
        const uint32_t stride = s + 1 <= last ? kFloatsBlock * 4u : 0u;
        from[0] += stride;
        from[1] += stride;
    }
    wait_direct_loads<(kSlots - 1) * kLoads>();
    __syncthreads();
    f32x4 fa[2][kI], fb[2][kJ];
#pragma unroll
    for (int i = 0; i < kI; ++i) fa[0][i] = read(base_a[0] + (uint32_t)i * 4096u);
#pragma unroll
    for (int j = 0; j < kJ; ++j) fb[0][j] = read(base_b[0] + (uint32_t)j * 4096u);
    // A step is four octets of k, 4 kI kJ MFMAs each, and the fragments of the next octet are read meanwhile.  Before the last one
    // every wavefront holds the step's fragments, so its slot is refilled, and the next step has to have landed.
    uint32_t cur = 0;
    for (int s = 0; s < steps; ++s) {
        const uint32_t next = cur + Ring::kSlotBytes == kSlots * Ring::kSlotBytes ? 0u : cur + Ring::kSlotBytes;
        static_for<4>([&](auto which) __attribute__((always_inline)) {
            constexpr int o = decltype(which)::value, set = o & 1;
            if constexpr (o == 3) {
                wait_direct_loads<(kSlots - 2) * kLoads>();
                __syncthreads();
            }
            const uint32_t slot = o < 3 ? cur : next;
#pragma unroll
            for (int i = 0; i < kI; ++i) fa[set ^ 1][i] = read(base_a[(o + 1) & 3] + slot + (uint32_t)i * 4096u);
#pragma unroll
            for (int j = 0; j < kJ; ++j) fb[set ^ 1][j] = read(base_b[(o + 1) & 3] + slot + (uint32_t)j * 4096u);
            static_for<4 * kI * kJ>([&](auto number) __attribute__((always_inline)) {
                constexpr int n = decltype(number)::value, t = n / (kI * kJ), i = n % (kI * kJ) / kJ, j = n % kJ;
                __builtin_amdgcn_sched_barrier(0);
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fb[set][j][t], fa[set][i][t], acc[i][j], 0, 0, 0);
                if constexpr (o == 3 && n * kLoads / (4 * kI * kJ) != (n + 1) * kLoads / (4 * kI * kJ)) {
                    __builtin_amdgcn_sched_barrier(0);
                    static_for<(n + 1) * kLoads / (4 * kI * kJ) - n * kLoads / (4 * kI * kJ)>([&](auto more) __attribute__((always_inline)) {
                        load(cur, n * kLoads / (4 * kI * kJ) + decltype(more)::value);
                    });
                }
            });
        });
        const uint32_t stride = s + kSlots + 1 <= last ? kFloatsBlock * 4u : 0u;
        from[0] += stride;
        from[1] += stride;
        cur = next;
    }
    wait_direct_loads<0>();
    __syncthreads();
    epi(FloatsCoord<kI, kJ>{m0 + wm * 32 * kI, n0 + wn * 32 * kJ, lane}, acc, reinterpret_cast<char*>(smem.data) + wave * Ring::kStageBytes);
}

}  // namespace pcm
