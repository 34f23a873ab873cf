// fp32 matrices as three bf16 matrices each (internal header): what lets the fp32 path of the actor step run on the bf16
// matrix cores without giving up a bit of its operands.
#pragma once

#include "actor.h"

namespace pcm {

// global memory of any float alignment: the hardware takes 8- and 16-byte accesses at every multiple of four bytes
typedef __attribute__((ext_vector_type(4), aligned(4))) float f32x4_any;

// Three matrices [rows][ld], `third` elements apart, whose sum is an fp32 matrix [rows][columns].  Columns and rows behind the
// matrix, as far as a reduction or a tile of 128 reads them, are zero.
struct Thirds {
    bf16* p;
    int64_t ld, third;
};
constexpr int kThirdsUnit = 128;         // columns are padded to a multiple of this
constexpr int kThirdsRows = 256;         // and rows (allocated, not cleared) to one of this

// x as the sum of three bf16 values, exactly (but for what lies below the smallest bf16 value): the leading eight bits of the
// significand by truncation, which cannot overflow, and twice the bf16 value nearest to the rest, the second of which leaves
// none.  out[t]: the t-th parts of kN values, two to a word.
template <int kN>
__device__ __forceinline__ void split_in_three(const float (&x)[kN], uint32_t (&out)[3][kN / 2]) {
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
#pragma unroll
    for (int q = 0; q < kN / 2; ++q) {
        const uint32_t x0 = __builtin_bit_cast(uint32_t, x[2 * q]), x1 = __builtin_bit_cast(uint32_t, x[2 * q + 1]);
        out[0][q] = __builtin_amdgcn_perm(x1, x0, 0x07060302);          // the upper halves
        float r0 = x[2 * q] - __builtin_bit_cast(float, x0 & 0xFFFF0000u), r1 = x[2 * q + 1] - __builtin_bit_cast(float, x1 & 0xFFFF0000u);
        const bf16x2 middle = {(__bf16)r0, (__bf16)r1};
        out[1][q] = __builtin_bit_cast(uint32_t, middle);
        r0 -= __builtin_bit_cast(float, out[1][q] << 16);
        r1 -= __builtin_bit_cast(float, out[1][q] & 0xFFFF0000u);
        const bf16x2 low = {(__bf16)r0, (__bf16)r1};
        out[2][q] = __builtin_bit_cast(uint32_t, low);
    }
}

// gather.hip: what an fp32 step does before its first product, in one launch: the kept chunks' rows of hidden as thirds (rows from
// the last live one to the end of its tile of 256 are zero) with their metadata, the weights as thirds, and zeros in the rows of
// dX (or null) behind the last live row's tile, which no product writes.
struct ThirdsJob {
    const float* src;     // [R, C]
    Thirds dst;
    int R, C, rows;       // rows written: R and zeros
    int mode;             // PackMode: as it is, or gate and up in blocks of 32 columns in turn (dst.ld covers both)
};
struct ThirdsList {
    static constexpr int kMax = 4;
    ThirdsJob job[kMax];
    int first[kMax];      // first workgroup of each
    int n, blocks;
    static constexpr int kUnits = 1024;       // groups of eight columns per workgroup
    void add(const ThirdsJob& j) {
        job[n] = j;
        first[n++] = blocks;
        const int64_t columns = j.mode == kPackNone ? j.dst.ld : j.dst.ld / 2;
        blocks += (int)ceil_div64(j.rows * (columns / 8), kUnits);
    }
};
[[nodiscard]] int launch_prepare_f32(const ActorShape& sh, const ActorIO& io, const Thirds& X, int64_t rows_pad, RowMeta meta,
                                     const ThirdsList& weights, float* dX, hipStream_t s);

}  // namespace pcm
