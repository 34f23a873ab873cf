// fp32 matrices as three bf16 matrices each (internal header): what lets the fp32 path of the actor step run on the bf16
// matrix cores without giving up a bit of its operands.
#pragma once

#include "actor.h"

namespace pcm {

// global memory of any float alignment: the hardware takes 8- and 16-byte accesses at every multiple of four bytes
typedef __attribute__((ext_vector_type(4), aligned(4))) float f32x4_any;

// An fp32 matrix [rows][columns] as three bf16 matrices whose sum it is, in blocks of 128 rows x 32 columns: a block's part 0, 1
// and 2 one behind the other, each [128][32]; the blocks of 128 rows in order of their columns, then the next 128 rows.  Columns
// are padded to ld, a multiple of 128, and rows to one of 128; what is padding is zero as far as a reduction reads it.
// A step of a product takes 32 of k of 128 rows, which is one block, 24 KB in a row (or 32 rows of four blocks, 2 KB of each
// part), so every line that it brings in is used whole.  (With the matrices of the parts stored row by row, a step takes a half
// of every 128-byte line of an operand [rows][K]: steps 3 to 23 % longer, 1792 rows of 169 -> 2026 197 -> 178 us.)
constexpr int kThirdsUnit = 128, kThirdsPart = kThirdsUnit * 32, kThirdsBlock = 3 * kThirdsPart;
struct Thirds {
    bf16* p;
    int64_t ld;
    // where part 0 of an element is; that of part t is t * kThirdsPart further
    __host__ __device__ static int64_t at(int64_t row, int64_t column, int64_t ld) {
        return ((row / kThirdsUnit) * (ld / 32) + column / 32) * kThirdsBlock + (row % kThirdsUnit) * 32 + column % 32;
    }
};

// An fp32 matrix in the same blocks of 128 rows x 32 columns, for products on the fp32 matrix instructions: of each eight columns
// the even ones, then the odd ones, which is what the two halves of a wavefront read.
constexpr int kFloatsBlock = kThirdsUnit * 32;
struct FloatBlocks {
    float* p;
    int64_t ld;
    // where column 0 of the eight that hold `column` is
    __host__ __device__ static int64_t at(int64_t row, int64_t column, int64_t ld) {
        return ((row / kThirdsUnit) * (ld / 32) + column / 32) * kFloatsBlock + (row % kThirdsUnit) * 32 + column % 32 / 8 * 8;
    }
};

// x as the sum of three bf16 values, exactly (but for what lies below the smallest bf16 value): the bf16 value nearest to x (or the
// largest finite one), and twice the one nearest to the rest, the second of which leaves none.  The second and third part are at
// most 2^-8 and 2^-17 of x, so the three products of parts that a product of two leaves out (second by third, third by second, third by
// third) come to less than 2^-24 of it, the rounding of one fp32 operation.  (With the first part cut off instead of rounded 2^-22.)
// out[t]: the t-th parts of kN values, two to a word.
template <int kN>
__device__ __forceinline__ void split_in_three(const float (&x)[kN], uint32_t (&out)[3][kN / 2]) {
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
    const float largest = __builtin_bit_cast(float, 0x7F7F0000u);
#pragma unroll
    for (int q = 0; q < kN / 2; ++q) {
        float r[2] = {x[2 * q], x[2 * q + 1]};
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            const float r0 = t == 0 ? __builtin_amdgcn_fmed3f(r[0], -largest, largest) : r[0];
            const float r1 = t == 0 ? __builtin_amdgcn_fmed3f(r[1], -largest, largest) : r[1];
            const bf16x2 part = {(__bf16)r0, (__bf16)r1};
            out[t][q] = __builtin_bit_cast(uint32_t, part);
            asm("" : "+v"(out[t][q]));              // (else the compiler converts the first of the two again, by itself)
            r[0] -= __builtin_bit_cast(float, out[t][q] << 16);
            r[1] -= __builtin_bit_cast(float, out[t][q] & 0xFFFF0000u);
        }
    }
}

// gather.hip: what an fp32 step does before its first product, in one launch: the kept chunks' rows of hidden, as floats and (if
// X3.p) as thirds, with their metadata (rows from the last live one to the end of its tile of 256 are zero), the weights, as floats
// (to.p) or as thirds (to3.p), and zeros in the rows of dX (or null) behind the last live row's tile, which no product writes.
struct WeightJob {
    const float* src;     // [R, C]
    FloatBlocks to;       // one of the two, its padding cleared
    Thirds to3;
    int R, C;
    bool transposed;      // to: columns of src as rows
    int mode;             // PackMode of the columns: as they are, or gate and up in blocks of 32 in turn (up to twice as many)
};
struct WeightJobs {
    static constexpr int kMax = 8;
    WeightJob job[kMax];
    int first[kMax];      // first workgroup of each
    int n, blocks;
    static constexpr int kUnits = 1024;       // groups of eight values per workgroup
    void add(const WeightJob& j) {
        job[n] = j;
        first[n++] = blocks;
        blocks += (int)ceil_div64(padded(j.R) * padded(j.C) / 8, kUnits);
    }
    static int64_t padded(int64_t n) { return ceil_div64(n, kThirdsUnit) * kThirdsUnit; }
};
// Its argument.
struct PrepareF32 {
    GatherArgs<float> gather;    // X unused
    FloatBlocks X;
    Thirds X3;
    WeightJobs weights;
    float* dX;
    int gather_blocks;
};
[[nodiscard]] int launch_prepare_f32(const ActorShape& sh, const ActorIO& io, const FloatBlocks& X, const Thirds& X3, int64_t rows_pad,
                                     RowMeta meta, const WeightJobs& weights, float* dX, hipStream_t s);

}  // namespace pcm
