// Device code shared by the translation units of libnmfmu.
#pragma once

#include "nmfmu_internal.h"

namespace nmfmu {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// Sum of N requested values, added in a fixed tree: long lists of partial results meet in batches of this
// kind, so that no value passes through a chain of more roundings than there are batches plus log2 N.
template <int N>
__device__ __forceinline__ float tree_sum(float (&t)[N])
{
#pragma unroll
    for (int w = N / 2; w > 0; w >>= 1)
#pragma unroll
        for (int i = 0; i < w; ++i) t[i] += t[i + w];
    return t[0];
}

// Row of the 32 x 32 accumulator held in register v of a lane in half `half`.
__device__ __forceinline__ int acc_row(int v, int half) { return (v & 3) + 4 * half + 8 * (v >> 2); }

// Side job of the pass kernels: the Gram tiles a finisher left behind (nsets sets of
// kt x kt tiles of 1024 floats) are needed, summed, by the finisher AFTER this pass.  The
// first workgroups of the pass add them up so that no separate launch is needed: job j = entries
// 64 j .. 64 j + 63, dealt to the nwg workgroups in order (first: this one); four lanes share an entry, lane q adds sets
// q, q + 4, ... a batch of 16 at a time, and the four sums meet in a fixed tree.  (Sums of 16 sets each, left to the
// finisher's workgroups to finish, cost every one of them 256 KiB of reads at 33 to 64 factors.)
__device__ __forceinline__ void sum_tile_sets(const float *__restrict__ gtiles, int nsets, int k,
                                              float *__restrict__ gsum, int first, int nwg)
{
    constexpr int B = 16;
    const int kt = (k + 31) >> 5;
    const int stride = kt * kt * 1024;
    const int q = threadIdx.x & 3;
    for (int job = first; job < stride / 64; job += nwg) {
        const float *src = gtiles + job * 64 + (threadIdx.x >> 2);
        float sum = 0.f;
        for (int s = q; s < nsets; s += 4 * B) {
            float t[B];
#pragma unroll
            for (int b = 0; b < B; ++b) t[b] = src[(int64_t)(s + 4 * b < nsets ? s + 4 * b : 0) * stride];
#pragma unroll
            for (int b = 0; b < B; ++b) t[b] = s + 4 * b < nsets ? t[b] : 0.f;
            sum += tree_sum(t);
        }
        sum += __shfl_xor(sum, 1);
        sum += __shfl_xor(sum, 2);
        if (q == 0) gsum[job * 64 + (threadIdx.x >> 2)] = sum;
    }
}

// ---- the same from pairs of halves --------------------------------------------------
// A float scaled by a power of two into the range of a half (11 significant bits) is cut into h = x rounded to nearest
// even and l = (x - h) rounded likewise: 22 bits and the two signs, so h + l is x or, for a quarter of all floats, its
// neighbour; below 2^-1 of the scaled range the halves' denormals end the second piece at 2^-25 instead.  THREE products,
// l h, h l and h h, do the work of the six of bf16 pieces (the one left out is below 2^-24 of the term, of either sign),
// and the cut is shorter.  The products have up to 22 bits, and fewer of them join an accumulator: against 64
// bits, root mean square over 4096 terms of U[0,1) in chains of 256, bf16 pieces 7.5e-8 and pairs 6.7e-8 (fp32
// instruction 8.0e-8); with one value down a column 1.9e-7 and 8.4e-8; one value on either side 6.3e-7 and 4.4e-7.
//
// Scales: a factor's column c has one for all of a pass, 2^(14 - exponent of its largest entry) (half_exponent of most[c]).
// The streamed operand's columns belong to lanes, and their scales change along the rows (see the passes).
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ f32x16 mfma_f16(u32x4 a, u32x4 b, f32x16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

// Exponent of the power of two below |x|, from the bits of |x|; held where 2^(14 - e) and its inverse are floats.  What is
// smaller than 2^-112 meets a scale of 2^126, under which the last bit of a denormal float is a half.
__device__ __forceinline__ int half_exponent(unsigned bits)
{
    const int e = (int)(bits >> 23) - 127;
    return e < -112 ? -112 : e;
}
__device__ __forceinline__ float power_of_two(int e) { return __uint_as_float((unsigned)(e + 127) << 23); }

// Halves of two consecutive elements of an operand, times s, into register pr of its two planes.
__device__ __forceinline__ void cut2h(float x0, float x1, float s, u32x4 (&at)[2], int pr)
{
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    const f16x2 h = __builtin_convertvector(f32x2{x0 * s, x1 * s}, f16x2);
    const float r0 = __builtin_fmaf(x0, s, -(float)h[0]), r1 = __builtin_fmaf(x1, s, -(float)h[1]);
    at[0][pr] = __builtin_bit_cast(unsigned, h);
    at[1][pr] = __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{r0, r1}, f16x2));
}

// Pair planes of a factor F (rows x k, contracted over its rows): unit (rows 8 g .. 8 g + 7, piece p, column c) = 16 bytes at
// (g * 2 + p) * ld + c, cut under a scale of the unit's own, its largest magnitude at 2^14; exps[g * ld + c] = that one's
// half_exponent + 112.  most[copy * ld + c] = the largest magnitudes of the column in parts of it, as bits, which scales it in the pass: what writes the
// planes need not know the other rows.  One unit; the largest magnitude is returned.
__device__ __forceinline__ unsigned put_pairs(const float (&x)[8], u32x4 *unit, int64_t ld, unsigned char *exps)
{
    unsigned top = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const unsigned b = __float_as_uint(x[e]) & 0x7fffffffu;
        top = b > top ? b : top;
    }
    const int e = half_exponent(top);
    const float sc = power_of_two(14 - e);
    u32x4 o[2];
#pragma unroll
    for (int pr = 0; pr < 4; ++pr) cut2h(x[2 * pr], x[2 * pr + 1], sc, o, pr);
    unit[0] = o[0];
    unit[ld] = o[1];
    *exps = (unsigned char)(e + 112);
    return top;
}

// The exponent of a column's scale.
__device__ __forceinline__ int column_exponent(const unsigned *__restrict__ most, int ld, int c)
{
    unsigned m[kPairCopies], top = 0;
#pragma unroll
    for (int i = 0; i < kPairCopies; ++i) m[i] = most[i * ld + c];
#pragma unroll
    for (int i = 0; i < kPairCopies; ++i) top = m[i] > top ? m[i] : top;
    return half_exponent(top);
}

// A unit brought from its own scale to its column's.
__device__ __forceinline__ u32x4 to_column_scale(u32x4 unit, unsigned exps, int exponent)
{
    const int d = exponent + 112 - (int)exps;
    const _Float16 r = (_Float16)power_of_two(-(d > 40 ? 40 : d));
    u32x4 o;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const unsigned u = unit[i];
        o[i] = __builtin_bit_cast(unsigned, __builtin_bit_cast(f16x2, u) * f16x2{r, r});
    }
    return o;
}

}  // namespace nmfmu
