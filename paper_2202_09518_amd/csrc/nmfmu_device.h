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

__device__ __forceinline__ f32x16 mfma32(float a, float b, f32x16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
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

// ---- exact fp32 products on the bf16 matrix cores ---------------------------------
// A float x is cut into three pieces h + m + l = x, each with at most 8
// significant bits (a bf16 holds 8): h = x truncated to its top 8 bits,
// m = (x - h) truncated likewise, l = the rest.  Both subtractions are exact,
// so the sum of the pieces is x bit for bit (for |x| >= 2^-110; below that the
// last piece can fall under the bf16 range and is dropped by the hardware).  A
// product of two pieces has at most 16 significant bits and is exact in the
// fp32 accumulator, so the nine piece products of x y add up to the exact x y:
// v_mfma_f32_32x32x16_bf16 on pieces computes the same sums of products as
// v_mfma_f32_32x32x2_f32 on the floats, with the roundings of the running sums
// only, at a quarter of the matrix-core time per product.
//
// Lane layout of v_mfma_f32_32x32x16_bf16: A_op (32 x 16): lane l holds
// A_op[l % 32][8 (l / 32) .. 8 (l / 32) + 7]; B_op (16 x 32): lane l holds
// B_op[8 (l / 32) .. + 7][l % 32]; D as for the fp32 instruction.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ f32x16 mfma_bf16(u32x4 a, u32x4 b, f32x16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// Bit patterns of the three pieces as floats (their low 16 bits are zero, or
// dropped by pack2: the top 16 bits are the bf16).
__device__ __forceinline__ void split3(float x, unsigned &h, unsigned &m, unsigned &l)
{
    h = __float_as_uint(x) & 0xffff0000u;
    const float r = x - __uint_as_float(h);
    m = __float_as_uint(r) & 0xffff0000u;
    l = __float_as_uint(r - __uint_as_float(m));
}

// Two bf16 in one register: `even` in the low half, `odd` in the high half.
__device__ __forceinline__ unsigned pack2(unsigned even, unsigned odd)
{
    return __builtin_amdgcn_perm(odd, even, 0x07060302u);
}

// The streamed operand is cut with rounding instead of truncation, two floats at a time (packed
// conversions, round to nearest even): h = x rounded to 8 significant bits, m = (x - h) rounded
// likewise, l = the rest; again exact, |m| <= 2^-8 |x|, |l| <= 2^-16 |x| and m, l have either
// sign.  Against a truncated operand (W or H from the planes: pieces of one sign, m < 2^-7,
// l < 2^-15 of the float) the passes issue SIX products, h h, h m, m h, m m, h l, l h: the three
// left out are below 2^-23 (twice) and 2^-31 of the term and signed like A's lower pieces.
// With the first two of them added back the errors against 64 bits were the same to the second
// digit on planted, uniform and repeated-value data (2003 x 4004 to 65536 x 1024, k = 20 to 64), and
// where A and W hold one value each the results agreed to every digit printed: the matrix adder
// drops bits of that size of every term that joins a grown accumulator (see the running totals
// below).  They would cost 4 (32768 x 16384, k = 32) to 15 % (rank 256, one pass) of an iteration.
// Against eight products of truncated pieces, which lose their low bits always downwards, the error
// is smaller at the same lengths of accumulation: 6.0e-8 against 6.7e-8 at 4096 rows, mean signed
// error -2e-9 against -28e-9.
// A value above the largest bf16 (3.39e38) would round to infinity and is held at that bf16.
__device__ __forceinline__ unsigned cvt_pk_bf16(float lo, float hi)
{
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}

// Pieces of two consecutive elements of an operand into register pr of its three planes.
__device__ __forceinline__ void cut2(float x0, float x1, u32x4 (&at)[3], int pr)
{
    typedef short i16x2 __attribute__((ext_vector_type(2)));
    const unsigned h = __builtin_bit_cast(unsigned, __builtin_elementwise_min(
        __builtin_bit_cast(i16x2, cvt_pk_bf16(x0, x1)), i16x2{0x7f7f, 0x7f7f}));
    const float r0 = x0 - __uint_as_float(h << 16), r1 = x1 - __uint_as_float(h & 0xffff0000u);
    const unsigned m = cvt_pk_bf16(r0, r1);
    at[0][pr] = h;
    at[1][pr] = m;
    at[2][pr] = cvt_pk_bf16(r0 - __uint_as_float(m << 16), r1 - __uint_as_float(m & 0xffff0000u));
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
//
// What the scales leave out: an entry below 2^-2 of the scaled range (2^-17 of the largest) is off by up to 2^-25 there, and
// a factor's, cut under a scale of its eight rows and brought to the column's, by up to 2^-23.  No scale holds every sum against that: a
// small entry of a factor is all there is to a sum whose other terms meet zeros of the streamed matrix, and the
// updates drive factors that far by themselves.  So every sum is looked at when it is done, against what is left out of it at most: 2^-23
// of the sum of the streamed column's magnitudes, and 2^15 (a factor's largest) times 2^-25 for each of its entries that is small and not
// zero, or simply 128 * 2^15 * (2^-23 + 2^-25) < 1 in its scaled range for up to 128 rows.  If any sum of a workgroup's tile is below kSure
// times that, or not finite, the whole tile is formed again from the floats as they are (floats_tile); what is left out of the others
// is 2^-22 of them at most.  Sums of uniform entries are 2^15 times as large as that asks.
constexpr float kSure = 4194304.f;
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

// The largest magnitude of a column, as bits; its half_exponent is that of the column's scale.
__device__ __forceinline__ unsigned column_most(const unsigned *__restrict__ most, int ld, int c)
{
    unsigned m[kPairCopies], top = 0;
#pragma unroll
    for (int i = 0; i < kPairCopies; ++i) m[i] = most[i * ld + c];
#pragma unroll
    for (int i = 0; i < kPairCopies; ++i) top = m[i] > top ? m[i] : top;
    return top;
}

// A unit brought from its own scale to its column's, in two steps: 2^-24 is the smallest half, and the largest of a unit reaches below
// the last place of the scaled range 2^-40 further down.  fill: what a column of zeros gets in place of its entries, else zero; added
// (FMA: 128 factors 2 % faster) or put in (64 factors 1 % faster).
template <bool FMA>
__device__ __forceinline__ u32x4 to_column_scale(u32x4 unit, unsigned exps, int exponent, _Float16 fill)
{
    const int by = exponent + 112 - (int)exps, d = by > 40 ? 40 : by;
    const _Float16 r = (_Float16)power_of_two(-(d >> 1)), s = (_Float16)power_of_two((d >> 1) - d);
    const f16x2 ff = {fill, fill};
    u32x4 o;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const unsigned u = unit[i];
        const f16x2 part = __builtin_bit_cast(f16x2, u) * f16x2{r, r};
        if (FMA) o[i] = __builtin_bit_cast(unsigned, __builtin_elementwise_fma(part, f16x2{s, s}, ff));
        else o[i] = __builtin_bit_cast(unsigned, part * f16x2{s, s}) | __builtin_bit_cast(unsigned, ff);
    }
    return o;
}

}  // namespace nmfmu
