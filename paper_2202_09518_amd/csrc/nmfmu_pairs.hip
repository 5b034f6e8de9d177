// Products of two fp32 matrices as pairs of halves on the fp16 matrix cores: more than 32 factors (see nmfmu_device.h for the
// arithmetic and the formats).
//   cut_pairs_kernel : A and A^T in the order in which the pass loads them, once per call
//   split_pairs_kernel : the planes of a factor (factor_update_kernel writes them itself)
//   pair_pass_kernel : the pass over A' or (A^T)' for slices of 64 or 128 factors
//   wta_pass_pair_kernel : the same over a matrix that is cut as it is loaded
//   floats_tile : a tile of either pass again from the floats, where a sum could have lost more to the halves than it may
#include "nmfmu_device.h"

namespace nmfmu {

// ---------------------------------------------------------------------------
// A itself as pairs of halves, in the order in which the pass loads its operands, so that nothing is cut more than once a call:
// A' and (A^T)' (see PairMatrix; a column's largest magnitude in a block of 128 rows goes to 2^14).  A workgroup takes a tile of
// 128 x 128 of A through LDS and writes it into both.  16384 x 8192: 300 us (a transposed copy alone: 200); 20011 x 9998: 480 (a
// transposed and an aligned copy: 595).
// clear: words to set to zero on the way.
// ---------------------------------------------------------------------------
constexpr int kCutTile = kPairBlock;
typedef int i32x4 __attribute__((ext_vector_type(4)));
template <bool VEC>
__global__ __launch_bounds__(512) void cut_pairs_kernel(const float *__restrict__ A, int64_t m, int64_t n, PairMatrix a, PairMatrix at_,
                                                        unsigned *__restrict__ clear, int nclear)
{
    __shared__ float tile[kCutTile][kCutTile + 1];
    __shared__ unsigned part[4][kCutTile];
    __shared__ float left[4][kCutTile];
    const int tid = threadIdx.x;
    if (blockIdx.x == 0)
        for (int i = tid; i < nclear; i += 512) clear[i] = 0u;
    const int64_t tc = (n + kCutTile - 1) / kCutTile;
    const int64_t br = blockIdx.x / tc, bc = blockIdx.x % tc;
    const int64_t r0 = br * kCutTile, c0 = bc * kCutTile;
    if (VEC) {
        const int x = (tid & 31) * 4, y = tid >> 5;
        f32x4 v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int64_t r = r0 + y + 16 * i;
            const bool ok = r < m && c0 + x < n;
            v[i] = *reinterpret_cast<const f32x4 *>(A + (ok ? r * n + c0 + x : 0));
            if (!ok) v[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) tile[y + 16 * i][x + e] = v[i][e];
    } else {
        const int x = tid & 127, y = tid >> 7;
#pragma unroll
        for (int b = 0; b < 32; b += 16) {
            float v[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int64_t r = r0 + y + 4 * (b + i);
                const bool ok = r < m && c0 + x < n;
                v[i] = A[ok ? r * n + c0 + x : 0];
                v[i] = ok ? v[i] : 0.f;
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) tile[y + 4 * (b + i)][x] = v[i];
        }
    }
    __syncthreads();
    const int at = tid & 127, quarter = tid >> 7;     // a column (then a row) of the tile and 32 of its entries
#pragma unroll
    for (int side = 0; side < 2; ++side) {
        float v[32];
#pragma unroll
        for (int i = 0; i < 32; ++i) v[i] = side ? tile[at][32 * quarter + i] : tile[32 * quarter + i][at];
        unsigned top = 0;
#pragma unroll
        for (int i = 0; i < 32; ++i) {
            const unsigned b = __float_as_uint(v[i]) & 0x7fffffffu;
            top = b > top ? b : top;
        }
        part[quarter][at] = top;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i) top = part[i][at] > top ? part[i][at] : top;
        const int e = half_exponent(top);
        const float sc = power_of_two(14 - e);
        // what the halves leave out (see kSure), a little more for the rounding of this sum
        float sum = 0.f, small = 0.f;
#pragma unroll
        for (int i = 0; i < 32; ++i) {
            const float b = __builtin_fabsf(v[i]);
            sum += b * sc;
            small += b * sc < 0.25f && b > 0.f ? 1.f : 0.f;
        }
        left[quarter][at] = sum * (1.0001f * 0x1p-23f) + small * 0x1p-10f;
        __syncthreads();
        const PairMatrix &x = side ? at_ : a;
        const int64_t col = (side ? r0 : c0) + at, ld = x.ld, block = side ? bc : br;
        if (col < ld) {
            u32x4 *dst = static_cast<u32x4 *>(x.units) + (block * 16 + 4 * quarter) * 2 * ld + col;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                u32x4 o[2];
#pragma unroll
                for (int pr = 0; pr < 4; ++pr) cut2h(v[8 * g + 2 * pr], v[8 * g + 2 * pr + 1], sc, o, pr);
                dst[(2 * g) * ld] = o[0];
                dst[(2 * g + 1) * ld] = o[1];
            }
            if (quarter == 0) {
                const float inv = top ? power_of_two(e - 14) : 0.f;
                x.scale[block * ld + col] = float2{inv, inv * ((left[0][at] + left[1][at]) + (left[2][at] + left[3][at]))};
            }
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// Pair planes of X (rows x k, row-major), see put_pairs; rows beyond `rows` and columns beyond k are zero.  blockIdx.y = 64 columns;
// a thread takes eight of a block's 32 row groups, so that a column's maximum costs one atomic per block.
// clear (optional): maxima to set to zero on the way.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void split_pairs_kernel(const float *__restrict__ X, int64_t rows, int k, PairFactor f, int ld,
                                                          unsigned *__restrict__ clear)
{
    __shared__ unsigned most[4][64];
    const int cw = threadIdx.x & 63, w = threadIdx.x >> 6, c = 64 * (int)blockIdx.y + cw;
    if (blockIdx.x == 0 && clear)
        for (int i = w; i < kPairCopies; i += 4) clear[i * ld + c] = 0u;
    unsigned top = 0;
    for (int i = 0; i < 8; ++i) {
        const int64_t g = (int64_t)blockIdx.x * 32 + 4 * i + w;
        if (g * 8 >= rows) break;
        float x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = (g * 8 + e < rows && c < k) ? X[(g * 8 + e) * k + c] : 0.f;
        const unsigned t = put_pairs(x, static_cast<u32x4 *>(f.units) + g * 2 * ld + c, ld, f.exps + g * ld + c);
        top = t > top ? t : top;
    }
    most[w][cw] = top;
    __syncthreads();
    if (w == 0 && c < k) {
#pragma unroll
        for (int i = 1; i < 4; ++i) top = most[i][cw] > top ? most[i][cw] : top;
        if (top) atomicMax(f.most + (int)(blockIdx.x % kPairCopies) * ld + c, top);
    }
}

// ---------------------------------------------------------------------------
// A workgroup's tile of F^T X from the floats as they are, cut into bf16 pieces (which have their exponents), for tiles whose sums the halves
// cannot hold (kSure): rows r0 .. r1, k of 32 T factors, a lane's two columns col, the totals as the passes have them.  F (entry
// (i, c) at f + i * fr + c * fc) goes through LDS, 64 rows at a time, double buffered, cut on the way; X (entry (i, j) at
// x + i * xr + j * xc) straight into registers, D steps of 16 rows ahead, along its rows or along its columns, four entries
// in one load or one.  What bounds it is the one wave per SIMD of the pass that it is part of: cutting and matrix instructions do not overlap.
// A of two blocks on the diagonal, all tiles so, 16384 x 8192, 64 factors: 150 us along the rows, 180 along the columns, where
// pairs take 98 and the mirrored plan, on pieces cut before and a transposed copy, 110 to 128; whole runs there 0.7 to 0.85 of the
// mirrored plan's speed.  On the fp32 instruction 190 and 200.  As a launch of its own it would cost every pass 3 us.
// ---------------------------------------------------------------------------
typedef const __attribute__((address_space(1))) float *GlobalFloats;      // read by global loads, wherever the pointer comes from
struct Floats {
    GlobalFloats f, x;
    int64_t fr, fc, xr, xc;
};

__device__ __forceinline__ uintptr_t uniform(uintptr_t p)
{
    return (uintptr_t)(unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)p) |
           (uintptr_t)(unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(p >> 32)) << 32;
}

enum class Along { rows, columns, columns4 };

template <int T, int D, Along ALONG>
__device__ __forceinline__ void floats_tile(u32x4 *stage, const Floats &o, int k, int64_t r0, int64_t r1, const int64_t (&col)[2],
                                            f32x16 (&tot)[T][2])
{
    constexpr int KP = 32 * T, kRows = 64, kSteps = kRows / 16, kUnits = kRows / 8 * 3 * KP;
    constexpr int kEach = KP / 32;           // row groups of F a thread cuts in a block
    constexpr int kRsrcFlags = 0x00020000;   // raw buffer, 32-bit data format (gfx9 family)
    const int tid = threadIdx.x, lane = tid & 63, jj = lane & 31, half = lane >> 5;
    const int fc = tid & (KP - 1), fg = tid / KP;                // group e of a thread: fg + e * 256 / KP, column fc
    const GlobalFloats f = o.f + (fc < k ? fc : 0) * o.fc;
    const GlobalFloats x[2] = {o.x + col[0] * o.xc + 16 * half, o.x + col[1] * o.xc + 16 * half};
    const unsigned rowb = (unsigned)o.xr * 4u;
    unsigned xoff[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) xoff[q] = (unsigned)(16 * half) * rowb + (unsigned)col[q] * 4u;
    struct Group { float v[8]; };
    auto load_f = [&](Group &u, int64_t ib, int e) {
        const int64_t i = ib + 8 * (fg + e * (256 / KP));
        if (ib + kRows <= r1) {
            const GlobalFloats p = f + i * o.fr;
#pragma unroll
            for (int v = 0; v < 8; ++v) u.v[v] = p[v * o.fr];
        } else {
#pragma unroll
            for (int v = 0; v < 8; ++v) {
                const float t = f[(i + v < r1 ? i + v : r1 - 1) * o.fr];
                u.v[v] = i + v < r1 ? t : 0.f;
            }
        }
    };
    auto store_f = [&](const Group &u, u32x4 *dst, int e) {
        u32x4 p[3];
#pragma unroll
        for (int pr = 0; pr < 4; ++pr) {
            unsigned h[2], m[2], l[2];
#pragma unroll
            for (int b = 0; b < 2; ++b) split3(fc < k ? u.v[2 * pr + b] : 0.f, h[b], m[b], l[b]);
            p[0][pr] = pack2(h[0], h[1]);
            p[1][pr] = pack2(m[0], m[1]);
            p[2][pr] = pack2(l[0], l[1]);
        }
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) dst[((fg + e * (256 / KP)) * 3 + pl) * KP + fc] = p[pl];
    };
    // A step contracts 16 rows: the s-th 8 rows (s = 0, 1) of either half of 32, so that a lane's two steps along a column are
    // 64 consecutive bytes, requested together.
    struct Step { float v[2][8]; };
    auto load_x = [&](Step &t, int64_t ib, int s) {      // ib: of the 32 rows
        if (ALONG == Along::rows) {
            const int64_t i = ib + 8 * s;
            int64_t av = r1 - i;
            av = av < 0 ? 0 : (av > 24 ? 24 : av);
            const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void *)uniform((uintptr_t)(o.x + (av ? i : 0) * o.xr)), 0,
                                                                               __builtin_amdgcn_readfirstlane((int)((unsigned)av * rowb)), kRsrcFlags);
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int v = 0; v < 8; ++v)
                    t.v[q][v] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, xoff[q] + v * rowb, 0, 0));
        } else if (ib + 32 <= r1) {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const GlobalFloats p = x[q] + ib + 8 * s;
                if (ALONG == Along::columns4) {
#pragma unroll
                    for (int b = 0; b < 2; ++b) {
                        const f32x4 u = *(const __attribute__((address_space(1))) f32x4 *)(p + 4 * b);
#pragma unroll
                        for (int v = 0; v < 4; ++v) t.v[q][4 * b + v] = u[v];
                    }
                } else {
#pragma unroll
                    for (int v = 0; v < 8; ++v) t.v[q][v] = p[v];
                }
            }
        } else {
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int v = 0; v < 8; ++v) {
                    const int64_t i = ib + 16 * half + 8 * s + v;
                    const float u = x[q][(i < r1 ? i : r1 - 1) - 16 * half];
                    t.v[q][v] = i < r1 ? u : 0.f;
                }
        }
    };
    f32x16 acc[T][2];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int q = 0; q < 2; ++q) tot[t][q] = f32x16{0};
    Step xs[D];
    Group fu[kEach];
#pragma unroll
    for (int s = 0; s < D; ++s) load_x(xs[s], r0 + 16 * (s & ~1), s & 1);
#pragma unroll
    for (int e = 0; e < kEach; ++e) load_f(fu[e], r0, e);
#pragma unroll
    for (int e = 0; e < kEach; ++e) store_f(fu[e], stage, e);
    __syncthreads();
    int buf = 0;
    for (int64_t i = r0; i < r1; i += kRows) {
        const u32x4 *mine = stage + buf * kUnits;
        u32x4 *next = stage + (buf ^ 1) * kUnits;
#pragma unroll
        for (int s = 0; s < kSteps; ++s) {
            if (s == 0) {      // F of the next block, cut and stored after the last steps
#pragma unroll
                for (int e = 0; e < kEach; ++e) load_f(fu[e], i + kRows, e);
            }
            u32x4 wt[T][3];
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int pl = 0; pl < 3; ++pl) wt[t][pl] = mine[((2 * (s & ~1) + 2 * half + (s & 1)) * 3 + pl) * KP + 32 * t + jj];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                u32x4 at[3];
#pragma unroll
                for (int pr = 0; pr < 4; ++pr) cut2(xs[s % D].v[q][2 * pr], xs[s % D].v[q][2 * pr + 1], at, pr);
                constexpr int PW[6] = {2, 1, 0, 1, 0, 0}, PA[6] = {0, 1, 2, 0, 1, 0};   // smallest first
#pragma unroll
                for (int e = 0; e < 6; ++e)
#pragma unroll
                    for (int t = 0; t < T; ++t)
                        acc[t][q] = mfma_bf16(wt[t][PW[e]], at[PA[e]], s == 0 && e == 0 ? f32x16{0} : acc[t][q]);
            }
            if (s & 1) {
                load_x(xs[(s - 1) % D], i + 16 * (s - 1 + D), 0);
                load_x(xs[s % D], i + 16 * (s - 1 + D), 1);
            }
#pragma unroll
            for (int e = 0; e < kEach; ++e)
                if (s == kSteps - 1 - (kEach - 1 - e) * 2 / kEach) store_f(fu[e], next, e);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int q = 0; q < 2; ++q) tot[t][q] += acc[t][q];
        __syncthreads();    // the next block is written, this one is read
        buf ^= 1;
    }
}

template <int T, int D>
__device__ __forceinline__ void exact_tile(u32x4 *stage, const Floats &o, int k, int64_t r0, int64_t r1, const int64_t (&col)[2],
                                           f32x16 (&tot)[T][2])
{
    // four along a column of X: r0 is a multiple of 16, and so is r1 or it is the end of that column
    if (o.xc == 1) floats_tile<T, D, Along::rows>(stage, o, k, r0, r1, col, tot);
    else if ((o.xc & 3) == 0 && ((uintptr_t)o.x & 15u) == 0) floats_tile<T, D, Along::columns4>(stage, o, k, r0, r1, col, tot);
    else floats_tile<T, D, Along::columns>(stage, o, k, r0, r1, col, tot);
}

// A kernel's arguments once more, for the few workgroups that need all of them: kept in scalar registers through the passes they
// cost the others 2 to 5 percent.
template <class A>
__device__ __forceinline__ const __attribute__((address_space(4))) A *arguments_again()
{
    uintptr_t p = (uintptr_t)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return (const __attribute__((address_space(4))) A *)p;
}

// Whether the sums of a lane in one column are at least kSure times what may be left out of them, and finite.
struct Sums {
    float least = __builtin_inff(), most = 0.f;
    __device__ __forceinline__ void add(float x, float y)
    {
        least = __builtin_elementwise_minimum(__builtin_elementwise_minimum(least, __builtin_fabsf(x)), __builtin_fabsf(y));
        most = __builtin_elementwise_maximum(__builtin_elementwise_maximum(most, __builtin_fabsf(x)), __builtin_fabsf(y));
    }
    __device__ __forceinline__ bool sure(float left) const { return least >= kSure * left && most < __builtin_inff(); }
};
// A factor of a slice that is zero (or is not there) is sure of itself: it is staged as the largest power of two, and its exponent makes its
// sums zero.
constexpr int kNoFactor = -4096;
constexpr _Float16 kLargeHalf = (_Float16)32768.f;

// Passes for which a tile whose sums were not sure is formed from the floats without another try of the pairs.
constexpr int kRedoPasses = 16;

// 32 T factors from f0 on of the workgroup's tile of pair_pass_kernel.
template <int T, int D>
__device__ __forceinline__ void from_floats(u32x4 *stage, int f0)
{
    const auto *a = arguments_again<PairPass>();
    const int gx = (int)((a->n + 255) / 256), within = blockIdx.x >> 3, z = within % a->nslices;
    const int t8 = (within / a->nslices) * 8 + (blockIdx.x & 7), bx = t8 % gx, by = t8 / gx, k = a->k[z];
    if (f0 >= k) return;
    const int lane = threadIdx.x & 63, jj = lane & 31, half = lane >> 5;
    const int64_t n = a->n, jw = (int64_t)bx * 256 + (threadIdx.x & ~63u);
    const int64_t r0 = (int64_t)by * a->rps, r1 = (r0 + a->rps < a->rows) ? r0 + a->rps : a->rows;
    const Floats o{(GlobalFloats)(a->f + z * a->slice_f + f0 * a->f_col), (GlobalFloats)a->x, a->f_row, a->f_col, a->x_row, a->x_col};
    int64_t col[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) col[q] = jw + 32 * q + jj < n ? jw + 32 * q + jj : n - 1;
    f32x16 tot[T][2];
    exact_tile<T, D>(stage, o, k - f0, r0, r1, col, tot);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        if (jw + 32 * q + jj >= n) continue;
        float *dst = a->ppart + z * a->slice_ppart + ((int64_t)by * k + f0) * n + col[q];
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int f = 32 * t + acc_row(v, half);
                if (f0 + f < k) dst[(int64_t)f * n] = tot[t][q][v];
            }
    }
}

// ---------------------------------------------------------------------------
// The pass on pairs with both operands cut before: P = F^T X for slices of 32 T factors.  Workgroup = 256 columns, wave = 64 of
// them (two tiles of 32), and all four waves walk the same 16-row steps; the planes of F are staged in LDS for the four, a block
// of 8 steps at a time, double buffered, and brought to their columns' scales on the way; X' is loaded straight into operand
// registers, D steps ahead.  No vector work but that and the joins: after a block (128 terms, one scale per column of X) the
// accumulators join the totals (DEEP: and those a sum after every eighth block: with six splits of 20011 rows in one
// chain the factors were 3.4e-7 off after 20 iterations, 3.1e-7 on bf16 pieces and twelve splits, 3.0e-7 so).
//
// Microseconds per product, bf16 pieces cut in the pass -> halves cut in the pass -> this: rank 256 on 16384 x 8192 380 -> 270 ->
// 200 (T = 4: 162 would be the matrix work at the rate of a library product); 64 factors 110 -> 113 -> 98; on 20011 x 10000
// 183 -> 160 -> 133 (148 in a long run, as the clock goes); on 32768 x 16384 400 -> 365 -> 331 (a bare read: 313 to 338).  One workgroup per compute unit: two, with
// twice the splits, 111 at 64 factors on 16384 x 8192.  T = 4 at one wave per SIMD (its accumulators and totals fill half
// of the registers) loads X' once for 128 factors: 200 against 210 to 240 as two slices of 64 each.
// ---------------------------------------------------------------------------
template <int T, int D, int OCC, int POLICY, bool DEEP>
__global__ __launch_bounds__(64 * kWtaWaves, OCC) void pair_pass_kernel(const PairPass a)
{
    constexpr int KP = 32 * T, kSteps = kPairBlock / 16;
    constexpr int kRsrcFlags = 0x00020000;   // raw buffer, 32-bit data format (gfx9 family)
    constexpr int kUnits = kSteps * 4 * KP;            // 16-byte units of planes in a block
    constexpr int kEach = kUnits / 256 / kSteps;       // a thread stages so many per step
    extern __shared__ u32x4 pst[];                     // two blocks
    __shared__ __align__(16) int fexp[KP];
    __shared__ int redone;                             // the tile's sums are not sure
    __shared__ int before;                             // passes for which it is formed from the floats as it is
    const int64_t rows = a.rows, n = a.n, ldx = a.X.ld;
    const int gx = (int)((n + 255) / 256), ldf = a.ldf;
    const int L = blockIdx.x, within = L >> 3;
    const int z = within % a.nslices;
    const int t8 = (within / a.nslices) * 8 + (L & 7);
    const int k = a.k[z];
    if (a.gtiles)
        sum_tile_sets(a.gtiles + z * a.slice_gtiles, a.nsets, k, a.gsum + z * a.slice_gsum, (int)gridDim.x / a.nslices - 1 - t8,
                      (int)gridDim.x / a.nslices);
    if (t8 >= gx * a.splits) return;      // on small matrices there are workgroups for the tiles alone
    const int bx = t8 % gx, by = t8 / gx;
    const u32x4 *F = static_cast<const u32x4 *>(a.F.units) + z * a.slice_units;
    const unsigned char *exps = a.F.exps + z * a.slice_exps;
    const unsigned *most = a.F.most + z * a.slice_most;
    float *ppart = a.ppart + z * a.slice_ppart;
    const u32x4 *X = static_cast<const u32x4 *>(a.X.units);
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int jj = lane & 31, half = lane >> 5;
    if (L == 0)
        for (int i = tid; i < a.nclear; i += 256) a.clear[i] = 0u;
    const int64_t jw = (int64_t)bx * 256 + 64 * w;
    const int64_t r0 = (int64_t)by * a.rps;
    const int64_t r1 = (r0 + a.rps < rows) ? r0 + a.rps : rows;
    // columns past the edge of X' read its last ones, whose sums are not stored
    unsigned xoff[2];
    int64_t xcol[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        xcol[q] = jw + 32 * q + jj < ldx ? jw + 32 * q + jj : ldx - 1;
        xoff[q] = (unsigned)((half * 2 * ldx + xcol[q]) * 16);
    }
    const unsigned xpiece = (unsigned)(ldx * 16);

    f32x16 acc[T][2], tot[T][2], sum[T][2];
    float unit[2] = {0.f, 0.f};            // what is left out of the sums of a column at most
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int q = 0; q < 2; ++q) tot[t][q] = sum[t][q] = f32x16{0};
    const int64_t redo = (int64_t)t8 * a.nslices + z;
    const int asked = tid == 0 ? (int)a.redo[redo] : 0;
    struct Stage { u32x4 x[2][2]; };
    Stage xs[D];
    auto load_x = [&](Stage &s, int64_t ib) {
        const int64_t i = ib < r1 ? ib : r0;           // past the end: anything that is there
        const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<u32x4 *>(X + (i >> 3) * 2 * ldx), 0, (int)(4 * xpiece), kRsrcFlags);
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int p = 0; p < 2; ++p) s.x[q][p] = __builtin_amdgcn_raw_buffer_load_b128(rx, xoff[q] + p * xpiece, 0, POLICY);
    };
    // planes of the block of rows from ib on; groups past the last row read as zero
    const int64_t groups = (rows + 7) >> 3;
    const int fc = tid & (KP - 1), fg = tid / KP;      // unit e of a thread: row group and piece fg + e * 256 / KP, column fc
    const unsigned ftop = fc < k ? column_most(most, ldf, fc) : 0u;
    const int fce = half_exponent(ftop);
    const _Float16 fill = ftop ? (_Float16)0.f : kLargeHalf;
    if (tid < KP) fexp[tid] = ftop ? fce - 14 : kNoFactor;      // read after the first barrier
    if (tid == 0) redone = 0;
    struct Rsrc { __amdgpu_buffer_rsrc_t u, e; };
    auto rsrc_f = [&](int64_t ib) {
        int64_t ng = ib < r1 ? groups - (ib >> 3) : 0;
        ng = ng < 0 ? 0 : (ng > 2 * kSteps ? 2 * kSteps : ng);
        const int64_t g = ng ? ib >> 3 : 0;
        return Rsrc{__builtin_amdgcn_make_buffer_rsrc(const_cast<u32x4 *>(F + g * 2 * ldf), 0, ng ? (int)(((ng * 2 - 1) * ldf + KP) * 16) : 0,
                                                      kRsrcFlags),
                    __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char *>(exps + g * ldf), 0, ng ? (int)((ng - 1) * ldf + KP) : 0,
                                                      kRsrcFlags)};
    };
    struct Units { u32x4 u[kEach]; unsigned e[kEach]; };
    Units th[3];
    auto load_f = [&](Units &t, const Rsrc &r, int s) {
#pragma unroll
        for (int e = 0; e < kEach; ++e) {
            const int gp = fg + (s * kEach + e) * (256 / KP);
            t.u[e] = __builtin_amdgcn_raw_buffer_load_b128(r.u, (unsigned)(gp * ldf + fc) * 16, 0, 0);
            t.e[e] = __builtin_amdgcn_raw_buffer_load_b8(r.e, (unsigned)((gp >> 1) * ldf + fc), 0, 0);
        }
    };
    auto store_f = [&](const Units &t, u32x4 *dst, int s) {
#pragma unroll
        for (int e = 0; e < kEach; ++e) dst[(s * kEach + e) * 256 + tid] = to_column_scale<T == 4>(t.u[e], t.e[e], fce, fill);
    };

#pragma unroll
    for (int s = 0; s < D; ++s) {
        load_x(xs[s], r0 + 16 * s);
        __builtin_amdgcn_sched_barrier(0);
    }
    {
        const Rsrc rf = rsrc_f(r0);
        Units first[kSteps];               // one trip to memory
#pragma unroll
        for (int s = 0; s < kSteps; ++s) load_f(first[s], rf, s);
#pragma unroll
        for (int s = 0; s < kSteps; ++s) store_f(first[s], pst, s);
    }
    if (tid == 0) before = asked;          // one look for all four waves: the word changes below
    __syncthreads();
    const int again = __builtin_amdgcn_readfirstlane(before);
    if (!again) {
        int buf = 0;
        for (int64_t i = r0; i < r1; i += kPairBlock) {
            const Rsrc rf = rsrc_f(i + kPairBlock);
            u32x4 *mine = pst + buf * kUnits, *next = pst + (buf ^ 1) * kUnits;
            float inv[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const float2 s = a.X.scale[i / kPairBlock * ldx + xcol[q]];
                inv[q] = s.x;
                unit[q] += s.y;
            }
#pragma unroll
            for (int s = 0; s < kSteps; ++s) {
                load_f(th[s % 3], rf, s);      // the next block's planes, stored two steps later
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    u32x4 wt[2];
#pragma unroll
                    for (int pl = 0; pl < 2; ++pl) wt[pl] = mine[((2 * s + half) * 2 + pl) * KP + 32 * t + jj];
                    constexpr int PW[3] = {1, 0, 0}, PA[3] = {0, 1, 0};   // smallest first
#pragma unroll
                    for (int e = 0; e < 3; ++e)
#pragma unroll
                        for (int q = 0; q < 2; ++q)
                            acc[t][q] = mfma_f16(wt[PW[e]], xs[s % D].x[q][PA[e]], s == 0 && e == 0 ? f32x16{0} : acc[t][q]);
                }
                load_x(xs[s % D], i + 16 * (s + D));
                if (s >= 2) store_f(th[(s - 2) % 3], next, s - 2);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int s = kSteps - 2; s < kSteps; ++s) store_f(th[s % 3], next, s);
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int v = 0; v < 16; ++v) tot[t][q][v] = __builtin_fmaf(acc[t][q][v], inv[q], tot[t][q][v]);
            if (DEEP && ((i - r0) / kPairBlock & 7) == 7) {
#pragma unroll
                for (int t = 0; t < T; ++t)
#pragma unroll
                    for (int q = 0; q < 2; ++q) sum[t][q] += tot[t][q], tot[t][q] = f32x16{0};
            }
            __syncthreads();    // the next block's planes are written, this block's are read
            buf ^= 1;
        }
        if (DEEP) {
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int q = 0; q < 2; ++q) tot[t][q] += sum[t][q];
        }
        unsigned off[2];                   // of a lane's columns in four rows of factors on; past the edge out of reach
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            Sums sums;
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int v = 0; v < 16; v += 2) sums.add(tot[t][q][v], tot[t][q][v + 1]);
            const bool in = jw + 32 * q + jj < n;
            off[q] = in ? ((unsigned)(4 * half) * (unsigned)n + (unsigned)(jw + 32 * q + jj)) * 4u : 0xffffffffu;
            if (in && !sums.sure(unit[q])) redone = 1;
        }
        // register v is factor 32 t + v % 4 + 8 (v / 4), or four on: a descriptor holds both rows, or the first if the second is past k
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const i32x4 e = *reinterpret_cast<const i32x4 *>(&fexp[32 * t + 8 * g + 4 * half]);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int f = 32 * t + 8 * g + u;
                    const __amdgpu_buffer_rsrc_t row = __builtin_amdgcn_make_buffer_rsrc(
                        ppart + ((int64_t)by * k + (f < k ? f : 0)) * n, 0, (int)(f + 4 < k ? 5 * n * 4 : f < k ? n * 4 : 0), kRsrcFlags);
#pragma unroll
                    for (int q = 0; q < 2; ++q)
                        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(ldexpf(tot[t][q][4 * g + u], e[u])), row, off[q], 0, 0);
                }
            }
        __syncthreads();
        if (!__builtin_amdgcn_readfirstlane(redone)) return;
    }
    // so are the next passes' tiles: such data stays so for a while
    if (tid == 0) a.redo[redo] = again ? again - 1 : kRedoPasses;
    // as many factors at once as the registers hold
    constexpr int kAtOnce = OCC == 1 ? 2 : 1, kAhead = OCC == 1 ? 4 : 2;
    from_floats<kAtOnce, kAhead>(pst, 0);
    if (T > kAtOnce) from_floats<kAtOnce, kAhead>(pst, 32 * kAtOnce);
}

// ---------------------------------------------------------------------------
// The pass for slices of 64 factors on pairs of halves (aligned A, n % 4 == 0, 64 n < 2^31; pair planes), for X that
// is not cut before.  Workgroup = 256 columns, wave = 64 of them (lane = 2 consecutive columns), the planes of a
// group of steps staged in LDS for the four waves, three register stages of A.  12 matrix instructions per 16 rows x 64
// columns x 64 factors instead of 24.  The accumulators join the totals after every group, 96 terms (192: a
// contraction over 384 factors 8e-8 off, so 4e-8).
// Ranks above 64 were bound by the matrix cores (power) on bf16 pieces; rank 256 on 16384 x 8192: 380 -> 270 us per product
// (of which loads without the matrix work 210, the matrix work without the loads 220), whole iterations 937 -> 718,
// error against 64 bits after five iterations 2.4 -> 2.3e-7.
//
// Scale of a column of A: a column of the accumulators belongs to a lane pair (l, l + 32), so the scale may change from group to
// group as long as the accumulators are unscaled when they join the totals (one fused multiply-add each).  The running maximum
// of a column's magnitudes costs half an instruction per element; if an element would leave the halves' range
// (2^15), the wave joins what it has to the totals and scales anew: the largest entry seen goes to 2^11, so that entries up to
// 8 times as large come without another change, and after every join the scale follows the maximum since the last one.
// ---------------------------------------------------------------------------
// Several 64-factor slices of a wider factor in one launch: workgroup L of a one-dimensional grid stands for (tile, slice) with
// the slices of one tile of A (slab x row split) 8 workgroups apart, i.e. on the same XCD at about the same time, so that A
// comes from HBM once and from that XCD's L2 for the other slices (default cache policy).  Slice z reads columns 64 z .. of
// the planes and writes ppart + z * slice_ppart; it holds min(64, ktotal - 64 z) factors.
struct PairSlices {
    const float *X, *f;                // X; F itself, rows x k
    PairFactor F;
    float *ppart;
    int64_t rows, n, rps, slice_ppart;
    int ldf, k, gx, gy, nslices;
};
__global__ __launch_bounds__(64 * kWtaWaves, 2) void wta_pass_pair_kernel(const PairSlices args)
{
    const float *A = args.X;
    const PairFactor &F = args.F;
    const int ldf = args.ldf, gx = args.gx, gy = args.gy, nslices = args.nslices;
    const int64_t rows = args.rows, n = args.n, rps = args.rps;
    int k = args.k;
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    constexpr int KP = 64;
    constexpr int kRsrcFlags = 0x00020000;   // raw buffer, 32-bit data format (gfx9 family)
    constexpr int kSteps = 6;                          // 16-row steps per group of staged planes
    constexpr int kUnits = kSteps * 2 * 2 * KP;        // 16-byte units of planes in a group
    constexpr float kMost = 32768.f;
    __shared__ u32x4 lds[2 * kUnits];                  // two groups; as much as floats_tile needs
    __shared__ int fexp[KP];
    __shared__ int redone;                             // the tile's sums are not sure
    const int L = blockIdx.x, within = L >> 3;
    const int z = within % nslices;
    const int t8 = (within / nslices) * 8 + (L & 7);
    if (t8 >= gx * gy) return;
    const int bx = t8 % gx, by = t8 / gx;
    const u32x4 *units = static_cast<const u32x4 *>(F.units) + KP * z;
    const unsigned char *exps = F.exps + KP * z;
    const unsigned *fmost = F.most + KP * z;
    float *ppart = args.ppart + (int64_t)z * args.slice_ppart;
    k = (k - 64 * z < 64) ? k - 64 * z : 64;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int jj = lane & 31, half = lane >> 5;
    const int64_t jw = (int64_t)bx * 256 + 64 * w;
    const bool live = jw < n;   // a wave wholly past the edge only helps to stage the planes
    const int64_t colr = jw + 2 * jj;
    const int64_t col = colr < n ? colr : 0;   // lanes past the edge read valid data that is never stored
    const int64_t r0 = (int64_t)by * rps;
    const int64_t r1 = (r0 + rps < rows) ? r0 + rps : rows;
    const unsigned rowb = (unsigned)(n * 4);
    const unsigned loff = (unsigned)(half * 8) * rowb + (unsigned)col * 4;
    const int64_t ngroups = (rows + 7) >> 3;
    const int fc = tid & 63, fg = tid >> 6;      // unit e of a thread: row group and piece fg + 4 e, column fc
    const unsigned ftop = fc < k ? column_most(fmost, ldf, fc) : 0u;
    const int fce = half_exponent(ftop);
    const _Float16 fill = ftop ? (_Float16)0.f : kLargeHalf;
    if (tid < KP) fexp[tid] = ftop ? fce - 14 : kNoFactor;      // read after the first barrier
    if (tid == 0) redone = 0;

    f32x16 acc[2][2], tot[2][2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int q = 0; q < 2; ++q) acc[t][q] = f32x16{0}, tot[t][q] = f32x16{0};
    // per column: scale, its inverse, largest magnitude since the last join
    float sc[2], inv[2], most[2] = {0.f, 0.f}, unit[2] = {0.f, 0.f};      // unit: what is left out at most, one in the scaled range of each join
#pragma unroll
    for (int q = 0; q < 2; ++q) sc[q] = power_of_two(126), inv[q] = power_of_two(-126);

    struct Stage { u32x2 a[8]; };
    auto load_stage = [&](Stage &s, int64_t ib) {
        int64_t av = live ? r1 - ib : 0;            // rows of this step inside the split
        av = av < 0 ? 0 : (av > 16 ? 16 : av);
        const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float *>(A + (av ? ib : 0) * n), 0, (int)(av * rowb), kRsrcFlags);
#pragma unroll
        for (int r = 0; r < 8; ++r) s.a[r] = __builtin_amdgcn_raw_buffer_load_b64(ra, loff + r * rowb, 0, 0);
    };
    // a third of the planes of the group of rows from ib on: 2 units per thread
    struct Third { u32x4 u[2]; unsigned e[2]; };
    auto load_third = [&](Third &p, int64_t ib, int part) {
        const int64_t g = ib >> 3;
        int64_t ng = ib < r1 ? ngroups - g : 0;     // 8-row groups of planes that exist
        ng = ng < 0 ? 0 : (ng > 2 * kSteps ? 2 * kSteps : ng);
        const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<u32x4 *>(units + (ng ? g * 2 * ldf : 0)), 0, ng ? (int)(((ng * 2 - 1) * ldf + KP) * 16) : 0, kRsrcFlags);
        const __amdgpu_buffer_rsrc_t re = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<unsigned char *>(exps + (ng ? g * ldf : 0)), 0, ng ? (int)((ng - 1) * ldf + KP) : 0, kRsrcFlags);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int gp = fg + 4 * (2 * part + e);
            p.u[e] = __builtin_amdgcn_raw_buffer_load_b128(rp, (unsigned)(gp * ldf + fc) * 16, 0, 0);
            p.e[e] = __builtin_amdgcn_raw_buffer_load_b8(re, (unsigned)((gp >> 1) * ldf + fc), 0, 0);
        }
    };
    auto store_third = [&](const Third &p, int buf, int part) {
#pragma unroll
        for (int e = 0; e < 2; ++e) lds[buf * kUnits + (2 * part + e) * 256 + tid] = to_column_scale<true>(p.u[e], p.e[e], fce, fill);
    };
    // the accumulators join the totals; the scales follow the maxima
    auto join = [&]() {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    tot[t][q][v] = __builtin_fmaf(acc[t][q][v], inv[q], tot[t][q][v]);
                    acc[t][q][v] = 0.f;
                }
            const float both = fmaxf(most[q], __shfl_xor(most[q], 32));
            // under the first scale `most` knows all that was added up; a column of zeros has no unit
            unit[q] += both > 0.f || sc[q] < power_of_two(126) ? inv[q] : 0.f;
            if (both > 0.f) {
                const int e = half_exponent(__float_as_uint(both));
                sc[q] = power_of_two(11 - e > 126 ? 126 : 11 - e);
                inv[q] = power_of_two(11 - e > 126 ? -126 : e - 11);
            }
            most[q] = 0.f;
        }
    };
    auto compute = [&](const Stage &c, int buf, int st) {
        u32x4 wt[2][2];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int pl = 0; pl < 2; ++pl) wt[t][pl] = lds[buf * kUnits + ((2 * st + half) * 2 + pl) * KP + 32 * t + jj];
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int r = 0; r < 8; ++r) most[q] = fmaxf(most[q], __builtin_fabsf(__uint_as_float(c.a[r][q])));
        if (__any(most[0] * sc[0] >= kMost || most[1] * sc[1] >= kMost)) join();
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            u32x4 at[2];
#pragma unroll
            for (int pr = 0; pr < 4; ++pr)
                cut2h(__uint_as_float(c.a[2 * pr][q]), __uint_as_float(c.a[2 * pr + 1][q]), sc[q], at, pr);
            constexpr int PW[3] = {1, 0, 0}, PA[3] = {0, 1, 0};   // smallest first
#pragma unroll
            for (int e = 0; e < 3; ++e)
#pragma unroll
                for (int t = 0; t < 2; ++t) acc[t][q] = mfma_f16(wt[t][PW[e]], at[PA[e]], acc[t][q]);
        }
    };
    Stage s0, s1, s2;
    Third th;
    load_stage(s0, r0);
    __builtin_amdgcn_sched_barrier(0);   // issue order = age order, also here: the waits in the loop count loads in flight
    load_stage(s1, r0 + 16);
#pragma unroll
    for (int part = 0; part < 3; ++part) {
        load_third(th, r0, part);
        store_third(th, 0, part);
    }
    __syncthreads();
    int buf = 0;
    for (int64_t i = r0; i < r1; i += 16 * kSteps) {
#pragma unroll
        for (int part = 0; part < 3; ++part) {
            const int64_t ib = i + 32 * part;
            Stage &x = part == 0 ? s0 : (part == 1 ? s2 : s1);
            Stage &y = part == 0 ? s1 : (part == 1 ? s0 : s2);
            Stage &z2 = part == 0 ? s2 : (part == 1 ? s1 : s0);
            load_third(th, i + 16 * kSteps, part);
            load_stage(z2, ib + 32);
            __builtin_amdgcn_sched_barrier(0);
            if (live && ib < r1) compute(x, buf, 2 * part);
            __builtin_amdgcn_sched_barrier(0);
            load_stage(x, ib + 48);
            __builtin_amdgcn_sched_barrier(0);
            if (live && ib + 16 < r1) compute(y, buf, 2 * part + 1);
            __builtin_amdgcn_sched_barrier(0);
            store_third(th, buf ^ 1, part);
        }
        join();
        __syncthreads();    // the next group's planes are written, this group's are read
        buf ^= 1;
    }
    join();
    float *dst = ppart + (int64_t)by * k * n + colr;
    auto store = [&](int t, const f32x16 (&sums)[2], bool scaled) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int c = 32 * t + acc_row(v, half);
            const int e = scaled ? fexp[c] : 0;
            if (c < k && colr < n) *reinterpret_cast<f32x2 *>(dst + (int64_t)c * n) = f32x2{ldexpf(sums[0][v], e), ldexpf(sums[1][v], e)};
        }
    };
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        Sums sums;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int v = 0; v < 16; v += 2) sums.add(tot[t][q][v], tot[t][q][v + 1]);
        if (colr < n && !sums.sure(unit[q])) redone = 1;
    }
    store(0, tot[0], true);
    store(1, tot[1], true);
    __syncthreads();
    if (!__builtin_amdgcn_readfirstlane(redone)) return;
    // 32 factors at a time, as many as the registers hold
    auto again = [&](int t) {
        const auto *b = arguments_again<PairSlices>();
        const Floats floats{(GlobalFloats)(b->f + KP * z + 32 * t), (GlobalFloats)b->X, b->k, 1, b->n, 1};
        const int64_t cols[2] = {col, col + 1};
        f32x16 some[1][2];
        floats_tile<1, 2, Along::rows>(lds, floats, k - 32 * t, r0, r1, cols, some);
        store(t, some[0], false);
    };
    again(0);
    if (k > 32) again(1);
}

// ---------------------------------------------------------------------------
// Update behind the products of ranks above 64: X[c][j] <- X[c][j] * (sum of the numerator's partials) / (sum of the denominator's +
// eps) for a tile of 64 factors (blockIdx.y) x CW columns, and from it X^T and its pair planes for the next half of
// the iteration.  As sums of either product, an element-wise update, a transpose and a split with
// its cleared maxima (seven launches) 56 us and more per half of an iteration at rank 256 on 16384 x 8192, now 21 to 29 (with
// tiles of 64 columns 33 to 42: what counts is loads in flight).
// clear: maxima to set to zero on the way.
// ---------------------------------------------------------------------------
template <int CW>
__global__ __launch_bounds__(256) void sliced_update_kernel(const SlicedUpdate a)
{
    constexpr int FG = 256 / CW, NE = 64 / FG;             // factors side by side, entries of a thread
    __shared__ float tile[64][CW + 1];
    __shared__ unsigned most[64];
    const int tid = threadIdx.x, jl = tid % CW, fl = tid / CW, f0 = 64 * (int)blockIdx.y;
    const int kb = a.k - f0 < 64 ? a.k - f0 : 64;          // factors of this block
    const int64_t j0 = (int64_t)blockIdx.x * CW, j = j0 + jl, len = a.len;
    const bool okj = j < len;
    if (tid < 64) most[tid] = 0u;
    if (blockIdx.x == 0 && blockIdx.y == 0)
        for (int i = tid; i < a.nclear; i += 256) a.clear[i] = 0u;
    // the partials of the numerator: slices of `width` factors; of the denominator: of 64
    const int zn = f0 / a.width, kn = a.k - a.width * zn < a.width ? a.k - a.width * zn : a.width;
    const float *num = a.num + ((int64_t)zn * a.snum * a.width + f0 - a.width * zn) * len;
    const float *den = a.den + (int64_t)blockIdx.y * a.sden * 64 * len;
    float old[NE], p[NE], d[NE];
    int64_t at[NE];
    bool ok[NE];
#pragma unroll
    for (int i = 0; i < NE; ++i) {
        const int c = fl + FG * i;
        ok[i] = okj && c < kb;
        at[i] = ok[i] ? (int64_t)c * len + j : 0;
        old[i] = ok[i] ? a.X[(int64_t)f0 * len + at[i]] : 0.f;
        p[i] = d[i] = 0.f;
    }
    auto add = [&](float (&sum)[NE], const float *from, int splits, int64_t stride) {
        int t = 0;
        for (; t + 4 <= splits; t += 4) {
            float v[NE][4];
#pragma unroll
            for (int i = 0; i < NE; ++i)
#pragma unroll
                for (int u = 0; u < 4; ++u) v[i][u] = ok[i] ? from[at[i] + (t + u) * stride] : 0.f;
#pragma unroll
            for (int i = 0; i < NE; ++i)
                sum[i] += (v[i][0] + v[i][1]) + (v[i][2] + v[i][3]);
        }
        for (; t < splits; ++t) {
            float v[NE];
#pragma unroll
            for (int i = 0; i < NE; ++i) v[i] = ok[i] ? from[at[i] + t * stride] : 0.f;
#pragma unroll
            for (int i = 0; i < NE; ++i) sum[i] += v[i];
        }
    };
    if (kb > 0) {
        add(p, num, a.snum, (int64_t)kn * len);
        add(d, den, a.sden, (int64_t)kb * len);
    }
#pragma unroll
    for (int i = 0; i < NE; ++i) {
        float x = 0.f;
        if (ok[i]) {
            x = old[i] * p[i] / (d[i] + a.eps);
            a.X[(int64_t)f0 * len + at[i]] = x;
        }
        tile[fl + FG * i][jl] = x;
    }
    __syncthreads();
    // X^T: rows of the tile's columns
    const int cl = tid & 63, w = tid >> 6;
#pragma unroll
    for (int row = w; row < CW; row += 4)
        if (j0 + row < len && cl < kb) a.Xt[(j0 + row) * a.k + f0 + cl] = tile[cl][row];
    // its planes; columns beyond k are zero
    for (int u = w; u < CW / 8; u += 4) {
        const int64_t g = j0 / 8 + u;
        if (g * 8 < len) {
            float x[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = tile[cl][8 * u + e];
            const unsigned t = put_pairs(x, static_cast<u32x4 *>(a.F.units) + g * 2 * a.ld + f0 + cl, a.ld, a.F.exps + g * a.ld + f0 + cl);
            if (t) atomicMax(&most[cl], t);
        }
    }
    __syncthreads();
    if (tid < kb && most[tid]) atomicMax(a.F.most + (int)(blockIdx.x % kPairCopies) * a.ld + f0 + tid, most[tid]);
}

// ---------------------------------------------------------------------------
// Factors of stacked runs: blockIdx.y = run; the first wblocks blocks turn 64 rows of its W each through LDS, the others
// copy its H.  One launch a slice instead of two or three copies a run.
// ---------------------------------------------------------------------------
template <bool IN>
__global__ __launch_bounds__(256) void stack_kernel(const StackedRuns runs, float *__restrict__ Wt, float *__restrict__ Hs, int64_t m,
                                                    int64_t n, int64_t wblocks)
{
    __shared__ float tile[64][65];
    const int run = blockIdx.y, k = runs.k[run], at = runs.at[run], tid = threadIdx.x;
    if ((int64_t)blockIdx.x >= wblocks) {
        float *one = runs.H[run], *all = Hs + at * n;
        const int64_t count = k * n, step = (int64_t)(gridDim.x - wblocks) * 256;
        for (int64_t e = ((int64_t)blockIdx.x - wblocks) * 256 + tid; e < count; e += step) {
            if (IN) all[e] = one[e];
            else one[e] = all[e];
        }
        return;
    }
    float *W = runs.W[run];
    const int64_t r0 = (int64_t)blockIdx.x * 64;
    const int rows = m - r0 < 64 ? (int)(m - r0) : 64;
    if (IN) {
        for (int e = tid; e < rows * k; e += 256) tile[e % k][e / k] = W[r0 * k + e];
        __syncthreads();
        for (int e = tid; e < 64 * k; e += 256)
            if ((e & 63) < rows) Wt[(at + (e >> 6)) * m + r0 + (e & 63)] = tile[e >> 6][e & 63];
    } else {
        for (int e = tid; e < 64 * k; e += 256)
            if ((e & 63) < rows) tile[e >> 6][e & 63] = Wt[(at + (e >> 6)) * m + r0 + (e & 63)];
        __syncthreads();
        for (int e = tid; e < rows * k; e += 256) W[r0 * k + e] = tile[e % k][e / k];
    }
}

// ---------------------------------------------------------------------------
// Host side launchers
// ---------------------------------------------------------------------------

hipError_t launch_cut_pairs(const float *A, int64_t m, int64_t n, const PairMatrix &a, const PairMatrix &at, unsigned *clear, int nclear,
                            hipStream_t st)
{
    const int64_t tiles = ((m + kCutTile - 1) / kCutTile) * ((n + kCutTile - 1) / kCutTile);
    if (tiles > 0x7fffffff) return hipErrorInvalidValue;
    if ((reinterpret_cast<uintptr_t>(A) & 15u) == 0 && (n & 3) == 0)
        hipLaunchKernelGGL(cut_pairs_kernel<true>, dim3((unsigned)tiles), dim3(512), 0, st, A, m, n, a, at, clear, nclear);
    else
        hipLaunchKernelGGL(cut_pairs_kernel<false>, dim3((unsigned)tiles), dim3(512), 0, st, A, m, n, a, at, clear, nclear);
    return hipGetLastError();
}

hipError_t launch_split_pairs(const float *X, int64_t rows, int k, const PairFactor &f, int ld, hipStream_t st, unsigned *clear)
{
    const int64_t groups = (rows + 7) / 8;
    hipLaunchKernelGGL(split_pairs_kernel, dim3((unsigned)((groups + 31) / 32), (unsigned)(ld / 64)), dim3(256), 0, st, X, rows, k, f, ld,
                       clear);
    return hipGetLastError();
}

hipError_t launch_sliced_update(const SlicedUpdate &a, hipStream_t st)
{
    // every 64 columns of the planes: those beyond k are read by slices of 128
    const int cw = a.len * (a.ld / 64) >= 32 * 1024 ? 32 : 16;      // 1024 workgroups, or as many as there are
    const int64_t blocks = (a.len + cw - 1) / cw;
    if (blocks > 0x7fffffff || a.k > a.ld) return hipErrorInvalidValue;
    const dim3 grid((unsigned)blocks, (unsigned)(a.ld / 64));
    if (cw == 32) hipLaunchKernelGGL(sliced_update_kernel<32>, grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL(sliced_update_kernel<16>, grid, dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_stack(const StackedRuns &runs, int count, bool in, float *Wt, float *H, int64_t m, int64_t n, hipStream_t st)
{
    const int64_t wblocks = (m + 63) / 64, hblocks = (n + 63) / 64;
    if (wblocks + hblocks > 0x7fffffff) return hipErrorInvalidValue;
    const dim3 grid((unsigned)(wblocks + hblocks), (unsigned)count);
    if (in) hipLaunchKernelGGL(stack_kernel<true>, grid, dim3(256), 0, st, runs, Wt, H, m, n, wblocks);
    else hipLaunchKernelGGL(stack_kernel<false>, grid, dim3(256), 0, st, runs, Wt, H, m, n, wblocks);
    return hipGetLastError();
}

hipError_t launch_pair_slices(const float *X, int64_t rows, int64_t n, int k, const float *F, const PairFactor &f, int ld,
                              float *ppart, int splits, int64_t rps, hipStream_t st)
{
    if (wta_planes_only_width(X, n) != 64 || rps % 16) return hipErrorInvalidValue;
    const int nslices = (k + 63) / 64;
    const int gx = (int)((n + 255) / 256), gy = splits;
    const int64_t tiles8 = ((int64_t)gx * gy + 7) / 8 * 8;
    const PairSlices args{X, F, f, ppart, rows, n, rps, (int64_t)splits * 64 * n, ld, k, gx, gy, nslices};
    hipLaunchKernelGGL(wta_pass_pair_kernel, dim3((unsigned)(tiles8 * nslices)), dim3(64 * kWtaWaves), 0, st, args);
    return hipGetLastError();
}

template <int T, int D, int OCC, int POLICY, bool DEEP>
static hipError_t pair_pass_launch(dim3 grid, hipStream_t st, const PairPass &p)
{
    constexpr int kLdsBytes = 2 * (kPairBlock / 16) * 4 * 32 * T * 16;
    static bool raised = false;      // more dynamic LDS than the default limit: asked for once per process
    if (!raised) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&pair_pass_kernel<T, D, OCC, POLICY, DEEP>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
        if (e != hipSuccess) return e;
        raised = true;
    }
    hipLaunchKernelGGL((pair_pass_kernel<T, D, OCC, POLICY, DEEP>), grid, dim3(64 * kWtaWaves), kLdsBytes, st, p);
    return hipGetLastError();
}

hipError_t launch_pair_pass(const PairPass &p, int tiles, bool stream, hipStream_t st)
{
    if (p.rps % kPairBlock || p.nslices < 1 || p.nslices > kPairSlices || (int64_t)(p.splits - 1) * p.rps >= p.rows ||
        p.X.ld >= ((int64_t)1 << 25) || p.X.ld < p.n || !p.f || !p.x || !p.redo)
        return hipErrorInvalidValue;
    for (int z = 0; z < p.nslices; ++z)
        if (p.k[z] < 1 || p.k[z] > 32 * tiles) return hipErrorInvalidValue;      // a pass that stores nothing, or not all
    int64_t tiles8 = ((p.n + 255) / 256 * p.splits + 7) / 8 * 8;
    if (p.gtiles && tiles8 < 192) tiles8 += 64;      // a workgroup per 64 entries of the Gram matrix
    const dim3 grid((unsigned)(tiles8 * p.nslices));
    if (tiles == 4) return stream ? pair_pass_launch<4, 4, 1, 2, false>(grid, st, p) : pair_pass_launch<4, 4, 1, 0, false>(grid, st, p);
    // slices that share X' keep it in the L2 for each other: three on 16384 x 8192 160 us per product, 230 marked for early eviction
    if (p.nslices > 1) return pair_pass_launch<2, 2, 2, 0, false>(grid, st, p);
    return stream ? pair_pass_launch<2, 4, 1, 2, true>(grid, st, p) : pair_pass_launch<2, 4, 1, 0, true>(grid, st, p);
}

// Workgroups side by side: one per compute unit; slices of 64 that share X' two.  The cost of `s` splits in blocks of 128 rows, as the
// workgroups walk them: rounds of workgroups times the blocks of each, half a block for its start and end, and the partial results, which are
// written and read again, against the bytes of a block in all places, with what the update's chain of reads waits for each.  Whole blocks of
// rows to each.  (Before, the fewest that leave the last round of workgroups nearly full, whatever they cost: 111913 x 448, k = 36 went
// over A^T in four splits of one block, 205 us an iteration, 177 on the mirrored plan, 167 now in one; 178 shapes as for pairs_least 1.03 times as
// fast, slower than the plan before 15, now 2, by 2 percent.)
int pair_splits(int64_t rows, int64_t cols, int tiles, int nslices)
{
    const int64_t blocks = (rows + kPairBlock - 1) / kPairBlock, slabs = (cols + 255) / 256, per = slabs * nslices;
    const int64_t places = tiles == 4 || nslices == 1 ? 256 : 512;
    const int64_t cap = slabs >= 16 ? 32 : 128, most = blocks < cap ? blocks : cap;
    const double block = (double)places / nslices * kPairBlock * 256 * 4, partial = 2.0 * 32 * tiles * nslices * (double)cols * 4;
    int64_t best = 1;
    double least = 0.0;
    for (int64_t s = 1; s <= most; ++s) {
        const int64_t each = (blocks + s - 1) / s, rounds = (per * s + places - 1) / places;
        const double cost = (double)rounds * ((double)each + 0.5) + (double)s * (partial / block + 0.015);
        if (s == 1 || cost < least) {
            least = cost;
            best = s;
        }
    }
    const int64_t each = (blocks + best - 1) / best;
    return (int)((blocks + each - 1) / each);
}

}  // namespace nmfmu
