// CSR kernels of the multiplicative-update iteration for gfx950 (MI355X).
//
// With A in CSR (paper, section 2.3: values, column indices, row pointers) the
// two products over A become sums over stored entries.  Both are run as
// gathers against a row-major factor table, so that one stored entry touches
// one contiguous run of k floats and no atomics are needed:
//   A H^T : Q[i][:]  = sum over the entries (i, j, a) of row i    of a * Ht[j][:]
//   W^T A : Pt[j][:] = sum over the entries (i, j, a) of column j of a * W[i][:]
// The first walks the caller's CSR arrays (read-only, never copied); the
// second walks a column-ordered copy (CSC: column pointers, row indices,
// values) that is built once per call by a stable radix sort of the column
// indices, so entries of a column keep their row order and sums are
// reproducible.  The two updates are then one kernel used twice (the H update
// is the W update of the transposed problem), each with its update fused.
// The sparse iteration works on Ht = H^T (n x k); H is transposed on entry
// and on exit.
//
// Work mapping: a row (of A for the W update, of A^T for the H update) is
// handled by a group of LPR lanes, LPR = smallest power of two >= k (at least
// 4): lane c of the group owns factor index c.  A wave holds 64 / LPR rows, so
// short rows are packed several to a wave.  The group reads its row's entries
// LPR at a time with coalesced loads and hands them round (from_lane for 5 to 16 factors, else lane shuffles).
// From 64 entries per row on average a whole wave takes one row at a time.
// Rows are dealt to wavefronts in contiguous ranges of equal work (stored
// entries plus a per-row cost), and rows too long for one wave are split
// over a whole workgroup.
#include <utility>

#include <hipcub/hipcub.hpp>

#include "nmfmu_internal.h"

namespace nmfmu {

template <int LPR>
__device__ __forceinline__ float group_bcast(float v, int src)
{
    return __shfl(v, src, LPR);
}
template <int LPR>
__device__ __forceinline__ int group_bcast(int v, int src)
{
    return __shfl(v, src, LPR);
}

// f(0), f(1), ... f(N - 1) with constant arguments.
template <int... I, class F>
__device__ __forceinline__ void for_each_index(std::integer_sequence<int, I...>, F f)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void unrolled(F f) { for_each_index(std::make_integer_sequence<int, N>{}, f); }

// The value of lane SRC of a group of 8 or 16 lanes, in all of its lanes, by data-parallel primitives of the vector unit:
// a shuffle goes through the LDS unit, and with two for every entry and one for every factor of the update that unit was what the
// launches on small tables waited for.  All lanes of the wave have to be active.  (Groups of 4: the registers spill, 0.94x.)
constexpr bool by_lane(int lpr) { return lpr == 8 || lpr == 16; }
template <int LPR, int SRC>
__device__ __forceinline__ int from_lane(int v)
{
    constexpr int kRowLane = 0x150;      // row_newbcast: a lane of every row of 16
    if constexpr (LPR == 16) return __builtin_amdgcn_mov_dpp(v, kRowLane + SRC, 0xf, 0xf, true);
    else {
        static_assert(LPR == 8, "groups within a row of 16 lanes");
        const int low = __builtin_amdgcn_mov_dpp(v, kRowLane + SRC, 0xf, 0xf, true);
        return __builtin_amdgcn_update_dpp(low, v, kRowLane + 8 + SRC, 0xf, 0xc, false);
    }
}
template <int LPR, int SRC>
__device__ __forceinline__ float from_lane(float v) { return __int_as_float(from_lane<LPR, SRC>(__float_as_int(v))); }

// den[c] as below, from column c of G in registers (zero beyond k, as x is).
template <int LPR>
__device__ __forceinline__ float row_times_column(float x, const float (&g)[LPR])
{
    float d0 = 0.f, d1 = 0.f;
    unrolled<LPR / 2>([&](auto i) {
        d0 += from_lane<LPR, 2 * i>(x) * g[2 * i];
        d1 += from_lane<LPR, 2 * i + 1>(x) * g[2 * i + 1];
    });
    return d0 + d1;
}

// den[c] = sum_d x[d] * G[d][c] for the row whose element c this lane holds.
template <int LPR>
__device__ __forceinline__ float row_times_gram(float x, const float *Gs, int ldg, int k, int c)
{
    float d0 = 0.f, d1 = 0.f;
    const int cc = (c < k) ? c : 0;
    constexpr int U = LPR <= 8 ? 1 : 4;
#pragma unroll U
    for (int d = 0; d + 1 < k; d += 2) {
        d0 += group_bcast<LPR>(x, d) * Gs[d * ldg + cc];
        d1 += group_bcast<LPR>(x, d + 1) * Gs[(d + 1) * ldg + cc];
    }
    if (k & 1) d0 += group_bcast<LPR>(x, k - 1) * Gs[(k - 1) * ldg + cc];
    return d0 + d1;
}

__device__ __forceinline__ void stage_gram(float *Gs, const float *__restrict__ G, int k, int ldg)
{
    for (int e = threadIdx.x; e < k * k; e += blockDim.x) Gs[(e / k) * ldg + (e % k)] = G[e];
    __syncthreads();
}

// ---------------------------------------------------------------------------
// Row-balanced work partition.  The work of row r is taken as its stored
// entries plus kRowCost (the fused update), so the running total
//     key(r) = rowptr[r] + kRowCost * r
// is increasing and part[w] = first r with key(r) >= w * share splits the rows
// into nparts contiguous ranges of (nearly) equal work, one per wavefront.
// Rows longer than kLongRow entries are taken out of the ranges (they would
// stall one wavefront) and handled by a whole workgroup each.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void csr_partition_kernel(const int64_t *__restrict__ rowptr,
                                                            int64_t m, int nparts,
                                                            int64_t *__restrict__ part)
{
    const int w = blockIdx.x * 256 + threadIdx.x;
    if (w > nparts) return;
    const int64_t total = rowptr[m] + kRowCost * m;
    const int64_t share = (total + nparts - 1) / nparts;
    const int64_t target = (int64_t)w * share;
    int64_t lo = 0, hi = m;                 // smallest r in [0, m] with key(r) >= target
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (rowptr[mid] + kRowCost * mid >= target) hi = mid;
        else lo = mid + 1;
    }
    part[w] = (w == nparts) ? m : lo;
}

// list[0 .. *count) = rows with more than kLongRow entries (any order).
// `cap` slots: row pointers that add up to nnz cannot name more such rows than nnz / kLongRow;
// malformed ones can, and what does not fit is dropped (the count keeps running).
__global__ __launch_bounds__(256) void csr_long_rows_kernel(const int64_t *__restrict__ rowptr,
                                                            int64_t m, int32_t *__restrict__ list,
                                                            unsigned *count, unsigned cap)
{
    for (int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x; r < m; r += (int64_t)gridDim.x * 256)
        if (rowptr[r + 1] - rowptr[r] > kLongRow) {
            const unsigned slot = atomicAdd(count, 1u);
            if (slot < cap) list[slot] = (int32_t)r;
        }
}

__global__ void zero_u32_kernel(unsigned *p) { if (threadIdx.x == 0 && blockIdx.x == 0) *p = 0u; }

// The entry a lane holds for its group: its table row (clamped: an index outside the table, from
// malformed input, is pulled to its edge, no stray access) as an offset into the table, and its value;
// past the row's end: row 0 of the table, value 0, which adds nothing.  NARROW: the table has at most 2^30
// floats, and the lane that loads an entry multiplies it by the table's row length once for the whole group.
template <bool NARROW>
__device__ __forceinline__ void load_entry(const int32_t *__restrict__ colidx, const float *__restrict__ vals,
                                           int trows, int ldt, int64_t e, bool ok, int &off, float &val)
{
    off = 0;
    val = 0.f;
    if (ok) {
        const int col = min(max(colidx[e], 0), trows - 1);
        off = NARROW ? col * ldt : col;
        val = vals[e];
    }
}

// acc + the products of the `cnt` entries the group's lanes hold (`any`: the largest cnt of the wave's
// groups), UNR at a time so that several table rows are in flight.
template <int LPR, bool NARROW>
__device__ __forceinline__ float gather_entries(const float *__restrict__ T, int ldt, int cc, int off, float val,
                                                int cnt, float acc)
{
    constexpr int UNR = (LPR < 8) ? LPR : 8;
    if constexpr (by_lane(LPR)) {
        auto some = [&](auto t0) {
            float a[UNR], h[UNR];
            unrolled<UNR>([&](auto u) {
                const int o = from_lane<LPR, t0 + u>(off);
                a[u] = from_lane<LPR, t0 + u>(val);
                if (NARROW) h[u] = *reinterpret_cast<const float *>(reinterpret_cast<const char *>(T) + (unsigned)(o + cc) * 4u);
                else h[u] = T[(int64_t)o * ldt + cc];
            });
#pragma unroll
            for (int u = 0; u < UNR; ++u) acc += a[u] * h[u];
        };
        if (__any(cnt > 0)) some(std::integral_constant<int, 0>{});
        if constexpr (LPR > UNR)
            if (__any(cnt > UNR)) some(std::integral_constant<int, UNR>{});
        return acc;
    }
    for (int t0 = 0; __any(t0 < cnt); t0 += UNR) {
        float a[UNR], h[UNR];
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            const int o = group_bcast<LPR>(off, t0 + u);
            a[u] = group_bcast<LPR>(val, t0 + u);
            if (NARROW) h[u] = *reinterpret_cast<const float *>(reinterpret_cast<const char *>(T) + (unsigned)(o + cc) * 4u);
            else h[u] = T[(int64_t)o * ldt + cc];
        }
#pragma unroll
        for (int u = 0; u < UNR; ++u) acc += a[u] * h[u];
    }
    return acc;
}

// One gather step of a lane group: entries [e, e + LPR) of a row (fewer at its end).
template <int LPR, bool NARROW>
__device__ __forceinline__ float gather_chunk(const int32_t *__restrict__ colidx,
                                              const float *__restrict__ vals,
                                              const float *__restrict__ T, int trows, int ldt, int k, int c,
                                              int64_t e, int64_t e1, float acc)
{
    const int64_t left = e1 - e;
    const int cnt = left < LPR ? (left > 0 ? (int)left : 0) : LPR;
    int off;
    float val;
    load_entry<NARROW>(colidx, vals, trows, ldt, e + c, c < cnt, off, val);
    return gather_entries<LPR, NARROW>(T, ldt, (c < k) ? c : 0, off, val, cnt, acc);
}

// ---------------------------------------------------------------------------
// X[i][:] <- X[i][:] * (sum over the entries (i, j, a) of row i of a T[j][:]) / (X[i][:] G + eps).
// With the CSR of A, T = Ht, G = H H^T, X = W: AHT, WHHT and the W update of
// Algorithm 3 in one kernel (the row of A H^T lives in one register per lane);
// with the column-ordered copy, T = W, G = W^T W, X = Ht: WTA and the H update.
// The first kCsrLongBlocks workgroups take the rows in `list` (more than kLongRow entries), one
// workgroup per row: its lane groups take the row's chunks round robin and their sums are added in
// group order; with none they end at once.  In the others wavefront gw works on rows
// [part[gw], part[gw + 1]):
//   SPLIT = false: 64 / LPR rows at a time, a lane group each, LPR entries of each per step;
//   SPLIT = true:  one row at a time, 64 entries per step dealt to all lane groups, the groups'
//                  sums added by butterfly (see launch_aht_csr for which).
// What bounds it depends on the size.  With a table beyond the caches: the bytes of the gathered rows.
// With small tables: the chain range -> row pointers -> entries -> table rows -> update, a trip to
// L2 or memory each; so G (one entry or a few per thread) and the row of X are requested before
// the entries and waited for after them, and the next step's entries are requested before the
// current ones are gathered.  65536 x 16384, 1.07 million entries, k = 12: 23 and 35 us for the two updates
// with a launch of 4.5 for the long rows each, 21 and 18.6 with the long rows in the same launch, and 16.5 and 14.6
// since from 5 to 16 factors nothing goes through the LDS unit (from_lane; G by columns in registers).  Tried there: half or a quarter
// as many waves with the next rows' pointers and entries on their way (no faster), 16 gathered rows in flight (slower).
// ldx, ldt: row lengths of W and of the table (at least k, see csr_row_length).
// accumulate != 0: no update; the gathered sums are added to W instead (the
// numerator of an update collected over several row batches of the matrix; GH unused).
// accumulate == 2: nothing is written to W (needs dpart; GH unused).
// dpart: dpart[blockIdx.x] = sum over this block's rows of gathered sum x value of W in double
// (the new value in an updating launch, the unchanged one with accumulate == 2), i.e. its
// share of <A H^T, W> for the objective ||A||^2 - 2 <A H^T, W> + <H H^T, W^T W>; lanes by
// butterfly, then the 4 waves in order.
// ---------------------------------------------------------------------------
template <int LPR, bool SPLIT, bool NARROW>
__global__ __launch_bounds__(256, LPR == 64 ? 6 : 8) void aht_csr_kernel(const int64_t *__restrict__ rowptr,
                                                      const int32_t *__restrict__ colidx,
                                                      const float *__restrict__ vals,
                                                      const int64_t *__restrict__ part,
                                                      const int32_t *__restrict__ list,
                                                      const unsigned *__restrict__ count, unsigned list_cap, int k,
                                                      const float *__restrict__ Ht,
                                                      const float *__restrict__ GH, float *W,
                                                      float eps, int accumulate,
                                                      double *__restrict__ dpart, int64_t nnz, int trows,
                                                      int ldx, int ldt)
{
    constexpr int LDG = LPR + 1, RPW = 64 / LPR, NG = 256 / LPR, EPG = (LPR * LPR + 255) / 256;
    constexpr bool REG = by_lane(LPR);      // G: a column of it in each lane's registers, else all of it in LDS
    __shared__ float Gs[REG ? 1 : LPR * LDG];
    __shared__ float part_acc[NG][LPR];
    __shared__ double dsum[4];
    const int lane = threadIdx.x & 63;
    const int c = lane % LPR, cc = (c < k) ? c : 0;
    double dacc = 0.0;
    // G: requested first, put into LDS (one barrier) when the first row's sums are there
    float gq[EPG], gc[REG ? LPR : 1];
    if constexpr (REG) {
#pragma unroll
        for (int d = 0; d < LPR; ++d)
            gc[d] = !accumulate && d < k && c < k ? GH[d * k + c] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < EPG; ++i) gq[i] = !REG && !accumulate && (int)threadIdx.x + 256 * i < k * k ? GH[threadIdx.x + 256 * i] : 0.f;
    bool staged = REG || accumulate != 0;      // uniform over a wave; every wave passes the barrier once
    auto stage = [&]() {
        if (staged) return;
        staged = true;
#pragma unroll
        for (int i = 0; i < EPG; ++i) {
            const int e = threadIdx.x + 256 * i;
            if (e < k * k) Gs[(e / k) * LDG + e % k] = gq[i];
        }
        __syncthreads();
    };
    // the row's update from its sum; `mine`: this lane writes factor c of it
    auto finish = [&](int64_t row, bool valid, bool mine, float w, float acc) {
        mine = mine && valid && c < k;
        if (accumulate == 2) {
            if (mine) dacc += (double)acc * (double)w;
        } else if (accumulate) {
            if (mine) W[row * ldx + c] = w + acc;
        } else {
            stage();
            float den;
            if constexpr (REG) den = row_times_column<LPR>(w, gc) + eps;
            else den = row_times_gram<LPR>(w, Gs, LDG, k, c) + eps;
            if (mine) {
                const float wn = w * acc / den;
                W[row * ldx + c] = wn;
                dacc += (double)acc * (double)wn;
            }
        }
    };
    if (blockIdx.x < kCsrLongBlocks) {
        const unsigned n_long = *count < list_cap ? *count : list_cap;
        const int grp = threadIdx.x / LPR;
        for (unsigned li = blockIdx.x; li < n_long; li += kCsrLongBlocks) {
            const int64_t row = list[li];
            const int64_t e0 = min(max(rowptr[row], (int64_t)0), nnz), e1 = min(max(rowptr[row + 1], (int64_t)0), nnz);
            float acc = 0.f;
            for (int64_t e = e0 + (int64_t)grp * LPR; __any(e < e1); e += (int64_t)NG * LPR)
                acc = gather_chunk<LPR, NARROW>(colidx, vals, Ht, trows, ldt, k, c, e, e1, acc);
            part_acc[grp][threadIdx.x % LPR] = acc;
            __syncthreads();
            float total = 0.f;           // every lane adds up its factor, the first group's lanes write it
            for (int gI = 0; gI < NG; ++gI) total += part_acc[gI][c];
            const float w = (c < k) ? W[row * ldx + c] : 0.f;
            finish(row, true, threadIdx.x < LPR, w, total);
            __syncthreads();
        }
    } else {
        const int gw = __builtin_amdgcn_readfirstlane((blockIdx.x - kCsrLongBlocks) * 4 + (threadIdx.x >> 6));
        const int64_t r_lo = part[gw], r_hi = part[gw + 1];          // same for the whole wavefront
        constexpr int STEP = SPLIT ? 1 : RPW;
        for (int64_t base = r_lo; base < r_hi; base += STEP) {
            const int64_t row = SPLIT ? base : base + lane / LPR;
            bool valid = row < r_hi;
            // row pointers outside [0, nnz] (malformed input) are pulled into the arrays
            int64_t p0, p1;
            float wv;
            if constexpr (REG) {
                // rows past the range read its last one's and drop it: loads without branches (groups of 64 lanes 0.8 % slower so)
                const int64_t at = valid ? row : r_hi - 1;
                p0 = rowptr[at], p1 = rowptr[at + 1];
                wv = W[at * ldx + cc];
            } else {
                p0 = valid ? rowptr[row] : 0, p1 = valid ? rowptr[row + 1] : 0;
                wv = valid && c < k ? W[row * ldx + c] : 0.f;
            }
            int64_t e = min(max(p0, (int64_t)0), nnz), e1 = min(max(p1, (int64_t)0), nnz);
            if (!valid || p1 - p0 > kLongRow) {       // long rows are left to the long-row workgroups
                valid = false;
                e1 = e;
            }
            const float w = (valid && c < k) ? wv : 0.f;
            float acc = 0.f;
            constexpr int CHUNK = SPLIT ? 64 : LPR;      // entries of a row per step
            if (SPLIT) e += lane - c;                    // this group's share of the first step
            int64_t left = e1 - e;
            int off;
            float val;
            load_entry<NARROW>(colidx, vals, trows, ldt, e + c, c < left, off, val);
            while (__any(left > 0)) {
                const int o = off, cnt = left < LPR ? (left > 0 ? (int)left : 0) : LPR;
                const float v = val;
                e += CHUNK;
                left -= CHUNK;
                load_entry<NARROW>(colidx, vals, trows, ldt, e + c, c < left, off, val);
                acc = gather_entries<LPR, NARROW>(Ht, ldt, cc, o, v, cnt, acc);
            }
            if (SPLIT) {
#pragma unroll
                for (int x = LPR; x < 64; x <<= 1) acc += __shfl_xor(acc, x);
            }
            finish(row, valid, !SPLIT || lane < LPR, w, acc);
        }
    }
    if (!(blockIdx.x < kCsrLongBlocks)) stage();      // a wave without rows still owes the others its barrier
    if (dpart) {     // uniform over the grid
        for (int off = 32; off > 0; off >>= 1) dacc += __shfl_xor(dacc, off);
        if (lane == 0) dsum[threadIdx.x >> 6] = dacc;
        __syncthreads();
        if (threadIdx.x == 0) dpart[blockIdx.x] = ((dsum[0] + dsum[1]) + dsum[2]) + dsum[3];
    }
}

// X[i][:] <- X[i][:] * Num[i][:] / (X[i][:] G + eps) for i < rows: the update once its
// numerator has been collected (out-of-memory CSR); lane group per row as above.
template <int LPR>
__global__ __launch_bounds__(256) void row_update_kernel(float *X, const float *__restrict__ Num,
                                                         const float *__restrict__ G, int k,
                                                         int64_t rows, float eps)
{
    constexpr int LDG = 65, RPW = 64 / LPR;
    __shared__ float Gs[64 * LDG];
    stage_gram(Gs, G, k, LDG);
    const int lane = threadIdx.x & 63;
    const int c = lane % LPR;
    const int64_t waves = (int64_t)gridDim.x * 4;
    for (int64_t base = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * RPW; base < rows; base += waves * RPW) {
        const int64_t row = base + lane / LPR;
        const bool valid = row < rows && c < k;
        const float x = valid ? X[row * k + c] : 0.f;
        const float den = row_times_gram<LPR>(x, Gs, LDG, k, c) + eps;
        if (valid) X[row * k + c] = x * Num[row * k + c] / den;
    }
}

// out[i] = in[i] - base: row pointers of a row batch made relative to the batch's first entry.
__global__ __launch_bounds__(256) void rebase_i64_kernel(const int64_t *__restrict__ in, int64_t count,
                                                         int64_t base, int64_t *__restrict__ out)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < count; i += (int64_t)gridDim.x * 256)
        out[i] = in[i] - base;
}

__global__ __launch_bounds__(256) void fill_f32_kernel(float *p, int64_t count, float v)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < count; i += (int64_t)gridDim.x * 256)
        p[i] = v;
}

// ---------------------------------------------------------------------------
// Column-ordered copy of the CSR matrix.
// ---------------------------------------------------------------------------
// payload[e] = (row of entry e) << 32 | bits of vals[e]; a group of 32 lanes per row.
__global__ __launch_bounds__(256) void csc_payload_kernel(const int64_t *__restrict__ rowptr,
                                                          const float *__restrict__ vals, int64_t m,
                                                          int64_t nnz, uint64_t *__restrict__ payload)
{
    const int c = threadIdx.x & 31;
    const int64_t group = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 5;
    const int64_t ngroups = (int64_t)gridDim.x * 8;
    for (int64_t row = group; row < m; row += ngroups) {
        const int64_t e1 = min(max(rowptr[row + 1], (int64_t)0), nnz);
        for (int64_t e = min(max(rowptr[row], (int64_t)0), nnz) + c; e < e1; e += 32)
            payload[e] = ((uint64_t)row << 32) | (uint64_t)__float_as_uint(vals[e]);
    }
}

// After the stable sort by column: sorted_cols[e'] is the column of the e'-th
// entry in column order and sorted_payload[e'] its (row, value).  Writes the CSC
// row indices and values and the column pointers (every column j with
// sorted_cols[e'-1] < j <= sorted_cols[e'] starts at e'; columns after the last
// stored one start at nnz).
// dup_part (optional, one double per block): repeated (row, column) pairs stand for their sum, so
// the squared norm of the matrix is the sum of the squared stored values plus, for every run of
// entries with the same row and column (adjacent here, because the sort is stable and a column's
// entries keep their row-major order), twice the products of its pairs; each entry adds
// 2 x its value x the sum of the run's entries before it.
__global__ __launch_bounds__(256) void csc_finish_kernel(const int32_t *__restrict__ sorted_cols,
                                                         const uint64_t *__restrict__ sorted_payload,
                                                         int64_t n, int64_t nnz,
                                                         int64_t *__restrict__ colptr,
                                                         int32_t *__restrict__ rowidx,
                                                         float *__restrict__ cvals,
                                                         double *__restrict__ dup_part)
{
    double corr = 0.0;
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < nnz; e += (int64_t)gridDim.x * 256) {
        const uint64_t pl = sorted_payload[e];
        rowidx[e] = (int32_t)(pl >> 32);
        cvals[e] = __uint_as_float((unsigned)pl);
        if (dup_part) {
            double before = 0.0;
            for (int64_t p = e - 1; p >= 0 && sorted_cols[p] == sorted_cols[e] && (sorted_payload[p] >> 32) == (pl >> 32); --p)
                before += (double)__uint_as_float((unsigned)sorted_payload[p]);
            corr += 2.0 * (double)__uint_as_float((unsigned)pl) * before;
        }
        // column indices outside [0, n) (malformed input) are pulled to the edge
        const int64_t cur = min(max((int64_t)sorted_cols[e], (int64_t)0), n - 1);
        const int64_t prev = (e > 0) ? min(max((int64_t)sorted_cols[e - 1], (int64_t)0), n - 1) : -1;
        for (int64_t j = prev + 1; j <= cur; ++j) colptr[j] = e;
        if (e == nnz - 1)
            for (int64_t j = cur + 1; j <= n; ++j) colptr[j] = nnz;
    }
    if (dup_part) {     // uniform over the grid; lanes by butterfly, then the 4 waves in order
        __shared__ double wsum[4];
        for (int off = 32; off > 0; off >>= 1) corr += __shfl_xor(corr, off);
        if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = corr;
        __syncthreads();
        if (threadIdx.x == 0) dup_part[blockIdx.x] = ((wsum[0] + wsum[1]) + wsum[2]) + wsum[3];
    }
}

__global__ __launch_bounds__(256) void fill_i64_kernel(int64_t *p, int64_t count, int64_t v)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < count; i += (int64_t)gridDim.x * 256)
        p[i] = v;
}

// dst (rows x ld_dst) = the first `cols` columns of src (rows x ld_src), columns cols .. ld_dst - 1
// of dst set to zero (cols <= ld_dst).  One workgroup per row at a time; a wave instruction moves
// 64 consecutive floats, eight per thread in flight.  No alignment is asked of either side.
__global__ __launch_bounds__(256) void pad_copy_kernel(const float *__restrict__ src, int64_t ld_src,
                                                       float *__restrict__ dst, int64_t ld_dst, int64_t rows,
                                                       int64_t cols)
{
    for (int64_t r = blockIdx.x; r < rows; r += gridDim.x) {
        const float *s = src + r * ld_src;
        float *d = dst + r * ld_dst;
        for (int64_t c0 = threadIdx.x; c0 < ld_dst; c0 += 2048) {
            float v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int64_t c = c0 + 256 * q;
                v[q] = c < cols ? s[c] : 0.f;
            }
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int64_t c = c0 + 256 * q;
                if (c < ld_dst) d[c] = v[q];
            }
        }
    }
}

// out (ldc x ld) = in^T, in is rows x cols (rows ldin apart) with ldc >= cols and ld >= rows: what lies beyond in is set to
// zero.  COPY: copy (rows x ldc) = in with the same zero columns, from the same reading of it.
// Tiles of 64 x 64: whole 256-byte runs on both sides at any alignment, 16 loads in flight per
// thread (20011 x 9998, the first iteration of a run at k = 50 with 32 x 32 tiles, four loads each,
// and a copy of its own: 940 us before the iterations, now 680; tiles in the other order 760).
template <bool COPY>
__global__ __launch_bounds__(256) void transpose_kernel(const float *__restrict__ in, int64_t rows,
                                                        int64_t cols, float *__restrict__ out, int64_t ld,
                                                        float *__restrict__ copy, int64_t ldc, int64_t ldin)
{
    __shared__ float tile[64][65];
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    const int64_t tiles_c = (ldc + 63) / 64, tiles_r = (ld + 63) / 64;
    for (int64_t t = blockIdx.x; t < tiles_c * tiles_r; t += gridDim.x) {
        const int64_t r0 = (t / tiles_c) * 64, c0 = (t % tiles_c) * 64;
        float v[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int64_t r = r0 + ty + 4 * i;
            const bool ok = r < rows && c0 + tx < cols;
            v[i] = in[ok ? r * ldin + c0 + tx : 0];
            v[i] = ok ? v[i] : 0.f;
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int64_t r = r0 + ty + 4 * i;
            tile[ty + 4 * i][tx] = v[i];
            if (COPY && r < rows && c0 + tx < ldc) copy[r * ldc + c0 + tx] = v[i];
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int y = ty + 4 * i;
            if (c0 + y < ldc && r0 + tx < ld) out[(c0 + y) * ld + r0 + tx] = tile[tx][y];
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------

static int lanes_per_row(int k)
{
    int l = 4;
    while (l < k) l <<= 1;
    return l;
}

#define NMFMU_LPR_SWITCH(lpr, CALL)      \
    switch (lpr) {                        \
    case 4: { constexpr int L = 4; CALL; } break;   \
    case 8: { constexpr int L = 8; CALL; } break;   \
    case 16: { constexpr int L = 16; CALL; } break; \
    case 32: { constexpr int L = 32; CALL; } break; \
    default: { constexpr int L = 64; CALL; } break; \
    }

hipError_t launch_csr_partition(const int64_t *rowptr, int64_t m, int nparts, int64_t *part,
                                hipStream_t st)
{
    hipLaunchKernelGGL(csr_partition_kernel, dim3((nparts + 1 + 255) / 256), dim3(256), 0, st, rowptr, m, nparts, part);
    return hipGetLastError();
}

hipError_t launch_csr_long_rows(const int64_t *rowptr, int64_t m, int32_t *list, unsigned *count,
                                unsigned cap, hipStream_t st)
{
    hipLaunchKernelGGL(zero_u32_kernel, dim3(1), dim3(64), 0, st, count);
    int64_t b = (m + 255) / 256;
    if (b > 4096) b = 4096;
    hipLaunchKernelGGL(csr_long_rows_kernel, dim3((unsigned)b), dim3(256), 0, st, rowptr, m, list, count, cap);
    return hipGetLastError();
}

template <int LPR, bool SPLIT>
static void aht_csr_dispatch(bool narrow, hipStream_t st, const int64_t *rowptr, const int32_t *colidx, const float *vals,
                             const int64_t *part, const int32_t *list, const unsigned *count, unsigned cap, int k,
                             const float *Ht, const float *GH, float *W, float eps, int acc, double *dpart, int64_t nnz,
                             int trows, int ldx, int ldt)
{
    const dim3 grid(kCsrLongBlocks + kCsrParts / 4), block(256);
    if (narrow)
        hipLaunchKernelGGL((aht_csr_kernel<LPR, SPLIT, true>), grid, block, 0, st, rowptr, colidx, vals, part, list, count, cap,
                           k, Ht, GH, W, eps, acc, dpart, nnz, trows, ldx, ldt);
    else
        hipLaunchKernelGGL((aht_csr_kernel<LPR, SPLIT, false>), grid, block, 0, st, rowptr, colidx, vals, part, list, count, cap,
                           k, Ht, GH, W, eps, acc, dpart, nnz, trows, ldx, ldt);
}

hipError_t launch_aht_csr(const int64_t *rowptr, const int32_t *colidx, const float *vals,
                          const int64_t *part, const int32_t *long_list, const unsigned *long_count,
                          int k, const float *Ht, const float *GH, float *W, float eps, int64_t nnz, int64_t rows,
                          int64_t trows, hipStream_t st, bool accumulate, double *dpart, bool dry, int ldx, int ldt)
{
    if (ldx == 0) ldx = k;
    if (ldt == 0) ldt = k;
    if (ldx < k || ldt < k) return hipErrorInvalidValue;
    if (trows < 1 || trows > 0x7fffffff || nnz < 0 || rows < 1) return hipErrorInvalidValue;
    if ((dpart && accumulate) || (dry && (!dpart || accumulate))) return hipErrorInvalidValue;
    const int lpr = lanes_per_row(k);
    const int acc = dry ? 2 : (accumulate ? 1 : 0);
    const bool narrow = trows * ldt <= ((int64_t)1 << 30);
    const unsigned cap = (unsigned)(nnz / kLongRow + 1);
    // From 64 entries per row on average a row fills the wave's lanes by itself, and fewer, longer rows
    // than lane groups leave no group idle: 16384 rows of 65 entries at k = 12 took 35 us a row per
    // group, 18.6 a row per wave; 524288 rows of 210 at k = 32, where the gathered bytes decide,
    // 2276 and 2254.  Shorter rows waste lanes at the end of their one step (65536 rows of 16 at k = 12: 21).
    const bool split = lpr < 64 && nnz >= 64 * rows;
    if (split) {
        NMFMU_LPR_SWITCH(lpr, (aht_csr_dispatch<L, (L < 64)>(narrow, st, rowptr, colidx, vals, part, long_list, long_count, cap, k, Ht,
                                                         GH, W, eps, acc, dpart, nnz, (int)trows, ldx, ldt)));
    } else {
        NMFMU_LPR_SWITCH(lpr, (aht_csr_dispatch<L, false>(narrow, st, rowptr, colidx, vals, part, long_list, long_count, cap, k, Ht,
                                                          GH, W, eps, acc, dpart, nnz, (int)trows, ldx, ldt)));
    }
    return hipGetLastError();
}

hipError_t launch_row_update(float *X, const float *Num, const float *G, int k, int64_t rows, float eps,
                             hipStream_t st)
{
    const int lpr = lanes_per_row(k);
    int64_t b = (rows * lpr / 64 + 3) / 4;
    if (b > 8192) b = 8192;
    if (b < 1) b = 1;
    const dim3 grid((unsigned)b), block(256);
    NMFMU_LPR_SWITCH(lpr, hipLaunchKernelGGL((row_update_kernel<L>), grid, block, 0, st, X, Num, G, k, rows, eps));
    return hipGetLastError();
}

hipError_t launch_rebase_i64(const int64_t *in, int64_t count, int64_t base, int64_t *out, hipStream_t st)
{
    int64_t b = (count + 255) / 256;
    if (b > 4096) b = 4096;
    hipLaunchKernelGGL(rebase_i64_kernel, dim3((unsigned)b), dim3(256), 0, st, in, count, base, out);
    return hipGetLastError();
}

hipError_t launch_fill_f32(float *p, int64_t count, float v, hipStream_t st)
{
    int64_t b = (count + 255) / 256;
    if (b > 8192) b = 8192;
    if (b < 1) b = 1;
    hipLaunchKernelGGL(fill_f32_kernel, dim3((unsigned)b), dim3(256), 0, st, p, count, v);
    return hipGetLastError();
}

// dst (rows of ldd) = the first k columns of src (rows of lds); a thread per entry of a few rows at a time.
__global__ __launch_bounds__(256) void restride_kernel(const float *__restrict__ src, int lds, float *__restrict__ dst,
                                                       int ldd, int64_t rows, int k)
{
    const int per = 256 / k, c = threadIdx.x % k, r = threadIdx.x / k;
    if (r >= per) return;
    for (int64_t row = (int64_t)blockIdx.x * per + r; row < rows; row += (int64_t)gridDim.x * per)
        dst[row * ldd + c] = src[row * lds + c];
}

hipError_t launch_restride(const float *src, int lds, float *dst, int ldd, int64_t rows, int k, hipStream_t st)
{
    if (k < 1 || k > 64 || lds < k || ldd < k) return hipErrorInvalidValue;
    int64_t b = (rows + 256 / k - 1) / (256 / k);
    if (b > 16384) b = 16384;
    hipLaunchKernelGGL(restride_kernel, dim3((unsigned)b), dim3(256), 0, st, src, lds, dst, ldd, rows, k);
    return hipGetLastError();
}

hipError_t launch_pad_copy(const float *src, int64_t ld_src, float *dst, int64_t ld_dst, int64_t rows, int64_t cols,
                           hipStream_t st)
{
    if (cols > ld_dst || cols > ld_src) return hipErrorInvalidValue;
    const int64_t b = rows < 8192 ? rows : 8192;
    hipLaunchKernelGGL(pad_copy_kernel, dim3((unsigned)(b < 1 ? 1 : b)), dim3(256), 0, st, src, ld_src, dst, ld_dst, rows, cols);
    return hipGetLastError();
}

hipError_t launch_transpose(const float *in, int64_t rows, int64_t cols, float *out, hipStream_t st, int64_t ld,
                            float *copy, int64_t ldc, int64_t ldin)
{
    if (ldin < cols) ldin = cols;
    if (ld < rows) ld = rows;
    if (ldc < cols) ldc = cols;
    int64_t tiles = ((ld + 63) / 64) * ((ldc + 63) / 64);
    if (tiles > 65536) tiles = 65536;
    if (copy) hipLaunchKernelGGL(transpose_kernel<true>, dim3((unsigned)tiles), dim3(256), 0, st, in, rows, cols, out, ld, copy, ldc, ldin);
    else hipLaunchKernelGGL(transpose_kernel<false>, dim3((unsigned)tiles), dim3(256), 0, st, in, rows, cols, out, ld, copy, ldc, ldin);
    return hipGetLastError();
}

static unsigned blocks_for(int64_t count)
{
    int64_t b = (count + 255) / 256;
    if (b > 65536) b = 65536;
    if (b < 1) b = 1;
    return (unsigned)b;
}

static int bits_for(int64_t n)
{
    int b = 1;
    while (((int64_t)1 << b) < n) ++b;
    return b;
}

size_t csc_sort_temp_bytes(int64_t nnz, int64_t n)
{
    size_t bytes = 0;
    const int32_t *kin = nullptr;
    int32_t *kout = nullptr;
    const uint64_t *vin = nullptr;
    uint64_t *vout = nullptr;
    (void)hipcub::DeviceRadixSort::SortPairs(nullptr, bytes, kin, kout, vin, vout, (int)nnz, 0, bits_for(n));
    return bytes;
}

hipError_t launch_csc_build(const int64_t *rowptr, const int32_t *colidx, const float *vals,
                            int64_t m, int64_t n, int64_t nnz, int32_t *sorted_cols,
                            uint64_t *payload, uint64_t *sorted_payload, void *sort_temp,
                            size_t sort_temp_bytes, int64_t *colptr, int32_t *rowidx, float *cvals,
                            hipStream_t st, double *dup_part)
{
    if (nnz == 0) {
        hipLaunchKernelGGL(fill_i64_kernel, dim3(blocks_for(n + 1)), dim3(256), 0, st, colptr, n + 1, (int64_t)0);
        if (dup_part) hipLaunchKernelGGL(fill_i64_kernel, dim3(1), dim3(256), 0, st, reinterpret_cast<int64_t *>(dup_part), (int64_t)1, (int64_t)0);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(csc_payload_kernel, dim3(blocks_for(m * 32)), dim3(256), 0, st, rowptr, vals, m, nnz, payload);
    hipError_t e = hipcub::DeviceRadixSort::SortPairs(sort_temp, sort_temp_bytes, colidx, sorted_cols,
                                                      (const uint64_t *)payload, sorted_payload,
                                                      (int)nnz, 0, bits_for(n), st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(csc_finish_kernel, dim3(blocks_for(nnz)), dim3(256), 0, st, sorted_cols,
                       sorted_payload, n, nnz, colptr, rowidx, cvals, dup_part);
    return hipGetLastError();
}

int csc_finish_blocks(int64_t nnz) { return (int)blocks_for(nnz); }

}  // namespace nmfmu
