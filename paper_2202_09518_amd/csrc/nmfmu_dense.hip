// Dense kernels of the multiplicative-update iteration for gfx950 (MI355X).
//
// One iteration (paper, Algorithm 3 on a single unit) is
//   WTW = W^T W,  WTA = W^T A,  H <- H * WTA / (WTW H + eps),
//   HHT = H H^T (new H),  AHT = A H^T (new H),  W <- W * AHT / (W HHT + eps),
// and the two products over A are all of its memory traffic.  Here they are
// streaming passes over A on the matrix cores, with everything else folded into
// them or into one small finisher kernel:
//   wta_pass_split_buf_kernel / wta_pass_split64_wide_kernel : W^T A as row-split
//       partials; lanes run along the columns of A, the reduction over rows is the
//       reduction of the matrix instruction
//   factor_update_kernel : sums the partials, updates H (or W^T in the mirrored
//       plan), writes the operand planes and the Gram tiles of the new factor
//   one_pass_kernel, one_pass16_kernel : up to 512 columns, A H^T, the W update and W^T A of the next
//       iteration in one reading of A
//   resident_kernel : up to 16 factors, a whole run in one launch while the compute units hold A
//   aht_rows_kernel : A H^T on the row-major A (coalesced loads turned through
//       LDS) with the W update, the planes and the Gram tiles of the new W fused
//   aht_pass_kernel : the older direct A H^T kernel (lanes down the rows), for
//       shapes the others do not serve (unaligned A, short wide matrices)
//   gram_kernel, gram_sum_kernel, residual_*_kernel, objective_kernel : the small rest.
// For k <= 32 and aligned A (and up to 64 where A is not cut into pairs of halves, see nmfmu_pairs.hip) the products are formed from pieces: fp32 operands cut into
// three bf16 pieces each, exactly, and the six leading of the nine piece products per term
// (the rest is below 2^-22 of the term, of either sign) on v_mfma_f32_32x32x16_bf16 with
// fp32 accumulation (see split3 and cut2 below).  wta_pass_kernel and aht_pass_kernel use
// v_mfma_f32_32x32x2_f32 on the floats themselves.
//
// Lane layout of v_mfma_f32_32x32x2_f32 (64 lanes, D = A_op B_op + C):
//   A_op (32 x 2):  lane l holds A_op[l % 32][l / 32]
//   B_op (2 x 32):  lane l holds B_op[l / 32][l % 32]
//   D    (32 x 32): lane l, register v holds D[(v % 4) + 4 (l / 32) + 8 (v / 4)][l % 32]
#include <atomic>

#include "nmfmu_device.h"

namespace nmfmu {

__device__ __forceinline__ f32x4 mfma_bf16_16(u32x4 a, u32x4 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// Running totals of the piece passes.  The bf16 matrix instruction aligns its 16 products
// and the accumulator on the largest exponent and drops what falls below its adder's
// width without rounding, so an accumulator that has grown over thousands of rows loses
// the low bits of every product it takes in, always downwards: measured on uniform data
// the sum over 2048 rows comes out 1.7e-6 low, over 4096 rows 1.1e-5, while up to 512 rows
// the loss is below 1e-7.  Where A repeats one value down a column, all products of that column
// lose the same bits: 4.0e-7 of the result with 512 rows to an accumulator (32768 x 16384, k = 32),
// 1.8e-7 with 256.  The pass kernels therefore keep a matrix accumulator for at most kFlushSteps
// 16-row steps (the kernels further down for as long, or for 96 rows) and then add it, with
// ordinary rounded fp32 adds, into a total that the wave keeps in its own 16 KiB of LDS (64
// accumulator registers x 64 lanes; no other wave touches it, so no barrier); 16 steps instead of
// 32 cost 0.1 % of an iteration.  Slot of register r of tile q for a lane: the
// lane index is flipped by 8 q so that the epilogue, which walks columns 4 jj + q, reads
// 32 different banks.
constexpr int kFlushSteps = 16;

// Cache policy of the buffer loads that stream A: the non-temporal bit.  Every element of A is
// used once per pass, so its lines are marked for early eviction and leave the L2 and the
// Infinity Cache to the operands that are re-read (the piece planes, the partial results).
// Measured on a bare read of 32768 x 16384 floats in the pass's launch shape: 0.313 ms
// (6.85 TB/s) against 0.345 ms (6.22 TB/s) with the default policy.
constexpr int kStreamLoad = 2;
constexpr int kTotFloats = 64 * 64;
__device__ __forceinline__ int tot_slot(int q, int v, int lane) { return (q * 16 + v) * 64 + (lane ^ (8 * q)); }

__device__ __forceinline__ void tot_clear(float *tot, int lane)
{
#pragma unroll
    for (int r = 0; r < 64; ++r) tot[r * 64 + lane] = 0.f;
}

// tot += acc; acc = 0 (four column tiles of one 32-factor tile)
__device__ __forceinline__ void tot_flush4(float *tot, f32x16 (&acc)[4], int lane)
{
    // a tile at a time: 16 reads in flight, then the adds, then the writes
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float t[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) t[v] = tot[tot_slot(q, v, lane)];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            tot[tot_slot(q, v, lane)] = t[v] + acc[q][v];
            acc[q][v] = 0.f;
        }
    }
}

// Epilogue of the 128-column kernels: the four waves' totals of (factor c, column x of the
// slab), added in wave order.
__device__ __forceinline__ float tot_sum4(const float *tot, int c, int x)
{
    const int q = x & 3, jj = x >> 2, half = (c >> 2) & 1, v = (c & 3) | ((c >> 3) << 2);
    const int idx = tot_slot(q, v, 32 * half + jj);
    float val = tot[idx];
#pragma unroll
    for (int ww = 1; ww < kWtaWaves; ++ww) val += tot[ww * kTotFloats + idx];
    return val;
}

// Four consecutive elements X[row][col .. col+3] of a row-major matrix with
// `ncols` columns; elements outside the matrix (or the whole group, if !ok)
// read as zero.  VEC needs a 16-byte aligned base and ncols % 4 == 0, col % 4 == 0.
template <bool VEC>
__device__ __forceinline__ f32x4 load4(const float *__restrict__ X, int64_t ncols, int64_t row,
                                       int64_t col, bool ok)
{
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (VEC) {
        // Branch free: lanes outside the matrix read element (0, 0) and discard
        // it, so the loads of a stage stay in one basic block and the waits on
        // them can be counted exactly (needed for the software prefetch).
        const bool in = ok && col < ncols;
        const f32x4 t = *reinterpret_cast<const f32x4 *>(X + (in ? row * ncols + col : 0));
        v.x = in ? t.x : 0.f;
        v.y = in ? t.y : 0.f;
        v.z = in ? t.z : 0.f;
        v.w = in ? t.w : 0.f;
    } else {
        if (ok) {
            const float *p = X + row * ncols + col;
            if (col + 0 < ncols) v.x = p[0];
            if (col + 1 < ncols) v.y = p[1];
            if (col + 2 < ncols) v.z = p[2];
            if (col + 3 < ncols) v.w = p[3];
        }
    }
    return v;
}

// ---------------------------------------------------------------------------
// Gram matrices.  MODE 0: G = X^T X, X is rows x k (the factor W), rows ld apart.
//                 MODE 1: G = X X^T, X is k x cols (the factor H).
// blockIdx.y selects one 32 x 32 tile (t1, t2) of G; every block sums a slice
// of the long dimension, writes its partial tile, and the block that arrives
// last adds the partials in block order (deterministic) and stores G.
// ---------------------------------------------------------------------------
template <int MODE, bool VEC>
__global__ __launch_bounds__(512) void gram_kernel(const float *__restrict__ X, int64_t len, int k,
                                                   float *__restrict__ G, float *gpart,
                                                   unsigned *counters, int ld)
{
    constexpr int NW = 8;
    __shared__ float red[NW * 1024];
    __shared__ unsigned ticket_s;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int jj = lane & 31, half = lane >> 5;
    const int kt = (k + 31) >> 5;
    const int t1 = blockIdx.y / kt, t2 = blockIdx.y % kt;
    const int c1 = 32 * t1 + jj, c2 = 32 * t2 + jj;
    const int64_t gw = (int64_t)blockIdx.x * NW + w, tw = (int64_t)gridDim.x * NW;

    // Operands of several steps are fetched before the first multiply so that
    // the loads overlap; all loads are branch free (out-of-range lanes read
    // element 0 and discard it).
    f32x16 acc = {0};
    if (MODE == 0) {
        constexpr int UN = 8;
        const int64_t npairs = (len + 1) >> 1;
        for (int64_t p = gw; p < npairs; p += tw * UN) {
            float a[UN], b[UN];
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const int64_t row = 2 * (p + u * tw) + half;
                const bool in1 = row < len && c1 < k, in2 = row < len && c2 < k;
                const float va = X[in1 ? row * ld + c1 : 0], vb = X[in2 ? row * ld + c2 : 0];
                a[u] = in1 ? va : 0.f;
                b[u] = in2 ? vb : 0.f;
            }
#pragma unroll
            for (int u = 0; u < UN; ++u) acc = mfma32(a[u], b[u], acc);
        }
    } else {
        constexpr int UN = 4;
        const int64_t ngroups = (len + 7) >> 3;
        for (int64_t g = gw; g < ngroups; g += tw * UN) {
            f32x4 a[UN], b[UN];
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const int64_t col = 8 * (g + u * tw) + 4 * half;
                a[u] = load4<VEC>(X, len, c1, col, c1 < k);
                b[u] = load4<VEC>(X, len, c2, col, c2 < k);
            }
#pragma unroll
            for (int u = 0; u < UN; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q) acc = mfma32(a[u][q], b[u][q], acc);
        }
    }

    // Every wave parks its tile, then all threads add the eight copies in wave order.
#pragma unroll
    for (int v = 0; v < 16; ++v) red[w * 1024 + v * 64 + lane] = acc[v];
    __syncthreads();
    const int ntiles = gridDim.y;
    float *mine = gpart + ((int64_t)blockIdx.x * ntiles + blockIdx.y) * 1024;
    for (int e = tid; e < 1024; e += 64 * NW) {
        float t = red[e];
#pragma unroll
        for (int ww = 1; ww < NW; ++ww) t += red[ww * 1024 + e];
        mine[e] = t;
    }
    if (G == nullptr) return;   // the consumer sums the partial tiles itself
    __threadfence();
    __syncthreads();
    if (tid == 0) ticket_s = atomicAdd(&counters[blockIdx.y], 1u);
    __syncthreads();
    if (ticket_s != gridDim.x - 1) return;
    // Last block to arrive: every partial tile is visible after this fence.
    // Loads are issued in groups of eight so that they overlap; the sum runs
    // in block order whatever the arrival order was.
    __threadfence();
    const volatile float *vp = gpart;
    for (int e = tid; e < 1024; e += 64 * NW) {
        float s = 0.f;
        const int64_t stride = (int64_t)ntiles * 1024;
        const int64_t base = (int64_t)blockIdx.y * 1024 + e;
        unsigned b = 0;
        for (; b + 8 <= gridDim.x; b += 8) {
            float t[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) t[u] = vp[base + (b + u) * stride];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += t[u];
        }
        for (; b < gridDim.x; ++b) s += vp[base + b * stride];
        const int v = e >> 6, l = e & 63;
        const int r1 = 32 * t1 + acc_row(v, l >> 5), r2 = 32 * t2 + (l & 31);
        if (r1 < k && r2 < k) G[r1 * k + r2] = s;
    }
    if (tid == 0) counters[blockIdx.y] = 0u;
}

// X^T X of a factor of up to 16 columns (rows ld apart) in one launch: 16 x 16 x 4 instructions, a share (lower triangle)
// per workgroup, the last workgroup to arrive adds the shares up, all its loads in flight together.  Sums of
// more than 16 rows are in double: an entry's error is the same for all rows of the other factor.  A tile set per
// workgroup and a launch for their sum took 4.8 + 3.9 us on 65536 x 12, a chain of trips to memory each.
constexpr int kGram16Blocks = 64;
__global__ __launch_bounds__(512) void gram16_kernel(const float *__restrict__ X, int64_t rows, int k, int ld, float *__restrict__ G,
                                                     float *shares, unsigned *counter)
{
    constexpr int kRsrcFlags = 0x00020000;   // raw buffer, 32-bit data format (gfx9 family)
    constexpr unsigned kOut = 0x7fffffffu;   // an offset outside the extent: reads as zero, stores nothing
    constexpr int kExchange = 16;            // sc1: coherent over the whole device
    constexpr int UN = 16, ROW = 136, GR = 15;     // ROW: floats of a share; GR x ROW / 4 threads add them up
    __shared__ double sums[8 * 256];         // of the waves, then of groups of shares
    __shared__ unsigned ticket;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, l16 = lane & 15, quad = lane >> 4;
    const int64_t per = (rows + gridDim.x - 1) / gridDim.x, r0 = blockIdx.x * per, r1 = r0 + per < rows ? r0 + per : rows;
    double tot[4] = {0.0, 0.0, 0.0, 0.0};
    for (int64_t base = r0 + 4 * w; base < r1; base += 32 * UN) {
        f32x4 acc[4];          // 16 rows each
        float x[UN];
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int64_t row = base + 32 * u + quad;
            const bool in = row < r1 && l16 < k;
            const float v = X[in ? row * ld + l16 : 0];
            x[u] = in ? v : 0.f;
        }
#pragma unroll
        for (int u = 0; u < UN; ++u) acc[u & 3] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[u], x[u], u < 4 ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[u & 3], 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) tot[v] += ((double)acc[0][v] + (double)acc[1][v]) + ((double)acc[2][v] + (double)acc[3][v]);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) sums[w * 256 + l16 * 16 + 4 * quad + v] = tot[v];
    __syncthreads();
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(shares, 0, (int)(gridDim.x * ROW * 4), kRsrcFlags);
    const int er = (tid >> 4) & 15, ec = tid & 15;
    if (tid < 256) {
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < 8; ++i) s += sums[i * 256 + tid];
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint((float)s), rs, er >= ec && er < k ? (unsigned)(blockIdx.x * ROW + er * (er + 1) / 2 + ec) * 4u : kOut, 0, kExchange);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) ticket = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (ticket != gridDim.x - 1) return;
    const int vec = tid % (ROW / 4), g = tid / (ROW / 4);
    if (g < GR) {
        constexpr int M = (kGram16Blocks + GR - 1) / GR;
        u32x4 x[M];
#pragma unroll
        for (int i = 0; i < M; ++i) x[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, (unsigned)((g + GR * i) * ROW + 4 * vec) * 4u, 0, kExchange);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            double s = 0.0;
#pragma unroll
            for (int i = 0; i < M; ++i) s += (double)__uint_as_float(x[i][j]);
            sums[g * ROW + 4 * vec + j] = s;
        }
    }
    __syncthreads();
    if (tid < 256 && er < k && ec < k) {
        const int hi = er > ec ? er : ec, lo = er > ec ? ec : er;
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < GR; ++i) s += sums[i * ROW + hi * (hi + 1) / 2 + lo];
        G[er * k + ec] = (float)s;
    }
    if (tid == 0) *counter = 0u;
}

// ---------------------------------------------------------------------------
// W^T A pass.  Workgroup = 4 waves on one 128-column slab of A and one row
// split; wave w takes row pairs w, w+4, ... of the split.  Per row pair a lane
// loads four consecutive columns (one 16-byte load, 512 contiguous bytes per
// row and wave) and one element of each W row; column tile q of the wave
// therefore holds columns j0 + 4 jj + q.  MFMA roles: A_op = W rows (factor
// index across lanes), B_op = A elements (column across lanes), reduction
// over the two rows.  The waves are summed through LDS in wave order and the
// slab is written (or added) to the split's partial result.
// Registers are capped (OCC waves per SIMD) so that several workgroups share a
// compute unit: one group's reduction epilogue then hides behind the others'
// streaming, and enough loads are in flight to cover the HBM latency.
// ---------------------------------------------------------------------------
template <int KT, int U, int OCC, bool VEC>
__global__ __launch_bounds__(64 * kWtaWaves, OCC) void wta_pass_kernel(const float *__restrict__ A,
                                                       const float *__restrict__ W,
                                                       float *__restrict__ ppart, int64_t rows,
                                                       int64_t n, int k, int64_t rps,
                                                       int accumulate,
                                                       const float *__restrict__ gtiles, int nsets,
                                                       float *__restrict__ gsum)
{
    constexpr int NW = kWtaWaves;
    constexpr int LD = 132;
    __shared__ float red[KT * 32 * LD];
    if (gtiles) sum_tile_sets(gtiles, nsets, k, gsum, blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int jj = lane & 31, half = lane >> 5;
    const int64_t j0 = (int64_t)blockIdx.x * kWtaCols;
    const int64_t col = j0 + 4 * jj;
    const int64_t r0 = (int64_t)blockIdx.y * rps;
    const int64_t r1 = (r0 + rps < rows) ? r0 + rps : rows;

    f32x16 acc[KT][4];
#pragma unroll
    for (int t = 0; t < KT; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[t][q] = f32x16{0};

    struct Stage {
        f32x4 a[U];
        float wv[U][KT];
    };
    auto load_stage = [&](Stage &s, int64_t ibase) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t row = ibase + 2 * NW * u + half;
            const bool ok = row < r1;
            s.a[u] = load4<VEC>(A, n, row, col, ok);
#pragma unroll
            for (int t = 0; t < KT; ++t) {
                const int c = 32 * t + jj;
                const bool in = ok && c < k;
                const float wv = W[in ? row * k + c : 0];
                s.wv[u][t] = in ? wv : 0.f;
            }
        }
    };
    const int64_t step = 2 * NW * U;
    Stage cur, nxt;
    int64_t i = r0 + 2 * w;
    load_stage(cur, i);
    for (; i < r1; i += step) {
        load_stage(nxt, i + step);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int t = 0; t < KT; ++t)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    acc[t][q] = mfma32(cur.wv[u][t], cur.a[u][q], acc[t][q]);
        cur = nxt;
    }

    for (int ww = 0; ww < NW; ++ww) {
        if (w == ww) {
#pragma unroll
            for (int t = 0; t < KT; ++t)
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int idx = (32 * t + acc_row(v, half)) * LD + q * 32 + jj;
                        if (ww == 0) red[idx] = acc[t][q][v];
                        else red[idx] += acc[t][q][v];
                    }
        }
        __syncthreads();
    }
    float *dst = ppart + (int64_t)blockIdx.y * k * n;
    for (int e = tid; e < k * kWtaCols; e += 64 * NW) {
        const int c = e >> 7, x = e & 127;
        const int64_t cj = j0 + x;
        if (cj < n) {
            float val = red[c * LD + (x & 3) * 32 + (x >> 2)];
            float *p = dst + (int64_t)c * n + cj;
            if (accumulate) val += *p;
            *p = val;
        }
    }
}

// ---------------------------------------------------------------------------
// Piece planes of kc <= kp columns c0 .. c0 + kc - 1 of a factor X (rows x ld,
// row-major), the A_op of the passes below; kp = 32 or 64 factor slots per row group:
// planes[(g * 3 + p) * kp + c] = the eight bf16 p-th pieces (p = 0: h, 1: m, 2: l)
// of X[8 g .. 8 g + 7][c0 + c], c < kp; rows beyond `rows` and columns beyond kc are zero.
// ---------------------------------------------------------------------------
// blockIdx.y = slice: columns c0 + kp * slice onwards (at most kp of the k left), planes + slice * slice_planes.
__global__ __launch_bounds__(256) void split_planes_kernel(const float *__restrict__ X, int64_t rows,
                                                           int64_t ld, int64_t c0, int k, int kp,
                                                           u32x4 *__restrict__ planes, int64_t slice_planes)
{
    c0 += (int64_t)kp * blockIdx.y;
    k -= kp * (int)blockIdx.y;
    if (k > kp) k = kp;
    planes += (int64_t)blockIdx.y * slice_planes;
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t g = t / kp;
    const int c = (int)(t % kp);
    if (g * 8 >= rows) return;
    u32x4 o[3];
#pragma unroll
    for (int pr = 0; pr < 4; ++pr) {
        unsigned h[2], m[2], l[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int64_t row = g * 8 + 2 * pr + e;
            const float x = (row < rows && c < k) ? X[row * ld + c0 + c] : 0.f;
            split3(x, h[e], m[e], l[e]);
        }
        o[0][pr] = pack2(h[0], h[1]);
        o[1][pr] = pack2(m[0], m[1]);
        o[2][pr] = pack2(l[0], l[1]);
    }
#pragma unroll
    for (int pl = 0; pl < 3; ++pl) planes[(g * 3 + pl) * kp + c] = o[pl];
}

// ---------------------------------------------------------------------------
// W^T A pass for k <= 32 on pieces, on the bf16 matrix cores (see
// split3 and cut2 above).  Geometry as wta_pass_kernel: 4 waves on a 128-column slab and
// one row split, lane = 4 consecutive columns; but a wave takes 16 rows per step
// (half-wave = 8 consecutive rows, the reduction depth of one instruction), loads
// them with eight 16-byte loads per lane, cuts each element into its pieces in
// registers and reads the pieces of W ready-made (planes, 3 x 16 bytes per lane
// and step).  Per column tile the six piece products are accumulated smallest
// first.  r0 of every split is a multiple of 16 (rps is), so a half-wave's rows
// are one 8-row group of the planes.  Two waves per SIMD (256 registers each).
// ---------------------------------------------------------------------------
template <bool VEC>
__global__ __launch_bounds__(64 * kWtaWaves, 2) void wta_pass_split_kernel(
    const float *__restrict__ A, const u32x4 *__restrict__ planes, float *__restrict__ ppart,
    int64_t rows, int64_t n, int k, int64_t rps, int accumulate,
    const float *__restrict__ gtiles, int nsets, float *__restrict__ gsum)
{
    constexpr int NW = kWtaWaves;
    __shared__ float tot[NW * kTotFloats];
    if (gtiles) sum_tile_sets(gtiles, nsets, k, gsum, blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    float *mytot = tot + w * kTotFloats;
    tot_clear(mytot, lane);
    const int jj = lane & 31, half = lane >> 5;
    const int64_t j0 = (int64_t)blockIdx.x * kWtaCols;
    const int64_t col = j0 + 4 * jj;
    const int64_t r0 = (int64_t)blockIdx.y * rps;
    const int64_t r1 = (r0 + rps < rows) ? r0 + rps : rows;

    f32x16 acc[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[q] = f32x16{0};

    struct Stage {
        f32x4 a[8];
        u32x4 wt[3];
    };
    auto load_stage = [&](Stage &s, int64_t ibase) {
        const int64_t rb = ibase + 8 * half;
#pragma unroll
        for (int r = 0; r < 8; ++r) s.a[r] = load4<VEC>(A, n, rb + r, col, rb + r < r1);
        // rows at or beyond r1 contribute nothing because their A elements read as zero
        const int64_t g = rb >> 3;
        const bool okg = rb < r1;
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) s.wt[pl] = planes[okg ? (g * 3 + pl) * 32 + jj : 0];
    };
    const int64_t step = 16 * NW;
    Stage cur, nxt;
    int64_t i = r0 + 16 * w;
    int steps = 0;
    load_stage(cur, i);
    for (; i < r1; i += step) {
        if (++steps > kFlushSteps) {
            tot_flush4(mytot, acc, lane);
            steps = 1;
        }
        load_stage(nxt, i + step);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            u32x4 at[3];
#pragma unroll
            for (int pr = 0; pr < 4; ++pr) {
                cut2(cur.a[2 * pr][q], cur.a[2 * pr + 1][q], at, pr);
            }
            acc[q] = mfma_bf16(cur.wt[2], at[0], acc[q]);      // six products, smallest first
            acc[q] = mfma_bf16(cur.wt[1], at[1], acc[q]);
            acc[q] = mfma_bf16(cur.wt[0], at[2], acc[q]);
            acc[q] = mfma_bf16(cur.wt[1], at[0], acc[q]);
            acc[q] = mfma_bf16(cur.wt[0], at[1], acc[q]);
            acc[q] = mfma_bf16(cur.wt[0], at[0], acc[q]);
        }
        cur = nxt;
    }

    tot_flush4(mytot, acc, lane);
    __syncthreads();
    float *dst = ppart + (int64_t)blockIdx.y * k * n;
    for (int e = tid; e < k * kWtaCols; e += 64 * NW) {
        const int c = e >> 7, x = e & 127;
        const int64_t cj = j0 + x;
        if (cj < n) {
            float val = tot_sum4(tot, c, x);
            float *p = dst + (int64_t)c * n + cj;
            if (accumulate) val += *p;
            *p = val;
        }
    }
}

// ---------------------------------------------------------------------------
// The same pass for 16-byte aligned A with n % 4 == 0 and 64 n < 2^31, on buffer
// loads: per 16-row step a wave builds one descriptor over those rows (base
// A + first row, extent = the rows that exist in this split) and every lane
// loads row r at byte offset (8 half + r) * 4 n + 4 col from it.  Rows past the
// end of the split are outside the extent and read as zero, without a compare
// or select per load, and the addresses cost one VALU add per load.  The planes
// are read the same way (extent = the 8-row groups that exist).  Two steps are
// written out so that the staging registers alternate without copies.
// ---------------------------------------------------------------------------
template <int POLICY>
__global__ __launch_bounds__(64 * kWtaWaves, 2) void wta_pass_split_buf_kernel(
    const float *__restrict__ A, const u32x4 *__restrict__ planes, float *__restrict__ ppart,
    int64_t rows, int64_t n, int k, int64_t rps, int accumulate,
    const float *__restrict__ gtiles, int nsets, float *__restrict__ gsum)
{
    constexpr int NW = kWtaWaves;
    constexpr int kRsrcFlags = 0x00020000;   // raw buffer, 32-bit data format (gfx9 family)
    __shared__ float tot[NW * kTotFloats];
    if (gtiles) sum_tile_sets(gtiles, nsets, k, gsum, blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    float *mytot = tot + w * kTotFloats;
    tot_clear(mytot, lane);
    const int jj = lane & 31, half = lane >> 5;
    const int64_t j0 = (int64_t)blockIdx.x * kWtaCols;
    int64_t col = j0 + 4 * jj;
    if (col >= n) col = 0;   // lanes past the edge read valid data that is never stored
    const int64_t r0 = (int64_t)blockIdx.y * rps;
    const int64_t r1 = (r0 + rps < rows) ? r0 + rps : rows;
    const unsigned rowb = (unsigned)(n * 4);
    const unsigned loff = (unsigned)(half * 8) * rowb + (unsigned)col * 4;
    const unsigned poff = (unsigned)(half * 3 * 32 + jj) * 16;
    const int64_t ngroups = (rows + 7) >> 3;

    f32x16 acc[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[q] = f32x16{0};

    struct Stage {
        u32x4 a[8];
        u32x4 wt[3];
    };
    auto load_stage = [&](Stage &s, int64_t ib) {
        int64_t av = r1 - ib;                       // rows of this step inside the split
        av = av < 0 ? 0 : (av > 16 ? 16 : av);
        const int64_t g = ib >> 3;
        int64_t ng = av ? ngroups - g : 0;          // 8-row groups of planes that exist
        ng = ng < 0 ? 0 : (ng > 2 ? 2 : ng);
        const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float *>(A + (av ? ib : 0) * n), 0, (int)(av * rowb), kRsrcFlags);
        const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<u32x4 *>(planes + (ng ? g : 0) * 3 * 32), 0, (int)(ng * 3 * 32 * 16), kRsrcFlags);
#pragma unroll
        for (int r = 0; r < 8; ++r) s.a[r] = __builtin_amdgcn_raw_buffer_load_b128(ra, loff + r * rowb, 0, POLICY);
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) s.wt[pl] = __builtin_amdgcn_raw_buffer_load_b128(rp, poff + pl * 32 * 16, 0, 0);
    };
    auto compute = [&](const Stage &c) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            u32x4 at[3];
#pragma unroll
            for (int pr = 0; pr < 4; ++pr) {
                cut2(__uint_as_float(c.a[2 * pr][q]), __uint_as_float(c.a[2 * pr + 1][q]), at, pr);
            }
            acc[q] = mfma_bf16(c.wt[2], at[0], acc[q]);      // six products, smallest first
            acc[q] = mfma_bf16(c.wt[1], at[1], acc[q]);
            acc[q] = mfma_bf16(c.wt[0], at[2], acc[q]);
            acc[q] = mfma_bf16(c.wt[1], at[0], acc[q]);
            acc[q] = mfma_bf16(c.wt[0], at[1], acc[q]);
            acc[q] = mfma_bf16(c.wt[0], at[0], acc[q]);
        }
    };
    const int64_t step = 16 * NW;
    Stage s0, s1;
    int64_t i = r0 + 16 * w;
    int pairs = 2 * w;   // the waves of a workgroup flush at different times
    load_stage(s0, i);
    while (i < r1) {
        load_stage(s1, i + step);
        compute(s0);
        i += step;
        if (i >= r1) break;
        load_stage(s0, i + step);
        compute(s1);
        i += step;
        if (++pairs == kFlushSteps / 2) {
            tot_flush4(mytot, acc, lane);
            pairs = 0;
        }
    }

    tot_flush4(mytot, acc, lane);
    __syncthreads();
    float *dst = ppart + (int64_t)blockIdx.y * k * n;
    for (int e = tid; e < k * kWtaCols; e += 64 * NW) {
        const int c = e >> 7, x = e & 127;
        const int64_t cj = j0 + x;
        if (cj < n) {
            float val = tot_sum4(tot, c, x);
            float *p = dst + (int64_t)c * n + cj;
            if (accumulate) val += *p;
            *p = val;
        }
    }
}

// ---------------------------------------------------------------------------
// The pass for 32 < k <= 64 on pieces (aligned A, n % 4 == 0, 64 n < 2^31; planes with
// 64 factor slots per row group).  The arithmetic of wta_pass_split_buf_kernel with two
// 32-factor accumulator tiles per column tile, and another geometry: workgroup = 256
// columns, wave w = columns 64 w .. 64 w + 63 of them (lane = 2 consecutive columns, 8-byte
// loads), and all four waves walk the same 16-row steps of the split.  The piece planes of a
// step are 1.5 times the bytes of a wave's share of A, and read by every wave through the
// vector cache they were the kernel's largest cost (32768 x 16384, k = 64: 474 us, 370 without
// them, 445 without cutting A, 383 with two products instead of six).  So the workgroup stages
// them in LDS once for its four waves: six steps (36 KiB) at a time, double buffered, three
// 16-byte units per thread requested every second step and written two steps later, one
// barrier per six steps; 72 KiB per workgroup, two workgroups per compute unit.  The running
// totals live in registers (the planes of the next steps no longer do) and take the
// accumulators in after every group, 96 terms: by then a sum of terms of one sign or of equal
// ones has lost little (a column of one value, 20011 rows at k = 50: 6.9e-8 of the float64
// result, 3.7e-7 with 480 terms; misaligned A, which ran on the fp32 instruction before, is
// as close as there), for 1 % of the time.  No sum across waves is needed, and each wave stores its own 64 x 64 result: register v of tile (t, q) is factor
// 32 t + row(v), column 2 jj + q, so (q = 0, q = 1) pair up to 8-byte stores, 256
// contiguous bytes per row.  Loads of A run two steps ahead of the arithmetic (three register
// stages), held there by scheduling barriers.  Measured in the iteration on 32768 x 16384:
// 480 -> 400 us (5.4 TB/s; its bare 8-byte loads take 338), on 16384 x 8192 131 -> 110 us.
// ---------------------------------------------------------------------------
template <int POLICY>
__global__ __launch_bounds__(64 * kWtaWaves, 2) void wta_pass_split64_wide_kernel(
    const float *__restrict__ A, const u32x4 *__restrict__ planes, float *__restrict__ ppart,
    int64_t rows, int64_t n, int k, int64_t rps, int accumulate,
    const float *__restrict__ gtiles, int nsets, float *__restrict__ gsum)
{
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    constexpr int KP = 64;
    constexpr int kRsrcFlags = 0x00020000;   // raw buffer, 32-bit data format (gfx9 family)
    constexpr int kSteps = 6;                          // 16-row steps per group of staged planes
    constexpr int kUnits = kSteps * 2 * 3 * KP;        // 16-byte units of planes in a group
    __shared__ u32x4 pst[2][kUnits];
    const int bx = blockIdx.x, by = blockIdx.y;
    if (gtiles) sum_tile_sets(gtiles, nsets, k, gsum, blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
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

    f32x16 acc[2][2], tot[2][2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int q = 0; q < 2; ++q) acc[t][q] = f32x16{0}, tot[t][q] = f32x16{0};

    struct Stage { u32x2 a[8]; };
    auto load_stage = [&](Stage &s, int64_t ib) {
        int64_t av = live ? r1 - ib : 0;            // rows of this step inside the split
        av = av < 0 ? 0 : (av > 16 ? 16 : av);
        const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float *>(A + (av ? ib : 0) * n), 0, (int)(av * rowb), kRsrcFlags);
#pragma unroll
        for (int r = 0; r < 8; ++r) s.a[r] = __builtin_amdgcn_raw_buffer_load_b64(ra, loff + r * rowb, 0, POLICY);
    };
    // a third of the planes of the group of rows from ib on: 3 units per thread
    struct Third { u32x4 u[3]; };
    auto load_third = [&](Third &p, int64_t ib, int part) {
        const int64_t g = ib >> 3;
        int64_t ng = ib < r1 ? ngroups - g : 0;     // 8-row groups of planes that exist
        ng = ng < 0 ? 0 : (ng > 2 * kSteps ? 2 * kSteps : ng);
        const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<u32x4 *>(planes + (ng ? g : 0) * 3 * KP), 0, (int)(ng * 3 * KP * 16), kRsrcFlags);
#pragma unroll
        for (int e = 0; e < 3; ++e)
            p.u[e] = __builtin_amdgcn_raw_buffer_load_b128(rp, (unsigned)((3 * part + e) * 256 + tid) * 16, 0, 0);
    };
    auto store_third = [&](const Third &p, int buf, int part) {
#pragma unroll
        for (int e = 0; e < 3; ++e) pst[buf][(3 * part + e) * 256 + tid] = p.u[e];
    };
    auto compute = [&](const Stage &c, int buf, int st) {     // step 0 of a group starts the accumulators
        u32x4 wt[2][3];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int pl = 0; pl < 3; ++pl) wt[t][pl] = pst[buf][((2 * st + half) * 3 + pl) * KP + 32 * t + jj];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            u32x4 at[3];
#pragma unroll
            for (int pr = 0; pr < 4; ++pr)
                cut2(__uint_as_float(c.a[2 * pr][q]), __uint_as_float(c.a[2 * pr + 1][q]), at, pr);
            constexpr int PW[6] = {2, 1, 0, 1, 0, 0}, PA[6] = {0, 1, 2, 0, 1, 0};   // smallest first
#pragma unroll
            for (int e = 0; e < 6; ++e)
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    acc[t][q] = mfma_bf16(wt[t][PW[e]], at[PA[e]], st == 0 && e == 0 ? f32x16{0} : acc[t][q]);
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
            Stage &z = part == 0 ? s2 : (part == 1 ? s1 : s0);
            load_third(th, i + 16 * kSteps, part);
            load_stage(z, ib + 32);
            __builtin_amdgcn_sched_barrier(0);
            if (live && ib < r1) compute(x, buf, 2 * part);
            __builtin_amdgcn_sched_barrier(0);
            load_stage(x, ib + 48);
            __builtin_amdgcn_sched_barrier(0);
            if (live && ib + 16 < r1) compute(y, buf, 2 * part + 1);
            __builtin_amdgcn_sched_barrier(0);
            store_third(th, buf ^ 1, part);
        }
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int q = 0; q < 2; ++q) tot[t][q] += acc[t][q];
        __syncthreads();    // the next group's planes are written, this group's are read
        buf ^= 1;
    }

    if (colr < n) {
        float *dst = ppart + (int64_t)by * k * n + colr;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int c = 32 * t + acc_row(v, half);
                if (c < k) {
                    f32x2 *p = reinterpret_cast<f32x2 *>(dst + (int64_t)c * n);
                    f32x2 val = {tot[t][0][v], tot[t][1][v]};
                    if (accumulate) {
                        const f32x2 old = *p;
                        val.x += old.x;
                        val.y += old.y;
                    }
                    *p = val;
                }
            }
    }
}

// ---------------------------------------------------------------------------
// Factor update ("finisher").  For X (k x len), partials of its numerator and
// the Gram matrix G of the other factor:
//     X[c][j] <- X[c][j] * (sum_s part[s][c][j]) / (sum_d G[c][d] X[d][j] + eps).
// With X = H, part = W^T A, G = W^T W this is the H-update line of Algorithm 3;
// with X = W^T, part = (A H^T)^T, G = H H^T it is the W-update line.
// A block covers CW columns at a time; thread (column j, group g of 512 / CW) holds the
// old column in registers and produces factor indices c = g, g + FG, ...; groups beyond the
// KP factors take a share of the row splits each, added up through LDS in order.
// Every element is written by the thread that computed it, after a block
// barrier that follows all reads of the old column.
// G comes either complete (Gfull, ld k) or as `nbin` partial 32 x 32 tiles in
// accumulator layout (gin), which every block sums in block order while
// staging G into LDS.  Optional outputs: Xt (len x k), staged through LDS so a
// block stores one contiguous run of CW k floats, and gout: this block's
// partial Gram tiles of the NEW X (X X^T), computed from the LDS copy (one tile: the
// same register as both MFMA operands; four tiles at 33 to 64 factors: each wave one
// tile over half of a chunk's columns); the next finisher consumes them, so no
// separate Gram kernel and no cross-block reduction are needed.  With
// part == nullptr (and splits == 0) nothing is updated and only gout is produced.
//
// The kernel is a chain of trips to L2 (G, the old column, the splits in batches) with little to
// compute, so what counts is how many trips are in flight: the first chunk's old values and first
// batch of splits are requested together with G, a batch holds up to 32 loads per thread, a
// thread loads only its own factors' old values (the column meets in LDS), and short factors are
// cut into narrower chunks so that more workgroups share the splits (see factor_update_width).
// With every thread loading the whole column, batches of 2 to 4 splits and G as 16 partial sums:
// 25 us at k = 50 on 9998 columns and 12 splits, now 19; 10.5 at k = 20 on 4096, now 6.7; 27 at
// k = 16 on 512 columns and 128 splits, now 10; 13 at k = 32 on 16384, now 9.6.
// ---------------------------------------------------------------------------
template <int KP, int CW, bool BIG, int PAIRS>
__global__ __launch_bounds__(512) void factor_update_kernel(float *X, float *Xt,
                                                            const float *__restrict__ part,
                                                            int splits,
                                                            const float *__restrict__ Gfull,
                                                            const float *__restrict__ gin, int nbin,
                                                            float *__restrict__ gout,
                                                            u32x4 *__restrict__ planes,
                                                            double *__restrict__ dpart, int k,
                                                            int64_t len, float eps, BlockMap bm_, FinisherSlices sl)
{
    // PAIRS: 1 one factor, 2 blockIdx.y = slice
    const int z = PAIRS == 2 ? blockIdx.y : 0;
    PairFactor pf{};
    if (PAIRS) {
        X = sl.X[z];
        Xt = sl.Xt[z];
        k = sl.k[z];
        if (part) part += z * sl.part;
        if (gin) gin += z * sl.gin;
        gout += z * sl.gout;
        pf.units = static_cast<u32x4 *>(sl.pairs.units) + z * sl.units;
        pf.exps = sl.pairs.exps + z * sl.exps;
        pf.most = sl.pairs.most + (z * kPairCopies + blockIdx.x % kPairCopies) * 64;
    }
    const BlockMap &bm = PAIRS ? sl.bm[z] : bm_;
    constexpr int NW = 8, KT = KP / 32 > 0 ? KP / 32 : 1, LD = KP + 4;
    constexpr int NG = 512 / CW, FG = NG < KP ? NG : KP, SPL = NG / FG, NC = KP / FG;
    constexpr int SB = 32 / NC < 16 ? 32 / NC : 16;   // splits per batch
    constexpr int LDT = 32 * KT + 1;   // the Gram tiles read 32 factor indices per tile
    // one LDS array: G and the chunk's new values during the updates, then (after a barrier)
    // the eight waves' copies of a Gram tile for the sum over waves
    constexpr int GS = KP * LD, XS = KP * CW, TS = CW * LDT, PS = (SPL - 1) * KP * CW;
    constexpr int SM = (GS + XS + TS + PS > NW * 1024) ? GS + XS + TS + PS : NW * 1024;
    __shared__ __align__(16) float Sm[SM];
    float *Gs = Sm, *Xs = Sm + GS, *Ts = Xs + XS, *Ps = Ts + TS;   // Xs: the chunk's old values [KP][CW]
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int kt = (k + 31) >> 5;
    const int jl = tid % CW, grp = tid / CW, fc = grp % FG;
    const int sp = __builtin_amdgcn_readfirstlane(grp / FG);   // CW x FG threads share it: whole waves
    const int64_t nchunks = (len + CW - 1) / CW;
    const int s_lo = SPL > 1 ? (int)((int64_t)splits * sp / SPL) : 0;
    const int s_hi = SPL > 1 ? (int)((int64_t)splits * (sp + 1) / SPL) : splits;

    // The loads below are buffer loads with 32-bit lane offsets, so that the many in flight hold no
    // addresses.  A descriptor covers the array from the chunk's first column on: what lies past its
    // end (a factor or a set that does not exist) reads as zero, and lanes past the last column or
    // factor read a neighbour's value that is never used.  BIG: k x len floats exceed 2^31 bytes, so
    // every row (one per wave at CW = 64) gets a descriptor of its own.
    static_assert(!BIG || CW == 64, "long factors have 64-column chunks");
    constexpr int kRsrcFlags = 0x00020000;   // raw buffer, 32-bit data format (gfx9 family)
    auto rsrc = [](const float *base, int64_t floats) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(base), 0, (int)(floats * 4), kRsrcFlags);
    };
    auto ld = [](__amdgpu_buffer_rsrc_t r, unsigned off) {
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
    };
    const int fu = BIG ? __builtin_amdgcn_readfirstlane(fc) : 0;
    const unsigned rowb = BIG ? 0u : (unsigned)len * 4u;
    float pb[SB][NC], xo[NC];
    // splits s .. s + SB - 1 of chunk ch
    auto request_splits = [&](int64_t ch, int s) {
        const int64_t left = len - ch * CW;
#pragma unroll
        for (int u = 0; u < SB; ++u) {
            const bool ok = s + u < s_hi;
            const float *base = part + (ok ? (int64_t)(s + u) * k * len + ch * CW : 0);
            if (BIG) {
#pragma unroll
                for (int ci = 0; ci < NC; ++ci) {
                    const int c = fu + FG * ci;
                    pb[u][ci] = ld(rsrc(base + (c < k ? c * len : 0), ok && c < k ? (left < CW ? left : CW) : 0), jl * 4u);
                }
            } else {
                const __amdgpu_buffer_rsrc_t r = rsrc(base, ok ? k * len - ch * CW : 0);
#pragma unroll
                for (int ci = 0; ci < NC; ++ci) pb[u][ci] = ld(r, (unsigned)(fc + FG * ci) * rowb + jl * 4u);
            }
        }
    };
    // the old column and the first batch of splits of chunk ch: requested, not waited for
    auto request = [&](int64_t ch) {
        const int64_t left = len - ch * CW;
        const __amdgpu_buffer_rsrc_t r = rsrc(X + ch * CW, BIG ? 0 : k * len - ch * CW);
#pragma unroll
        for (int ci = 0; ci < NC; ++ci) {
            const int c = (BIG ? fu : fc) + FG * ci;
            xo[ci] = BIG ? ld(rsrc(X + (c < k ? c * len + ch * CW : 0), c < k ? (left < CW ? left : CW) : 0), jl * 4u)
                         : ld(r, c * rowb + jl * 4u);
        }
        if (part) request_splits(ch, s_lo);
    };
    request(blockIdx.x);

    // A thread's entries of G (8 at KP = 64) are independent: the loads of up to four entries are
    // requested together, kGramBatch sets per entry at a time (each trip to L2 costs a microsecond
    // here), and each batch is added in a tree.
    constexpr int kGramBatch = 16;
    constexpr int EPT = (KP * KP + 64 * NW - 1) / (64 * NW), EG = EPT < 4 ? EPT : 4;
    for (int i0 = 0; i0 < EPT; i0 += EG) {
        float gv[EG];
        unsigned off[EG];
        const int64_t stride = (int64_t)kt * kt * 1024;
#pragma unroll
        for (int i = 0; i < EG; ++i) {
            const int e = tid + 64 * NW * (i0 + i);
            const int c = e / KP, d = e % KP;
            // Stacked independent runs: factor indices of different runs do not interact.
            const bool use = e < KP * KP && c < k && d < k && (!bm.on || bm.id[c] == bm.id[d]);
            const int r1 = c & 31, r2 = d & 31;
            const int pos = ((r1 & 3) + 4 * (r1 >> 3)) * 64 + r2 + 32 * ((r1 >> 2) & 1);
            off[i] = !use ? 0x7fffffffu : 4u * (unsigned)(Gfull ? c * k + d : ((c >> 5) * kt + (d >> 5)) * 1024 + pos);
            gv[i] = 0.f;
        }
        if (Gfull || nbin == 1) {
            const __amdgpu_buffer_rsrc_t r = rsrc(Gfull ? Gfull : gin, Gfull ? k * k : stride);
#pragma unroll
            for (int i = 0; i < EG; ++i) gv[i] = ld(r, off[i]);
        } else {
            const __amdgpu_buffer_rsrc_t r = rsrc(gin, nbin * stride);
            for (int b = 0; b < nbin; b += kGramBatch) {
                float t[EG][kGramBatch];
#pragma unroll
                for (int i = 0; i < EG; ++i)
#pragma unroll
                    for (int u = 0; u < kGramBatch; ++u) t[i][u] = ld(r, off[i] + (unsigned)(b + u) * (unsigned)stride * 4u);
#pragma unroll
                for (int i = 0; i < EG; ++i) gv[i] += tree_sum(t[i]);
            }
        }
#pragma unroll
        for (int i = 0; i < EG; ++i) {
            const int e = tid + 64 * NW * (i0 + i);
            if (e < KP * KP) Gs[(e / KP) * LD + e % KP] = gv[i];
        }
    }

    // Gram tiles of the new X.  One tile (KT = 1): every wave adds up its share of the columns.
    // Four tiles (KT = 2): wave w adds up tile w % 4 over half w / 4 of a chunk's columns, which
    // leaves one accumulator per wave and one round through LDS at the end instead of four.
    constexpr bool G2 = KT == 2;
    f32x16 acc = {0};

    double dacc = 0.0;   // sum over this thread's entries of numerator x new value (objective monitor)
    __shared__ unsigned most[64];    // of each factor, over this block's chunks (pair planes)
    if (PAIRS && tid < 64) most[tid] = 0u;    // the barriers of the first chunk come before its use
    unsigned top = 0;
    for (int64_t ch = blockIdx.x; ch < nchunks; ch += gridDim.x) {
        const int64_t j = ch * CW + jl;
        const bool okj = j < len;
        float p[NC];
#pragma unroll
        for (int ci = 0; ci < NC; ++ci) p[ci] = 0.f;
        // Partial sums in split order, a batch of splits at a time: the batch is added up by itself.
        for (int s = s_lo; s < s_hi; s += SB) {
            if (s > s_lo) request_splits(ch, s);
#pragma unroll
            for (int ci = 0; ci < NC; ++ci) {
                float b = pb[0][ci];
#pragma unroll
                for (int u = 1; u < SB; ++u) b += pb[u][ci];
                p[ci] += b;
            }
        }
        if (sp == 0) {
#pragma unroll
            for (int ci = 0; ci < NC; ++ci) Xs[(fc + FG * ci) * CW + jl] = okj && fc + FG * ci < k ? xo[ci] : 0.f;
        }
        if (SPL > 1 && sp > 0) {
#pragma unroll
            for (int ci = 0; ci < NC; ++ci) Ps[((sp - 1) * KP + fc + FG * ci) * CW + jl] = p[ci];
        }
        __syncthreads();   // Gs and the chunk's old values are complete, Ts is free
        if (PAIRS) {
            // denominators on 16 x 16 x 4 instructions, G being symmetric: 16 x 16 tiles of G X dealt to the waves, four chains of
            // 16 terms each, left in Ts where the thread of an entry finds it
            if (part) {
                const int l16 = lane & 15, quad = lane >> 4;
                for (int t = w; t < KP / 16 * (CW / 16); t += NW) {
                    const int f0 = t % (KP / 16) * 16, j0 = t / (KP / 16) * 16;
                    f32x4 d[4];
#pragma unroll
                    for (int i = 0; i < KP / 4; ++i)
                        d[i % 4] = __builtin_amdgcn_mfma_f32_16x16x4f32(Gs[(4 * i + quad) * LD + f0 + l16], Xs[(4 * i + quad) * CW + j0 + l16],
                                                                        i < 4 ? f32x4{0.f, 0.f, 0.f, 0.f} : d[i % 4], 0, 0, 0);
                    const f32x4 den = (d[0] + d[1]) + (d[2] + d[3]);
#pragma unroll
                    for (int v = 0; v < 4; ++v) Ts[(j0 + l16) * LDT + f0 + 4 * quad + v] = den[v];
                }
                __syncthreads();
            }
#pragma unroll
            for (int ci = 0; ci < NC; ++ci) {
                const int c = fc + FG * ci;
                if (c >= k) continue;
                float nv = okj ? xo[ci] : 0.f;      // Gram-only: as it is
                if (part && okj) {
                    nv = xo[ci] * p[ci] / (Ts[jl * LDT + c] + eps);
                    X[(int64_t)c * len + j] = nv;
                    dacc += (double)p[ci] * (double)nv;
                }
                Ts[jl * LDT + c] = nv;   // columns past the end contribute zeros
            }
        } else if (sp == 0) {
            // denominators: 16 old values of the column at a time against all of the thread's rows of G
            float den[NC][4];
#pragma unroll
            for (int ci = 0; ci < NC; ++ci)
#pragma unroll
                for (int u = 0; u < 4; ++u) den[ci][u] = 0.f;
            constexpr int DB = KP < 16 ? KP : 16;
#pragma unroll 1   // unrolled, every LDS read is scheduled first and the registers spill
            for (int d0 = 0; d0 < KP; d0 += DB) {
                float h[DB];
#pragma unroll
                for (int d = 0; d < DB; ++d) h[d] = Xs[(d0 + d) * CW + jl];
#pragma unroll
                for (int ci = 0; ci < NC; ++ci) {
                    const float *g = Gs + (fc + FG * ci) * LD + d0;
#pragma unroll
                    for (int d = 0; d < DB; d += 4) {
                        const f32x4 gq = *reinterpret_cast<const f32x4 *>(g + d);
#pragma unroll
                        for (int u = 0; u < 4; ++u) den[ci][u] += gq[u] * h[d + u];
                    }
                }
            }
#pragma unroll
            for (int ci = 0; ci < NC; ++ci) {
                const int c = fc + FG * ci;
#pragma unroll
                for (int q = 1; q < SPL; ++q) p[ci] += Ps[((q - 1) * KP + c) * CW + jl];
                if (c < k && part == nullptr) {
                    // Gram-only mode: no update, the tiles of the current X are produced
                    // with exactly the summation order an updating launch would use.
                    Ts[jl * LDT + c] = okj ? xo[ci] : 0.f;
                } else if (c < k) {
                    float nv = 0.f;
                    if (okj) {
                        const int64_t at = (int64_t)c * len + j;
                        nv = xo[ci] * p[ci] / (((den[ci][0] + den[ci][1]) + (den[ci][2] + den[ci][3])) + eps);
                        X[at] = nv;
                        dacc += (double)p[ci] * (double)nv;
                    }
                    Ts[jl * LDT + c] = nv;   // columns past the end contribute zeros
                }
            }
        }
        if (ch + gridDim.x < nchunks) request(ch + gridDim.x);   // other columns: nobody writes them
        __syncthreads();
        if (Xt) {
            for (int e = tid; e < CW * k; e += 64 * NW) {
                const int jj = e / k, c = e % k;
                if (ch * CW + jj < len) Xt[(ch * CW + jj) * k + c] = Ts[jj * LDT + c];
            }
        }
        constexpr int PKP = KP <= 32 ? 32 : 64;   // factor slots per row group of the planes
        if (!PAIRS && planes && tid < (CW / 8) * PKP) {
            // bf16 piece planes of the new X^T rows of this chunk (layout of split_planes_kernel)
            const int gl = tid / PKP, c = tid % PKP;
            const int64_t grow = ch * (CW / 8) + gl;
            if (grow * 8 < len) {
                u32x4 o[3];
#pragma unroll
                for (int pr = 0; pr < 4; ++pr) {
                    unsigned hh[2], mm[2], ll[2];
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const float x = (c < k) ? Ts[(8 * gl + 2 * pr + e) * LDT + c] : 0.f;
                        split3(x, hh[e], mm[e], ll[e]);
                    }
                    o[0][pr] = pack2(hh[0], hh[1]);
                    o[1][pr] = pack2(mm[0], mm[1]);
                    o[2][pr] = pack2(ll[0], ll[1]);
                }
#pragma unroll
                for (int pl = 0; pl < 3; ++pl) planes[(grow * 3 + pl) * PKP + c] = o[pl];
            }
        }
        if (PAIRS && tid < (CW / 8) * PKP) {
            // pair planes of the same rows (layout of split_pairs_kernel)
            const int gl = tid / PKP, c = tid % PKP;
            const int64_t grow = ch * (CW / 8) + gl;
            if (grow * 8 < len) {
                float x[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) x[e] = c < k ? Ts[(8 * gl + e) * LDT + c] : 0.f;
                const unsigned t = put_pairs(x, static_cast<u32x4 *>(pf.units) + grow * 2 * PKP + c, PKP, pf.exps + grow * PKP + c);
                top = t > top ? t : top;
            }
        }
        if (gout && G2) {
            const int jj = lane & 31, half = lane >> 5;
            const int ta = (w & 3) >> 1, tb = w & 1, hb = w >> 2;
#pragma unroll
            for (int q = 0; q < CW / 4; ++q) {
                const int row = (CW / 2) * hb + 2 * q + half;    // column pair of this chunk
                acc = mfma32(Ts[row * LDT + 32 * ta + jj], Ts[row * LDT + 32 * tb + jj], acc);
            }
        } else if (gout) {
            const int jj = lane & 31, half = lane >> 5;
#pragma unroll
            for (int q = 0; q < CW / 16; ++q) {
                const int row = 2 * (w + NW * q) + half;   // column pair of this chunk
                const float va = Ts[row * LDT + jj];
                acc = mfma32(va, va, acc);
            }
        }
    }
    if (dpart) {
        // <numerator, new X> of this block, summed in a fixed order (waves, then lanes by tree)
        __shared__ double dsum[NW];
        for (int off = 32; off > 0; off >>= 1) dacc += __shfl_xor(dacc, off);
        if (lane == 0) dsum[w] = dacc;
        __syncthreads();
        if (tid == 0) {
            double t = 0.0;
            for (int i = 0; i < NW; ++i) t += dsum[i];
            dpart[blockIdx.x] = t;
        }
    }
    if (!gout) return;
    if (PAIRS && top) atomicMax(&most[tid % 64], top);
    __syncthreads();   // the last chunk's readers of Ts are done: Sm changes hands
    if (PAIRS && tid < k && most[tid]) atomicMax(pf.most + tid, most[tid]);
    // Rows and columns of a tile at factor indices >= k hold whatever LDS held;
    // consumers never read them.
    // every wave parks its tile, then all threads add the copies in wave order: the two halves
    // of each of four tiles, or the eight shares of the one tile
#pragma unroll
    for (int v = 0; v < 16; ++v) Sm[w * 1024 + v * 64 + lane] = acc[v];
    __syncthreads();
    if (G2) {
        for (int e = tid; e < 4096; e += 64 * NW) {
            const int a = e >> 11, b = (e >> 10) & 1;
            if (a < kt && b < kt) gout[((int64_t)blockIdx.x * kt * kt + a * kt + b) * 1024 + (e & 1023)] = Sm[e] + Sm[4096 + e];
        }
    } else {
        float *dst = gout + (int64_t)blockIdx.x * 1024;
        for (int e = tid; e < 1024; e += 64 * NW) {
            float t = Sm[e];
#pragma unroll
            for (int ww = 1; ww < NW; ++ww) t += Sm[ww * 1024 + e];
            dst[e] = t;
        }
    }
}

// ---------------------------------------------------------------------------
// A H^T pass with the W update fused.  Workgroup = 8 waves on RT*32 rows of A;
// the waves split the columns in groups of 32 (one 128-byte line per row).
// MFMA roles: A_op = A elements (row across lanes), B_op = H elements (factor
// index across lanes), reduction over two columns; a lane's 16-byte load gives
// four instructions their operands, so both A and H are read with the same
// pattern: lane l, load u -> row l % 32, columns jb + 8u + 4 (l / 32) .. +3.
// Epilogue: waves summed through LDS in wave order, then
//   W[i][c] <- W[i][c] * Q[i][c] / (sum_d W[i][d] GH[d][c] + eps).
// dpart != nullptr: dpart[blockIdx.x] = sum over the block's entries of Q x new W in double
// (its share of <A H^T, W_new> for the objective), lanes by butterfly, then the waves in order.
// ---------------------------------------------------------------------------
template <int KT, int RT, bool VEC>
__global__ __launch_bounds__(512) void aht_pass_kernel(const float *__restrict__ A,
                                                       const float *__restrict__ H,
                                                       const float *__restrict__ GH, float *W,
                                                       int64_t rows, int64_t n, int k, float eps,
                                                       double *__restrict__ dpart)
{
    constexpr int NW = kAhtWaves;
    constexpr int RB = 32 * RT;
    constexpr int KP = 32 * KT;
    constexpr int LDQ = KP + 1;
    __shared__ float Qs[RB * LDQ];
    __shared__ float Ws[RB * LDQ];
    __shared__ float Gs[KP * LDQ];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int r = lane & 31, half = lane >> 5;
    const int64_t i0 = (int64_t)blockIdx.x * RB;

    // Stage GH (zero padded) and the old W rows of this block.
    for (int e = tid; e < KP * KP; e += 512) {
        const int d = e / KP, c = e % KP;
        Gs[d * LDQ + c] = (d < k && c < k) ? GH[d * k + c] : 0.f;
    }
    for (int e = tid; e < RB * KP; e += 512) {
        const int i = e / KP, c = e % KP;
        Ws[i * LDQ + c] = (i0 + i < rows && c < k) ? W[(i0 + i) * k + c] : 0.f;
    }

    int64_t arow[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        const int64_t row = i0 + 32 * rt + r;
        arow[rt] = (row < rows) ? row : rows - 1;   // clamped rows are discarded below
    }

    f32x16 acc[RT][KT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int t = 0; t < KT; ++t) acc[rt][t] = f32x16{0};

    struct Stage {
        f32x4 a[RT][4];
        f32x4 h[KT][4];
    };
    auto load_stage = [&](Stage &s, int64_t g) {
        const int64_t jb = 32 * g + 4 * half;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) s.a[rt][u] = load4<VEC>(A, n, arow[rt], jb + 8 * u, true);
#pragma unroll
            for (int t = 0; t < KT; ++t) s.h[t][u] = load4<VEC>(H, n, 32 * t + r, jb + 8 * u, 32 * t + r < k);
        }
    };
    const int64_t ngroups = (n + 31) >> 5;
    Stage cur, nxt;
    int64_t g = w;
    load_stage(cur, g);
    for (; g < ngroups; g += NW) {
        load_stage(nxt, g + NW);   // columns >= n read as zero, no memory access
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                    for (int t = 0; t < KT; ++t)
                        acc[rt][t] = mfma32(cur.a[rt][u][q], cur.h[t][u][q], acc[rt][t]);
        cur = nxt;
    }

    for (int ww = 0; ww < NW; ++ww) {
        if (w == ww) {
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int t = 0; t < KT; ++t)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int idx = (32 * rt + acc_row(v, half)) * LDQ + 32 * t + r;
                        if (ww == 0) Qs[idx] = acc[rt][t][v];
                        else Qs[idx] += acc[rt][t][v];
                    }
        }
        __syncthreads();
    }

    double dacc = 0.0;
    for (int e = tid; e < RB * k; e += 512) {
        const int i = e / k, c = e % k;
        if (i0 + i < rows) {
            float d0 = 0.f, d1 = 0.f;
            for (int d = 0; d + 1 < k; d += 2) {
                d0 += Ws[i * LDQ + d] * Gs[d * LDQ + c];
                d1 += Ws[i * LDQ + d + 1] * Gs[(d + 1) * LDQ + c];
            }
            if (k & 1) d0 += Ws[i * LDQ + k - 1] * Gs[(k - 1) * LDQ + c];
            const float den = (d0 + d1) + eps;
            const float wn = Ws[i * LDQ + c] * Qs[i * LDQ + c] / den;
            W[(i0 + i) * k + c] = wn;
            dacc += (double)Qs[i * LDQ + c] * (double)wn;
        }
    }
    if (dpart) {     // uniform over the grid
        __shared__ double dsum[NW];
        for (int off = 32; off > 0; off >>= 1) dacc += __shfl_xor(dacc, off);
        if (lane == 0) dsum[w] = dacc;
        __syncthreads();
        if (tid == 0) {
            double t = 0.0;
            for (int ww = 0; ww < NW; ++ww) t += dsum[ww];
            dpart[blockIdx.x] = t;
        }
    }
}

// ---------------------------------------------------------------------------
// A H^T pass on the row-major A with the W update fused, k <= 32 KT ("row plan"; 16-byte aligned
// A, n % 4 == 0, n < 2^24; the text below describes KT = 1, the end of it what KT = 2 changes).  A workgroup of 8 waves owns 32 R rows of A and W at a time
// (row blocks blockIdx.x, + gridDim.x, ...); the waves split the 64-column chunks of the
// block between them, and a wave's sub-tile is 32 rows x 64 columns, R per chunk.  MFMA
// roles: A_op = A elements (32 rows x 16 columns, a lane holds 8 consecutive columns of one
// row, cut into bf16 pieces in registers), B_op = the piece planes of H^T (16 columns x 32
// factors: the planes the H update writes for its new H; the 48 registers of a chunk serve
// all R row tiles), so the sums are the piece sums of the W^T A pass, and like there a
// matrix accumulator runs over at most 256 terms (4 chunks) before it is added, in
// rounded fp32, to totals: here totals in LDS shared by the wave pairs (w, w + 4), because
// R accumulator tiles and R total tiles do not fit a wave's registers beside the planes.
// An operand layout with lanes down the rows would make every lane of a load touch its own
// cache line, so A is loaded coalesced (a wave instruction = 4 rows x 256 contiguous bytes,
// non-temporal) and turned through a wave-private 8 KiB tile of LDS (16-byte chunks
// swizzled by row, conflict free both ways; no barrier: only the wave itself touches its
// tile).  Every row block starts its walk over the columns at another chunk (17 x block
// index): launched in step on the same columns, the workgroups would crowd the same memory
// channels (0.338 against 0.318 ms for the bare loads on 32768 x 16384).
// LDS: 64 KiB of staging tiles + 16 R KiB of totals, dynamic (above the 64 KiB a static
// array may have; a workgroup may use all 160 KiB of a compute unit).
//
// Epilogue per row block: the four totals are added in order; W <- W * Q / (W GH + eps) for
// the block's rows with GH = H H^T (k x k, complete); then from the new rows in LDS: their
// bf16 piece planes (operand of the next W^T A pass), this workgroup's share of W^T W (fp32
// matrix instruction, one tile set per workgroup in gout, which the next W^T A pass adds
// up) and, with dpart, its share of <A H^T, W_new> in double.
// KT = 2 (33 <= k <= 64): planes of 64 factor slots (96 registers per chunk), every cut of A
// feeds two accumulator chains, R = 2 (four accumulator tiles), 65-float rows in the epilogue,
// and the block's four tiles of W^T W are added to running tiles in LDS (wave w: tile w % 4
// over half w / 4 of the block's rows) instead of living in registers across row blocks.
// mode 1: no pass and no update, only the planes and the Gram share of W as it is (the
// same summation order, so that a run cut into two calls gives the same bits).  mode 2: the
// whole pass with the stores to W and its planes left out (timing).
// ---------------------------------------------------------------------------
extern __shared__ float aht_rows_lds[];
template <int R, int KT, int POLICY>
__global__ __launch_bounds__(512, 2) void aht_rows_kernel(
    const float *__restrict__ A, const u32x4 *__restrict__ planesH, const float *__restrict__ GH,
    float *W, u32x4 *__restrict__ planesW, float *__restrict__ gout,
    double *__restrict__ dpart, int64_t rows, int64_t n, int k, float eps, int mode, BlockMap bm)
{
    constexpr int NW = 8, RB = 32 * R, KP = 32 * KT, LDW = KP + 1, RT = R * KT * 1024;
    constexpr int kRsrcFlags = 0x00020000;   // raw buffer, 32-bit data format (gfx9 family)
    float *lds = aht_rows_lds;             // staging tiles: 8 x 2048 floats
    float *T = aht_rows_lds + NW * 2048;   // totals of the four wave pairs: 4 x (R x KT x 1024) floats
    float *Grun = T + 4 * RT;              // KT = 2: this workgroup's W^T W over its row blocks, 4 tiles
    double *dsum = reinterpret_cast<double *>(lds + 16368);      // used after the last row block only
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    float *stg = lds + w * 2048;
    const int jj = lane & 31, half = lane >> 5;
    const unsigned rowb = (unsigned)(n * 4);
    const int64_t nchunks = (n + 63) >> 6;
    const int64_t ngroups = (n + 7) >> 3;
    const int64_t nblocks = (rows + RB - 1) / RB;
    // coalesced loads: instruction u of a sub-tile covers rows 4u .. 4u+3, lane = (row, 16-byte chunk)
    const int lrow = lane >> 4, lch = lane & 15;
    const unsigned loff = (unsigned)lrow * rowb + (unsigned)lch * 16;
    // epilogue arrays (they alias the staging tiles; barriers separate the phases)
    float *Ws = lds;                      // old rows   [RB][LDW]
    float *Wn = lds + RB * LDW;           // new rows   [RB][LDW]
    float *Gs = lds + 2 * RB * LDW;       // H H^T      [KP][LDW]
    static_assert(2 * RB * LDW + KP * LDW <= 16368, "epilogue arrays must fit the staging tiles");
    f32x16 gacc = {0};                    // KT = 1: this wave's share of W^T W over all row blocks
    if (KT == 2)
        for (int e = tid; e < 4096; e += 64 * NW) Grun[e] = 0.f;   // first read after many barriers
    double dacc = 0.0;
    // a round = up to 4 chunks per wave (8: rows of one value 4.2e-7 off at 16384 columns, 4: 1.8e-7, in the same time)
    const int rounds = (int)((nchunks + 31) >> 5);

    for (int64_t blk = blockIdx.x; blk < nblocks; blk += gridDim.x) {
        const int64_t i0 = blk * RB;
        if (mode != 1) {
            const int64_t rot = (blk * 17) % nchunks;
            f32x16 acc[R][KT];
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int ft = 0; ft < KT; ++ft) acc[r][ft] = f32x16{0};
            struct Stage { u32x4 a[8]; };
            auto phys = [&](int64_t ch) { const int64_t c = ch + rot; return c >= nchunks ? c - nchunks : c; };
            auto load_stage = [&](Stage &s, int64_t chl, int rt) {
                const int64_t rbase = i0 + 32 * rt;
                int64_t av = rows - rbase;                  // rows of this sub-tile that exist
                av = av < 0 ? 0 : (av > 32 ? 32 : av);
                if (chl >= nchunks) av = 0;                 // past the last chunk: nothing is loaded
                const int64_t ch = av ? phys(chl) : 0;
                const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
                    const_cast<float *>(A + (av ? rbase * n + ch * 64 : 0)), 0,
                    (int)(av ? av * (int64_t)rowb - ch * 256 : 0), kRsrcFlags);
                // columns at or past n (last chunk only): the lane's offset is pushed out of range
                const unsigned lo = (ch * 64 + lch * 4 < n) ? loff : 0x7fffffffu;
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    s.a[u] = __builtin_amdgcn_raw_buffer_load_b128(ra, lo + (unsigned)(4 * u) * rowb, 0, POLICY);
            };
            u32x4 bp[4][3][KT];
            auto load_b = [&](int64_t chl) {
                const int64_t g = phys(chl) * 8;
                int64_t ng = ngroups - g;                   // 8-column groups of planes that exist
                ng = ng < 0 ? 0 : (ng > 8 ? 8 : ng);
                const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(
                    const_cast<u32x4 *>(planesH + (ng ? g : 0) * 3 * KP), 0, (int)(ng * 3 * KP * 16), kRsrcFlags);
#pragma unroll
                for (int s = 0; s < 4; ++s)
#pragma unroll
                    for (int pl = 0; pl < 3; ++pl)
#pragma unroll
                        for (int ft = 0; ft < KT; ++ft)
                            bp[s][pl][ft] = __builtin_amdgcn_raw_buffer_load_b128(
                                rp, (unsigned)((((2 * s + half) * 3 + pl) * KP + 32 * ft + jj) * 16), 0, 0);
            };
            auto to_lds = [&](const Stage &s) {
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int row = 4 * u + lrow;
                    *reinterpret_cast<f32x4 *>(stg + row * 64 + ((lch ^ (row & 15)) << 2)) = __builtin_bit_cast(f32x4, s.a[u]);
                }
            };
            auto compute = [&](f32x16 (&a)[KT]) {
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const int c0 = 4 * s + 2 * half;
                    const f32x4 x0 = *reinterpret_cast<const f32x4 *>(stg + jj * 64 + ((c0 ^ (jj & 15)) << 2));
                    const f32x4 x1 = *reinterpret_cast<const f32x4 *>(stg + jj * 64 + (((c0 + 1) ^ (jj & 15)) << 2));
                    u32x4 at[3];
                    cut2(x0.x, x0.y, at, 0);
                    cut2(x0.z, x0.w, at, 1);
                    cut2(x1.x, x1.y, at, 2);
                    cut2(x1.z, x1.w, at, 3);
                    // six piece products, smallest first (per 32-factor tile: independent chains)
                    constexpr int PA[6] = {2, 1, 0, 1, 0, 0}, PB[6] = {0, 1, 2, 0, 1, 0};
#pragma unroll
                    for (int e = 0; e < 6; ++e)
#pragma unroll
                        for (int ft = 0; ft < KT; ++ft) a[ft] = mfma_bf16(at[PA[e]], bp[s][PB[e]][ft], a[ft]);
                }
            };
            // Sub-tiles in the order (chunk, row tile); the loads of the next one are requested as soon
            // as the current one has gone to LDS.  After every round (4 chunks = 256 columns) the
            // matrix accumulators are added, in rounded fp32, to totals in LDS that the waves w and w + 4
            // share: first the lower four waves, then the upper four, a barrier after each.
            Stage s0;
            load_stage(s0, w, 0);
            float *Tp = T + (w & 3) * RT;
            for (int r = 0; r < rounds; ++r) {
                for (int t = 0; t < 4; ++t) {
                    const int64_t ch = w + 8 * (int64_t)(4 * r + t);
                    if (ch >= nchunks) break;        // this wave has no more chunks (loads already requested nothing)
                    load_b(ch);
#pragma unroll
                    for (int rt = 0; rt < R; ++rt) {
                        to_lds(s0);
                        __builtin_amdgcn_sched_barrier(0);
                        if (rt + 1 < R) load_stage(s0, ch, rt + 1);
                        else load_stage(s0, ch + 8, 0);
                        __builtin_amdgcn_sched_barrier(0);
                        compute(acc[rt]);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                if (w < 4) {
#pragma unroll
                    for (int rt = 0; rt < R * KT; ++rt) {
                        float old[16];
#pragma unroll
                        for (int v = 0; v < 16; ++v) old[v] = r ? Tp[(rt * 16 + v) * 64 + lane] : 0.f;
#pragma unroll
                        for (int v = 0; v < 16; ++v) {
                            Tp[(rt * 16 + v) * 64 + lane] = old[v] + acc[rt / KT][rt % KT][v];
                            acc[rt / KT][rt % KT][v] = 0.f;
                        }
                    }
                }
                __syncthreads();
                if (w >= 4) {
#pragma unroll
                    for (int rt = 0; rt < R * KT; ++rt) {
                        float old[16];
#pragma unroll
                        for (int v = 0; v < 16; ++v) old[v] = Tp[(rt * 16 + v) * 64 + lane];
#pragma unroll
                        for (int v = 0; v < 16; ++v) {
                            Tp[(rt * 16 + v) * 64 + lane] = old[v] + acc[rt / KT][rt % KT][v];
                            acc[rt / KT][rt % KT][v] = 0.f;
                        }
                    }
                }
                __syncthreads();
            }
            // the four pairs' totals, added in order, in place
            for (int e = tid; e < RT; e += 64 * NW)
                T[e] = ((T[e] + T[RT + e]) + T[2 * RT + e]) + T[3 * RT + e];
            __syncthreads();
        }
        // ---- H H^T and the block's rows of W ----
        if (mode != 1) {
            for (int e = tid; e < KP * KP; e += 64 * NW) {
                const int c = e / KP, d = e % KP;
                // stacked independent runs: factor indices of different runs do not interact
                const bool in = c < k && d < k && (!bm.on || bm.id[c] == bm.id[d]);
                const float v = GH[in ? c * k + d : 0];
                Gs[c * LDW + d] = in ? v : 0.f;
            }
        }
        for (int e = tid; e < RB * KP; e += 64 * NW) {
            const int i = e / KP, c = e % KP;
            const bool in = i0 + i < rows && c < k;
            const float v = W[in ? (i0 + i) * k + c : 0];
            (mode != 1 ? Ws : Wn)[i * LDW + c] = in ? v : 0.f;
        }
        __syncthreads();
        if (mode != 1) {
            for (int e = tid; e < RB * KP; e += 64 * NW) {
                const int i = e / KP, c = e % KP;
                float wn = 0.f;
                if (i0 + i < rows && c < k) {
                    float d0 = 0.f, d1 = 0.f, d2 = 0.f, d3 = 0.f;
                    const float *wr = Ws + i * LDW;
#pragma unroll
                    for (int d = 0; d < KP; d += 4) {
                        d0 += wr[d + 0] * Gs[(d + 0) * LDW + c];
                        d1 += wr[d + 1] * Gs[(d + 1) * LDW + c];
                        d2 += wr[d + 2] * Gs[(d + 2) * LDW + c];
                        d3 += wr[d + 3] * Gs[(d + 3) * LDW + c];
                    }
                    const float den = ((d0 + d1) + (d2 + d3)) + eps;
                    const int r = i & 31;
                    const float q = T[(((i >> 5) * KT + (c >> 5)) * 16 + ((r & 3) | ((r >> 3) << 2))) * 64 + 32 * ((r >> 2) & 1) + (c & 31)];
                    wn = wr[c] * q / den;
                    if (mode == 0) W[(i0 + i) * k + c] = wn;
                    dacc += (double)q * (double)wn;
                }
                Wn[i * LDW + c] = wn;
            }
            __syncthreads();
        }
        // ---- by-products of the new rows: piece planes, Gram share ----
        if (tid < (RB / 8) * KP) {
            const int gl = tid / KP, c = tid % KP;
            const int64_t grow = (i0 >> 3) + gl;
            if (grow * 8 < rows && mode != 2) {
                u32x4 o[3];
#pragma unroll
                for (int pr = 0; pr < 4; ++pr) {
                    unsigned hh[2], mm[2], ll[2];
#pragma unroll
                    for (int e = 0; e < 2; ++e) split3(Wn[(8 * gl + 2 * pr + e) * LDW + c], hh[e], mm[e], ll[e]);
                    o[0][pr] = pack2(hh[0], hh[1]);
                    o[1][pr] = pack2(mm[0], mm[1]);
                    o[2][pr] = pack2(ll[0], ll[1]);
                }
#pragma unroll
                for (int pl = 0; pl < 3; ++pl) planesW[(grow * 3 + pl) * KP + c] = o[pl];
            }
        }
        if (KT == 1) {
#pragma unroll
            for (int q = 0; q < RB / 16; ++q) {
                const float va = Wn[(2 * (w + NW * q) + half) * LDW + jj];
                gacc = mfma32(va, va, gacc);
            }
        } else {
            // the block's share of the four tiles of W^T W: wave w takes tile w % 4 over the rows of
            // half w / 4 of the block; the two halves meet in the (now free) totals and are added,
            // in order, to the running tiles
            const int ta = (w & 3) >> 1, tb = w & 1, hb = w >> 2;
            f32x16 g2 = {0};
#pragma unroll
            for (int q = 0; q < RB / 4; ++q) {
                const int row = hb * (RB / 2) + 2 * q + half;
                g2 = mfma32(Wn[row * LDW + 32 * ta + jj], Wn[row * LDW + 32 * tb + jj], g2);
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) T[hb * 4096 + (w & 3) * 1024 + v * 64 + lane] = g2[v];
            __syncthreads();
            for (int e = tid; e < 4096; e += 64 * NW) Grun[e] += T[e] + T[4096 + e];
        }
        __syncthreads();                           // LDS goes back to the staging tiles
    }
    if (dpart) {
        for (int off = 32; off > 0; off >>= 1) dacc += __shfl_xor(dacc, off);
        if (lane == 0) dsum[w] = dacc;
        __syncthreads();
        if (tid == 0) { double t = 0.0; for (int i = 0; i < NW; ++i) t += dsum[i]; dpart[blockIdx.x] = t; }
    }
    if (KT == 1) {
        // this workgroup's share of W^T W: the eight waves' tiles added in wave order
#pragma unroll
        for (int v = 0; v < 16; ++v) lds[w * 1024 + v * 64 + lane] = gacc[v];
        __syncthreads();
        for (int e = tid; e < 1024; e += 64 * NW) {
            float t = lds[e];
#pragma unroll
            for (int ww = 1; ww < NW; ++ww) t += lds[ww * 1024 + e];
            gout[(int64_t)blockIdx.x * 1024 + e] = t;
        }
    } else {
        for (int e = tid; e < 4096; e += 64 * NW) gout[(int64_t)blockIdx.x * 4096 + e] = Grun[e];
    }
}

// ---------------------------------------------------------------------------
// Both products in one reading of A, for few columns (k <= 32, 16-byte aligned A, n % 4 == 0,
// n <= 512 / NRW; the "one-pass plan").  A block of 32 NRW rows is all that the W update of these rows
// needs, and W^T A of the NEXT iteration needs only their new values: so a workgroup takes a
// block, forms A H^T, updates W and at once adds the new rows' share of W^T A and W^T W.
//   update:  W <- W * (A H^T) / (W H H^T + eps) for the block's rows (else W is taken as it is)
//   product: this workgroup's sum of W^T A over its row blocks goes to ppart[blockIdx.x] (k x n)
// and its W^T W, always, to gout (one tile set); with dpart its share of <A H^T, W> in double.
//
// 8 waves = NRW row tiles x NCW column groups; wave (rw, cw) owns 32 rows and 64 columns of the
// block.  The arithmetic is that of the other passes: A cut with rounding against truncated
// pieces of H and W, six piece products, fp32 accumulation.
//   1. A arrives coalesced (4 rows x 256 bytes per instruction, requested a block ahead) and goes
//      to the wave's 8 KiB of LDS, swizzled by row as in aht_rows_kernel; read back row by lane it
//      is the operand of A H^T (B_op: the planes of the wave's 64 columns of H^T, which stay in
//      registers over all blocks).
//   2. The waves' 32 x 32 shares of A H^T meet in LDS; each lane owns 2 NRW entries of the
//      block's rows (factor = lane % 32), for which it has formed W H H^T meanwhile; it
//      updates them, and leaves the pieces of the new rows in LDS.
//   3. Every wave reads its tile again, columns by lane, for W^T A.
// Two barriers per block.  An accumulator of W^T A takes in at most kOnePassFlush blocks (256 rows a
// wave) before it is added, in rounded fp32, to ppart (twice as many: columns of one value 4.5e-7 off
// instead of 1.9e-7, for 1 to 3 % less time).
// The pieces of W never leave the chip, and A comes from memory once per iteration instead of
// twice.  One workgroup (8 waves, 116 KiB of LDS) fills a compute unit; its chain of LDS round
// trips, not the memory, bounds it: 200000 x 400 at k = 30 takes 141 us per iteration.  It runs for 17 to 32
// factors; up to 16 one_pass16_kernel does (524288 x 512, k = 16, per pass: 215 us for the W^T A pass and 340 for
// aht_rows_kernel; averages of a trace of three ten-iteration calls, and the shortest: 357 and 314 for this kernel, 259 and
// 212 for that one).  Two chunks of columns
// per wave (n up to 1024), with the second reading from the caches, gained 0.95 to 1.15x only,
// three lost to the row plan (0.73 to 1.01x): hence the limit.
// ---------------------------------------------------------------------------
constexpr int kOnePassFlush = 8;
template <int NRW, int POLICY, bool update, bool product>
__global__ __launch_bounds__(512, 2) void one_pass_kernel(
    const float *__restrict__ A, const u32x4 *__restrict__ planesH, const float *__restrict__ GH,
    const float *__restrict__ ghsets, int nbh, const float *W, float *Wnew, float *__restrict__ ppart,
    float *__restrict__ gout, double *__restrict__ dpart, int64_t rows, int64_t n, int k, float eps)
{
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    constexpr int NCW = 8 / NRW, RB = 32 * NRW, NO = 2 * NRW, LDW = 36;
    constexpr int kRsrcFlags = 0x00020000;   // raw buffer, 32-bit data format (gfx9 family)
    constexpr unsigned kOut = 0x7fffffffu;   // an offset outside every extent: reads as zero
    float *lds = aht_rows_lds;               // staging tiles: 8 x 2048 floats
    float *Qp = lds + 8 * 2048;              // the waves' shares of A H^T: 8 x 1024
    u32x4 *Wp = reinterpret_cast<u32x4 *>(Qp + 8 * 1024);              // pieces of the new rows [3][RB / 8][32]
    float *Ws = reinterpret_cast<float *>(Wp + 3 * (RB / 8) * 32);     // old rows [RB][LDW]
    float *Gs = Ws + RB * LDW;               // H H^T [32][LDW], symmetric: row c is column c
    __shared__ double dsum[8];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rw = w / NCW, cw = w % NCW;
    const int jj = lane & 31, half = lane >> 5;
    float *stg = lds + w * 2048;
    const unsigned rowb = (unsigned)(n * 4);
    const int nchunks = (int)((n + 63) >> 6);
    const int64_t ngroups = (n + 7) >> 3;
    const int64_t nblocks = (rows + RB - 1) / RB;
    const int lrow = lane >> 4, lch = lane & 15;

    struct Rows { u32x4 a[8]; };       // coalesced: instruction u = rows 4 u .. 4 u + 3, lane = (row, 16-byte chunk)
    auto load_rows = [&](Rows &s, int64_t blk) {
        const int64_t rbase = blk * RB + 32 * rw;
        int64_t av = rows - rbase;                  // rows of this wave's tile that exist
        av = av < 0 || blk >= nblocks || cw >= nchunks ? 0 : (av > 32 ? 32 : av);
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float *>(A + (av ? rbase * n + cw * 64 : 0)), 0,
            (int)(av ? av * (int64_t)rowb - cw * 256 : 0), kRsrcFlags);
        unsigned lo = (cw * 64 + lch * 4 < n) ? (unsigned)lrow * rowb + (unsigned)lch * 16 : kOut;
        asm volatile("" : "+v"(lo));   // the rows' offsets are added here, not kept in registers across the block
#pragma unroll
        for (int u = 0; u < 8; ++u) s.a[u] = __builtin_amdgcn_raw_buffer_load_b128(r, lo + (unsigned)(4 * u) * rowb, 0, POLICY);
    };
    float wnext[NO];                   // this lane's entries of W of the next block
    const int ob = w * 4 * NRW + half * NO;
    auto load_w = [&](int64_t blk) {
        int64_t av = rows - blk * RB;
        av = av < 0 || blk >= nblocks ? 0 : (av > RB ? RB : av);
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(W + (av ? blk * RB * k : 0)), 0, (int)(av * k * 4), kRsrcFlags);
#pragma unroll
        for (int i = 0; i < NO; ++i)
            wnext[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, jj < k ? (unsigned)((ob + i) * k + jj) * 4u : kOut, 0, 0));
    };
    u32x4 bp[4][3];                    // planes of H^T, this wave's 64 columns
    if (update) {
        const int64_t g = (int64_t)cw * 8;
        int64_t ng = ngroups - g;                   // 8-column groups of planes that exist
        ng = ng < 0 ? 0 : (ng > 8 ? 8 : ng);
        const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<u32x4 *>(planesH + (ng ? g : 0) * 3 * 32), 0, (int)(ng * 3 * 32 * 16), kRsrcFlags);
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int pl = 0; pl < 3; ++pl)
                bp[s][pl] = __builtin_amdgcn_raw_buffer_load_b128(rp, (unsigned)(((2 * s + half) * 3 + pl) * 32 + jj) * 16, 0, 0);
    }
    auto to_lds = [&](const Rows &s) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int row = 4 * u + lrow;
            *reinterpret_cast<f32x4 *>(stg + row * 64 + ((lch ^ (row & 15)) << 2)) = __builtin_bit_cast(f32x4, s.a[u]);
        }
    };

    Rows ra;
    int64_t blk = blockIdx.x;
    load_rows(ra, blk);
    load_w(blk);
    if (update) {
        // H H^T: complete, or the H update's tile sets added up, a batch of 16 at a time
        constexpr int B = 16;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int e = tid + 512 * i, d = e >> 5, c = e & 31;
            const bool in = c < k && d < k;
            const int pos = ((d & 3) + 4 * (d >> 3)) * 64 + c + 32 * ((d >> 2) & 1);
            float g = 0.f;
            if (GH) {
                g = GH[in ? d * k + c : 0];
            } else {
                for (int b = 0; b < nbh; b += B) {
                    float t[B];
#pragma unroll
                    for (int u = 0; u < B; ++u) t[u] = ghsets[(b + u < nbh ? b + u : 0) * 1024 + (in ? pos : 0)];
#pragma unroll
                    for (int u = 0; u < B; ++u) t[u] = b + u < nbh ? t[u] : 0.f;
                    g += tree_sum(t);
                }
            }
            Gs[d * LDW + c] = in ? g : 0.f;
        }
        __syncthreads();
    }

    f32x16 acc[2], gacc = {0};
    acc[0] = f32x16{0};
    acc[1] = f32x16{0};
    double dacc = 0.0;
    bool first = true;      // nothing in ppart yet
    // adds the accumulators to this workgroup's partial; the row tiles of a column group in order
    auto flush = [&]() {
        if (NRW > 1) {
            __syncthreads();          // the staging tiles are free
            if (rw > 0) {
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int v = 0; v < 16; ++v) stg[(q * 16 + v) * 64 + lane] = acc[q][v];
            }
            __syncthreads();
        }
        if (rw == 0) {
            // nothing to add to yet: an extent of zero reads as zeros; factors and columns that do not
            // exist lie outside the extent and are dropped
            float *part = ppart + (int64_t)blockIdx.x * k * n;
            const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(part, 0, first ? 0 : k * (int)rowb, kRsrcFlags);
            const __amdgpu_buffer_rsrc_t rn = __builtin_amdgcn_make_buffer_rsrc(part, 0, k * (int)rowb, kRsrcFlags);
            const int col = cw * 64 + 2 * jj;
            unsigned at = col < n ? (unsigned)(4 * half) * rowb + (unsigned)col * 4 : kOut;
            asm volatile("" : "+v"(at));
            u32x2 old[16];
#pragma unroll
            for (int v = 0; v < 16; ++v) old[v] = __builtin_amdgcn_raw_buffer_load_b64(ro, at + (unsigned)acc_row(v, 0) * rowb, 0, 0);
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                f32x2 val = {acc[0][v], acc[1][v]};
#pragma unroll
                for (int r = 1; r < NRW; ++r) {
                    const float *o = lds + (r * NCW + cw) * 2048;
                    val.x += o[v * 64 + lane];
                    val.y += o[(16 + v) * 64 + lane];
                }
                val.x += __uint_as_float(old[v].x);
                val.y += __uint_as_float(old[v].y);
                __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, val), rn, at + (unsigned)acc_row(v, 0) * rowb, 0, 0);
            }
        }
        if (NRW > 1) __syncthreads();
        acc[0] = f32x16{0};
        acc[1] = f32x16{0};
        first = false;
    };
    constexpr int PA[6] = {2, 1, 0, 1, 0, 0}, PB[6] = {0, 1, 2, 0, 1, 0};   // smallest first
    int done = 0;
    for (; blk < nblocks; blk += gridDim.x) {
        const int64_t i0 = blk * RB, next = blk + gridDim.x;
        float wold[NO];
#pragma unroll
        for (int i = 0; i < NO; ++i) {
            wold[i] = wnext[i];
            Ws[(ob + i) * LDW + jj] = wold[i];
        }
        to_lds(ra);
        __builtin_amdgcn_sched_barrier(0);
        load_rows(ra, next);
        load_w(next);
        __builtin_amdgcn_sched_barrier(0);
        float wn[NO];
        if (update) {
            f32x16 q[2];
            q[0] = f32x16{0};
            q[1] = f32x16{0};
#pragma unroll
            for (int s = 0; s < 4; s += 2) {      // two steps, two chains of products
                u32x4 at[2][3];
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const int c0 = 4 * (s + t) + 2 * half;
                    const f32x4 x0 = *reinterpret_cast<const f32x4 *>(stg + jj * 64 + ((c0 ^ (jj & 15)) << 2));
                    const f32x4 x1 = *reinterpret_cast<const f32x4 *>(stg + jj * 64 + (((c0 + 1) ^ (jj & 15)) << 2));
                    cut2(x0.x, x0.y, at[t], 0);
                    cut2(x0.z, x0.w, at[t], 1);
                    cut2(x1.x, x1.y, at[t], 2);
                    cut2(x1.z, x1.w, at[t], 3);
                }
#pragma unroll
                for (int e = 0; e < 6; ++e)
#pragma unroll
                    for (int t = 0; t < 2; ++t) q[t] = mfma_bf16(at[t][PA[e]], bp[s + t][PB[e]], q[t]);
                __builtin_amdgcn_sched_barrier(0);   // hoisted LDS reads would spill
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) Qp[w * 1024 + v * 64 + lane] = q[0][v] + q[1][v];
            // W H H^T of this lane's entries (its wave wrote their rows above)
            float den[NO];
#pragma unroll
            for (int i = 0; i < NO; ++i) den[i] = 0.f;
            // 16 factors in two sums, then into the total: four running sums of all take the registers that the block in
            // flight needs (262144 x 256, k = 32: 141 us per iteration, 131 so)
            for (int d0 = 0; d0 < k; d0 += 16) {
                float s0[NO], s1[NO];
#pragma unroll
                for (int i = 0; i < NO; ++i) s0[i] = s1[i] = 0.f;
#pragma unroll 2
                for (int d = d0; d < d0 + 16; d += 4) {
                    const f32x4 g = *reinterpret_cast<const f32x4 *>(Gs + jj * LDW + d);
#pragma unroll
                    for (int i = 0; i < NO; ++i) {
                        const f32x4 x = *reinterpret_cast<const f32x4 *>(Ws + (ob + i) * LDW + d);
                        s0[i] += x.x * g.x;
                        s1[i] += x.y * g.y;
                        s0[i] += x.z * g.z;
                        s1[i] += x.w * g.w;
                    }
                }
#pragma unroll
                for (int i = 0; i < NO; ++i) den[i] += s0[i] + s1[i];
            }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < NO; ++i) {
                const int row = ob + i, rt = row >> 5, r = row & 31;
                const float *src = Qp + rt * NCW * 1024 + ((r & 3) | ((r >> 3) << 2)) * 64 + 32 * ((r >> 2) & 1) + jj;
                float qs = src[0];
#pragma unroll
                for (int c = 1; c < NCW; ++c) qs += src[c * 1024];
                wn[i] = 0.f;
                if (i0 + row < rows && jj < k) {
                    wn[i] = wold[i] * qs / (den[i] + eps);
                    if (Wnew) Wnew[(i0 + row) * k + jj] = wn[i];
                    dacc += (double)qs * (double)wn[i];
                }
            }
        } else {
            __syncthreads();           // the last block's readers of Wp are done
#pragma unroll
            for (int i = 0; i < NO; ++i) wn[i] = wold[i];
        }
#pragma unroll
        for (int i = 0; i < NO; ++i) gacc = mfma32(wn[i], wn[i], gacc);   // rows of the two halves
        if (product) {
#pragma unroll
            for (int i = 0; i < NO; i += 2) {
                unsigned h[2], m[2], l[2];
                split3(wn[i], h[0], m[0], l[0]);
                split3(wn[i + 1], h[1], m[1], l[1]);
                const int row = ob + i;
                unsigned *dst = reinterpret_cast<unsigned *>(Wp + (row >> 3) * 32 + jj) + ((row & 7) >> 1);
                dst[0] = pack2(h[0], h[1]);
                dst[(RB / 8) * 32 * 4] = pack2(m[0], m[1]);
                dst[2 * (RB / 8) * 32 * 4] = pack2(l[0], l[1]);
            }
            __syncthreads();
#pragma unroll
            for (int st = 0; st < 2; ++st) {
                u32x2 x[8];            // columns 2 jj, 2 jj + 1 of rows 16 st + 8 half + e
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int row = 16 * st + 8 * half + e;
                    x[e] = *reinterpret_cast<const u32x2 *>(stg + row * 64 + (((jj >> 1) ^ (row & 15)) << 2) + ((jj & 1) << 1));
                }
                u32x4 wt[3], at[2][3];
#pragma unroll
                for (int pl = 0; pl < 3; ++pl) wt[pl] = Wp[(pl * (RB / 8) + 4 * rw + 2 * st + half) * 32 + jj];
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int pr = 0; pr < 4; ++pr) cut2(__uint_as_float(x[2 * pr][q]), __uint_as_float(x[2 * pr + 1][q]), at[q], pr);
#pragma unroll
                for (int e = 0; e < 6; ++e)
#pragma unroll
                    for (int q = 0; q < 2; ++q) acc[q] = mfma_bf16(wt[PB[e]], at[q][PA[e]], acc[q]);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (++done == kOnePassFlush) {
                flush();
                done = 0;
            }
        } else {
            __syncthreads();           // the shares of A H^T are read; the next block writes its own
        }
    }
    if (product && done) flush();
    if (dpart) {
        for (int off = 32; off > 0; off >>= 1) dacc += __shfl_xor(dacc, off);
        if (lane == 0) dsum[w] = dacc;
    }
    // this workgroup's W^T W: the eight waves' tiles added in wave order
    __syncthreads();
#pragma unroll
    for (int v = 0; v < 16; ++v) Qp[w * 1024 + v * 64 + lane] = gacc[v];
    __syncthreads();
    for (int e = tid; e < 1024; e += 512) {
        float t = Qp[e];
#pragma unroll
        for (int ww = 1; ww < 8; ++ww) t += Qp[ww * 1024 + e];
        gout[(int64_t)blockIdx.x * 1024 + e] = t;
    }
    if (dpart && tid == 0) {
        double t = 0.0;
        for (int i = 0; i < 8; ++i) t += dsum[i];
        dpart[blockIdx.x] = t;
    }
}

// ---------------------------------------------------------------------------
// one_pass_kernel for up to 16 factors and many rows, on 16 x 16 x 32 instructions: the same block of 32 NRW rows, the
// same partials and tile sets per workgroup, but 16 waves with 32 columns and 32 rows each.  With 32 factor slots half
// of the matrix work, of the planes and of the accumulators would be padding, and 8 waves that pass through a chain of
// LDS round trips in step left the memory idle for half of it: 357 us per pass on 524288 x 512 at k = 16 on average.  Here a
// wave's share of a block is half as long, and its registers (four loads, one step of planes, two column tiles) leave room
// for 16 waves; the running totals stay in registers (8 per lane) instead of going to ppart every 8 blocks.
//   1. A arrives coalesced (8 rows x 128 bytes per instruction, a block ahead) and goes to the wave's 4 KiB of LDS, 16-byte
//      chunks flipped by (row / 2) % 8; read back row by lane for A H^T: two 16-row tiles, one step of 32 columns.
//   2. The column groups' shares of A H^T meet in LDS; thread tid owns entry (row tid / 16, factor tid % 16).
//   3. The wave reads its tile again, columns by lane (two per lane), all 32 rows the depth of one instruction.
// The largest products have an accumulator of their own (see resident_kernel).
// ---------------------------------------------------------------------------
template <int NRW, int POLICY, bool update, bool product>
__global__ __launch_bounds__(1024, 1) void one_pass16_kernel(
    const float *__restrict__ A, const u32x4 *__restrict__ planesH, const float *__restrict__ GH,
    const float *__restrict__ ghsets, int nbh, const float *W, float *Wnew, float *__restrict__ ppart,
    float *__restrict__ gout, double *__restrict__ dpart, int64_t rows, int64_t n, int k, float eps)
{
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    constexpr int NW = 16, NCW = NW / NRW, RB = 32 * NRW, LD = 20;
    constexpr int kRsrcFlags = 0x00020000;   // raw buffer, 32-bit data format (gfx9 family)
    constexpr unsigned kOut = 0x7fffffffu;   // an offset outside every extent: reads as zero
    float *lds = aht_rows_lds;               // staging tiles: 16 x 1024 floats
    float *Qp = lds + NW * 1024;             // the waves' shares of A H^T: 16 x 512
    float *Ws = Qp + NW * 512;               // old rows [RB][LD]
    float *Gs = Ws + RB * LD;                // H H^T [16][LD]
    unsigned short *Wp = reinterpret_cast<unsigned short *>(Gs + 16 * LD);   // pieces of the new rows [3][RB / 8][16][8]
    __shared__ double dsum[NW];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rw = w / NCW, cw = w % NCW;
    const int l16 = lane & 15, quad = lane >> 4;
    float *stg = lds + w * 1024;
    const unsigned rowb = (unsigned)(n * 4);
    const int64_t nblocks = (rows + RB - 1) / RB;
    const bool has_cols = cw * 32 < n;
    const int lrow = lane >> 3, lch = lane & 7;

    struct Rows { u32x4 a[4]; };       // coalesced: instruction u = rows 8 u .. 8 u + 7, lane = (row, 16-byte chunk)
    auto load_rows = [&](Rows &s, int64_t blk) {
        const int64_t rbase = blk * RB + 32 * rw;
        int64_t av = rows - rbase;                  // rows of this wave's tile that exist
        av = av < 0 || blk >= nblocks || !has_cols ? 0 : (av > 32 ? 32 : av);
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float *>(A + (av ? rbase * n + cw * 32 : 0)), 0,
            (int)(av ? av * (int64_t)rowb - cw * 128 : 0), kRsrcFlags);
        unsigned lo = (cw * 32 + lch * 4 < n) ? (unsigned)lrow * rowb + (unsigned)lch * 16 : kOut;
        asm volatile("" : "+v"(lo));   // the rows' offsets are added here, not kept in registers across the block
#pragma unroll
        for (int u = 0; u < 4; ++u) s.a[u] = __builtin_amdgcn_raw_buffer_load_b128(r, lo + (unsigned)(8 * u) * rowb, 0, POLICY);
    };
    const int er = tid >> 4, ec = tid & 15;         // this thread's entry of the block's rows of W
    const bool entry = tid < RB * 16;
    float wnext;
    auto load_w = [&](int64_t blk) {
        int64_t av = rows - blk * RB;
        av = av < 0 || blk >= nblocks ? 0 : (av > RB ? RB : av);
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(W + (av ? blk * RB * k : 0)), 0, (int)(av * k * 4), kRsrcFlags);
        wnext = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, entry && ec < k ? (unsigned)(er * k + ec) * 4u : kOut, 0, 0));
    };
    u32x4 bp[3];                       // planes of H^T (32 factor slots), this wave's 32 columns
    if (update) {
        const int64_t ngroups = (n + 7) >> 3, g = (int64_t)cw * 4;
        int64_t ng = ngroups - g;                   // 8-column groups of planes that exist
        ng = ng < 0 ? 0 : (ng > 4 ? 4 : ng);
        const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<u32x4 *>(planesH + (ng ? g : 0) * 3 * 32), 0, (int)(ng * 3 * 32 * 16), kRsrcFlags);
#pragma unroll
        for (int pl = 0; pl < 3; ++pl)
            bp[pl] = __builtin_amdgcn_raw_buffer_load_b128(rp, (unsigned)((quad * 3 + pl) * 32 + l16) * 16, 0, 0);
    }
    Rows ra;
    int64_t blk = blockIdx.x;
    load_rows(ra, blk);
    load_w(blk);
    if (update) {
        // H H^T: complete, or the H update's tile sets added up, a batch of 16 at a time
        constexpr int B = 16;
        if (tid < 256) {
            const bool in = ec < k && er < k;
            const int pos = ((er & 3) + 4 * (er >> 3)) * 64 + ec + 32 * ((er >> 2) & 1);
            float g = 0.f;
            if (GH) {
                g = GH[in ? er * k + ec : 0];
            } else {
                for (int b = 0; b < nbh; b += B) {
                    float t[B];
#pragma unroll
                    for (int u = 0; u < B; ++u) t[u] = ghsets[(b + u < nbh ? b + u : 0) * 1024 + pos];
#pragma unroll
                    for (int u = 0; u < B; ++u) t[u] = b + u < nbh ? t[u] : 0.f;
                    g += tree_sum(t);
                }
            }
            Gs[er * LD + ec] = in ? g : 0.f;
        }
        __syncthreads();
    }

    f32x4 acc[2][2], tot[2], gacc = {0.f, 0.f, 0.f, 0.f};      // acc: [column parity][small products, large ones]
#pragma unroll
    for (int q = 0; q < 2; ++q) acc[q][0] = acc[q][1] = tot[q] = f32x4{0.f, 0.f, 0.f, 0.f};
    double dacc = 0.0;
    constexpr int PA[6] = {2, 1, 0, 1, 0, 0}, PB[6] = {0, 1, 2, 0, 1, 0};   // smallest first
    int done = 0;
    auto settle = [&]() {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            tot[q] += acc[q][0] + acc[q][1];
            acc[q][0] = acc[q][1] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        done = 0;
    };
    for (; blk < nblocks; blk += gridDim.x) {
        const int64_t i0 = blk * RB, next = blk + gridDim.x;
        const float wold = wnext;
        if (entry) Ws[er * LD + ec] = wold;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int row = 8 * u + lrow;
            *reinterpret_cast<f32x4 *>(stg + row * 32 + ((lch ^ ((row >> 1) & 7)) << 2)) = __builtin_bit_cast(f32x4, ra.a[u]);
        }
        __builtin_amdgcn_sched_barrier(0);
        load_rows(ra, next);
        load_w(next);
        __builtin_amdgcn_sched_barrier(0);
        float wn = wold;
        if (update) {
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int row = 16 * t + l16, sw = (row >> 1) & 7;
                const f32x4 x0 = *reinterpret_cast<const f32x4 *>(stg + row * 32 + (((2 * quad) ^ sw) << 2));
                const f32x4 x1 = *reinterpret_cast<const f32x4 *>(stg + row * 32 + (((2 * quad + 1) ^ sw) << 2));
                u32x4 at[3];
                cut2(x0.x, x0.y, at, 0);
                cut2(x0.z, x0.w, at, 1);
                cut2(x1.x, x1.y, at, 2);
                cut2(x1.z, x1.w, at, 3);
                f32x4 q[2];
                q[0] = q[1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int e = 0; e < 6; ++e) q[e / 5] = mfma_bf16_16(at[PA[e]], bp[PB[e]], q[e / 5]);
#pragma unroll
                for (int v = 0; v < 4; ++v) Qp[w * 512 + (16 * t + 4 * quad + v) * 16 + l16] = q[0][v] + q[1][v];
            }
            float den = 0.f;           // W H H^T of this thread's entry (its wave wrote the row above)
            if (entry) {
                float s0 = 0.f, s1 = 0.f;
#pragma unroll
                for (int d = 0; d < 16; d += 4) {
                    const f32x4 g = *reinterpret_cast<const f32x4 *>(Gs + ec * LD + d);
                    const f32x4 x = *reinterpret_cast<const f32x4 *>(Ws + er * LD + d);
                    s0 += x.x * g.x;
                    s1 += x.y * g.y;
                    s0 += x.z * g.z;
                    s1 += x.w * g.w;
                }
                den = s0 + s1;
            }
            __syncthreads();
            if (entry) {
                const float *src = Qp + (er >> 5) * NCW * 512 + (er & 31) * 16 + ec;
                float t[NCW];
#pragma unroll
                for (int c = 0; c < NCW; ++c) t[c] = src[c * 512];
                const float qs = tree_sum(t);
                wn = 0.f;
                if (i0 + er < rows && ec < k) {
                    wn = wold * qs / (den + eps);
                    if (Wnew) Wnew[(i0 + er) * k + ec] = wn;
                    dacc += (double)qs * (double)wn;
                }
            }
        } else {
            __syncthreads();           // the last block's readers of Wp are done
        }
        gacc = __builtin_amdgcn_mfma_f32_16x16x4f32(wn, wn, gacc, 0, 0, 0);     // the wave's four rows (no entry: zeros)
        if (product) {
            if (entry) {
                unsigned h, m, l;
                split3(wn, h, m, l);
                unsigned short *dst = Wp + ((er >> 3) * 16 + ec) * 8 + (er & 7);
                dst[0] = (unsigned short)(h >> 16);
                dst[(RB / 8) * 128] = (unsigned short)(m >> 16);
                dst[2 * (RB / 8) * 128] = (unsigned short)(l >> 16);
            }
            __syncthreads();
            u32x2 x[8];                // columns 2 l16, 2 l16 + 1 of rows 8 quad + e
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int row = 8 * quad + e;
                x[e] = *reinterpret_cast<const u32x2 *>(stg + row * 32 + (((l16 >> 1) ^ ((row >> 1) & 7)) << 2) + ((l16 & 1) << 1));
            }
            u32x4 wt[3];
#pragma unroll
            for (int pl = 0; pl < 3; ++pl) wt[pl] = reinterpret_cast<const u32x4 *>(Wp)[(pl * (RB / 8) + 4 * rw + quad) * 16 + l16];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                u32x4 at[3];
#pragma unroll
                for (int pr = 0; pr < 4; ++pr) cut2(__uint_as_float(x[2 * pr][q]), __uint_as_float(x[2 * pr + 1][q]), at, pr);
#pragma unroll
                for (int e = 0; e < 6; ++e) acc[q][e / 5] = mfma_bf16_16(at[PA[e]], wt[PB[e]], acc[q][e / 5]);
            }
            if (++done == kOnePassFlush) settle();
        } else {
            __syncthreads();           // the shares of A H^T are read; the next block writes its own
        }
    }
    if (product) {
        settle();
        if (NRW > 1) {                 // the row tiles of a column group in order
            __syncthreads();
            if (rw > 0) {
#pragma unroll
                for (int q = 0; q < 2; ++q) *reinterpret_cast<f32x4 *>(stg + (q * 64 + lane) * 4) = tot[q];
            }
            __syncthreads();
            if (rw == 0) {
#pragma unroll
                for (int r = 1; r < NRW; ++r)
#pragma unroll
                    for (int q = 0; q < 2; ++q) tot[q] += *reinterpret_cast<const f32x4 *>(lds + (r * NCW + cw) * 1024 + (q * 64 + lane) * 4);
            }
        }
        if (rw == 0) {                 // lane: factor l16, columns 8 quad .. 8 quad + 7 of the wave's
            const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(ppart + (int64_t)blockIdx.x * k * n, 0, k * (int)rowb, kRsrcFlags);
#pragma unroll
            for (int v = 0; v < 4; v += 2) {
                const int col = cw * 32 + 8 * quad + 2 * v;
                const f32x4 val = {tot[0][v], tot[1][v], tot[0][v + 1], tot[1][v + 1]};
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, val), ro, l16 < k && col < n ? (unsigned)l16 * rowb + (unsigned)col * 4u : kOut, 0, 0);
            }
        }
    }
    if (dpart) {
        for (int off = 32; off > 0; off >>= 1) dacc += __shfl_xor(dacc, off);
        if (lane == 0) dsum[w] = dacc;
    }
    // this workgroup's W^T W: the waves' tiles added in wave order
    __syncthreads();
    *reinterpret_cast<f32x4 *>(Qp + w * 256 + l16 * 16 + 4 * quad) = gacc;
    __syncthreads();
    {
        // a tile set in the layout of the 32 x 32 accumulators; beyond 16 factors zero
        const int v = tid >> 6, r = acc_row(v, (tid >> 5) & 1), c = tid & 31;
        float t = 0.f;
        if (r < 16 && c < 16)
            for (int ww = 0; ww < NW; ++ww) t += Qp[ww * 256 + c * 16 + r];
        gout[(int64_t)blockIdx.x * 1024 + tid] = t;
    }
    if (dpart && tid == 0) {
        double t = 0.0;
        for (int i = 0; i < NW; ++i) t += dsum[i];
        dpart[blockIdx.x] = t;
    }
}

// ---------------------------------------------------------------------------
// A whole run in one launch, for matrices that the chip holds on its compute units (k <= 16; the "resident
// plan").  What such a run costs otherwise is launches and trips to L2: four dependent kernels of 3 to 12 us
// per iteration whatever the work in them.  Here a workgroup keeps a tile of A, 16 RT rows x 256 columns, on its
// compute unit over all iterations; workgroup (r, c) of R x C has rows 16 RT r .. and columns 256 c ...
//   product:   the share of its rows in W^T A (its columns) and in W^T W, for column group c;
//   H update:  the 16-column tiles of group c are dealt to its R workgroups, which add up the R shares;
//   A H^T:     the share of its columns in A H^T (its rows) and in H H^T, for row group r;
//   W update:  the 16-row tiles of group r are dealt to its C workgroups, which add up the C shares.
// Each of the four hands its result through memory to the other workgroups of the group (with C = 1 the last two
// stay on chip): the workgroup posts a flag behind its stores and waits for the flags of its group.  Cutting
// A both ways keeps what is handed over small: with 16-row blocks of whole rows, 2000 x 1201 at k = 12 wrote
// and read 9.6 MB of shares of W^T A per iteration, against 2.4 MB in all, and took 18.4 us.
//
// The arithmetic is that of the other passes, on 16 x 16 x 32 instructions: six products of pieces, A cut with
// rounding once per run.  For A H^T (operand: lane = row, 8 columns) the pieces stay in registers: wave
// (rt, cw) has row tile rt and RT of the tile's eight 32-column steps.  For W^T A (lane = column, 8 rows) they
// stay in LDS: wave w has columns 32 w .. 32 w + 31.  16 rows fill only half of an instruction's depth, so its
// halves take two different piece products: three instructions for the six.  H H^T and W^T W are on the
// fp32 instruction.  A matrix accumulator takes in at most 256 terms, and the largest products have one of their own
// that meets the others in a rounded add: what the instruction drops when they join it is always downwards and shows
// as a drift of the factors' scale over many iterations.
//
// Who waits for a flag must know that its writer runs.  The workgroups first report in, and when all have (all hold
// their compute units then) the run starts.  If they have not after `patience` ticks of the 100 MHz counter (other
// kernels, another such launch, a stream with few compute units), those that have start without the others: an
// iteration's work of all R C is dealt to them, each does its share one workgroup's after the other, tiles loaded anew,
// with barriers of all (the "shared" run).  After each iteration the first looks who has reported in meanwhile and
// deals again; as soon as all have, each keeps its own tile from there on.  So every wait is for a
// workgroup that runs, whatever else the device does; the sums, and so the bits, are the same.  Microseconds per iteration
// with all, all but one, half and a quarter of the workgroups, and with one: 2000 x 1201, k = 12 11.5, 29.6, 35.2, 59, 1900;
// 16384 x 256, k = 16 17.2, 37.3, 38.5, 63, 3500 (the other plans on the whole device: 27.8 and 33.6; on half of it 28.5 and 43).  The two bodies apart
// also took a tenth off the iterations of all (256 x 192, k = 4: 7.3 -> 6.5 us): fewer scalar registers to spill.
// Only a caller that breaks the rule of one call at a time per workspace can take flags away from a run that waits for
// them: each wait has `polls` looks (ten seconds or more), then the launch is marked as lost, nobody waits in it any
// longer and it ends; the last workgroup to leave stores a NaN in W[0] and H[0].  The last updates store to W and H behind the
// L2s, so that no line of an L2 is written back over it.  (A launch behind the run for this: 2 to 6 us more per call.)
// A launch does a bounded number of iterations (resident_piece): a longer run is cut, which gives the same bits.
// Stores and loads of what workgroups exchange carry the sc1 bit: they meet behind the L2s of the XCDs.
// (Plain loads after an acquire at the flags, which drops the L2's copies, were slower: 19.5 for 18.4 us.)
// ---------------------------------------------------------------------------
constexpr int kExchange = 16;            // sc1: coherent over the whole device
constexpr unsigned kLostPolls = 1u << 24;     // looks, not time: a process that is switched out does not look
constexpr int kPRec = kResidentPRec;
__host__ __device__ constexpr int resident_lds_floats(int rt)
{
    return 8 * 2 * rt * 384 + 3 * 32 * 16 * 4 + 2 * 2048 + rt * 16 * 20 + 3 * 16 * 20 + 3 * rt * 128 + 24;
}

__device__ __forceinline__ unsigned peek(const unsigned *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void post(unsigned *p, unsigned x) { __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ unsigned add_one(unsigned *p) { return __hip_atomic_fetch_add(p, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void put_through(float *p, float x) { __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ bool decide(unsigned *p, unsigned x)      // if nobody has
{
    unsigned none = 0u;
    return __hip_atomic_compare_exchange_strong(p, &none, x, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// How many have reported in, within what a deal may say whatever other calls do to the word.
__device__ __forceinline__ unsigned resident_here(const ResidentArgs &a, int most)
{
    const int here = (int)peek(a.sync + kResidentHere);
    return (unsigned)(here < 1 ? 1 : here > most ? most : here);
}

// Waits of one thread for a word to reach a value.
struct Patient {
    unsigned *lost_word;
    unsigned polls;
    unsigned lost;                     // this thread waits no more
    __device__ __forceinline__ void await(const unsigned *from, unsigned least)
    {
        for (unsigned looks = 1; !lost && peek(from) < least; ++looks) {
            __builtin_amdgcn_s_sleep(1);
            lost = looks >= polls || (looks % 4096 == 0 && peek(lost_word) != 0u);
            if (lost) post(lost_word, 1u);
        }
    }
};

// Iterations `s` .. of the workgroup.  SHARED: the work of several, dealt anew after every iteration; returns
// the iteration from which all workgroups are there, or -1 after the last.  EVERY: all updates of W leave their part of the
// objective (a.gw), not only the last (if a.dpart).  (A launch per reported iteration took 20 us more each: 4096 x 1024,
// k = 8, 20 iterations 903 us a call, 802 on the row plan, 340 so.  As a run-time case: 3 % on runs that report nothing.)
template <int RT, bool EVERY, bool SHARED>
__device__ __forceinline__ int resident_iterations(const ResidentArgs &a, int s, unsigned ticket, unsigned deal)
{
    constexpr int kRsrcFlags = 0x00020000;         // raw buffer, 32-bit data format (gfx9 family)
    constexpr unsigned kOut = 0x7fffffffu;         // an offset outside every extent: reads as zero, stores nothing
    constexpr int LD = 20, RB = 16 * RT, CW = 8 / RT, NE = (RT * 256 + 511) / 512, kQRec = resident_qrec(RT);
    constexpr int PA[6] = {2, 1, 0, 1, 0, 0}, PB[6] = {0, 1, 2, 0, 1, 0};   // smallest first
    float *lds = aht_rows_lds;
    u32x4 *Ap = reinterpret_cast<u32x4 *>(lds);                    // [wave][2 tiles][RT][3 pieces][2][16 columns]
    u32x4 *Hp = Ap + 8 * 2 * RT * 96;                              // pieces of H: [3][32 groups of 8 columns][16]
    float *Qs = reinterpret_cast<float *>(Hp + 3 * 32 * 16);       // shares of the waves: [8][256]
    float *Gq = Qs + 2048;
    float *Ws = Gq + 2048;                                         // [RB rows][LD]
    float *Gs = Ws + RB * LD;                                      // H H^T or W^T W [16][LD]
    float *Gl = Gs + 16 * LD;                                      // what the float of an entry of Gs leaves out
    float *Hs = Gl + 16 * LD;                                      // [16 columns][LD]
    unsigned short *Wp = reinterpret_cast<unsigned short *>(Hs + 16 * LD);   // pieces of the rows [3][RB / 8][16][8]
    unsigned *word = reinterpret_cast<unsigned *>(Hs + 16 * LD + 3 * RT * 128);
    double *dsum = reinterpret_cast<double *>(word + 2);
    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int er = (tid >> 4) & 15, ec = tid & 15;
    // The lane, with 4 row tiles found again in every iteration: what follows from it (offsets, masks) would else be kept in
    // registers over the loop, 15 more than there are (2000 x 1201, k = 12: 12.3 us an iteration instead of 11.2).
    int lane, l16, quad, hr, half;
    auto place = [&]() {
        lane = tid & 63;
        if (RT > 2) asm volatile("" : "+v"(lane));
        l16 = lane & 15;
        quad = lane >> 4;
        hr = quad & 1;
        half = lane >> 5;
    };
    place();
    const int k = a.k, R = a.R, C = a.C, nwg = R * C, n = (int)a.n;
    const int nt = (n + 15) >> 4;                                  // 16-column tiles in all
    const int rpad = (R + 31) & ~31, box = rpad + 32;              // words of a workgroup's letter box: column group, row group

    // The workgroups this one stands for.  Shared: far apart, as the first ones own the column tiles.
    const int v0 = SHARED ? (int)ticket : (int)blockIdx.x, v1 = SHARED ? nwg : v0 + 1, r0 = v0 / C, c0 = v0 % C;
    int step = SHARED ? (int)(deal & 511) : 1;
    unsigned epoch = 0, target = 0;
    unsigned *boxes = a.sync + kResidentHead;
    // Posts a flag behind all stores of this workgroup to every other of its column or row group, then waits for
    // theirs.  Each has its own letter box: with one array of flags that all poll, the few lines of it are what a
    // wait of 125 workgroups waits for (9000 cycles instead of 3000 of 16).
    Patient thread{a.sync + kResidentLost, a.polls, 0u};
    auto meet = [&](bool column) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        ++epoch;
        if (SHARED) {                  // all that are here
            if (tid == 0) {
                add_one(a.sync + kResidentArrived);
                if (ticket == 0) {
                    target += deal & 511;
                    thread.await(a.sync + kResidentArrived, target);
                    post(a.sync + kResidentRelease, epoch);
                } else {
                    thread.await(a.sync + kResidentRelease, epoch);
                }
            }
        } else if (tid < (column ? R : C)) {
            post(boxes + (column ? (tid * C + c0) * box + r0 : (r0 * C + tid) * box + rpad + c0), epoch);
            thread.await(boxes + v0 * box + (column ? 0 : rpad) + tid, epoch);
        }
        asm volatile("" ::: "memory");
        __syncthreads();
    };

    u32x4 at[RT][3];                   // operand of A H^T
    // The tile as the operand of A H^T, of W^T A, or both (a shared run loads what the half it is at needs).
    auto load_tile = [&](int r, int c, bool for_aht, bool for_wta) {
        const int64_t row0 = (int64_t)r * RB;
        int64_t av = a.m - row0;
        av = av > RB ? RB : av;
        const int col0 = c * 256, rt = w / CW;
        const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float *>(a.A + row0 * n), 0, (int)(av * n * 4), kRsrcFlags);
        int opaque = 0;
        asm volatile("" : "+s"(opaque));      // the offsets are formed here, once, and not kept in registers over the run
#pragma unroll
        for (int i = 0; i < (for_aht ? RT : 0); ++i) {
            const int cc = opaque + col0 + 32 * (w % CW + CW * i) + 8 * quad;
            float x[8];
#pragma unroll
            for (int e = 0; e < 8; ++e)
                x[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ra, cc + e < n ? (unsigned)((16 * rt + l16) * n + cc + e) * 4u : kOut, 0, 0));
#pragma unroll
            for (int pr = 0; pr < 4; ++pr) cut2(x[2 * pr], x[2 * pr + 1], at[i], pr);
            if (!SHARED) __builtin_amdgcn_sched_barrier(0);     // one group of loads at a time: all of them would spill
        }
        const int cc = opaque + col0 + 32 * w + 16 * half + l16;
#pragma unroll
        for (int i = 0; i < (for_wta ? RT : 0); ++i) {      // columns by lane: 8 rows of one of the wave's two tiles
            float x[8];
#pragma unroll
            for (int e = 0; e < 8; ++e)
                x[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ra, cc < n ? (unsigned)((16 * i + 8 * hr + e) * n + cc) * 4u : kOut, 0, 0));
            u32x4 p[3];
#pragma unroll
            for (int pr = 0; pr < 4; ++pr) cut2(x[2 * pr], x[2 * pr + 1], p, pr);
            u32x4 *dst = Ap + ((w * 2 + half) * RT + i) * 96;
#pragma unroll
            for (int q = 0; q < 3; ++q) dst[(q * 2 + hr) * 16 + l16] = p[q];
            if (!SHARED) __builtin_amdgcn_sched_barrier(0);
        }
    };
    // a row of W in LDS: the float and its pieces
    auto put_w = [&](int row, int f, float x) {
        Ws[row * LD + f] = x;
        unsigned h, mm, l;
        split3(x, h, mm, l);
        unsigned short *dst = Wp + ((row >> 3) * 16 + f) * 8 + (row & 7);
        dst[0] = (unsigned short)(h >> 16);
        dst[RT * 256] = (unsigned short)(mm >> 16);
        dst[2 * RT * 256] = (unsigned short)(l >> 16);
    };
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(a.wx, 0, R * RB * 64, kRsrcFlags);
    const __amdgpu_buffer_rsrc_t rh = __builtin_amdgcn_make_buffer_rsrc(a.hx, 0, nt * 1024, kRsrcFlags);
    // the rows of row group r: as handed in, or as exchanged
    auto load_w = [&](int r, bool handed_in) {
        float x[NE];
#pragma unroll
        for (int i = 0; i < NE; ++i) {
            const int e = tid + 512 * i, row = e >> 4, f = e & 15;
            const int64_t grow = (int64_t)r * RB + row;
            if (handed_in) x[i] = row < RB && grow < a.m && f < k ? a.Win[grow * k + f] : 0.f;
            else x[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rw, row < RB ? (unsigned)(r * RB * 16 + e) * 4u : kOut, 0, kExchange));
        }
#pragma unroll
        for (int i = 0; i < NE; ++i) {
            const int e = tid + 512 * i;
            if (e < RT * 256) put_w(e >> 4, e & 15, x[i]);
        }
    };
    // The Gram matrix of either update, up to 8 factors in two floats an entry: an entry's rounding is the same in all
    // rows or columns and, near a fixed point, in all iterations, so that the factors' scale drifts by it (256 x 192,
    // k = 4, 100 iterations, median of 48 inputs: 4.2e-7 off with one float, 3.6 with two, 3.7 on the one-pass plan;
    // 1000 x 300, k = 12, 50 iterations: 3.5, 3.4, 3.7).
    auto put_g = [&](double x) {
        const float hi = (float)x;
        Gs[er * LD + ec] = hi;
        Gl[er * LD + ec] = fabsf(hi) < __builtin_inff() ? (float)(x - (double)hi) : 0.f;     // an infinite denominator stays one
    };
    auto dot = [&](const float *x, int row) -> float {     // x . row of the Gram matrix
        const float *gh = Gs + row * LD, *gl = Gl + row * LD;
        float s0 = 0.f, s1 = 0.f, l = 0.f;
        auto four = [&](int d) {
            const f32x4 u = *reinterpret_cast<const f32x4 *>(x + d), v = *reinterpret_cast<const f32x4 *>(gh + d);
            s0 += u.x * v.x;
            s1 += u.y * v.y;
            s0 += u.z * v.z;
            s1 += u.w * v.w;
        };
        auto rest = [&](int d) {
            const f32x4 u = *reinterpret_cast<const f32x4 *>(x + d), v = *reinterpret_cast<const f32x4 *>(gl + d);
            l += u.x * v.x + u.y * v.y + u.z * v.z + u.w * v.w;
        };
        if (k <= 8) {
            four(0), rest(0);
            four(4), rest(4);
        } else {
            four(0), four(4), four(8), four(12);
        }
        return (s0 + s1) + l;
    };
    // new entry of W; with the last update also to the caller's W and the objective's terms
    auto update_w = [&](int r, int row, int f, float num, bool last, double &dacc) -> float {
        const int64_t grow = (int64_t)r * RB + row;
        if (grow >= a.m || f >= k) return 0.f;
        const float x = Ws[row * LD + f] * num / (dot(Ws + row * LD, f) + a.eps);   // H H^T is symmetric
        if (last) put_through(a.W + grow * k + f, x);
        dacc += (double)num * (double)x;
        return x;
    };
    // what the last update of W, or every one (lead = 0), leaves for the objective
    auto report = [&](int v, double dacc) {
        const int u = EVERY ? s - 1 : 0;
        for (int off = 32; off > 0; off >>= 1) dacc += __shfl_xor(dacc, off);
        __syncthreads();
        if (lane == 0) dsum[w] = dacc;
        __syncthreads();
        if (tid == 0) {
            double t = 0.0;
            for (int i = 0; i < 8; ++i) t += dsum[i];
            a.dpart[u * nwg + v] = t;
        }
        if (v == 0 && tid < 256 && er < k && ec < k) a.gh[(u * k + er) * k + ec] = Gs[er * LD + ec];
    };

    bool have_tile = false;
    for (; s <= a.nprod; ++s) {
        place();
        epoch = 8 * s;                 // more than an iteration's meetings
        if (s == 0) {
            for (int v = v0; v < v1; v += step)      // H as handed in, to where its owners look for it
                for (int t = v / C; t < 16; t += R) {
                    const int tile = 16 * (v % C) + t, col = 16 * tile + ec;
                    if (tid < 256)
                        __builtin_amdgcn_raw_buffer_store_b32(er < k && col < n ? __float_as_uint(a.Hin[(int64_t)er * n + col]) : 0u, rh,
                                                              (unsigned)((2 * tile + (ec >> 3)) * 128 + er * 8 + (ec & 7)) * 4u, 0, kExchange);
                }
            if (a.lead) meet(true);
        }
        const bool stored = s > 1 || (s == 1 && a.lead);     // wx holds the rows
        const bool product = s < a.nprod, update = s ? (product || a.trail) : a.lead;
        if (!product && !update) break;
        const bool last_w = update && (!product || (s == a.nprod - 1 && !a.trail));
        const bool last_h = s == a.nprod - 1;
        if (update) {
            // ---- A H^T
            for (int v = v0; v < v1; v += step) {
                const int r = v / C, c = v % C;
                if (SHARED) __syncthreads();
                if (SHARED || !have_tile) {
                    load_tile(r, c, true, !SHARED);
                    load_w(r, !stored);
                }
                // thread tid: group tid / 16 of 8 columns, factor tid % 16; the floats are its wave's operand of H H^T
                const unsigned off = (tid & 15) < k ? (unsigned)(c * 4096 + tid * 8) * 4u : kOut;
                const u32x4 x0 = __builtin_amdgcn_raw_buffer_load_b128(rh, off, 0, kExchange);
                const u32x4 x1 = __builtin_amdgcn_raw_buffer_load_b128(rh, off + 16, 0, kExchange);
                {
                    u32x4 p[3];
                    cut2(__uint_as_float(x0.x), __uint_as_float(x0.y), p, 0);
                    cut2(__uint_as_float(x0.z), __uint_as_float(x0.w), p, 1);
                    cut2(__uint_as_float(x1.x), __uint_as_float(x1.y), p, 2);
                    cut2(__uint_as_float(x1.z), __uint_as_float(x1.w), p, 3);
#pragma unroll
                    for (int q = 0; q < 3; ++q) Hp[q * 512 + tid] = p[q];
                }
                __syncthreads();
                f32x4 q[2], g = {0.f, 0.f, 0.f, 0.f};
                q[0] = q[1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int i = 0; i < RT; ++i) {
                    u32x4 b[3];
#pragma unroll
                    for (int p = 0; p < 3; ++p) b[p] = Hp[p * 512 + (4 * (w % CW + CW * i) + quad) * 16 + l16];
#pragma unroll
                    for (int e = 0; e < 6; ++e) q[e / 5] = mfma_bf16_16(at[i][PA[e]], b[PB[e]], q[e / 5]);
                }
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float x = __uint_as_float(e < 4 ? x0[e & 3] : x1[e & 3]);
                    g = __builtin_amdgcn_mfma_f32_16x16x4f32(x, x, g, 0, 0, 0);
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    Qs[w * 256 + (4 * quad + i) * 16 + l16] = q[0][i] + q[1][i];
                    Gq[w * 256 + (4 * quad + i) * 16 + l16] = g[i];
                }
                __syncthreads();
                float num[NE];
                double gsum = 0.0;
#pragma unroll
                for (int i = 0; i < NE; ++i) {
                    const int e = tid + 512 * i;
                    float t[CW];
#pragma unroll
                    for (int u = 0; u < CW; ++u) t[u] = e < RT * 256 ? Qs[((e >> 8) * CW + u) * 256 + (e & 255)] : 0.f;
                    num[i] = tree_sum(t);
                }
                if (RT > 1 ? tid < 256 : tid >= 256) {      // one row tile: the threads without an entry of it
#pragma unroll
                    for (int u = 0; u < 8; ++u) gsum += (double)Gq[u * 256 + (tid & 255)];
                }
                const bool has_g = RT > 1 ? tid < 256 : tid >= 256;
                if (C == 1) {
                    if (has_g) put_g(gsum);
                    __syncthreads();
                    double dacc = 0.0;
                    float x[NE];
#pragma unroll
                    for (int i = 0; i < NE; ++i) {
                        const int e = tid + 512 * i;
                        x[i] = e < RT * 256 ? update_w(r, e >> 4, e & 15, num[i], last_w, dacc) : 0.f;
                    }
                    __syncthreads();
#pragma unroll
                    for (int i = 0; i < NE; ++i) {
                        const int e = tid + 512 * i;
                        if (e < RT * 256) {
                            put_w(e >> 4, e & 15, x[i]);
                            if (SHARED) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x[i]), rw, (unsigned)(r * RB * 16 + e) * 4u, 0, kExchange);
                        }
                    }
                    if (a.dpart && (last_w || EVERY)) report(v, dacc);
                } else {
                    const __amdgpu_buffer_rsrc_t rq = __builtin_amdgcn_make_buffer_rsrc(a.qpart + (int64_t)v * kQRec, 0, kQRec * 4, kRsrcFlags);
#pragma unroll
                    for (int i = 0; i < NE; ++i)
                        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(num[i]), rq, tid + 512 * i < RT * 256 ? (unsigned)(tid + 512 * i) * 4u : kOut, 0, kExchange);
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint((float)gsum), rq, has_g ? (unsigned)(RT * 256 + (tid & 255)) * 4u : kOut, 0, kExchange);
                }
            }
            if (C > 1) {
                meet(false);
                // ---- W update: the 16-row tiles dealt to the workgroups of the row group
                for (int v = v0; v < v1; v += step) {
                    const int r = v / C, c = v % C;
                    if (SHARED) {
                        __syncthreads();
                        load_w(r, !stored);
                    }
                    const __amdgpu_buffer_rsrc_t rq = __builtin_amdgcn_make_buffer_rsrc(a.qpart + (int64_t)r * C * kQRec, 0, C * kQRec * 4, kRsrcFlags);
                    // first tile of this workgroup: threads 0 .. 255, H H^T: the others; shares in batches of 8
                    const int t = c;
                    float sum = 0.f;
                    double gsum = 0.0;
                    unsigned qo = tid >= 256 ? (unsigned)(RT * 256 + tid - 256) * 4u : t < RT ? (unsigned)(t * 256 + tid) * 4u : kOut;
                    for (int b = 0; b < C; b += 8) {
                        float x[8];
#pragma unroll
                        for (int u = 0; u < 8; ++u)
                            x[u] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rq, qo + (unsigned)((b + u) * kQRec) * 4u, 0, kExchange));
                        if (tid >= 256) {
#pragma unroll
                            for (int u = 0; u < 8; ++u) gsum += (double)x[u];
                        }
                        sum += tree_sum(x);
                    }
                    if (tid >= 256) put_g(gsum);
                    __syncthreads();
                    double dacc = 0.0;
                    for (int tt = t; tt < RT; tt += C) {
                        if (tt != t && tid < 256) {
                            sum = 0.f;
                            for (int u = 0; u < C; ++u)
                                sum += __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rq, (unsigned)(u * kQRec + tt * 256 + tid) * 4u, 0, kExchange));
                        }
                        if (tid < 256) {
                            const float x = update_w(r, 16 * tt + er, ec, sum, last_w, dacc);
                            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x), rw, (unsigned)((r * RB + 16 * tt) * 16 + tid) * 4u, 0, kExchange);
                        }
                    }
                    if (a.dpart && (last_w || EVERY)) report(v, dacc);
                }
                if (product || a.gout) meet(false);
            }
        }
        if (!product && !a.gout) break;
        // ---- product
        for (int v = v0; v < v1; v += step) {
            const int r = v / C, c = v % C;
            if (SHARED) {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // the rows of an update that did not wait for others
                __syncthreads();
            }
            if (SHARED || !have_tile) {
                if (SHARED || !update) load_tile(r, c, !SHARED, true);
                if (SHARED || !update) load_w(r, !(stored || update));
            }
            if (!SHARED && update && C > 1) load_w(r, false);
            __syncthreads();
            if (product) {
                f32x4 d[2][2];         // [tile][small products, large ones]
#pragma unroll
                for (int t = 0; t < 2; ++t) d[t][0] = d[t][1] = f32x4{0.f, 0.f, 0.f, 0.f};
                const u32x4 *wsrc = reinterpret_cast<const u32x4 *>(Wp);
                const int p0 = half ? 1 : 2, p1 = half ? 1 : 0;
#pragma unroll
                for (int i = 0; i < RT; ++i) {
                    u32x4 wf[3];
                    wf[0] = wsrc[(p0 * 2 * RT + 2 * i + hr) * 16 + l16];    // l | m   against h | m
                    wf[1] = wsrc[(p1 * 2 * RT + 2 * i + hr) * 16 + l16];    // h | m           l | h
                    wf[2] = wsrc[(2 * i + hr) * 16 + l16];                  // h | h           m | h
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        const u32x4 *src = Ap + ((w * 2 + t) * RT + i) * 96;
                        u32x4 af[3];
                        af[0] = src[((half ? 1 : 0) * 2 + hr) * 16 + l16];
                        af[1] = src[((half ? 0 : 2) * 2 + hr) * 16 + l16];
                        af[2] = src[((half ? 0 : 1) * 2 + hr) * 16 + l16];
#pragma unroll
                        for (int e = 0; e < 3; ++e) d[t][e / 2] = mfma_bf16_16(af[e], wf[e], d[t][e / 2]);
                    }
                }
                const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(a.part + (int64_t)v * kPRec, 0, kPRec * 4, kRsrcFlags);
                const unsigned off = l16 < k ? (unsigned)(l16 * 16 + 4 * quad) * 4u + (unsigned)w * 2048u : kOut;
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, d[t][0] + d[t][1]), rp, off + t * 1024u, 0, kExchange);
            }
            if (w == 7) {              // the rows' W^T W
                f32x4 d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int i = 0; i < 4 * RT; ++i) {
                    const float x = Ws[(4 * i + quad) * LD + l16];
                    d = __builtin_amdgcn_mfma_f32_16x16x4f32(x, x, d, 0, 0, 0);
                }
                if (product) {
                    const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(a.part + (int64_t)v * kPRec, 0, kPRec * 4, kRsrcFlags);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {      // the lower triangle
                        const int row = 4 * quad + i;
                        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(d[i]), rp, row >= l16 && row < k ? (unsigned)(4096 + row * (row + 1) / 2 + l16) * 4u : kOut, 0, kExchange);
                    }
                }
                if (last_w && a.gout && c == 0) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int row = 4 * quad + i;
                        a.gout[(int64_t)r * 1024 + ((row & 3) + 4 * (row >> 3)) * 64 + l16 + 32 * ((row >> 2) & 1)] = d[i];
                    }
                }
            }
        }
        have_tile = true;
        if (!product) break;
        meet(true);
        // ---- H update: the 16-column tiles dealt to the workgroups of the column group
        for (int v = v0; v < v1; v += step) {
            const int r = v / C, c = v % C;
            for (int t = r; t < 16 && 16 * c + t < nt; t += R) {
                const int tile = 16 * c + t, col = 16 * tile + ec;
                const unsigned hoff = (unsigned)((2 * tile + (ec >> 3)) * 128 + er * 8 + (ec & 7)) * 4u;
                const float hold = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rh, tid < 256 ? hoff : kOut, 0, kExchange));
                constexpr int B = 8;
                const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(a.part + (int64_t)c * kPRec, 0, ((R - 1) * C + 1) * kPRec * 4, kRsrcFlags);
                f32x4 ps = {0.f, 0.f, 0.f, 0.f}, gs = {0.f, 0.f, 0.f, 0.f};
                for (int g0 = w; g0 < R; g0 += 8 * B) {
                    u32x4 p[B], gg[B];
                    unsigned pstep = (unsigned)(8 * C * kPRec) * 4u, po = (unsigned)(g0 * C * kPRec) * 4u, go = po;
                    po = l16 < k ? po + (unsigned)(t * 256 + l16 * 16 + 4 * quad) * 4u : kOut;
                    go = 8 * lane < k * (k + 1) ? go + (unsigned)(4096 + 4 * lane) * 4u : kOut;
                    asm volatile("" : "+v"(po), "+v"(go), "+s"(pstep));
#pragma unroll
                    for (int i = 0; i < B; ++i) {
                        p[i] = gg[i] = u32x4{0u, 0u, 0u, 0u};
                        if (g0 + 8 * i < R) {
                            p[i] = __builtin_amdgcn_raw_buffer_load_b128(rp, po + i * pstep, 0, kExchange);
                            gg[i] = __builtin_amdgcn_raw_buffer_load_b128(rp, go + i * pstep, 0, kExchange);
                        }
                    }
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        float x[B], y[B];
#pragma unroll
                        for (int i = 0; i < B; ++i) x[i] = __uint_as_float(p[i][j]), y[i] = __uint_as_float(gg[i][j]);
                        ps[j] += tree_sum(x);
                        gs[j] += tree_sum(y);
                    }
                }
                __syncthreads();       // the last readers of these
                *reinterpret_cast<f32x4 *>(Qs + w * 256 + l16 * 16 + 4 * quad) = ps;
                *reinterpret_cast<f32x4 *>(Gq + w * 256 + lane * 4) = gs;
                if (tid < 256) Hs[ec * LD + er] = hold;
                __syncthreads();
                float sum = 0.f;
                if (tid < 256) {
                    float x[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) x[i] = Qs[i * 256 + tid];
                    sum = tree_sum(x);
                } else {
                    const int hi = er > ec ? er : ec, lo = er > ec ? ec : er;
                    double x = 0.0;
#pragma unroll
                    for (int i = 0; i < 8; ++i) x += (double)Gq[i * 256 + hi * (hi + 1) / 2 + lo];
                    put_g(hi < k ? x : 0.0);
                    if (EVERY && s > 0 && v == 0 && t == 0 && hi < k) a.gw[((s - 1) * k + er) * k + ec] = (float)x;
                }
                __syncthreads();
                if (tid < 256) {
                    const float den = dot(Hs + ec * LD, er);
                    const float h = er < k && col < n ? hold * sum / (den + a.eps) : 0.f;
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(h), rh, hoff, 0, kExchange);
                    if (last_h && er < k && col < n) put_through(a.H + (int64_t)er * n + col, h);
                }
            }
        }
        if (last_h && !a.trail) break;
        meet(true);
        if (SHARED) {
            if (tid == 0) {
                const unsigned next = (unsigned)(s + 2) << 9;
                unsigned now;
                if (ticket == 0) {
                    now = next | resident_here(a, nwg);
                    post(a.sync + kResidentDeal, now);
                } else {
                    thread.await(a.sync + kResidentDeal, next);
                    now = peek(a.sync + kResidentDeal);
                }
                word[0] = now >> 9 == next >> 9 && (now & 511) > ticket ? now : deal;      // else a lost run
            }
            __syncthreads();
            deal = __builtin_amdgcn_readfirstlane(word[0]);
            step = deal & 511;
            if (step >= nwg) return s + 1;
        }
    }
    if (SHARED && ticket == 0 && tid == 0) post(a.sync + kResidentDeal, kResidentOver);
    return -1;
}

template <int RT, bool EVERY>
__global__ __launch_bounds__(512, 2) void resident_kernel(const ResidentArgs a)
{
    unsigned *word = reinterpret_cast<unsigned *>(aht_rows_lds);
    if (threadIdx.x == 0) {
        const unsigned ticket = add_one(a.sync + kResidentHere);
        if (ticket == gridDim.x - 1) decide(a.sync + kResidentDeal, 1u << 9 | gridDim.x);
        const long long end = wall_clock64() + a.patience;
        unsigned deal;
        // the low nine bits: how many of those that have reported in are at work; the others: from which iteration on, plus one
        for (unsigned looks = 1; ((deal = peek(a.sync + kResidentDeal)) & 511) <= ticket; ++looks) {
            if (ticket == 0 && (long long)wall_clock64() >= end) decide(a.sync + kResidentDeal, 1u << 9 | resident_here(a, gridDim.x));
            __builtin_amdgcn_s_sleep(1);
            if (looks >= a.polls) {
                post(a.sync + kResidentLost, 1u);
                deal = kResidentOver;
                break;
            }
        }
        word[0] = deal;
        word[1] = ticket;
    }
    __syncthreads();
    const unsigned deal = __builtin_amdgcn_readfirstlane(word[0]), ticket = __builtin_amdgcn_readfirstlane(word[1]);
    __syncthreads();
    if (deal != kResidentOver) {
        int s = (int)(deal >> 9) - 1;      // beyond the last iteration, if it is not this run's deal: nothing is done
        if (s >= 0 && (int)(deal & 511) < a.R * a.C) s = resident_iterations<RT, EVERY, true>(a, s, ticket, deal);
        if (s >= 0) resident_iterations<RT, EVERY, false>(a, s, 0u, 0u);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // what this workgroup has stored, marks among it
    __syncthreads();
    if (threadIdx.x == 0 && add_one(a.sync + kResidentOut) == gridDim.x - 1 && peek(a.sync + kResidentLost)) {
        put_through(a.W, __builtin_nanf(""));
        put_through(a.H, __builtin_nanf(""));
    }
}


// G (k x k, ld k) = sum over nb sets of partial 32 x 32 tiles (accumulator layout).
// Eight lanes share one entry: lane q adds sets q, q+8, ..., a batch of 16 at a time, then the
// eight sums are combined in a fixed tree, so the result does not depend on timing.
__device__ __forceinline__ void gram_sum(const float *__restrict__ gpart, int nb, int k, float *__restrict__ G, int block)
{
    const int kt = (k + 31) >> 5;
    const int64_t stride = (int64_t)kt * kt * 1024;
    const int gid = block * 256 + threadIdx.x;
    const int entry = gid >> 3, q = gid & 7;
    const bool ok = entry < kt * kt * 1024;
    const float *src = gpart + (ok ? entry : 0);
    float s = 0.f;
    // 16 sets of the lane requested together (256 sets: two trips to L2 instead of eight)
    for (int b = q; b < nb; b += 128) {
        float t[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) t[u] = src[(b + 8 * u < nb ? b + 8 * u : 0) * stride];
#pragma unroll
        for (int u = 0; u < 16; ++u) t[u] = b + 8 * u < nb ? t[u] : 0.f;
        s += tree_sum(t);
    }
    s += __shfl_xor(s, 1, 8);
    s += __shfl_xor(s, 2, 8);
    s += __shfl_xor(s, 4, 8);
    if (ok && q == 0) {
        const int tile = entry >> 10, e = entry & 1023;
        const int v = e >> 6, l = e & 63;
        const int r1 = 32 * (tile / kt) + acc_row(v, l >> 5), r2 = 32 * (tile % kt) + (l & 31);
        if (r1 < k && r2 < k) G[r1 * k + r2] = s;
    }
}
__global__ __launch_bounds__(256) void gram_sum_kernel(const float *__restrict__ gpart, int nb, int k,
                                                       float *__restrict__ G)
{
    gram_sum(gpart, nb, k, G, blockIdx.x);
}

// The shares of W^T A that the workgroups of a one-pass launch leave (nb of count4 x 4 floats), added up to kShareGroups
// for the H update, and beside them the sum of their Gram tile sets.  The H update alone, 16 or 32 columns a workgroup,
// has 10 to 32 of them for the 8 MiB of 256 shares: 17.5 us at k = 16, n = 512.
__global__ __launch_bounds__(256) void share_sum_kernel(const float *__restrict__ ppart, int nb, int count4, f32x4 *__restrict__ psum,
                                                        int pblocks, const float *__restrict__ gpart, int k, float *__restrict__ G)
{
    if ((int)blockIdx.x >= pblocks) {
        gram_sum(gpart, nb, k, G, (int)blockIdx.x - pblocks);
        return;
    }
    const int t = blockIdx.x * 256 + threadIdx.x, e = t % count4, g = t / count4;
    if (g >= kShareGroups) return;
    const int per = (nb + kShareGroups - 1) / kShareGroups, s0 = g * per, s1 = s0 + per < nb ? s0 + per : nb;
    const f32x4 *src = reinterpret_cast<const f32x4 *>(ppart) + e;
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
    for (int b = s0; b < s1; b += 16) {
        f32x4 x[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) x[u] = src[(int64_t)(b + u < s1 ? b + u : s0) * count4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            float y[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) y[u] = b + u < s1 ? x[u][j] : 0.f;
            sum[j] += tree_sum(y);
        }
    }
    psum[(int64_t)g * count4 + e] = sum;
}

// ---------------------------------------------------------------------------
// Objective ||A - W H||_F^2 in row tiles of W (the tiling of the paper's
// section 3.2 for its convergence check: W H is produced tile by tile and never
// stored).  Workgroup = 32 rows of A and W, 4 waves; a wave takes 128-column
// slabs w, w+4, ...  Per slab: X = W_tile H[:, slab] by MFMA (A_op = W tile
// from LDS, B_op = H elements, reduction over two factor indices per
// instruction; column tile q holds columns j0 + 4 jj + q), then A is loaded in
// the accumulator layout (16-byte loads, 512 contiguous bytes per row) and
// (a - x)^2 is summed.  One double per workgroup goes to `partial`.
// ---------------------------------------------------------------------------
template <int KT, bool VEC>
__global__ __launch_bounds__(256) void residual_kernel(const float *__restrict__ A,
                                                       const float *__restrict__ W,
                                                       const float *__restrict__ H, int64_t m,
                                                       int64_t n, int k, double *__restrict__ partial)
{
    constexpr int KP = 32 * KT, LDW = KP + 1;
    __shared__ float Ws[32 * LDW];
    __shared__ double wsum[4];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int jj = lane & 31, half = lane >> 5;
    const int64_t i0 = (int64_t)blockIdx.x * 32;
    for (int e = tid; e < 32 * KP; e += 256) {
        const int i = e / KP, c = e % KP;
        Ws[i * LDW + c] = (i0 + i < m && c < k) ? W[(i0 + i) * k + c] : 0.f;
    }
    __syncthreads();
    const int kpairs = (k + 1) >> 1;
    float local = 0.f;
    double total = 0.0;
    const int64_t nslabs = (n + 127) >> 7;
    for (int64_t sl = w; sl < nslabs; sl += 4) {
        const int64_t col = sl * 128 + 4 * jj;
        f32x16 acc[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[q] = f32x16{0};
        for (int s = 0; s < kpairs; ++s) {
            const int c = 2 * s + half;
            const float a = Ws[jj * LDW + c];                 // c <= KP - 1 always; zero beyond k
            const f32x4 h = load4<VEC>(H, n, c, col, c < k);
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[q] = mfma32(a, h[q], acc[q]);
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int64_t row = i0 + acc_row(v, half);
            const f32x4 a = load4<VEC>(A, n, row, col, row < m);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const bool in = row < m && col + q < n;
                const float d = in ? a[q] - acc[q][v] : 0.f;
                local += d * d;
            }
        }
        total += (double)local;     // fp32 within a slab (2048 terms per lane), double across slabs
        local = 0.f;
    }
    for (int off = 32; off > 0; off >>= 1) total += __shfl_xor(total, off);
    if (lane == 0) wsum[w] = total;
    __syncthreads();
    if (tid == 0) partial[blockIdx.x] = (wsum[0] + wsum[1]) + (wsum[2] + wsum[3]);
}

// ---------------------------------------------------------------------------
// The same objective as a streaming pass for k = 16 or 32, 16-byte aligned A, W and H,
// n % 4 == 0 and m % 32 == 0 (the launcher gives the rows left over to the general kernel):
// the geometry and the pieces of the W^T A pass, turned round (both operands cut with rounding): here the
// 32 x 32 tile of an instruction is rows of A by columns of A and the reduction runs over the
// factor index.  Workgroup = 4 waves on 256 consecutive columns and one row split; a wave
// owns 64 of the columns and walks down all the rows of the split, a lane 2 consecutive
// columns.  Once per wave its slab of H is cut into bf16 pieces (B_op: lane l holds factors
// 8 (l / 32) .. + 7 of 16 for column l % 32), kept in registers for every row tile.  Per
// 32-row tile a wave forms the two 32 x 32 tiles of A - W H with 6 instructions per 16 factors
// each from pieces of the rows of -W (A_op: lane l holds 8 consecutive factors of row l % 32) that
// the workgroup makes once for its four waves (wave w cuts tile w of every group of
// four tiles into LDS, double buffered, one barrier per group), and the
// tile of A, loaded in the accumulator layout (lane l, register v: row (v % 4) + 4 (l / 32) +
// 8 (v / 4), its 2 columns: 8-byte loads, 1 KiB contiguous per row over the workgroup).  The
// accumulators start as A and take the largest products first, so that near a good fit they are
// small when the small products come and lose little of them: with W H summed up and subtracted
// afterwards the objective of a fit to 1e-4 was 1.4e-5 (k = 32) to 2.6e-5 (k = 16) too large, now
// 6e-7, as at other ranks (residual_stream_f32_kernel: 4e-7 to 1.2e-6), in the same time.  The
// next tile of A is requested before the current tile's arithmetic, the rows of W two groups
// ahead.  One double per workgroup.  On the 32768 x 16384, k = 32 case the kernel takes
// 0.37 ms on random operands and 0.31 ms, the time of its loads alone, on all-zero ones:
// what is left is the chip's power limit under matrix work and streaming together.
// ---------------------------------------------------------------------------
template <int KSTEPS>
__global__ __launch_bounds__(256, 2) void residual_stream_kernel(const float *__restrict__ A,
                                                                 const float *__restrict__ W,
                                                                 const float *__restrict__ H, int64_t m,
                                                                 int64_t n, int64_t rps,
                                                                 double *__restrict__ partial)
{
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    constexpr int k = 16 * KSTEPS;
    __shared__ double wsum[4];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int jj = lane & 31, half = lane >> 5;
    const int64_t jw = (int64_t)blockIdx.x * 256 + 64 * w;   // this wave's 64 columns
    const int64_t col = jw + 2 * jj;
    const bool colok = col < n;                       // n is even: both columns or none
    const int64_t j0 = jw < n ? jw : 0;               // a wave wholly past column n fetches the first slab
    const int64_t r0 = (int64_t)blockIdx.y * rps;     // rps % 32 == 0
    const int64_t r1 = (r0 + rps < m) ? r0 + rps : m;

    // B_op pieces of the slab of H: hp[s][q][piece]
    u32x4 hp[KSTEPS][2][3];
#pragma unroll
    for (int s = 0; s < KSTEPS; ++s) {
        f32x2 hv[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int c = 16 * s + 8 * half + r;
            const f32x2 t = *reinterpret_cast<const f32x2 *>(H + (colok ? (int64_t)c * n + col : 0));
            hv[r].x = colok ? t.x : 0.f;
            hv[r].y = colok ? t.y : 0.f;
        }
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int pr = 0; pr < 4; ++pr) {
                cut2(hv[2 * pr][q], hv[2 * pr + 1][q], hp[s][q], pr);
            }
    }

    // Requests only: nothing below reads a loaded value before the products of the previous
    // tile are issued, so the loads stay in flight.  m % 32 == 0 and rps % 32 == 0: every tile
    // is whole; a request past the split fetches tile 0 instead and is never used.
    // this lane's row of W for tile i0: 8 consecutive factors per 16-factor step
    f32x4 wv[KSTEPS][2];
    auto load_w = [&](int64_t i0) {
        const float *src = W + ((i0 < r1 ? i0 : 0) + jj) * k + 8 * half;
#pragma unroll
        for (int s = 0; s < KSTEPS; ++s) {
            wv[s][0] = *reinterpret_cast<const f32x4 *>(src + 16 * s);
            wv[s][1] = *reinterpret_cast<const f32x4 *>(src + 16 * s + 4);
        }
    };
    // A in the accumulator layout: wave-uniform row address plus one 32-bit lane offset
    // (4 n + 62 < 2^32); lanes past column n fetch the slab's first columns
    typedef f32x2 ATile[16];
    const unsigned lane_off = colok ? (unsigned)(4 * half) * (unsigned)n + 2u * jj : 0u;
    auto load_a = [&](ATile &a, int64_t i0) {
        const float *tp = A + (i0 < r1 ? i0 : 0) * n + j0;
#pragma unroll
        for (int v = 0; v < 16; ++v)
            a[v] = __builtin_nontemporal_load(reinterpret_cast<const f32x2 *>(tp + (int64_t)((v & 3) + 8 * (v >> 2)) * n + lane_off));
    };

    double total = 0.0;
    // The four waves walk the same row tiles, so the pieces of a tile of W are made once per
    // workgroup: of every group of four tiles wave w cuts tile w and stores it in LDS in
    // operand order (entry [tile][step * 3 + piece][lane], 16 bytes each), while the group
    // before it is consumed from the other buffer; one barrier per group.
    __shared__ u32x4 wlds[2][4][KSTEPS * 3][64];
    auto cut_store = [&](int buf) {
#pragma unroll
        for (int s = 0; s < KSTEPS; ++s) {
            u32x4 wp[3];
#pragma unroll
            for (int pr = 0; pr < 4; ++pr) {
                cut2(wv[s][pr >> 1][(2 * pr) & 3], wv[s][pr >> 1][(2 * pr + 1) & 3], wp, pr);
            }
#pragma unroll
            for (int pc = 0; pc < 3; ++pc) wlds[buf][w][s * 3 + pc][lane] = wp[pc] ^ 0x80008000u;
        }
    };
    // one tile, its A already requested: pieces of -W from LDS, products, squares.  The two
    // 32-column halves are two chains of 6 KSTEPS instructions one after the other, so the
    // squares of the first half can issue under the products of the second.
    auto tile = [&](const ATile &a, int buf, int t, bool valid) {
        u32x4 wp[KSTEPS][3];
#pragma unroll
        for (int s = 0; s < KSTEPS; ++s)
#pragma unroll
            for (int pc = 0; pc < 3; ++pc) wp[s][pc] = wlds[buf][t][s * 3 + pc][lane];
        f32x16 acc[2];
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[0][v] = a[v].x, acc[1][v] = a[v].y;
        constexpr int PW[6] = {0, 0, 1, 1, 0, 2}, PH[6] = {0, 1, 0, 1, 2, 0};   // largest first
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int e = 0; e < 6; ++e)
#pragma unroll
                for (int s = 0; s < KSTEPS; ++s) acc[q] = mfma_bf16(wp[s][PW[e]], hp[s][q][PH[e]], acc[q]);
        float local = 0.f;      // 32 terms per lane in fp32, double across tiles
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            local += acc[0][v] * acc[0][v];
            local += acc[1][v] * acc[1][v];
        }
        total += valid ? (double)local : 0.0;
    };
    // four tiles per trip (every wave of the workgroup makes the same trips: r0 and r1 are the
    // workgroup's); a tile past the split is tile 0 again, and its sum is dropped
    ATile a0, a1;
    int64_t i = r0;
    load_w(i + 32 * w);
    cut_store(0);
    load_w(i + 128 + 32 * w);
    load_a(a0, i);
    __syncthreads();
    int buf = 0;
    for (; i < r1; i += 128) {
        cut_store(buf ^ 1);
        load_w(i + 256 + 32 * w);
        load_a(a1, i + 32);
        __builtin_amdgcn_sched_barrier(0);
        tile(a0, buf, 0, true);
        load_a(a0, i + 64);
        __builtin_amdgcn_sched_barrier(0);
        tile(a1, buf, 1, i + 32 < r1);
        load_a(a1, i + 96);
        __builtin_amdgcn_sched_barrier(0);
        tile(a0, buf, 2, i + 64 < r1);
        load_a(a0, i + 128);
        __builtin_amdgcn_sched_barrier(0);
        tile(a1, buf, 3, i + 96 < r1);
        __syncthreads();    // the group's buffer is free, the next group's is written
        buf ^= 1;
    }
    if (!colok) total = 0.0;   // such lanes subtracted a zero product from columns of other lanes
    for (int off = 32; off > 0; off >>= 1) total += __shfl_xor(total, off);
    if (lane == 0) wsum[w] = total;
    __syncthreads();
    if (tid == 0) partial[(int64_t)blockIdx.y * gridDim.x + blockIdx.x] = (wsum[0] + wsum[1]) + (wsum[2] + wsum[3]);
}

// ---------------------------------------------------------------------------
// The objective as a streaming pass for any k <= 2 KS <= 48, 16-byte aligned A and H and
// n % 4 == 0, with the fp32 matrix instruction, which takes two factors per step instead of 16 and
// the floats as they are: no rank is rounded up to 16, and the sums are those of residual_kernel.  The
// geometry of residual_stream_kernel: a wave owns 64 columns and walks down the rows of a split, a
// lane 2 consecutive columns; its slab of H stays in registers, the rows of W go through LDS four
// 32-row tiles at a time, and the next tile of A is requested before the current one's arithmetic.
// Half h of the wave takes factors KS h .. KS h + KS - 1, one per instruction, so that a lane's
// share of a row of W is one contiguous run.  Rows from m on read as zero, of A (outside the
// tile's buffer extent) and of W, and add nothing; a request past the split fetches tile 0 instead
// and is never used.  Against residual_kernel, whose waves wait for H, the products and A of every
// slab in turn: see launch_residual.
// ---------------------------------------------------------------------------
template <int KS>
__global__ __launch_bounds__(256, 2) void residual_stream_f32_kernel(const float *__restrict__ A,
                                                                     const float *__restrict__ W,
                                                                     const float *__restrict__ H, int64_t m,
                                                                     int64_t n, int k, int64_t rps,
                                                                     double *__restrict__ partial)
{
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    constexpr int kRsrcFlags = 0x00020000;   // raw buffer, 32-bit data format (gfx9 family)
    __shared__ double wsum[4];
    __shared__ f32x4 wlds[2][4][KS / 4][64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int jj = lane & 31, half = lane >> 5;
    const int64_t jw = (int64_t)blockIdx.x * 256 + 64 * w;   // this wave's 64 columns
    const int64_t col = jw + 2 * jj;
    const bool colok = col < n;                       // n is even: both columns or none
    const int64_t j0 = jw < n ? jw : 0;               // a wave wholly past column n fetches the first slab
    const int64_t r0 = (int64_t)blockIdx.y * rps;     // rps % 32 == 0
    const int64_t r1 = (r0 + rps < m) ? r0 + rps : m;
    const unsigned rowb = (unsigned)(n * 4);
    const unsigned lane_off = colok ? (unsigned)(4 * half) * rowb + 8u * jj : 0u;

    f32x2 hv[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        const int c = KS * half + s;
        const bool in = colok && c < k;
        const f32x2 t = *reinterpret_cast<const f32x2 *>(H + (in ? (int64_t)c * n + col : 0));
        hv[s].x = in ? t.x : 0.f;
        hv[s].y = in ? t.y : 0.f;
    }

    f32x4 wv[KS / 4];
    bool wok = false;
    auto load_w = [&](int64_t i0) {
        const int64_t row = (i0 < r1 ? i0 : 0) + jj;
        wok = row < m;
        const float *src = W + (wok ? row : 0) * k;
#pragma unroll
        for (int s = 0; s < KS; ++s) wv[s >> 2][s & 3] = src[KS * half + s < k ? KS * half + s : 0];
    };
    auto store_w = [&](int buf) {
#pragma unroll
        for (int s = 0; s < KS; s += 4) {
            f32x4 t;
#pragma unroll
            for (int e = 0; e < 4; ++e) t[e] = wok && KS * half + s + e < k ? wv[s >> 2][e] : 0.f;
            wlds[buf][w][s >> 2][lane] = t;
        }
    };
    typedef f32x2 ATile[16];
    auto load_a = [&](ATile &a, int64_t i0) {
        const int64_t base = i0 < r1 ? i0 : 0;
        const int64_t av = m - base < 32 ? m - base : 32;
        const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float *>(A + base * n + j0), 0, (int)(av * rowb - j0 * 4), kRsrcFlags);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const u32x2 t = __builtin_amdgcn_raw_buffer_load_b64(ra, lane_off + (unsigned)acc_row(v, 0) * rowb, 0, kStreamLoad);
            a[v] = __builtin_bit_cast(f32x2, t);
        }
    };
    double total = 0.0;
    auto tile = [&](const ATile &a, int buf, int t, bool valid) {
        f32x16 acc[2];
        acc[0] = f32x16{0};
        acc[1] = f32x16{0};
#pragma unroll
        for (int s = 0; s < KS; s += 4) {
            const f32x4 x = wlds[buf][t][s >> 2][lane];
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int q = 0; q < 2; ++q) acc[q] = mfma32(x[e], hv[s + e][q], acc[q]);
        }
        float local = 0.f;      // 32 terms per lane in fp32, double across tiles
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const float d0 = a[v].x - acc[0][v], d1 = a[v].y - acc[1][v];
            local += d0 * d0;
            local += d1 * d1;
        }
        total += valid ? (double)local : 0.0;
    };
    // four tiles per trip, as in residual_stream_kernel
    ATile a0, a1;
    int64_t i = r0;
    load_w(i + 32 * w);
    store_w(0);
    load_w(i + 128 + 32 * w);
    load_a(a0, i);
    __syncthreads();
    int buf = 0;
    for (; i < r1; i += 128) {
        store_w(buf ^ 1);
        load_w(i + 256 + 32 * w);
        load_a(a1, i + 32);
        __builtin_amdgcn_sched_barrier(0);
        tile(a0, buf, 0, true);
        load_a(a0, i + 64);
        __builtin_amdgcn_sched_barrier(0);
        tile(a1, buf, 1, i + 32 < r1);
        load_a(a1, i + 96);
        __builtin_amdgcn_sched_barrier(0);
        tile(a0, buf, 2, i + 64 < r1);
        load_a(a0, i + 128);
        __builtin_amdgcn_sched_barrier(0);
        tile(a1, buf, 3, i + 96 < r1);
        __syncthreads();    // the group's buffer is free, the next group's is written
        buf ^= 1;
    }
    if (!colok) total = 0.0;   // such lanes subtracted a zero product from columns of other lanes
    for (int off = 32; off > 0; off >>= 1) total += __shfl_xor(total, off);
    if (lane == 0) wsum[w] = total;
    __syncthreads();
    if (tid == 0) partial[(int64_t)blockIdx.y * gridDim.x + blockIdx.x] = (wsum[0] + wsum[1]) + (wsum[2] + wsum[3]);
}

// ---------------------------------------------------------------------------
// The objective as a streaming pass on pairs of halves, any k <= 16 S <= 64 and any alignment, in the
// geometry of residual_stream_kernel; VEC (16-byte aligned A, n % 4 == 0): a lane's two columns are consecutive, else 32 apart.
// The reduction runs over columns of W and rows of H that may be in units of their own, so each row of H is first brought to
// its largest entry in the workgroup's columns, the power of two going to that column of W.  H is then cut under a scale per column and
// the rows of W under one per row.  Three instructions per 16 factors do the work of eight of the fp32 kernel; the
// large products and the cross products have accumulators of their own and
// are taken from A one after the other, so that near a good fit the second meets a small difference and
// few instructions round at the size of W H (a fit to 1e-4: objective 3e-8 to 2.4e-7 off, residual_stream_f32_kernel
// 5e-9 to 9e-7).  Rows from m on read as zero, of A and of W (outside the tile's buffer extent), and
// add nothing.
// ---------------------------------------------------------------------------
template <int S, bool VEC>
__global__ __launch_bounds__(256, 2) void residual_pair_kernel(const float *__restrict__ A,
                                                                 const float *__restrict__ W,
                                                                 const float *__restrict__ H, int64_t m,
                                                                 int64_t n, int k, int64_t rps,
                                                                 double *__restrict__ partial)
{
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    constexpr int kRsrcFlags = 0x00020000;   // raw buffer, 32-bit data format (gfx9 family)
    __shared__ double wsum[4];
    __shared__ u32x4 wlds[2][4][S * 2][64];  // [tile][step * 2 + piece][lane]
    __shared__ f32x4 wunit[2][4][8];         // 2^(exponent - 14) of the tile's rows
    __shared__ unsigned fmost[4][16 * S];
    __shared__ float funit[2][16 * S];       // the factors' units, and one over them
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int jj = lane & 31, half = lane >> 5;
    const int64_t jw = (int64_t)blockIdx.x * 256 + 64 * w;   // this wave's 64 columns
    const int64_t j0 = jw < n ? jw : 0;               // a wave wholly past column n fetches the first slab
    const int64_t r0 = (int64_t)blockIdx.y * rps;     // rps % 32 == 0
    const int64_t r1 = (r0 + rps < m) ? r0 + rps : m;
    const unsigned rowb = (unsigned)(n * 4);
    bool ok[2];                                       // VEC: n is even, both columns or none
    unsigned off[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int c = VEC ? 2 * jj + q : 32 * q + jj;
        ok[q] = jw + c < n;
        off[q] = ok[q] ? (unsigned)(4 * half) * rowb + 4u * c : 0u;
    }

    float hv[2][S * 8];
#pragma unroll
    for (int s = 0; s < S * 8; ++s) {
        const int c = 16 * (s >> 3) + 8 * half + (s & 7);
        unsigned top = 0;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const bool in = ok[q] && c < k;
            const float t = H[in ? (int64_t)c * n + jw + (VEC ? 2 * jj + q : 32 * q + jj) : 0];
            hv[q][s] = in ? t : 0.f;
            const unsigned x = __float_as_uint(hv[q][s]) & 0x7fffffffu;
            top = x > top ? x : top;
        }
        for (int o = 16; o > 0; o >>= 1) {
            const unsigned x = __shfl_xor(top, o);
            top = x > top ? x : top;
        }
        if (jj == 0) fmost[w][c] = top;
    }
    __syncthreads();
    if (tid < 16 * S) {
        unsigned top = 0;
#pragma unroll
        for (int x = 0; x < 4; ++x) top = fmost[x][tid] > top ? fmost[x][tid] : top;
        const int e = half_exponent(top);
        funit[0][tid] = power_of_two(e < 126 ? e : 126);
        funit[1][tid] = power_of_two(e < 126 ? -e : -126);
    }
    __syncthreads();
    u32x4 hp[S][2][2];
    float unit[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        unsigned top = 0;
#pragma unroll
        for (int s = 0; s < S * 8; ++s) {
            hv[q][s] *= funit[1][16 * (s >> 3) + 8 * half + (s & 7)];
            const unsigned x = __float_as_uint(hv[q][s]) & 0x7fffffffu;
            top = x > top ? x : top;
        }
        const unsigned other = __shfl_xor(top, 32);
        const int e = half_exponent(other > top ? other : top);
        const float sc = power_of_two(14 - e);
        unit[q] = power_of_two(e - 14);
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int pr = 0; pr < 4; ++pr) cut2h(hv[q][8 * s + 2 * pr], hv[q][8 * s + 2 * pr + 1], sc, hp[s][q], pr);
    }

    // Requests only: nothing below reads a loaded value before the products of the previous
    // tile are issued, so the loads stay in flight.
    float wv[S * 8];
    const unsigned woff = (unsigned)(jj * k + 8 * half) * 4u;
    auto load_w = [&](int64_t i0) {
        const int64_t base = i0 < r1 ? i0 : 0;
        const int64_t av = m - base < 32 ? m - base : 32;
        const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(W + base * k), 0, (int)(av * k * 4), kRsrcFlags);
#pragma unroll
        for (int s = 0; s < S * 8; ++s)      // factors from k on are the next row's
            wv[s] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rw, woff + 64u * (s >> 3) + 4u * (s & 7), 0, 0));
    };
    auto store_w = [&](int buf) {
        unsigned top = 0;
#pragma unroll
        for (int s = 0; s < S * 8; ++s) {
            const int c = 16 * (s >> 3) + 8 * half + (s & 7);
            wv[s] = c < k ? wv[s] * funit[0][c] : 0.f;
            const unsigned b = __float_as_uint(wv[s]) & 0x7fffffffu;
            top = b > top ? b : top;
        }
        const unsigned other = __shfl_xor(top, 32);
        const int e = half_exponent(other > top ? other : top);
        const float sc = power_of_two(14 - e);
#pragma unroll
        for (int s = 0; s < S; ++s) {
            u32x4 wp[2];
#pragma unroll
            for (int pr = 0; pr < 4; ++pr) cut2h(wv[8 * s + 2 * pr], wv[8 * s + 2 * pr + 1], sc, wp, pr);
            wlds[buf][w][2 * s][lane] = wp[0];
            wlds[buf][w][2 * s + 1][lane] = wp[1];
        }
        if (half == 0) reinterpret_cast<float *>(wunit[buf][w])[jj] = power_of_two(e - 14);
    };
    typedef f32x2 ATile[16];
    auto load_a = [&](ATile &a, int64_t i0) {
        const int64_t base = i0 < r1 ? i0 : 0;
        const int64_t av = m - base < 32 ? m - base : 32;
        const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float *>(A + base * n + j0), 0, (int)(av * rowb - j0 * 4), kRsrcFlags);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            unsigned row = (unsigned)acc_row(v, 0) * rowb;
            asm volatile("" : "+s"(row));            // sixteen sums kept in registers otherwise
            if (VEC) {
                const u32x2 t = __builtin_amdgcn_raw_buffer_load_b64(ra, off[0] + row, 0, kStreamLoad);
                a[v] = __builtin_bit_cast(f32x2, t);
            } else {
                a[v].x = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ra, off[0] + row, 0, kStreamLoad));
                a[v].y = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ra, off[1] + row, 0, kStreamLoad));
            }
        }
    };
    double total = 0.0;
    // one tile, its A already requested: pairs of W from LDS, products, squares
    auto tile = [&](const ATile &a, int buf, int t, bool valid) {
        f32x4 u[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) u[g] = wunit[buf][t][2 * g + half];
        f32x16 big[2], rest[2];
        auto products = [&](int q) {
            big[q] = f32x16{0}, rest[q] = f32x16{0};
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const u32x4 w0 = wlds[buf][t][2 * s][lane], w1 = wlds[buf][t][2 * s + 1][lane];
                rest[q] = mfma_f16(w1, hp[s][q][0], rest[q]);
                big[q] = mfma_f16(w0, hp[s][q][0], big[q]);
                rest[q] = mfma_f16(w0, hp[s][q][1], rest[q]);
            }
        };
        auto squares = [&](int q) {
            float local = 0.f;      // 16 terms per lane in fp32, double across
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const float p = u[v >> 2][v & 3] * unit[q];
                const float d = __builtin_fmaf(-rest[q][v], p, __builtin_fmaf(-big[q][v], p, a[v][q]));
                local = __builtin_fmaf(d, d, local);
            }
            // not a branch: with one the compiler mixes the tiles' work and spills
            asm volatile("" : "+v"(local));
            total += valid && ok[q] ? (double)local : 0.0;
        };
        products(0);
        if (S > 2) __builtin_amdgcn_sched_barrier(0);
        if (S <= 2) products(1);
        squares(0);
        if (S > 2) {
            __builtin_amdgcn_sched_barrier(0);
            products(1);
        }
        squares(1);
        __builtin_amdgcn_sched_barrier(0);
    };
    // four tiles per trip (every wave of the workgroup makes the same trips: r0 and r1 are the
    // workgroup's); a tile past the split is tile 0 again, and its sum is dropped
    ATile at[2];
    int64_t i = r0;
    load_w(i + 32 * w);
    store_w(0);
    load_w(i + 128 + 32 * w);
    load_a(at[0], i);
    __syncthreads();
    int buf = 0;
    for (; i < r1; i += 128) {
        store_w(buf ^ 1);
        load_w(i + 256 + 32 * w);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            load_a(at[(t + 1) & 1], i + 32 * (t + 1));
            __builtin_amdgcn_sched_barrier(0);
            tile(at[t & 1], buf, t, i + 32 * t < r1);
        }
        __syncthreads();    // the group's buffer is free, the next group's is written
        buf ^= 1;
    }
    auto sum = [&]() {
        for (int off = 32; off > 0; off >>= 1) total += __shfl_xor(total, off);
        if (lane == 0) wsum[w] = total;
        __syncthreads();
        total = (wsum[0] + wsum[1]) + (wsum[2] + wsum[3]);
    };
    sum();
    if (!(total < __builtin_inf())) {
        // An infinity has no two halves, their differences are no number.  What the floats give, a column a thread.
        total = 0.0;
        const int64_t j = (int64_t)blockIdx.x * 256 + tid;
        if (j < n)
#pragma unroll 1
            for (int64_t i = r0; i < r1; ++i) {
                float p = 0.f;
#pragma unroll 4
                for (int c = 0; c < k; ++c) p = __builtin_fmaf(W[i * k + c], H[c * n + j], p);
                const float d = A[i * n + j] - p;
                total += (double)(d * d);
            }
        __syncthreads();      // wsum is read
        sum();
    }
    if (tid == 0) partial[(int64_t)blockIdx.y * gridDim.x + blockIdx.x] = total;
}

// Sum of `count` doubles by one block of 256 threads in a fixed order: thread t adds entries
// t, t + 256, ..., then the lanes of a wave by butterfly and the four waves in order (one thread
// alone needs a dependent load per entry: 33 us for 512 entries, 0.3 ms for 4096).
__device__ __forceinline__ double block_sum_f64(const double *__restrict__ partial, int64_t count)
{
    __shared__ double part[4];
    double s = 0.0;
    for (int64_t i = threadIdx.x; i < count; i += 256) s += partial[i];
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
    __syncthreads();
    return (part[0] + part[1]) + (part[2] + part[3]);
}

// out[0] = sqrt(sum of `count` partials).  One block of 256 threads.
__global__ __launch_bounds__(256) void residual_finish_kernel(const double *__restrict__ partial, int64_t count,
                                                              double *out)
{
    const double s = block_sum_f64(partial, count);
    if (threadIdx.x == 0) out[0] = sqrt(s);
}

// partial[b] = sum of squares of a slice of X (double), for ||A||_F^2.
__global__ __launch_bounds__(256) void sumsq_kernel(const float *__restrict__ X, int64_t count,
                                                    double *__restrict__ partial)
{
    __shared__ double wsum[4];
    double acc = 0.0;
    // eight loads in flight per thread: one at a time, 192 MiB took 65 us
    const int64_t step = (int64_t)gridDim.x * 256;
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < count; e += 8 * step) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = e + u * step < count ? X[e + u * step] : 0.f;
#pragma unroll
        for (int u = 0; u < 8; ++u) acc += (double)v[u] * (double)v[u];
    }
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) partial[blockIdx.x] = (wsum[0] + wsum[1]) + (wsum[2] + wsum[3]);
}

// out[0] = sum of `count` partials.  One block of 256 threads.
__global__ __launch_bounds__(256) void sum_f64_kernel(const double *__restrict__ partial, int64_t count, double *out)
{
    const double s = block_sum_f64(partial, count);
    if (threadIdx.x == 0) out[0] = s;
}

// Objective from quantities the W update leaves behind (the expansion of section 2.1's norm):
// ||A - W H||_F^2 = ||A||_F^2 - 2 <A H^T, W> + <H H^T, W^T W>, with <A H^T, W> = sum of dpart
// (numerator of the W update against the new W), GH = H H^T and GW = W^T W of the new factors.
// out[0] = square root of that, clamped at zero.  One block.
__global__ __launch_bounds__(256) void objective_kernel(const double *__restrict__ dpart, int nb,
                                                        const float *__restrict__ GW,
                                                        const float *__restrict__ GH, int k,
                                                        const double *__restrict__ normA2, double *out)
{
    __shared__ double part[256], dsum[256];
    double gg = 0.0, dd = 0.0;
    dpart += (int64_t)blockIdx.x * nb;       // a workgroup per iteration
    GW += blockIdx.x * k * k;
    GH += blockIdx.x * k * k;
    out += blockIdx.x;
    for (int e = threadIdx.x; e < k * k; e += 256) gg += (double)GW[e] * (double)GH[e];
    // shares b, b + 256, ... per thread, then the threads in order (the sparse and the streamed
    // runs hand over thousands of shares: one thread alone would spend 0.3 ms on them)
    for (int b = threadIdx.x; b < nb; b += 256) dd += dpart[b];
    part[threadIdx.x] = gg;
    dsum[threadIdx.x] = dd;
    __syncthreads();
    if (threadIdx.x == 0) {
        double g2 = 0.0, dot = 0.0;
        for (int i = 0; i < 256; ++i) g2 += part[i];
        for (int i = 0; i < 256; ++i) dot += dsum[i];
        const double f2 = normA2[0] - 2.0 * dot + g2;
        out[0] = f2 > 0.0 ? sqrt(f2) : 0.0;
    }
}

// P = sum over the row splits of the partial W^T A results (test entry point only).
// blockIdx.y = slice of 64 factors (ranks above 64): partials at ppart + slice * slice_ppart, `count`
// floats of P per full slice, count_last for the last one.
// Eight splits are requested together and added in a tree: one load at a time, a 256 x 256
// Gram matrix over 32 splits took 35 us on 64 workgroups per slice, a chain of trips to memory
// (rank 256 on 16384 x 8192: 1041 -> 977 us per iteration).
__global__ __launch_bounds__(256) void sum_partials_kernel(const float *__restrict__ ppart,
                                                           int splits, int64_t count,
                                                           float *__restrict__ P, int accumulate,
                                                           int64_t slice_ppart, int64_t count_last)
{
    ppart += (int64_t)blockIdx.y * slice_ppart;
    P += (int64_t)blockIdx.y * count;
    if (blockIdx.y == gridDim.y - 1) count = count_last;
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < count; e += (int64_t)gridDim.x * 256) {
        float s = 0.f;
        int t = 0;
        for (; t + 8 <= splits; t += 8) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = ppart[(int64_t)(t + u) * count + e];
            s += tree_sum(v);
        }
        for (; t < splits; ++t) s += ppart[(int64_t)t * count + e];
        P[e] = accumulate ? P[e] + s : s;
    }
}

// X <- X * P / (D + eps) element by element: the multiplicative update with its numerator P
// and the product D of the other factor's Gram matrix with X already formed (ranks above 64).
__global__ __launch_bounds__(256) void mu_apply_kernel(float *__restrict__ X, const float *__restrict__ P,
                                                       const float *__restrict__ D, float eps,
                                                       int64_t count)
{
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < count; e += (int64_t)gridDim.x * 256)
        X[e] = X[e] * P[e] / (D[e] + eps);
}

// ---------------------------------------------------------------------------
// Host side launchers
// ---------------------------------------------------------------------------

static inline bool vec_ok(const void *p, int64_t ld)
{
    return (reinterpret_cast<uintptr_t>(p) & 15u) == 0 && (ld & 3) == 0;
}

// A that the last-level cache (256 MiB) keeps from one pass to the next is loaded to stay there, not
// marked for eviction: 12288 x 4096, k = 20 (192 MiB): A H^T pass 39.4 -> 34.2 us, W^T A 38.2 -> 36.0;
// 2000 x 1204, k = 12: 13.7 -> 11.7 and 8.3 -> 8.0.  A run that reads A and A^T in turn has two matrices to
// keep; per iteration there, marked against kept: 2 x 120 MiB, k = 40 102 and 97 us, 2 x 144 110 and 110 (k = 20 83 and
// 81), 2 x 160, k = 64 124 and 128, 2 x 192, k = 40 132 and 137, 2 x 220, k = 64 147 and 155.
bool stream_a(int64_t rows, int64_t n, bool two)
{
    return rows * n * 4 > ((int64_t)(two ? 152 : 224) << 20);
}

int wta_splits(int64_t rows, int64_t n, int k)
{
    // Enough workgroups to fill the chip once at the kernels' occupancy (2 groups per
    // compute unit), but long row ranges per group: every split costs a k x n partial
    // result written and read again.  A workgroup covers 128 columns up to 32 factors and
    // 256 above.
    const int64_t width = k > 32 ? 256 : kWtaCols;
    const int64_t slabs = (n + width - 1) / width;
    // Rounded down: 512 workgroups are resident at once, and one more split than fits leaves its
    // last workgroups to a second round (20011 x 10000 at k = 50: 40 slabs x 13 splits = 520
    // workgroups take 213 us back to back; 40 x 12 170).
    const int64_t target = 512;
    int64_t s = target / slabs;
    // With one split on fewer than 384 slabs (three quarters of the places) the chip is better served by two rounds of
    // half as long workgroups: pass and finisher, 1 -> 2 splits, k = 32 on 16384 rows: 258 slabs 577 -> 529 us, 300 540
    // -> 507, 400 634 -> 639, 500 690 -> 711; k = 64 on 8192 rows: 258 672 -> 606, 300 728 -> 644, 400 867 -> 844,
    // but 252 -> 259 per iteration at k = 40 on 2048 rows (A^T of 102400 x 2048).
    // (Two splits against three on 172 and 200 slabs: 302 and 317 us against 329 and 356.)
    if (s == 1 && slabs < 384) s = 2;
    int64_t max_by_rows = (rows + 255) / 256;         // at least 256 rows per split ...
    if (slabs * max_by_rows < 128) {
        // ... unless that leaves most of the chip idle: small matrices are split down to one
        // 16-row step per wave, up to 128 workgroups (256 x 192: 19.6 instead of 26.0 us per
        // iteration; with many workgroups the fixed cost of a split outweighs it)
        const int64_t fine = (rows + 63) / 64, want = (128 + slabs - 1) / slabs;
        max_by_rows = fine < want ? fine : want;
    }
    if (s > max_by_rows) s = max_by_rows;
    // every split is a k x n partial that the finisher reads again, a few splits per trip to L2:
    // 32 at most, but up to 128 while there are fewer than 16 column slabs (1048576 x 256: the pass
    // ran on 64 workgroups)
    const int64_t cap = slabs >= 16 ? 32 : 128;
    if (s > cap) s = cap;
    if (s < 1) s = 1;
    return (int)s;
}

int wta_splits_bound(int64_t rows, int64_t n, int k)
{
    // within a column width the count shrinks as slabs grow and does not depend on k
    const int a = wta_splits(rows, n, 1), b = k > 32 ? wta_splits(rows, n, 64) : a;
    return a > b ? a : b;
}

int64_t wta_rows_per_split(int64_t rows, int splits)
{
    int64_t rps = (rows + splits - 1) / splits;
    return (rps + 15) & ~(int64_t)15;   // whole 16-row steps of a wave (and whole row pairs)
}

static int gram_blocks(int64_t len, int per_block)
{
    int64_t b = (len + per_block - 1) / per_block;
    if (b > kGramMaxBlocks) b = kGramMaxBlocks;
    if (b < 1) b = 1;
    return (int)b;
}

hipError_t launch_gram_w(const float *X, int64_t rows, int k, float *G, float *gpart,
                         unsigned *counters, hipStream_t st)
{
    const int kt = k_tiles(k);
    dim3 grid(gram_blocks(rows, 512), kt * kt);
    hipLaunchKernelGGL((gram_kernel<0, false>), grid, dim3(512), 0, st, X, rows, k, G, gpart, counters, k);
    return hipGetLastError();
}

// Up to 2048 rows per workgroup, four trips; beyond, 256 workgroups and a launch for the sum read faster.  Sparse iterations
// (two Gram matrices of this many rows, one entry per row), gram16_kernel against the two launches, in us: k = 12 16384 rows 29.0, 31.3,
// 65536 38.9, 41.3, 98304 51.9, 53.2, 131072 55.4, 55.9, 262144 93.3, 89.9; k = 4 131072 39.8, 40.5, 262144 53.8, 51.2; k = 16 131072
// 58.7, 58.9, 262144 99.5, 96.2.
constexpr int64_t kGram16Rows = 1 << 17;
hipError_t launch_gram_w_wide(const float *X, int64_t rows, int k, float *G, float *tiles, unsigned *counters, hipStream_t st, int ld)
{
    if (k <= 16 && rows <= kGram16Rows) {
        int64_t nb = (rows + 63) / 64;
        if (nb > kGram16Blocks) nb = kGram16Blocks;
        hipLaunchKernelGGL(gram16_kernel, dim3((unsigned)nb), dim3(512), 0, st, X, rows, k, ld ? ld : k, G, tiles, counters);
        return hipGetLastError();
    }
    const int kt = k_tiles(k);
    // 256 rows per workgroup: two trips of eight row pairs per wave (65536 x 12: 7.8 us with 512 rows)
    int64_t nb = (rows + 255) / 256;
    if (nb > kFinMaxBlocks) nb = kFinMaxBlocks;
    if (nb < 1) nb = 1;
    hipLaunchKernelGGL((gram_kernel<0, false>), dim3((unsigned)nb, kt * kt), dim3(512), 0, st, X, rows, k,
                       static_cast<float *>(nullptr), tiles, static_cast<unsigned *>(nullptr), ld ? ld : k);
    return launch_gram_sum(tiles, (int)nb, k, G, st);
}

hipError_t launch_gram_h(const float *X, int k, int64_t cols, float *G, float *gpart,
                         unsigned *counters, hipStream_t st)
{
    const int kt = k_tiles(k);
    dim3 grid(gram_blocks(cols, 512), kt * kt);
    if (vec_ok(X, cols))
        hipLaunchKernelGGL((gram_kernel<1, true>), grid, dim3(512), 0, st, X, cols, k, G, gpart, counters, k);
    else
        hipLaunchKernelGGL((gram_kernel<1, false>), grid, dim3(512), 0, st, X, cols, k, G, gpart, counters, k);
    return hipGetLastError();
}

template <int KT>
static void wta_dispatch(bool vec, dim3 grid, hipStream_t st, const float *A, const float *W,
                         float *ppart, int64_t rows, int64_t n, int k, int64_t rps, int acc,
                         const float *gtiles, int nsets, float *gsum)
{
    constexpr int U = 5, OCC = 2;
    const dim3 block(64 * kWtaWaves);
    if (vec)
        hipLaunchKernelGGL((wta_pass_kernel<KT, U, OCC, true>), grid, block, 0, st, A, W, ppart, rows, n, k, rps, acc, gtiles, nsets, gsum);
    else
        hipLaunchKernelGGL((wta_pass_kernel<KT, U, OCC, false>), grid, block, 0, st, A, W, ppart, rows, n, k, rps, acc, gtiles, nsets, gsum);
}

int wta_planes_only_width(const float *A, int64_t n)
{
    return (vec_ok(A, n) && n < ((int64_t)1 << 25)) ? 64 : 32;
}

size_t planes_bytes(int64_t rows) { return (size_t)((rows + 7) / 8) * 3 * 64 * 16; }   // 64 factor slots

hipError_t launch_split_planes_slice(const float *X, int64_t rows, int64_t ld, int64_t c0, int kc,
                                     void *planes, hipStream_t st)
{
    if (kc < 1 || kc > 64) return hipErrorInvalidValue;
    const int kp = kc <= 32 ? 32 : 64;
    const int64_t threads = ((rows + 7) / 8) * kp;
    hipLaunchKernelGGL(split_planes_kernel, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, st, X,
                       rows, ld, c0, kc, kp, static_cast<u32x4 *>(planes), (int64_t)0);
    return hipGetLastError();
}

hipError_t launch_sum_partials_slices(const float *ppart, int splits, int k, int64_t cols, float *P, hipStream_t st,
                                      bool accumulate)
{
    const int nslices = (k + 63) / 64;
    const int64_t count = 64 * cols, count_last = (int64_t)(k - 64 * (nslices - 1)) * cols;
    int64_t b = (count + 255) / 256;
    if (b > 4096) b = 4096;
    // the partials of slice z hold splits x (factors of z) x cols floats, packed for that slice's width
    hipLaunchKernelGGL(sum_partials_kernel, dim3((unsigned)b, (unsigned)nslices), dim3(256), 0, st, ppart, splits, count, P,
                       accumulate ? 1 : 0, (int64_t)splits * 64 * cols, count_last);
    return hipGetLastError();
}

hipError_t launch_split_planes(const float *X, int64_t rows, int k, void *planes, hipStream_t st)
{
    if (!wta_uses_planes(k)) return hipSuccess;
    return launch_split_planes_slice(X, rows, k, 0, k, planes, st);
}

hipError_t launch_mu_apply(float *X, const float *P, const float *D, float eps, int64_t count,
                           hipStream_t st)
{
    int64_t b = (count + 255) / 256;
    if (b > 8192) b = 8192;
    hipLaunchKernelGGL(mu_apply_kernel, dim3((unsigned)b), dim3(256), 0, st, X, P, D, eps, count);
    return hipGetLastError();
}

hipError_t launch_wta_pass(const float *A, int64_t rows, int64_t n, int k, const float *W,
                           void *planes, bool planes_ready, float *ppart, int splits, int64_t rps,
                           bool accumulate, hipStream_t st, const float *gtiles, int nsets, float *gsum, bool two)
{
    dim3 grid((unsigned)((n + kWtaCols - 1) / kWtaCols), (unsigned)splits);
    const bool vec = vec_ok(A, n);
    const int acc = accumulate ? 1 : 0;
    if (rps % 16) return hipErrorInvalidValue;
    switch (k_tiles(k)) {
    case 1: {
        if (!planes) return hipErrorInvalidValue;
        if (!planes_ready) {
            hipError_t e = launch_split_planes(W, rows, k, planes, st);
            if (e != hipSuccess) return e;
        }
        const u32x4 *pl = static_cast<const u32x4 *>(planes);
        const dim3 block(64 * kWtaWaves);
        // buffer loads address 16 rows with 32-bit offsets: 64 n bytes must stay below 2^31
        if (vec && n < ((int64_t)1 << 25))
            if (stream_a(rows, n, two)) hipLaunchKernelGGL(wta_pass_split_buf_kernel<kStreamLoad>, grid, block, 0, st, A, pl, ppart, rows, n, k, rps, acc, gtiles, nsets, gsum);
            else hipLaunchKernelGGL(wta_pass_split_buf_kernel<0>, grid, block, 0, st, A, pl, ppart, rows, n, k, rps, acc, gtiles, nsets, gsum);
        else
            hipLaunchKernelGGL((wta_pass_split_kernel<false>), grid, block, 0, st, A, pl, ppart, rows, n, k, rps, acc, gtiles, nsets, gsum);
        break;
    }
    case 2:
        if (vec && planes && n < ((int64_t)1 << 25)) {
            if (!planes_ready) {
                hipError_t e = launch_split_planes(W, rows, k, planes, st);
                if (e != hipSuccess) return e;
            }
            const dim3 grid256((unsigned)((n + 255) / 256), (unsigned)splits);
            if (stream_a(rows, n, two))
                hipLaunchKernelGGL(wta_pass_split64_wide_kernel<kStreamLoad>, grid256, dim3(64 * kWtaWaves), 0, st, A,
                                   static_cast<const u32x4 *>(planes), ppart, rows, n, k, rps, acc, gtiles, nsets, gsum);
            else
                hipLaunchKernelGGL(wta_pass_split64_wide_kernel<0>, grid256, dim3(64 * kWtaWaves), 0, st, A,
                                   static_cast<const u32x4 *>(planes), ppart, rows, n, k, rps, acc, gtiles, nsets, gsum);
        } else {
            if (!W) return hipErrorInvalidValue;   // this kernel reads the factor itself, not its planes
            wta_dispatch<2>(vec, grid, st, A, W, ppart, rows, n, k, rps, acc, gtiles, nsets, gsum);
        }
        break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

int gram_w_blocks(int64_t rows) { return gram_blocks(rows, 512); }

hipError_t launch_gram_sum(const float *gpart, int nb, int k, float *G, hipStream_t st)
{
    const int kt = k_tiles(k);
    const int threads = kt * kt * 1024 * 8;
    hipLaunchKernelGGL(gram_sum_kernel, dim3((threads + 255) / 256), dim3(256), 0, st, gpart, nb, k, G);
    return hipGetLastError();
}

// Columns per workgroup and chunk of the finisher: 64 fill whole cache lines and leave a row to a
// wave; shorter factors take narrower chunks, which put up to 256 workgroups on the splits
// (k = 16 on 512 columns and 128 splits: 27 us with 8 workgroups of 64 columns, 11 with 32 of 16;
// k = 20 on 4096: 10.5 with 64 workgroups, 7.8 with 128 of 32).
static int factor_update_width(int64_t len) { return len <= 2048 ? 16 : (len <= 8192 ? 32 : 64); }

int factor_update_blocks(int64_t len)
{
    const int cw = factor_update_width(len);
    int64_t b = (len + cw - 1) / cw;
    if (b > kFinMaxBlocks) b = kFinMaxBlocks;
    return (int)b;
}

template <int CW, bool BIG>
static void factor_update_dispatch(dim3 grid, hipStream_t st, float *X, float *Xt, const float *part, int splits,
                                   const float *Gfull, const float *gin, int nbin, float *gout, u32x4 *pl,
                                   double *dpart, int k, int64_t len, float eps, const BlockMap &bm, const FinisherSlices &sl)
{
    const dim3 block(512);
#define NMFMU_FINISHER(KP, PAIRS) \
    hipLaunchKernelGGL((factor_update_kernel<KP, CW, BIG, PAIRS>), grid, block, 0, st, X, Xt, part, splits, Gfull, gin, nbin, gout, pl, dpart, k, len, eps, bm, sl)
    if (sl.pairs.units && grid.y > 1) NMFMU_FINISHER(64, 2);
    else if (sl.pairs.units) NMFMU_FINISHER(64, 1);
    else if (k <= 8) NMFMU_FINISHER(8, 0);
    else if (k <= 16) NMFMU_FINISHER(16, 0);
    else if (k <= 32) NMFMU_FINISHER(32, 0);
    else NMFMU_FINISHER(64, 0);
#undef NMFMU_FINISHER
}

static hipError_t factor_update(float *X, float *Xt, const float *part, int splits, const float *Gfull, const float *gin, int nbin,
                                float *gout, u32x4 *pl, double *dpart, int k, int64_t len, float eps, hipStream_t st,
                                const BlockMap &bm, int slices, const FinisherSlices &sl)
{
    // Without Gram output there is no reason to cap the grid: one block per chunk.
    const int cw = factor_update_width(len);
    int64_t blocks = gout ? factor_update_blocks(len) : (len + cw - 1) / cw;
    if (blocks > 65535) blocks = 65535;
    const dim3 grid((unsigned)blocks, (unsigned)slices);
    if (cw == 16) factor_update_dispatch<16, false>(grid, st, X, Xt, part, splits, Gfull, gin, nbin, gout, pl, dpart, k, len, eps, bm, sl);
    else if (cw == 32) factor_update_dispatch<32, false>(grid, st, X, Xt, part, splits, Gfull, gin, nbin, gout, pl, dpart, k, len, eps, bm, sl);
    else if (k * len < ((int64_t)1 << 29)) factor_update_dispatch<64, false>(grid, st, X, Xt, part, splits, Gfull, gin, nbin, gout, pl, dpart, k, len, eps, bm, sl);
    else factor_update_dispatch<64, true>(grid, st, X, Xt, part, splits, Gfull, gin, nbin, gout, pl, dpart, k, len, eps, bm, sl);
    return hipGetLastError();
}

hipError_t launch_factor_update(float *X, float *Xt, const float *part, int splits,
                                const float *Gfull, const float *gin, int nbin, float *gout, int k,
                                int64_t len, float eps, hipStream_t st, const BlockMap *map,
                                void *planes, double *dpart)
{
    u32x4 *pl = wta_uses_planes(k) ? static_cast<u32x4 *>(planes) : nullptr;
    BlockMap bm;
    if (map) bm = *map;
    else bm.on = 0;
    return factor_update(X, Xt, part, splits, Gfull, gin, nbin, gout, pl, dpart, k, len, eps, st, bm, 1, FinisherSlices{});
}

hipError_t launch_pair_update(const FinisherSlices &sl, int slices, const float *part, int splits, const float *gin, float *gout,
                              int64_t len, float eps, hipStream_t st, double *dpart)
{
    int kmax = 0;
    for (int z = 0; z < slices; ++z) kmax = sl.k[z] > kmax ? sl.k[z] : kmax;
    if (slices < 1 || slices > kPairGroup || kmax > 64 || !gout || (dpart && slices > 1)) return hipErrorInvalidValue;
    return factor_update(nullptr, nullptr, part, splits, nullptr, gin, gin ? 1 : 0, gout, nullptr, dpart, kmax, len, eps, st, sl.bm[0], slices, sl);
}

hipError_t launch_sum_partials(const float *ppart, int splits, int64_t count, float *P,
                               hipStream_t st, bool accumulate)
{
    int64_t b = (count + 255) / 256;
    if (b > 4096) b = 4096;
    hipLaunchKernelGGL(sum_partials_kernel, dim3((unsigned)b), dim3(256), 0, st, ppart, splits, count, P, accumulate ? 1 : 0,
                       (int64_t)0, count);
    return hipGetLastError();
}

hipError_t launch_sumsq(const float *X, int64_t count, double *partial, double *out, hipStream_t st)
{
    int64_t b = (count + 256 * 64 - 1) / (256 * 64);
    if (b > 4096) b = 4096;
    if (b < 1) b = 1;
    hipLaunchKernelGGL(sumsq_kernel, dim3((unsigned)b), dim3(256), 0, st, X, count, partial);
    hipLaunchKernelGGL(sum_f64_kernel, dim3(1), dim3(256), 0, st, partial, b, out);
    return hipGetLastError();
}

hipError_t launch_objective(const double *dpart, int nb, const float *GW, const float *GH, int k,
                            const double *normA2, double *out, hipStream_t st, int iters)
{
    hipLaunchKernelGGL(objective_kernel, dim3((unsigned)iters), dim3(256), 0, st, dpart, nb, GW, GH, k, normA2, out);
    return hipGetLastError();
}

// Row splits of the streaming objective kernel: one resident set of workgroups, whole 32-row tiles.
static int residual_splits(int64_t m, int64_t n)
{
    const int64_t slabs = (n + 255) / 256;
    int64_t s = (512 + slabs - 1) / slabs;
    const int64_t by_rows = (m + 31) / 32;
    if (s > by_rows) s = by_rows;
    if (s < 1) s = 1;
    return (int)s;
}

static int64_t residual_rows_per_split(int64_t m, int64_t n)
{
    const int splits = residual_splits(m, n);
    return ((m + splits - 1) / splits + 31) & ~(int64_t)31;
}

int64_t residual_partials(int64_t m, int64_t n)
{
    const int64_t a = (m + 31) / 32, b = ((n + 255) / 256) * residual_splits(m, n) + 1;
    return a > b ? a : b;
}

hipError_t launch_residual(const float *A, int64_t m, int64_t n, int k, const float *W,
                           const float *H, double *partial, double *out, hipStream_t st)
{
    const int64_t m32 = m & ~(int64_t)31;
    // the streaming kernel adds a 32-bit lane offset of up to 4 n + 62 floats to a row address
    if (m32 > 0 && k <= 32 && k % 16 == 0 && n < ((int64_t)1 << 29) && vec_ok(A, n) && vec_ok(H, n) && vec_ok(W, k)) {
        // whole 32-row tiles by the streaming kernel, the up to 31 rows left by one workgroup
        // of the general one
        const int splits = residual_splits(m32, n);
        int64_t rps = (m32 + splits - 1) / splits;
        rps = (rps + 31) & ~(int64_t)31;
        const dim3 grid((unsigned)((n + 255) / 256), (unsigned)splits);
        int64_t count = (int64_t)grid.x * grid.y;
        if (k == 16)
            hipLaunchKernelGGL(residual_stream_kernel<1>, grid, dim3(256), 0, st, A, W, H, m32, n, rps, partial);
        else
            hipLaunchKernelGGL(residual_stream_kernel<2>, grid, dim3(256), 0, st, A, W, H, m32, n, rps, partial);
        if (m > m32) {
            hipLaunchKernelGGL((residual_kernel<1, true>), dim3(1), dim3(256), 0, st, A + m32 * n, W + m32 * k, H,
                               m - m32, n, k, partial + count);
            ++count;
        }
        hipLaunchKernelGGL(residual_finish_kernel, dim3(1), dim3(256), 0, st, (const double *)partial, count, out);
        return hipGetLastError();
    }
    // The other streaming kernels (32 rows of A with 32-bit byte offsets: 128 n < 2^31) from four row
    // tiles per workgroup on, about 2^24 elements; below that their pipelines do not fill.  On aligned operands the fp32 instruction up to 24
    // factors and, where a workgroup has fewer than eight tiles for the longer start of the other, up to 48; else pairs of halves.
    // Whole call in us: 16384 x 8192, k = 10 / 17 / 29 / 64: fp32 101 / 109 / 128 / 237, pairs 103 / 114 / 118 / 180; 8192 x 2048,
    // k = 20 / 40 / 64: 37 / 50 / 72 and 44 / 54 / 65; 65536 x 1024, k = 40: 102 and 98.  k = 32 on the kernel above 104, pairs 126.
    // Misaligned: residual_kernel 16384 x 8190, k = 10 192, pairs 118; 9001 x 7003, k = 50 319 and 142; 2050 x 8191, k = 20 162 and 50.
    if (n < ((int64_t)1 << 24) && residual_rows_per_split(m, n) >= 128) {
        const int splits = residual_splits(m, n);
        const int64_t rps = residual_rows_per_split(m, n);
        const dim3 grid((unsigned)((n + 255) / 256), (unsigned)splits);
        const int64_t count = (int64_t)grid.x * grid.y;
#define NMFMU_RESIDUAL(...) hipLaunchKernelGGL((__VA_ARGS__), grid, dim3(256), 0, st, A, W, H, m, n, k, rps, partial)
        if (vec_ok(A, n) && vec_ok(H, n) && (k <= 24 || (k <= 48 && rps < 256))) {
            if (k <= 8) NMFMU_RESIDUAL(residual_stream_f32_kernel<4>);
            else if (k <= 16) NMFMU_RESIDUAL(residual_stream_f32_kernel<8>);
            else if (k <= 24) NMFMU_RESIDUAL(residual_stream_f32_kernel<12>);
            else if (k <= 32) NMFMU_RESIDUAL(residual_stream_f32_kernel<16>);
            else NMFMU_RESIDUAL(residual_stream_f32_kernel<24>);
        } else if (k <= 16) NMFMU_RESIDUAL(residual_pair_kernel<1, false>);
        else if (vec_ok(A, n)) {
            if (k <= 32) NMFMU_RESIDUAL(residual_pair_kernel<2, true>);
            else if (k <= 48) NMFMU_RESIDUAL(residual_pair_kernel<3, true>);
            else NMFMU_RESIDUAL(residual_pair_kernel<4, true>);
        } else {
            if (k <= 32) NMFMU_RESIDUAL(residual_pair_kernel<2, false>);
            else if (k <= 48) NMFMU_RESIDUAL(residual_pair_kernel<3, false>);
            else NMFMU_RESIDUAL(residual_pair_kernel<4, false>);
        }
#undef NMFMU_RESIDUAL
        hipLaunchKernelGGL(residual_finish_kernel, dim3(1), dim3(256), 0, st, (const double *)partial, count, out);
        return hipGetLastError();
    }
    const int64_t blocks = (m + 31) / 32;
    const bool vec = vec_ok(A, n) && vec_ok(H, n);
    const dim3 grid((unsigned)blocks), block(256);
    if (k_tiles(k) == 1) {
        if (vec) hipLaunchKernelGGL((residual_kernel<1, true>), grid, block, 0, st, A, W, H, m, n, k, partial);
        else hipLaunchKernelGGL((residual_kernel<1, false>), grid, block, 0, st, A, W, H, m, n, k, partial);
    } else {
        if (vec) hipLaunchKernelGGL((residual_kernel<2, true>), grid, block, 0, st, A, W, H, m, n, k, partial);
        else hipLaunchKernelGGL((residual_kernel<2, false>), grid, block, 0, st, A, W, H, m, n, k, partial);
    }
    hipLaunchKernelGGL(residual_finish_kernel, dim3(1), dim3(256), 0, st, (const double *)partial, blocks, out);
    return hipGetLastError();
}

template <int KT>
static void aht_dispatch(bool vec, dim3 grid, hipStream_t st, const float *A, const float *H,
                         const float *GH, float *W, int64_t rows, int64_t n, int k, float eps, double *dpart)
{
    constexpr int RT = kAhtRowTiles;
    if (vec)
        hipLaunchKernelGGL((aht_pass_kernel<KT, RT, true>), grid, dim3(512), 0, st, A, H, GH, W, rows, n, k, eps, dpart);
    else
        hipLaunchKernelGGL((aht_pass_kernel<KT, RT, false>), grid, dim3(512), 0, st, A, H, GH, W, rows, n, k, eps, dpart);
}

int64_t aht_pass_blocks(int64_t rows) { return (rows + 32 * kAhtRowTiles - 1) / (32 * kAhtRowTiles); }

hipError_t launch_aht_pass(const float *A, int64_t rows, int64_t n, int k, const float *H,
                           const float *GH, float *W, float eps, hipStream_t st, double *dpart)
{
    dim3 grid((unsigned)aht_pass_blocks(rows));
    const bool vec = vec_ok(A, n) && vec_ok(H, n);
    switch (k_tiles(k)) {
    case 1: aht_dispatch<1>(vec, grid, st, A, H, GH, W, rows, n, k, eps, dpart); break;
    case 2: aht_dispatch<2>(vec, grid, st, A, H, GH, W, rows, n, k, eps, dpart); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

bool aht_rows_can(const float *A, int64_t n, int k)
{
    // 32 rows of A are addressed with 32-bit byte offsets: 128 n < 2^31
    return k <= 64 && vec_ok(A, n) && n < ((int64_t)1 << 24);
}

bool aht_rows_ok(const float *A, int64_t m, int64_t n, int k)
{
    // Short and wide matrices leave most of the chip without a row block (64-row blocks: 12288 rows
    // are 192 of them), and with fewer than eight 64-column chunks some of a workgroup's waves have
    // none: such shapes do better on a transposed copy, unless the whole problem is small enough to be
    // latency bound anyway.
    return aht_rows_can(A, n, k) && ((m >= 12288 && n >= 512) || m * n <= ((int64_t)1 << 22));
}

// row tiles per workgroup: 128-row blocks when they fill the chip, else 64-row or 32-row blocks; two
// 32-factor tiles leave registers for two row tiles only
int aht_rows_tiles(int64_t rows, int k)
{
    if (k > 32) return 2;
    // 32-row blocks below 8192 rows: 2000 x 1204, k = 12, 18.0 us on 32 workgroups of 64 rows, 13.7 on 63
    return (rows + 127) / 128 >= 192 ? 4 : (rows + 63) / 64 >= 128 ? 2 : 1;
}

int aht_rows_blocks(int64_t rows, int k, int tiles)
{
    const int64_t rb = 32 * (tiles ? tiles : aht_rows_tiles(rows, k));
    int64_t b = (rows + rb - 1) / rb;
    if (b > kFinMaxBlocks) b = kFinMaxBlocks;
    return (int)b;
}

template <int R, int KT, int POLICY>
static hipError_t aht_rows_launch(dim3 grid, hipStream_t st, const float *A, const u32x4 *ph, const float *GH, float *W,
                                  u32x4 *pw, float *gout, double *dpart, int64_t rows, int64_t n, int k, float eps,
                                  int mode, const BlockMap &bm)
{
    constexpr int kLdsBytes = (8 * 2048 + 4 * R * KT * 1024 + (KT == 2 ? 4096 : 0)) * (int)sizeof(float);
    static bool raised = false;      // more dynamic LDS than the default limit: asked for once per process
    if (!raised) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&aht_rows_kernel<R, KT, POLICY>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
        if (e != hipSuccess) return e;
        raised = true;
    }
    hipLaunchKernelGGL((aht_rows_kernel<R, KT, POLICY>), grid, dim3(512), kLdsBytes, st, A, ph, GH, W, pw, gout, dpart, rows, n, k, eps, mode, bm);
    return hipGetLastError();
}

hipError_t launch_aht_rows(const float *A, int64_t rows, int64_t n, int k, const void *planesH,
                           const float *GH, float *W, void *planesW, float *gout, float eps, hipStream_t st,
                           bool gram_only, const BlockMap *map, double *dpart, bool dry, int tiles)
{
    if (tiles == 0) tiles = aht_rows_tiles(rows, k);
    if (k > 64 || !planesW || !gout || (k > 32 ? tiles != 2 : tiles != 1 && tiles != 2 && tiles != 4)) return hipErrorInvalidValue;
    if (!gram_only && (!A || !planesH || !GH || !vec_ok(A, n) || n >= ((int64_t)1 << 24))) return hipErrorInvalidValue;
    BlockMap bm;
    if (map) bm = *map;
    else bm.on = 0;
    const dim3 grid((unsigned)aht_rows_blocks(rows, k, tiles));
    const u32x4 *ph = static_cast<const u32x4 *>(planesH);
    u32x4 *pw = static_cast<u32x4 *>(planesW);
    const int mode = gram_only ? 1 : (dry ? 2 : 0);
    const bool stream = stream_a(rows, n);
#define NMFMU_AHT_ROWS(R, KT) \
    return stream ? aht_rows_launch<R, KT, kStreamLoad>(grid, st, A, ph, GH, W, pw, gout, dpart, rows, n, k, eps, mode, bm) \
                  : aht_rows_launch<R, KT, 0>(grid, st, A, ph, GH, W, pw, gout, dpart, rows, n, k, eps, mode, bm)
    if (k > 32) NMFMU_AHT_ROWS(2, 2);
    if (tiles == 4) NMFMU_AHT_ROWS(4, 1);
    if (tiles == 2) NMFMU_AHT_ROWS(2, 1);
    NMFMU_AHT_ROWS(1, 1);
#undef NMFMU_AHT_ROWS
}

bool one_pass_ok(const float *A, int64_t n, int k)
{
    // Whatever the number of rows: per iteration against the row plan (us), n = 160, k = 16, m = 256 /
    // 16000 / 262144: 26.6 / 41.9 / 192 -> 17.0 / 33.8 / 103; n = 512: 27.2 / 48.4 / 326 -> 17.5 / 39.7 /
    // 175.  1.07 to 2.06x over n = 160 to 512, m = 256 to 262144, k = 4 to 32.
    return k <= 32 && vec_ok(A, n) && n <= 512;
}

int one_pass_blocks(int64_t rows, int64_t n)
{
    const int rb = n <= 256 ? 64 : 32;
    const int64_t b = (rows + rb - 1) / rb;
    return (int)(b < kFinMaxBlocks ? b : kFinMaxBlocks);
}

template <int NRW, int POLICY, bool update, bool product>
static hipError_t one_pass_launch(dim3 grid, hipStream_t st, const float *A, const u32x4 *planesH, const float *GH,
                                  const float *ghsets, int nbh, const float *W, float *Wnew, float *ppart, float *gout, double *dpart,
                                  int64_t rows, int64_t n, int k, float eps)
{
    constexpr int kLdsBytes = (8 * 2048 + 8 * 1024 + 3 * 4 * NRW * 32 * 4 + 32 * NRW * 36 + 32 * 36) * (int)sizeof(float);
    static bool raised = false;      // more dynamic LDS than the default limit: asked for once per process
    if (!raised) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&one_pass_kernel<NRW, POLICY, update, product>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
        if (e != hipSuccess) return e;
        raised = true;
    }
    hipLaunchKernelGGL((one_pass_kernel<NRW, POLICY, update, product>), grid, dim3(512), kLdsBytes, st, A, planesH, GH, ghsets, nbh, W, Wnew,
                       ppart, gout, dpart, rows, n, k, eps);
    return hipGetLastError();
}

template <int NRW, int POLICY, bool update, bool product>
static hipError_t one_pass16_launch(dim3 grid, hipStream_t st, const float *A, const u32x4 *planesH, const float *GH,
                                    const float *ghsets, int nbh, const float *W, float *Wnew, float *ppart, float *gout, double *dpart,
                                    int64_t rows, int64_t n, int k, float eps)
{
    constexpr int kLdsBytes = (16 * 1024 + 16 * 512 + 32 * NRW * 20 + 16 * 20 + 3 * 4 * NRW * 64) * (int)sizeof(float);
    static bool raised = false;      // more dynamic LDS than the default limit: asked for once per process
    if (!raised) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&one_pass16_kernel<NRW, POLICY, update, product>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
        if (e != hipSuccess) return e;
        raised = true;
    }
    hipLaunchKernelGGL((one_pass16_kernel<NRW, POLICY, update, product>), grid, dim3(1024), kLdsBytes, st, A, planesH, GH, ghsets, nbh, W, Wnew,
                       ppart, gout, dpart, rows, n, k, eps);
    return hipGetLastError();
}

hipError_t launch_one_pass(const float *A, int64_t rows, int64_t n, int k, const void *planesH, const float *GH,
                           const float *ghsets, int nbh, const float *W, float *Wnew, float *ppart, float *gout, float eps,
                           hipStream_t st, bool update, bool product, double *dpart)
{
    if (!one_pass_ok(A, n, k) || !gout || (!update && !product) || (product && !ppart) || (update && (!planesH || (!GH && !ghsets))))
        return hipErrorInvalidValue;
    const dim3 grid((unsigned)one_pass_blocks(rows, n));
    const u32x4 *ph = static_cast<const u32x4 *>(planesH);
    const bool stream = stream_a(rows, n);
#define NMFMU_ONE_PASS16(NRW, POL) \
    return !update ? one_pass16_launch<NRW, POL, false, true>(grid, st, A, ph, GH, ghsets, nbh, W, Wnew, ppart, gout, dpart, rows, n, k, eps) \
         : product ? one_pass16_launch<NRW, POL, true, true>(grid, st, A, ph, GH, ghsets, nbh, W, Wnew, ppart, gout, dpart, rows, n, k, eps) \
                   : one_pass16_launch<NRW, POL, true, false>(grid, st, A, ph, GH, ghsets, nbh, W, Wnew, ppart, gout, dpart, rows, n, k, eps)
    if (k <= 16) {
        if (n <= 256) {
            if (stream) NMFMU_ONE_PASS16(2, kStreamLoad);
            NMFMU_ONE_PASS16(2, 0);
        }
        if (stream) NMFMU_ONE_PASS16(1, kStreamLoad);
        NMFMU_ONE_PASS16(1, 0);
    }
#undef NMFMU_ONE_PASS16
#define NMFMU_ONE_PASS(NRW, POL) \
    return !update ? one_pass_launch<NRW, POL, false, true>(grid, st, A, ph, GH, ghsets, nbh, W, Wnew, ppart, gout, dpart, rows, n, k, eps) \
         : product ? one_pass_launch<NRW, POL, true, true>(grid, st, A, ph, GH, ghsets, nbh, W, Wnew, ppart, gout, dpart, rows, n, k, eps) \
                   : one_pass_launch<NRW, POL, true, false>(grid, st, A, ph, GH, ghsets, nbh, W, Wnew, ppart, gout, dpart, rows, n, k, eps)
    if (n <= 256) {
        if (stream) NMFMU_ONE_PASS(2, kStreamLoad);
        NMFMU_ONE_PASS(2, 0);
    }
    if (stream) NMFMU_ONE_PASS(1, kStreamLoad);
    NMFMU_ONE_PASS(1, 0);
#undef NMFMU_ONE_PASS
}

// Compute units of the current device (asked for once per device).
static int compute_units()
{
    static std::atomic<int> known[64];
    int dev = -1, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
    if ((cus = known[dev].load(std::memory_order_relaxed)) == 0) {
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
        known[dev].store(cus, std::memory_order_relaxed);
    }
    return cus;
}

// Row tiles per workgroup of the resident plan, 0: the plan does not apply.  One workgroup per compute unit, so the tiles
// of A must be at most 256; within that the plan was faster at every size tried (us per iteration of 50, other plans ->
// this one): 200 x 150 17.0 -> 6.4, 512 x 512 17.3 -> 9.8, 64 x 4096 33.7 -> 12.9, 2048 x 2048 31.9 -> 12.4, 8000 x 512
// 34.8 -> 16.2, 16384 x 256 33.6 -> 17.3, 16384 x 64 31.7 -> 16.1; two iterations in a call, with its wait, 47 -> 36 us to 89 -> 68.
// One iteration in a call takes as long as on the others, 4 us less to 2 more; it stays here for the bits of a run cut in pieces.
// Low tiles first, as a workgroup's own work is shorter, but not more than 32 row groups if higher ones avoid that:
// every owner of columns adds up a share per group (2000 x 192: 125 groups 10.4 us, 32 groups 8.5; 4096 x 256: 256 groups
// 15.8, 64 groups 9.9).
int resident_tiles(int64_t m, int64_t n, int k)
{
    if (k > 16 || m > 1 << 16 || n > 1 << 12) return 0;
    const int64_t cols = (n + 255) / 256, most = compute_units() < 256 ? compute_units() : 256;
    for (int rt = 1; rt <= 4; rt *= 2) {
        const int64_t groups = (m + 16 * rt - 1) / (16 * rt);
        if (groups * cols <= most && (groups <= 32 || rt == 4)) return rt;
    }
    return 0;
}

template <int RT, bool EVERY>
static hipError_t resident_launch(unsigned blocks, hipStream_t st, const ResidentArgs &a)
{
    constexpr int kLdsBytes = resident_lds_floats(RT) * (int)sizeof(float);
    static bool raised = false;      // more dynamic LDS than the default limit: asked for once per process
    if (!raised) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&resident_kernel<RT, EVERY>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
        if (e != hipSuccess) return e;
        raised = true;
    }
    hipLaunchKernelGGL((resident_kernel<RT, EVERY>), dim3(blocks), dim3(512), kLdsBytes, st, a);
    return hipGetLastError();
}

hipError_t launch_resident(const ResidentArgs &args, int tiles, hipStream_t st, int workgroups)
{
    ResidentArgs a = args;
    if (a.k < 1 || a.k > 16 || a.m < 1 || a.n < 1 || !a.A || !a.part || !a.qpart || !a.hx || !a.wx || !a.sync ||
        (a.dpart && (!a.gout || !a.gh)) || (a.gw && (!a.dpart || a.lead || !a.trail)) || (tiles != 1 && tiles != 2 && tiles != 4))
        return hipErrorInvalidValue;
    const int64_t R = (a.m + 16 * tiles - 1) / (16 * tiles), C = (a.n + 255) / 256;
    if (R * C > 256) return hipErrorInvalidValue;
    a.R = (int)R;
    a.C = (int)C;
    // 200 us: a launch's workgroups are all there after 10 to 20 if nothing is in the way, and who comes later joins in
    if (!a.patience) a.patience = 20000;
    if (!a.polls) a.polls = kLostPolls;
    const unsigned blocks = workgroups > 0 && workgroups < R * C ? (unsigned)workgroups : (unsigned)(R * C);
    hipError_t e = launch_fill_f32(reinterpret_cast<float *>(a.sync), resident_sync_words(R, C), 0.f, st);
    if (e != hipSuccess) return e;
    if (a.gw) return tiles == 1 ? resident_launch<1, true>(blocks, st, a) : tiles == 2 ? resident_launch<2, true>(blocks, st, a) : resident_launch<4, true>(blocks, st, a);
    return tiles == 1 ? resident_launch<1, false>(blocks, st, a) : tiles == 2 ? resident_launch<2, false>(blocks, st, a) : resident_launch<4, false>(blocks, st, a);
}

hipError_t launch_resident_run(const ResidentArgs &args, int tiles, hipStream_t st, int workgroups)
{
    const int piece = resident_piece((args.m + 16 * tiles - 1) / (16 * tiles) * ((args.n + 255) / 256));
    ResidentArgs a = args;
    a.trail = 1;
    for (int left = args.nprod; left > 0; left -= a.nprod) {
        a.nprod = left < piece ? left : piece;
        a.dpart = a.nprod == left ? args.dpart : nullptr;
        a.gout = a.nprod == left ? args.gout : nullptr;
        if (hipError_t e = launch_resident(a, tiles, st, workgroups)) return e;
        a.Win = a.W;
        a.Hin = a.H;
    }
    return hipSuccess;
}

hipError_t launch_share_sum(const float *ppart, int nb, int k, int64_t n, float *psum, const float *gtiles, float *G, hipStream_t st)
{
    if (k < 1 || k > 32 || n % 4 || nb < 1) return hipErrorInvalidValue;
    const int count4 = (int)(k * n / 4), pblocks = (count4 * kShareGroups + 255) / 256;
    hipLaunchKernelGGL(share_sum_kernel, dim3((unsigned)pblocks + 32u), dim3(256), 0, st, ppart, nb, count4, reinterpret_cast<f32x4 *>(psum),
                       pblocks, gtiles, k, G);
    return hipGetLastError();
}

hipError_t launch_sum_f64(const double *in, int64_t count, double *out, hipStream_t st)
{
    hipLaunchKernelGGL(sum_f64_kernel, dim3(1), dim3(256), 0, st, in, count, out);
    return hipGetLastError();
}

}  // namespace nmfmu
