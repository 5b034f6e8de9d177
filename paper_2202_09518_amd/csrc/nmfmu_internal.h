// Internal declarations shared by the HIP translation units of libnmfmu.
// Not part of the public ABI (that is include/nmfmu.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace nmfmu {

// ---- launch geometry shared between the host scheduler and the kernels ----

constexpr int kWtaWaves = 4;        // waves per workgroup in the W^T A pass
constexpr int kWtaCols = 128;       // columns of A per workgroup in that pass
constexpr int kAhtWaves = 8;        // waves per workgroup in the A H^T pass
constexpr int kAhtRowTiles = 2;     // 32-row tiles per workgroup in that pass
constexpr int kGramMaxBlocks = 64;  // partial Gram matrices before the final sum
constexpr int kFinMaxBlocks = 256;  // finisher blocks when they also emit Gram partials
constexpr int kMaxKTiles = 2;       // 32-wide rank tiles: k <= 64

inline int k_tiles(int k) { return (k + 31) / 32; }

// Which independent run a factor index belongs to when several runs on the same A
// are stacked side by side (id[c] for c < k); passed to kernels by value.
struct BlockMap {
    int on;
    unsigned char id[64];
};

// Row split of the W^T A pass: number of partial k x n results, rows in each.
int wta_splits(int64_t rows, int64_t n, int k);
// Largest split count of any rank up to k on these dimensions (workspace sizing).
int wta_splits_bound(int64_t rows, int64_t n, int k);
int64_t wta_rows_per_split(int64_t rows, int splits);

// The largest magnitudes of the columns meet in atomics; a block takes one of several copies, the reader the largest: 256
// blocks on the same 64 words cost 2 us.
constexpr int kPairCopies = 8;
// Planes of a factor (rows x k) in units of 8 rows x 1 column, ld columns per row group (see put_pairs).
struct PairFactor {
    void *units;              // pair_units_bytes(rows, ld)
    unsigned char *exps;      // pair_exps_bytes(rows, ld)
    unsigned *most;           // kPairCopies x ld words; zero before the planes are written
};

// ---- kernel launchers (all asynchronous on `st`; return hipGetLastError) ----

// G (k x k, ld k) = X^T X for X rows x k (row-major, ld k).
hipError_t launch_gram_w(const float *X, int64_t rows, int k, float *G, float *gpart,
                         unsigned *counters, hipStream_t st);
// The same for a long factor (millions of rows): up to kFinMaxBlocks blocks write partial tiles
// (tiles: kFinMaxBlocks sets), summed by launch_gram_sum.
// counters: as for launch_gram_w.
hipError_t launch_gram_w_wide(const float *X, int64_t rows, int k, float *G, float *tiles, unsigned *counters, hipStream_t st,
                              int ld = 0);
// G (k x k, ld k) = X X^T for X k x cols (row-major, ld cols).
hipError_t launch_gram_h(const float *X, int k, int64_t cols, float *G, float *gpart,
                         unsigned *counters, hipStream_t st);
// Ranks whose W^T A pass reads its factor as bf16 piece planes (planes_bytes(rows) bytes,
// written by launch_split_planes from the rows x k factor) instead of the floats.
inline bool wta_uses_planes(int k) { return k <= 64; }
size_t planes_bytes(int64_t rows);
// Largest rank for which launch_wta_pass on this A (n columns) reads only the planes, never
// the float factor W (which may then be null): 64 for aligned A with n % 4 == 0, else 32.
int wta_planes_only_width(const float *A, int64_t n);
hipError_t launch_split_planes(const float *X, int64_t rows, int k, void *planes, hipStream_t st);
// The same for columns c0 .. c0 + kc - 1 (kc <= 64; 32 factor slots per row group up to kc = 32, else 64)
// of X with leading dimension ld.
hipError_t launch_split_planes_slice(const float *X, int64_t rows, int64_t ld, int64_t c0, int kc,
                                     void *planes, hipStream_t st);
// ppart[s] (+)= W[r0_s:r1_s]^T A[r0_s:r1_s] for each row split s (k x n each).  `planes`:
// scratch of planes_bytes(rows) bytes (unused unless wta_uses_planes(k)); with planes_ready it
// already holds the planes of W, otherwise they are produced first.
hipError_t launch_wta_pass(const float *A, int64_t rows, int64_t n, int k, const float *W,
                           void *planes, bool planes_ready, float *ppart, int splits,
                           int64_t rows_per_split, bool accumulate, hipStream_t st,
                           const float *gtiles = nullptr, int nsets = 0, float *gsum = nullptr, bool two = false);
// two: A is read in turn with its transpose (what the last-level cache would have to keep).
// gtiles (optional): nsets sets of partial Gram tiles for rank k that the first workgroups of
// the pass add up into gsum (one set).
// Whether a pass marks A (rows x n) for early eviction; two: A^T is read in turn with it.
bool stream_a(int64_t rows, int64_t n, bool two = false);
// ---- pairs of halves ----
// Sizes of a factor's planes:
inline size_t pair_units_bytes(int64_t rows, int64_t ld) { return (size_t)((rows + 7) / 8) * 2 * ld * 16; }
inline size_t pair_exps_bytes(int64_t rows, int64_t ld) { return (size_t)((rows + 7) / 8) * ld; }
// X' of a matrix X (rows x cols, contracted over its rows): the same units, cut under one scale per column and kPairBlock
// rows; scale[(row / kPairBlock) * ld + column] = {its inverse, what the halves leave out of these rows' sum with a factor in its scaled range
// at most (see kSure)}; rows are filled up to whole blocks with zeros.
constexpr int kPairBlock = 128;
struct PairMatrix {
    void *units;              // pair_matrix_units(rows, ld) bytes
    float2 *scale;            // pair_matrix_scales(rows, ld) bytes
    int64_t ld;               // pair_matrix_ld(cols)
};
inline int64_t pair_matrix_ld(int64_t cols) { return (cols + 63) / 64 * 64; }
inline size_t pair_matrix_units(int64_t rows, int64_t ld) { return (size_t)((rows + kPairBlock - 1) / kPairBlock) * kPairBlock * ld * 4; }
inline size_t pair_matrix_scales(int64_t rows, int64_t ld) { return (size_t)((rows + kPairBlock - 1) / kPairBlock) * ld * sizeof(float2); }
// A' and (A^T)' of A (m x n, any alignment) in one reading; clear (optional): words to set to zero on the way.
hipError_t launch_cut_pairs(const float *A, int64_t m, int64_t n, const PairMatrix &a, const PairMatrix &at, unsigned *clear, int nclear,
                            hipStream_t st);
// Planes of X (rows x k, row-major) with ld columns per row group, ld >= k a multiple of 64; clear (optional): a like array of maxima to
// set to zero on the way.
hipError_t launch_split_pairs(const float *X, int64_t rows, int k, const PairFactor &f, int ld, hipStream_t st,
                              unsigned *clear = nullptr);
// One pass: F^T X for slices of `tiles` * 32 factors side by side, slice z with k[z] factors, its operands the z-th along the
// strides, its partials (splits x k[z] x n) at ppart + z * slice_ppart.
constexpr int kPairSlices = 16;
struct PairPass {
    PairFactor F;
    int ldf;
    int64_t slice_units, slice_exps, slice_most;      // from slice to slice: in units of 16 bytes, bytes and words
    PairMatrix X;
    // F and X themselves, for tiles whose sums the halves cannot hold: entries (i, c) of the first slice of F and (i, j) of X
    const float *f, *x;
    int64_t f_row, f_col, slice_f, x_row, x_col;
    unsigned *redo;                                   // pair_pass_tiles words, zero before a run's first pass: which tiles they are
    float *ppart;
    int64_t slice_ppart;
    int64_t rows, n, rps;                             // rps: rows of a split, a multiple of kPairBlock
    int splits, nslices;
    short k[kPairSlices];
    const float *gtiles;                              // optional, as in launch_wta_pass: tile sets to add up,
    int nsets;
    float *gsum;
    int64_t slice_gtiles, slice_gsum;
    unsigned *clear;                                  // optional: words to set to zero on the way
    int nclear;
};
// tiles: 2 or 4.  stream: X' is marked for early eviction.
hipError_t launch_pair_pass(const PairPass &p, int tiles, bool stream, hipStream_t st);
int pair_splits(int64_t rows, int64_t cols, int tiles, int nslices);
inline int64_t pair_pass_tiles(int64_t cols, int splits, int nslices) { return (cols + 255) / 256 * splits * nslices; }
inline int64_t pair_rows_per_split(int64_t rows, int splits)
{
    const int64_t blocks = (rows + kPairBlock - 1) / kPairBlock;
    return (blocks + splits - 1) / splits * kPairBlock;
}
// The same product with X itself, cut as it is loaded (16-byte aligned, n % 4 == 0), for all slices of 64 of k factors whose
// planes f (of F, rows x k) have ld columns per row group; partials of slice z at ppart + z * splits * 64 * n.  rps: a multiple of 16.
hipError_t launch_pair_slices(const float *X, int64_t rows, int64_t n, int k, const float *F, const PairFactor &f, int ld,
                              float *ppart, int splits, int64_t rps, hipStream_t st);
// Update of ranks above 64 from the partials of its products (see sliced_update_kernel).
struct SlicedUpdate {
    float *X, *Xt;                // k x len, len x k
    const float *num;             // numerator: slices of `width` factors, snum splits each
    const float *den;             // denominator: slices of 64, sden splits each
    int k, width, snum, sden;
    int64_t len;
    float eps;
    PairFactor F;                 // planes of Xt, ld columns per row group; maxima zero before
    int ld;
    unsigned *clear;              // other maxima to set to zero on the way
    int nclear;
};
hipError_t launch_sliced_update(const SlicedUpdate &a, hipStream_t st);
// P (k x cols) (+)= the sums over the splits, slices of 64 factors.
hipError_t launch_sum_partials_slices(const float *ppart, int splits, int k, int64_t cols, float *P, hipStream_t st,
                                      bool accumulate = false);
// P[e] (+)= sum_s ppart[s][e], e < count.
hipError_t launch_sum_partials(const float *ppart, int splits, int64_t count, float *P,
                               hipStream_t st, bool accumulate = false);
// X[e] <- X[e] * P[e] / (D[e] + eps), e < count.
hipError_t launch_mu_apply(float *X, const float *P, const float *D, float eps, int64_t count,
                           hipStream_t st);
// X (k x len) <- X * (sum_s part[s]) / (G X + eps), in place.  G is given complete (Gfull, ld k)
// or as nbin partial tiles (gin).  Optional: Xt (len x k) = new X^T; gout = partial Gram tiles
// of the new X, one set per block (factor_update_blocks(len) blocks); planes = the bf16 piece
// planes of the new X^T (planes_bytes(len) bytes; written only if wta_uses_planes(k)).
hipError_t launch_factor_update(float *X, float *Xt, const float *part, int splits,
                                const float *Gfull, const float *gin, int nbin, float *gout, int k,
                                int64_t len, float eps, hipStream_t st,
                                const BlockMap *map = nullptr, void *planes = nullptr,
                                double *dpart = nullptr);
// The same for runs on pairs: up to kPairGroup factors side by side, slice z's arrays the z-th along the strides; the pair planes
// of the new X^T (64 columns per row group) are written, the tile set gin is complete.  part null: only planes and gout of X.
constexpr int kPairGroup = 4;
struct FinisherSlices {
    float *X[kPairGroup], *Xt[kPairGroup];      // Xt: optional
    int k[kPairGroup];
    BlockMap bm[kPairGroup];
    int64_t part, gin, gout, units, exps;       // from slice to slice: floats, floats, floats, units, bytes
    PairFactor pairs;                           // most: kPairCopies x 64 words a slice
};
hipError_t launch_pair_update(const FinisherSlices &sl, int slices, const float *part, int splits, const float *gin, float *gout,
                              int64_t len, float eps, hipStream_t st, double *dpart = nullptr);
// Factors of up to 64 runs to (in) or from one slice: run r's W (m x k[r]) and rows `at` .. of Wt (ks x m), its H and the
// same rows of H of the slice (ks x n).
struct StackedRuns {
    float *W[64], *H[64];
    short k[64], at[64];
};
hipError_t launch_stack(const StackedRuns &runs, int count, bool in, float *Wt, float *H, int64_t m, int64_t n, hipStream_t st);
// dpart (with an updating launch): per block, the sum of numerator x new value over its entries
// (factor_update_blocks(len) doubles when gout is given, else one per chunk of 16, 32 or 64 columns).
// out[0] = sum of squares of X[0 .. count) in double; partial: 4096 doubles of scratch.
hipError_t launch_sumsq(const float *X, int64_t count, double *partial, double *out, hipStream_t st);
// out[0] = sqrt(max(0, normA2[0] - 2 sum(dpart[0 .. nb)) + <GW, GH>)).
// iters: of that many iterations, their nb shares and matrices one behind the other.
hipError_t launch_objective(const double *dpart, int nb, const float *GW, const float *GH, int k,
                            const double *normA2, double *out, hipStream_t st, int iters = 1);
int factor_update_blocks(int64_t len);
// G (k x k, ld k) = sum of nb sets of partial tiles.
hipError_t launch_gram_sum(const float *gpart, int nb, int k, float *G, hipStream_t st);
// Blocks (= partial tile sets) launch_gram_w uses for `rows` rows; with G == nullptr it only
// writes the partial tiles to gpart.
int gram_w_blocks(int64_t rows);
// W <- W * (A H^T) / (W GH + eps), in place, for `rows` rows of A and W.
// dpart (aht_pass_blocks(rows) doubles): per workgroup, the sum of (A H^T) x new W over its rows.
hipError_t launch_aht_pass(const float *A, int64_t rows, int64_t n, int k, const float *H,
                           const float *GH, float *W, float eps, hipStream_t st, double *dpart = nullptr);
int64_t aht_pass_blocks(int64_t rows);
// The same update for k <= 64 as one streaming pass over the row-major A (coalesced loads turned
// through LDS, products from pieces): planesH = piece planes of H^T (what launch_factor_update
// writes for X = H), GH = H H^T (k x k).  Also written: the piece planes of the new W (planesW),
// aht_rows_blocks(rows, k) tile sets of W^T W (gout) and dpart as above (aht_rows_blocks(rows, k)
// doubles).  gram_only: no pass and no update, only planesW and gout of W as it is.  dry: the
// pass and the update without the stores to W and planesW (timing runs).  aht_rows_can: the
// operands this kernel takes; aht_rows_ok: and a shape on which it fills the chip.
bool aht_rows_can(const float *A, int64_t n, int k);
bool aht_rows_ok(const float *A, int64_t m, int64_t n, int k);
// tiles: 32-row tiles per workgroup, 0: aht_rows_tiles(rows, k).  The count of workgroups grows with the rows only at a
// fixed number of tiles: a caller that sizes for one height and launches a smaller one names the tiles.
int aht_rows_tiles(int64_t rows, int k);
int aht_rows_blocks(int64_t rows, int k, int tiles = 0);
hipError_t launch_aht_rows(const float *A, int64_t rows, int64_t n, int k, const void *planesH,
                           const float *GH, float *W, void *planesW, float *gout, float eps, hipStream_t st,
                           bool gram_only = false, const BlockMap *map = nullptr, double *dpart = nullptr,
                           bool dry = false, int tiles = 0);
// Both products in one reading of A (few columns; see one_pass_kernel).  ppart: one k x n partial
// of W^T A per workgroup (one_pass_blocks of them), gout: one tile set of W^T W each, dpart
// (optional): one double each.  H H^T either complete (GH) or as nbh tile sets (ghsets).
// update: W is updated first, into Wnew (W itself, or null: not stored; planesH: piece planes of H^T);
// product: W^T A is wanted.
bool one_pass_ok(const float *A, int64_t n, int k);
int one_pass_blocks(int64_t rows, int64_t n);
hipError_t launch_one_pass(const float *A, int64_t rows, int64_t n, int k, const void *planesH, const float *GH,
                           const float *ghsets, int nbh, const float *W, float *Wnew, float *ppart, float *gout, float eps,
                           hipStream_t st, bool update, bool product, double *dpart = nullptr);

// psum (kShareGroups x k x n) = the nb shares of W^T A of a one-pass launch, added up group by group; G = the sum of its
// nb tile sets.
constexpr int kShareGroups = 16;
hipError_t launch_share_sum(const float *ppart, int nb, int k, int64_t n, float *psum, const float *gtiles, float *G, hipStream_t st);

// A whole run in one launch (see resident_kernel): up to 16 factors, R x C workgroups, each with a tile of A of
// 16 * tiles rows (tiles: 1, 2, 4) x 256 columns.
struct ResidentArgs {
    const float *A, *Win, *Hin;      // the matrix and the factors as handed in
    float *W, *H;                    // where they go
    float *part;                     // shares of W^T A and W^T W: per workgroup [16 tiles][16 factors][16 columns], lower triangle
    float *qpart;                    // shares of A H^T and H H^T: per workgroup [16 tiles rows][16], [16][16]
    float *hx;                       // the new H: [group of 8 columns][16 factors][8]
    float *wx;                       // the new W: [row][16]
    unsigned *sync;                  // kResidentLost ..; from kResidentHead on the letter boxes; zero at the start
    double *dpart;                   // optional, of the last W update: <A H^T, W> in R C shares,
    float *gout, *gh;                // R tile sets of W^T W (32 x 32 accumulator layout) and H H^T (k x k)
    float *gw;                       // optional: dpart and gh of every update of W, one behind the other, and here W^T W (k x k) of
                                     // all but the last (lead = 0, trail = 1, one launch)
    int64_t m, n;
    int k, R, C;
    float eps;
    int nprod;                       // updates of H; updates of W: between them,
    int lead, trail;                 // one before the first (lead) and one after the last (trail)
    long long patience;              // ticks until those that are there start without the others (0: the default)
    unsigned polls;                  // looks of one wait before the run is given up (0: the default)
};
// Words of sync, a cache line each:
constexpr int kResidentLost = 0,     // set when a wait has run out of looks
    kResidentHere = 32,              // workgroups that have reported in
    kResidentDeal = 64,              // how many of them are at work, from which iteration on
    kResidentArrived = 96, kResidentRelease = 128,     // barriers of a shared run
    kResidentOut = 160,              // workgroups that are done
    kResidentHead = 192;
constexpr unsigned kResidentOver = ~0u;     // in kResidentDeal: who comes now is not needed
constexpr int kResidentPRec = 4096 + 160;     // floats of a workgroup's record in part,
constexpr int resident_qrec(int tiles) { return 256 * (tiles + 1); }     // and in qpart
inline int64_t resident_sync_words(int64_t R, int64_t C) { return kResidentHead + R * C * (((R + 31) & ~(int64_t)31) + 32); }
int resident_tiles(int64_t m, int64_t n, int k);
// Iterations of one launch of R * C = `groups` workgroups: it holds its compute units for up to some 30 ms, or seconds if one
// workgroup does the run of all, and the flags (8 an iteration) stay far from their end.  Loading A again costs 10
// to 20 us.
inline int resident_piece(int64_t groups) { return (int)(groups > 256 ? 256 : groups < 16 ? 4096 : 65536 / groups); }
// Fills in R, C and the defaults and clears sync.  workgroups > 0: that many are launched instead of R * C (and share
// the run).
hipError_t launch_resident(const ResidentArgs &args, int tiles, hipStream_t st, int workgroups = 0);
// nprod updates of H, each followed by one of W, in launches of resident_piece iterations.
hipError_t launch_resident_run(const ResidentArgs &args, int tiles, hipStream_t st, int workgroups = 0);

// out[0] = sum of in[0 .. count), added in a fixed order (strided per thread, then the threads in order).
hipError_t launch_sum_f64(const double *in, int64_t count, double *out, hipStream_t st);

// out[0] = ||A - W H||_F; partial: residual_partials(m, n) doubles of scratch.
int64_t residual_partials(int64_t m, int64_t n);
hipError_t launch_residual(const float *A, int64_t m, int64_t n, int k, const float *W,
                           const float *H, double *partial, double *out, hipStream_t st);

// ---- CSR (everything in terms of Ht = H^T, n x k) ----
// X[i][:] <- X[i][:] * (sum over the stored entries (i, j, a) of a * T[j][:]) / (X[i][:] G + eps)
// for i < rows.  W update: (rowptr, colidx, vals) = CSR of A, T = Ht, G = H H^T, X = W.
// H update: the CSC arrays of A, T = W, G = W^T W, X = Ht.
constexpr int kCsrParts = 16384;      // row ranges (= wavefronts) of a sparse update launch
constexpr int64_t kRowCost = 8;       // work of a row besides its entries, in entries
constexpr int64_t kLongRow = 16384;   // rows with more entries go to a whole workgroup
constexpr int kCsrLongBlocks = 256;   // workgroups of it that take long rows, the first of the launch
constexpr int kCsrDparts = kCsrParts / 4 + kCsrLongBlocks;
// part[0 .. nparts]: row ranges of equal work; part[w] = first row r with
// rowptr[r] + kRowCost * r >= w * ceil((rowptr[m] + kRowCost * m) / nparts), part[nparts] = m.
hipError_t launch_csr_partition(const int64_t *rowptr, int64_t m, int nparts, int64_t *part,
                                hipStream_t st);
// list[0 .. min(*count, cap)): the rows with more than kLongRow entries (cap = nnz / kLongRow + 1 slots).
hipError_t launch_csr_long_rows(const int64_t *rowptr, int64_t m, int32_t *list, unsigned *count,
                                unsigned cap, hipStream_t st);
hipError_t launch_aht_csr(const int64_t *rowptr, const int32_t *colidx, const float *vals,
                          const int64_t *part, const int32_t *long_list, const unsigned *long_count,
                          int k, const float *Ht, const float *GH, float *W, float eps, int64_t nnz, int64_t rows,
                          int64_t trows, hipStream_t st, bool accumulate = false, double *dpart = nullptr, bool dry = false,
                          int ldx = 0, int ldt = 0);
// ldx, ldt: row lengths of W and of the table Ht (0: k).
// Row length at which a factor of k columns is gathered row by row without straddling cache lines (128
// bytes): whole fractions of a line up to 32, one and a half or two lines above.
inline int csr_row_length(int k) { return k <= 4 ? 4 : k <= 8 ? 8 : k <= 16 ? 16 : k <= 32 ? 32 : k <= 48 ? 48 : 64; }
hipError_t launch_restride(const float *src, int lds, float *dst, int ldd, int64_t rows, int k, hipStream_t st);
// nnz, rows, trows: lengths of the entry arrays, of W and of the table Ht (rows); row pointers and column
// indices beyond them are pulled to the edge, so that malformed input cannot cause a stray access.
// accumulate: X[i][:] += (gathered sum) instead of the update (GH unused).
// dpart (updating launch only; kCsrDparts doubles): per workgroup, the sum of
// gathered sum x new value over its rows, i.e. <A H^T, W_new> in pieces (objective monitor).
// dry (needs dpart): W is left alone and dpart gets <A H^T, W> of the factors as they are.
// X[i][:] <- X[i][:] * Num[i][:] / (X[i][:] G + eps), i < rows (X, Num rows x k).
hipError_t launch_row_update(float *X, const float *Num, const float *G, int k, int64_t rows, float eps,
                             hipStream_t st);
// out[i] = in[i] - base, i < count.
hipError_t launch_rebase_i64(const int64_t *in, int64_t count, int64_t base, int64_t *out, hipStream_t st);
hipError_t launch_fill_f32(float *p, int64_t count, float v, hipStream_t st);
// Column-ordered copy (colptr int64[n+1], rowidx int32[nnz], cvals float[nnz]) of a CSR matrix
// by a stable sort on the column index.  Scratch: sorted_cols int32[nnz], payload and
// sorted_payload uint64[nnz], sort_temp of csc_sort_temp_bytes(nnz, n) bytes.
// nnz < 2^31, m < 2^31.
size_t csc_sort_temp_bytes(int64_t nnz, int64_t n);
hipError_t launch_csc_build(const int64_t *rowptr, const int32_t *colidx, const float *vals,
                            int64_t m, int64_t n, int64_t nnz, int32_t *sorted_cols,
                            uint64_t *payload, uint64_t *sorted_payload, void *sort_temp,
                            size_t sort_temp_bytes, int64_t *colptr, int32_t *rowidx, float *cvals,
                            hipStream_t st, double *dup_part = nullptr);
// dup_part (csc_finish_blocks(nnz) doubles, at least one): their sum is what repeated (row, column)
// pairs add to the squared Frobenius norm of the matrix beyond the sum of the squared stored values.
int csc_finish_blocks(int64_t nnz);
// dst (rows x ld_dst) = the first `cols` columns of src (rows x ld_src); the columns of dst from
// `cols` on are set to zero.  Any alignment.
hipError_t launch_pad_copy(const float *src, int64_t ld_src, float *dst, int64_t ld_dst, int64_t rows, int64_t cols,
                           hipStream_t st);
// out = in^T (in: rows x cols, rows ldin apart).  ld > rows: rows of out are ld long, ldc > cols: out has ldc rows, what lies
// beyond in is zero; copy (optional): in with its rows extended to ldc, read once for both.
hipError_t launch_transpose(const float *in, int64_t rows, int64_t cols, float *out, hipStream_t st, int64_t ld = 0,
                            float *copy = nullptr, int64_t ldc = 0, int64_t ldin = 0);

}  // namespace nmfmu
