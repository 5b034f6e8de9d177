// C ABI of libnmfmu: argument checking, workspace management and the host-side
// schedules (resident loop, out-of-memory batch pipeline, CSR loop, ensemble).
// Public contract: include/nmfmu.h; the hooks of the tests: include/nmfmu_test.h.
#include "nmfmu.h"
#include "nmfmu_test.h"
#include "nmfmu_internal.h"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <vector>

using namespace nmfmu;

namespace {

thread_local char t_err[256] = "";

int fail(int status, const char *fmt, const char *detail = "")
{
    snprintf(t_err, sizeof(t_err), fmt, detail);
    return status;
}

#define NMF_HIP(call)                                                         \
    do {                                                                      \
        hipError_t e_ = (call);                                               \
        if (e_ != hipSuccess) return fail(NMF_EHIP, #call ": %s", hipGetErrorString(e_)); \
    } while (0)

constexpr size_t kAlign = 256;
size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

// ---- process-wide device memory owned by the library ----------------------

struct State {
    std::mutex mu;
    void *ws = nullptr;         // workspace in use (owned or caller's)
    size_t ws_bytes = 0;
    bool ws_owned = true;
    void *stage = nullptr;      // staging slots of the out-of-memory path
    size_t stage_bytes = 0;
    hipStream_t copy_stream = nullptr;
    hipEvent_t ev_copied[3] = {nullptr, nullptr, nullptr};
    hipEvent_t ev_freed[3] = {nullptr, nullptr, nullptr};
    hipEvent_t ev_entry = nullptr;
    double *pinned = nullptr;   // host memory that kernels write: results of blocking calls
    // rank-sliced out-of-memory path: up to kMaxSlots staging slots, factor rows copied back
    void *sl_stage = nullptr;
    size_t sl_stage_bytes = 0;
    hipStream_t back_stream = nullptr;
    hipEvent_t sl_copied[16] = {}, sl_done[16] = {}, sl_freed[16] = {};
};
State g;

// Workspace carving.  Slot 0 holds the arrival counters of the Gram kernels and
// must be zero whenever no kernel is running; the kernels restore that.
struct Carve {
    char *base;
    size_t off = 0;
    explicit Carve(void *b) : base(static_cast<char *>(b)) {}
    template <class T> T *take(size_t count)
    {
        T *p = reinterpret_cast<T *>(base + off);
        off = align_up(off + count * sizeof(T));
        return p;
    }
};

struct Common {
    unsigned *counters;
    float *gw, *gh, *gpart;
    float *gwp, *ghp;   // partial Gram tiles handed from one finisher to the next
    float *gws, *ghs;   // the same, added up by the pass that runs in between
};

Common carve_common(Carve &c, int k)
{
    Common r;
    r.counters = c.take<unsigned>(64);
    r.gw = c.take<float>((size_t)k * k);
    r.gh = c.take<float>((size_t)k * k);
    const int kt = k_tiles(k);
    r.gpart = c.take<float>((size_t)kGramMaxBlocks * kt * kt * 1024);
    r.gwp = c.take<float>((size_t)kFinMaxBlocks * kt * kt * 1024);
    r.ghp = c.take<float>((size_t)kFinMaxBlocks * kt * kt * 1024);
    r.gws = c.take<float>((size_t)kt * kt * 1024);
    r.ghs = c.take<float>((size_t)kt * kt * 1024);
    return r;
}

size_t common_bytes(int k)
{
    Carve c(nullptr);
    carve_common(c, k);
    return c.off;
}

int ensure_workspace(size_t need, void **out)
{
    if (g.ws && g.ws_bytes >= need) {
        *out = g.ws;
        return NMF_OK;
    }
    if (!g.ws_owned) return fail(NMF_ENOMEM, "caller-provided workspace is too small%s");
    if (g.ws) {
        NMF_HIP(hipDeviceSynchronize());
        NMF_HIP(hipFree(g.ws));
        g.ws = nullptr;
        g.ws_bytes = 0;
    }
    void *p = nullptr;
    hipError_t e = hipMalloc(&p, need);
    if (e != hipSuccess) return fail(NMF_ENOMEM, "hipMalloc(workspace): %s", hipGetErrorString(e));
    NMF_HIP(hipMemset(p, 0, kAlign));
    g.ws = p;
    g.ws_bytes = need;
    *out = p;
    return NMF_OK;
}

int check_common(const void *a, const void *w, const void *h, int64_t m, int64_t n, int32_t k,
                 int32_t iters, float eps, int32_t kmax = NMF_MU_MAX_K)
{
    if (!a || !w || !h) return fail(NMF_EINVAL, "null pointer%s");
    if (m < 1 || n < 1 || k < 1) return fail(NMF_EINVAL, "m, n, k must be >= 1%s");
    if (k > kmax) return fail(NMF_EUNSUPPORTED, "k exceeds the rank this entry point supports%s");
    if (iters < 0) return fail(NMF_EINVAL, "iters must be >= 0%s");
    if (!(eps >= 0.f) || !std::isfinite(eps)) return fail(NMF_EINVAL, "eps must be finite and >= 0%s");
    if (m > (int64_t)1 << 40 || n > (int64_t)1 << 31) return fail(NMF_EINVAL, "matrix too large%s");
    return NMF_OK;
}

// Plan of one resident dense run.  The fast plan ("mirrored") keeps A^T, W^T
// and H^T next to A, W, H, so that the A H^T product becomes the same
// row-streaming contraction as W^T A (on A^T with H^T: the two updates are
// transposes of each other) and its update the same finisher on W^T.  It costs
// one extra copy of A in the workspace; without it the direct A H^T kernel runs.
template <class T> T max3(T a, T b, T c) { return a > b ? (a > c ? a : c) : (b > c ? b : c); }

constexpr int kPairMost = kPairGroup * kPairCopies * 64;      // words of maxima of a factor's slices
enum class PairPlanes { none, there };      // of A, in the workspace

// The slices of a run on pairs: one of up to 64 factors, or up to kPairGroup stacks of runs on the same A side by side.
struct PairSlices {
    int count = 1;
    int k[kPairGroup];
    BlockMap bm[kPairGroup];
};

struct DensePlan {
    bool mirrored;
    bool one_pass = false;     // both products in one reading of A: ppart and planes2 only
    bool pairs = false;        // mirrored, with A and A^T as pairs of halves: ppart, pa, pt, fw, fh and Wt
    PairMatrix pa, pt;         // A' and (A^T)'
    PairFactor fw, fh;         // planes of W and of H^T
    float *Wts[kPairGroup], *Hs[kPairGroup];      // slices of stacked runs: W^T and H
    unsigned *redo;                               // tiles of either pass that are formed from the floats
    int64_t nredo[2];
    int64_t slice_gw, slice_gh, slice_gs;         // from slice to slice: tile sets of either factor, summed sets
    PairSlices sl;
    int resident = 0;          // the run in one launch, this many row tiles per workgroup: `res` and dry only
    ResidentArgs res;          // its exchange buffers
    float *dry;                // room for factors that a timing run leaves behind
    int64_t a_rows = 0;        // mirrored: rows of A itself when those of W are padded (0: the same)
    Common c;
    float *ppart;              // row-split partials of either pass
    float *psum;               // one-pass plan: the workgroups' shares of W^T A added up to kShareGroups
    void *planes;              // bf16 piece planes of the factor a pass contracts with
    void *planes2;             // row plan: piece planes of H^T (planes then holds those of W)
    float *At, *Wt, *Ht;       // mirrored only
    int s1, s2;                // row splits of the pass over A / over A^T
    int64_t rps1, rps2;
};

size_t dense_bytes(int64_t m, int64_t n, int k, bool mirrored)
{
    const size_t p1 = (size_t)wta_splits_bound(m, n, k) * k * n, p2 = (size_t)wta_splits_bound(n, m, k) * k * m;
    size_t b = common_bytes(k) + align_up(((mirrored && p2 > p1) ? p2 : p1) * sizeof(float)) +
               align_up(planes_bytes((mirrored && n > m) ? n : m)) + align_up(planes_bytes(n));
    if (mirrored)
        b += align_up((size_t)m * n * sizeof(float)) + align_up((size_t)k * m * sizeof(float)) +
             align_up((size_t)n * k * sizeof(float));
    return b;
}

DensePlan carve_dense(void *ws, int64_t m, int64_t n, int k, bool mirrored)
{
    Carve cv(ws);
    DensePlan p;
    p.mirrored = mirrored;
    p.c = carve_common(cv, k);
    p.s1 = wta_splits(m, n, k);
    p.rps1 = wta_rows_per_split(m, p.s1);
    p.s2 = wta_splits(n, m, k);
    p.rps2 = wta_rows_per_split(n, p.s2);
    const size_t p1 = (size_t)wta_splits_bound(m, n, k) * k * n, p2 = (size_t)wta_splits_bound(n, m, k) * k * m;
    p.ppart = cv.take<float>((mirrored && p2 > p1) ? p2 : p1);
    p.planes = cv.take<char>(planes_bytes((mirrored && n > m) ? n : m));
    p.planes2 = cv.take<char>(planes_bytes(n));
    p.At = p.Wt = p.Ht = nullptr;
    if (mirrored) {
        p.At = cv.take<float>((size_t)m * n);
        p.Wt = cv.take<float>((size_t)k * m);
        p.Ht = cv.take<float>((size_t)n * k);
    }
    return p;
}

// What launch_pair_pass takes: the rows of A' and (A^T)' are as long as A's rounded up.
bool pair_lengths_ok(int64_t m, int64_t n) { return pair_matrix_ld(m) < (int64_t)1 << 25 && pair_matrix_ld(n) < (int64_t)1 << 25; }

// 33 to 64 factors: the mirrored plan on pairs of halves.
bool pairs_ok(int64_t m, int64_t n, int k) { return k > 32 && k <= NMF_MU_MAX_K && pair_lengths_ok(m, n); }

// The iterations a call has to have for the cut (A read, two copies written; 300 us on 16384 x 8192, a transposed copy 200) to pay, without ->
// with it: 2000 x 1000, k = 40, one 67 -> 63 us; 16384 x 8192, k = 40, one 456 -> 524, two 685 -> 734, three 917 -> 943, k = 64, three 970 -> 968;
// 6000 x 4000, k = 64, two 226 -> 210; 100000 x 512, k = 40, two 491 -> 497.  A that would be copied first: 20011 x 9998, k = 50, two 1471 -> 1145.
// Of 178 shapes of 0.5 to 270 million entries, k = 33 to 64, narrow, short and square, none is slower by more than 1 percent from here on (with
// four iterations above 2^27, 193 and 257 million entries 5 and 4 percent).
int pairs_least(int64_t m, int64_t n, bool copy_a, bool rows_on_a_copy)
{
    if (m * n <= 1 << 22) return rows_on_a_copy ? 2 : 1;
    if (copy_a || m * n <= 1 << 25) return 2;
    return m * n <= 1 << 27 ? 4 : 6;
}

PairMatrix carve_pair_matrix(Carve &cv, int64_t rows, int64_t cols)
{
    PairMatrix x;
    x.ld = pair_matrix_ld(cols);
    x.units = cv.take<char>(pair_matrix_units(rows, x.ld));
    x.scale = cv.take<float2>(pair_matrix_scales(rows, x.ld) / sizeof(float2));
    return x;
}

PairFactor carve_pair_factor(Carve &cv, int64_t rows, int64_t ld, int slices)
{
    PairFactor f;
    f.units = cv.take<char>(pair_units_bytes(rows, ld) * slices);
    f.exps = cv.take<unsigned char>(pair_exps_bytes(rows, ld) * slices);
    f.most = nullptr;
    return f;
}

void set_slices(DensePlan *p, int64_t m, int64_t n, int count)
{
    p->sl.count = count;
    p->s1 = pair_splits(m, n, 2, count);
    p->rps1 = pair_rows_per_split(m, p->s1);
    p->s2 = pair_splits(n, m, 2, count);
    p->rps2 = pair_rows_per_split(n, p->s2);
}

// groups = 0: one run of k factors; else up to that many slices of stacked runs side by side.
DensePlan carve_pairs(Carve &cv, int64_t m, int64_t n, int k, int groups = 0)
{
    DensePlan p{};
    p.mirrored = p.pairs = true;
    p.c = carve_common(cv, k);
    size_t part = 0;
    p.nredo[0] = p.nredo[1] = 0;
    for (int c = 1; c <= (groups ? groups : 1); ++c) {
        set_slices(&p, m, n, c);
        const int64_t t1 = pair_pass_tiles(n, p.s1, c), t2 = pair_pass_tiles(m, p.s2, c);
        p.nredo[0] = t1 > p.nredo[0] ? t1 : p.nredo[0];
        p.nredo[1] = t2 > p.nredo[1] ? t2 : p.nredo[1];
        const size_t p1 = (size_t)p.s1 * c * (groups ? 64 : k) * n, p2 = (size_t)p.s2 * c * (groups ? 64 : k) * m;
        part = max3(part, p1, p2);
    }
    p.ppart = cv.take<float>(part);
    p.pa = carve_pair_matrix(cv, m, n);
    p.pt = carve_pair_matrix(cv, n, m);
    p.fw = carve_pair_factor(cv, m, 64, groups ? groups : 1);
    p.fh = carve_pair_factor(cv, n, 64, groups ? groups : 1);
    p.fw.most = cv.take<unsigned>(2 * kPairMost + p.nredo[0] + p.nredo[1]);
    p.fh.most = p.fw.most + kPairMost;
    p.redo = p.fh.most + kPairMost;
    if (!groups) {
        p.Wt = p.Wts[0] = cv.take<float>((size_t)k * m);
        p.sl.k[0] = k;
        return p;
    }
    p.slice_gw = p.slice_gh = (int64_t)kFinMaxBlocks * 4 * 1024;
    p.slice_gs = 4 * 1024;
    p.c.gwp = cv.take<float>((size_t)groups * p.slice_gw);
    p.c.ghp = cv.take<float>((size_t)groups * p.slice_gh);
    p.c.gws = cv.take<float>((size_t)groups * p.slice_gs);
    p.c.ghs = cv.take<float>((size_t)groups * p.slice_gs);
    for (int z = 0; z < groups; ++z) {
        p.Wts[z] = cv.take<float>((size_t)64 * m);
        p.Hs[z] = cv.take<float>((size_t)64 * n);
    }
    return p;
}

size_t pairs_bytes(int64_t m, int64_t n, int k, int groups = 0)
{
    Carve c(nullptr);
    carve_pairs(c, m, n, k, groups);
    return c.off;
}

// One-pass plan: up to this many shares and tile sets are added by the H update's workgroups themselves.
constexpr int kFewSets = 32;

size_t one_pass_bytes(int64_t m, int64_t n, int k)
{
    return common_bytes(k) + align_up((size_t)one_pass_blocks(m, n) * k * n * sizeof(float)) + align_up(planes_bytes(n)) +
           align_up(one_pass_blocks(m, n) > kFewSets ? (size_t)kShareGroups * k * n * sizeof(float) : 0);
}

DensePlan carve_resident(Carve &cv, int64_t m, int64_t n, int k, int tiles)
{
    const size_t R = (size_t)(m + 16 * tiles - 1) / (16 * tiles), C = (size_t)(n + 255) / 256, wgs = R * C;
    DensePlan p{};
    p.resident = tiles;
    p.c = carve_common(cv, k);
    p.res.part = cv.take<float>(wgs * kResidentPRec);
    p.res.qpart = cv.take<float>(wgs * resident_qrec(tiles));
    p.res.hx = cv.take<float>(C * 4096);
    p.res.wx = cv.take<float>(R * 256 * tiles);
    p.res.sync = cv.take<unsigned>((size_t)resident_sync_words((int64_t)R, (int64_t)C));
    p.dry = cv.take<float>((size_t)(m + n) * k);
    return p;
}

size_t resident_bytes(int64_t m, int64_t n, int k)
{
    Carve c(nullptr);
    carve_resident(c, m, n, k, resident_tiles(m, n, k));
    return c.off;
}

DensePlan carve_one_pass(void *ws, int64_t m, int64_t n, int k)
{
    Carve cv(ws);
    DensePlan p;
    p.mirrored = false;
    p.one_pass = true;
    p.c = carve_common(cv, k);
    p.ppart = cv.take<float>((size_t)one_pass_blocks(m, n) * k * n);
    p.planes2 = cv.take<char>(planes_bytes(n));
    p.psum = cv.take<float>(one_pass_blocks(m, n) > kFewSets ? (size_t)kShareGroups * k * n : 0);
    p.planes = nullptr;
    p.At = p.Wt = p.Ht = nullptr;
    p.s1 = p.s2 = 0;
    p.rps1 = p.rps2 = 0;
    return p;
}

// Which plan runs.  Up to 32 factors the row plan comes first wherever its kernel applies.  From 33
// to 64 factors its A H^T pass is slower than the W^T A kernel on a transposed copy (622 against
// 525 us on 32768 x 16384, 167 against 132 us on 16384 x 8192), so there the mirrored plan comes
// first and the row plan serves when the workspace cannot hold the copy.
static bool rows_plan_first(const float *A, int64_t m, int64_t n, int k) { return k <= 32 && aht_rows_ok(A, m, n, k); }
static bool rows_plan_runs(const float *A, int64_t m, int64_t n, int k, bool mirrored)
{
    // without a transposed copy the row kernel beats the direct one on every shape it can take
    return aht_rows_can(A, n, k) && (!mirrored || rows_plan_first(A, m, n, k));
}

// Workspace for a dense run: the mirrored plan if it can be had, else the small one.
int dense_workspace(const float *A, int64_t m, int64_t n, int k, void **ws, bool *mirrored)
{
    const size_t big = dense_bytes(m, n, k, true), small = dense_bytes(m, n, k, false);
    if (rows_plan_first(A, m, n, k)) {     // the row plan streams A itself for both products
        *mirrored = false;
        return ensure_workspace(small, ws);
    }
    if (g.ws && g.ws_bytes >= big) {
        *ws = g.ws;
        *mirrored = true;
        return NMF_OK;
    }
    if (g.ws_owned && ensure_workspace(big, ws) == NMF_OK) {
        *mirrored = true;
        return NMF_OK;
    }
    (void)hipGetLastError();
    *mirrored = false;
    return ensure_workspace(small, ws);
}

// Workspace for a plan that a smaller one can stand in for: whether it is there or can be had.  Under capture of
// `st` nothing is grown (that synchronises, which would end the capture), and the block that is held is not given
// up for one that the device has no room for (the calls that follow would free and allocate it every time).
bool have_workspace(size_t need, hipStream_t st)
{
    if (g.ws && g.ws_bytes >= need) return true;
    if (!g.ws_owned) return false;
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    size_t left = 0, total = 0;
    void *ws = nullptr;
    const bool can = hipStreamIsCapturing(st, &cap) == hipSuccess && cap == hipStreamCaptureStatusNone &&
                     hipMemGetInfo(&left, &total) == hipSuccess && need <= left + g.ws_bytes &&
                     ensure_workspace(need, &ws) == NMF_OK;
    if (!can) (void)hipGetLastError();
    return can;
}

// Whether a run comes first to the pair plan, among those that the workspace decides.
bool takes_pairs(const float *A, int64_t m, int64_t n, int k, int iters, float eps)
{
    const int64_t n4 = (n + 3) & ~(int64_t)3;
    const bool copy_a = (reinterpret_cast<uintptr_t>(A) & 15u) != 0 || n != n4;
    const bool rows_on_a_copy = copy_a && aht_rows_ok(nullptr, m, n4, k) && eps >= 1.17549435e-38f;
    return pairs_ok(m, n, k) && iters > 0 && iters >= pairs_least(m, n, copy_a, rows_on_a_copy);
}

// The plan of a dense run with `extra` bytes behind it (*tail): the resident plan where it applies, then the
// one-pass plan, else the row or the mirrored plan, else the small one; whatever the workspace can hold.
int dense_plan(const float *A, int64_t m, int64_t n, int k, size_t extra, hipStream_t st, DensePlan *p, char **tail, bool pairs)
{
    void *ws = nullptr;
    const int tiles = resident_tiles(m, n, k);
    size_t bytes = tiles ? resident_bytes(m, n, k) : 0;
    if (tiles && have_workspace(bytes + extra, st)) {
        Carve cv(g.ws);
        *p = carve_resident(cv, m, n, k, tiles);
        if (tail) *tail = static_cast<char *>(g.ws) + bytes;
        return NMF_OK;
    }
    bytes = one_pass_bytes(m, n, k);
    if (one_pass_ok(A, n, k) && have_workspace(bytes + extra, st)) {
        *p = carve_one_pass(g.ws, m, n, k);
    } else if (pairs && have_workspace(pairs_bytes(m, n, k) + extra, st)) {
        bytes = pairs_bytes(m, n, k);
        Carve cv(g.ws);
        *p = carve_pairs(cv, m, n, k);
    } else {
        bool mirrored = false;
        bytes = dense_bytes(m, n, k, true);
        if (!rows_plan_first(A, m, n, k) && have_workspace(bytes + extra, st)) {
            mirrored = true;
        } else {
            bytes = dense_bytes(m, n, k, false);
            if (int rc = ensure_workspace(bytes + extra, &ws)) return rc;
        }
        *p = carve_dense(g.ws, m, n, k, mirrored);
    }
    if (tail) *tail = static_cast<char *>(g.ws) + bytes;
    return NMF_OK;
}

// What a dense run works on: A, W and H as handed in, or copies the streaming kernels can take.
struct DenseRun {
    DensePlan p;
    const float *A;
    float *W, *H;
    int64_t m, n;
    char *tail;      // `extra` bytes
    bool have_at;    // the mirrored plan's A^T is made
};

// A that the streaming kernels cannot take as it is (base not 16-byte aligned, or n % 4 != 0) is
// copied once per call into an aligned array of n4 = n rounded up to 4 columns, the new columns
// zero, and H likewise: a zero column of A keeps its column of H at zero and adds nothing to any
// product, so the run on the copies is the run on A and H.  The one-pass and the row plan run on
// those.  The mirrored plan also reads A^T, whose columns are the rows of A: m is rounded up to 4
// in A^T and in a copy of W, whose new rows are zero and stay zero for the same reason.
// Only with a normal positive eps (with eps = 0 a zero column gives 0 / 0), and where the workspace
// can hold the copies.  Microseconds per iteration, 20 or 30 per call, copies included, against the
// plan that ran before (the kernels for any alignment, or the row plan at 33 factors and up):
// 32768 x 16382, k = 32: 1020 -> 800 (row plan); mirrored plan: 20011 x 9998, k = 50 634 -> 424;
// 20011 x 10000, k = 40 788 -> 409; 2001 x 6001, k = 50 169 -> 68; 5001 x 3000, k = 12 62 -> 50;
// one iteration: 5001 x 3001, k = 12 117 -> 119, k = 40 192 -> 124.
// The mirrored plan on pairs of halves takes any A as it is; with `aligned` it works on the copies all the same
// (a caller that evaluates the objective on r->A).
int open_run(const float *A, int64_t m, int64_t n, int k, float *W, float *H, int iters, float eps, size_t extra,
             hipStream_t st, DenseRun *r, bool aligned = false)
{
    const int64_t n4 = (n + 3) & ~(int64_t)3, m4 = (m + 3) & ~(int64_t)3;
    const bool copy_a = (reinterpret_cast<uintptr_t>(A) & 15u) != 0 || n != n4;
    const size_t copies = (copy_a ? align_up((size_t)m * n4 * sizeof(float)) : 0) +
                          (n != n4 ? align_up((size_t)k * n4 * sizeof(float)) : 0);
    *r = DenseRun{};
    r->A = A;
    r->W = W;
    r->H = H;
    r->m = m;
    r->n = n;
    bool padded = false, pad_w = false;
    size_t base = 0;
    if (resident_tiles(m, n, k) && have_workspace(resident_bytes(m, n, k) + extra, st))      // takes any A
        return dense_plan(A, m, n, k, extra, st, &r->p, &r->tail, false);
    const bool can_rows = aht_rows_ok(nullptr, m, n4, k), copies_can = eps >= 1.17549435e-38f && iters > 0;
    const bool pairs = takes_pairs(A, m, n, k, iters, eps);
    if (pairs) {
        if (aligned && copy_a && copies_can && have_workspace(pairs_bytes(m, n4, k) + copies + extra, st)) {
            base = pairs_bytes(m, n4, k);
            Carve cv(g.ws);
            r->p = carve_pairs(cv, m, n4, k);
            padded = true;
        } else if (have_workspace(pairs_bytes(m, n, k) + extra, st)) {
            return dense_plan(A, m, n, k, extra, st, &r->p, &r->tail, true);
        }
    }
    if (!padded && copies_can && (copy_a || m != m4)) {
        const bool one = one_pass_ok(nullptr, n4, k), rows = rows_plan_first(nullptr, m, n4, k);
        if (one || rows) {
            if (copy_a) {
                base = one_pass_bytes(m, n4, k);
                if (one && have_workspace(base + copies + extra, st)) {
                    r->p = carve_one_pass(g.ws, m, n4, k);
                    padded = true;
                } else if (rows) {
                    base = dense_bytes(m, n4, k, false);
                    if ((padded = have_workspace(base + copies + extra, st))) r->p = carve_dense(g.ws, m, n4, k, false);
                }
            }
        } else {
            pad_w = m != m4;
            base = dense_bytes(m4, n4, k, true);
            const size_t wcopy = pad_w ? align_up((size_t)m4 * k * sizeof(float)) : 0;
            if ((iters > 1 || !copy_a || !can_rows) && (padded = have_workspace(base + copies + wcopy + extra, st))) {
                r->p = carve_dense(g.ws, m4, n4, k, true);
                r->p.a_rows = m;
                r->m = m4;
            } else {
                pad_w = false;
                base = dense_bytes(m, n4, k, false);
                if (copy_a && can_rows && (padded = have_workspace(base + copies + extra, st)))
                    r->p = carve_dense(g.ws, m, n4, k, false);
            }
        }
    }
    if (!padded) return dense_plan(A, m, n, k, extra, st, &r->p, &r->tail, pairs);
    Carve cv(static_cast<char *>(g.ws) + base);
    if (copy_a) {
        float *Ap = cv.take<float>((size_t)m * n4);
        if (r->p.mirrored && !r->p.pairs) NMF_HIP(launch_transpose(A, m, n, r->p.At, st, r->m, Ap, n4));
        else NMF_HIP(launch_pad_copy(A, n, Ap, n4, m, n, st));
        r->have_at = r->p.mirrored && !r->p.pairs;
        r->A = Ap;
        r->n = n4;
    }
    if (n != n4) {
        r->H = cv.take<float>((size_t)k * n4);
        NMF_HIP(launch_pad_copy(H, n, r->H, n4, k, n, st));
    }
    if (pad_w) {
        r->W = cv.take<float>((size_t)m4 * k);
        NMF_HIP(launch_pad_copy(W, k, r->W, k, m, k, st));
        NMF_HIP(launch_fill_f32(r->W + m * k, (m4 - m) * k, 0.f, st));
    }
    r->tail = cv.base + cv.off;
    return NMF_OK;
}

// The factors of a run on copies go back to the caller's.
int close_run(const DenseRun &r, int k, float *W, float *H, int64_t m, int64_t n, hipStream_t st)
{
    if (r.H != H) NMF_HIP(launch_pad_copy(r.H, r.n, H, n, k, n, st));
    if (r.W != W) NMF_HIP(launch_pad_copy(r.W, k, W, k, m, k, st));
    return NMF_OK;
}

// A dense_body on this plan streams A itself for both products and leaves the plan's A^T alone.
bool takes_row_plan(const DensePlan &p, const float *A, int64_t m, int64_t n, int k)
{
    return !p.one_pass && !p.resident && !p.pairs && !p.a_rows && rows_plan_runs(A, m, n, k, p.mirrored);
}

constexpr int kDenseKernels = 6;

// Per-iteration objective of a dense run (device memory): out[it] after iteration it.
struct Monitor {
    double *dpart;      // kFinMaxBlocks: <numerator, new W> per finisher block (batch times that, batch > 1)
    double *normA2;     // [0] = ||A||_F^2, followed by 4096 doubles of scratch for its sum
    double *out;        // iters values
    double *res;        // direct plan: scratch of the tiled evaluation (ceil(m / 32) + 1 doubles)
    bool last_only;     // only the last iteration of the call reports (into out[0])
    int batch = 1;      // resident plan: iterations per launch that reports them all, with
    float *gw = nullptr, *gh = nullptr;      // batch Gram matrices each
};
// 32 iterations: what a launch costs beyond its iterations (20 us) no longer shows.
constexpr int kMonitored = 32;
size_t monitored_bytes(int batch, int k)
{
    return align_up((size_t)(batch - 1) * kFinMaxBlocks * sizeof(double)) + 2 * align_up((size_t)batch * k * k * sizeof(float));
}

// A pass of a run on pairs: over A' with the planes of W, or (transposed) over (A^T)' with those of H^T.  The maxima of the planes
// that come next are set to zero on the way: those planes were read by the pass before.
hipError_t pass_over(const DensePlan &p, const float *A, int64_t m, int64_t n, bool transposed, int nsets, hipStream_t st)
{
    const Common &c = p.c;
    PairPass a{};
    a.f = transposed ? p.Hs[0] : p.Wts[0];
    a.f_row = 1;
    a.f_col = transposed ? n : m;
    a.slice_f = p.sl.count > 1 ? (transposed ? p.Hs[1] : p.Wts[1]) - a.f : 0;
    a.x = A;
    a.x_row = transposed ? 1 : n;
    a.x_col = transposed ? n : 1;
    a.redo = p.redo + (transposed ? p.nredo[0] : 0);
    a.F = transposed ? p.fh : p.fw;
    a.ldf = 64;
    a.slice_units = (int64_t)(pair_units_bytes(transposed ? n : m, 64) / 16);
    a.slice_exps = (int64_t)pair_exps_bytes(transposed ? n : m, 64);
    a.slice_most = kPairCopies * 64;
    a.X = transposed ? p.pt : p.pa;
    a.ppart = p.ppart;
    a.rows = transposed ? n : m;
    a.n = transposed ? m : n;
    a.splits = transposed ? p.s2 : p.s1;
    a.rps = transposed ? p.rps2 : p.rps1;
    a.slice_ppart = (int64_t)a.splits * 64 * a.n;
    a.nslices = p.sl.count;
    for (int z = 0; z < p.sl.count; ++z) a.k[z] = (short)p.sl.k[z];
    if (nsets) {
        a.gtiles = transposed ? c.ghp : c.gwp;
        a.slice_gtiles = transposed ? p.slice_gh : p.slice_gw;
        a.nsets = nsets;
        a.gsum = transposed ? c.ghs : c.gws;
        a.slice_gsum = p.slice_gs;
        a.clear = transposed ? p.fw.most : p.fh.most;
        a.nclear = p.sl.count * kPairCopies * 64;
    }
    return launch_pair_pass(a, 2, stream_a(m, n, true), st);
}

// The update behind that pass: of H, or (transposed) of W^T, whose rows go to W if that is given.  start: no update, the planes and tiles
// of W^T as it is, with the summation order of an updating launch (so that a run split into two calls equals one call).
hipError_t update_behind(const DensePlan &p, int64_t m, int64_t n, bool transposed, bool start, float *W, float eps, hipStream_t st,
                         double *dpart = nullptr)
{
    const Common &c = p.c;
    FinisherSlices f{};
    for (int z = 0; z < p.sl.count; ++z) {
        f.X[z] = transposed ? p.Wts[z] : p.Hs[z];
        f.k[z] = p.sl.k[z];
        f.bm[z] = p.sl.bm[z];
    }
    f.Xt[0] = W;
    const int64_t len = transposed ? m : n;
    f.part = (int64_t)(transposed ? p.s2 : p.s1) * 64 * len;
    f.gin = p.slice_gs;
    f.gout = transposed ? p.slice_gw : p.slice_gh;
    f.units = (int64_t)(pair_units_bytes(len, 64) / 16);
    f.exps = (int64_t)pair_exps_bytes(len, 64);
    f.pairs = transposed ? p.fw : p.fh;
    return launch_pair_update(f, p.sl.count, start ? nullptr : p.ppart, start ? 0 : (transposed ? p.s2 : p.s1),
                              start ? nullptr : (transposed ? c.ghs : c.gws), transposed ? c.gwp : c.ghp, len, eps, st, dpart);
}

// A run on pairs, or a group of stacked ones: p.Wts and p.Hs hold the factors; W: takes the rows of the first W at the end.
// As the mirrored plan, on A' and (A^T)'; the finishers write the planes that the next pass contracts with.
int pairs_body(const float *A, int64_t m, int64_t n, float *W, int iters, float eps, const DensePlan &p, hipStream_t st,
               PairPlanes cut, hipEvent_t *ev = nullptr, const Monitor *mon = nullptr)
{
    const Common &c = p.c;
    const int64_t words = 2 * kPairMost + p.nredo[0] + p.nredo[1];      // maxima, and all tiles are formed from pairs at first
    if (cut == PairPlanes::none) NMF_HIP(launch_cut_pairs(A, m, n, p.pa, p.pt, p.fw.most, (int)words, st));
    else NMF_HIP(launch_fill_f32(reinterpret_cast<float *>(p.fw.most), words, 0.f, st));
    NMF_HIP(update_behind(p, m, n, true, true, nullptr, eps, st));
    const int nbw = factor_update_blocks(m), nbh = factor_update_blocks(n), k = p.sl.k[0];
    if (ev) NMF_HIP(hipEventRecord(*ev++, st));
    for (int it = 0; it < iters; ++it) {
        if (ev) NMF_HIP(hipEventRecord(*ev++, st));
        NMF_HIP(pass_over(p, A, m, n, false, nbw, st));
        if (ev) NMF_HIP(hipEventRecord(*ev++, st));
        NMF_HIP(update_behind(p, m, n, false, false, nullptr, eps, st));
        if (ev) NMF_HIP(hipEventRecord(*ev++, st));
        if (ev) NMF_HIP(hipEventRecord(*ev++, st));
        NMF_HIP(pass_over(p, A, m, n, true, nbh, st));
        if (ev) NMF_HIP(hipEventRecord(*ev++, st));
        const bool report = mon && (!mon->last_only || it == iters - 1);
        NMF_HIP(update_behind(p, m, n, true, false, it == iters - 1 ? W : nullptr, eps, st, report ? mon->dpart : nullptr));
        if (ev) NMF_HIP(hipEventRecord(*ev++, st));
        if (report) {
            NMF_HIP(launch_gram_sum(c.gwp, nbw, k, c.gw, st));
            NMF_HIP(launch_gram_sum(c.ghs, 1, k, c.gh, st));
            NMF_HIP(launch_objective(mon->dpart, nbw, c.gw, c.gh, k, mon->normA2, mon->out + (mon->last_only ? 0 : it), st));
        }
    }
    return NMF_OK;
}

// One resident dense run on `st`.  With `ev` (kDenseKernels * iters + 1 events)
// an event is recorded before the first kernel of the loop and after every
// kernel, for per-kernel timing; slots of kernels a plan does not use collapse
// to zero duration.  `a_is_mirrored`: At already holds this A's transpose.
int dense_body(const float *A, int64_t m, int64_t n, int k, float *W, float *H, int iters,
               float eps, const DensePlan &p, hipStream_t st, bool a_is_mirrored = false,
               hipEvent_t *ev = nullptr, const BlockMap *map = nullptr, const Monitor *mon = nullptr)
{
    const Common &c = p.c;
    if (p.resident) {
        if (iters < 1) return NMF_OK;
        ResidentArgs a = p.res;
        a.A = A;
        a.Win = a.W = W;
        a.Hin = a.H = H;
        a.m = m;
        a.n = n;
        a.k = k;
        a.eps = eps;
        if (ev) {      // the halves of an iteration one by one: the same sums
            NMF_HIP(hipEventRecord(*ev++, st));
            for (int it = 0; it < iters; ++it)
                for (int slot = 0; slot < kDenseKernels; ++slot) {
                    a.nprod = slot == 1;
                    a.lead = slot == 4;
                    if (slot == 1 || slot == 4) NMF_HIP(launch_resident(a, p.resident, st));
                    NMF_HIP(hipEventRecord(*ev++, st));
                }
            return NMF_OK;
        }
        const bool all = mon && !mon->last_only;
        const int step = all ? mon->batch : iters;
        const int R = (int)((m + 16 * p.resident - 1) / (16 * p.resident)), C = (int)((n + 255) / 256);
        float *gw = c.gw;
        if (mon) a.dpart = mon->dpart, a.gout = c.gwp, a.gh = c.gh;
        if (all && step > 1) a.gw = gw = mon->gw, a.gh = mon->gh;
        for (int i = 0; i < iters; i += step) {
            const int some = iters - i < step ? iters - i : step, report = all ? some : 1;
            a.nprod = some;
            NMF_HIP(launch_resident_run(a, p.resident, st));
            if (mon) {
                NMF_HIP(launch_gram_sum(c.gwp, R, k, gw + (size_t)(report - 1) * k * k, st));
                NMF_HIP(launch_objective(mon->dpart, R * C, gw, a.gh, k, mon->normA2, mon->out + i, st, report));
            }
        }
        return NMF_OK;
    }
    if (p.one_pass) {
        // Per iteration: the pass that finishes the previous one (A H^T, the W update) and leaves W^T A
        // and W^T W of the new W as one share per workgroup, then the H update; the last W update has a
        // pass of its own without W^T A.  Up to kFewSets tile sets are added by the consumer's
        // workgroups themselves, more by a launch of their own (for W^T W: with the shares of W^T A).
        const int nbw = one_pass_blocks(m, n), nbh = factor_update_blocks(n);
        auto pass = [&](int done, bool product) -> int {       // `done` H updates so far
            const bool report = done && mon && (!mon->last_only || done == iters);
            const bool whole = nbh > kFewSets;      // whether or not the objective is wanted: same bits
            if (done && (whole || report)) NMF_HIP(launch_gram_sum(c.ghp, nbh, k, c.gh, st));
            NMF_HIP(launch_one_pass(A, m, n, k, p.planes2, whole ? c.gh : nullptr, c.ghp, nbh, W, W, p.ppart, c.gwp, eps, st,
                                    done > 0, product, report ? mon->dpart : nullptr));
            if (report) {
                NMF_HIP(launch_gram_sum(c.gwp, nbw, k, c.gw, st));
                NMF_HIP(launch_objective(mon->dpart, nbw, c.gw, c.gh, k, mon->normA2,
                                         mon->out + (mon->last_only ? 0 : done - 1), st));
            }
            return NMF_OK;
        };
        if (ev) NMF_HIP(hipEventRecord(*ev++, st));
        for (int it = 0; it < iters; ++it) {
            if (ev) NMF_HIP(hipEventRecord(*ev++, st));
            if (int rc = pass(it, true)) return rc;
            if (ev) NMF_HIP(hipEventRecord(*ev++, st));
            const bool many = nbw > kFewSets;
            if (many) NMF_HIP(launch_share_sum(p.ppart, nbw, k, n, p.psum, c.gwp, c.gw, st));
            NMF_HIP(launch_factor_update(H, nullptr, many ? p.psum : p.ppart, many ? kShareGroups : nbw, many ? c.gw : nullptr, c.gwp,
                                         nbw, c.ghp, k, n, eps, st, map, p.planes2));
            if (ev) NMF_HIP(hipEventRecord(*ev++, st));
            if (ev) NMF_HIP(hipEventRecord(*ev++, st));
            if (it == iters - 1)
                if (int rc = pass(iters, false)) return rc;
            if (ev) NMF_HIP(hipEventRecord(*ev++, st));
            if (ev) NMF_HIP(hipEventRecord(*ev++, st));
        }
        return NMF_OK;
    }
    if (p.pairs) {
        const PairPlanes cut = a_is_mirrored ? PairPlanes::there : PairPlanes::none;
        NMF_HIP(launch_transpose(W, m, k, p.Wt, st));
        DensePlan q = p;
        q.Hs[0] = H;
        if (map) q.sl.bm[0] = *map;
        else q.sl.bm[0].on = 0;
        return pairs_body(A, m, n, W, iters, eps, q, st, cut, ev, mon);
    }
    // The plan may have been carved for a larger rank (stacks of an ensemble): split
    // counts follow the rank actually run; the partial buffer holds the largest case.
    const int s1 = wta_splits(m, n, k), s2 = wta_splits(n, m, k);
    const int64_t rps1 = wta_rows_per_split(m, s1), rps2 = wta_rows_per_split(n, s2);
    if (takes_row_plan(p, A, m, n, k)) {
        // Row plan: both products stream the row-major A.  The W^T A pass reads the piece
        // planes of W and, on the side, adds the tile sets of W^T W up; the H update writes
        // the planes of H^T and the tile sets of H H^T, which a small launch adds up; the A H^T pass
        // with the fused W update writes the planes of the new W and the tile sets of its W^T W.
        const int nbw = aht_rows_blocks(m, k), nbh = factor_update_blocks(n);
        // up to 16 sets are one trip to L2 for the finisher itself: the side job would cost a small pass
        // more than that (256 x 192, k = 4: 5.9 instead of 4.8 us)
        const bool few = nbw <= 16;
        // planes and W^T W of the W handed in, with the summation order of an updating launch
        NMF_HIP(launch_aht_rows(nullptr, m, n, k, nullptr, nullptr, W, p.planes, c.gwp, eps, st, true));
        if (ev) NMF_HIP(hipEventRecord(*ev++, st));
        for (int it = 0; it < iters; ++it) {
            if (ev) NMF_HIP(hipEventRecord(*ev++, st));
            NMF_HIP(launch_wta_pass(A, m, n, k, W, p.planes, true, p.ppart, s1, rps1, false, st, few ? nullptr : c.gwp, nbw, c.gws));
            if (ev) NMF_HIP(hipEventRecord(*ev++, st));
            NMF_HIP(launch_factor_update(H, nullptr, p.ppart, s1, nullptr, few ? c.gwp : c.gws, few ? nbw : 1, c.ghp, k, n, eps, st, map, p.planes2));
            if (ev) NMF_HIP(hipEventRecord(*ev++, st));
            NMF_HIP(launch_gram_sum(c.ghp, nbh, k, c.gh, st));
            if (ev) NMF_HIP(hipEventRecord(*ev++, st));
            const bool report = mon && (!mon->last_only || it == iters - 1);
            NMF_HIP(launch_aht_rows(A, m, n, k, p.planes2, c.gh, W, p.planes, c.gwp, eps, st, false, map,
                                    report ? mon->dpart : nullptr));
            if (ev) NMF_HIP(hipEventRecord(*ev++, st));
            if (ev) NMF_HIP(hipEventRecord(*ev++, st));
            if (report) {
                NMF_HIP(launch_gram_sum(c.gwp, nbw, k, c.gw, st));
                NMF_HIP(launch_objective(mon->dpart, nbw, c.gw, c.gh, k, mon->normA2,
                                         mon->out + (mon->last_only ? 0 : it), st));
            }
        }
        return NMF_OK;
    }
    const int64_t ma = p.a_rows ? p.a_rows : m;
    if (p.mirrored) {
        if (!a_is_mirrored) NMF_HIP(launch_transpose(A, ma, n, p.At, st, m));
        NMF_HIP(launch_transpose(W, m, k, p.Wt, st));
        NMF_HIP(launch_transpose(H, k, n, p.Ht, st));
    }
    if (p.mirrored) {
        // W^T W of the initial W as partial tiles, from the finisher in its Gram-only
        // mode (same bits as the tiles a preceding W update would have left, so that
        // a run split into two calls equals one call); afterwards every finisher
        // hands the Gram tiles of its new factor to the next one.
        NMF_HIP(launch_factor_update(p.Wt, nullptr, nullptr, 0, nullptr, nullptr, 0, c.gwp, k, m, eps, st, nullptr, p.planes));
        const int nbw = factor_update_blocks(m), nbh = factor_update_blocks(n);
        if (ev) NMF_HIP(hipEventRecord(*ev++, st));
        // The tiles of a finisher are needed, summed, by the next finisher; the pass that runs
        // in between adds them up on the side (its first workgroups): no launch of its own.
        for (int it = 0; it < iters; ++it) {
            if (ev) NMF_HIP(hipEventRecord(*ev++, st));
            NMF_HIP(launch_wta_pass(A, ma, n, k, W, p.planes, true, p.ppart, s1, rps1, false, st, c.gwp, nbw, c.gws, true));
            if (ev) NMF_HIP(hipEventRecord(*ev++, st));
            NMF_HIP(launch_factor_update(H, p.Ht, p.ppart, s1, nullptr, c.gws, 1, c.ghp, k, n, eps, st, map, p.planes));
            if (ev) NMF_HIP(hipEventRecord(*ev++, st));
            if (ev) NMF_HIP(hipEventRecord(*ev++, st));
            NMF_HIP(launch_wta_pass(p.At, n, m, k, p.Ht, p.planes, true, p.ppart, s2, rps2, false, st, c.ghp, nbh, c.ghs, true));
            if (ev) NMF_HIP(hipEventRecord(*ev++, st));
            const bool report = mon && (!mon->last_only || it == iters - 1);
            NMF_HIP(launch_factor_update(p.Wt, W, p.ppart, s2, nullptr, c.ghs, 1, c.gwp, k, m, eps, st, map, p.planes,
                                         report ? mon->dpart : nullptr));
            if (ev) NMF_HIP(hipEventRecord(*ev++, st));
            if (report) {
                // ||A - W H||_F from what this W update leaves behind: <A H^T, W>, H H^T, W^T W
                NMF_HIP(launch_gram_sum(c.gwp, nbw, k, c.gw, st));
                NMF_HIP(launch_gram_sum(c.ghs, 1, k, c.gh, st));
                NMF_HIP(launch_objective(mon->dpart, nbw, c.gw, c.gh, k, mon->normA2,
                                         mon->out + (mon->last_only ? 0 : it), st));
            }
        }
        return NMF_OK;
    }
    if (ev) NMF_HIP(hipEventRecord(*ev++, st));
    for (int it = 0; it < iters; ++it) {
        NMF_HIP(launch_gram_w(W, m, k, c.gw, c.gpart, c.counters, st));
        NMF_HIP(launch_split_planes(W, m, k, p.planes, st));
        if (ev) NMF_HIP(hipEventRecord(*ev++, st));
        NMF_HIP(launch_wta_pass(A, m, n, k, W, p.planes, true, p.ppart, s1, rps1, false, st));
        if (ev) NMF_HIP(hipEventRecord(*ev++, st));
        NMF_HIP(launch_factor_update(H, nullptr, p.ppart, s1, c.gw, nullptr, 0, nullptr, k, n, eps, st));
        if (ev) NMF_HIP(hipEventRecord(*ev++, st));
        NMF_HIP(launch_gram_h(H, k, n, c.gh, c.gpart, c.counters, st));
        if (ev) NMF_HIP(hipEventRecord(*ev++, st));
        NMF_HIP(launch_aht_pass(A, m, n, k, H, c.gh, W, eps, st));
        if (ev) NMF_HIP(hipEventRecord(*ev++, st));
        if (ev) NMF_HIP(hipEventRecord(*ev++, st));
        if (mon && (!mon->last_only || it == iters - 1))   // exact, tiled
            NMF_HIP(launch_residual(A, m, n, k, W, H, mon->res + 1, mon->out + (mon->last_only ? 0 : it), st));
    }
    return NMF_OK;
}

size_t csr_bytes(int64_t n, int64_t nnz, int k)
{
    return common_bytes(k) + align_up((size_t)n * k * sizeof(float)) +      // Ht
           align_up((size_t)(n + 1) * sizeof(int64_t)) +                      // column pointers
           align_up((size_t)nnz * sizeof(int32_t)) + align_up((size_t)nnz * sizeof(float)) +
           2 * align_up((size_t)(kCsrParts + 1) * sizeof(int64_t)) +          // row ranges, CSR and CSC
           2 * align_up((size_t)(nnz / kLongRow + 2) * sizeof(int32_t)) +     // long-row lists
           kAlign +                                                           // their counts
           // scratch of the one-time sort that builds the column-ordered copy
           align_up((size_t)nnz * sizeof(int32_t)) + 2 * align_up((size_t)nnz * sizeof(uint64_t)) +
           align_up(nnz ? csc_sort_temp_bytes(nnz, n) : 0);
}

// Column-ordered copy of a CSR matrix into caller-provided arrays (test hook); the sort
// scratch is transient (allocated and freed here, which synchronises with `st`).
int build_csc(const int64_t *rowptr, const int32_t *colidx, const float *vals, int64_t m,
              int64_t n, int64_t nnz, int64_t *colptr, int32_t *rowidx, float *cvals, hipStream_t st)
{
    const size_t idx_bytes = align_up((size_t)nnz * sizeof(int32_t));
    const size_t pl_bytes = align_up((size_t)nnz * sizeof(uint64_t));
    const size_t temp_bytes = nnz ? csc_sort_temp_bytes(nnz, n) : 0;
    void *scratch = nullptr;
    if (nnz) {
        hipError_t e = hipMalloc(&scratch, idx_bytes + 2 * pl_bytes + align_up(temp_bytes) + kAlign);
        if (e != hipSuccess) return fail(NMF_ENOMEM, "hipMalloc(sort scratch): %s", hipGetErrorString(e));
    }
    char *sp = static_cast<char *>(scratch);
    hipError_t e = launch_csc_build(rowptr, colidx, vals, m, n, nnz,
                                    reinterpret_cast<int32_t *>(sp + 2 * pl_bytes),
                                    reinterpret_cast<uint64_t *>(sp),
                                    reinterpret_cast<uint64_t *>(sp + pl_bytes),
                                    sp + 2 * pl_bytes + idx_bytes, temp_bytes, colptr, rowidx, cvals, st);
    hipError_t e2 = scratch ? hipStreamSynchronize(st) : hipSuccess;
    if (scratch) (void)hipFree(scratch);
    if (e != hipSuccess) return fail(NMF_EHIP, "csc build: %s", hipGetErrorString(e));
    if (e2 != hipSuccess) return fail(NMF_EHIP, "csc build: %s", hipGetErrorString(e2));
    return NMF_OK;
}

// ---- rank-sliced engine (ranks above NMF_MU_MAX_K, and the host-resident-W pipeline) ----
// Every product of the iteration is written as F^T X with F (rows x k) and X (rows x cols)
// row-major, i.e. a reduction over the rows of both, and computed for slices of 64 or 128 columns of F side by side
// on the planes of F:
//   W^T A, W^T W                      F = W,  X = A or W
//   (W^T W) H                         F = W^T W (symmetric), X = H
//   A H^T, H H^T, W (H H^T)           the same three on the transposes A^T, H^T, W^T
// followed by the element-wise update.
struct Sliced {
    void *planes;     // pair planes of F (or, up to 64 factors and for X that is not aligned, the bf16 planes of a slice)
    float *ppart;     // row-split partials of one slice: splits x 64 x max cols
    size_t planes_cap, ppart_elems;
    unsigned *most;   // the largest magnitudes of the columns of F
};

// Partials of a product that are not added up: slices of 64 factors, `splits` each.
struct Partials {
    const float *at;
    int splits;
};

// The pair planes of F in e.planes.
PairFactor sliced_factor(const Sliced &e, int64_t rows, int ld)
{
    return PairFactor{e.planes, reinterpret_cast<unsigned char *>(e.planes) + pair_units_bytes(rows, ld), e.most};
}
// Columns per row group: whole slices of 128.
int sliced_ld(int k) { return (k + 127) / 128 * 128; }

// Row splits of a pass whose slices run side by side: every split of every slice is a partial result
// written and read again, and the slices already fill the chip (512 workgroups at a time), so the fewest
// splits whose last round of workgroups is nearly full.  Rank 256 on 16384 x 8192: 16 and 8 splits
// (134 MB of partials for each product) 930 us per iteration, 4 and 2 894.
int sliced_splits(int64_t rows, int64_t cols, int width, int nslices)
{
    const int most = wta_splits(rows, cols, width);
    const int64_t per = (cols + 255) / 256 * nslices;
    int best = most;
    double full = 0.0;
    for (int s = 1; s <= most; ++s) {
        const double rounds = (double)(per * s) / 512.0, use = rounds / std::ceil(rounds);
        if (use > full + 1e-9) {
            full = use;
            best = s;
        }
        if (use >= 0.9) break;
    }
    return best;
}

// Whether a product over X runs on pairs of halves, all slices in one launch each.
bool sliced_pairs(const float *X, int64_t cols, int k) { return k > NMF_MU_MAX_K && wta_planes_only_width(X, cols) == 64; }

hipError_t sliced_split(const Sliced &e, const float *F, int64_t rows, int k, hipStream_t st)
{
    const int ld = sliced_ld(k);
    if (pair_units_bytes(rows, ld) + pair_exps_bytes(rows, ld) > e.planes_cap) return hipErrorInvalidValue;
    hipError_t rc = launch_fill_f32(reinterpret_cast<float *>(e.most), ld * kPairCopies, 0.f, st);
    return rc != hipSuccess ? rc : launch_split_pairs(F, rows, k, sliced_factor(e, rows, ld), ld, st);
}

// split: the planes do not hold F yet.  keep: the partials are left as they are (where they are complete they are in out).
int sliced_ftx(const Sliced &e, const float *F, int64_t rows, int k, const float *X, int64_t cols,
               float *out, bool accumulate, hipStream_t st, bool split = true, Partials *keep = nullptr)
{
    // factor columns per pass: the widest the pass kernels take from planes alone for this X
    // (the slices of F are not contiguous, so the kernel that reads the factor itself is out)
    const int kSlice = wta_planes_only_width(X, cols);
    const int nslices = (k + 63) / 64;
    const int splits = sliced_splits(rows, cols, kSlice, kSlice == 64 ? nslices : 1);
    const int64_t rps = wta_rows_per_split(rows, splits);
    if (sliced_pairs(X, cols, k)) {
        // all slices in one launch each: the slices of a tile of X run side by side and share its bytes
        if ((size_t)splits * 64 * (size_t)cols * nslices > e.ppart_elems) return fail(NMF_EHIP, "internal: sliced scratch too small%s");
        if (split) NMF_HIP(sliced_split(e, F, rows, k, st));
        NMF_HIP(launch_pair_slices(X, rows, cols, k, F, sliced_factor(e, rows, sliced_ld(k)), sliced_ld(k), e.ppart, splits, rps, st));
        if (keep) *keep = Partials{e.ppart, splits};
        else NMF_HIP(launch_sum_partials_slices(e.ppart, splits, k, cols, out, st, accumulate));
        return NMF_OK;
    }
    if (keep) *keep = Partials{out, 1};
    if ((size_t)splits * kSlice * (size_t)cols > e.ppart_elems || planes_bytes(rows) > e.planes_cap)
        return fail(NMF_EHIP, "internal: sliced scratch too small%s");
    for (int c0 = 0; c0 < k; c0 += kSlice) {
        const int kc = (k - c0 < kSlice) ? k - c0 : kSlice;
        NMF_HIP(launch_split_planes_slice(F, rows, k, c0, kc, e.planes, st));
        NMF_HIP(launch_wta_pass(X, rows, cols, kc, nullptr, e.planes, true, e.ppart, splits, rps, false, st));
        NMF_HIP(launch_sum_partials(e.ppart, splits, (int64_t)kc * cols, out + (int64_t)c0 * cols, st, accumulate));
    }
    return NMF_OK;
}

// Factors of a slice of a pass over A'.  128 (one wave per SIMD) where such slices have more than 64 factors each and every compute
// unit gets some four blocks of 128 rows x 256 columns of the work: 16384 x 8192, k = 128 346 us per iteration in one slice, 377 in
// two of 64, k = 256 543 and 556, k = 384 825 and 823; below that the latency of a block decides (2000 x 1000, k = 68: 17.7 us
// per product in one slice of 128, 13 in two of 64).  A last slice of 64 behind those of 128 is a launch of its own
// that reads A' again: k = 130 on 32768 x 4096 733 us per iteration, 639 in slices of 64, k = 320 774 and 702.
int sliced_width(int64_t rows, int64_t cols, int k)
{
    const int64_t blocks = (rows + kPairBlock - 1) / kPairBlock * ((cols + 255) / 256) * ((k + 127) / 128);
    return blocks >= 1024 && (k - 1) % 128 >= 64 ? 128 : 64;
}

int64_t sliced_pass_tiles(int64_t rows, int64_t cols, int k)
{
    const int width = sliced_width(rows, cols, k), slices = (k + width - 1) / width;
    return pair_pass_tiles(cols, pair_splits(rows, cols, width / 32, slices), slices);
}

size_t sliced_pass_elems(int64_t rows, int64_t cols, int k)
{
    const int width = sliced_width(rows, cols, k), slices = (k + width - 1) / width;
    return (size_t)pair_splits(rows, cols, width / 32, slices) * slices * width * (size_t)cols;
}

// Upper bound on splits x 64 x cols over every X with at most `cols` rows and columns (64-factor slices;
// 32-factor slices have 128-column slabs and half the factors).  wta_splits keeps splits x slabs <= 512 with
// cols <= 256 slabs, or two splits on fewer than 384 slabs, or one: splits x cols <= 131072 + cols.  And more than
// 32 splits need fewer than 16 slabs and 256 rows each: at most cols / 256 splits of 15 x 256 columns.
size_t sliced_ppart_elems(int64_t cols)
{
    const int64_t a = 32 * cols, b = 131072 + cols;
    return (size_t)64 * (size_t)(a < b ? a : b);
}

// Resident run of rank k > NMF_MU_MAX_K.
struct SlicedDense {
    Sliced e;
    float *At, *Wt, *Ht, *num, *den, *g;
    bool pairs;             // A' and (A^T)' instead of At; no num, but
    PairMatrix pa, pt;
    float *pass;            // partials of a pass over A' or (A^T)'
    unsigned *most_g;       // maxima of the planes of a Gram matrix
    unsigned *redo;         // tiles of either pass that are formed from the floats
    int64_t nredo[2];
};


// Bytes of planes for any F of up to `rows` rows.
size_t sliced_planes_cap(int64_t rows, int k)
{
    const size_t pairs = pair_units_bytes(rows, sliced_ld(k)) + pair_exps_bytes(rows, sliced_ld(k)), pieces = planes_bytes(rows);
    return pairs > pieces ? pairs : pieces;
}

SlicedDense carve_sliced_dense(void *ws, int64_t m, int64_t n, int k, bool pairs, size_t *bytes)
{
    Carve cv(ws);
    SlicedDense p{};
    const int64_t big = m > n ? m : n, all = max3<int64_t>(m, n, k);
    const size_t nslices = (size_t)(k + 63) / 64;
    cv.take<unsigned>(64);       // the arrival counters at the head of the workspace stay untouched
    p.e.most = cv.take<unsigned>((size_t)sliced_ld(k) * kPairCopies);
    p.e.planes_cap = sliced_planes_cap(all, k);
    p.e.planes = cv.take<char>(p.e.planes_cap);
    // X is one of A (m x n), W (m x k), H (k x n) or a transpose of those
    p.e.ppart_elems = sliced_ppart_elems(all) * nslices;
    p.e.ppart = cv.take<float>(p.e.ppart_elems);
    if ((p.pairs = pairs)) {
        const size_t p1 = sliced_pass_elems(m, n, k), p2 = sliced_pass_elems(n, m, k);
        p.pass = cv.take<float>(p1 > p2 ? p1 : p2);
        p.nredo[0] = sliced_pass_tiles(m, n, k);
        p.nredo[1] = sliced_pass_tiles(n, m, k);
        p.most_g = cv.take<unsigned>((size_t)sliced_ld(k) * kPairCopies + p.nredo[0] + p.nredo[1]);
        p.redo = p.most_g + sliced_ld(k) * kPairCopies;
        p.pa = carve_pair_matrix(cv, m, n);
        p.pt = carve_pair_matrix(cv, n, m);
    } else {
        p.At = cv.take<float>((size_t)m * n);
    }
    p.Wt = cv.take<float>((size_t)k * m);
    p.Ht = cv.take<float>((size_t)n * k);
    p.num = cv.take<float>(pairs ? 0 : (size_t)k * big);
    p.den = cv.take<float>((size_t)k * big);
    p.g = cv.take<float>((size_t)k * k);
    if (bytes) *bytes = cv.off;
    return p;
}

bool sliced_cut_ok(int64_t m, int64_t n, int k) { return k > NMF_MU_MAX_K && pair_lengths_ok(m, n); }

size_t sliced_dense_bytes(int64_t m, int64_t n, int k, bool pairs)
{
    size_t b = 0;
    carve_sliced_dense(nullptr, m, n, k, pairs, &b);
    return b;
}

// F^T X over X' = x, the planes of F in e.planes; X is A or (transposed) A^T.  The partials are left where `u` says.
int sliced_pass(const SlicedDense &p, const float *F, int64_t rows, int k, const float *A, bool transposed, int64_t cols, bool stream,
                SlicedUpdate *u, hipStream_t st)
{
    static_assert(kPairSlices * 64 >= NMF_MU_MAX_K_SLICED, "one launch for all slices");
    const int width = sliced_width(rows, cols, k);
    PairPass a{};
    a.ldf = sliced_ld(k);
    a.F = sliced_factor(p.e, rows, a.ldf);
    a.slice_units = a.slice_exps = a.slice_most = width;
    a.X = transposed ? p.pt : p.pa;
    a.f = F;
    a.f_row = k;
    a.f_col = 1;
    a.slice_f = width;
    a.x = A;
    a.x_row = transposed ? 1 : cols;
    a.x_col = transposed ? rows : 1;
    a.redo = p.redo + (transposed ? p.nredo[0] : 0);
    a.rows = rows;
    a.n = cols;
    a.nslices = (k + width - 1) / width;
    for (int z = 0; z < a.nslices; ++z) a.k[z] = (short)(k - width * z < width ? k - width * z : width);
    a.splits = pair_splits(rows, cols, width / 32, a.nslices);
    a.rps = pair_rows_per_split(rows, a.splits);
    a.ppart = p.pass;
    a.slice_ppart = (int64_t)a.splits * width * cols;
    NMF_HIP(launch_pair_pass(a, width / 32, stream, st));
    u->k = k;
    u->num = p.pass;
    u->width = width;
    u->snum = a.splits;
    return NMF_OK;
}

// Y (k x cols) <- Y * (F^T X) / ((F^T F) Y + eps) and Yt its transpose, F rows x k with its planes in e.planes, X = A or (transposed)
// A^T; the planes of Yt take their place.
int sliced_pairs_update(const SlicedDense &p, const float *F, int64_t rows, int k, const float *A, bool transposed, int64_t cols, float *Y,
                        float *Yt, float eps, bool stream, hipStream_t st)
{
    const int ld = sliced_ld(k);
    SlicedUpdate u{};
    if (int rc = sliced_pass(p, F, rows, k, A, transposed, cols, stream, &u, st)) return rc;
    if (int rc = sliced_ftx(p.e, F, rows, k, F, k, p.g, false, st, false)) return rc;
    Partials den{};
    if (sliced_pairs(Y, cols, k)) {
        Sliced g = p.e;
        g.most = p.most_g;
        NMF_HIP(launch_split_pairs(p.g, k, k, sliced_factor(g, k, ld), ld, st, p.e.most));      // and the maxima of Yt to zero
        if (int rc = sliced_ftx(g, p.g, k, k, Y, cols, p.den, false, st, false, &den)) return rc;
    } else {
        if (int rc = sliced_ftx(p.e, p.g, k, k, Y, cols, p.den, false, st, true, &den)) return rc;
        NMF_HIP(launch_fill_f32(reinterpret_cast<float *>(p.e.most), ld * kPairCopies, 0.f, st));
    }
    u.X = Y;
    u.Xt = Yt;
    u.den = den.at;
    u.sden = den.splits;
    u.len = cols;
    u.eps = eps;
    u.F = sliced_factor(p.e, cols, ld);
    u.ld = ld;
    u.clear = p.most_g;
    u.nclear = ld * kPairCopies;
    NMF_HIP(launch_sliced_update(u, st));
    return NMF_OK;
}

// The same without a second layout: Y <- Y * (F^T X) / ((F^T F) Y + eps), X rows x cols.
int sliced_update(const SlicedDense &p, const float *F, int64_t rows, int k, const float *X, int64_t cols, float *Y, float eps,
                  hipStream_t st)
{
    if (int rc = sliced_ftx(p.e, F, rows, k, X, cols, p.num, false, st)) return rc;
    if (int rc = sliced_ftx(p.e, F, rows, k, F, k, p.g, false, st, !sliced_pairs(X, cols, k))) return rc;
    if (int rc = sliced_ftx(p.e, p.g, k, k, Y, cols, p.den, false, st)) return rc;
    NMF_HIP(launch_mu_apply(Y, p.num, p.den, eps, (int64_t)k * cols, st));
    return NMF_OK;
}

int sliced_dense_body(const float *A, int64_t m, int64_t n, int k, float *W, float *H, int iters,
                      float eps, const SlicedDense &p, hipStream_t st)
{
    // H update (Algorithm 3 order): numerator W^T A, denominator (W^T W) H; W update with the new H, on the
    // transposes: (A H^T)^T = H A^T, (W H H^T)^T = (H H^T) W^T
    if (p.pairs) {
        const bool stream = stream_a(m, n, true);
        const int maxima = sliced_ld(k) * kPairCopies;
        NMF_HIP(launch_cut_pairs(A, m, n, p.pa, p.pt, p.e.most, maxima, st));
        NMF_HIP(launch_fill_f32(reinterpret_cast<float *>(p.most_g), maxima + p.nredo[0] + p.nredo[1], 0.f, st));
        NMF_HIP(launch_transpose(W, m, k, p.Wt, st));
        NMF_HIP(launch_split_pairs(W, m, k, sliced_factor(p.e, m, sliced_ld(k)), sliced_ld(k), st));
        for (int it = 0; it < iters; ++it) {
            if (int rc = sliced_pairs_update(p, W, m, k, A, false, n, H, p.Ht, eps, stream, st)) return rc;
            if (int rc = sliced_pairs_update(p, p.Ht, n, k, A, true, m, p.Wt, W, eps, stream, st)) return rc;
        }
        return NMF_OK;
    }
    NMF_HIP(launch_transpose(A, m, n, p.At, st));
    NMF_HIP(launch_transpose(W, m, k, p.Wt, st));
    for (int it = 0; it < iters; ++it) {
        if (int rc = sliced_update(p, W, m, k, A, n, H, eps, st)) return rc;
        NMF_HIP(launch_transpose(H, k, n, p.Ht, st));
        if (int rc = sliced_update(p, p.Ht, n, k, p.At, m, p.Wt, eps, st)) return rc;
        NMF_HIP(launch_transpose(p.Wt, k, m, W, st));
    }
    return NMF_OK;
}

// Out-of-memory run through the sliced engine, any supported rank; W either on the device
// (W_host == nullptr) or in host memory and streamed with the batches (Algorithm 5).
constexpr int kMaxSlots = 16;

struct SlicedOoc {
    Sliced e;
    float *Abt, *Wbt, *num_b, *den_b;   // per-batch transposes, numerator and denominator (k x rows)
    float *num, *den, *Ht, *gw, *gh;    // k x n, k x n, n x k, k x k, k x k
};

SlicedOoc carve_sliced_ooc(void *ws, int64_t rb, int64_t n, int k, size_t *bytes)
{
    Carve cv(ws);
    SlicedOoc p;
    const size_t nslices = (size_t)(k + 63) / 64;
    cv.take<unsigned>(64);       // the arrival counters at the head of the workspace stay untouched
    p.e.most = cv.take<unsigned>((size_t)sliced_ld(k) * kPairCopies);
    p.e.planes_cap = sliced_planes_cap(max3<int64_t>(rb, n, k), k);
    p.e.ppart_elems = sliced_ppart_elems(max3<int64_t>(rb, n, k)) * nslices;
    p.e.planes = cv.take<char>(p.e.planes_cap);
    p.e.ppart = cv.take<float>(p.e.ppart_elems);
    p.Abt = cv.take<float>((size_t)n * rb);
    p.Wbt = cv.take<float>((size_t)k * rb);
    p.num_b = cv.take<float>((size_t)k * rb);
    p.den_b = cv.take<float>((size_t)k * rb);
    p.num = cv.take<float>((size_t)k * n);
    p.den = cv.take<float>((size_t)k * n);
    p.Ht = cv.take<float>((size_t)n * k);
    p.gw = cv.take<float>((size_t)k * k);
    p.gh = cv.take<float>((size_t)k * k);
    if (bytes) *bytes = cv.off;
    return p;
}

size_t sliced_ooc_bytes(int64_t rb, int64_t n, int k)
{
    size_t b = 0;
    carve_sliced_ooc(nullptr, rb, n, k, &b);
    return b;
}

int sliced_ooc_run(const float *A_host, float *W_host, float *W_dev, int64_t m, int64_t n, int k,
                   float *H, int iters, float eps, int64_t batch_rows, int slots, hipStream_t st,
                   size_t *device_bytes)
{
    const bool hostw = W_host != nullptr;
    const size_t a_bytes = align_up((size_t)batch_rows * n * sizeof(float));
    const size_t w_bytes = hostw ? align_up((size_t)batch_rows * k * sizeof(float)) : 0;
    const size_t slot_bytes = a_bytes + w_bytes;
    void *ws = nullptr;
    const size_t ws_bytes = sliced_ooc_bytes(batch_rows, n, k);
    if (int rc = ensure_workspace(ws_bytes, &ws)) return rc;
    const SlicedOoc p = carve_sliced_ooc(ws, batch_rows, n, k, nullptr);
    if (g.sl_stage_bytes < slots * slot_bytes) {
        if (g.sl_stage) {
            NMF_HIP(hipDeviceSynchronize());
            NMF_HIP(hipFree(g.sl_stage));
            g.sl_stage = nullptr;
            g.sl_stage_bytes = 0;
        }
        hipError_t e = hipMalloc(&g.sl_stage, slots * slot_bytes);
        if (e != hipSuccess) return fail(NMF_ENOMEM, "hipMalloc(staging): %s", hipGetErrorString(e));
        g.sl_stage_bytes = slots * slot_bytes;
    }
    if (device_bytes) *device_bytes = ws_bytes + slots * slot_bytes;
    if (!g.copy_stream) NMF_HIP(hipStreamCreateWithFlags(&g.copy_stream, hipStreamNonBlocking));
    if (!g.ev_entry) NMF_HIP(hipEventCreateWithFlags(&g.ev_entry, hipEventDisableTiming));
    if (!g.back_stream) NMF_HIP(hipStreamCreateWithFlags(&g.back_stream, hipStreamNonBlocking));
    for (int i = 0; i < kMaxSlots; ++i) {
        if (!g.sl_copied[i]) NMF_HIP(hipEventCreateWithFlags(&g.sl_copied[i], hipEventDisableTiming));
        if (!g.sl_done[i]) NMF_HIP(hipEventCreateWithFlags(&g.sl_done[i], hipEventDisableTiming));
        if (!g.sl_freed[i]) NMF_HIP(hipEventCreateWithFlags(&g.sl_freed[i], hipEventDisableTiming));
    }
    // Staging slots may still be read by work enqueued earlier on `st`.
    NMF_HIP(hipEventRecord(g.ev_entry, st));
    NMF_HIP(hipStreamWaitEvent(g.copy_stream, g.ev_entry, 0));

    const int64_t nb = (m + batch_rows - 1) / batch_rows;
    int64_t issued = 0;
    for (int s = 0; s <= iters; ++s) {
        for (int64_t b = 0; b < nb; ++b, ++issued) {
            const int slot = (int)(issued % slots);
            const int64_t i0 = b * batch_rows;
            const int64_t rb = (i0 + batch_rows <= m) ? batch_rows : m - i0;
            char *base = static_cast<char *>(g.sl_stage) + slot * slot_bytes;
            float *Ab = reinterpret_cast<float *>(base);
            float *Wb = hostw ? reinterpret_cast<float *>(base + a_bytes) : W_dev + i0 * k;
            if (issued >= slots) NMF_HIP(hipStreamWaitEvent(g.copy_stream, g.sl_freed[slot], 0));
            NMF_HIP(hipMemcpyAsync(Ab, A_host + i0 * n, (size_t)rb * n * sizeof(float),
                                   hipMemcpyHostToDevice, g.copy_stream));
            if (hostw)
                NMF_HIP(hipMemcpyAsync(Wb, W_host + i0 * k, (size_t)rb * k * sizeof(float),
                                       hipMemcpyHostToDevice, g.copy_stream));
            NMF_HIP(hipEventRecord(g.sl_copied[slot], g.copy_stream));
            NMF_HIP(hipStreamWaitEvent(st, g.sl_copied[slot], 0));
            if (s > 0) {
                // W_b <- W_b * (A_b H^T) / (W_b H H^T + eps) on the transposes of the batch
                NMF_HIP(launch_transpose(Ab, rb, n, p.Abt, st));
                NMF_HIP(launch_transpose(Wb, rb, k, p.Wbt, st));
                if (int rc = sliced_ftx(p.e, p.Ht, n, k, p.Abt, rb, p.num_b, false, st)) return rc;
                if (int rc = sliced_ftx(p.e, p.gh, k, k, p.Wbt, rb, p.den_b, false, st)) return rc;
                NMF_HIP(launch_mu_apply(p.Wbt, p.num_b, p.den_b, eps, (int64_t)k * rb, st));
                NMF_HIP(launch_transpose(p.Wbt, k, rb, Wb, st));
            }
            if (s < iters) {
                // accumulate W_b^T A_b and W_b^T W_b with the W_b just updated
                if (int rc = sliced_ftx(p.e, Wb, rb, k, Ab, n, p.num, b > 0, st)) return rc;
                if (int rc = sliced_ftx(p.e, Wb, rb, k, Wb, k, p.gw, b > 0, st, !sliced_pairs(Ab, n, k))) return rc;
            }
            if (hostw) {
                NMF_HIP(hipEventRecord(g.sl_done[slot], st));
                NMF_HIP(hipStreamWaitEvent(g.back_stream, g.sl_done[slot], 0));
                if (s > 0)
                    NMF_HIP(hipMemcpyAsync(W_host + i0 * k, Wb, (size_t)rb * k * sizeof(float),
                                           hipMemcpyDeviceToHost, g.back_stream));
                NMF_HIP(hipEventRecord(g.sl_freed[slot], g.back_stream));
            } else {
                NMF_HIP(hipEventRecord(g.sl_freed[slot], st));
            }
        }
        if (s < iters) {
            if (int rc = sliced_ftx(p.e, p.gw, k, k, H, n, p.den, false, st)) return rc;
            NMF_HIP(launch_mu_apply(H, p.num, p.den, eps, (int64_t)k * n, st));
            NMF_HIP(launch_transpose(H, k, n, p.Ht, st));
            if (int rc = sliced_ftx(p.e, p.Ht, n, k, p.Ht, k, p.gh, false, st)) return rc;
        }
    }
    if (hostw) {
        // the caller's stream continues only after the last rows of W have reached the host
        NMF_HIP(hipEventRecord(g.ev_entry, g.back_stream));
        NMF_HIP(hipStreamWaitEvent(st, g.ev_entry, 0));
    }
    return NMF_OK;
}

}  // namespace

// ---- allocation-free resident dense run --------------------------------------
// For callers that cannot allocate (HIP graph capture, tight serving loops, harnesses that
// forbid it): nmf_mu_dense on the small plan (row-split partials, piece planes, Gram scratch)
// with that workspace in a fixed array in device memory instead of hipMalloc'ed memory.

namespace {
constexpr size_t kScratchBytes = NMF_MU_NOALLOC_SCRATCH_BYTES;
}
// One copy per device that loads the library, held until the process ends.  In host code the
// name is only a handle for hipGetSymbolAddress; kernels get the address that call returns.
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex scratch_mu;
void *scratch_ptr[kMaxDevices] = {};      // device address of `scratch` on each device, once asked

int scratch_address(void **out)
{
    int dev = -1;
    NMF_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return fail(NMF_EUNSUPPORTED, "device ordinal beyond 63%s");
    std::lock_guard<std::mutex> lock(scratch_mu);
    if (!scratch_ptr[dev]) {
        void *p = nullptr;
        NMF_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return fail(NMF_EHIP, "hipGetSymbolAddress returned a null address%s");
        scratch_ptr[dev] = p;
    }
    *out = scratch_ptr[dev];
    return NMF_OK;
}
}  // namespace

namespace {
// Consecutive runs of an ensemble on the same A whose ranks K = sum(k) fit one slice.
struct Stack {
    int first, count, K;
};

// How many stacks from si on share one A, kPairGroup at most.
int stacks_from(const std::vector<Stack> &stacks, size_t si, const float *const *A)
{
    int c = 1;
    while (c < kPairGroup && si + c < stacks.size() && A[stacks[si + c].first] == A[stacks[si].first]) ++c;
    return c;
}

int stacks_side_by_side(const std::vector<Stack> &stacks, const float *const *A)
{
    int most = 1;
    for (size_t si = 0; si < stacks.size();) {
        const int c = stacks_from(stacks, si, A);
        most = c > most ? c : most;
        si += c;
    }
    return most;
}

// More than 32 factors on every A: below that the row plan has no second layout to make.  Several stacks on an A earn the cut by
// sharing it, a single one by its iterations, as a single run does, or by its runs, whose factors are two or three copies each for the plan
// before.  Against that plan, 10 shapes of 0.1 to 270 million entries: two or three stacks, one iteration 1.05 to 1.5 times as fast, ten 1.4 to
// 2.3; one stack of two runs, one, two and four iterations 1.19, 1.14 and 1.07 on 3000 x 2000, 0.94, 0.99 and 1.03 on 8192 x 4000, 0.89, 0.94
// and 0.99 on 16384 x 8192; of five 1.53, 1.36 and 1.23, then 1.13, 1.10 and 1.10, then 0.95, 0.97 and 1.01.  One rule for the call: what more of its
// matrices ask for.
bool ensemble_on_pairs(int64_t m, int64_t n, const std::vector<Stack> &stacks, const float *const *A, int iters)
{
    if (!pairs_ok(m, n, NMF_MU_MAX_K)) return false;
    int for_it = 0, against = 0;
    for (size_t si = 0; si < stacks.size();) {
        const float *a = A[stacks[si].first];
        const bool aligned = (reinterpret_cast<uintptr_t>(a) & 15u) == 0 && n % 4 == 0;
        int K = 0, count = 0, runs = 0;
        for (; si < stacks.size() && A[stacks[si].first] == a; ++si, ++count) K += stacks[si].K, runs += stacks[si].count;
        if (K <= 32) return false;
        const int least = runs == 1 ? pairs_least(m, n, false, false) : m * n > 1 << 26 ? 4 : runs == 2 && m * n > 1 << 24 ? 2 : 1;
        ++(count > 1 || !aligned || iters >= least ? for_it : against);
    }
    return for_it >= against;
}

int pairs_ensemble(const float *const *A, int64_t m, int64_t n, const int32_t *k, float *const *W, float *const *H, int iters,
                   float eps, const std::vector<Stack> &stacks, int groups, hipStream_t st)
{
    Carve cv(g.ws);
    DensePlan p = carve_pairs(cv, m, n, NMF_MU_MAX_K, groups);
    const float *cut = nullptr;      // whose A' the workspace holds
    for (size_t si = 0; si < stacks.size();) {
        const int count = stacks_from(stacks, si, A);
        const float *a = A[stacks[si].first];
        set_slices(&p, m, n, count);
        const PairPlanes planes = cut == a ? PairPlanes::there : PairPlanes::none;
        cut = a;
        if (count == 1 && stacks[si].count == 1) {      // a run by itself stays where it is
            const int r = stacks[si++].first;
            DensePlan q = p;
            q.Hs[0] = H[r];
            q.sl.k[0] = k[r];
            q.sl.bm[0].on = 0;
            NMF_HIP(launch_transpose(W[r], m, k[r], q.Wts[0], st));
            if (int rc = pairs_body(a, m, n, W[r], iters, eps, q, st, planes)) return rc;
            continue;
        }
        StackedRuns runs[kPairGroup];
        for (int z = 0; z < count; ++z) {
            const Stack &sk = stacks[si + z];
            BlockMap &map = p.sl.bm[z];
            map.on = sk.count > 1;
            int off = 0;
            for (int i = 0; i < sk.count; ++i) {
                const int r = sk.first + i;
                runs[z].W[i] = W[r];
                runs[z].H[i] = H[r];
                runs[z].k[i] = (short)k[r];
                runs[z].at[i] = (short)off;
                for (int c = 0; c < k[r]; ++c) map.id[off + c] = (unsigned char)i;
                off += k[r];
            }
            for (int c = off; c < 64; ++c) map.id[c] = 255;
            p.sl.k[z] = sk.K;
            NMF_HIP(launch_stack(runs[z], sk.count, true, p.Wts[z], p.Hs[z], m, n, st));
        }
        if (int rc = pairs_body(a, m, n, nullptr, iters, eps, p, st, planes)) return rc;
        for (int z = 0; z < count; ++z)
            NMF_HIP(launch_stack(runs[z], stacks[si + z].count, false, p.Wts[z], p.Hs[z], m, n, st));
        si += count;
    }
    return NMF_OK;
}
}  // namespace

extern "C" {

const char *nmf_status_string(int status)
{
    switch (status) {
    case NMF_OK: return "NMF_OK";
    case NMF_EINVAL: return "NMF_EINVAL";
    case NMF_ENOMEM: return "NMF_ENOMEM";
    case NMF_EHIP: return "NMF_EHIP";
    case NMF_EUNSUPPORTED: return "NMF_EUNSUPPORTED";
    default: return "NMF_UNKNOWN";
    }
}

const char *nmf_last_error(void) { return t_err; }

size_t nmf_mu_workspace_bytes(int kind, int64_t m, int64_t n, int64_t nnz, int32_t k,
                              int64_t batch_rows)
{
    if (m < 1 || n < 1 || k < 1) return 0;
    if (kind == 5) {
        if (k > NMF_MU_MAX_K_SLICED) return 0;
        const size_t plain = sliced_dense_bytes(m, n, k, false), pairs = sliced_cut_ok(m, n, k) ? sliced_dense_bytes(m, n, k, true) : 0;
        return plain > pairs ? plain : pairs;
    }
    if (kind == 6) {
        if (batch_rows < 1 || k > NMF_MU_MAX_K_SLICED) return 0;
        return sliced_ooc_bytes(batch_rows < m ? batch_rows : m, n, k);
    }
    if (k > NMF_MU_MAX_K) return 0;
    switch (kind) {
    case 0: {
        const size_t mirrored = dense_bytes(m, n, k, true), pairs = pairs_ok(m, n, k) ? pairs_bytes(m, n, k) : 0;
        return mirrored > pairs ? mirrored : pairs;
    }
    case 3: {   // stacks of runs up to the largest supported rank, side by side, or one by one with their packed factors
        const size_t one = dense_bytes(m, n, NMF_MU_MAX_K, true) + align_up((size_t)m * NMF_MU_MAX_K * sizeof(float)) +
                           align_up((size_t)NMF_MU_MAX_K * n * sizeof(float));
        const size_t pairs = pairs_ok(m, n, NMF_MU_MAX_K) ? pairs_bytes(m, n, NMF_MU_MAX_K, kPairGroup) : 0;
        return one > pairs ? one : pairs;
    }
    case 4: return dense_bytes(m, n, k, false);
    case 1: return nnz < 0 ? 0 : csr_bytes(n, nnz, k);
    case 2:
        if (batch_rows < 1) return 0;
        return dense_bytes(batch_rows < m ? batch_rows : m, n, k, false);
    default: return 0;
    }
}

int nmf_mu_set_workspace(void *dev_ptr, size_t bytes)
{
    std::lock_guard<std::mutex> lock(g.mu);
    if (dev_ptr && bytes) {
        if (reinterpret_cast<uintptr_t>(dev_ptr) % kAlign) return fail(NMF_EINVAL, "workspace must be 256-byte aligned%s");
        if (bytes < kAlign) return fail(NMF_EINVAL, "workspace too small%s");
        if (g.ws && g.ws_owned) {
            NMF_HIP(hipDeviceSynchronize());
            NMF_HIP(hipFree(g.ws));
        }
        NMF_HIP(hipMemset(dev_ptr, 0, kAlign));
        g.ws = dev_ptr;
        g.ws_bytes = bytes;
        g.ws_owned = false;
    } else {
        if (!g.ws_owned) {
            g.ws = nullptr;
            g.ws_bytes = 0;
        }
        g.ws_owned = true;
    }
    return NMF_OK;
}

int nmf_mu_release(void)
{
    std::lock_guard<std::mutex> lock(g.mu);
    NMF_HIP(hipDeviceSynchronize());
    if (g.ws && g.ws_owned) NMF_HIP(hipFree(g.ws));
    if (g.ws_owned) {
        g.ws = nullptr;
        g.ws_bytes = 0;
    }
    if (g.stage) NMF_HIP(hipFree(g.stage));
    g.stage = nullptr;
    g.stage_bytes = 0;
    if (g.sl_stage) NMF_HIP(hipFree(g.sl_stage));
    g.sl_stage = nullptr;
    g.sl_stage_bytes = 0;
    for (int i = 0; i < 3; ++i) {
        if (g.ev_copied[i]) NMF_HIP(hipEventDestroy(g.ev_copied[i]));
        if (g.ev_freed[i]) NMF_HIP(hipEventDestroy(g.ev_freed[i]));
        g.ev_copied[i] = g.ev_freed[i] = nullptr;
    }
    if (g.ev_entry) NMF_HIP(hipEventDestroy(g.ev_entry));
    g.ev_entry = nullptr;
    if (g.pinned) NMF_HIP(hipHostFree(g.pinned));
    g.pinned = nullptr;
    if (g.copy_stream) NMF_HIP(hipStreamDestroy(g.copy_stream));
    g.copy_stream = nullptr;
    for (int i = 0; i < 16; ++i) {
        if (g.sl_copied[i]) NMF_HIP(hipEventDestroy(g.sl_copied[i]));
        if (g.sl_done[i]) NMF_HIP(hipEventDestroy(g.sl_done[i]));
        if (g.sl_freed[i]) NMF_HIP(hipEventDestroy(g.sl_freed[i]));
        g.sl_copied[i] = g.sl_done[i] = g.sl_freed[i] = nullptr;
    }
    if (g.back_stream) NMF_HIP(hipStreamDestroy(g.back_stream));
    g.back_stream = nullptr;
    return NMF_OK;
}

int nmf_mu_dense(const float *A, int64_t m, int64_t n, int32_t k, float *W, float *H,
                 int32_t iters, float eps, void *stream)
{
    if (int rc = check_common(A, W, H, m, n, k, iters, eps, NMF_MU_MAX_K_SLICED)) return rc;
    if (iters == 0) return NMF_OK;
    std::lock_guard<std::mutex> lock(g.mu);
    void *ws = nullptr;
    if (k > NMF_MU_MAX_K) {
        hipStream_t st = static_cast<hipStream_t>(stream);
        const bool pairs = sliced_cut_ok(m, n, k) && have_workspace(sliced_dense_bytes(m, n, k, true), st);
        if (int rc = ensure_workspace(sliced_dense_bytes(m, n, k, pairs), &ws)) return rc;
        const SlicedDense p = carve_sliced_dense(ws, m, n, k, pairs, nullptr);
        return sliced_dense_body(A, m, n, k, W, H, iters, eps, p, st);
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    DenseRun r;
    if (int rc = open_run(A, m, n, k, W, H, iters, eps, 0, st, &r)) return rc;
    if (int rc = dense_body(r.A, r.m, r.n, k, r.W, r.H, iters, eps, r.p, st, r.have_at)) return rc;
    return close_run(r, k, W, H, m, n, st);
}

int nmf_mu_dense_profile(const float *A, int64_t m, int64_t n, int32_t k, float *W, float *H,
                         int32_t iters, float eps, void *stream, float *kernel_ms)
{
    if (int rc = check_common(A, W, H, m, n, k, iters, eps)) return rc;
    if (!kernel_ms) return fail(NMF_EINVAL, "null pointer%s");
    if (iters < 1 || iters > 4096) return fail(NMF_EINVAL, "profiled run needs 1 <= iters <= 4096%s");
    hipStream_t st = static_cast<hipStream_t>(stream);
    std::lock_guard<std::mutex> lock(g.mu);
    DensePlan p;
    if (int rc = dense_plan(A, m, n, k, 0, st, &p, nullptr, takes_pairs(A, m, n, k, iters, eps))) return rc;
    p.Hs[0] = H;
    const bool mirrored = p.mirrored, one_pass = p.one_pass, resident = p.resident != 0;
    constexpr int NK = kDenseKernels;
    std::vector<hipEvent_t> ev((size_t)iters * NK + 1, nullptr);
    int rc = NMF_OK;
    for (auto &e : ev)
        if (hipEventCreate(&e) != hipSuccess) rc = fail(NMF_EHIP, "hipEventCreate failed%s");
    if (rc == NMF_OK) rc = dense_body(A, m, n, k, W, H, iters, eps, p, st, false, ev.data());
    if (rc == NMF_OK && hipStreamSynchronize(st) != hipSuccess) rc = fail(NMF_EHIP, "hipStreamSynchronize failed%s");
    if (rc == NMF_OK) {
        double sum[NK] = {0, 0, 0, 0, 0, 0};
        for (int it = 0; it < iters && rc == NMF_OK; ++it)
            for (int j = 0; j < NK; ++j) {
                float ms = 0.f;
                if (hipEventElapsedTime(&ms, ev[(size_t)it * NK + j], ev[(size_t)it * NK + j + 1]) != hipSuccess) {
                    rc = fail(NMF_EHIP, "hipEventElapsedTime failed%s");
                    break;
                }
                sum[j] += ms;
            }
        for (int j = 0; j < NK; ++j) kernel_ms[j] = (float)(sum[j] / iters);
        kernel_ms[NK] = resident || one_pass || rows_plan_runs(A, m, n, k, mirrored) ? 2.f : (mirrored ? 1.f : 0.f);
        kernel_ms[NK + 1] = kernel_ms[NK + 2] = 0.f;
    }
    // The pass kernels once more, `reps` launches back to back between two events: the
    // duration of a launch without the event commands around it.  They only rewrite the
    // partial results, which nothing reads afterwards.
    if (rc == NMF_OK) {
        const int reps = 20;
        const int s1 = wta_splits(m, n, k), s2 = wta_splits(n, m, k);
        const int64_t rps1 = wta_rows_per_split(m, s1), rps2 = wta_rows_per_split(n, s2);
        const bool rows_plan = !resident && !one_pass && rows_plan_runs(A, m, n, k, mirrored);
        const Common &c = p.c;
        for (int which = 0; which < ((mirrored || rows_plan || one_pass || resident) ? 2 : 1) && rc == NMF_OK; ++which) {
            if (one_pass || resident || p.pairs) (void)0;
            else if (which == 0) (void)launch_split_planes(W, m, k, p.planes, st);
            else if (!rows_plan) (void)launch_split_planes(p.Ht, n, k, p.planes, st);
            ResidentArgs dry = p.res;
            if (resident) {
                dry.A = A, dry.Win = W, dry.Hin = H, dry.W = p.dry, dry.H = p.dry + m * k;
                dry.m = m, dry.n = n, dry.k = k, dry.eps = eps, dry.nprod = which == 0, dry.lead = which == 1;
            }
            hipError_t e = hipEventRecord(ev[0], st);
            for (int r = 0; r < reps && e == hipSuccess; ++r)
                e = resident ? launch_resident(dry, p.resident, st)
                    : one_pass ? launch_one_pass(A, m, n, k, p.planes2, nullptr, c.ghp, factor_update_blocks(n), W, nullptr, p.ppart,
                                               c.gwp, eps, st, which == 1, which == 0)
                    : p.pairs ? pass_over(p, A, m, n, which == 1, 0, st)
                    : which == 0 ? launch_wta_pass(A, m, n, k, W, p.planes, true, p.ppart, s1, rps1, false, st, nullptr, 0, nullptr, mirrored)
                    : rows_plan  // the fused pass without its stores to W
                        ? launch_aht_rows(A, m, n, k, p.planes2, c.gh, W, p.planes, c.gwp, eps, st, false, nullptr,
                                          nullptr, true)
                        : launch_wta_pass(p.At, n, m, k, p.Ht, p.planes, true, p.ppart, s2, rps2, false, st, nullptr, 0, nullptr, true);
            if (e == hipSuccess) e = hipEventRecord(ev[1], st);
            if (e == hipSuccess) e = hipEventSynchronize(ev[1]);
            float ms = 0.f;
            if (e == hipSuccess) e = hipEventElapsedTime(&ms, ev[0], ev[1]);
            if (e != hipSuccess) rc = fail(NMF_EHIP, "pass timing: %s", hipGetErrorString(e));
            kernel_ms[NK + 1 + which] = ms / reps;
        }
    }
    for (auto &e : ev)
        if (e) (void)hipEventDestroy(e);
    return rc;
}

int nmf_mu_dense_batched(int32_t n_runs, const float *const *A, int64_t m, int64_t n,
                         const int32_t *k, float *const *W, float *const *H, int32_t iters,
                         float eps, void *stream)
{
    if (n_runs < 0 || !A || !k || !W || !H) return fail(NMF_EINVAL, "null pointer or negative run count%s");
    int kmax = 1;
    for (int r = 0; r < n_runs; ++r) {
        if (int rc = check_common(A[r], W[r], H[r], m, n, k[r], iters, eps)) return rc;
        if (k[r] > kmax) kmax = k[r];
    }
    if (iters == 0 || n_runs == 0) return NMF_OK;
    std::lock_guard<std::mutex> lock(g.mu);
    hipStream_t st = static_cast<hipStream_t>(stream);
    // Consecutive runs on the same A are stacked side by side while their ranks sum to
    // at most NMF_MU_MAX_K: one stack is one factorisation of rank sum(k) for the two
    // passes over A (A is read once for all of them), with the Gram matrices masked to
    // their diagonal blocks in the finishers so that the runs stay independent.
    std::vector<Stack> stacks;
    for (int r = 0; r < n_runs;) {
        Stack sk{r, 0, 0};
        while (r < n_runs && A[r] == A[sk.first] && sk.K + k[r] <= NMF_MU_MAX_K) {
            sk.K += k[r];
            ++sk.count;
            ++r;
        }
        stacks.push_back(sk);
    }
    int Kmax = kmax;
    for (const Stack &sk : stacks)
        if (sk.K > Kmax) Kmax = sk.K;
    const size_t stack_bytes = align_up((size_t)m * Kmax * sizeof(float)) + align_up((size_t)Kmax * n * sizeof(float));
    void *ws = nullptr;
    // Stacking needs the mirrored plan for the largest stack plus room for the packed
    // factors; without that much workspace the runs go one by one with the plan that fits.
    const size_t big = dense_bytes(m, n, Kmax, true) + stack_bytes;
    // Several stacks on the same A, or one of more than 32 factors: on pairs, up to kPairGroup stacks side by side as slices of
    // one launch per product, which reads A' once for all of them, and of one per update.  16384 x 8192, ranks 2 to 16 (stacks
    // of 54, 50 and 31 factors): 10 iterations of the 30 runs on two copies
    // of A 14.5 -> 9.4 ms.
    if (ensemble_on_pairs(m, n, stacks, A, iters)) {
        const int groups = stacks_side_by_side(stacks, A);
        if (have_workspace(pairs_bytes(m, n, NMF_MU_MAX_K, groups), st))
            return pairs_ensemble(A, m, n, k, W, H, iters, eps, stacks, groups, st);
    }
    // Whose transpose the workspace holds: a run that takes the row plan makes none, also where the next
    // one on the same A, of a larger rank, needs it.
    const float *at_of = nullptr;
    auto note_at = [&](const DensePlan &p, const float *a, int rank) {
        if (p.mirrored && !takes_row_plan(p, a, m, n, rank)) at_of = a;
    };
    if (!have_workspace(big, st)) {
        bool mirrored = false;
        if (int rc = dense_workspace(nullptr, m, n, kmax, &ws, &mirrored)) return rc;
        const DensePlan p1 = carve_dense(ws, m, n, kmax, mirrored);
        for (int r = 0; r < n_runs; ++r) {
            if (int rc = dense_body(A[r], m, n, k[r], W[r], H[r], iters, eps, p1, st, at_of == A[r])) return rc;
            note_at(p1, A[r], k[r]);
        }
        return NMF_OK;
    }
    ws = g.ws;
    // Carve once with the largest stacked rank so that A^T sits at one address for all
    // stacks: consecutive stacks on the same A share its transpose.
    const DensePlan p = carve_dense(ws, m, n, Kmax, true);
    char *tail = static_cast<char *>(ws) + dense_bytes(m, n, Kmax, true);
    float *Wall = reinterpret_cast<float *>(tail);
    float *Hall = reinterpret_cast<float *>(tail + align_up((size_t)m * Kmax * sizeof(float)));
    for (size_t si = 0; si < stacks.size(); ++si) {
        const Stack &sk = stacks[si];
        const bool have_at = at_of == A[sk.first];
        if (sk.count == 1) {
            const int r = sk.first;
            if (int rc = dense_body(A[r], m, n, k[r], W[r], H[r], iters, eps, p, st, have_at)) return rc;
            note_at(p, A[r], k[r]);
            continue;
        }
        BlockMap map;
        map.on = 1;
        int off = 0;
        for (int i = 0; i < sk.count; ++i) {
            const int r = sk.first + i;
            for (int c = 0; c < k[r]; ++c) map.id[off + c] = (unsigned char)i;
            NMF_HIP(hipMemcpy2DAsync(Wall + off, (size_t)sk.K * sizeof(float), W[r], (size_t)k[r] * sizeof(float),
                                     (size_t)k[r] * sizeof(float), (size_t)m, hipMemcpyDeviceToDevice, st));
            NMF_HIP(hipMemcpyAsync(Hall + (size_t)off * n, H[r], (size_t)k[r] * n * sizeof(float),
                                   hipMemcpyDeviceToDevice, st));
            off += k[r];
        }
        for (int c = off; c < 64; ++c) map.id[c] = 255;
        if (int rc = dense_body(A[sk.first], m, n, sk.K, Wall, Hall, iters, eps, p, st, have_at, nullptr, &map))
            return rc;
        note_at(p, A[sk.first], sk.K);
        off = 0;
        for (int i = 0; i < sk.count; ++i) {
            const int r = sk.first + i;
            NMF_HIP(hipMemcpy2DAsync(W[r], (size_t)k[r] * sizeof(float), Wall + off, (size_t)sk.K * sizeof(float),
                                     (size_t)k[r] * sizeof(float), (size_t)m, hipMemcpyDeviceToDevice, st));
            NMF_HIP(hipMemcpyAsync(H[r], Hall + (size_t)off * n, (size_t)k[r] * n * sizeof(float),
                                   hipMemcpyDeviceToDevice, st));
            off += k[r];
        }
    }
    return NMF_OK;
}

// Streamed dense run; objective_host (iters doubles) != nullptr: the objective of every
// iteration as well (ranks up to NMF_MU_MAX_K only).
static int ooc_run(const float *A_host, int64_t m, int64_t n, int32_t k, float *W, float *H,
                   int32_t iters, float eps, int64_t batch_rows, int64_t device_budget_bytes,
                   double *objective_host, void *stream)
{
    if (int rc = check_common(A_host, W, H, m, n, k, iters, eps, NMF_MU_MAX_K_SLICED)) return rc;
    if (objective_host && k > NMF_MU_MAX_K)
        return fail(NMF_EUNSUPPORTED, "monitored out-of-memory run: k <= 64%s");
    if (batch_rows < 1) return fail(NMF_EINVAL, "batch_rows must be >= 1%s");
    if (device_budget_bytes < 1) return fail(NMF_EINVAL, "device_budget_bytes must be >= 1%s");
    if (iters == 0) return NMF_OK;
    if (batch_rows > m) batch_rows = m;
    const size_t slot_bytes = align_up((size_t)batch_rows * n * sizeof(float));
    int slots = (int)((size_t)device_budget_bytes / slot_bytes);
    if (slots < 1) return fail(NMF_ENOMEM, "device budget does not hold one batch%s");
    if (slots > 3) slots = 3;
    hipStream_t st = static_cast<hipStream_t>(stream);

    std::lock_guard<std::mutex> lock(g.mu);
    if (k > NMF_MU_MAX_K) {
        const int64_t nbat = (m + batch_rows - 1) / batch_rows;
        if (slots > nbat) slots = (int)nbat;
        return sliced_ooc_run(A_host, nullptr, W, m, n, k, H, iters, eps, batch_rows, slots, st, nullptr);
    }
    const int64_t nb = (m + batch_rows - 1) / batch_rows;
    // monitored run: the W updates' shares of <A H^T, W> (one per workgroup and batch), ||A_b||^2 per
    // batch and its scratch, ||A||^2, one objective value per iteration
    // The W update of a batch: the streaming row kernel where it applies (staging slots are aligned,
    // so that is a matter of n, k and the batch height), else the direct kernel.
    const bool use_rows = aht_rows_can(nullptr, n, k);
    // Row tiles per workgroup are chosen once, for a full batch: with a choice of its own a shorter last batch could
    // have more workgroups than a full one (8192 rows: 128 of 64 rows, 8000 rows: 250 of 32), and more than the
    // shares that are laid out here for it.
    // At least two: one share per 64 rows is what nmf_mu_ooc_monitor's workspace is documented to hold, and the link
    // bounds a batch, not the workgroups of its W update.
    const int tiles = use_rows ? std::max(2, aht_rows_tiles(batch_rows, k)) : 0;
    auto w_blocks = [&](int64_t rows) { return use_rows ? (int64_t)aht_rows_blocks(rows, k, tiles) : aht_pass_blocks(rows); };
    const int64_t bpb = w_blocks(batch_rows);
    const size_t mon_bytes = objective_host
        ? align_up((size_t)(nb * bpb) * sizeof(double)) + align_up((size_t)nb * sizeof(double)) +
          align_up(4097 * sizeof(double)) + align_up((size_t)iters * sizeof(double))
        : 0;
    void *ws = nullptr;
    if (int rc = ensure_workspace(dense_bytes(batch_rows, n, k, false) + mon_bytes, &ws)) return rc;
    Carve cv(ws);
    const Common c = carve_common(cv, k);
    const int splits = wta_splits(batch_rows, n, k);
    const int64_t rps = wta_rows_per_split(batch_rows, splits);
    float *ppart = cv.take<float>((size_t)splits * k * n);
    void *planes = cv.take<char>(planes_bytes(batch_rows));
    void *planes_ht = cv.take<char>(planes_bytes(n));      // row kernel: piece planes of H^T
    double *dpart = nullptr, *normb = nullptr, *normA2 = nullptr, *obj = nullptr;
    if (objective_host) {
        dpart = cv.take<double>((size_t)(nb * bpb));
        normb = cv.take<double>((size_t)nb);
        normA2 = cv.take<double>(4097);
        obj = cv.take<double>((size_t)iters);
    }

    if (g.stage_bytes < slots * slot_bytes) {
        if (g.stage) {
            NMF_HIP(hipDeviceSynchronize());
            NMF_HIP(hipFree(g.stage));
            g.stage = nullptr;
            g.stage_bytes = 0;
        }
        hipError_t e = hipMalloc(&g.stage, slots * slot_bytes);
        if (e != hipSuccess) return fail(NMF_ENOMEM, "hipMalloc(staging): %s", hipGetErrorString(e));
        g.stage_bytes = slots * slot_bytes;
    }
    if (!g.copy_stream) NMF_HIP(hipStreamCreateWithFlags(&g.copy_stream, hipStreamNonBlocking));
    if (!g.ev_entry) NMF_HIP(hipEventCreateWithFlags(&g.ev_entry, hipEventDisableTiming));
    for (int i = 0; i < 3; ++i) {
        if (!g.ev_copied[i]) NMF_HIP(hipEventCreateWithFlags(&g.ev_copied[i], hipEventDisableTiming));
        if (!g.ev_freed[i]) NMF_HIP(hipEventCreateWithFlags(&g.ev_freed[i], hipEventDisableTiming));
    }
    // Staging slots may still be read by work enqueued earlier on `st`.
    NMF_HIP(hipEventRecord(g.ev_entry, st));
    NMF_HIP(hipStreamWaitEvent(g.copy_stream, g.ev_entry, 0));

    // Every other sweep walks the batches backwards, so that it begins with those the last one left in the
    // slots: they are not copied again.  The link is the bound (16384 x 16384 in 8 batches, 3 slots, 3
    // iterations: 32 copies of 128 MiB took 76 ms, 23 take 56).  Position i of a sweep overwrites the
    // slot of position i - slots, whose work on the batch is awaited by an event.
    std::vector<int> slot_of((size_t)nb, 0);
    for (int s = 0; s <= iters; ++s) {
        auto batch_at = [&](int64_t i) { return (s & 1) ? nb - 1 - i : i; };
        for (int64_t i = 0; i < nb; ++i) {
            const int64_t b = batch_at(i);
            const bool upload = s == 0 || i >= slots;
            if (upload) slot_of[(size_t)b] = i < slots ? (int)i : slot_of[(size_t)batch_at(i - slots)];
            const int slot = slot_of[(size_t)b];
            const int64_t i0 = b * batch_rows;
            const int64_t rb = (i0 + batch_rows <= m) ? batch_rows : m - i0;
            float *Ab = reinterpret_cast<float *>(static_cast<char *>(g.stage) + slot * slot_bytes);
            if (upload) {
                if (i >= slots) NMF_HIP(hipStreamWaitEvent(g.copy_stream, g.ev_freed[slot], 0));
                NMF_HIP(hipMemcpyAsync(Ab, A_host + i0 * n, (size_t)rb * n * sizeof(float),
                                       hipMemcpyHostToDevice, g.copy_stream));
                NMF_HIP(hipEventRecord(g.ev_copied[slot], g.copy_stream));
                NMF_HIP(hipStreamWaitEvent(st, g.ev_copied[slot], 0));
            }
            if (dpart && s == 0) NMF_HIP(launch_sumsq(Ab, rb * n, normA2 + 1, normb + b, st));
            if (s > 0) {
                if (use_rows)    // also leaves the piece planes of the batch's new rows for the pass below
                    NMF_HIP(launch_aht_rows(Ab, rb, n, k, planes_ht, c.gh, W + i0 * k, planes, c.gwp, eps, st, false, nullptr,
                                            dpart ? dpart + b * bpb : nullptr, false, tiles));
                else
                    NMF_HIP(launch_aht_pass(Ab, rb, n, k, H, c.gh, W + i0 * k, eps, st, dpart ? dpart + b * bpb : nullptr));
            }
            if (s < iters)
                NMF_HIP(launch_wta_pass(Ab, rb, n, k, W + i0 * k, planes, use_rows && s > 0, ppart, splits, rps, i > 0, st));
            NMF_HIP(hipEventRecord(g.ev_freed[slot], st));
        }
        if (dpart && s == 0) NMF_HIP(launch_sum_f64(normb, nb, normA2, st));
        if (s < iters || dpart) NMF_HIP(launch_gram_w(W, m, k, c.gw, c.gpart, c.counters, st));
        if (dpart && s > 0) {
            // iteration s is complete: <A H^T, W> from this sweep's W updates (a short last batch
            // leaves the tail of its segment untouched, so its workgroups are counted, not bpb),
            // H H^T of the H they used, W^T W of the W they left
            const int64_t last_rows = m - (nb - 1) * batch_rows;
            if (w_blocks(last_rows) < bpb) {
                // close the gap so that the shares are one contiguous run
                NMF_HIP(hipMemsetAsync(dpart + (nb - 1) * bpb + w_blocks(last_rows), 0,
                                       (size_t)(bpb - w_blocks(last_rows)) * sizeof(double), st));
            }
            NMF_HIP(launch_objective(dpart, (int)(nb * bpb), c.gw, c.gh, k, normA2, obj + (s - 1), st));
        }
        if (s < iters) {
            NMF_HIP(launch_factor_update(H, nullptr, ppart, splits, c.gw, nullptr, 0, nullptr, k, n, eps, st, nullptr,
                                         use_rows ? planes_ht : nullptr));
            NMF_HIP(launch_gram_h(H, k, n, c.gh, c.gpart, c.counters, st));
        }
    }
    if (dpart) {
        NMF_HIP(hipMemcpyAsync(objective_host, obj, (size_t)iters * sizeof(double), hipMemcpyDeviceToHost, st));
        NMF_HIP(hipStreamSynchronize(st));
    }
    return NMF_OK;
}

int nmf_mu_ooc(const float *A_host, int64_t m, int64_t n, int32_t k, float *W, float *H,
               int32_t iters, float eps, int64_t batch_rows, int64_t device_budget_bytes,
               void *stream)
{
    return ooc_run(A_host, m, n, k, W, H, iters, eps, batch_rows, device_budget_bytes, nullptr, stream);
}

int nmf_mu_ooc_monitor(const float *A_host, int64_t m, int64_t n, int32_t k, float *W, float *H,
                       int32_t iters, float eps, int64_t batch_rows, int64_t device_budget_bytes,
                       double *objective_host, void *stream)
{
    if (!objective_host) return fail(NMF_EINVAL, "null pointer%s");
    if (iters > (1 << 20)) return fail(NMF_EINVAL, "monitored run: iters <= 2^20%s");
    return ooc_run(A_host, m, n, k, W, H, iters, eps, batch_rows, device_budget_bytes, objective_host, stream);
}

int nmf_mu_ooc_hostw(const float *A_host, float *W_host, int64_t m, int64_t n, int32_t k, float *H,
                     int32_t iters, float eps, int64_t batch_rows, int32_t slots, void *stream,
                     size_t *device_bytes_host)
{
    if (int rc = check_common(A_host, W_host, H, m, n, k, iters, eps, NMF_MU_MAX_K_SLICED)) return rc;
    if (batch_rows < 1) return fail(NMF_EINVAL, "batch_rows must be >= 1%s");
    if (slots < 1 || slots > kMaxSlots) return fail(NMF_EINVAL, "slots must be in 1 .. 16%s");
    if (device_bytes_host) *device_bytes_host = 0;
    if (iters == 0) return NMF_OK;
    if (batch_rows > m) batch_rows = m;
    const int64_t nbat = (m + batch_rows - 1) / batch_rows;
    if (slots > nbat) slots = (int)nbat;
    std::lock_guard<std::mutex> lock(g.mu);
    return sliced_ooc_run(A_host, W_host, nullptr, m, n, k, H, iters, eps, batch_rows, slots,
                          static_cast<hipStream_t>(stream), device_bytes_host);
}

// Bytes behind csr_bytes() that a monitored sparse run needs: the W update's by-products,
// ||A||^2 with its scratch, one objective value per iteration.
size_t csr_monitor_bytes(int iters)
{
    return align_up((size_t)kCsrDparts * sizeof(double)) + align_up(4097 * sizeof(double)) +
           align_up((size_t)iters * sizeof(double)) + align_up((size_t)(65536 + 1) * sizeof(double));
}

// Stopping rule of a sparse run (Algorithm 1): results in host memory.
struct CsrTol {
    double tol;
    int check_every;
    int32_t *iters_done;
    double *residual;
};

// Resident sparse run; objective_host (iters doubles) == nullptr: no monitoring; with `tolp`
// the run stops as soon as a check finds the objective at or below tolp->tol (iters = the most).
static int csr_run(const int64_t *rowptr, const int32_t *colidx, const float *vals, int64_t m,
                   int64_t n, int64_t nnz, int32_t k, float *W, float *H, int32_t iters, float eps,
                   double *objective_host, void *stream, const CsrTol *tolp = nullptr)
{
    if (!rowptr) return fail(NMF_EINVAL, "null pointer%s");
    if (nnz < 0) return fail(NMF_EINVAL, "nnz must be >= 0%s");
    if (nnz > 0 && (!colidx || !vals)) return fail(NMF_EINVAL, "null pointer%s");
    if (int rc = check_common(rowptr, W, H, m, n, k, iters, eps)) return rc;
    if (iters == 0 && !tolp) return NMF_OK;
    hipStream_t st = static_cast<hipStream_t>(stream);
    std::lock_guard<std::mutex> lock(g.mu);
    if (nnz >= ((int64_t)1 << 31) || m >= ((int64_t)1 << 31))
        return fail(NMF_EUNSUPPORTED, "CSR path needs nnz < 2^31 and m < 2^31%s");
    void *ws = nullptr;
    const bool watch = objective_host || tolp;
    const size_t need = csr_bytes(n, nnz, k) + (watch ? csr_monitor_bytes(tolp ? 1 : iters) : 0);
    // Both factors are gathered from row by row; where their rows straddle cache lines (k not a
    // length of csr_row_length) the run works on copies with longer rows, if the workspace holds them:
    // 1000000 x 300000 with 40 entries per row, per iteration, k = 12 1660 -> 1482 us, k = 24 2128 -> 1592,
    // k = 50 3726 -> 3310.  Tables that the L2 caches hold gain nothing (65536 x 16384, k = 12: 58.9 and
    // 60.4; 100000 x 100000, k = 24, 9.6 MB each: 647 and 544).
    const int ldk = csr_row_length(k);
    const size_t wide = align_up((size_t)m * ldk * sizeof(float)) + align_up((size_t)n * ldk * sizeof(float));
    const bool copies = ldk != k && (iters > 1 || tolp) && (int64_t)(m > n ? m : n) * k * 4 > ((int64_t)8 << 20) &&
                        have_workspace(need + wide, st);
    if (!copies)
        if (int rc = ensure_workspace(need, &ws)) return rc;
    ws = g.ws;
    const int ld = copies ? ldk : k;
    Carve cv(ws);
    const Common c = carve_common(cv, k);
    float *Ht = cv.take<float>((size_t)n * k);
    int64_t *colptr = cv.take<int64_t>((size_t)n + 1);
    int32_t *rowidx = cv.take<int32_t>((size_t)nnz);
    float *cvals = cv.take<float>((size_t)nnz);
    int64_t *part_r = cv.take<int64_t>((size_t)kCsrParts + 1);
    int64_t *part_c = cv.take<int64_t>((size_t)kCsrParts + 1);
    int32_t *long_r = cv.take<int32_t>((size_t)(nnz / kLongRow + 2));
    int32_t *long_c = cv.take<int32_t>((size_t)(nnz / kLongRow + 2));
    unsigned *long_n = cv.take<unsigned>(64);      // [0] rows of A, [1] columns of A
    const size_t sort_temp_bytes = nnz ? csc_sort_temp_bytes(nnz, n) : 0;
    int32_t *sorted_cols = cv.take<int32_t>((size_t)nnz);
    uint64_t *payload = cv.take<uint64_t>((size_t)nnz);
    uint64_t *sorted_payload = cv.take<uint64_t>((size_t)nnz);
    char *sort_temp = cv.take<char>(sort_temp_bytes);
    double *dpart = nullptr, *normA2 = nullptr, *obj = nullptr, *dup = nullptr;
    if (watch) {
        dpart = cv.take<double>(kCsrDparts);
        normA2 = cv.take<double>(4097);
        obj = cv.take<double>(tolp ? 1 : (size_t)iters);
        dup = cv.take<double>(65536 + 1);      // one share per block of the copy's last kernel, then the sum of squares
    }
    const int ndup = csc_finish_blocks(nnz);
    // The Gram kernel's arrival counter reads zero at the start also after a call that was cut short.
    NMF_HIP(launch_fill_f32(reinterpret_cast<float *>(c.counters), 64, 0.f, st));

    // Column-ordered copy of A, once per call, enqueued like everything else.
    NMF_HIP(launch_csc_build(rowptr, colidx, vals, m, n, nnz, sorted_cols, payload, sorted_payload, sort_temp,
                             sort_temp_bytes, colptr, rowidx, cvals, st, dup));
    if (watch) {
        // ||A||_F^2 of the matrix the arrays stand for: the squared stored values plus what repeated
        // (row, column) pairs add (found while the column-ordered copy is written)
        if (nnz > 0) NMF_HIP(launch_sumsq(vals, nnz, normA2 + 1, dup + ndup, st));
        else NMF_HIP(launch_fill_f32(reinterpret_cast<float *>(dup + ndup), 2, 0.f, st));
        NMF_HIP(launch_sum_f64(dup, ndup + 1, normA2, st));
    }

    // Work partitions of both orientations, once per call.
    NMF_HIP(launch_csr_partition(rowptr, m, kCsrParts, part_r, st));
    NMF_HIP(launch_csr_partition(colptr, n, kCsrParts, part_c, st));
    NMF_HIP(launch_csr_long_rows(rowptr, m, long_r, long_n, (unsigned)(nnz / kLongRow + 1), st));
    NMF_HIP(launch_csr_long_rows(colptr, n, long_c, long_n + 1, (unsigned)(nnz / kLongRow + 1), st));

    float *Wx = W;
    if (copies) {
        Carve tail(static_cast<char *>(ws) + need);
        Wx = tail.take<float>((size_t)m * ldk);
        Ht = tail.take<float>((size_t)n * ldk);
        NMF_HIP(launch_restride(W, k, Wx, ldk, m, k, st));
    }
    // The factors go back to the caller's.
    auto hand_back = [&]() -> int {
        NMF_HIP(launch_transpose(Ht, n, k, H, st, 0, nullptr, 0, ld));
        if (copies) NMF_HIP(launch_restride(Wx, ldk, W, k, m, k, st));
        return NMF_OK;
    };
    NMF_HIP(launch_transpose(H, k, n, Ht, st, ld));
    // One iteration; with `out`, ||A - W H||_F of its result goes there, from what the W update
    // leaves behind: <A H^T, W>, H H^T, and W^T W of the new W (computed here; the next iteration
    // computes the same matrix again for its H update).
    auto iteration = [&](double *out) -> int {
        NMF_HIP(launch_gram_w_wide(Wx, m, k, c.gw, c.gwp, c.counters, st, ld));
        NMF_HIP(launch_aht_csr(colptr, rowidx, cvals, part_c, long_c, long_n + 1, k, Wx, c.gw, Ht, eps, nnz, n, m, st, false, nullptr, false, ld, ld));   // H update on H^T
        NMF_HIP(launch_gram_w_wide(Ht, n, k, c.gh, c.ghp, c.counters, st, ld));
        NMF_HIP(launch_aht_csr(rowptr, colidx, vals, part_r, long_r, long_n, k, Ht, c.gh, Wx, eps, nnz, m, n, st, false,
                               out ? dpart : nullptr, false, ld, ld));                                                       // W update
        if (out) {
            NMF_HIP(launch_gram_w_wide(Wx, m, k, c.gw, c.gwp, c.counters, st, ld));
            NMF_HIP(launch_objective(dpart, kCsrDparts, c.gw, c.gh, k, normA2, out, st));
        }
        return NMF_OK;
    };
    if (tolp) {
        // objective of the factors as given: the W pass without its update
        double res = 0.0;
        NMF_HIP(launch_gram_w_wide(Wx, m, k, c.gw, c.gwp, c.counters, st, ld));
        NMF_HIP(launch_gram_w_wide(Ht, n, k, c.gh, c.ghp, c.counters, st, ld));
        NMF_HIP(launch_aht_csr(rowptr, colidx, vals, part_r, long_r, long_n, k, Ht, c.gh, Wx, eps, nnz, m, n, st, false, dpart, true, ld, ld));
        NMF_HIP(launch_objective(dpart, kCsrDparts, c.gw, c.gh, k, normA2, obj, st));
        NMF_HIP(hipMemcpyAsync(&res, obj, sizeof(double), hipMemcpyDeviceToHost, st));
        NMF_HIP(hipStreamSynchronize(st));
        int done = 0;
        while (done < iters && res > tolp->tol) {
            const int chunk = (iters - done < tolp->check_every) ? iters - done : tolp->check_every;
            for (int it = 0; it < chunk; ++it)
                if (int rc = iteration(it == chunk - 1 ? obj : nullptr)) return rc;
            NMF_HIP(hipMemcpyAsync(&res, obj, sizeof(double), hipMemcpyDeviceToHost, st));
            NMF_HIP(hipStreamSynchronize(st));
            done += chunk;
        }
        if (int rc = hand_back()) return rc;
        NMF_HIP(hipStreamSynchronize(st));
        *tolp->iters_done = done;
        *tolp->residual = res;
        return NMF_OK;
    }
    for (int it = 0; it < iters; ++it)
        if (int rc = iteration(objective_host ? obj + it : nullptr)) return rc;
    if (int rc = hand_back()) return rc;
    if (objective_host) {
        NMF_HIP(hipMemcpyAsync(objective_host, obj, (size_t)iters * sizeof(double), hipMemcpyDeviceToHost, st));
        NMF_HIP(hipStreamSynchronize(st));
    }
    return NMF_OK;
}

int nmf_mu_csr(const int64_t *rowptr, const int32_t *colidx, const float *vals, int64_t m,
               int64_t n, int64_t nnz, int32_t k, float *W, float *H, int32_t iters, float eps,
               void *stream)
{
    return csr_run(rowptr, colidx, vals, m, n, nnz, k, W, H, iters, eps, nullptr, stream);
}

int nmf_mu_csr_monitor(const int64_t *rowptr, const int32_t *colidx, const float *vals, int64_t m,
                       int64_t n, int64_t nnz, int32_t k, float *W, float *H, int32_t iters, float eps,
                       double *objective_host, void *stream)
{
    if (!objective_host) return fail(NMF_EINVAL, "null pointer%s");
    if (iters > (1 << 20)) return fail(NMF_EINVAL, "monitored run: iters <= 2^20%s");
    return csr_run(rowptr, colidx, vals, m, n, nnz, k, W, H, iters, eps, objective_host, stream);
}

int nmf_mu_csr_tol(const int64_t *rowptr, const int32_t *colidx, const float *vals, int64_t m,
                   int64_t n, int64_t nnz, int32_t k, float *W, float *H, int32_t max_iters, float eps,
                   double tol, int32_t check_every, int32_t *iters_done_host, double *residual_host,
                   void *stream)
{
    if (!iters_done_host || !residual_host) return fail(NMF_EINVAL, "null pointer%s");
    if (check_every < 1) return fail(NMF_EINVAL, "check_every must be >= 1%s");
    if (!(tol >= 0.0)) return fail(NMF_EINVAL, "tol must be >= 0%s");
    const CsrTol t = {tol, check_every, iters_done_host, residual_host};
    *iters_done_host = 0;
    return csr_run(rowptr, colidx, vals, m, n, nnz, k, W, H, max_iters, eps, nullptr, stream, &t);
}

// Out-of-memory CSR: row batches of about batch_nnz stored entries each, streamed from host
// memory every sweep in the order of nmf_mu_ooc (W update of the batch with the current H, then
// the batch's share of W^T A for the next H update).  A batch is a CSR matrix of its own once
// its row pointers are made relative; its column-ordered copy is rebuilt on the device each
// time (a sort of the batch, which runs beside the upload of the next one).
int nmf_mu_csr_ooc(const int64_t *rowptr_host, const int32_t *colidx_host, const float *vals_host,
                   int64_t m, int64_t n, int64_t nnz, int32_t k, float *W, float *H, int32_t iters,
                   float eps, int64_t batch_nnz, int64_t device_budget_bytes, void *stream)
{
    if (!rowptr_host) return fail(NMF_EINVAL, "null pointer%s");
    if (nnz < 0) return fail(NMF_EINVAL, "nnz must be >= 0%s");
    if (nnz > 0 && (!colidx_host || !vals_host)) return fail(NMF_EINVAL, "null pointer%s");
    if (int rc = check_common(rowptr_host, W, H, m, n, k, iters, eps)) return rc;
    if (batch_nnz < 1) return fail(NMF_EINVAL, "batch_nnz must be >= 1%s");
    if (device_budget_bytes < 1) return fail(NMF_EINVAL, "device_budget_bytes must be >= 1%s");
    if (m >= ((int64_t)1 << 31)) return fail(NMF_EUNSUPPORTED, "CSR path needs m < 2^31%s");
    if (iters == 0) return NMF_OK;
    if (rowptr_host[0] != 0 || rowptr_host[m] != nnz) return fail(NMF_EINVAL, "rowptr[0] != 0 or rowptr[m] != nnz%s");
    hipStream_t st = static_cast<hipStream_t>(stream);

    // Row batches: as many whole rows as fit batch_nnz entries, at least one row.
    struct Batch { int64_t r0, r1, e0, e1; };
    std::vector<Batch> batches;
    int64_t max_rows = 1, max_nnz = 1;
    for (int64_t r0 = 0; r0 < m;) {
        const int64_t e0 = rowptr_host[r0];
        const int64_t *hi = std::upper_bound(rowptr_host + r0 + 1, rowptr_host + m + 1, e0 + batch_nnz);
        int64_t r1 = (hi - rowptr_host) - 1;
        if (r1 <= r0) r1 = r0 + 1;
        const int64_t e1 = rowptr_host[r1];
        if (e1 < e0) return fail(NMF_EINVAL, "rowptr is not non-decreasing%s");
        if (e1 - e0 >= ((int64_t)1 << 31)) return fail(NMF_EUNSUPPORTED, "a row batch needs fewer than 2^31 entries%s");
        batches.push_back({r0, r1, e0, e1});
        if (r1 - r0 > max_rows) max_rows = r1 - r0;
        if (e1 - e0 > max_nnz) max_nnz = e1 - e0;
        r0 = r1;
    }
    const size_t rp_bytes = align_up((size_t)(max_rows + 1) * sizeof(int64_t));
    const size_t ci_bytes = align_up((size_t)max_nnz * sizeof(int32_t));
    const size_t va_bytes = align_up((size_t)max_nnz * sizeof(float));
    const size_t slot_bytes = rp_bytes + ci_bytes + va_bytes;
    int slots = (int)((size_t)device_budget_bytes / slot_bytes);
    if (slots < 1) return fail(NMF_ENOMEM, "device budget does not hold one batch%s");
    if (slots > 3) slots = 3;

    std::lock_guard<std::mutex> lock(g.mu);
    const size_t temp_bytes = csc_sort_temp_bytes(max_nnz, n);
    const size_t need = common_bytes(k) + 2 * align_up((size_t)n * k * sizeof(float)) + rp_bytes +
                        align_up((size_t)(n + 1) * sizeof(int64_t)) + 2 * ci_bytes + va_bytes +
                        2 * align_up((size_t)max_nnz * sizeof(uint64_t)) + align_up(temp_bytes) +
                        2 * align_up((size_t)(kCsrParts + 1) * sizeof(int64_t)) +
                        2 * align_up((size_t)(max_nnz / kLongRow + 2) * sizeof(int32_t)) + kAlign;
    void *ws = nullptr;
    if (int rc = ensure_workspace(need, &ws)) return rc;
    Carve cv(ws);
    const Common c = carve_common(cv, k);
    float *Ht = cv.take<float>((size_t)n * k);
    float *Num = cv.take<float>((size_t)n * k);
    int64_t *rowptr_loc = cv.take<int64_t>((size_t)max_rows + 1);
    int64_t *colptr = cv.take<int64_t>((size_t)n + 1);
    int32_t *rowidx = cv.take<int32_t>((size_t)max_nnz);
    float *cvals = cv.take<float>((size_t)max_nnz);
    int32_t *sorted_cols = cv.take<int32_t>((size_t)max_nnz);
    uint64_t *payload = cv.take<uint64_t>((size_t)max_nnz);
    uint64_t *sorted_payload = cv.take<uint64_t>((size_t)max_nnz);
    char *sort_temp = cv.take<char>(temp_bytes);
    int64_t *part_r = cv.take<int64_t>((size_t)kCsrParts + 1);
    int64_t *part_c = cv.take<int64_t>((size_t)kCsrParts + 1);
    int32_t *long_r = cv.take<int32_t>((size_t)(max_nnz / kLongRow + 2));
    int32_t *long_c = cv.take<int32_t>((size_t)(max_nnz / kLongRow + 2));
    unsigned *long_n = cv.take<unsigned>(64);
    if (cv.off > need) return fail(NMF_EHIP, "internal: csr_ooc workspace accounting%s");

    if (g.sl_stage_bytes < slots * slot_bytes) {
        if (g.sl_stage) {
            NMF_HIP(hipDeviceSynchronize());
            NMF_HIP(hipFree(g.sl_stage));
            g.sl_stage = nullptr;
            g.sl_stage_bytes = 0;
        }
        hipError_t e = hipMalloc(&g.sl_stage, slots * slot_bytes);
        if (e != hipSuccess) return fail(NMF_ENOMEM, "hipMalloc(staging): %s", hipGetErrorString(e));
        g.sl_stage_bytes = slots * slot_bytes;
    }
    if (!g.copy_stream) NMF_HIP(hipStreamCreateWithFlags(&g.copy_stream, hipStreamNonBlocking));
    if (!g.ev_entry) NMF_HIP(hipEventCreateWithFlags(&g.ev_entry, hipEventDisableTiming));
    for (int i = 0; i < 3; ++i) {
        if (!g.sl_copied[i]) NMF_HIP(hipEventCreateWithFlags(&g.sl_copied[i], hipEventDisableTiming));
        if (!g.sl_freed[i]) NMF_HIP(hipEventCreateWithFlags(&g.sl_freed[i], hipEventDisableTiming));
    }
    NMF_HIP(hipEventRecord(g.ev_entry, st));
    NMF_HIP(hipStreamWaitEvent(g.copy_stream, g.ev_entry, 0));

    NMF_HIP(launch_fill_f32(reinterpret_cast<float *>(c.counters), 64, 0.f, st));      // as in csr_run
    NMF_HIP(launch_transpose(H, k, n, Ht, st));
    int64_t issued = 0;
    for (int s = 0; s <= iters; ++s) {
        if (s < iters) NMF_HIP(launch_fill_f32(Num, n * (int64_t)k, 0.f, st));
        for (size_t b = 0; b < batches.size(); ++b, ++issued) {
            const Batch &bt = batches[b];
            const int64_t rows = bt.r1 - bt.r0, cnt = bt.e1 - bt.e0;
            const int slot = (int)(issued % slots);
            char *base = static_cast<char *>(g.sl_stage) + slot * slot_bytes;
            int64_t *rp = reinterpret_cast<int64_t *>(base);
            int32_t *ci = reinterpret_cast<int32_t *>(base + rp_bytes);
            float *va = reinterpret_cast<float *>(base + rp_bytes + ci_bytes);
            if (issued >= slots) NMF_HIP(hipStreamWaitEvent(g.copy_stream, g.sl_freed[slot], 0));
            NMF_HIP(hipMemcpyAsync(rp, rowptr_host + bt.r0, (size_t)(rows + 1) * sizeof(int64_t),
                                   hipMemcpyHostToDevice, g.copy_stream));
            if (cnt > 0) {
                NMF_HIP(hipMemcpyAsync(ci, colidx_host + bt.e0, (size_t)cnt * sizeof(int32_t),
                                       hipMemcpyHostToDevice, g.copy_stream));
                NMF_HIP(hipMemcpyAsync(va, vals_host + bt.e0, (size_t)cnt * sizeof(float),
                                       hipMemcpyHostToDevice, g.copy_stream));
            }
            NMF_HIP(hipEventRecord(g.sl_copied[slot], g.copy_stream));
            NMF_HIP(hipStreamWaitEvent(st, g.sl_copied[slot], 0));
            NMF_HIP(launch_rebase_i64(rp, rows + 1, bt.e0, rowptr_loc, st));
            float *Wb = W + bt.r0 * k;
            if (s > 0) {
                NMF_HIP(launch_csr_partition(rowptr_loc, rows, kCsrParts, part_r, st));
                NMF_HIP(launch_csr_long_rows(rowptr_loc, rows, long_r, long_n, (unsigned)(max_nnz / kLongRow + 1), st));
                NMF_HIP(launch_aht_csr(rowptr_loc, ci, va, part_r, long_r, long_n, k, Ht, c.gh, Wb, eps, cnt, rows, n, st));
            }
            if (s < iters) {
                NMF_HIP(launch_csc_build(rowptr_loc, ci, va, rows, n, cnt, sorted_cols, payload, sorted_payload,
                                         sort_temp, temp_bytes, colptr, rowidx, cvals, st));
                NMF_HIP(launch_csr_partition(colptr, n, kCsrParts, part_c, st));
                NMF_HIP(launch_csr_long_rows(colptr, n, long_c, long_n + 1, (unsigned)(max_nnz / kLongRow + 1), st));
                NMF_HIP(launch_aht_csr(colptr, rowidx, cvals, part_c, long_c, long_n + 1, k, Wb, nullptr, Num, eps,
                                       cnt, n, rows, st, true));
            }
            NMF_HIP(hipEventRecord(g.sl_freed[slot], st));
        }
        if (s < iters) {
            NMF_HIP(launch_gram_w_wide(W, m, k, c.gw, c.gwp, c.counters, st));
            NMF_HIP(launch_row_update(Ht, Num, c.gw, k, n, eps, st));
            NMF_HIP(launch_gram_w_wide(Ht, n, k, c.gh, c.ghp, c.counters, st));
        }
    }
    NMF_HIP(launch_transpose(Ht, n, k, H, st));
    return NMF_OK;
}

// ---- objective and tolerance-driven run ---------------------------------------

namespace {
// Host memory for the few doubles a blocking call waits for, written by the kernel that has them: a copy to the caller's
// pageable memory costs 8 us more.  Null if there is none (the value is then copied).  Used under the lock only, which a
// blocking call holds until it has read the value.
double *pinned_doubles()
{
    if (!g.pinned && hipHostMalloc(reinterpret_cast<void **>(&g.pinned), kAlign, hipHostMallocPortable | hipHostMallocMapped) != hipSuccess) {
        (void)hipGetLastError();
        g.pinned = nullptr;
    }
    return g.pinned;
}

// Waits for `st` and reads the double that a kernel on it wrote to `at` (pinned host memory or device memory).
int read_double(const double *at, double *out_host, hipStream_t st)
{
    const bool host = g.pinned && at >= g.pinned && at < g.pinned + kAlign / sizeof(double);
    if (!host) NMF_HIP(hipMemcpyAsync(out_host, at, sizeof(double), hipMemcpyDeviceToHost, st));
    NMF_HIP(hipStreamSynchronize(st));
    if (host) *out_host = *static_cast<const volatile double *>(at);
    return NMF_OK;
}

// ||A - W H||_F into *out_host; synchronises `st`.  Scratch sits behind the dense plan.
int residual_to_host(const float *A, int64_t m, int64_t n, int k, const float *W, const float *H,
                     double *scratch, double *out_host, hipStream_t st)
{
    double *pin = pinned_doubles(), *out = pin ? pin : scratch;
    NMF_HIP(launch_residual(A, m, n, k, W, H, scratch + 1, out, st));
    return read_double(out, out_host, st);
}
// the same for a run that may work on a copy of A with padded columns
size_t run_scratch_bytes(int64_t m, int64_t n)
{
    const int64_t a = residual_partials(m, n), b = residual_partials(m, (n + 3) & ~(int64_t)3);
    return align_up(((size_t)(a > b ? a : b) + 1) * sizeof(double));
}
size_t residual_scratch_bytes(int64_t m, int64_t n) { return align_up(((size_t)residual_partials(m, n) + 1) * sizeof(double)); }
}  // namespace

int nmf_residual_dense(const float *A, int64_t m, int64_t n, int32_t k, const float *W,
                       const float *H, double *residual_host, void *stream)
{
    if (int rc = check_common(A, W, H, m, n, k, 0, 0.f)) return rc;
    if (!residual_host) return fail(NMF_EINVAL, "null pointer%s");
    std::lock_guard<std::mutex> lock(g.mu);
    void *ws = nullptr;
    if (int rc = ensure_workspace(kAlign + residual_scratch_bytes(m, n), &ws)) return rc;
    Carve cv(ws);
    cv.take<unsigned>(64);   // the arrival counters at the head of the workspace stay untouched
    double *scratch = cv.take<double>((size_t)residual_partials(m, n) + 1);
    return residual_to_host(A, m, n, k, W, H, scratch, residual_host, static_cast<hipStream_t>(stream));
}

int nmf_mu_dense_tol(const float *A, int64_t m, int64_t n, int32_t k, float *W, float *H,
                     int32_t max_iters, float eps, double tol, int32_t check_every,
                     int32_t *iters_done_host, double *residual_host, void *stream)
{
    if (int rc = check_common(A, W, H, m, n, k, max_iters, eps)) return rc;
    if (!iters_done_host || !residual_host) return fail(NMF_EINVAL, "null pointer%s");
    if (!(tol >= 0.0) || check_every < 1) return fail(NMF_EINVAL, "tol must be >= 0 and check_every >= 1%s");
    hipStream_t st = static_cast<hipStream_t>(stream);
    std::lock_guard<std::mutex> lock(g.mu);
    // the residual scratch and the monitor's few doubles ride behind whichever dense plan fits
    const size_t extra = run_scratch_bytes(m, n) + align_up((size_t)kFinMaxBlocks * sizeof(double)) +
                         align_up(4097 * sizeof(double)) + kAlign;
    DenseRun r;
    if (int rc = open_run(A, m, n, k, W, H, max_iters, eps, extra, st, &r, true)) return rc;
    const bool mirrored = r.p.mirrored;
    // plans whose W update leaves the objective's terms behind
    const bool fast = mirrored || r.p.one_pass || r.p.resident || rows_plan_runs(r.A, m, r.n, k, mirrored);
    Carve cv(r.tail);
    double *scratch = cv.take<double>(run_scratch_bytes(m, n) / sizeof(double));
    Monitor mon;
    mon.dpart = cv.take<double>(kFinMaxBlocks);
    mon.normA2 = cv.take<double>(4097);
    mon.out = cv.take<double>(1);
    if (double *pin = pinned_doubles()) mon.out = pin + 1;
    mon.res = scratch;
    mon.last_only = true;
    int done = 0;
    double res = 0.0;
    bool exact = true;       // `res` comes from the tiled evaluation (not from the expansion)
    if (int rc = residual_to_host(r.A, m, r.n, k, r.W, r.H, scratch, &res, st)) return rc;
    double normA2 = 0.0;
    if (fast && max_iters > 0 && res > tol) {
        NMF_HIP(launch_sumsq(r.A, m * r.n, mon.normA2 + 1, mon.normA2, st));
        NMF_HIP(hipMemcpyAsync(&normA2, mon.normA2, sizeof(double), hipMemcpyDeviceToHost, st));
        NMF_HIP(hipStreamSynchronize(st));
    }
    bool have_at = r.have_at;
    while (done < max_iters && res > tol) {
        const int chunk = (max_iters - done < check_every) ? max_iters - done : check_every;
        if (int rc = dense_body(r.A, r.m, r.n, k, r.W, r.H, chunk, eps, r.p, st, have_at, nullptr, nullptr, fast ? &mon : nullptr))
            return rc;
        have_at = mirrored;
        done += chunk;
        if (fast) {
            // The objective of the chunk's last iteration from the by-products of its W update
            // (no pass over A); its error is bounded by the fp32 sums of its three terms.  Only
            // when it comes within that bound of the tolerance is the exact value needed.
            double approx = 0.0;
            if (int rc = read_double(mon.out, &approx, st)) return rc;
            const double slack = 1e-3 * approx + 2e-6 * normA2 / (approx > 1e-300 ? approx : 1e-300);
            if (approx > tol + slack) {
                res = approx;
                exact = false;
                continue;
            }
        }
        if (int rc = residual_to_host(r.A, m, r.n, k, r.W, r.H, scratch, &res, st)) return rc;
        exact = true;
    }
    if (!exact)
        if (int rc = residual_to_host(r.A, m, r.n, k, r.W, r.H, scratch, &res, st)) return rc;
    if (int rc = close_run(r, k, W, H, m, n, st)) return rc;
    if (r.W != W || r.H != H) NMF_HIP(hipStreamSynchronize(st));    // blocking also where the factors are copied back
    *iters_done_host = done;
    *residual_host = res;
    return NMF_OK;
}

int nmf_mu_dense_monitor(const float *A, int64_t m, int64_t n, int32_t k, float *W, float *H,
                         int32_t iters, float eps, double *objective_host, void *stream)
{
    if (int rc = check_common(A, W, H, m, n, k, iters, eps)) return rc;
    if (!objective_host) return fail(NMF_EINVAL, "null pointer%s");
    if (iters > (1 << 20)) return fail(NMF_EINVAL, "monitored run: iters <= 2^20%s");
    if (iters == 0) return NMF_OK;
    hipStream_t st = static_cast<hipStream_t>(stream);
    std::lock_guard<std::mutex> lock(g.mu);
    size_t extra = align_up((size_t)kFinMaxBlocks * sizeof(double)) + align_up(4097 * sizeof(double)) +
                   align_up((size_t)iters * sizeof(double)) + run_scratch_bytes(m, n);
    Monitor mon;
    if (resident_tiles(m, n, k) && iters > 1) {
        const int batch = iters < kMonitored ? iters : kMonitored;
        const size_t more = monitored_bytes(batch, k);
        if (have_workspace(resident_bytes(m, n, k) + extra + more, st)) {
            mon.batch = batch;
            extra += more;
        }
    }
    DenseRun r;
    if (int rc = open_run(A, m, n, k, W, H, iters, eps, extra, st, &r)) return rc;
    Carve cv(r.tail);
    mon.dpart = cv.take<double>((size_t)mon.batch * kFinMaxBlocks);
    if (mon.batch > 1) {
        mon.gw = cv.take<float>((size_t)mon.batch * k * k);
        mon.gh = cv.take<float>((size_t)mon.batch * k * k);
    }
    mon.normA2 = cv.take<double>(4097);
    mon.out = cv.take<double>((size_t)iters);
    mon.res = cv.take<double>(run_scratch_bytes(m, n) / sizeof(double));
    mon.last_only = false;
    if (r.p.mirrored || r.p.one_pass || r.p.resident || rows_plan_runs(r.A, m, r.n, k, r.p.mirrored))
        NMF_HIP(launch_sumsq(r.A, m * r.n, mon.normA2 + 1, mon.normA2, st));
    if (int rc = dense_body(r.A, r.m, r.n, k, r.W, r.H, iters, eps, r.p, st, r.have_at, nullptr, nullptr, &mon)) return rc;
    if (int rc = close_run(r, k, W, H, m, n, st)) return rc;
    NMF_HIP(hipMemcpyAsync(objective_host, mon.out, (size_t)iters * sizeof(double), hipMemcpyDeviceToHost, st));
    NMF_HIP(hipStreamSynchronize(st));
    return NMF_OK;
}

// ---- allocation-free resident dense run --------------------------------------

int nmf_mu_dense_noalloc(const float *A, int64_t m, int64_t n, int32_t k, float *W, float *H,
                         int32_t iters, float eps, void *stream)
{
    if (int rc = check_common(A, W, H, m, n, k, iters, eps)) return rc;
    if (dense_bytes(m, n, k, false) > kScratchBytes)
        return fail(NMF_ENOMEM, "problem needs more than the fixed scratch array of nmf_mu_dense_noalloc "
                                "(see nmf_mu_workspace_bytes kind 4)%s");
    if (iters == 0) return NMF_OK;
    void *ws = nullptr;
    if (int rc = scratch_address(&ws)) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    // The arrival counters at the head of the array must read zero when the first kernel starts;
    // the kernels restore that, but an earlier call may have been cut short.  A fill kernel, not
    // a memset: the call may be under graph capture.
    NMF_HIP(launch_fill_f32(static_cast<float *>(ws), 64, 0.f, st));
    const int tiles = resident_tiles(m, n, k);
    if (tiles && resident_bytes(m, n, k) <= kScratchBytes) {
        Carve cv(ws);
        return dense_body(A, m, n, k, W, H, iters, eps, carve_resident(cv, m, n, k, tiles), st);
    }
    const bool one = one_pass_ok(A, n, k) && one_pass_bytes(m, n, k) <= kScratchBytes;
    const DensePlan p = one ? carve_one_pass(ws, m, n, k) : carve_dense(ws, m, n, k, false);
    return dense_body(A, m, n, k, W, H, iters, eps, p, st);
}

// ---- single steps ----------------------------------------------------------

int nmfmu_dense_plan(const float *A, int64_t m, int64_t n, int32_t k, float *W, float *H, int32_t iters, float eps,
                     int32_t *plan, void *stream)
{
    if (int rc = check_common(A, W, H, m, n, k, iters, eps)) return rc;
    if (!plan) return fail(NMF_EINVAL, "null pointer%s");
    std::lock_guard<std::mutex> lock(g.mu);
    DenseRun r;
    if (int rc = open_run(A, m, n, k, W, H, iters, eps, 0, static_cast<hipStream_t>(stream), &r)) return rc;
    *plan = r.p.resident ? 4 : r.p.one_pass ? 3 : takes_row_plan(r.p, r.A, r.m, r.n, k) ? 2 : r.p.mirrored ? 1 : 0;
    if (r.A != A || r.W != W || r.H != H) *plan += 8;
    if (r.p.pairs) *plan += 16;
    return NMF_OK;
}

static int resident_hook(const float *A, int64_t m, int64_t n, int k, float *W, float *H, int iters, float eps, int workgroups,
                         long long patience, unsigned polls, hipStream_t st)
{
    if (int rc = check_common(A, W, H, m, n, k, iters, eps)) return rc;
    const int tiles = resident_tiles(m, n, k);
    if (!tiles) return fail(NMF_EUNSUPPORTED, "not a shape of the resident plan%s");
    if (iters == 0) return NMF_OK;
    std::lock_guard<std::mutex> lock(g.mu);
    void *ws = nullptr;
    if (int rc = ensure_workspace(resident_bytes(m, n, k), &ws)) return rc;
    Carve cv(ws);
    ResidentArgs a = carve_resident(cv, m, n, k, tiles).res;
    a.A = A, a.Win = a.W = W, a.Hin = a.H = H;
    a.m = m, a.n = n, a.k = k, a.eps = eps, a.nprod = iters, a.patience = patience, a.polls = polls;
    NMF_HIP(launch_resident_run(a, tiles, st, workgroups));
    return NMF_OK;
}

int nmfmu_resident_by_one(const float *A, int64_t m, int64_t n, int32_t k, float *W, float *H, int32_t iters, float eps,
                          void *stream)
{
    return resident_hook(A, m, n, k, W, H, iters, eps, 1, 0, 0, static_cast<hipStream_t>(stream));
}

int nmfmu_resident_shared(const float *A, int64_t m, int64_t n, int32_t k, float *W, float *H, int32_t iters, float eps,
                          int32_t workgroups, int64_t patience, void *stream)
{
    return resident_hook(A, m, n, k, W, H, iters, eps, workgroups, patience, 0, static_cast<hipStream_t>(stream));
}

int nmfmu_resident_polls(const float *A, int64_t m, int64_t n, int32_t k, float *W, float *H, int32_t iters, float eps,
                         uint32_t polls, void *stream)
{
    return resident_hook(A, m, n, k, W, H, iters, eps, 0, 0, polls, static_cast<hipStream_t>(stream));
}

int nmf_csr_partition(const int64_t *rowptr, int64_t m, int32_t nparts, int64_t *part, void *stream)
{
    if (!rowptr || !part) return fail(NMF_EINVAL, "null pointer%s");
    if (m < 1 || nparts < 1) return fail(NMF_EINVAL, "bad size%s");
    NMF_HIP(launch_csr_partition(rowptr, m, nparts, part, static_cast<hipStream_t>(stream)));
    return NMF_OK;
}

int nmf_split_planes(const float *X, int64_t rows, int32_t k, uint16_t *planes, void *stream)
{
    if (!X || !planes) return fail(NMF_EINVAL, "null pointer%s");
    if (rows < 1 || k < 1) return fail(NMF_EINVAL, "bad size%s");
    if (!wta_uses_planes(k)) return fail(NMF_EUNSUPPORTED, "piece planes are used for k <= 64 only%s");
    if (reinterpret_cast<uintptr_t>(planes) % 16) return fail(NMF_EINVAL, "planes must be 16-byte aligned%s");
    NMF_HIP(launch_split_planes(X, rows, k, planes, static_cast<hipStream_t>(stream)));
    return NMF_OK;
}

int nmf_csr_to_csc(const int64_t *rowptr, const int32_t *colidx, const float *vals, int64_t m,
                   int64_t n, int64_t nnz, int64_t *colptr, int32_t *rowidx, float *cvals,
                   void *stream)
{
    if (!rowptr || !colptr) return fail(NMF_EINVAL, "null pointer%s");
    if (m < 1 || n < 1 || nnz < 0) return fail(NMF_EINVAL, "bad size%s");
    if (nnz > 0 && (!colidx || !vals || !rowidx || !cvals)) return fail(NMF_EINVAL, "null pointer%s");
    if (nnz >= ((int64_t)1 << 31) || m >= ((int64_t)1 << 31))
        return fail(NMF_EUNSUPPORTED, "CSR path needs nnz < 2^31 and m < 2^31%s");
    return build_csc(rowptr, colidx, vals, m, n, nnz, colptr, rowidx, cvals,
                     static_cast<hipStream_t>(stream));
}

int nmf_gram_w(const float *W, int64_t m, int32_t k, float *G, void *stream)
{
    if (int rc = check_common(W, W, G, m, 1, k, 0, 0.f)) return rc;
    std::lock_guard<std::mutex> lock(g.mu);
    void *ws = nullptr;
    if (int rc = ensure_workspace(common_bytes(k), &ws)) return rc;
    Carve cv(ws);
    const Common c = carve_common(cv, k);
    NMF_HIP(launch_gram_w(W, m, k, G, c.gpart, c.counters, static_cast<hipStream_t>(stream)));
    return NMF_OK;
}

int nmf_wta_dense(const float *A, int64_t m, int64_t n, int32_t k, const float *W, float *P,
                  void *stream)
{
    if (int rc = check_common(A, W, P, m, n, k, 0, 0.f)) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    std::lock_guard<std::mutex> lock(g.mu);
    void *ws = nullptr;
    if (int rc = ensure_workspace(dense_bytes(m, n, k, false), &ws)) return rc;
    Carve cv(ws);
    carve_common(cv, k);
    const int splits = wta_splits(m, n, k);
    float *ppart = cv.take<float>((size_t)splits * k * n);
    void *planes = cv.take<char>(planes_bytes(m));
    NMF_HIP(launch_wta_pass(A, m, n, k, W, planes, false, ppart, splits, wta_rows_per_split(m, splits), false, st));
    NMF_HIP(launch_sum_partials(ppart, splits, (int64_t)k * n, P, st));
    return NMF_OK;
}

int nmf_h_update(float *H, const float *P, const float *G, int32_t k, int64_t n, float eps,
                 float *GH, void *stream)
{
    if (int rc = check_common(H, P, G, 1, n, k, 0, eps)) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    std::lock_guard<std::mutex> lock(g.mu);
    void *ws = nullptr;
    if (int rc = ensure_workspace(common_bytes(k), &ws)) return rc;
    Carve cv(ws);
    const Common c = carve_common(cv, k);
    NMF_HIP(launch_factor_update(H, nullptr, P, 1, G, nullptr, 0, nullptr, k, n, eps, st));
    if (GH) NMF_HIP(launch_gram_h(H, k, n, GH, c.gpart, c.counters, st));
    return NMF_OK;
}

int nmf_aht_w_update_dense(const float *A, int64_t m, int64_t n, int32_t k, const float *H,
                           const float *GH, float *W, float eps, void *stream)
{
    if (int rc = check_common(A, W, H, m, n, k, 0, eps)) return rc;
    if (!GH) return fail(NMF_EINVAL, "null pointer%s");
    NMF_HIP(launch_aht_pass(A, m, n, k, H, GH, W, eps, static_cast<hipStream_t>(stream)));
    return NMF_OK;
}

}  // extern "C"
