"""Products on pairs of halves over data whose parts lie many powers of two apart: what the halves cannot hold has to come out right
all the same, part by part."""
import numpy as np
import pytest

EPS = 1e-16


def reference(A, W, H, iters):
    A, W, H = (x.astype(np.float64) for x in (A, W, H))
    eps = float(np.float32(EPS))
    for _ in range(iters):
        H = H * (W.T @ A) / ((W.T @ W) @ H + eps)
        W = W * (A @ H.T) / (W @ (H @ H.T) + eps)
    return W, H


def off(got, want):
    return np.linalg.norm(got.astype(np.float64) - want) / np.linalg.norm(want)


def dense(A, W, H, iters):
    import torch

    import paper_2202_09518_amd as nmf
    Wd, Hd = torch.from_numpy(W).cuda(), torch.from_numpy(H).cuda()
    nmf.nmf_mu_dense(torch.from_numpy(A).cuda(), A.shape[0], A.shape[1], W.shape[1], Wd, Hd, iters, EPS)
    return Wd.cpu().numpy(), Hd.cpu().numpy()


def stacked(A, Ws, Hs, iters):
    import torch

    import paper_2202_09518_amd as nmf
    Ad = torch.from_numpy(A).cuda()
    Wd, Hd = [torch.from_numpy(w).cuda() for w in Ws], [torch.from_numpy(h).cuda() for h in Hs]
    nmf.nmf_mu_dense_batched(len(Ws), [Ad] * len(Ws), A.shape[0], A.shape[1], [w.shape[1] for w in Ws], Wd, Hd, iters, EPS)
    return [w.cpu().numpy() for w in Wd], [h.cpu().numpy() for h in Hd]


def streamed(A, W, H, iters):
    import torch

    import paper_2202_09518_amd as nmf
    Ah = torch.empty(A.shape, pin_memory=True)
    Ah.copy_(torch.from_numpy(A))
    Wd, Hd = torch.from_numpy(W).cuda(), torch.from_numpy(H).cuda()
    m, n = A.shape
    nmf.nmf_mu_ooc(Ah, m, n, W.shape[1], Wd, Hd, iters, EPS, 128, 3 * 128 * n * 4 + 1024)
    return Wd.cpu().numpy(), Hd.cpu().numpy()


def brought_to_column_scale(x, top):
    """Halves of units of 8 entries (rows of x), each cut under its own scale, brought to that of a column whose largest entry has
    exponent `top`, as the kernels do it; also the entries in that range."""
    e = np.floor(np.log2(np.abs(x).max(axis=1))).astype(int)
    s = np.ldexp(x.astype(np.float64), (14 - e)[:, None])
    h = s.astype(np.float16)
    low = (s - h.astype(np.float64)).astype(np.float32).astype(np.float16)
    d = np.minimum(top - e, 40)
    r1, r2 = np.ldexp(1.0, -(d >> 1)).astype(np.float16)[:, None], np.ldexp(1.0, (d >> 1) - d).astype(np.float16)[:, None]
    pieces = [(p * r1) * r2 for p in (h, low)]
    assert all(p.dtype == np.float16 for p in pieces)
    return np.ldexp(x.astype(np.float64), 14 - top), sum(p.astype(np.float64) for p in pieces)


def test_what_the_column_scale_leaves_out():
    r = np.random.default_rng(2)
    for d in range(46):
        x = np.ldexp(r.random((4000, 8)) + 1, -d - r.integers(0, 30, (4000, 8))).astype(np.float32)
        x[:, 0] = np.ldexp(r.random(4000) + 1, -d)
        want, got = brought_to_column_scale(x, 0)
        assert (np.abs(want - got) <= np.maximum(np.ldexp(want, -22), np.ldexp(1.0, -23))).all()
        if d < 38:
            assert (got[:, 0] > 0).all()      # the largest of a unit is there 2^38 below the largest of its column
    # so 128 products of scaled entries are off by less than a 2^-22nd of a sum that counts as sure
    assert 128 * 2.0**15 * (2.0**-23 + 2.0**-25) < 1


def two_blocks(r, m, n, s, permuted):
    """Two dense blocks on the diagonal, the second s times as large; which rows and columns are the second's."""
    rows, cols = np.arange(m) >= m // 2, np.arange(n) >= n // 2
    if permuted:
        rows, cols = rows[r.permutation(m)], cols[r.permutation(n)]
    A = r.random((m, n), dtype=np.float32)
    A *= np.where(rows[:, None] == cols, np.where(rows[:, None], np.float32(s), np.float32(1)), np.float32(0))
    return A, rows, cols


def check_blocks(W, H, Wr, Hr, rows, cols, tol):
    for part in (False, True):
        assert off(H[:, cols == part], Hr[:, cols == part]) < tol
        assert off(W[rows == part], Wr[rows == part]) < tol


# The multiplicative update drives the factors of the smaller block through a wide range by itself.  While it does, what W and H are off
# by goes into each other's next update, H' = H (W ..) and then W' = W (H' ..), so that it grows by up to ((1 + 5^0.5) / 2)^2 = 2.6 an
# iteration: 2^-24 becomes 8e-4 in ten at most.  Exact products of bf16 pieces are 2.0e-5 off in the worst of these cases, at ten iterations;
# four times that.  A block that is lost is off by 1.
TOL = 8e-5


@pytest.mark.gpu
@pytest.mark.parametrize("permuted", [False, True])
@pytest.mark.parametrize("s,iters", [(0.2, 5), (0.2, 10), (0.2, 50), (0.07, 5), (0.07, 10), (0.07, 50), (0.02, 5)])     # 0.02: below 1e-38 by 10
@pytest.mark.parametrize("m,n,k", [(256, 256, 40), (384, 260, 64), (260, 388, 96), (301, 203, 50)])
def test_small_block_beside_a_large_one(m, n, k, s, permuted, iters):
    r = np.random.default_rng(3)
    A, rows, cols = two_blocks(r, m, n, s, permuted)
    W, H = r.random((m, k), dtype=np.float32), r.random((k, n), dtype=np.float32)
    check_blocks(*dense(A, W, H, iters), *reference(A, W, H, iters), rows, cols, TOL)


@pytest.mark.gpu
@pytest.mark.parametrize("iters", [5, 10])
@pytest.mark.parametrize("permuted", [False, True])
@pytest.mark.parametrize("s", [0.2, 0.1])
def test_small_block_in_a_stack(s, permuted, iters):
    m, n, ks = 256, 256, [8, 9, 8, 20, 8, 16, 30]
    r = np.random.default_rng(4)
    A, rows, cols = two_blocks(r, m, n, s, permuted)
    Ws, Hs = [r.random((m, k), dtype=np.float32) for k in ks], [r.random((k, n), dtype=np.float32) for k in ks]
    got = stacked(A, Ws, Hs, iters)
    for W, H, Wg, Hg in zip(Ws, Hs, *got):
        check_blocks(Wg, Hg, *reference(A, W, H, iters), rows, cols, TOL)


@pytest.mark.gpu
@pytest.mark.parametrize("iters", [1, 5])
@pytest.mark.parametrize("way", [dense, streamed])
def test_factors_in_units_of_their_own(way, iters):
    """Columns of W in units u and rows of H in 1 / u: every factor's sums are as exact as any other's."""
    m, n, k = 512, 388, 96
    r = np.random.default_rng(5)
    A = (r.random((m, 8)) @ r.random((8, n))).astype(np.float32)
    u = np.ldexp(np.float32(1), r.integers(-25, 26, k)).astype(np.float32)
    W, H = r.random((m, k), dtype=np.float32) * u, r.random((k, n), dtype=np.float32) / u[:, None]
    Wg, Hg = way(A, W, H, iters)
    Wr, Hr = reference(A, W, H, iters)
    for c in range(k):
        assert off(Hg[c], Hr[c]) < 5e-6 and off(Wg[:, c], Wr[:, c]) < 5e-6


@pytest.mark.gpu
@pytest.mark.parametrize("order", [20, 34, 60])
@pytest.mark.parametrize("way,k", [(dense, 40), (dense, 96), (dense, 200), (streamed, 96), ("stack", 50)])
def test_factors_that_leave_out_the_large_rows(way, k, order):
    """Half of the factors are zero on the rows of A that are 2^order times as large: their sums are made of the small rows alone."""
    m, n = 640, 260
    r = np.random.default_rng(6)
    A = r.random((m, n), dtype=np.float32) + np.float32(0.1)
    small = r.random(m) < 0.5
    A[small] *= np.ldexp(np.float32(1), -order)
    W, H = r.random((m, k), dtype=np.float32), r.random((k, n), dtype=np.float32)
    W[np.ix_(~small, np.arange(k) % 2 == 0)] = 0
    if way == "stack":
        (Wg, W2), (Hg, _) = stacked(A, [W, W[:, :10]], [H, H[:10]], 1)
        assert np.isfinite(W2).all()
    else:
        Wg, Hg = way(A, W, H, 1)
    Wr, Hr = reference(A, W, H, 1)
    for part in (0, 1):
        assert off(Hg[part::2], Hr[part::2]) < 5e-6
    assert off(Wg[small], Wr[small]) < 5e-6 and off(Wg[~small], Wr[~small]) < 5e-6


@pytest.mark.gpu
@pytest.mark.parametrize("k", [40, 96])
@pytest.mark.parametrize("a,w", [(122, -8), (-110, 10), (90, -60), (-60, -50)])
def test_ends_of_the_range(k, a, w):
    """A, the factors and all sums are floats; the sums of A alone, or times the largest factor, are not."""
    m, n = 256, 132
    r = np.random.default_rng(7)
    A = np.ldexp(r.random((m, n), dtype=np.float32) + np.float32(0.5), a).astype(np.float32)
    W, H = np.ldexp(r.random((m, k), dtype=np.float32), w).astype(np.float32), r.random((k, n), dtype=np.float32)
    W[3] = np.ldexp(r.random(k, dtype=np.float32), w - 20)
    Wd, Hd = dense(A, W, H, 1)
    Wr, Hr = reference(A, W, H, 1)
    with np.errstate(over="ignore"):
        fits = np.abs(Hr) < 1e38
    assert np.isfinite(Hd[fits]).all()
    if fits.all():
        assert off(Hd, Hr) < 5e-6


@pytest.mark.gpu
@pytest.mark.parametrize("k", [40, 96])
def test_factors_that_are_zero(k):
    m, n = 512, 260
    r = np.random.default_rng(8)
    A = r.random((m, n), dtype=np.float32)
    A[:, 7] = 0
    A[128:256] = 0
    W, H = r.random((m, k), dtype=np.float32), r.random((k, n), dtype=np.float32)
    W[:, 5] = 0
    H[9] = 0
    Wg, Hg = dense(A, W, H, 3)
    Wr, Hr = reference(A, W, H, 3)
    assert off(Hg, Hr) < 5e-6 and off(Wg, Wr) < 5e-6
    assert (Hg[:, 7] == 0).all() and (Wg[128:256] == 0).all() and (Wg[:, 5] == 0).all() and (Hg[9] == 0).all()


# The same over many workgroups: several splits, ragged edges, A along its rows, along its columns four entries at a time and one at
# a time, slices of 128 factors and of 64 side by side.
@pytest.mark.gpu
@pytest.mark.parametrize("m,n,ks", [(5001, 3003, [50]), (4100, 4100, [64]), (3001, 4096, [33]), (8200, 4100, [128]), (8197, 4101, [200]),
                                    (4100, 3000, [20, 30, 14, 40, 24]), (2049, 5003, [64, 64, 33])])
def test_blocks_over_many_workgroups(m, n, ks):
    import torch

    import paper_2202_09518_amd as nmf
    g = torch.Generator(device="cuda")
    g.manual_seed(m + n)
    rows, cols = torch.rand(m, generator=g, device="cuda") < 0.5, torch.rand(n, generator=g, device="cuda") < 0.5
    A = torch.rand((m, n), generator=g, device="cuda")
    A *= (rows[:, None] == cols).float() * torch.where(rows, 0.07, 1.0)[:, None]
    Ws, Hs = [torch.rand((m, k), generator=g, device="cuda") for k in ks], [torch.rand((k, n), generator=g, device="cuda") for k in ks]
    Wg, Hg = [w.clone() for w in Ws], [h.clone() for h in Hs]
    if len(ks) == 1:
        nmf.nmf_mu_dense(A, m, n, ks[0], Wg[0], Hg[0], 6, EPS)
    else:
        nmf.nmf_mu_dense_batched(len(ks), [A] * len(ks), m, n, ks, Wg, Hg, 6, EPS)
    A = A.double()
    At = A.t().contiguous()
    eps = float(np.float32(EPS))
    for W, H, Wd, Hd in zip(Ws, Hs, Wg, Hg):
        W, Ht = W.double(), H.double().t().contiguous()
        for _ in range(6):
            Ht = Ht * (At @ W) / (Ht @ (W.t().contiguous() @ W) + eps)
            W = W * (A @ Ht) / (W @ (Ht.t().contiguous() @ Ht) + eps)
        for part in (False, True):
            r, c = rows == part, cols == part
            assert ((Wd.double() - W)[r].norm() / W[r].norm()).item() < TOL
            assert ((Hd.double().t() - Ht)[c].norm() / Ht[c].norm()).item() < TOL


# Sums of one sign are as exact as their terms, entry by entry, whatever lies beside them.
@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["A", "W", "H", "all", "rows", "columns", "sparse", "decayed"])
@pytest.mark.parametrize("way,m,n,k", [(dense, 700, 516, 40), (dense, 1301, 333, 64), (dense, 640, 1028, 96), (dense, 333, 700, 130),
                                       (streamed, 640, 260, 70), ("stack", 516, 700, 30)])
def test_every_entry_of_wide_data(way, m, n, k, kind):
    r = np.random.default_rng(9)

    def wide(orders, *shape):
        return np.ldexp(r.random(shape) + 0.5, r.integers(-orders, orders + 1, shape)).astype(np.float32)
    A, W, H = (r.random(s, dtype=np.float32) for s in ((m, n), (m, k), (k, n)))
    if kind in ("A", "all"):
        A = wide(15, m, n)
    if kind in ("W", "all"):
        W = wide(15, m, k)
    if kind in ("H", "all"):
        H = wide(12, k, n)
    if kind == "rows":
        A *= wide(25, m, 1)
    elif kind == "columns":
        A *= wide(25, 1, n)
    elif kind == "sparse":
        A, W = wide(20, m, n) * (r.random((m, n)) < 0.05), wide(20, m, k) * (r.random((m, k)) < 0.05) + np.float32(1e-12) * W
    elif kind == "decayed":
        A, W, H = A * (r.random((m, n)) < 0.3), np.exp2(-60 * W), np.exp2(-30 * H)
    A, W, H = (np.ascontiguousarray(x, dtype=np.float32) for x in (A, W, H))
    if way == "stack":
        got = [x[0] for x in stacked(A, [W, W[:, :20].copy()], [H, H[:20].copy()], 1)]
    else:
        got = way(A, W, H, 1)
    for x, want in zip(got, reference(A, W, H, 1)):
        live = (want > 1e-25) & (want < 1e30)
        assert live.any() and (np.abs(x - want)[live] <= 6e-6 * want[live]).all()      # 2e-6 at most on exact pieces
