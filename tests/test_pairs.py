"""Pairs of halves: what the two pieces of a scaled float hold, and the scales that follow the data."""
import numpy as np
import pytest

EPS = 1e-16


def cut(x, e):
    """Pieces of x under the scale 2^(14 - e), as the kernels cut them."""
    s = np.ldexp(x.astype(np.float64), 14 - e)
    h = s.astype(np.float16)
    low = (s - h.astype(np.float64)).astype(np.float32).astype(np.float16)
    return s, h.astype(np.float64), low.astype(np.float64)


def test_two_halves_hold_a_float_to_its_last_bit():
    r = np.random.default_rng(1)
    x = r.random(200000).astype(np.float32) + np.float32(1)           # [1, 2): exponent 0 under any scale above its own
    for e in (0, 3, 10):
        s, h, low = cut(x, e)
        ulp = np.ldexp(1.0, 14 - e - 23)
        err = s - h - low
        assert np.abs(err).max() <= ulp                                # the neighbour at worst,
        assert (err == 0).mean() > 0.7                                 # and three quarters exact
        assert abs(err.mean()) < 0.01 * ulp                            # of either sign
        # the product left out: the lower pieces of both operands
        assert np.abs(low).max() <= np.ldexp(1.0, 14 - e - 11)


def test_small_entries_keep_an_absolute_error_of_the_largest():
    r = np.random.default_rng(2)
    x = np.ldexp(r.random(200000) + 1, r.integers(-60, 1, 200000)).astype(np.float32)
    s, h, low = cut(x, 0)
    err = np.abs(s - h - low)
    assert (err <= np.maximum(np.ldexp(s, -23), np.ldexp(1.0, -25))).all()


def reference(A, W, H):
    A, W, H = (x.astype(np.float64) for x in (A, W, H))
    eps = float(np.float32(EPS))
    H = H * (W.T @ A) / ((W.T @ W) @ H + eps)
    W = W * (A @ H.T) / (W @ (H @ H.T) + eps)
    return W, H


def plan_of(A, m, n, k, W, H, iters):
    import ctypes

    import torch

    import paper_2202_09518_amd as nmf
    fn = nmf.lib().nmfmu_dense_plan
    fn.argtypes = [ctypes.c_void_p, ctypes.c_int64, ctypes.c_int64, ctypes.c_int32, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int32,
                   ctypes.c_float, ctypes.POINTER(ctypes.c_int32), ctypes.c_void_p]
    plan = ctypes.c_int32(-1)
    assert fn(A.data_ptr(), m, n, k, W.data_ptr(), H.data_ptr(), iters, EPS, ctypes.byref(plan), torch.cuda.current_stream().cuda_stream) == 0
    return plan.value


def columns_off(got, want):
    """Largest relative error of a column (2-norm)."""
    d = np.linalg.norm(got.astype(np.float64) - want, axis=0) / np.linalg.norm(want, axis=0)
    return d.max()


# odd sizes, ranks that fill one slice and part of the next; sizes at which the other paths of a product run.  Up to 64 factors two iterations
# where one would not earn the cut of a matrix that is not aligned.
@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["plain", "columns", "rows", "growing", "late", "spikes"])
@pytest.mark.parametrize("m,n,k", [(1300, 516, 68), (517, 1028, 132), (700, 333, 96), (900, 1030, 200),      # above 64
                                   (1300, 2516, 33), (517, 1029, 64), (128, 257, 40), (1, 300, 50)])          # up to 64
def test_scales_follow_the_data(m, n, k, kind):
    import torch

    import paper_2202_09518_amd as nmf
    r = np.random.default_rng(7)
    A = (r.random((m, 8)) @ r.random((8, n))).astype(np.float32)
    W, H = r.random((m, k), dtype=np.float32), r.random((k, n), dtype=np.float32)
    if kind == "columns":       # units of their own
        A *= np.ldexp(np.float32(1), r.integers(-30, 30, n)).astype(np.float32)
    elif kind == "rows":
        A *= np.ldexp(np.float32(1), r.integers(-12, 12, m)).astype(np.float32)[:, None]
        W *= np.ldexp(np.float32(1), r.integers(-20, 20, k)).astype(np.float32)
    elif kind == "growing":     # every few rows leave the scale of those before
        A *= np.ldexp(np.float32(1), np.arange(m) * 60 // m - 30).astype(np.float32)[:, None]
    elif kind == "late":        # nothing, and then something
        A[: m // 2] = 0
        A[:, n // 3] = 0
        A[m - 1, n // 3] = 1
    elif kind == "spikes":
        A[r.random((m, n)) < 0.001] *= 1000
    iters = 2 if k <= 64 and n % 4 else 1
    Wr, Hr = iterate(A, W, H, iters)
    Ad, Wd, Hd = (torch.from_numpy(x).cuda() for x in (A, W, H))
    assert k > 64 or plan_of(Ad, m, n, k, Wd, Hd, iters) == 17
    nmf.nmf_mu_dense(Ad, m, n, k, Wd, Hd, iters, EPS)
    Wd, Hd = Wd.cpu().numpy(), Hd.cpu().numpy()
    # sums of up to 1300 positive terms in single precision, a product of three of them and a quotient, each iteration
    live = np.linalg.norm(Hr, axis=0) > 0
    assert columns_off(Hd[:, live], Hr[:, live]) < 4e-6 * iters
    live = np.linalg.norm(Wr, axis=1) > 0
    assert columns_off(Wd.T[:, live], Wr.T[:, live]) < 4e-6 * iters
    assert not Hd[:, np.linalg.norm(Hr, axis=0) == 0].any()


@pytest.mark.gpu
@pytest.mark.parametrize("bad", [np.inf, np.nan])
def test_infinities_and_nan_reach_their_columns_only(bad):
    import torch

    import paper_2202_09518_amd as nmf
    m, n, k = 600, 260, 68
    r = np.random.default_rng(3)
    A = r.random((m, n)).astype(np.float32)
    W, H = r.random((m, k), dtype=np.float32), r.random((k, n), dtype=np.float32)
    A[400, 17] = bad
    P = torch.from_numpy(A).cuda()
    Wd, Hd = torch.from_numpy(W).cuda(), torch.from_numpy(H).cuda()
    nmf.nmf_mu_dense(P, m, n, k, Wd, Hd, 1, EPS)
    Hd = Hd.cpu().numpy()
    assert not np.isfinite(Hd[:, 17]).any()
    assert np.isfinite(np.delete(Hd, 17, axis=1)).all()


def iterate(A, W, H, iters):
    for _ in range(iters):
        W, H = reference(A, W, H)
    return W, H


def off(got, want):
    return np.linalg.norm(got.astype(np.float64) - want) / np.linalg.norm(want)


# Ranks above 64 without room for A' and (A^T)': A is cut as it is loaded.
@pytest.mark.gpu
@pytest.mark.parametrize("m,n,k", [(1300, 516, 68), (517, 1028, 132), (400, 700, 193)])
def test_without_room_for_a_second_layout(m, n, k):
    import torch

    import paper_2202_09518_amd as nmf
    r = np.random.default_rng(11)
    A, W, H = (r.random(s, dtype=np.float32) for s in ((m, n), (m, k), (k, n)))
    size = nmf.nmf_mu_workspace_bytes(5, m, n, 0, k, 0)
    runs = []
    for short in (0, 2 * m * n):        # half a matrix less than the second layout takes
        ws = torch.empty(size - short, dtype=torch.uint8, device="cuda")
        Wd, Hd = torch.from_numpy(W).cuda(), torch.from_numpy(H).cuda()
        nmf.nmf_mu_set_workspace(ws)
        try:
            nmf.nmf_mu_dense(torch.from_numpy(A).cuda(), m, n, k, Wd, Hd, 2, EPS)
            torch.cuda.synchronize()
        finally:
            nmf.nmf_mu_set_workspace(None)
        runs.append((Wd.cpu().numpy(), Hd.cpu().numpy()))
    Wr, Hr = iterate(A, W, H, 2)
    for w, h in runs:
        assert off(w, Wr) < 2e-6 and off(h, Hr) < 2e-6


@pytest.mark.gpu
@pytest.mark.parametrize("m,n,k", [(1500, 700, 40), (4001, 1003, 64), (300, 129, 33), (9000, 260, 50)])
def test_a_run_cut_in_two_has_the_same_bits(m, n, k):
    import torch

    import paper_2202_09518_amd as nmf
    g = torch.Generator(device="cuda")
    g.manual_seed(m + n)
    A, W, H = (torch.rand(s, generator=g, device="cuda") for s in ((m, n), (m, k), (k, n)))
    runs = []
    for parts in ((5,), (2, 3)):
        w, h = W.clone(), H.clone()
        for it in parts:
            nmf.nmf_mu_dense(A, m, n, k, w, h, it, EPS)
        runs.append((w, h))
    assert torch.equal(runs[0][0], runs[1][0]) and torch.equal(runs[0][1], runs[1][1])


# Ensembles: stacks side by side (up to four in a launch, then the rest on the same A), single runs among them, two matrices.
@pytest.mark.gpu
@pytest.mark.parametrize("m,n,ranks", [(700, 515, [[2, 3, 4, 30], [40, 50, 20]]), (1025, 300, [[64, 64, 33, 60, 50, 7], [1, 63, 5]]),
                                       (130, 2049, [[33], [12, 11, 30]])])
def test_stacks_side_by_side(m, n, ranks):
    import torch

    import paper_2202_09518_amd as nmf
    r = np.random.default_rng(5)
    As, ks, Ws, Hs, want = [], [], [], [], []
    for group in ranks:
        A = (r.random((m, 6)) @ r.random((6, n))).astype(np.float32)
        Ad = torch.from_numpy(A).cuda()
        for k in group:
            W, H = r.random((m, k), dtype=np.float32), r.random((k, n), dtype=np.float32)
            As.append(Ad), ks.append(k), Ws.append(torch.from_numpy(W).cuda()), Hs.append(torch.from_numpy(H).cuda())
            want.append(iterate(A, W, H, 2))
    nmf.nmf_mu_dense_batched(len(ks), As, m, n, ks, Ws, Hs, 2, EPS)
    for W, H, (Wr, Hr) in zip(Ws, Hs, want):
        # two updates of each factor, sums of one sign: a few roundings of 2^-24 per sum
        assert off(W.cpu().numpy(), Wr) < 2e-6 and off(H.cpu().numpy(), Hr) < 2e-6


# One stack on a large matrix earns the cut by its iterations, as a single run does: below that the runs go one by one, and a single run is
# that of nmf_mu_dense in either case.  An A that is not aligned, and several stacks, are cut for one iteration.
@pytest.mark.gpu
@pytest.mark.parametrize("m,n,ranks,iters", [(8200, 4100, [40], 3), (8200, 4100, [40], 4), (8200, 8200, [20, 20], 3), (8200, 8200, [20, 20], 4),
                                             (2100, 2001, [33], 1), (700, 516, [50], 1), (8200, 4100, [64, 33], 1)])
def test_ensembles_by_iterations(m, n, ranks, iters):
    import torch

    import paper_2202_09518_amd as nmf
    g = torch.Generator(device="cuda")
    g.manual_seed(m + n)
    A = torch.rand((m, n), generator=g, device="cuda")
    Ws, Hs = [torch.rand((m, k), generator=g, device="cuda") for k in ranks], [torch.rand((k, n), generator=g, device="cuda") for k in ranks]
    W, H = [w.clone() for w in Ws], [h.clone() for h in Hs]
    nmf.nmf_mu_dense_batched(len(ranks), [A] * len(ranks), m, n, ranks, W, H, iters, EPS)
    for k, w0, h0, w, h in zip(ranks, Ws, Hs, W, H):
        nmf.nmf_mu_dense(A, m, n, k, w0, h0, iters, EPS)
        if len(ranks) == 1 and n % 4 == 0:      # the same plan
            assert torch.equal(w0, w) and torch.equal(h0, h)
        else:      # `iters` updates of each factor, a few roundings of 2^-24 per sum
            assert ((w - w0).norm() / w0.norm()).item() < 4e-6 and ((h - h0).norm() / h0.norm()).item() < 4e-6


# The arrival counters at the head of the workspace are other kernels': a run above 64 factors leaves them at zero.
@pytest.mark.gpu
def test_counters_are_left_alone():
    import torch

    import paper_2202_09518_amd as nmf
    A = torch.rand((600, 260), device="cuda")
    W, H = torch.rand((600, 68), device="cuda"), torch.rand((68, 260), device="cuda")
    nmf.nmf_mu_dense(A, 600, 260, 68, W, H, 1, EPS)
    X, G = torch.rand((4099, 40), device="cuda"), torch.empty((40, 40), device="cuda")
    nmf.nmf_gram_w(X, 4099, 40, G)
    want = X.double().t().contiguous() @ X.double()
    assert ((G.double() - want).norm() / want.norm()).item() < 1e-6


# the streaming objective: ragged rows and columns, each number of factor steps, aligned and not, one slab and several
@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["plain", "units", "fit"])
@pytest.mark.parametrize("m,n,k", [(2591, 8201, 3), (2600, 8204, 17), (4133, 4099, 33), (4100, 4100, 64), (66001, 61, 48), (66000, 260, 16),
                                   (66000, 260, 30), (66100, 256, 40)])
def test_objective(m, n, k, kind):
    import torch

    import paper_2202_09518_amd as nmf
    r = np.random.default_rng(11)
    W, H = r.random((m, k), dtype=np.float32), r.random((k, n), dtype=np.float32)
    A = r.random((m, n), dtype=np.float32)
    if kind != "plain":
        A = ((W.astype(np.float64) @ H) * (1 + 1e-3 * (A - 0.5))).astype(np.float32)
    if kind == "units":     # of the factors, up to 2^60 apart, of the rows and of the columns
        u = np.ldexp(np.float32(1), r.integers(-30, 31, k)).astype(np.float32)
        W, H = W * u, H / u[:, None]
        rows, cols = (np.ldexp(np.float32(1), r.integers(-6, 7, x)).astype(np.float32) for x in (m, n))
        A, W, H = A * rows[:, None] * cols, W * rows[:, None], H * cols
    want = np.linalg.norm(A - W.astype(np.float64) @ H)
    got = nmf.nmf_residual_dense(torch.from_numpy(A).cuda(), m, n, k, torch.from_numpy(W).cuda(), torch.from_numpy(H).cuda())
    # an error of 2^-22 per entry of W H adds to the difference in the squares: (2^-22 / 3e-4)^2 / 2 of a fit to 3e-4 of A
    assert abs(got - want) <= 1e-6 * want


# The profile is of the plan that nmf_mu_dense runs for as many iterations: pairs of halves or, for few on a large aligned matrix,
# the plan that needs no second copy.  (The launcher refuses a timed pass of no factors.)
@pytest.mark.gpu
@pytest.mark.parametrize("m,n,k,iters", [(8200, 4100, 40, 1), (8200, 4100, 40, 4), (700, 516, 64, 1), (2100, 2001, 33, 1), (2100, 2001, 33, 2)])
def test_profile_is_of_the_plan_that_runs(m, n, k, iters):
    import torch

    import paper_2202_09518_amd as nmf
    g = torch.Generator(device="cuda")
    g.manual_seed(m + n)
    A, W, H = (torch.rand(s, generator=g, device="cuda") for s in ((m, n), (m, k), (k, n)))
    w, h = W.clone(), H.clone()
    nmf.nmf_mu_dense(A, m, n, k, w, h, iters, EPS)
    ms = nmf.nmf_mu_dense_profile(A, m, n, k, W, H, iters, EPS)
    assert ms[7] > 0 and ms[8] > 0
    if n % 4 == 0 or iters > 1:     # the profile makes no aligned copy of A
        assert torch.equal(W, w) and torch.equal(H, h)


# An infinite entry of a factor makes the objective infinite, as in single precision; NaN where the floats give NaN.
@pytest.mark.gpu
@pytest.mark.parametrize("m,n,k", [(2591, 8201, 10), (4100, 4100, 64), (66001, 61, 48)])
def test_objective_of_infinite_factors(m, n, k):
    import torch

    import paper_2202_09518_amd as nmf
    g = torch.Generator(device="cuda")
    g.manual_seed(m + n)
    A, W, H = (torch.rand(s, generator=g, device="cuda") + 0.1 for s in ((m, n), (m, k), (k, n)))

    def objective():
        return nmf.nmf_residual_dense(A, m, n, k, W, H)
    assert np.isfinite(objective())
    for x, at in ((W, (m - 1, k // 2)), (H, (k - 1, n - 1)), (A, (m // 2, 0))):
        old = x[at].clone()
        x[at] = np.inf
        assert objective() == np.inf
        x[at] = np.nan
        assert np.isnan(objective())
        x[at] = old
    W[5, 0], H[0, 7] = np.inf, 0
    assert np.isnan(objective())
