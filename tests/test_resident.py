"""A whole run in one launch (up to 16 factors, A on the compute units): edges of the row and column tiles, of the groups
that exchange and of the factor count, against the oracle; the same bits from a run cut in two, from the allocation-free
call, from a monitored and a stopped run, and from one workgroup that does the run of all."""
import ctypes

import numpy as np
import pytest

from oracle import nmf_oracle as orc

EPS = 1e-16
# one group of columns and 1, 2, 4 row tiles per workgroup (1, 32, 33, 63, 65 row groups, an odd rest); two to 16 groups
# of columns; more groups of rows than 16 (owners of no column tile), more groups of columns than row tiles; 4 row tiles
# on two or three groups of columns (an owner's second tile in the W update)
SHAPES = [(1, 1), (16, 16), (17, 15), (256, 192), (513, 255), (1000, 256), (1025, 31), (4161, 97), (16380, 256), (40, 257),
          (100, 513), (600, 1003), (2000, 1201), (1030, 2047), (63, 4096), (4096, 1024),
          (1100, 300), (8192, 512), (2001, 700)]


def data(m, n, k):
    r = np.random.default_rng(m + 3 * n + 7 * k)
    return r.random((m, n), dtype=np.float32), r.random((m, k), dtype=np.float32), r.random((k, n), dtype=np.float32)


def by_one(nmf, A, m, n, k, W, H, iters):
    import torch

    fn = nmf.lib().nmfmu_resident_by_one
    fn.argtypes = [ctypes.c_void_p, ctypes.c_int64, ctypes.c_int64, ctypes.c_int32, ctypes.c_void_p, ctypes.c_void_p,
                   ctypes.c_int32, ctypes.c_float, ctypes.c_void_p]
    assert fn(A.data_ptr(), m, n, k, W.data_ptr(), H.data_ptr(), iters, EPS, torch.cuda.current_stream().cuda_stream) == 0


@pytest.mark.gpu
@pytest.mark.parametrize("m,n", SHAPES)
@pytest.mark.parametrize("k", [1, 5, 16])
def test_runs_of_the_resident_plan(m, n, k):
    import torch

    import paper_2202_09518_amd as nmf
    A, W, H = data(m, n, k)
    Ad = torch.empty(m * n + 1, device="cuda")[1:]        # not 16-byte aligned: the plan takes any A
    Ad.copy_(torch.from_numpy(A).reshape(-1))
    eps = float(np.float32(EPS))

    def run(fn, *iters):
        Wd, Hd = torch.from_numpy(W).cuda(), torch.from_numpy(H).cuda()
        for it in iters:
            fn(Wd, Hd, it)
        torch.cuda.synchronize()
        return Wd, Hd

    ref = run(lambda w, h, it: nmf.nmf_mu_dense(Ad, m, n, k, w, h, it, EPS), 3)
    Wr, Hr = orc.mu_dense(A, W, H, 3, eps)
    # three updates of each factor, sums of one sign: a few roundings of 2^-24 per sum
    assert orc.rel_fro(ref[0].cpu().numpy(), Wr) < 3e-6 and orc.rel_fro(ref[1].cpu().numpy(), Hr) < 3e-6
    res = {}
    others = [run(lambda w, h, it: nmf.nmf_mu_dense(Ad, m, n, k, w, h, it, EPS), 2, 1),
              run(lambda w, h, it: nmf.nmf_mu_dense_noalloc(Ad, m, n, k, w, h, it, EPS), 3),
              run(lambda w, h, it: by_one(nmf, Ad, m, n, k, w, h, it), 3),
              run(lambda w, h, it: res.update(mon=nmf.nmf_mu_dense_monitor(Ad, m, n, k, w, h, it, EPS)), 3)]
    for Wd, Hd in others:
        assert torch.equal(Wd, ref[0]) and torch.equal(Hd, ref[1])
    Wd, Hd = run(lambda w, h, it: res.update(tol=nmf.nmf_mu_dense_tol(Ad, m, n, k, w, h, it, EPS, 0.0, 2)), 3)
    if res["tol"][0] == 3 or (m, n) != (1, 1):            # one entry may be met exactly
        assert res["tol"][0] == 3 and torch.equal(Wd, ref[0]) and torch.equal(Hd, ref[1])
    normA2 = float((A.astype(np.float64) ** 2).sum())
    for it in range(3):
        W, H = orc.mu_dense(A, W, H, 1, eps)
        want = orc.residual_dense(A, W, H)
        # ||A||^2 - 2 <A H^T, W> + <H H^T, W^T W>: three sums of relative error 2^-21 or less that cancel
        assert abs(res["mon"][it] ** 2 - want ** 2) <= 1e-6 * normA2 + 1e-5 * want ** 2


@pytest.mark.gpu
@pytest.mark.parametrize("eps", [0.0, EPS])
def test_zeros_of_the_resident_plan(eps):
    """A zero row and a zero column of A empty their row of W and column of H; with eps = 0 padded factors and columns
    (0 / 0) stay out of the result."""
    import torch

    import paper_2202_09518_amd as nmf
    m, n, k = 70, 300, 3
    A, W, H = data(m, n, k)
    if eps:
        A[5] = 0
        A[:, 270] = 0
    Wd, Hd = torch.from_numpy(W).cuda(), torch.from_numpy(H).cuda()
    nmf.nmf_mu_dense(torch.from_numpy(A).cuda(), m, n, k, Wd, Hd, 3, eps)
    Wr, Hr = orc.mu_dense(A, W, H, 3, float(np.float32(eps)))
    assert orc.rel_fro(Wd.cpu().numpy(), Wr) < 3e-6 and orc.rel_fro(Hd.cpu().numpy(), Hr) < 3e-6
    if eps:
        assert not Wd[5].any() and not Hd[:, 270].any()


@pytest.mark.gpu
def test_replays_of_a_captured_resident_run():
    import torch

    import paper_2202_09518_amd as nmf
    m, n, k = 600, 1003, 7
    A, W, H = (torch.from_numpy(x).cuda() for x in data(m, n, k))
    We, He = W.clone(), H.clone()
    nmf.nmf_mu_dense(A, m, n, k, We, He, 5, EPS)
    torch.cuda.synchronize()
    Wd, Hd = W.clone(), H.clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        Wd.copy_(W)
        Hd.copy_(H)
        nmf.nmf_mu_dense(A, m, n, k, Wd, Hd, 5, EPS)
    for _ in range(4):
        Wd.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(Wd, We) and torch.equal(Hd, He)
        W2, H2 = W.clone(), H.clone()
        nmf.nmf_mu_dense(A, m, n, k, W2, H2, 5, EPS)      # the same workspace between the replays
        torch.cuda.synchronize()
        assert torch.equal(W2, We) and torch.equal(H2, He)


def polled(nmf, A, m, n, k, W, H, iters, polls):
    import torch

    fn = nmf.lib().nmfmu_resident_polls
    fn.argtypes = [ctypes.c_void_p, ctypes.c_int64, ctypes.c_int64, ctypes.c_int32, ctypes.c_void_p, ctypes.c_void_p,
                   ctypes.c_int32, ctypes.c_float, ctypes.c_uint32, ctypes.c_void_p]
    assert fn(A.data_ptr(), m, n, k, W.data_ptr(), H.data_ptr(), iters, EPS, polls, torch.cuda.current_stream().cuda_stream) == 0


@pytest.mark.gpu
@pytest.mark.parametrize("m,n,k,iters", [(16, 16, 2, 9000), (256, 192, 4, 9000), (100, 513, 5, 9000), (4096, 1024, 16, 1500)])
def test_long_runs(m, n, k, iters):
    """More iterations than a launch does: the bits of short calls.  The looks of all waits together are many times the
    looks that a wait has, which belong to each wait (2^13: milliseconds, where a wait takes one or two microseconds)."""
    import torch

    import paper_2202_09518_amd as nmf
    A, W, H = (torch.from_numpy(x).cuda() for x in data(m, n, k))
    runs = []
    for calls, fn in ((1, lambda *a: polled(nmf, *a, 1 << 13)), (1, lambda *a: nmf.nmf_mu_dense(*a, EPS)),
                      (30, lambda *a: nmf.nmf_mu_dense(*a, EPS))):
        Wd, Hd = W.clone(), H.clone()
        for _ in range(calls):
            fn(A, m, n, k, Wd, Hd, iters // calls)
        torch.cuda.synchronize()
        assert bool(torch.isfinite(Wd).all()) and bool(torch.isfinite(Hd).all())
        runs.append((Wd, Hd))
    for Wd, Hd in runs[1:]:
        assert torch.equal(Wd, runs[0][0]) and torch.equal(Hd, runs[0][1])


@pytest.mark.gpu
def test_a_lost_run_is_marked():
    """One look a wait: a run of many workgroups does not get by with that, ends all the same and says so."""
    import torch

    import paper_2202_09518_amd as nmf
    m, n, k = 4096, 1024, 16
    A, W, H = (torch.from_numpy(x).cuda() for x in data(m, n, k))
    Wd, Hd = W.clone(), H.clone()
    polled(nmf, A, m, n, k, Wd, Hd, 300, 1)
    torch.cuda.synchronize()
    assert bool(torch.isnan(Wd[0, 0])) and bool(torch.isnan(Hd[0, 0]))
    runs = [(W.clone(), H.clone()) for _ in range(2)]
    polled(nmf, A, m, n, k, *runs[0], 3, 0)         # the next run on the same workspace is none the worse for it
    by_one(nmf, A, m, n, k, *runs[1], 3)
    torch.cuda.synchronize()
    assert torch.equal(runs[0][0], runs[1][0]) and torch.equal(runs[0][1], runs[1][1])
    assert bool(torch.isfinite(runs[0][0]).all())


@pytest.mark.gpu
@pytest.mark.parametrize("m,n", [(300, 200), (600, 1003)])
@pytest.mark.parametrize("k", [3, 8, 9])
def test_gram_matrices_beyond_the_largest_float(m, n, k):
    """W^T W overflows: the denominators are infinite and H becomes zero, and W with it, as on the plan of a workspace without
    room for this one."""
    import torch

    import paper_2202_09518_amd as nmf
    A, W, H = (torch.from_numpy(x + np.float32(0.1)).cuda() for x in data(m, n, k))
    A *= 1e-3
    W *= 1e20
    small = torch.empty(nmf.nmf_mu_workspace_bytes(4, m, n, 0, k, 0), dtype=torch.uint8, device="cuda")
    for ws in (None, small):
        Wd, Hd = W.clone(), H.clone()
        nmf.nmf_mu_set_workspace(ws)
        try:
            nmf.nmf_mu_dense(A, m, n, k, Wd, Hd, 2, EPS)
            torch.cuda.synchronize()
        finally:
            nmf.nmf_mu_set_workspace(None)
        assert torch.equal(Wd, torch.zeros_like(W)) and torch.equal(Hd, torch.zeros_like(H))


def shared(nmf, A, m, n, k, W, H, iters, workgroups, patience):
    import torch

    fn = nmf.lib().nmfmu_resident_shared
    fn.argtypes = [ctypes.c_void_p, ctypes.c_int64, ctypes.c_int64, ctypes.c_int32, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int32,
                   ctypes.c_float, ctypes.c_int32, ctypes.c_int64, ctypes.c_void_p]
    assert fn(A.data_ptr(), m, n, k, W.data_ptr(), H.data_ptr(), iters, EPS, workgroups, patience,
              torch.cuda.current_stream().cuda_stream) == 0


# 1, 2 and 4 row tiles per workgroup with one and with several groups of columns; (1100, 300) and (2001, 700): second row
# tiles of one owner; launched: a few workgroups, half, all but one, and all, who start at once with those that are there
@pytest.mark.gpu
@pytest.mark.parametrize("m,n,k", [(256, 192, 4), (513, 255, 9), (4161, 97, 16), (40, 257, 5), (600, 1003, 8), (1100, 300, 12),
                                   (2001, 700, 3), (4096, 1024, 16), (16380, 256, 10)])
def test_runs_shared_by_those_that_are_there(m, n, k):
    import torch

    import paper_2202_09518_amd as nmf
    A, W, H = (torch.from_numpy(x).cuda() for x in data(m, n, k))
    iters = 12
    We, He = W.clone(), H.clone()
    nmf.nmf_mu_dense(A, m, n, k, We, He, iters, EPS)
    torch.cuda.synchronize()
    Wr, Hr = orc.mu_dense(A.cpu().numpy(), W.cpu().numpy(), H.cpu().numpy(), iters, float(np.float32(EPS)))
    # twelve updates of each factor: as for three, times their number
    assert orc.rel_fro(We.cpu().numpy(), Wr) < 1.2e-5 and orc.rel_fro(He.cpu().numpy(), Hr) < 1.2e-5
    rows = 16
    while -(-m // rows) > 32 and rows < 64:
        rows *= 2
    groups = -(-m // rows) * -(-n // 256)
    for workgroups, patience in ((2, 0), (3, -1), (max(1, groups // 2), 0), (max(1, groups - 1), 0), (0, -1), (0, 1), (0, 100)):
        Wd, Hd = W.clone(), H.clone()
        shared(nmf, A, m, n, k, Wd, Hd, iters, workgroups, patience)
        torch.cuda.synchronize()
        assert torch.equal(Wd, We) and torch.equal(Hd, He), (workgroups, patience)


@pytest.mark.gpu
@pytest.mark.parametrize("first,second", [((16380, 256, 16), (16380, 256, 16)), ((6400, 256, 8), (16380, 256, 16)),
                                          ((2000, 1201, 12), (4096, 1024, 5))])
def test_two_runs_at_once(first, second):
    """A run on the library's workspace and one on the fixed scratch array, on two streams: together they want more
    compute units than there are."""
    import torch

    import paper_2202_09518_amd as nmf
    problems, results = [], []
    for m, n, k in (first, second):
        A, W, H = (torch.from_numpy(x).cuda() for x in data(m, n, k))
        problems.append((A, m, n, k, W, H))
    calls = (nmf.nmf_mu_dense, nmf.nmf_mu_dense_noalloc)
    streams = [torch.cuda.Stream() for _ in calls]
    for together in (False, True):
        factors = [(p[4].clone(), p[5].clone()) for p in problems]
        torch.cuda.synchronize()
        for _ in range(3):
            for call, st, (A, m, n, k, _, _), (Wd, Hd) in zip(calls, streams, problems, factors):
                with torch.cuda.stream(st):
                    call(A, m, n, k, Wd, Hd, 400, EPS)
                if not together:
                    torch.cuda.synchronize()
        torch.cuda.synchronize()
        results.append(factors)
    for (Wa, Ha), (Wb, Hb) in zip(*results):
        assert torch.equal(Wa, Wb) and torch.equal(Ha, Hb)


@pytest.mark.gpu
@pytest.mark.parametrize("m,n,k", [(256, 192, 4), (40, 257, 5), (16380, 256, 16), (2000, 1201, 12)])
def test_objectives_of_several_launches(m, n, k):
    """More iterations than a launch reports: the factors of a plain run and its objectives, also from a workspace that has no
    room to report several iterations at once."""
    import torch

    import paper_2202_09518_amd as nmf
    A, W, H = (torch.from_numpy(x).cuda() for x in data(m, n, k))
    iters, want = 70, {}
    We, He = W.clone(), H.clone()
    for it in range(iters):
        nmf.nmf_mu_dense(A, m, n, k, We, He, 1, EPS)
        if it in (0, 30, 31, 32, 63, 64, 69):
            want[it] = nmf.nmf_residual_dense(A, m, n, k, We, He)
    normA2 = float(A.double().square().sum())
    short = nmf.nmf_mu_workspace_bytes(4, m, n, 0, k, 0) + (48 << 10) * (-(-m // 16) * -(-n // 256))
    for size in (None, short):
        Wd, Hd = W.clone(), H.clone()
        nmf.nmf_mu_set_workspace(None if size is None else torch.empty(size, dtype=torch.uint8, device="cuda"))
        try:
            got = nmf.nmf_mu_dense_monitor(A, m, n, k, Wd, Hd, iters, EPS)
        finally:
            nmf.nmf_mu_set_workspace(None)
        assert torch.equal(Wd, We) and torch.equal(Hd, He)
        for it, f in want.items():
            # ||A||^2 - 2 <A H^T, W> + <H H^T, W^T W>: three sums of relative error 2^-21 or less that cancel
            assert abs(got[it] ** 2 - f ** 2) <= 1e-6 * normA2 + 1e-5 * f ** 2, (size, it)


@pytest.mark.gpu
def test_monitored_run_beside_another():
    """Its launches find part of the compute units taken: the factors and objectives of an undisturbed run."""
    import torch

    import paper_2202_09518_amd as nmf
    m, n, k = 4096, 1024, 7
    A, W, H = (torch.from_numpy(x).cuda() for x in data(m, n, k))
    A2, W2, H2 = (torch.from_numpy(x).cuda() for x in data(6400, 256, 16))
    side, runs = torch.cuda.Stream(), []
    for disturbed in (False, True, True):
        Wd, Hd = W.clone(), H.clone()
        torch.cuda.synchronize()
        if disturbed:
            with torch.cuda.stream(side):
                for _ in range(20):
                    nmf.nmf_mu_dense_noalloc(A2, 6400, 256, 16, W2, H2, 100, EPS)
        got = nmf.nmf_mu_dense_monitor(A, m, n, k, Wd, Hd, 70, EPS)
        runs.append((Wd, Hd, list(got)))
    torch.cuda.synchronize()
    for Wd, Hd, got in runs[1:]:
        assert torch.equal(Wd, runs[0][0]) and torch.equal(Hd, runs[0][1]) and got == runs[0][2]
