"""Both products in one reading of A (up to 32 factors, up to 512 columns): edges of the row tiles,
the column groups, the factor count and the rows an accumulator may take in, against the oracle;
a run cut in two; the objective from its by-products.  Up to 16 factors the smaller ones run in one launch
(test_resident.py) unless the workspace is short (test_short_workspaces.py)."""
import numpy as np
import pytest

from oracle import nmf_oracle as orc

EPS = 1e-16


def data(m, n, k):
    r = np.random.default_rng(m + 3 * n + 7 * k)
    return r.random((m, n), dtype=np.float32), r.random((m, k), dtype=np.float32), r.random((k, n), dtype=np.float32)


# 140001 x 260: more than 16 blocks of 32 rows per workgroup; 280100 x 68: the same with 64 rows;
# 259, 511: taken after a copy with padded columns
@pytest.mark.gpu
@pytest.mark.parametrize("m,n", [(1, 64), (31, 4), (32, 60), (33, 256), (64, 252), (65, 260), (1000, 68), (999, 508),
                                 (8193, 512), (16500, 192), (700, 259), (700, 511), (140001, 260), (280100, 68)])
@pytest.mark.parametrize("k", [1, 8, 17, 32])
def test_iterations_of_narrow_matrices(m, n, k):
    import torch

    import paper_2202_09518_amd as nmf
    A, W, H = data(m, n, k)
    Ad, eps = torch.from_numpy(A).cuda(), float(np.float32(EPS))
    Wd, Hd = torch.from_numpy(W).cuda(), torch.from_numpy(H).cuda()
    nmf.nmf_mu_dense(Ad, m, n, k, Wd, Hd, 3, EPS)
    W2, H2 = torch.from_numpy(W).cuda(), torch.from_numpy(H).cuda()
    nmf.nmf_mu_dense(Ad, m, n, k, W2, H2, 2, EPS)
    nmf.nmf_mu_dense(Ad, m, n, k, W2, H2, 1, EPS)
    torch.cuda.synchronize()
    assert torch.equal(Wd, W2) and torch.equal(Hd, H2)
    Wr, Hr = orc.mu_dense(A, W, H, 3, eps)
    # three updates of each factor, sums of one sign: a few roundings of 2^-24 per sum
    assert orc.rel_fro(Wd.cpu().numpy(), Wr) < 3e-6
    assert orc.rel_fro(Hd.cpu().numpy(), Hr) < 3e-6


@pytest.mark.gpu
@pytest.mark.parametrize("m,n,k", [(700, 192, 5), (20000, 500, 32)])
def test_objective_of_every_iteration(m, n, k):
    import torch

    import paper_2202_09518_amd as nmf
    A, W, H = data(m, n, k)
    Wd, Hd = torch.from_numpy(W).cuda(), torch.from_numpy(H).cuda()
    got = nmf.nmf_mu_dense_monitor(torch.from_numpy(A).cuda(), m, n, k, Wd, Hd, 4, EPS)
    for it in range(4):
        W, H = orc.mu_dense(A, W, H, 1, float(np.float32(EPS)))
        want = orc.residual_dense(A, W, H)
        # ||A||^2 - 2 <A H^T, W> + <H H^T, W^T W>: three sums of relative error 2^-22 or less, cancelling to
        # about a tenth of ||A||^2 for uniform data
        assert abs(got[it] - want) <= 1e-5 * want


@pytest.mark.gpu
def test_workspace_of_the_small_plan_still_serves():
    """A workspace sized for the plan without the extra partials runs that plan."""
    import torch

    import paper_2202_09518_amd as nmf
    m, n, k = 9000, 300, 12
    A, W, H = data(m, n, k)
    size = nmf.nmf_mu_workspace_bytes(4, m, n, 0, k, 0)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    Wd, Hd = torch.from_numpy(W).cuda(), torch.from_numpy(H).cuda()
    nmf.nmf_mu_set_workspace(ws)
    try:
        nmf.nmf_mu_dense(torch.from_numpy(A).cuda(), m, n, k, Wd, Hd, 2, EPS)
        torch.cuda.synchronize()
    finally:
        nmf.nmf_mu_set_workspace(None)
    Wr, Hr = orc.mu_dense(A, W, H, 2, float(np.float32(EPS)))
    assert orc.rel_fro(Wd.cpu().numpy(), Wr) < 2e-6 and orc.rel_fro(Hd.cpu().numpy(), Hr) < 2e-6
