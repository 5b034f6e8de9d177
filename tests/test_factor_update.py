"""The factor update at the edges of its chunk widths (16, 32 and 64 columns), factor counts and split
batches, and on a factor of more than 2^31 bytes.  Up to 16 factors the smaller ones run in one launch
(test_resident.py) unless the workspace is short (test_short_workspaces.py)."""
import numpy as np
import pytest

from oracle import nmf_oracle as orc

EPS = 1e-16


@pytest.mark.gpu
@pytest.mark.parametrize("m,n", [(300, 15), (9000, 17), (700, 2048), (700, 2049), (333, 8192), (333, 8193), (40000, 130),
                                 (333, 16500)])
@pytest.mark.parametrize("k", [1, 8, 9, 16, 17, 32, 33, 64])
def test_two_iterations_across_the_chunk_widths(m, n, k):
    import torch

    import paper_2202_09518_amd as nmf
    r = np.random.default_rng(m + n + k)
    A, W, H = r.random((m, n), dtype=np.float32), r.random((m, k), dtype=np.float32), r.random((k, n), dtype=np.float32)
    Wd, Hd = torch.from_numpy(W).cuda(), torch.from_numpy(H).cuda()
    nmf.nmf_mu_dense(torch.from_numpy(A).cuda(), m, n, k, Wd, Hd, 2, EPS)
    torch.cuda.synchronize()
    Wr, Hr = orc.mu_dense(A, W, H, 2, float(np.float32(EPS)))
    # two updates of each factor, sums of one sign: a few roundings of 2^-24 per sum
    assert orc.rel_fro(Wd.cpu().numpy(), Wr) < 2e-6
    assert orc.rel_fro(Hd.cpu().numpy(), Hr) < 2e-6


@pytest.mark.gpu
@pytest.mark.parametrize("k,n", [(64, (1 << 23) + 5), (33, (1 << 24) - 3)])
def test_update_of_a_factor_beyond_two_gigabytes(k, n):
    import torch

    import paper_2202_09518_amd as nmf
    g = torch.Generator(device="cuda").manual_seed(k)
    H = torch.rand((k, n), generator=g, device="cuda")
    P = torch.rand((k, n), generator=g, device="cuda")
    G = torch.rand((k, k), generator=g, device="cuda")
    G = G + G.t()
    new = H.clone()
    nmf.nmf_h_update(new, P, G, k, n, EPS)
    torch.cuda.synchronize()
    worst = 0.0
    for j in [0, n // 2 // 64 * 64, n - 70000]:      # the first columns, some in the middle, the ragged end
        s = slice(j, j + 70000)
        h = H[:, s].double()
        want = h * P[:, s].double() / (G.double() @ h + EPS)
        worst = max(worst, float(((new[:, s].double() - want).abs() / want).max()))
    assert worst < 64 * 2.0 ** -24       # 64 terms of one sign
