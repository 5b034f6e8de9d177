"""The streamed run walks its batches forwards and backwards in turn and keeps what the slots hold: any number of
batches, slots and iterations, a short last batch, the kernels for each kind of n and k, against the oracle; the slots
change nothing, and the monitored run reports the objective of the same factors."""
import numpy as np
import pytest

from oracle import nmf_oracle as orc

EPS = 1e-16


@pytest.mark.gpu
@pytest.mark.parametrize("rows,batch", [(64, 64), (100, 64), (192, 64), (200, 50), (201, 50), (333, 48)])
@pytest.mark.parametrize("iters", [1, 2, 3, 4])
# W update fused into the pass over A; the direct kernel (n % 4 != 0); the passes for 33 factors and more
@pytest.mark.parametrize("n,k", [(132, 7), (131, 7), (132, 40)])
def test_batches_slots_and_iterations(rows, batch, iters, n, k):
    import torch

    import paper_2202_09518_amd as nmf
    r = np.random.default_rng(rows + iters)
    A, W, H = r.random((rows, n), dtype=np.float32), r.random((rows, k), dtype=np.float32), r.random((k, n), dtype=np.float32)
    Ah = torch.from_numpy(A).pin_memory()
    runs = []
    for slots in (1, 2, 3):
        Wd, Hd = torch.from_numpy(W).cuda(), torch.from_numpy(H).cuda()
        nmf.nmf_mu_ooc(Ah, rows, n, k, Wd, Hd, iters, EPS, batch, slots * ((batch * n * 4 + 255) // 256 * 256))
        torch.cuda.synchronize()
        runs.append((Wd, Hd))
    for Wd, Hd in runs[1:]:
        assert torch.equal(Wd, runs[0][0]) and torch.equal(Hd, runs[0][1])
    Wr, Hr = orc.mu_dense(A, W, H, iters, float(np.float32(EPS)))
    # up to four updates of each factor, sums of one sign: a few roundings of 2^-24 per sum
    assert orc.rel_fro(runs[0][0].cpu().numpy(), Wr) < 4e-6
    assert orc.rel_fro(runs[0][1].cpu().numpy(), Hr) < 4e-6
    Wd, Hd = torch.from_numpy(W).cuda(), torch.from_numpy(H).cuda()
    got = nmf.nmf_mu_ooc_monitor(Ah, rows, n, k, Wd, Hd, iters, EPS, batch, 2 * ((batch * n * 4 + 255) // 256 * 256))
    assert torch.equal(Wd, runs[0][0]) and torch.equal(Hd, runs[0][1])
    normA2 = float((A.astype(np.float64) ** 2).sum())
    for it in range(iters):
        W, H = orc.mu_dense(A, W, H, 1, float(np.float32(EPS)))
        # ||A||^2 - 2 <A H^T, W> + <H H^T, W^T W>: errors of 2^-22 of ||A||^2
        assert abs(got[it] ** 2 - orc.residual_dense(A, W, H) ** 2) <= 6e-7 * normA2
