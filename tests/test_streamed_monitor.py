"""The monitored streamed run where the last batch is shorter than the others: the workgroups of its W update may not
outnumber those of a full batch, whose number the list of shares is laid out for."""
import ctypes

import numpy as np
import pytest

from oracle import nmf_oracle as orc

EPS = 1e-16


def blocks(rows, k, batch):
    """Workgroups of the W update on `rows` rows of a run in batches of `batch` (host functions of the library; a run
    takes two 32-row tiles per workgroup at least)."""
    import paper_2202_09518_amd as nmf
    tiles = getattr(nmf.lib(), "_ZN5nmfmu14aht_rows_tilesEli")
    count = getattr(nmf.lib(), "_ZN5nmfmu15aht_rows_blocksElii")
    i64, i32 = ctypes.c_int64, ctypes.c_int
    return count(i64(rows), i32(k), i32(max(2, tiles(i64(batch), i32(k)))))


@pytest.mark.parametrize("batch", [1, 64, 8128, 8129, 8192, 16200, 24448, 24449, 24576, 32768, 200000])
@pytest.mark.parametrize("k", [1, 32, 33, 64])
def test_a_shorter_batch_has_no_more_workgroups(batch, k):
    full = blocks(batch, k, batch)
    assert 1 <= full <= 256
    for rows in {1, 32, 4097, 7808, 8000, 8128, 24000, 24448, batch // 2, batch - 1}:
        if 1 <= rows <= batch:
            assert blocks(rows, k, batch) <= full, rows


# a last batch that would take 32-row blocks by itself, one that would take 64-row blocks where a full one takes 128
@pytest.mark.gpu
@pytest.mark.parametrize("batch,last", [(8192, 4100), (8192, 8000), (24576, 24000)])
def test_objective_with_a_short_last_batch(batch, last):
    import torch

    import paper_2202_09518_amd as nmf
    m, n, k, iters = 2 * batch + last, 36, 5, 2
    r = np.random.default_rng(batch + last)
    A, W, H = r.random((m, n), dtype=np.float32), r.random((m, k), dtype=np.float32), r.random((k, n), dtype=np.float32)
    Wd, Hd = torch.from_numpy(W).cuda(), torch.from_numpy(H).cuda()
    got = nmf.nmf_mu_ooc_monitor(torch.from_numpy(A).pin_memory(), m, n, k, Wd, Hd, iters, EPS, batch, 3 * batch * n * 4 + 1024)
    normA2 = float((A.astype(np.float64) ** 2).sum())
    for it in range(iters):
        W, H = orc.mu_dense(A, W, H, 1, float(np.float32(EPS)))
        want = orc.residual_dense(A, W, H)
        # ||A||^2 - 2 <A H^T, W> + <H H^T, W^T W>: absolute error about 2^-22 of ||A||^2 in the square
        assert abs(got[it] - want) <= 3e-7 * normA2 / want
    # two updates of each factor, sums of one sign: a few roundings of 2^-24 per sum
    assert orc.rel_fro(Wd.cpu().numpy(), W) < 2e-6 and orc.rel_fro(Hd.cpu().numpy(), H) < 2e-6


@pytest.mark.gpu
@pytest.mark.parametrize("m,batch", [(700, 256), (9000, 4000), (9000, 8192)])
def test_a_workspace_of_the_documented_size_is_enough(m, batch):
    import torch

    import paper_2202_09518_amd as nmf
    n, k, iters = 40, 6, 2
    r = np.random.default_rng(m + batch)
    A, W, H = r.random((m, n), dtype=np.float32), r.random((m, k), dtype=np.float32), r.random((k, n), dtype=np.float32)
    batches = -(-m // batch)
    size = nmf.nmf_mu_workspace_bytes(2, m, n, 0, k, batch)
    for doubles in (batches * -(-batch // 64), batches, 4097, iters):
        size += -(-8 * doubles // 256) * 256
    Wd, Hd = torch.from_numpy(W).cuda(), torch.from_numpy(H).cuda()
    buf = torch.empty(size, dtype=torch.uint8, device="cuda")
    nmf.nmf_mu_set_workspace(buf)
    try:
        got = nmf.nmf_mu_ooc_monitor(torch.from_numpy(A).pin_memory(), m, n, k, Wd, Hd, iters, EPS, batch, 3 * batch * n * 4 + 1024)
    finally:
        nmf.nmf_mu_set_workspace(None)
    W, H = orc.mu_dense(A, W, H, iters, float(np.float32(EPS)))
    want = orc.residual_dense(A, W, H)
    assert abs(got[-1] - want) <= 3e-7 * float((A.astype(np.float64) ** 2).sum()) / want
