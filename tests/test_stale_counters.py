"""A sparse run finds its arrival counters as a run that was cut short left them: the results are those of a clean workspace."""
import numpy as np
import pytest

EPS = 1e-16


@pytest.mark.gpu
@pytest.mark.parametrize("streamed", [False, True])
def test_sparse_runs(streamed):
    import torch

    import paper_2202_09518_amd as nmf
    r = np.random.default_rng(5)
    m, n, k, per = 3000, 1700, 12, 4
    rowptr = torch.arange(0, m * per + 1, per, dtype=torch.int64)
    col = torch.from_numpy(r.integers(0, n, m * per).astype(np.int32))
    vals, W, H = (torch.from_numpy(r.random(s, dtype=np.float32)) for s in (m * per, (m, k), (k, n)))
    ws = torch.zeros(64 << 20, dtype=torch.uint8, device="cuda")

    def run():
        Wd, Hd = W.cuda(), H.cuda()
        if streamed:
            nmf.nmf_mu_csr_ooc(rowptr.pin_memory(), col.pin_memory(), vals.pin_memory(), m, n, m * per, k, Wd, Hd, 3, EPS,
                               m * per // 3, 32 << 20)
        else:
            nmf.nmf_mu_csr(rowptr.cuda(), col.cuda(), vals.cuda(), m, n, m * per, k, Wd, Hd, 3, EPS)
        torch.cuda.synchronize()
        return Wd, Hd

    nmf.nmf_mu_set_workspace(ws)
    try:
        clean = run()
        ws[:256] = 7            # the counters are the head of the workspace
        stale = run()
    finally:
        nmf.nmf_mu_set_workspace(None)
    assert torch.equal(clean[0], stale[0]) and torch.equal(clean[1], stale[1])
