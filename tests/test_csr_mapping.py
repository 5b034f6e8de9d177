"""The two mappings of the sparse update (a row per lane group, a row per wave) at the edges of a step,
with empty, full-step and long rows, against the oracle."""
import numpy as np
import pytest

from oracle import nmf_oracle as orc

EPS = 1e-16


def matrix(m, n, lengths, seed):
    r = np.random.default_rng(seed)
    counts = np.resize(np.asarray(lengths, dtype=np.int64), m)
    rowptr = np.zeros(m + 1, dtype=np.int64)
    np.cumsum(counts, out=rowptr[1:])
    colidx = np.concatenate([np.sort(r.choice(n, int(c), replace=False)) for c in counts] or [np.zeros(0)]).astype(np.int32)
    return rowptr, colidx, r.random(colidx.size, dtype=np.float32)


@pytest.mark.gpu
@pytest.mark.parametrize("lengths", [[0, 1, 3, 4, 5, 15, 16, 17], [63, 64, 65, 127, 128, 129, 300], [0, 64, 0, 700], [70],
                                     [20000, 5, 0, 64], [1]])
@pytest.mark.parametrize("k", [1, 4, 7, 12, 16, 24, 32, 50, 64])
def test_rows_at_the_edges_of_a_step(lengths, k):
    import torch

    import paper_2202_09518_amd as nmf
    m, n = 333, max(max(lengths), 40) + 11
    rowptr, colidx, vals = matrix(m, n, lengths, 7 * k + len(lengths))
    r = np.random.default_rng(k)
    W, H = r.random((m, k), dtype=np.float32), r.random((k, n), dtype=np.float32)
    Wd, Hd = torch.from_numpy(W).cuda(), torch.from_numpy(H).cuda()
    nmf.nmf_mu_csr(torch.from_numpy(rowptr).cuda(), torch.from_numpy(colidx).cuda(), torch.from_numpy(vals).cuda(),
                   m, n, int(vals.size), k, Wd, Hd, 2, EPS)
    torch.cuda.synchronize()
    Wr, Hr = orc.mu_csr(rowptr, colidx, vals, m, n, W, H, 2, float(np.float32(EPS)))
    # two updates of each factor, sums of at most 20000 terms of one sign: a few roundings of 2^-24 per sum
    assert orc.rel_fro(Wd.cpu().numpy(), Wr) < 3e-6
    assert orc.rel_fro(Hd.cpu().numpy(), Hr) < 3e-6


@pytest.mark.gpu
@pytest.mark.parametrize("m,n,k", [(100001, 1000, 21), (900, 130003, 17), (190001, 300, 11), (70001, 500, 33), (50001, 500, 50)])
def test_tables_with_longer_rows(m, n, k):
    """Factors large enough for the copies whose rows do not straddle cache lines; the plain, the monitored and
    the stopped run, and a workspace without room for the copies (same sums, same bits)."""
    import torch

    import paper_2202_09518_amd as nmf
    r = np.random.default_rng(m + k)
    counts = r.integers(0, 9, m)
    rowptr = np.zeros(m + 1, dtype=np.int64)
    np.cumsum(counts, out=rowptr[1:])
    colidx = r.integers(0, n, int(rowptr[-1])).astype(np.int32)
    vals = r.random(colidx.size, dtype=np.float32)
    W, H = r.random((m, k), dtype=np.float32), r.random((k, n), dtype=np.float32)
    nnz = int(vals.size)
    rp, ci, va = torch.from_numpy(rowptr).cuda(), torch.from_numpy(colidx).cuda(), torch.from_numpy(vals).cuda()
    runs = []
    for how in ("plain", "monitored", "stopped", "small"):
        Wd, Hd = torch.from_numpy(W).cuda(), torch.from_numpy(H).cuda()
        if how == "monitored":
            nmf.nmf_mu_csr_monitor(rp, ci, va, m, n, nnz, k, Wd, Hd, 2, EPS)
        elif how == "stopped":
            nmf.nmf_mu_csr_tol(rp, ci, va, m, n, nnz, k, Wd, Hd, 2, EPS, 0.0, 1)
        elif how == "small":
            ws = torch.empty(nmf.nmf_mu_workspace_bytes(1, m, n, nnz, k, 0), dtype=torch.uint8, device="cuda")
            nmf.nmf_mu_set_workspace(ws)
            try:
                nmf.nmf_mu_csr(rp, ci, va, m, n, nnz, k, Wd, Hd, 2, EPS)
                torch.cuda.synchronize()
            finally:
                nmf.nmf_mu_set_workspace(None)
        else:
            nmf.nmf_mu_csr(rp, ci, va, m, n, nnz, k, Wd, Hd, 2, EPS)
        torch.cuda.synchronize()
        runs.append((Wd, Hd))
    for Wd, Hd in runs[1:]:
        assert torch.equal(Wd, runs[0][0]) and torch.equal(Hd, runs[0][1])
    Wr, Hr = orc.mu_csr(rowptr, colidx, vals, m, n, W, H, 2, float(np.float32(EPS)))
    assert orc.rel_fro(runs[0][0].cpu().numpy(), Wr) < 3e-6
    assert orc.rel_fro(runs[0][1].cpu().numpy(), Hr) < 3e-6
