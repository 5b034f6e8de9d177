"""A caller's workspace of the documented size gets the plan that the library's own would: the same bits."""
import numpy as np
import pytest

EPS = 1e-16


def same_bits(call, size, shapes):
    import torch

    import paper_2202_09518_amd as nmf
    g = torch.Generator(device="cuda")
    g.manual_seed(size & 0xffff)
    first = [torch.rand(s, generator=g, device="cuda") for s in shapes]
    own = [x.clone() for x in first]
    call(*own)
    torch.cuda.synchronize()
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    given = [x.clone() for x in first]
    nmf.nmf_mu_set_workspace(ws)
    try:
        call(*given)
        torch.cuda.synchronize()
    finally:
        nmf.nmf_mu_set_workspace(None)
    return all(torch.equal(a, b) for a, b in zip(own, given))


# one-pass plan; the same, the row plan and the mirrored plan on copies of A (odd n; odd n and m; odd m only)
@pytest.mark.gpu
@pytest.mark.parametrize("m,n,k,plan", [(9000, 300, 12, "one"), (9000, 299, 12, "one"), (12289, 513, 12, "row"),
                                        (1501, 2001, 40, "mirrored"), (5001, 3000, 12, "mirrored")])
def test_dense(m, n, k, plan):
    import torch

    import paper_2202_09518_amd as nmf
    n4, m4 = -(-n // 4) * 4, -(-m // 4) * 4
    if plan == "mirrored":
        size = nmf.nmf_mu_workspace_bytes(0, m4, n4, 0, k, 0)
    else:
        size = nmf.nmf_mu_workspace_bytes(4, m, n4, 0, k, 0) + (1024 * k * n4 if plan == "one" else 0)
    if n != n4 or m != m4:
        size += 4 * (m * n4 + k * n4 + m4 * k) + 768
    A = torch.rand((m, n), device="cuda")
    nmf.nmf_mu_release()
    assert same_bits(lambda W, H: nmf.nmf_mu_dense(A, m, n, k, W, H, 2, EPS), size, [(m, k), (k, n)])


@pytest.mark.gpu
def test_sparse():
    import torch

    import paper_2202_09518_amd as nmf
    m, n, k, per = 200000, 3000, 12, 3
    r = np.random.default_rng(5)
    rowptr = torch.arange(0, m * per + 1, per, dtype=torch.int64, device="cuda")
    col = torch.from_numpy(r.integers(0, n, m * per).astype(np.int32)).cuda()
    vals = torch.from_numpy(r.random(m * per, dtype=np.float32)).cuda()
    size = nmf.nmf_mu_workspace_bytes(1, m, n, m * per, k, 0) + 4 * 16 * (m + n) + 512
    nmf.nmf_mu_release()
    assert same_bits(lambda W, H: nmf.nmf_mu_csr(rowptr, col, vals, m, n, m * per, k, W, H, 2, EPS), size, [(m, k), (k, n)])


# Cut copies (8 bytes an entry) are planned up to the length that their launches take, which is rounded up to 64: 2^25 - 64.
@pytest.mark.parametrize("kind,k", [(0, 40), (3, 64), (5, 96)])
@pytest.mark.parametrize("turned", [False, True])
def test_cut_copies_end_where_their_launches_do(kind, k, turned):
    import paper_2202_09518_amd as nmf

    def size(m, n):
        return nmf.nmf_mu_workspace_bytes(kind, *((n, m) if turned else (m, n)), 0, k, 0) / (m * n)
    last = (1 << 25) - 64
    assert size(last, 8192) >= 8
    for m in (last + 1, last + 32, (1 << 25) - 1, 1 << 25):
        assert size(m, 8192) < 6
