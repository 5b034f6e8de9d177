"""Up to 16 factors: every plan that a workspace too short for the resident plan leaves, named, against the oracle; the same
bits from a run cut in two."""
import ctypes

import numpy as np
import pytest

from oracle import nmf_oracle as orc

EPS = 1e-16
SMALL, MIRRORED, ROW, ONE_PASS, RESIDENT, COPIES = 0, 1, 2, 3, 4, 8


def data(m, n, k):
    r = np.random.default_rng(m + 3 * n + 7 * k)
    return r.random((m, n), dtype=np.float32), r.random((m, k), dtype=np.float32), r.random((k, n), dtype=np.float32)


def plan_of(nmf, A, m, n, k, W, H, eps):
    import torch

    fn = nmf.lib().nmfmu_dense_plan
    fn.argtypes = [ctypes.c_void_p, ctypes.c_int64, ctypes.c_int64, ctypes.c_int32, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int32,
                   ctypes.c_float, ctypes.POINTER(ctypes.c_int32), ctypes.c_void_p]
    plan = ctypes.c_int32(-1)
    assert fn(A.data_ptr(), m, n, k, W.data_ptr(), H.data_ptr(), 3, eps, ctypes.byref(plan), torch.cuda.current_stream().cuda_stream) == 0
    return plan.value


# plans: those that workspaces from kind 4 on leave before the resident plan fits (where it fits kind 4 there are none).
# One-pass: up to 32 workgroups (the finisher adds their shares up itself) and more; waves without columns.
# Row: m n <= 2^22.  Small: n % 4 or the base of A not what the others take, or that on padded copies
# (eps > 0).  Mirrored: room for A^T beyond that size.
CASES = [
    (1, 64, 1, 0, {ONE_PASS}), (999, 508, 5, 0, {ONE_PASS}), (1000, 68, 16, 0, {ONE_PASS}), (2000, 512, 4, 0, {ONE_PASS}),
    (4096, 512, 3, 0, {ONE_PASS}), (4096, 512, 12, 0, {ROW}), (300, 516, 8, 0, {ROW}), (640, 1200, 16, 0, {ROW}),
    (2000, 2048, 9, 0, {ROW}), (4096, 1024, 3, 0, {ROW}), (2600, 2000, 12, 0, {ROW, MIRRORED}), (5000, 768, 16, 0, {ROW}),
    (300, 203, 8, 0, {SMALL, ONE_PASS + COPIES}), (700, 259, 16, 0, {SMALL}), (500, 517, 8, 0, {SMALL, ROW + COPIES}),
    (100, 513, 5, 0, {SMALL}), (1000, 68, 4, 1, {ONE_PASS + COPIES}), (333, 4094, 9, 0, {SMALL}),
]


@pytest.mark.gpu
@pytest.mark.parametrize("m,n,k,offset,plans", CASES)
@pytest.mark.parametrize("eps", [EPS, 0.0])
def test_plans(m, n, k, offset, plans, eps):
    import torch

    import paper_2202_09518_amd as nmf
    A, W, H = data(m, n, k)
    Ad = torch.empty(m * n + 4, device="cuda")[offset:offset + m * n]
    Ad.copy_(torch.from_numpy(A).reshape(-1))
    least = nmf.nmf_mu_workspace_bytes(4, m, n, 0, k, 0)
    most = least + (48 << 10) * (-(-m // 16) * -(-n // 256))
    ws = torch.zeros(most, dtype=torch.uint8, device="cuda")
    want, seen, size = None, set(), least
    try:
        while size <= most:
            nmf.nmf_mu_set_workspace(ws, size)
            W0, H0 = torch.from_numpy(W).cuda(), torch.from_numpy(H).cuda()
            plan = plan_of(nmf, Ad, m, n, k, W0, H0, eps)
            if plan == RESIDENT:
                break
            size += 32 << 10
            if plan in seen:
                continue
            seen.add(plan)
            runs = []
            for iters in ((3,), (2, 1)):
                Wd, Hd = W0.clone(), H0.clone()
                for it in iters:
                    nmf.nmf_mu_dense(Ad, m, n, k, Wd, Hd, it, eps)
                runs.append((Wd, Hd))
            torch.cuda.synchronize()
            assert torch.equal(runs[0][0], runs[1][0]) and torch.equal(runs[0][1], runs[1][1]), plan
            if want is None:
                want = orc.mu_dense(A, W, H, 3, float(np.float32(eps)))
            # three updates of each factor, sums of one sign: a few roundings of 2^-24 per sum
            e = orc.rel_fro(runs[0][0].cpu().numpy(), want[0]), orc.rel_fro(runs[0][1].cpu().numpy(), want[1])
            assert max(e) < 3e-6, plan
    finally:
        torch.cuda.synchronize()
        nmf.nmf_mu_set_workspace(None)
    assert {p if eps or p < COPIES else SMALL for p in plans} <= seen, seen
