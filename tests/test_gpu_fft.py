"""The power-of-two transform path of A_p^{-1} (M = n + 1 = 64, 128, 256, 512,
xform_fft.hip) against the FP64 oracle: sine and cosine bases, x lines and y
columns, line and column counts off the workgroup's, FP64 and complex64
plans, the accumulating last pass (one SKS step), the choice through the
autotuner's cache (code 3, refused by plans without the tables) and the queued
batch, whose lanes take the plan's path.  Bounds as for the other A_p^{-1}
parity tests: 1e-12 in FP64, 5e-5 for complex64."""
import numpy as np
import pytest

import oracle
from paper_1212_1397_amd.workloads import random_field

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def relerr(a, b):
    return float(np.abs(a - b).max() / np.abs(b).max())


@pytest.mark.parametrize("prec,bound", [("fp64", 1e-12), ("mixed", 5e-5)])
@pytest.mark.parametrize("M", [64, 128, 256, 512])
@pytest.mark.parametrize("axis,other", [(0, 3), (0, 11), (1, 3), (1, 33)])
def test_fft_pinv_parity(M, axis, other, prec, bound):
    from paper_1212_1397_amd import helmholtz6 as h6
    for basis in "DN":
        n = [other, other, 3]
        n[axis] = M - 1
        bc = ["D"] * 4 + ["S", "D"]
        bc[2 * axis] = bc[2 * axis + 1] = basis
        prob = oracle.Problem(tuple(n), 1.0 / M, 3.0 + 0.2j, tuple(bc))
        x = random_field(prob.shape, seed=M + other)
        plan = h6.Plan(prob.n, prob.h, prob.k, "".join(bc), precision=prec)
        z = plan.apply_Pinv(torch.from_numpy(x).cuda())
        assert relerr(z.cpu().numpy(), oracle.apply_Pinv(prob, x)) <= bound, basis
        U0 = torch.from_numpy(random_field(prob.shape, seed=7)).cuda()
        F = torch.from_numpy(x).cuda() + plan.apply_A(U0)
        U, _ = plan.solve(F, U0.clone(), method="sks", tol=0.0, maxit=1, zero_guess=False)
        plan.close()
        assert float((U - U0 - z).abs().max() / z.abs().max()) <= 10 * bound, basis


def test_cache_code_selects_the_path(monkeypatch, tmp_path):
    from paper_1212_1397_amd import helmholtz6 as h6
    arch = torch.cuda.get_device_properties(0).gcnArchName
    prob = oracle.Problem((63, 63, 5), 1.0 / 64, 4.0 + 0.1j, tuple("DDDDDD"))
    x = torch.from_numpy(random_field(prob.shape, seed=4)).cuda()
    got = {}
    for env in (False, True):
        if env:
            monkeypatch.setenv("H6_DENSE_TRANSFORMS", "1")
        plan = h6.Plan(prob.n, prob.h, prob.k, "DDDDDD")
        for code in (0, 3):
            path = tmp_path / f"tune{env}{code}.txt"
            path.write_text(f"h6tune3 {arch} 63 63 5 0 tz=16 xfast={code} yfast={code} xlines=4 ylines=16\n")
            plan.autotune(str(path))
            got[env, code] = plan.apply_Pinv(x)
        plan.close()
    assert not torch.equal(got[False, 0], got[False, 3])
    assert torch.equal(got[True, 0], got[False, 0]) and torch.equal(got[True, 3], got[False, 0])


def test_queue_on_the_fft_path():
    from paper_1212_1397_amd import helmholtz6 as h6
    n, h = 63, 1.0 / 64
    plans = [h6.Plan(n, h, k * (1 + 0.01j), "DDNNSS", precision="mixed") for k in (8.0, 12.0, 15.0)]
    Fs = [p.rhs_gaussians([[0.4, 0.5, 0.6]], [1.0 + 0.5j], 4 * h) for p in plans]
    ref = [p.solve(F, method="fgmres", restart=30, tol=1e-10, maxit=300)[0] for p, F in zip(plans, Fs)]
    Us = [torch.full_like(F, float("nan")) for F in Fs]
    infos = h6.solve_batch_queue(plans, Fs, Us, restart=30, tol=1e-10, maxit=300, lanes=2)
    for i, U, R in zip(infos, Us, ref):
        assert i["status"] == "ok" and float(torch.linalg.norm(U - R) / torch.linalg.norm(R)) < 1e-8
