"""The rule between the slab and the K-chunked kernels of the dense transforms
(xform_dense.hip) by the number of lines: long lines, whose slabs take more than one
round of outputs, on both sides of it (16 lines or columns a slab; 256 slabs along
complex128 x, two along complex64 x, 128 along y), against the FP64 oracle, with the
accumulating last pass (one SKS step).  Bounds as for the other A_p^{-1} parity tests:
1e-12 in FP64, 5e-5 for complex64."""
import numpy as np
import pytest

import oracle
from paper_1212_1397_amd.workloads import random_field

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SHAPES = [((300, 16, 255), "fp64"), ((300, 17, 241), "fp64"), ((514, 24, 170), "fp64"), ((516, 24, 171), "fp64"),
          ((300, 4, 4), "mixed"), ((300, 17, 1), "mixed"), ((516, 5, 5), "mixed"),
          ((15, 300, 127), "fp64"), ((15, 300, 128), "fp64"), ((33, 632, 43), "fp64"), ((49, 630, 31), "fp64"),
          ((15, 900, 127), "mixed"), ((15, 900, 128), "mixed"), ((17, 1262, 64), "mixed"), ((49, 1264, 31), "mixed")]


@pytest.mark.parametrize("n,prec", SHAPES)
@pytest.mark.parametrize("code", ["D", "N"])
def test_long_lines_few_and_many(monkeypatch, n, prec, code):
    from paper_1212_1397_amd import helmholtz6 as h6
    monkeypatch.setenv("H6_DENSE_TRANSFORMS", "1")
    bound = 1e-12 if prec == "fp64" else 5e-5
    off = 0 if code == "D" else 2
    bc = code * 4 + "DD"
    prob = oracle.Problem((n[0] - off, n[1] - off, n[2]), 1.0 / max(n), 3.0 + 0.2j, tuple(bc))
    x = random_field(prob.shape, seed=n[0])
    plan = h6.Plan(prob.n, prob.h, prob.k, bc, precision=prec)
    z = plan.apply_Pinv(torch.from_numpy(x).cuda())
    ref = oracle.apply_Pinv(prob, x)
    assert np.abs(z.cpu().numpy() - ref).max() <= bound * np.abs(ref).max()
    U0 = torch.from_numpy(random_field(prob.shape, seed=n[1])).cuda()
    F = torch.from_numpy(x).cuda() + plan.apply_A(U0)
    U, _ = plan.solve(F, U0.clone(), method="sks", tol=0.0, maxit=1, zero_guess=False)
    plan.close()
    assert float((U - U0 - z).abs().max() / z.abs().max()) <= 10 * bound



@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("n", [(32, 32, 3), (33, 33, 3), (31, 32, 1), (7, 20, 40), (24, 300, 1), (20, 24, 110),
                               (80, 32, 307), (48, 32, 512), (33, 64, 511), (33, 64, 512), (96, 40, 511), (96, 40, 512),
                               (300, 43, 96), (300, 44, 128), (416, 10, 472), (416, 10, 473)])
def test_short_lines_and_the_last_slabs(monkeypatch, n, prec):
    """Lines of up to 64 values and their neighbours, on both sides of the numbers of slabs
    that decide along y (complex64 1536 and 3072, complex128 12288), and complex128 x lines
    with 258 and 352 slabs.  Shifts near kappa = 64 keep the z solve from amplifying
    anything; root mean square against the oracle within 4 u sqrt(L), L the longest line: a
    random walk of L / 2 roundings in the two transforms of both axes is a quarter of it."""
    from paper_1212_1397_amd import helmholtz6 as h6
    monkeypatch.setenv("H6_DENSE_TRANSFORMS", "1")
    u = 2.0 ** (-53 if prec == "fp64" else -24)
    for code in "DN":
        off, bc = (0 if code == "D" else 2), code * 4 + "DD"
        h = 1.0 / max(n)
        prob = oracle.Problem((n[0] - off, n[1] - off, n[2]), h, (8.0 + 0.1j) / h, tuple(bc))
        x = random_field(prob.shape, seed=n[0])
        plan = h6.Plan(prob.n, prob.h, prob.k, bc, precision=prec)
        z = plan.apply_Pinv(torch.from_numpy(x).cuda()).cpu().numpy()
        plan.close()
        ref = oracle.apply_Pinv(prob, x)
        err = np.linalg.norm(z - ref) / np.linalg.norm(ref)
        print(f"{n} {code} {prec}: {err:.2e}", flush=True)
        assert err <= 4 * u * max(n[:2]) ** 0.5, code
