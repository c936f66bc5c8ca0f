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
