"""The slab kernels of the dense transforms (xform_dense.hip) at the edges of
their tiles and of the rule that picks them, against the FP64 oracle: line
lengths with every remainder class of H = ceil(L / 2) (whole 16-row tiles, one
and two border rows, a padded tile, K remainders), partial slabs (line and
column counts off the multiples of 16), odd row pitches, lines at the limits
of the slab rule (two units per wave along x, the LDS sizes along x and y),
and the accumulating last pass (one SKS step).  Bounds as for the other
A_p^{-1} parity tests: 1e-12 in FP64, 5e-5 for complex64."""
import numpy as np
import pytest

import oracle
from paper_1212_1397_amd.workloads import random_field

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# (n'x, n'y) of the unknown grid; the faces are chosen per case
SHAPES = [(32, 17), (33, 15), (34, 50), (35, 31), (36, 33), (38, 66), (48, 98), (63, 64), (65, 129), (99, 16),
          (160, 37), (161, 20), (255, 18), (516, 3), (518, 3), (3, 516), (17, 632), (16, 636), (5, 1264), (4, 1268)]


@pytest.mark.parametrize("prec,bound", [("fp64", 1e-12), ("mixed", 5e-5)])
@pytest.mark.parametrize("lx,ly", SHAPES)
def test_slab_pinv_parity(monkeypatch, lx, ly, prec, bound):
    from paper_1212_1397_amd import helmholtz6 as h6
    monkeypatch.setenv("H6_DENSE_TRANSFORMS", "1")
    for bc in ("DDDDSS", "NNNNDD"):
        off = 0 if bc[0] == "D" else 2
        if min(lx, ly) - off < 1:
            continue
        prob = oracle.Problem((lx - off, ly - off, 3), 1.0 / max(lx, ly), 3.0 + 0.2j, tuple(bc))
        x = random_field(prob.shape, seed=lx)
        plan = h6.Plan(prob.n, prob.h, prob.k, bc, precision=prec)
        z = plan.apply_Pinv(torch.from_numpy(x).cuda())
        ref = oracle.apply_Pinv(prob, x)
        e = float(np.abs(z.cpu().numpy() - ref).max() / np.abs(ref).max())
        assert e <= bound, (bc, e)
        # U_1 = U_0 + A_p^{-1} (F - A U_0) with F = x + A U_0: the accumulating pass adds the same z
        U0 = torch.from_numpy(random_field(prob.shape, seed=ly)).cuda()
        F = torch.from_numpy(x).cuda() + plan.apply_A(U0)
        U, _ = plan.solve(F, U0.clone(), method="sks", tol=0.0, maxit=1, zero_guess=False)
        e = float((U - U0 - z).abs().max() / z.abs().max())
        plan.close()
        assert e <= 10 * bound, (bc, e)
