"""Every launch shape of the operator kernel (tile width 64 or 32, chunks of 2
to 32 planes) gives the FP64 oracle's A x, and all depths the same bits: the
untuned choice for grids on both sides of the width and depth rules, and each
depth forced through the autotuner's cache; one SKS step covers the residual
form and its norm partials."""
import numpy as np
import pytest

import oracle
from paper_1212_1397_amd.workloads import random_field

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# n'x: 64 and 32 wide tiles with and without a partial tile; depths 2, 4, 8 and 16 by the rule
SHAPES = [((1, 1, 1), "DDDDDD"), ((31, 15, 1), "NNNNSS"), ((64, 8, 5), "DDNNSS"), ((65, 17, 33), "NNDDSN"),
          ((96, 95, 96), "DDNNSS"), ((160, 160, 60), "DDDDND"), ((200, 161, 97), "DDNNSS"), ((255, 128, 128), "DDDDSS")]


@pytest.mark.parametrize("n,bc", SHAPES)
def test_stencil_shapes(tmp_path, n, bc):
    from paper_1212_1397_amd import helmholtz6 as h6
    arch = torch.cuda.get_device_properties(0).gcnArchName
    prob = oracle.Problem(n, 1.0 / (max(n) + 1), 5.0 + 0.3j, tuple(bc))
    x = random_field(prob.shape, seed=n[0])
    ref = oracle.apply_A(prob, x)
    xg = torch.from_numpy(x).cuda()
    plan = h6.Plan(prob.n, prob.h, prob.k, bc)
    y0 = plan.apply_A(xg)
    assert np.abs(y0.cpu().numpy() - ref).max() <= 1e-12 * np.abs(ref).max()
    F = torch.from_numpy(random_field(prob.shape, seed=3)).cuda()
    rn = float(np.linalg.norm(F.cpu().numpy() - ref) / torch.linalg.norm(F))

    def resid():            # tol above the first residual: the solve only measures F - A x
        _, info = plan.solve(F, xg.clone(), method="sks", tol=2.0 * rn, maxit=1, zero_guess=False)
        assert info["iters"] == 0
        return info["rel_resid"]

    assert abs(resid() - rn) <= 1e-12 * rn
    nx, ny, nz = plan.dims
    for tz in (2, 4, 8, 16, 32):
        path = tmp_path / f"tune{tz}.txt"
        path.write_text(f"h6tune3 {arch} {nx} {ny} {nz} 0 tz={tz} xfast=0 yfast=0 xlines=4 ylines=16\n")
        plan.autotune(str(path))
        assert torch.equal(plan.apply_A(xg), y0), tz
        assert abs(resid() - rn) <= 1e-12 * rn, tz
    plan.close()
