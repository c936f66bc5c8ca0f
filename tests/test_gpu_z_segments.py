"""The z solver's launch rule around its lines: 8 segments of up to 5 or 9 rows
(n'z <= 40, 72), then 16 or 32, in both precisions, on mode counts that leave the
last workgroup ragged.  Bounds of the other A_p^{-1} parity tests: 1e-12 relative
in complex128, 5e-5 for the complex64 preconditioner."""
import numpy as np
import pytest
import torch

import oracle
from paper_1212_1397_amd.workloads import random_field

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,bound", [("fp64", 1e-12), ("mixed", 5e-5)])
@pytest.mark.parametrize("nz", [1, 7, 8, 9, 39, 40, 41, 71, 72, 73])
def test_pinv_around_the_segment_rule(nz, precision, bound):
    from paper_1212_1397_amd import helmholtz6 as h6
    for bc, n3 in (("DDNNDD", nz), ("DDNNSS", nz - 2)):
        if n3 < 1:
            continue
        prob = oracle.Problem((11, 5, n3), 1.0 / 12, 6.0 + 0.3j, tuple(bc))
        x = random_field(prob.shape, nz)
        plan = h6.Plan(prob.n, prob.h, prob.k, bc, precision=precision)
        z = plan.apply_Pinv(torch.from_numpy(x).cuda()).cpu().numpy()
        ref = oracle.apply_Pinv(prob, x)
        err = float(np.abs(z - ref).max() / np.abs(ref).max())
        print(f"n'z {nz} {bc} {precision}: {err:.2e}", flush=True)
        assert err <= bound
