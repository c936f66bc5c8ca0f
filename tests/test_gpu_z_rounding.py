"""Rounding errors of the complex64 z solve on short lines against A_p^{-1} in 80-bit
arithmetic.  Near resonance they come from the inverse pivots, which each segment of a
line replays from stored ones; the longer the replay, the larger they are.  LIMIT holds
the errors of lines split into 16 segments (two rows each at 32 planes), root mean square
over the same ten right-hand sides; 1.1 is left for another order of the remaining sums
(one stored pivot per segment of eight gave 1.2 to 1.8)."""
import numpy as np
import pytest

import oracle
from paper_1212_1397_amd.workloads import random_field
from test_gpu_fft_rounding import exact_pinv

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

LIMIT = {((32, 32, 32), "D", 0.3 + 0.01j): 1.218e-6, ((32, 32, 32), "D", 0.6 + 0.02j): 9.32e-7,
         ((32, 32, 32), "N", 0.3 + 0.01j): 1.282e-6, ((32, 32, 32), "N", 0.6 + 0.02j): 9.12e-7,
         ((48, 48, 20), "D", 0.3 + 0.01j): 9.61e-7, ((48, 48, 20), "D", 0.6 + 0.02j): 7.91e-7,
         ((48, 48, 20), "N", 0.3 + 0.01j): 9.31e-7, ((48, 48, 20), "N", 0.6 + 0.02j): 8.40e-7}


@pytest.mark.parametrize("n,code,kh", list(LIMIT))
def test_short_lines_no_less_exact_than_16_segments(n, code, kh):
    from paper_1212_1397_amd import helmholtz6 as h6
    h, bc = 1.0 / (max(n) + 1), code * 4 + "DD"
    prob = oracle.Problem(n, h, kh / h, tuple(bc))
    plan = h6.Plan(n, h, prob.k, bc, precision="mixed")
    total = 0.0
    for s in range(10):
        x = random_field(prob.shape, seed=1000 * s + n[2])
        ref = exact_pinv(prob, x)
        z = plan.apply_Pinv(torch.from_numpy(x).cuda()).cpu().numpy()
        total += float((np.abs(z - ref) ** 2).sum() / (np.abs(ref) ** 2).sum())
    plan.close()
    err = (total / 10) ** 0.5
    print(f"{n} {code} {kh}: {err:.3e} (limit {LIMIT[n, code, kh]:.3e})", flush=True)
    assert err <= 1.1 * LIMIT[n, code, kh]


@pytest.mark.parametrize("nz", [73, 79, 80, 81, 144, 145, 272, 273])
def test_rows_per_thread_of_16_segments(nz):
    """complex64 lines beyond 72 planes: five, nine or seventeen rows a thread, 32 segments
    from 273 on; the bound of the other complex64 parity tests."""
    from paper_1212_1397_amd import helmholtz6 as h6
    for bc, n3 in (("DDNNDD", nz), ("DDNNSS", nz - 2)):
        prob = oracle.Problem((11, 5, n3), 1.0 / 12, 6.0 + 0.3j, tuple(bc))
        x = random_field(prob.shape, nz)
        plan = h6.Plan(prob.n, prob.h, prob.k, bc, precision="mixed")
        z = plan.apply_Pinv(torch.from_numpy(x).cuda()).cpu().numpy()
        plan.close()
        ref = oracle.apply_Pinv(prob, x)
        assert np.abs(z - ref).max() <= 5e-5 * np.abs(ref).max()
