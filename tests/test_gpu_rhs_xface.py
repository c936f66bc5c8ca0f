"""Neumann x faces of the right-hand sides (rhs.hip) where the end nodes meet the edges
of the 16-node x tiles: both ends in one tile, an end node alone in its tile, ends in a
full tile's first and last column, and grids whose tiles are shared out over several
workgroups.  FP64 oracle, 1e-12 of max |F| as in the other right-hand-side tests."""
import numpy as np
import pytest

import oracle
from oracle.functions import Separable, Sin, Term, gaussian_sources

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("count", [1, 4, 5, 12])
@pytest.mark.parametrize("bc", ["NNNNNN", "NNDDSS", "NNNNDS"])
@pytest.mark.parametrize("lx", [3, 15, 16, 17, 31, 32, 33, 49, 160])
def test_end_nodes_and_tiles(lx, bc, count):
    from manufactured import factor_tables
    from paper_1212_1397_amd import helmholtz6 as h6
    n = (lx - 2, 6, 7)
    h = 1.0 / (max(n) + 1)
    prob = oracle.Problem(n, h, 7.0 + 0.2j, tuple(bc))
    rng = np.random.default_rng(lx + count)
    centres = rng.uniform(0.0, 1.0, size=(count, 3)) * np.array([prob.length(a) for a in range(3)])
    amps = rng.standard_normal(count) + 1j * rng.standard_normal(count)
    plan = h6.Plan(prob.n, prob.h, prob.k, bc)
    nan = torch.full(plan.shape, float("nan"), dtype=torch.complex128, device="cuda")
    F = plan.rhs_gaussians(centres, amps, 4.0 * h, out=nan.clone()).cpu().numpy()
    ref = oracle.rhs(prob, gaussian_sources(centres, amps, 4.0 * h))
    assert np.abs(F - ref).max() <= 1e-12 * np.abs(ref).max()
    f = Separable([Term(complex(rng.standard_normal(), rng.standard_normal()),
                        *(Sin(float(w)) for w in rng.uniform(1.0, 6.0, 3))) for _ in range(count)])
    S = plan.rhs_separable(*factor_tables(f, prob.points()), out=nan.clone()).cpu().numpy()
    plan.close()
    ref = oracle.rhs(prob, f)
    assert np.abs(S - ref).max() <= 1e-12 * np.abs(ref).max()
