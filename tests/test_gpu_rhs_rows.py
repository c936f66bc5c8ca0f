"""The row kernels of the right-hand sides (rhs.hip) where their tiles and
source groups end, against the FP64 oracle: source counts around the groups of
four and eight (further groups are added by a second pass over the rows), no
source at all, grids with a partial row tile, a partial x tile and a single
node, and Neumann x faces (their own kernel).  FP64, the same terms in another
order: 1e-12 of max |F| as in the other right-hand-side tests."""
import numpy as np
import pytest

import oracle
from oracle.functions import Separable, Sin, Term, gaussian_sources

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

GRIDS = [((17, 5, 7), "DDNNSS"), ((16, 8, 3), "NNNNNN"), ((33, 3, 5), "NNDDSN"), ((1, 2, 1), "NNNNSS"),
         ((30, 9, 11), "DDDDND")]


@pytest.mark.parametrize("nsrc", [0, 1, 4, 5, 8, 9, 17, 64])
@pytest.mark.parametrize("n,bc", GRIDS)
def test_gaussian_source_groups(n, bc, nsrc):
    from paper_1212_1397_amd import helmholtz6 as h6
    h = 1.0 / (max(n) + 1)
    prob = oracle.Problem(n, h, 9.0 + 0.3j, tuple(bc))
    rng = np.random.default_rng(nsrc)
    centres = rng.uniform(0.0, 1.0, size=(nsrc, 3)) * np.array([prob.length(a) for a in range(3)])
    amps = rng.standard_normal(nsrc) + 1j * rng.standard_normal(nsrc)
    plan = h6.Plan(prob.n, prob.h, prob.k, bc)
    F = plan.rhs_gaussians(centres, amps, 4.0 * h, out=torch.full(plan.shape, float("nan"), dtype=torch.complex128,
                                                                  device="cuda")).cpu().numpy()
    plan.close()
    if nsrc == 0:
        assert not F.any()
        return
    ref = oracle.rhs(prob, gaussian_sources(centres, amps, 4.0 * h))
    assert np.abs(F - ref).max() <= 1e-12 * np.abs(ref).max()


@pytest.mark.parametrize("nterms", [1, 4, 5, 8, 9, 13])
@pytest.mark.parametrize("n,bc", GRIDS)
def test_separable_term_groups(n, bc, nterms):
    from manufactured import factor_tables
    from paper_1212_1397_amd import helmholtz6 as h6
    prob = oracle.Problem(n, 1.0 / (max(n) + 1), 5.0 + 0.2j, tuple(bc))
    rng = np.random.default_rng(nterms)
    f = Separable([Term(complex(rng.standard_normal(), rng.standard_normal()),
                        *(Sin(float(w)) for w in rng.uniform(1.0, 6.0, 3))) for _ in range(nterms)])
    ref = oracle.rhs(prob, f)
    plan = h6.Plan(prob.n, prob.h, prob.k, bc)
    F = plan.rhs_separable(*factor_tables(f, prob.points()),
                           out=torch.full(plan.shape, float("nan"), dtype=torch.complex128, device="cuda")).cpu().numpy()
    plan.close()
    assert np.abs(F - ref).max() <= 1e-12 * np.abs(ref).max()
