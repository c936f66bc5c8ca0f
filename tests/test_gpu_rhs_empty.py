"""No source: F = 0 exactly, whatever width the call names (the smallest ones have no
finite 1 / sigma or no finite fourth power of it)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("sigma", [5e-324, 1e-300, 1e-80, 0.1, 1e300, float("inf")])
@pytest.mark.parametrize("bc", ["DDDDDD", "NNNNSS"])
def test_no_source_is_zero(bc, sigma):
    from paper_1212_1397_amd import helmholtz6 as h6
    plan = h6.Plan((17, 5, 3), 1.0 / 18, 4.0 + 0.2j, bc)
    out = torch.full(plan.shape, float("nan"), dtype=torch.complex128, device="cuda")
    F = plan.rhs_gaussians(np.empty((0, 3)), np.empty(0), sigma, out=out)
    plan.close()
    assert not F.any()
