"""The Arnoldi step's coefficient kernels across their dispatch line (16 vectors):
whole GMRES cycles shorter than, at and beyond it against the oracle.  The
device sums differ from the oracle's by their order only, 1e-13 relative over a
few thousand terms; a cycle of up to 20 steps to 1e-11 leaves 1e-9 of room."""
import numpy as np
import pytest
import torch

import oracle
from paper_1212_1397_amd.workloads import random_field

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("restart", [1, 2, 15, 16, 17, 20])
def test_gmres_cycles_around_the_small_kernel(restart):
    from paper_1212_1397_amd import helmholtz6 as h6
    prob = oracle.Problem((14, 11, 9), 1.0 / 15, 9.0 + 0.3j, tuple("DDNNSS"))
    F = random_field(prob.shape, 11)
    plan = h6.Plan(prob.n, prob.h, prob.k, "DDNNSS")
    U, info = plan.solve(torch.from_numpy(F).cuda(), method="gmres", restart=restart, tol=1e-11, maxit=400)
    ref, oinfo = oracle.solve(prob, F, "gmres", restart=restart, tol=1e-11, maxit=400)
    err = np.abs(U.cpu().numpy() - ref).max() / np.abs(ref).max()
    print(f"restart {restart}: {info['iters']} steps (oracle {oinfo.iters}), {err:.2e}", flush=True)
    assert info["status"] == "ok" and abs(info["iters"] - oinfo.iters) <= 1 and err <= 1e-9
